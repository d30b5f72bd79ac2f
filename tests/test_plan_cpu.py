"""Host-side plans of the large passes (csrc/pp_plan.h) and the offsets of their
loads (csrc/pp_core.h), built host-only into a small library: no GPU and no
device code."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
IT, OT, DT = 0, 1, 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "plan.so")
    cmd = [CLANG, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC",
           "-I", os.path.join(ROOT, "paper_2312_06881_amd", "csrc"), os.path.join(ROOT, "tests", "host", "plan.cpp"),
           "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    so = ctypes.CDLL(lib)
    i64, ci = ctypes.c_int64, ctypes.c_int
    so.pp_pays.argtypes = [ci, i64, i64, i64, i64, ci, ci, ci]
    so.pp_outside.argtypes = [ci, ci, i64, i64, ci, ctypes.POINTER(ci)]
    return so


def weight_bytes(n_in, n_out, D):
    return 2 * n_in * n_out // D


@pytest.mark.parametrize("variant", (IT, OT, DT))
@pytest.mark.parametrize("dx", (0, 1))
def test_large_tiles_refuse_offsets_past_32_bits(plan, variant, dx):
    """Weight tensors of 2^31 bytes and more (at 2^32 the buffer range itself wraps to zero), and
    rows whose 256-token panel of fp32 sums passes 2^31 bytes, stay with the kernels that count in
    64 bits; just below either bound the pass is taken."""
    for n_in, n_out, D in ((65536, 65536, 4), (65536, 131072, 8), (65536, 65536, 2), (131072, 131072, 8),
                           (65536, 131072, 4), (131072, 262144, 8)):
        assert weight_bytes(n_in, n_out, D) >= 1 << 31
        assert not plan.pp_pays(variant, n_in, n_out, D, 4096, dx, 0, 0), (n_in, n_out, D)
    # 2^21 columns: a 256-token fp32 panel is 2^31 bytes, the weights 2^30
    wide, narrow = 1 << 21, 2048
    n_in, n_out = (wide, narrow) if dx else (narrow, wide)
    assert weight_bytes(n_in, n_out, 8) < 1 << 31
    assert not plan.pp_pays(variant, n_in, n_out, 8, 4096, dx, 0, 0)
    # below both bounds: the pass without an output transpose is taken at n_dyad 8
    plain = OT if dx else IT
    assert plan.pp_pays(plain, 32768, 65536, 8, 4096, dx, 0, 0)


@pytest.mark.parametrize("n", (64, 128, 192, 256))
@pytest.mark.parametrize("tr", (0, 1))
@pytest.mark.parametrize("bk", (32, 64, 96, 160, 288, 512))
def test_unit_loads_stay_inside_the_block(plan, n, tr, bk):
    """A reduction block of an odd number of 32-index steps ends in a unit of one new step: started
    at that step, its second half would read past the block (for the last block, past the tensor)."""
    wrong = ctypes.c_int()
    units = (bk // 32 + 1) // 2
    for k in range(units):
        assert plan.pp_outside(n, tr, bk, k, 0, ctypes.byref(wrong)) == 0
        assert wrong.value == 0                 # every step is multiplied once, from its own bytes
    past = plan.pp_outside(n, tr, bk, units - 1, 1, ctypes.byref(wrong))
    assert (past > 0) == (bk % 64 == 32)
