"""Host-side plans of the grouped passes (csrc/pp_plan.h, csrc/tile_plan.h) and the
offsets of the large tiles' loads (csrc/pp_core.h), built host-only into a small
library: no GPU and no device code.  The shapes of the GPU tests are checked here
to take the form, the number of token chunks and the tile they are there for."""
import ctypes
import os
import subprocess

import pytest

from tests.test_gpu_permuted import PLAIN_CHUNK, STASH_CHUNK, WIDE
from tests.test_gpu_pp import FORMS, PADDED_FORMS
from tests.test_gpu_tiles import TILES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
IT, OT, DT = 0, 1, 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "plan.so")
    cmd = [CLANG, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2312_06881_amd", "csrc"), os.path.join(ROOT, "tests", "host", "plan.cpp"),
           "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    so = ctypes.CDLL(lib)
    i64, ci = ctypes.c_int64, ctypes.c_int
    so.pp_pays.argtypes = [ci, i64, i64, i64, i64, ci, ci, ci]
    so.pp_plan.argtypes = [ci, i64, i64, i64, i64, ci, ci, ci, ctypes.POINTER(i64)]
    so.padded_fused.argtypes = [ci, i64, i64, i64, i64, ci]
    so.tile_choice.restype = None
    so.tile_choice.argtypes = [ci, i64, i64, i64, i64, ci, ctypes.POINTER(i64 * 5)]
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


NAMES = {0: "none", 1: "pair", 2: "slice", 6: "res"}


@pytest.mark.parametrize("case", FORMS, ids=lambda c: "-".join(map(str, c)))
def test_gpu_cases_take_their_form(plan, case):
    n_in, n_out, D, M, variant, which, form, chunks = case
    dx, act, stash = which in ("dx", "dx_gelu"), which != "forward" and which != "dx", which == "gelu_h"
    chunk = ctypes.c_int64()
    got = plan.pp_plan(("IT", "OT", "DT").index(variant), n_in, n_out, D, M, dx, act, stash, ctypes.byref(chunk))
    assert NAMES[got] == form
    assert -(-M // chunk.value) == chunks


def test_wide_chunks(plan):
    """The chunks whose boundaries the wide layer's GPU test samples."""
    chunk = ctypes.c_int64()
    for v, m in PLAIN_CHUNK.items():
        assert plan.pp_plan(("IT", "OT", "DT").index(v), *WIDE, 0, 0, 0, ctypes.byref(chunk)) and chunk.value == m
    n_in, n_out, _, M = WIDE
    for v, m in STASH_CHUNK.items():
        assert not plan.pp_plan(("IT", "OT", "DT").index(v), *WIDE, 0, 1, 1, ctypes.byref(chunk))
        per_token = n_out * 4 + (n_in * 2 if v == "DT" else 0)     # the slice, the de-interleaved input
        assert (2 << 30) // per_token // 256 * 256 == m < M


@pytest.mark.parametrize("case", PADDED_FORMS, ids=lambda c: "-".join(map(str, c)))
def test_gpu_padded_cases_take_their_tiles(plan, case):
    n_in, n_out, D, M, variant, dx, fused = case
    assert bool(plan.padded_fused(("IT", "OT", "DT").index(variant), n_in, n_out, D, M, dx)) == fused


@pytest.mark.parametrize("case", TILES, ids=lambda c: "-".join(map(str, c)))
def test_gpu_cases_take_their_tile(plan, case):
    n_in, n_out, D, M, variant, dx, tile = case
    out = (ctypes.c_int64 * 5)()
    plan.tile_choice(("IT", "OT", "DT").index(variant), n_in, n_out, D, M, dx, ctypes.byref(out))
    assert tuple(out[:3]) == tile


def test_tile_plans_over_the_range(plan):
    """Every choice divides its block and its reduction, and its fp32 slices stay within the
    larger of 64 MiB and half the weights' bytes (written and read once: the weights' bytes)."""
    out = (ctypes.c_int64 * 5)()
    seen = set()
    for d, f in ((768, 3072), (1024, 4096), (640, 2560), (2048, 8192), (8192, 32768)):
        for n_in, n_out in ((d, d), (d, f), (f, d)):
            for D in (2, 3, 4, 6, 8, 16):
                for dx in (0, 1):
                    kin, nout = (n_out, n_in) if dx else (n_in, n_out)
                    if kin % (32 * D) or nout % (64 * D):
                        continue
                    for M in (1, 33, 64, 200, 1000, 4097):
                        for v in (IT, OT, DT):
                            plan.tile_choice(v, n_in, n_out, D, M, dx, ctypes.byref(out))
                            bm, bn, sp = out[:3]
                            if bm == 0:       # no 4-wave tile under this output transpose
                                continue
                            seen.add((bm, bn))
                            assert nout // D % bn == 0 and kin // D // 32 % sp == 0
                            weights = 4 * n_in * n_out // D
                            assert sp == 1 or sp * M * nout * 4 <= max(64 << 20, weights // 2)
                            # and it is one of the two plans
                            assert (-(-M // bm)) * (nout // bn) * sp in (out[3], out[4])
    assert len(seen) >= 6
