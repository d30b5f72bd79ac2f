"""GPU parity of the fp32 matrix-core kernels: edges of their 128 / 64 tiles and
32-index stages (ragged tokens, blocks of 4 to 260, classes of a few columns
under an output transpose), against the CPU oracle with the fp32 bounds of the
other parity tests."""
import pytest
import torch

import oracle
import paper_2312_06881_amd as dy
from workloads import layer_inputs
from tests.parity_util import assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [  # (n_in, n_out, n_dyad, tokens)
    (4, 8, 1, 1),           # one block of 4
    (24, 36, 3, 5),         # blocks of 8 and 12
    (64, 256, 4, 128),
    (272, 528, 4, 130),     # blocks of 68 and 132: ragged stages and tiles, columns D apart
    (1040, 520, 2, 257),    # blocks of 520 and 260
    (512, 256, 16, 700),    # blocks of 32 and 16: one column per class; split tokens
    (384, 192, 6, 1030),    # two token splits
]


@pytest.mark.parametrize("variant", ("IT", "OT", "DT"))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_f32(shape, variant):
    n_in, n_out, D, M = shape
    print("CASE", variant, *shape, flush=True)
    L = layer_inputs(n_in, n_out, D, M, dtype="f32")
    x, w1, w2, b, dz, h_in = (t.to(DEV) for t in (L.X, L.W1, L.W2, L.bias, L.dZ, L.H_in))
    f = {k: L.f64(k) for k in ("X", "W1", "W2", "bias", "dZ", "H_in")}
    y, h = dy.forward(x, w1, w2, b, variant, act="gelu", stash_h=True)
    ry, rh = oracle.forward(variant, n_in, n_out, D, f["X"], f["W1"], f["W2"], f["bias"], act=oracle.ACT_GELU, want_h=True)
    assert_close(y, ry, "f32", "gelu")
    assert_close(h, rh, "f32", "pre-activation")
    rx = oracle.backward_dx(variant, n_in, n_out, D, f["dZ"], f["W1"], f["W2"])
    assert_close(dy.backward_dx(dz, w1, w2, variant), rx, "f32", "dx")
    rg = oracle.backward_dx(variant, n_in, n_out, D, f["dZ"], f["W1"], f["W2"], act_in=oracle.ACT_GELU, H_in=f["H_in"])
    assert_close(dy.backward_dx(dz, w1, w2, variant, act_in="gelu", h_in=h_in), rg, "f32", "dx gelu'")
    got = dy.backward_dw(dz, x, D, variant)
    for g, r, what in zip(got, oracle.backward_dw(variant, n_in, n_out, D, f["dZ"], f["X"]), ("dW1", "dW2", "db")):
        assert_close(g, r, "f32", what)
