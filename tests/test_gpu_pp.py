"""GPU parity of the plain-block forms on the large ping-pong tiles.

Above 1024 tokens, n_dyad 2, 4, 8 and 16: both components in one loop over a
de-interleaved input copy (no output transpose), over residue-major columns
that a copy then interleaves (output transpose, whole tiles per block and
residue), or component 2 through an fp32 slice.  Shapes are the smallest that
take each form, with ragged token counts, reduction blocks that end in half a
unit (32 of 64 indices), every tile width and several token chunks.

Reference: the dense weight in float64 on the GPU (torch), elementwise bound
of the other parity tests.
"""
import pytest
import torch

import paper_2312_06881_amd as dy
from tests.parity_util import assert_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dense(w1, w2, variant):
    D, bo, bi = w1.shape
    i = torch.arange(D, device=DEV).view(D, 1, 1)
    j = torch.arange(bo, device=DEV).view(1, bo, 1)
    k = torch.arange(bi, device=DEV).view(1, 1, bi)
    r2 = j * D + i if variant in ("OT", "DT") else i * bo + j
    c2 = k * D + i if variant in ("IT", "DT") else i * bi + k
    W = torch.zeros(D * bo * D * bi, dtype=torch.float64, device=DEV)
    W[((i * bo + j) * (D * bi) + i * bi + k).flatten()] += w1.double().flatten()
    W[(r2 * (D * bi) + c2).flatten()] += w2.double().flatten()
    return W.view(D * bo, D * bi)


def gelu(h):
    return 0.5 * h * torch.erfc(-h / 2 ** 0.5)


def gelu_grad(h):
    return 0.5 * torch.erfc(-h / 2 ** 0.5) + h * torch.exp(-0.5 * h * h) / (2 * torch.pi) ** 0.5


def normal(seed, *shape, std=1.0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=DEV) * std).bfloat16()


CASES = [  # (n_in, n_out, n_dyad, tokens)
    (2048, 1024, 8, 1025),    # pair: 256 x 128 tiles; slice off, fused tiles beside it
    (2304, 1536, 8, 1100),    # blocks of 288 (half a unit at the end) and 192
    (1024, 1536, 16, 1290),   # blocks of 64 and 96
    (4096, 2048, 8, 1300),    # slice (blocks of 512 and 256) and pair
    (2048, 8192, 8, 1040),    # residue-major, 128 columns a pair
    (2048, 3072, 4, 4097),    # n_dyad 4 pair (blocks of 512 and 768), residue-major 192
    (2048, 4096, 2, 3100),    # n_dyad 2
    (4096, 2048, 4, 6200),    # n_dyad 4 slice (blocks of 1024 and 512)
    (4096, 32768, 16, 1600),  # residue-major at n_dyad 16, more than one token chunk
]


@pytest.mark.parametrize("variant", ("IT", "OT", "DT"))
@pytest.mark.parametrize("shape", CASES, ids=lambda c: "x".join(map(str, c)))
def test_forward_and_dx(shape, variant):
    n_in, n_out, D, M = shape
    print("CASE", variant, *shape, flush=True)
    x, dz = normal(1, M, n_in), normal(2, M, n_out)
    w1, w2 = (normal(s, D, n_out // D, n_in // D, std=0.02) for s in (3, 4))
    b, h_in = normal(5, n_out, std=0.02), normal(6, M, n_in)
    W = dense(w1, w2, variant)
    rows = torch.cat([torch.arange(0, M, 37, device=DEV), torch.arange(M - 70, M, device=DEV)])

    def check(got, ref, what):
        assert got.shape[0] == M
        assert_close(got[rows].float().cpu().numpy(), ref.cpu().numpy(), "bf16", what)

    rh = x[rows].double() @ W.t() + b.double()
    check(dy.forward(x, w1, w2, b, variant), rh, "forward")
    y, h = dy.forward(x, w1, w2, b, variant, act="gelu", stash_h=True)
    check(h, rh, "pre-activation")
    check(y, gelu(rh), "gelu")
    rx = dz[rows].double() @ W
    check(dy.backward_dx(dz, w1, w2, variant), rx, "dx")
    check(dy.backward_dx(dz, w1, w2, variant, act_in="gelu", h_in=h_in), rx * gelu_grad(h_in[rows].double()), "dx gelu'")
