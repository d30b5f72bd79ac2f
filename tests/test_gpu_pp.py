"""GPU parity of the plain-block forms on the large ping-pong tiles.

Above 1024 tokens, n_dyad 2, 4, 8 and 16: both components in one loop over a
de-interleaved input copy (no output transpose), over residue-major columns
that a copy then interleaves (output transpose, whole tiles per block and
residue), or component 2 through an fp32 slice.  CASES runs every pass of shapes
around the rules' lines, some of which stay with the other tiles; FORMS names the
passes that take each form, with ragged token counts, reduction blocks that end in
half a unit (32 of 64 indices) and more than one token chunk, and test_plan_cpu.py
checks on the CPU that they do.  PADDED_FORMS: zero-padded blocks on the large
tiles and on the fused-stage ones, rows of a width that 8 does not divide and more
residues than the slice's staging holds among them.

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
    (2048, 1024, 8, 1025),    # blocks too narrow for the form
    (2304, 1536, 8, 1100),    # blocks of 288 and 192: too few tokens for them
    (1024, 1536, 16, 1290),   # blocks of 64 and 96: the Dyad-OT input gradient alone
    (4096, 2048, 8, 1300),    # slice (blocks of 512 and 256) and pair
    (2048, 8192, 8, 1040),    # residue-major, 128 columns a pair
    (2048, 3072, 4, 4097),    # n_dyad 4 pair (blocks of 512 and 768), residue-major 192
    (2048, 4096, 2, 3100),    # n_dyad 2
    (4096, 2048, 4, 6200),    # n_dyad 4 residue-major and pair (blocks of 1024 and 512)
    (4096, 32768, 16, 1600),  # residue-major at n_dyad 16
]

FORMS = [  # (n_in, n_out, n_dyad, tokens, variant, pass, form, token chunks)
    (4352, 2048, 8, 1300, "IT", "gelu_h", "pair", 1),      # blocks of 544: 17 steps
    (2048, 4352, 8, 1300, "OT", "dx_gelu", "pair", 1),     # the same, weights read transposed
    (512, 1024, 16, 1100, "IT", "forward", "pair", 1),     # blocks of 32: half a unit alone
    (1024, 512, 16, 1100, "OT", "dx", "pair", 1),
    (1536, 6144, 8, 3328, "OT", "dx", "pair", 1),          # 192-wide tiles on part of the GPU
    (16384, 4096, 8, 4500, "IT", "gelu_h", "pair", 2),
    (4096, 16384, 8, 4500, "OT", "dx_gelu", "pair", 2),
    (4352, 8192, 8, 1100, "OT", "forward", "res", 1),      # 17 steps
    (8192, 4352, 8, 1100, "IT", "dx", "res", 1),
    (4096, 4096, 4, 3100, "DT", "gelu", "res", 1),
    (4096, 32768, 16, 2600, "OT", "gelu", "res", 2),
    (8448, 2048, 8, 2100, "OT", "gelu_h", "slice", 1),     # blocks of 1056 (33 steps) and 256
    (2048, 8448, 8, 2100, "DT", "dx_gelu", "slice", 1),
    (4096, 1280, 4, 9990, "OT", "forward", "slice", 1),    # n_dyad 4, blocks of 320
    (16384, 4096, 8, 4500, "DT", "gelu_h", "slice", 2),
]

PADDED_FORMS = [  # (n_in, n_out, n_dyad, tokens, variant, input gradient, fused-stage tiles)
    (768, 3070, 5, 600, "OT", 0, False),     # rows of 3070: no aligned piece, blocks of 614
    (768, 3070, 5, 600, "IT", 0, False),
    (770, 3072, 5, 600, "IT", 1, False),     # the same for the input gradient
    (770, 3072, 5, 600, "OT", 1, False),
    (5600, 2520, 70, 520, "OT", 0, False),   # 70 residues: the slice is read in place
    (2520, 5600, 70, 520, "IT", 1, False),
    (768, 3072, 12, 3000, "OT", 0, True),    # blocks of 64 and 256
    (776, 1544, 24, 700, "DT", 0, False),    # blocks of 33 and 65
    (776, 2000, 48, 700, "DT", 0, True),     # blocks of 17 and 42: short reductions
    (768, 768, 16, 1000, "DT", 1, True),     # blocks of 48
    (640, 10400, 10, 530, "OT", 1, True),    # blocks of 64 and 1040, weights read transposed
]


def run_passes(shape, variant, passes):
    """The named passes of one layer against float64 on every 37th token and the last 70."""
    n_in, n_out, D, M = shape
    print("CASE", variant, *shape, *passes, flush=True)
    x, dz = normal(1, M, n_in), normal(2, M, n_out)
    w1, w2 = (normal(s, D, -(-n_out // D), -(-n_in // D), std=0.02) for s in (3, 4))
    b, h_in = normal(5, n_out, std=0.02), normal(6, M, n_in)
    W = dense(w1, w2, variant)[:n_out, :n_in]
    rows = torch.cat([torch.arange(0, M, 37, device=DEV), torch.arange(max(0, M - 70), M, device=DEV)])

    def check(got, ref, what):
        assert got.shape[0] == M
        assert_close(got[rows].float().cpu().numpy(), ref.cpu().numpy(), "bf16", what)

    rh = x[rows].double() @ W.t() + b.double()
    rx = dz[rows].double() @ W
    if "forward" in passes:
        check(dy.forward(x, w1, w2, b, variant), rh, "forward")
    if "gelu" in passes:
        check(dy.forward(x, w1, w2, b, variant, act="gelu"), gelu(rh), "gelu")
    if "gelu_h" in passes:
        y, h = dy.forward(x, w1, w2, b, variant, act="gelu", stash_h=True)
        check(h, rh, "pre-activation")
        check(y, gelu(rh), "gelu, stashed")
    if "dx" in passes:
        check(dy.backward_dx(dz, w1, w2, variant, n_in=n_in), rx, "dx")
    if "dx_gelu" in passes:
        check(dy.backward_dx(dz, w1, w2, variant, act_in="gelu", h_in=h_in), rx * gelu_grad(h_in[rows].double()),
              "dx gelu'")


@pytest.mark.parametrize("variant", ("IT", "OT", "DT"))
@pytest.mark.parametrize("shape", CASES, ids=lambda c: "x".join(map(str, c)))
def test_forward_and_dx(shape, variant):
    run_passes(shape, variant, ("forward", "gelu_h", "dx", "dx_gelu"))


@pytest.mark.parametrize("case", FORMS, ids=lambda c: "-".join(map(str, c)))
def test_forms(case):
    run_passes(case[:4], case[4], (case[5],))


@pytest.mark.parametrize("case", PADDED_FORMS, ids=lambda c: "-".join(map(str, c)))
def test_padded_forms(case):
    run_passes(case[:4], case[4], ("dx", "dx_gelu") if case[5] else ("forward", "gelu_h"))


SPECIAL = [  # (n_in, n_out, n_dyad, tokens, variant, dtype): pair, residue-major, slice, padded (large and fused-stage), fp32
    (4352, 2048, 8, 1300, "IT", torch.bfloat16),
    (4352, 8192, 8, 1100, "OT", torch.bfloat16),
    (8448, 2048, 8, 2100, "OT", torch.bfloat16),
    (768, 3072, 5, 700, "IT", torch.bfloat16),
    (768, 3072, 5, 700, "DT", torch.bfloat16),
    (768, 3072, 12, 700, "OT", torch.bfloat16),
    (272, 528, 4, 130, "DT", torch.float32),
]


@pytest.mark.parametrize("value", (float("inf"), float("nan")))
@pytest.mark.parametrize("case", SPECIAL, ids=lambda c: "-".join(map(str, c)))
def test_infinity_and_nan_stay_in_their_outputs(case, value):
    """One infinite (NaN) input reaches the outputs that its weights feed, in its own token, and
    no other: neither zero padding nor a step that is loaded and not multiplied spreads it."""
    n_in, n_out, D, M, variant, dt = case
    print("CASE special", *case, value, flush=True)
    x = normal(1, M, n_in).to(dt)
    w1, w2 = (normal(s, D, -(-n_out // D), -(-n_in // D), std=0.02).to(dt) for s in (3, 4))
    one = torch.ones_like(w1)
    none = torch.zeros_like(w1)
    for col in (0, n_in // D - 1, n_in // 2 + 3, n_in - 1):
        row = (37 * col + 11) % M
        clean = x.clone()
        clean[row, col] = 0
        y0 = dy.forward(clean, w1, w2, None, variant, n_out=n_out)
        bad = clean.clone()
        bad[row, col] = value
        y = dy.forward(bad, w1, w2, None, variant, n_out=n_out)
        fed = (dense(one, none, variant) + dense(none, one, variant))[:n_out, col] != 0
        assert bool(torch.isfinite(y0).all())
        assert bool((~torch.isfinite(y[row][fed])).all())
        assert torch.equal(y[row][~fed], y0[row][~fed])
        others = torch.arange(M, device=DEV) != row
        assert torch.equal(y[others], y0[others])
