"""GPU parity of the 4-wave tiles at the plans their choice makes: the widest tile
with many splits of a long reduction, small tiles with few, no split, both passes;
test_plan_cpu.py checks on the CPU that each case takes the plan it names.
Against the dense weight in float64, every output."""
import pytest
import torch

from tests.test_gpu_pp import run_passes

pytestmark = pytest.mark.gpu

TILES = [  # (n_in, n_out, n_dyad, tokens, variant, input gradient, (tile rows, columns, splits))
    (32768, 8192, 8, 64, "IT", 0, (64, 256, 16)),
    (16384, 4096, 4, 200, "IT", 0, (128, 256, 8)),
    (3072, 768, 4, 200, "IT", 0, (64, 64, 4)),
    (3072, 768, 4, 2047, "IT", 0, (64, 64, 1)),
    (768, 3072, 4, 700, "IT", 0, (64, 64, 1)),
    (768, 3072, 4, 2047, "OT", 0, (64, 256, 1)),
    (768, 3072, 4, 2047, "IT", 1, (128, 192, 3)),
    (4096, 16384, 2, 33, "DT", 1, (64, 256, 32)),
    (768, 3072, 6, 300, "IT", 0, (64, 64, 1)),
    (8192, 2048, 2, 500, "OT", 1, (128, 256, 2)),
]


@pytest.mark.parametrize("case", TILES, ids=lambda c: "-".join(map(str, c)))
def test_tiles(case):
    run_passes(case[:4], case[4], ("dx", "dx_gelu") if case[5] else ("forward", "gelu", "gelu_h"))
