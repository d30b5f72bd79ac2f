"""Inference without autograd: the same results as the recorded path (up to the order of fp32 sums
where a stashed pre-activation changes the form), which every call that could need a derivative
still takes."""
import pytest
import torch
from torch.autograd import forward_ad

from paper_2312_06881_amd import nn
from paper_2312_06881_amd.nn import DyadFF, DyadLinear


def test_plain_only_without_derivatives():
    t, p = torch.zeros(2, 2), torch.nn.Parameter(torch.zeros(2))
    assert not nn._plain(t, p)                       # gradients on
    with torch.no_grad():
        assert nn._plain(t, p, None)
        with forward_ad.dual_level():
            assert not nn._plain(t, p)
        seen = []
        torch.func.vmap(lambda a: (seen.append(nn._plain(a)), a)[1])(t)
        assert seen == [False]

        class Sub(torch.Tensor):
            pass

        assert not nn._plain(t.as_subclass(Sub))


@pytest.mark.gpu
@pytest.mark.parametrize("tokens", (1, 33, 1500))
@pytest.mark.parametrize("variant", ("IT", "OT", "DT"))
def test_no_grad_matches_recorded(tokens, variant):
    torch.manual_seed(0)
    x = torch.randn(1, tokens, 256, device="cuda").bfloat16()
    for m in (DyadLinear(256, 512, 4, variant, device="cuda"), DyadFF(256, 1024, 4, variant, device="cuda")):
        y = m(x)
        assert y.requires_grad
        with torch.no_grad():
            z = m(x)
        assert not z.requires_grad and torch.equal(y.detach(), z)
