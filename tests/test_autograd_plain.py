"""Which tensors the autograd wrappers' backward may hand to the library by their pointers (no GPU)."""
import types

import pytest
import torch
from torch.autograd import forward_ad

from paper_2603_16428_amd import lce
from paper_2603_16428_amd.lce import _bytes_are_values, _differentiated, _scaled


def test_bytes_are_values():
    assert _bytes_are_values(torch.ones(3)) and _bytes_are_values(torch.ones(0)) and _bytes_are_values(torch.ones(()))
    negated = torch.complex(torch.tensor(0.0), torch.tensor(2.0)).conj().imag
    assert negated.item() == -2.0 and not _bytes_are_values(negated)
    assert _bytes_are_values(negated.resolve_neg())
    assert not _bytes_are_values(torch._efficientzerotensor((2, 3)))
    assert not _bytes_are_values(torch.nn.Parameter(torch.ones(3))) and not _bytes_are_values(torch.ones(3).to_sparse())
    assert not _bytes_are_values(torch.zeros(0).to_sparse())
    seen = []
    torch.func.vmap(lambda t: (seen.append(_bytes_are_values(t)), t + 1)[1])(torch.ones(2, 3))
    torch.func.grad(lambda t: (seen.append(_bytes_are_values(t)), t.sum())[1])(torch.ones(3))
    assert seen == [False, False]


@pytest.mark.parametrize("level_told", [True, False])
def test_differentiated(monkeypatch, level_told):
    if not level_told:  # a torch that has no name for the current level: every tensor is asked
        monkeypatch.setattr(lce.torch.autograd, "forward_ad", types.SimpleNamespace(unpack_dual=forward_ad.unpack_dual))
    x = torch.ones(3, requires_grad=True)
    assert _differentiated((torch.ones(3), x)) and not _differentiated((x.detach(),))
    with torch.no_grad():  # a backward pass without create_graph
        assert not _differentiated((x,))
    with forward_ad.dual_level():
        assert _differentiated((torch.ones(3), forward_ad.make_dual(torch.ones(3), torch.ones(3))))
        assert not _differentiated((torch.ones(3),))


@pytest.mark.parametrize("modes", [None, lambda: 1, lambda: 0])
def test_torch_without_the_private_names(monkeypatch, modes):
    """A torch that has none of its private names any more scales with its own operators."""
    for name in ("_has_storage", "_len_torch_dispatch_stack"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(lce, "_dispatch_modes", modes)
    ts = (torch.randn(5).bfloat16(), torch.randn(3, 4).bfloat16())
    for got, t in zip(_scaled(torch.tensor(0.5), ts), ts):
        assert got.dtype == t.dtype and torch.equal(got, t * 0.5)
