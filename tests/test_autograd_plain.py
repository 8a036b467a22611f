"""Which tensors the autograd wrappers' backward may hand to the library by their pointers (no GPU)."""
import torch

from paper_2603_16428_amd.lce import _bytes_are_values


def test_bytes_are_values():
    assert _bytes_are_values(torch.ones(3)) and _bytes_are_values(torch.ones(0)) and _bytes_are_values(torch.ones(()))
    negated = torch.complex(torch.tensor(0.0), torch.tensor(2.0)).conj().imag
    assert negated.item() == -2.0 and not _bytes_are_values(negated)
    assert _bytes_are_values(negated.resolve_neg())
    assert not _bytes_are_values(torch._efficientzerotensor((2, 3)))
