"""Host-only: the addresses that the binding passes on, and what it refuses."""
import types

import pytest
import torch

from paper_2603_09983_amd import binding as B


def _fake(cuda=True, contiguous=True, address=4096):
    return types.SimpleNamespace(is_cuda=cuda, is_contiguous=lambda: contiguous, data_ptr=lambda: address)


def test_addresses_in_order():
    assert B._pointers() == ()
    assert B._pointers(None, _fake(), None, _fake(address=0)) == (None, 4096, None, 0)


@pytest.mark.parametrize("bad", [torch.zeros(3), torch.nn.Parameter(torch.zeros(3)), _fake(cuda=False), _fake(contiguous=False)])
def test_refused_as_by_the_python_form(bad):
    for f in (B._pointers, B._ptr):
        with pytest.raises(ValueError, match="device-resident contiguous tensors only"):
            f(bad)


@pytest.mark.parametrize("bad", [3, "x", object()])
def test_not_a_tensor(bad):
    for f in (B._pointers, B._ptr):
        with pytest.raises(AttributeError):
            f(bad)


def test_subclass_keeps_its_own_attributes():
    class Sub(torch.Tensor):
        is_cuda = True

        def data_ptr(self):
            return 77
    assert B._pointers(torch.zeros(3).as_subclass(Sub)) == (77,)
