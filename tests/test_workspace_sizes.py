"""Host-only: how much workspace shapes ask for."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_09983_amd", "libmoe_spac.so")


class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("T", "H", "E", "k", "F", "C", "n_shared", "F_shared", "launch_form")]


@pytest.mark.parametrize("T,n_shared", [(33, 8), (64, 900), (64, 1100), (128, 2000)])
def test_any_number_of_shared_experts(T, n_shared):
    """More than 32 tokens: room for every shared expert's activations (4 bytes) and outputs (8 bytes), not for its partial
    sums over slices of its width, however many shared experts there are."""
    lib = ctypes.CDLL(LIB)
    H, E, k, F, C, Fs = 2048, 1024, 8, 64, 1000, 2048
    n = ctypes.c_size_t(0)
    sh = Shape(T, H, E, k, F, C, n_shared, Fs)
    assert lib.moe_workspace_bytes(ctypes.byref(sh), ctypes.byref(n)) == 0
    assert n.value <= n_shared * T * (4 * Fs + 8 * H) + T * k * (4 * F + 8 * H) + (1 << 20)
