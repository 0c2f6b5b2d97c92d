"""The native reading of tensor addresses: used with the torch that it was built for, done without otherwise; on the device, what
it answers itself and what it leaves to the Python form."""
import os
import subprocess
import sys
import types

import pytest
import torch

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_native_form_of_this_torch_is_used():
    if build.pointers_cmd() is None:
        pytest.skip("no g++")
    assert B._native is not None and B._native.torch_build == build.torch_build()
    assert B._pointers is B._native.pointers


@pytest.mark.parametrize("native", [None, types.SimpleNamespace(torch_build="1.0 0", pointers=None), types.SimpleNamespace(pointers=None)])
def test_python_form_without_it_or_with_another_torch(native):
    f = B._choose_pointers(native)
    assert f() == () and f(None, None) == (None, None)
    with pytest.raises(ValueError, match="device-resident contiguous tensors only"):
        f(torch.zeros(3))


def test_binding_imports_without_the_native_module():
    code = ("import sys; sys.modules['paper_2603_09983_amd._pointers'] = None\n"
            "from paper_2603_09983_amd import binding as B\n"
            "assert B._native is None and B._pointers(None) == (None,)\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


def test_build_knows_the_torch_it_was_built_for(monkeypatch, tmp_path):
    if build.pointers_cmd() is None:
        pytest.skip("no g++")
    monkeypatch.setattr(build, "LIB_POINTERS", str(tmp_path / "lib"))
    monkeypatch.setattr(build, "POINTERS_STAMP", str(tmp_path / "stamp"))
    assert build.pointers_stale()
    (tmp_path / "lib").write_text("")
    (tmp_path / "stamp").write_text(" ".join(build.pointers_cmd()))
    assert not build.pointers_stale()
    monkeypatch.setattr(build, "torch_build", lambda: "1.0 0")
    assert build.pointers_stale() and build.stale()


def test_build_names_the_command_that_failed():
    with pytest.raises(RuntimeError, match="^false --flag failed"):
        build._run(["false", "--flag"], False)


@pytest.mark.gpu
@pytest.mark.parametrize("make,good", [
    (lambda: torch.zeros(6, 4, device="cuda"), True),
    (lambda: torch.zeros(6, 4, device="cuda")[2:], True),                   # (an address behind its storage's start)
    (lambda: torch.nn.Parameter(torch.zeros(6, device="cuda")), True),
    (lambda: torch.zeros(0, 4, device="cuda"), True),
    (lambda: torch.zeros(1, 5, device="cuda").t(), True),                   # (strides of lengths of one do not count)
    (lambda: torch.zeros(6, 4, device="cuda").t(), False),
    (lambda: torch.zeros(6, 4, device="cuda")[:, 1:], False),
    (lambda: torch.zeros(8, device="cuda")[::2], False),
    (lambda: torch.zeros(1, device="cuda").expand(4), False),
    (lambda: torch.zeros(8, pin_memory=True), False),
    (lambda: torch.zeros(8, device="meta"), False),
])
def test_device_tensors(make, good):
    t = make()
    if good:
        assert B._pointers(None, t, t) == (None, t.data_ptr(), t.data_ptr()) == tuple(map(B._ptr, (None, t, t)))
    else:
        for f in (B._pointers, B._ptr):
            with pytest.raises(ValueError, match="device-resident contiguous tensors only"):
                f(t)
