"""The native marshalling is taken only by the interpreter, the torch and the
library ABI that it was built for, and the build does without it where its
compiler is missing."""
import importlib.machinery
import types

import pytest
import torch

from paper_2510_22876_amd import build as hip_build


@pytest.fixture(scope="module")
def sd():
    from paper_2510_22876_amd import specdec
    return specdec


def test_file_is_named_for_the_interpreter():
    assert hip_build.MARSHAL.name == "_marshal" + importlib.machinery.EXTENSION_SUFFIXES[0]
    assert "cpython" in hip_build.MARSHAL.name


def test_taken_by_the_torch_and_abi_it_was_built_for(sd):
    if not hip_build.MARSHAL.exists():
        pytest.skip("the native marshalling is not built")
    assert sd._native.built_for == (str(torch.__version__), sd.abi_version())
    assert sd._load_native() is sd._native


@pytest.mark.parametrize("differs", ["torch", "abi", "nothing said"])
def test_left_alone_by_another(sd, monkeypatch, differs):
    connected = []
    fake = types.SimpleNamespace(connect=lambda *a: connected.append(a))
    built_for = (str(torch.__version__), sd.abi_version())
    if differs == "torch":
        fake.built_for = ("0.0.1", built_for[1])
    elif differs == "abi":
        fake.built_for = (built_for[0], built_for[1] + 1)
    import paper_2510_22876_amd as pkg
    monkeypatch.setattr(pkg, "_marshal", fake, raising=False)
    assert sd._load_native() is None and not connected
    fake.built_for = built_for
    assert sd._load_native() is fake and len(connected) == 1


def test_build_without_a_compiler(monkeypatch, tmp_path):
    left = tmp_path / "_marshal.so"
    left.write_bytes(b"of an earlier build")
    monkeypatch.setattr(hip_build, "MARSHAL", left)
    monkeypatch.setenv("CXX", "no-such-compiler")
    assert hip_build.build_marshal() is None
    assert not left.exists()
