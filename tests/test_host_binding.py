"""Loading the binding without a GPU."""
import pytest
import torch

from paper_2105_00053_amd import binding


@pytest.fixture
def unloaded(monkeypatch):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)


@pytest.mark.parametrize("content", [None, b"", b"no shared object"])
def test_the_library_loads_without_the_extension_module(unloaded, monkeypatch, tmp_path, content):
    """Missing, or built for something else: a warning, and the Python code takes the calls."""
    path = tmp_path / "positnn_native.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(binding, "_NATIVE_PATH", str(path))
    with pytest.warns(RuntimeWarning, match="positnn_native.so"):
        library = binding.load()
    assert binding._native is None and binding._ready() is None
    assert binding.posit_gemm_workspace("p32", "p32", 0, 0, 512, 512, 512) > 0
    assert binding.load() is library


def test_the_extension_module_knows_the_formats_of_the_python_code():
    """It has no table of its own: rows that are no formats are refused."""
    binding.load()
    module = binding._load_native()
    addresses = [1] * len(binding._NATIVE_ORDER)
    for rows in (None, ((128, 1, torch.uint8, (torch.uint8,)),), ((0, 1, "uint8", (torch.uint8,)),), ((0, 1, torch.uint8, (1,)),), ((0, 1, torch.uint8),)):
        with pytest.raises((TypeError, ValueError)):
            module.init(rows, *addresses)
    with pytest.raises(TypeError):
        module.init((), *addresses[:-1])
