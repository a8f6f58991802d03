"""The C-ABI library builds, loads without a GPU and exports every function that
include/hdc.h declares; status texts are defined.  No compute is called here."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "hdc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(hdc_[a-z_]+)\s*\(", text)))


def test_header_declares_the_four_entry_points_and_helpers():
    names = declared_functions()
    for must in ("hdc_encode", "hdc_train_classical", "hdc_train_online", "hdc_search",
                 "hdc_create", "hdc_destroy", "hdc_binarize_classical", "hdc_binarize_online",
                 "hdc_strerror"):
        assert must in names


def test_library_exports_every_declared_symbol():
    from paper_2206_04746_amd import binding
    assert os.path.exists(binding.LIB_PATH)
    lib = ctypes.CDLL(binding.LIB_PATH)
    for name in declared_functions():
        assert hasattr(lib, name), name
    assert sorted(binding.SYMBOLS) == declared_functions()


def test_status_texts_and_version():
    from paper_2206_04746_amd import binding
    for code in (0, -1, -2, -3, -4, -99):
        assert binding.strerror(code)
    assert binding.strerror(0) == "ok"
    assert re.fullmatch(r"\d+\.\d+\.\d+", binding.version())


def test_binding_imports_and_finds_the_stream_without_private_names_of_torch(monkeypatch):
    import importlib.util
    import types

    import torch

    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name, raising=False)
    spec = importlib.util.spec_from_file_location("binding_again", os.path.join(ROOT, "paper_2206_04746_amd", "binding.py"))
    binding = importlib.util.module_from_spec(spec)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=1000 + device))
    spec.loader.exec_module(binding)
    assert binding._stream(None) == 1003
    assert binding._stream(17) == 17 and binding._stream(types.SimpleNamespace(cuda_stream=5)) == 5


def test_product_package_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2206_04746_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                src = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in src and "from oracle" not in src, f
                assert "hdc_oracle" not in src and "liboracle" not in src, f
