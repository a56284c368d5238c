"""The C-ABI library builds, loads without a GPU and exports every function include/sgnn.h declares."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "sgnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sgnn_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_four_calls():
    names = _declared()
    for n in ("sgnn_sample_uniform", "sgnn_induced_csr", "sgnn_gcn_fwd", "sgnn_gcn_bwd"):
        assert n in names


def test_library_exports_every_declared_symbol():
    from paper_2604_02651_amd import build as b
    path = b.build(force=False)
    L = ctypes.CDLL(path)
    for n in _declared():
        assert hasattr(L, n), n


def test_binding_refuses_to_run_without_the_library(monkeypatch, tmp_path):
    import paper_2604_02651_amd.binding as binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "missing.so"))
    import pytest
    with pytest.raises(ImportError):
        binding.lib()


def test_product_never_imports_the_oracle():
    pkg = os.path.join(ROOT, "paper_2604_02651_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                src = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in src.lower(), f


def test_launchers_remember_nothing_for_the_whole_process():
    # attributes of kernels belong to a device: a flag of the process would hold for the first one only
    csrc = os.path.join(ROOT, "paper_2604_02651_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        found = re.findall(r"^\s+static\s+(?:const\s+)?(?:bool|int|hipError_t)\s+\w+\s*=.*$", open(os.path.join(csrc, f)).read(), flags=re.M)
        assert not [x for x in found if "constexpr" not in x], (f, found)
