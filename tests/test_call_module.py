"""The binding's module in C++ where it cannot be built or does not load: the build goes on, the import says so, the calls go through
ctypes (no GPU)."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2605_07330_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_file_carries_the_python_it_was_built_for():
    assert os.path.basename(build.CALL) == "_call" + sysconfig.get_config_var("EXT_SUFFIX") != "_call.so"


def test_the_build_goes_on_without_a_compiler(monkeypatch, tmp_path, capsys):
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_call.tag.so"))
    for name in ("_call.so", "_call.tag.so"):                               # of an earlier build
        (tmp_path / name).write_bytes(b"")
    monkeypatch.setenv("CXX", "no-such-compiler")
    assert build.build_call() == ""
    assert "no-such-compiler" in capsys.readouterr().err and not list(tmp_path.iterdir())


def test_a_module_that_does_not_compile_is_an_error(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_call.tag.so"))
    monkeypatch.setattr(build, "CALL_SRC", str(tmp_path / "call.cpp"))
    (tmp_path / "call.cpp").write_text("int x = ;\n")
    with pytest.raises(subprocess.CalledProcessError):
        build.build_call()


@pytest.mark.parametrize("why", ["absent", "other torch"])
def test_the_import_says_what_is_missing(why):
    code = """
import sys, types, warnings
if %r == "absent":
    sys.modules["paper_2605_07330_amd._call"] = None
else:
    m = types.ModuleType("paper_2605_07330_amd._call"); m.torch_version = "0.0"; sys.modules[m.__name__] = m
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    import paper_2605_07330_amd
    if "paper_2605_07330_amd._call" in sys.modules and sys.modules["paper_2605_07330_amd._call"] is not None:
        paper_2605_07330_amd._call = sys.modules["paper_2605_07330_amd._call"]
    from paper_2605_07330_amd import srs
assert srs._call is None
assert any("take longer" in str(x.message) for x in w), [str(x.message) for x in w]
""" % why
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=300)
