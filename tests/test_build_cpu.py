"""The call module is optional: without a C compiler that takes it the library is built all the same, and no older module stays."""
import os
import sys

import pytest

from paper_2210_12415_amd import build


@pytest.fixture
def package(tmp_path, monkeypatch):
    """A package of one library source, with a compiler that only writes what it is asked for."""
    for folder in ("csrc", "native"):
        (tmp_path / "pkg" / folder).mkdir(parents=True)
    (tmp_path / "include").mkdir()
    (tmp_path / "include" / "alt.h").write_text("")
    (tmp_path / "pkg" / "csrc" / "one.cpp").write_text("")
    (tmp_path / "pkg" / "native" / "altcall.c").write_text("#error not today\n")
    compiler = tmp_path / "compiler"
    compiler.write_text("#!%s\nimport sys\nopen(sys.argv[sys.argv.index('-o') + 1], 'w').close()\n" % sys.executable)
    compiler.chmod(0o755)
    here = str(tmp_path / "pkg")
    for name, value in dict(HERE=here, CSRC=os.path.join(here, "csrc"), OBJ=os.path.join(here, "csrc", "_build"), LIB=os.path.join(here, "libalt.so"),
                            HIPCC=str(compiler)).items():
        monkeypatch.setattr(build, name, value)
    return tmp_path


@pytest.mark.parametrize("compiler", ["/nonexistent/cc", None], ids=["no_compiler", "compile_error"])
def test_library_is_built_without_the_call_module(package, compiler, monkeypatch, capsys):
    if compiler:
        monkeypatch.setenv("CC", compiler)
    else:
        monkeypatch.delenv("CC", raising=False)
    module = os.path.join(build.HERE, "_altcall" + build.sysconfig.get_config_var("EXT_SUFFIX"))
    open(module, "w").close()
    os.utime(module, (1, 1))                  # older than its source
    assert build.build(jobs=1) == build.LIB and os.path.exists(build.LIB)
    assert not os.path.exists(module)
    assert "through ctypes" in capsys.readouterr().out
