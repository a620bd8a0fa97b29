"""What build.py compiles for whom.  Nothing is compiled here."""
import os
import sys
import sysconfig

import pytest

from paper_2410_16926_amd import build


@pytest.fixture
def commands(monkeypatch):
    """The commands that a build would run."""
    ran = []

    def run(command):
        ran.append(command)
        return ""
    monkeypatch.setattr(build, "_run", run)
    return ran


def outputs(commands):
    return [os.path.basename(c[c.index("-o") + 1]) for c in commands]


def test_the_library_is_built_without_torch(commands, monkeypatch):
    monkeypatch.setitem(sys.modules, "torch", None)            # importing it raises ImportError
    build.build()
    assert outputs(commands) == [s + ".o" for s in build.SOURCES] + ["libpvq.so"]
    python = sysconfig.get_paths()["include"]
    assert not any("torch" in a or a == f"-I{python}" for c in commands for a in c)
    with pytest.raises(ImportError):
        build.build(library=False, binding=True)


def test_the_binding_alone(commands):
    pytest.importorskip("torch")
    build.build(library=False, binding=True)
    assert outputs(commands) == ["pvq_torch.cpp.o", os.path.basename(build.TORCH_PATH)]


def test_a_module_fits_one_python_and_one_torch(monkeypatch, tmp_path):
    torch = pytest.importorskip("torch")
    assert build.TORCH_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert build.binding_fits()
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", torch.__version__ + ".1")
        assert not build.binding_fits() and build.binding_is_stale()
        m.setattr(torch, "__version__", "2.1")
        assert not build.binding_fits()
    with monkeypatch.context() as m:
        m.setattr(build, "TORCH_PATH", str(tmp_path / "none.so"))
        assert not build.binding_fits()


def test_up_to_date_parts_are_left_out(commands, monkeypatch):
    monkeypatch.setattr(build, "library_is_stale", lambda: False)
    monkeypatch.setattr(build, "binding_is_stale", lambda: True)
    build.build(force=False)
    assert outputs(commands) == ["pvq_torch.cpp.o", os.path.basename(build.TORCH_PATH)]
    del commands[:]
    monkeypatch.setattr(build, "binding_is_stale", lambda: False)
    build.build(force=False)
    assert commands == []


def test_every_header_counts_for_staleness():
    headers = {n for n in os.listdir(os.path.join(os.path.dirname(build.__file__), "csrc")) if n.endswith(".h")}
    assert headers == set(build.HEADERS)
