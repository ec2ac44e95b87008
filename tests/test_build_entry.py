"""build() compiles the library, the oracle and the package whichever test programs are
there: none, some, or one that does not compile (CPU; the compilers are stood in for)."""
import os

import pytest

import __graft_entry__ as entry
from oracle import build_oracle
from paper_2609_39185_amd import build as hip_build

GOOD = "def build(verbose=False):\n    open(__file__ + '.built', 'w').close()\n"
BAD = "import subprocess\ndef build(verbose=False):\n    subprocess.run(['false'], check=True)\n"
CASES = {"no folder": None, "no programs": {}, "one": {"build_c_abi_test": GOOD},
         "other names": {"build_some_program": GOOD},
         "one fails": {"build_a": BAD, "build_c_abi_test": GOOD, "build_z": "import no_such_module\n"}}


@pytest.mark.parametrize("case", sorted(CASES))
def test_build_does_not_depend_on_the_test_programs(case, tmp_path, monkeypatch):
    programs = CASES[case]
    if programs is not None:
        (tmp_path / "tests").mkdir()
        (tmp_path / "tests" / "__init__.py").write_text("")
        for name, text in programs.items():
            (tmp_path / "tests" / f"{name}.py").write_text(text)
    done = []
    monkeypatch.setattr(entry, "ROOT", str(tmp_path))
    monkeypatch.setattr(hip_build, "build", lambda verbose=False: done.append("library"))
    monkeypatch.setattr(build_oracle, "build", lambda verbose=False: done.append("oracle"))
    entry.build()
    assert done == ["library", "oracle"]
    for name, text in (programs or {}).items():
        built = os.path.exists(tmp_path / "tests" / f"{name}.py.built")
        assert built == (text is GOOD), name


@pytest.mark.parametrize("how", ["no compiler", "compile error"])
def test_library_is_usable_without_the_module(how, tmp_path, monkeypatch):
    """Where the marshalling module does not compile, build() keeps the library and leaves
    no older module beside it."""
    import subprocess

    def stand_in(cmd, **kw):
        if cmd[0] == "g++":
            if how == "no compiler":
                raise FileNotFoundError("g++")
            raise subprocess.CalledProcessError(1, cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()

    library, native = str(tmp_path / "libssmq.so"), str(tmp_path / "_native.so")
    open(native, "w").close()
    monkeypatch.setattr(hip_build, "LIBRARY", library)
    monkeypatch.setattr(hip_build, "NATIVE", native)
    monkeypatch.setattr(hip_build.subprocess, "run", stand_in)
    assert hip_build.build() == library
    assert os.path.exists(library) and not os.path.exists(native)
