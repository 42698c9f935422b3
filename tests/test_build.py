"""The in-tree build: what a partial build may keep, what is built without g++, and an extension module that does not fit."""
import os
import stat
import subprocess
import sys

import pytest

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd import build as hb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPILER = '#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\ndate +%s%N > "$2"\n'        # writes the file that -o names


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A copy of the sources whose compilers only leave files."""
    pkg = tmp_path / "pkg"
    (pkg / "csrc").mkdir(parents=True)
    (tmp_path / "include").mkdir()
    files = [pkg / "csrc" / f for f in (*hb.SOURCES, "osdn_native.cpp", "osdn_device.h")] + [tmp_path / "include" / "osdn.h"]
    for f in files:
        f.write_text("")
        os.utime(f, (1e9, 1e9))
    for name, text in (("hipcc", COMPILER), ("cxx", COMPILER), ("no_cxx", "#!/bin/sh\necho no headers\nexit 1\n")):
        (tmp_path / name).write_text(text)
        (tmp_path / name).chmod(stat.S_IRWXU)
    monkeypatch.setenv("HIPCC", str(tmp_path / "hipcc"))
    monkeypatch.setenv("CXX", str(tmp_path / "cxx"))
    for name, path in (("HERE", pkg), ("CSRC", pkg / "csrc"), ("OBJ", pkg / "_build"), ("LIB", pkg / "libosdn.so"),
                       ("NATIVE", pkg / os.path.basename(hb.NATIVE)), ("NATIVE_SOURCE", pkg / "csrc" / "osdn_native.cpp")):
        monkeypatch.setattr(hb, name, str(path), raising=False)
    hb.build()
    return tmp_path, pkg, lambda: open(hb.NATIVE).read()


@pytest.mark.parametrize("changed", ["include/osdn.h", "pkg/csrc/osdn_native.cpp"])
def test_a_partial_build_renews_a_module_of_an_older_interface(tree, changed):
    root, pkg, native = tree
    first = native()
    hb.build(only=["osdn_step.hip"])
    assert native() == first
    t = os.path.getmtime(hb.NATIVE) + 1
    os.utime(root / changed, (t, t))
    hb.build(only=["osdn_step.hip"])
    assert native() != first


def test_the_library_is_built_without_a_host_compiler(tree, monkeypatch):
    root, pkg, native = tree
    (pkg / "_native.so").write_text("of an earlier build")
    os.remove(hb.LIB)
    for cxx in ("no_cxx", "not_there"):
        monkeypatch.setenv("CXX", str(root / cxx))
        with pytest.warns(UserWarning, match="not built"):
            hb.build()
        assert os.path.exists(hb.LIB) and not list(pkg.glob("_native*"))


def test_a_module_that_does_not_fit_is_refused():
    ob.lib()
    from paper_2605_13473_amd import _native
    size = ob.ctypes.sizeof(ob.OsdnParams)
    for args in ((0, size + 4, ob.torch.__version__), (0, size, "1.0")):
        with pytest.raises(ImportError, match="built for"):
            _native.bind(*args)


def test_a_missing_module_is_not_passed_over_in_silence():
    code = ("import sys, warnings; sys.modules['paper_2605_13473_amd._native'] = None\n"
            "from paper_2605_13473_amd import binding\n"
            "with warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always'); binding.lib(); binding.lib()\n"
            "assert binding._step_native is None and len([x for x in w if 'extension module' in str(x.message)]) == 1, w\n")
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True)
