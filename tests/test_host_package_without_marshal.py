"""The package around its native argument marshalling: what works where that is damaged, missing or built later.  Each case is a
copy of the package in a process of its own; nothing here needs a GPU."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = "paper_2505_20776_amd"
LIBRARY = os.path.join(ROOT, PACKAGE, "libspecext.so")
MARSHAL = os.path.join(ROOT, PACKAGE, "_marshal.so")
SPLITS = ("sx.num_splits(sx.make_desc(dtype=1, n_q_heads=8, n_kv_heads=2, head_dim=128, prefix_len=300, n_tree=8, num_splits=200))")


@pytest.fixture
def copy(tmp_path):
    """The package's Python files and the built library, without the marshalling."""
    if not (os.path.exists(LIBRARY) and os.path.exists(MARSHAL)):
        from paper_2505_20776_amd.build import build_library
        build_library(verbose=False)
    package = tmp_path / PACKAGE
    package.mkdir()
    for name in os.listdir(os.path.join(ROOT, PACKAGE)):
        if name.endswith(".py"):
            shutil.copy(os.path.join(ROOT, PACKAGE, name), package)
    os.symlink(LIBRARY, package / "libspecext.so")
    return package


def _run(copy, code, *options, **env):
    env = {k: v for k, v in dict(os.environ, **env).items() if k not in ("SPECEXT_LIBRARY", "PYTHONPATH")}
    run = subprocess.run([sys.executable, *options, "-c", code], cwd=copy.parent, env=env, stdout=subprocess.PIPE,
                         stderr=subprocess.STDOUT, text=True, timeout=250)
    assert run.returncode == 0, run.stdout[-3000:]
    return run.stdout


@pytest.mark.parametrize("what", ["empty", "text", "another library"])
def test_marshalling_that_does_not_load(copy, what):
    """The package imports, its functions and its build work, and loading the library says what to do."""
    if what == "another library":
        shutil.copy(LIBRARY, copy / "_marshal.so")
    else:
        (copy / "_marshal.so").write_bytes(b"" if what == "empty" else b"no shared object" * 400)
    out = _run(copy, f"import {PACKAGE} as sx, {PACKAGE}.build, types; print({SPLITS}); print(type(sx.verify_attn) is types.FunctionType)")
    assert "3\nTrue" in out and "RuntimeWarning" in out and f"python -m {PACKAGE}.build" in out


def test_without_marshalling(copy):
    out = _run(copy, f"import {PACKAGE} as sx; print({SPLITS})")
    assert out.endswith("3\n") and "RuntimeWarning" in out and "_marshal.so is missing" in out


def test_without_torch(copy):
    """Addresses instead of tensors: nothing of the marshalling is asked for."""
    for _ in range(2):
        out = _run(copy, f"import sys; sys.modules['torch'] = None; import {PACKAGE} as sx; print({SPLITS}); "
                         "print(sx.select_chunks(4096, 0, 2, 4096, 4096, stream=0, check=False))")
        assert out == "3\n-1\n"
        os.path.exists(copy / "_marshal.so") or os.symlink(MARSHAL, copy / "_marshal.so")


def test_built_after_the_import(copy):
    """Loading the library takes the marshalling over that was built since the package was imported."""
    out = _run(copy, f"import os, {PACKAGE} as sx; from {PACKAGE} import binding; os.symlink({MARSHAL!r}, {str(copy / '_marshal.so')!r}); "
                     "sx.load_library(); print(len(binding._marshal.FUNCTIONS)); "
                     "print(all(type(getattr(m, n)).__name__ == 'Call' for m in (sx, binding) for n in binding._marshal.FUNCTIONS)); "
                     "print(sx.select_chunks(4096, 0, 2, 4096, 4096, stream=0, check=False))")
    assert out == "10\nTrue\n-1\n"


@pytest.mark.parametrize("missing", ["torch", "headers"])
def test_build_without_what_the_marshalling_needs(copy, tmp_path, missing):
    """The library is built, the build says what is not, and an older _marshal.so does not stay beside a newer library.  A script
    stands in for hipcc: it notes each call and writes the output file."""
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\necho "$@" >> calls\nwhile [ "$1" != -o ]; do shift; done; echo built > "$2"\n')
    hipcc.chmod(0o755)
    os.remove(copy / "libspecext.so")
    os.symlink(MARSHAL, copy / "_marshal.so")
    hide = "sys.modules['torch'] = None; " if missing == "torch" else ""
    out = _run(copy, f"import sys; {hide}from {PACKAGE}.build import build_library, SOURCES; build_library(); print(len(SOURCES))",
               HIPCC=str(hipcc), CXX="false")
    assert "_marshal.so is not" in out and not os.path.lexists(copy / "_marshal.so")
    assert (copy / "libspecext.so").read_text() == "built\n"
    assert len(open(tmp_path / "calls").readlines()) == int(out.splitlines()[-1]) + 1
