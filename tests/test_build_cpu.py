"""What the build makes where torch or a compiler of the binding's module is missing: the C library is complete, and the binding does without
the module."""
import subprocess
import sys

import pytest

from paper_2312_00752_amd import build

ROOT = build.ROOT


@pytest.fixture
def commands(monkeypatch, tmp_path):
    """The build with its commands noted instead of run (their outputs are made empty), in a folder of its own."""
    ran = []

    def run(cmd, cwd, verbose):
        ran.append(cmd)
        if "ss_marshal.cpp" in " ".join(cmd) and fail:
            raise RuntimeError("compiler failed")
        open(cmd[cmd.index("-o") + 1], "w").close()
    fail = []
    for name, path in (("BUILD_DIR", "_build"), ("LIB", "libss_scan.so"), ("MARSHAL", "_marshal.so")):
        monkeypatch.setattr(build, name, str(tmp_path / path))
    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "_check_device_code", lambda directory: None)
    return ran, fail, tmp_path


def test_module_after_library(commands):
    ran, _, path = commands
    assert build.build_library() == str(path / "libss_scan.so")
    assert (path / "libss_scan.so").exists() and (path / "_marshal.so").exists()
    linked = [i for i, c in enumerate(ran) if c[c.index("-o") + 1].endswith("libss_scan.so")]
    assert len(linked) == 1 and all(("ss_marshal" in " ".join(c)) == (i > linked[0]) for i, c in enumerate(ran) if i != linked[0])


@pytest.mark.parametrize("what", ["torch", "the Python headers", "g++"])
def test_library_without_what_the_module_needs(commands, monkeypatch, capsys, what):
    ran, _, path = commands
    (path / "_marshal.so").write_text("of an earlier build")
    if what == "torch":
        monkeypatch.setitem(sys.modules, "torch.utils", None)
    elif what == "g++":
        which = build.shutil.which
        monkeypatch.setattr(build.shutil, "which", lambda name: None if name == "g++" else which(name))
    else:
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(path)})
    assert build.build_library() == str(path / "libss_scan.so")
    assert (path / "libss_scan.so").exists() and not (path / "_marshal.so").exists()
    assert what in capsys.readouterr().out and not any(c[0] == "g++" for c in ran)


def test_library_where_the_module_does_not_compile(commands):
    _, fail, path = commands
    fail.append(True)
    with pytest.raises(RuntimeError):
        build.build_library()
    assert (path / "libss_scan.so").exists() and not (path / "_marshal.so").exists()


def test_binding_without_the_module():
    code = ("import sys, warnings; sys.modules['paper_2312_00752_amd._marshal'] = None; from paper_2312_00752_amd import binding as B\n"
            "with warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always')\n"
            "    m = B._marshal(); B._marshal()\n"
            "print(len(w), [getattr(m, n)(1, 2) for n in ('step', 'layer_step', 'scan_fwd', 'scan_bwd', 'layer_fwd', 'layer_bwd')])")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert r.stdout.strip() == "1 " + str([None] * 6)
