"""What a build makes and what the binding can be loaded with: the library is enough, and the native calls are used only
beside the library, the torch and the Python that they were built for."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

from paper_2106_10796_amd import binding as B, build


@pytest.fixture(scope="module", autouse=True)
def built():
    build.ensure_built()


def _package(tmp_path, with_calls):
    """A copy of the package's Python files with the library, and the native calls or not."""
    pkg = tmp_path / "paper_2106_10796_amd"
    pkg.mkdir()
    for name in ("__init__.py", "binding.py", "libcdsgd.so"):
        shutil.copy(os.path.join(build.PKG, name), pkg / name)
    if with_calls is not None:
        (pkg / "_calls.so").write_bytes(with_calls)
    return tmp_path


def _run(where, code):
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(code)], cwd=where, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout.split()


USE = """
    import torch
    from paper_2106_10796_amd import binding as B
    B._stream = lambda: 0                                                # (no GPU is needed here)
    try:
        B.StaticLayerList([], None, 1).step(0, 1, 4, 0.5, 0.1, 0.1)      # the first call of a program
    except B.CdsgdError as e:
        print(e.status)
    print(B.cdsgd_cost_period_mean(1.0, 16.0, 2.0, 0.5, 4)["t_cd"] > 0)
    try:
        B.cdsgd_quantize_pack(torch.zeros(4), torch.zeros(4), torch.zeros(1, dtype=torch.int32), 0.5)
    except TypeError as e:
        print("contiguous" in str(e))
    print(type(B._native()).__name__)
"""


def _calls_bytes():
    with open(build.CALLS, "rb") as fh:
        return fh.read()


def test_the_native_calls_are_used(tmp_path):
    assert _run(_package(tmp_path, _calls_bytes()), USE) == [str(B.ERR_SIZE), "True", "True", "module"]


def test_without_the_native_calls(tmp_path):
    assert _run(_package(tmp_path, None), USE) == [str(B.ERR_SIZE), "True", "True", "_Declines"]


@pytest.mark.parametrize("part", range(3))
def test_native_calls_made_for_something_else_are_left_alone(tmp_path, part):
    ours = build.calls_for(build.built_id())[part].encode() + b"\0"
    data = _calls_bytes()
    assert ours in data
    other = ours[:-2] + bytes([ours[-2] ^ 1]) + b"\0"
    assert _run(_package(tmp_path, data.replace(ours, other)), USE) == [str(B.ERR_SIZE), "True", "True", "_Declines"]


@pytest.fixture
def dry(tmp_path, monkeypatch):
    """The default places in a folder of their own, and compilers that only write their output's name."""
    ran = []

    def run(cmd, **_):
        out = cmd[cmd.index("-o") + 1]
        ran.append(os.path.basename(out).split(".")[0])
        broken = ran[-1] in dry_run.broken
        if not broken:
            with open(out, "wb") as fh:
                fh.write(" ".join(cmd).encode())
        return subprocess.CompletedProcess(cmd, int(broken), "no such header" if broken else "")

    class dry_run:
        broken = ()
        made = ran
    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(build, "hipcc_path", lambda: "hipcc")
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libcdsgd.so"))
    monkeypatch.setattr(build, "CALLS", str(tmp_path / "_calls.so"))
    monkeypatch.setattr(build.build, "__defaults__", ((), build.LIB, False))
    return dry_run


def test_build_makes_the_library_and_the_native_calls(dry):
    build.build()
    assert dry.made == ["libcdsgd", "_calls"]
    del dry.made[:]
    build.build(extra_flags=("-DX=1",))
    with open(build.CALLS) as fh:
        assert build.source_id(("-DX=1",)) in fh.read()          # built for the library that is beside them
    del dry.made[:]
    build.build(out=build.LIB + ".variant")
    assert dry.made == ["libcdsgd"]


def test_a_library_without_the_native_calls_is_a_build(dry, capsys):
    dry.broken = ("_calls",)
    build.build()
    assert os.path.exists(build.LIB) and not os.path.exists(build.CALLS)
    assert "no such header" in capsys.readouterr().err
    dry.broken = ("libcdsgd",)
    with pytest.raises(RuntimeError, match="no such header"):
        build.build()


def test_the_library_does_not_depend_on_the_marshalling(tmp_path, monkeypatch):
    csrc = tmp_path / "csrc"
    shutil.copytree(os.path.dirname(build.SRC), csrc)
    for name in ("SRC", "SRC_CALLS"):
        monkeypatch.setattr(build, name, str(csrc / os.path.basename(getattr(build, name))))
    monkeypatch.setattr(build, "SRC_HOST", [str(csrc / os.path.basename(p)) for p in build.SRC_HOST])
    library, calls = build.source_id(), build.calls_id()
    with open(build.SRC_CALLS, "a") as fh:
        fh.write("// changed\n")
    assert build.source_id() == library and build.calls_id() != calls
    calls = build.calls_id()
    with open(build.SRC, "a") as fh:
        fh.write("// changed\n")
    assert build.source_id() != library and build.calls_id() != calls
