"""The native half of the binding: one file per interpreter and torch, whole when it appears, built by the command that builds the
library; and a library that is there loads without it and without a compiler."""
import os
import subprocess
import sys

import pytest

from paper_2301_00391_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_file_of_this_interpreter_and_torch(monkeypatch):
    import torch
    mine = build.host_path()
    assert mine.endswith(".so") and sys.implementation.cache_tag in os.path.basename(mine) and not set("+ ") & set(os.path.basename(mine))
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    assert build.host_path() != mine
    monkeypatch.undo()
    assert build.host_path() == mine


@pytest.mark.parametrize("fails", [False, True])
def test_whole_when_it_appears(monkeypatch, tmp_path, fails):
    path = tmp_path / "half.so"
    path.write_bytes(b"before")

    def compiler(cmd, check):
        with open(cmd[cmd.index("-o") + 1], "wb") as part:
            part.write(b"some")
            part.flush()
            assert path.read_bytes() == b"before"
            if fails:
                raise subprocess.CalledProcessError(1, cmd)

    monkeypatch.setattr(subprocess, "run", compiler)
    if fails:
        with pytest.raises(subprocess.CalledProcessError):
            build.build_host(output=str(path))
    else:
        build.build_host(output=str(path))
    assert [p.name for p in tmp_path.iterdir()] == ["half.so"] and path.read_bytes() == (b"before" if fails else b"some")


@pytest.mark.parametrize("args,built", [([], ["library", "half"]), (["-v"], ["library", "half"]), (["-o", "elsewhere.so"], ["library"]),
                                        (["-D", "PIPAD_AGG_DEPTH=2"], ["library"])])
def test_command_line_builds_both(monkeypatch, args, built):
    seen = []
    monkeypatch.setattr(build, "build", lambda **_: seen.append("library"))
    monkeypatch.setattr(build, "build_host", lambda **_: seen.append("half"))
    build.main(args)
    assert seen == built


def test_a_library_loads_without_it(tmp_path):
    """Another torch (so no file for it), nothing on the path that compiles."""
    binding.load_library()
    code = """if True:
        import torch, warnings
        torch.__version__ = "0.0.other"
        import paper_2301_00391_amd as pipad
        from paper_2301_00391_amd import binding
        with warnings.catch_warnings(record=True) as seen:
            warnings.simplefilter("always")
            lib = pipad.load_library()
        assert binding._host is None and [w.category for w in seen] == [RuntimeWarning], seen
        assert lib.pipad_strerror(0) == b"ok" and pipad.get_option("agg_nt") >= 0
        """
    env = {**os.environ, "PATH": str(tmp_path), "PIPAD_LIBRARY": binding.LIB_PATH}
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    assert not [f for f in os.listdir(os.path.dirname(binding.LIB_PATH)) if "0.0.other" in f]
