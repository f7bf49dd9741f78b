"""Launch shapes of the run-time-length passes: every line length the library takes, with few
and with many lines, against the limits of the kernels behind them.  The shapes come from the
built library; a small program compiled for the host asks for them (no GPU)."""
import os
import subprocess

import pytest

from paper_1601_04640_amd import binding, build_lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not os.path.exists(build_lib.HIPCC), reason="needs hipcc")
def test_every_accepted_length_has_launchable_shapes(tmp_path):
    binding.load()  # fails loudly if the library is not built
    obj, exe = str(tmp_path / "shapes.o"), str(tmp_path / "shapes")
    where, name = os.path.split(build_lib.LIB)
    for cmd in (
            [build_lib.HIPCC, *build_lib.FLAGS, "--offload-host-only", "-O1", "-c",
             "-I", os.path.join(ROOT, "paper_1601_04640_amd", "csrc"),
             os.path.join(ROOT, "tests", "host", "shapes_main.hip"), "-o", obj],
            [build_lib.HIPCC, obj, f"-L{where}", f"-l:{name}", f"-Wl,-rpath,{where}", "-o", exe]):
        b = subprocess.run(cmd, capture_output=True, text=True)
        assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("ok "), r.stdout
