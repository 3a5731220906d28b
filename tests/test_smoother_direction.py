"""The multigrid smoother keeps its Chebyshev direction as a vector: it is not
formed again from the iterates, whose rounding would then enter it (CPU;
smoother_direction.cpp runs the device code's own functions on the host)."""
import os
import shutil
import subprocess

import pytest

from paper_2603_07038_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(not shutil.which(B.HIPCC) and not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_direction_does_not_carry_the_rounding_of_the_iterate(tmp_path):
    obj, exe = str(tmp_path / "smoother_direction.o"), str(tmp_path / "smoother_direction")
    for cmd in ([f for f in B.FLAGS if f != "-O3"] + ["-O1", "-x", "hip", "-c",
                 os.path.join(HERE, "smoother_direction.cpp"), "-o", obj],
                ["--offload-arch=gfx950", obj, B.LIB, "-Wl,-rpath," + B.HERE, "-o", exe]):
        r = subprocess.run([B.HIPCC] + cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    rows = [x.split() for x in r.stdout.splitlines()]
    assert len(rows) == 8
    for row in rows:
        assert row[-2:] == ["0", "0"], row
