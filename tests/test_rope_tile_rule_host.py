"""The tile that carries the rotation of Q and K in the forward, over the sizes of layers: what the rule takes is costed as it
goes out.  No GPU: the planning functions of the library run on the host."""
import os
import shutil
import subprocess

import pytest

from paper_2510_16415_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_a_rotating_launch_is_never_much_longer_than_one_without(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not os.path.exists(build.LIB):
        pytest.skip("needs hipcc and the built library")
    exe = str(tmp_path / "rule")
    r = subprocess.run([hipcc, "-x", "hip", *build.FLAGS[:1], "--offload-host-only", "-O1", "-std=c++17", "-I", build.CSRC,
                        os.path.join(HERE, "rope_tile_rule.cpp"), "-x", "none", build.LIB, "-Wl,-rpath," + build.LIBDIR,
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    rows = [line.split() for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()]
    assert len(rows) == 2 * 32 * 29
    # the allowance for the rotation's own launch is 6 us
    late = [r for r in rows if float(r[4]) > float(r[5]) + 6.01]
    assert not late, f"{len(late)} of {len(rows)}: {late[:5]}"
    assert {int(r[3]) for r in rows} >= {-1, 0, 1}      # a launch of its own, 256 x 256 and 128 x 128 tiles are all taken
