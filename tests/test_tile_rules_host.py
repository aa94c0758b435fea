"""What the model of the GEMM tiles chooses, over the sizes of layers and against times measured on the chip.  No GPU: the
planning functions of the library run on the host."""
import os
import shutil
import subprocess

import pytest

from paper_2510_16415_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
GRAD, SWIGLU_BWD, STORE = 2, 4, 0
K_TILE = 5


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not os.path.exists(build.LIB):
        pytest.skip("needs hipcc and the built library")
    exe = str(tmp_path_factory.mktemp("rules") / "tile_rules")
    r = subprocess.run([hipcc, "-x", "hip", *build.FLAGS[:1], "--offload-host-only", "-O1", "-std=c++17", "-I", build.CSRC,
                        os.path.join(HERE, "tile_rules.cpp"), "-x", "none", build.LIB, "-Wl,-rpath," + build.LIBDIR,
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return lambda *a: [line.split() for line in subprocess.run([exe, *(str(int(x)) if not isinstance(x, str) else x for x in a)],
                                                               capture_output=True, text=True, check=True).stdout.splitlines()]


def test_the_tile_that_rotates_is_costed_as_it_goes_out(rules):
    """The shortest of those that can, and where it is no more than the allowance of 6 us behind the best whole tiles."""
    rows = rules("rope")
    assert len(rows) == 2 * 32 * 29
    wrong = [r for r in rows if (int(r[3]) >= 0) != (float(r[4]) <= float(r[6]) + 6) or float(r[5]) > float(r[4])]
    assert not wrong, f"{len(wrong)} of {len(rows)}: {wrong[:5]}"
    assert {int(r[3]) for r in rows} >= {-1, 0, 1}      # a launch of its own, 256 x 256 and 128 x 128 tiles are all taken


# (epilogue, second operand K-contiguous, M, N, K): us measured on the 192-row tile, and on 256 x 256 tiles, last round cut up
@pytest.mark.parametrize("epi,bkc,M,N,K,k_tile,large", [(SWIGLU_BWD, 1, 3584, 7168, 4096, 467, 360),
                                                        (SWIGLU_BWD, 1, 4352, 6144, 3072, 348, 293),
                                                        (SWIGLU_BWD, 1, 4864, 5888, 5120, 579, 508),
                                                        (STORE, 0, 6656, 7936, 3072, 343, 295)])
def test_rounds_of_the_192_row_tile(rules, epi, bkc, M, N, K, k_tile, large):
    """More than four rounds of them: the last one counts in full, like the first ones.  The model is good to 20 %."""
    k, l, _, taken = map(float, rules("cost", epi, 1, bkc, 1, M, N, K, 0)[0])
    assert abs(k / k_tile - 1) <= 0.2 and abs(l / large - 1) <= 0.2
    assert int(taken) != K_TILE


# us of three expansions [f x d] of rank r with a whole last round and with one that is cut up, measured
@pytest.mark.parametrize("f,d,r,f32,whole,cut", [(11008, 4096, 1024, 1, 296, 318), (8192, 3072, 384, 1, 96, 118),
                                                 (4352, 3072, 512, 1, 79, 86), (2560, 5120, 1024, 1, 109, 114),
                                                 (5461, 2048, 512, 1, 66.6, 62.7), (5461, 2048, 512, 0, 61.5, 52),
                                                 (1792, 4096, 1024, 0, 61, 57), (6144, 4096, 256, 0, 79, 85)])
def test_the_last_round_of_short_gradients(rules, f, d, r, f32, whole, cut):
    saved = float(rules("cost", GRAD, 1, 1, 3, f, d, r, f32)[0][2])
    assert (saved > 0) == (cut < whole)
