"""The rule that spreads a mixture population over waves and lanes
(paper_1306_5583_amd/csrc/smc_gmm_split.hpp), compiled for the host: what it
may return at all, and that the shapes of the GPU tests take the forms that
those tests mean to reach."""
import os
import random
import shutil
import subprocess

import pytest

from gpu_helpers import DRAW_SHAPES, UNSLICED

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("split") / "gmm_split")
    subprocess.run([gxx, "-std=c++17", "-O1", "-o", exe,
                    os.path.join(HERE, "support", "gmm_split.cpp")], check=True)

    def run(rows):
        text = "".join("%d %d %d %s\n" % r for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return run


def test_bounds_of_the_split(split):
    rng = random.Random(5)
    rows = [(int(2 ** rng.uniform(0, 24)), int(2 ** rng.uniform(0, 16)), rng.randint(1, 16),
             rng.choice(["step", "init", "loglik"])) for _ in range(4000)]
    rows += [(1, 1, 1, "step"), (1 << 17, 10000, 4, "step"), ((1 << 17) + 1, 10000, 4, "step")]
    for (n, nd, K, what), (W, lsl) in zip(rows, split(rows)):
        assert W in (1, 2, 4, 8) and 0 <= lsl <= 6
        if lsl:  # every lane of a particle has a point
            assert W == 4 and n <= 1 << 17 and W << lsl <= nd
        elif W > 1 and W != 4:
            assert nd >= 32 * W


def test_shapes_of_the_gpu_tests(split):
    n, nd = UNSLICED
    rows = [(n, nd, K, what) for K in range(1, 17) for what in ("loglik", "step", "init")]
    assert split(rows) == [(4, 0)] * len(rows)


def test_shapes_of_the_draws(split):
    rows = [(n, nd, K, "step") for n, nd, K, _ in DRAW_SHAPES]
    assert split(rows) == [(W, 0) for _, _, _, W in DRAW_SHAPES]
