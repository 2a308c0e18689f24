"""CPU: the launch planning (decode partition and workspace slots, the
prefill's XCD-aware work order, the automatic key-split count) at several
machine shapes, through a small C++ harness built with g++ against the
library's planning header."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "plan_harness.cpp")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_harness")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", SRC, "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("cus,xcds", [(32, 4), (64, 8), (256, 8), (256, 1), (80, 1)])
def test_partition_arithmetic(harness, cus, xcds):
    res = subprocess.run([harness, str(cus), str(xcds)], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout + res.stderr


# The decodes that the GPU tests of the two routes run (tests/test_gpu_decode_routes.py),
# (KV heads, head_dim, contexts), at the CU count of the part they run on.
EDGES = [1, 16, 17, 31, 32, 33, 64, 225, 255, 256]
LONG = [8233 - 17 * (i % 5 == 0) for i in range(32)]
DIRECT = [(8, 128, EDGES), (4, 128, EDGES), (1, 64, EDGES), (5, 64, EDGES), (8, 64, LONG)]
UNEVEN = [(4, 128, np.random.default_rng(73 + n).integers(lo, hi + 1, n))
          for n, lo, hi in ((1, 3000, 3000), (80, 1, 900), (40, 100, 4000))]


@pytest.mark.parametrize("fp8", [False, True])
def test_routes_of_the_decodes_tested_on_the_gpu(harness, fp8):
    for want, cases in (("direct", DIRECT), ("partition", UNEVEN)):
        for hkv, d, ctx in cases:
            seg = (16 if d == 64 else 12) if fp8 else 8
            res = subprocess.run([harness, "route", "256", str(seg), str(hkv), *map(str, ctx)], capture_output=True,
                                 text=True, check=True)
            assert res.stdout.strip() == want, (hkv, d, list(ctx))
