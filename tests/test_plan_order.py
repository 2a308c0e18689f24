"""CPU: the prefill's XCD-aware order at several XCD counts, through a small
C++ harness built with g++ against the library's planning header."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "order_harness.cpp")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("order") / "order_harness")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", SRC, "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("xcds", [1, 4, 6, 8])
def test_order_covers_every_item_once(harness, xcds):
    res = subprocess.run([harness, str(xcds)], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout + res.stderr
