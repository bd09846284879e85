"""Order of resident launches on several streams (tests/native/resident_order_check.cpp): whatever the streams, sizes
and times, the launches that run together have at most a block per CU, and small ones do not wait for each other."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("order") / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_07780_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "resident_order_check.cpp"), "-o", exe], check=True)
    return lambda *a: [int(v) for v in subprocess.run([exe, *map(str, a)], capture_output=True, text=True,
                                                      check=True).stdout.split()]


@pytest.mark.parametrize("streams", [1, 2, 3, 8, 31, 32, 33, 60])
@pytest.mark.parametrize("most", [256, 130, 60])
def test_never_more_blocks_than_places(check, streams, most):
    worst, free_runs, launches = check(streams, most)
    assert worst <= 256
    if streams * most <= 256:
        assert free_runs == launches
