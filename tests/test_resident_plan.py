"""Brick plans of resident solves, checked on the host (tests/native/resident_check.cpp).

* every LDS row that a thread of a finite-difference brick reads lies in its brick's box, for the threads
  without nodes too;
* the problems of resident_forms take the kernel variants that they are there for.
"""

import math
import os
import random
import subprocess

import pytest

from tests.resident_forms import STEPS, VARIANTS, variant

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_07780_amd", "csrc")
CUS = 256


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("resident") / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "resident_check.cpp"), os.path.join(CSRC, "resident.cpp"),
                    "-o", exe, "-lpthread"], check=True)

    def run(problems):
        text = "\n".join(" ".join(str(int(v)) for v in p) for p in problems)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        rows = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
        assert len(rows) == len(problems)
        return rows

    return run


def _random_problems(n):
    rng = random.Random(2508)
    out = [(CUS, 25, 25, 25, 8, 8, 8, 8, 8, 8, 300, 63, 3, a, r) for a, r in ((0, 0), (1, 0), (1, 1))]
    while len(out) < n:
        size = [int(math.exp(rng.uniform(math.log(5), math.log(110)))) for _ in range(3)]
        cells = [rng.randint(2, s - 3) for s in size]
        lo = [rng.randint(1, s - 2 - c) for s, c in zip(size, cells)]
        adj = rng.randrange(2)
        out.append((CUS, *size, *lo, *cells, rng.randint(4, 40), rng.randrange(1, 64), rng.randrange(64), adj,
                    adj and rng.randrange(2)))
    return out


def test_rows_stay_in_the_brick(check):
    problems = _random_problems(300)
    rows = check(problems)
    assert sum(r[0] > 0 for r in rows) > 200
    for p, r in zip(problems, rows):
        assert r[4] == 0, (p, r)


def test_forms_take_every_variant(check):
    problems = []
    for n, lo, cells, det, damp, ck, *_ in VARIANTS.values():
        for adj in (0, 1):
            problems.append((CUS, *n, *lo, *cells, STEPS, det, damp, adj, adj and ck < STEPS))
    rows = check(problems)
    seen = set()
    for i, (name, form) in enumerate(VARIANTS.items()):
        for adj in (0, 1):
            r = rows[2 * i + adj]
            assert r[0] and variant(r[1], r[2]) == form[7 + adj], (name, adj, r)
            rec = adj and form[5] < STEPS
            seen |= {("run", adj, rec, form[7 + adj][0]), ("fem", adj, rec, form[7 + adj][1])}
    # the adjoint with recompute holds more per node: its cuts have two planes per thread nowhere
    assert seen >= {("run", 0, 0, k) for k in (2, 4, 8, 12)} | {("run", 1, False, k) for k in (2, 4, 8, 12)}
    assert seen >= {("run", 1, True, k) for k in (4, 8, 12)}
    assert seen >= {("fem", a, r, k) for a, r in ((0, 0), (1, False), (1, True)) for k in (1, 2, 3)}
