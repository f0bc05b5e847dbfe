"""The distribution of work items over workgroups (xcd_pair_item in
csrc/common.hpp): every (pair, rank) item is given to exactly one workgroup of
the launch, each pair's items stay in its group of XCDs, and an XCD's share of
a pair starts with that pair's first items.  Host code, run on the CPU."""
import math
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_19242_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("items") / "work_items_harness")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-x", "hip", "-I", CSRC,
                    os.path.join(HERE, "work_items_harness.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def test_every_item_goes_to_one_workgroup(harness):
    cases = [(nbk, T, il) for nbk in (1, 2, 3, 4, 6, 7, 8, 12, 16, 20, 24) for T in (1, 2, 5, 8, 33, 100)
             for il in (0, 1)]
    inp = "".join(f"{a} {b} {c}\n" for a, b, c in cases)
    lines = subprocess.run([harness], input=inp, capture_output=True, text=True, check=True).stdout.split("\n")
    for (nbk, T, il), line in zip(cases, lines):
        n, *items = line.split()
        assert int(n) == len(items) and int(n) >= nbk * T
        got = [(wg % 8, *map(int, x.split(","))) for wg, x in enumerate(items) if x != "-"]
        assert sorted((p, r) for _, p, r in got) == [(p, r) for p in range(nbk) for r in range(T)], (nbk, T, il)
        g = math.gcd(nbk, 8)
        for xcd, p, r in got:
            assert xcd // (8 // g) == p // (nbk // g), (nbk, T, il)
        # the ranks an XCD gets of a pair are spread over the pair's range
        for p in range(nbk):
            for xcd in {x for x, q, _ in got if q == p}:
                mine = sorted(r for x, q, r in got if q == p and x == xcd)
                assert mine[0] < 8 and all(b - a <= 8 for a, b in zip(mine, mine[1:])), (nbk, T, il, p, xcd)
