"""The plan of cut dK/dV walks (csrc/split_plan.hpp) against every form of call:
the partial sums of two chunks or tiles never share a row, all lie inside the
workspace that the size query asks for, whatever the ranges into which the keys
are divided, and the chunks of a walk do not depend on that division.  Host
code, run on the CPU; the walks are counted as the kernels count them."""
import os
import random
import re
import shutil
import subprocess

import pytest

import paper_2609_19242_amd as bd
from tests.asm_listing import kernel_resources, listing
from paper_2609_19242_amd import CLEAN, CORRUPTED

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2609_19242_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("split") / "split_harness")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-x", "hip", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "split_harness.cpp"), "-o", exe],
                   check=True, capture_output=True)

    def run(calls):
        inp = ""
        for c in calls:
            head = (c["batch"], c["L"], c["M"], c["H"], c["KV"], c["D"], c["f32"], c["intra"], c["hilo"], c["window"],
                    len(c["table"]), *c["table"])
            flat = lambda rs: " ".join([str(len(rs))] + [f"{s} {p} {n}" for s, p, n in rs])  # noqa: E731
            inp += " ".join(map(str, head)) + f" {flat(c['q'])} {flat(c['k'])}\n"
        lines = iter(subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout.split("\n"))
        out = []
        for c in calls:
            keys = ("unit", "rows", "tiles", "counts_bytes", "bytes", "stats", "wgs_per_cu")
            r = dict(zip(keys, map(int, next(lines).split())), ranges=[])
            for s, pos0, n in c["k"]:
                head, *tiles = next(lines).split(" | ")
                ch, nt = map(int, head.split())
                assert len(tiles) == nt
                r["ranges"].append((s, pos0, n, ch, [tuple(map(int, t.split())) for t in tiles]))
            out.append(r)
        return out

    return run


def tile_rows(c):
    return 16 if c["f32"] else 128


def divide(rng, lo, hi, n):
    """[lo, hi) as n consecutive ranges, some empty or short."""
    cuts = sorted(rng.choice([rng.randint(lo, hi), lo + rng.randrange(1, 40)]) for _ in range(n - 1))
    ends = [lo] + [min(x, hi) for x in cuts] + [hi]
    return [(a, b - a) for a, b in zip(ends, ends[1:])]


def draw(rng):
    f32 = rng.random() < 0.3
    M = rng.randint(1, 130)
    L = M * max(1, int(2 ** rng.uniform(5, 10.5 if f32 else 13)) // M)
    H, KV = rng.choice([(4, 2), (16, 16), (24, 8), (32, 8), (32, 4), (12, 2), (56, 8), (3, 1), (2, 2)])
    window = rng.choice([0, 0, 0, rng.randint(1, 2000)])
    table = sorted(rng.randint(0, L) for _ in range(L // M)) if rng.random() < 0.2 else []
    q = [(CORRUPTED, 0, L), (CLEAN, 0, L)]
    kind = rng.random()
    if kind < 0.35:
        a = rng.randint(0, L)
        q = [(rng.choice([CLEAN, CORRUPTED]), a, rng.randint(0, L - a))]
    elif kind < 0.5:
        q = [(rng.choice([CLEAN, CORRUPTED]), p, n) for p, n in divide(rng, 0, L, rng.randint(2, 4))]
    return dict(batch=rng.choice([1, 1, 2, 3]), L=L, M=M, H=H, KV=KV, D=rng.choice([64, 128]), f32=int(f32),
                intra=rng.randint(0, 1), hilo=rng.choice([0, 0, 15, 7]), window=window, table=table, q=q,
                k=[(CORRUPTED, 0, L), (CLEAN, 0, L)])


def check(c, r):
    pairs = c["batch"] * c["KV"]
    row_bytes = 2 * c["D"] * (8 if c["f32"] else 4)
    used, tiles = [], 0
    for s, pos0, n, ch, walks in r["ranges"]:
        tiles += len(walks) if ch > 1 else 0
        for t, (steps, nch, *rows) in enumerate(walks):
            assert nch == (max(1, -(-steps // r["unit"])) if ch > 1 else 1), (c, t)
            assert ch > 1 or r["rows"] == 0 or steps <= r["unit"], c
            nk = min(tile_rows(c), n - t * tile_rows(c))
            used += [(x, x + nk) for x in rows]
    assert tiles == r["tiles"]
    if not tiles:
        return
    used.sort()
    assert used == [] or (used[0][0] >= 0 and used[-1][1] <= r["rows"]), c
    assert all(a[1] <= b[0] for a, b in zip(used, used[1:])), c
    assert 4 * tiles * pairs <= r["counts_bytes"]
    assert r["counts_bytes"] + r["rows"] * pairs * row_bytes <= r["bytes"], c
    assert r["stats"] + r["bytes"] <= bd.NOALLOC_SCRATCH_BYTES, c


def test_partial_sums_stay_apart_and_inside(harness):
    rng = random.Random(3)
    calls = []
    for _ in range(1500):
        c = draw(rng)
        calls.append(c)
        for _ in range(2):
            n = rng.randint(1, 31)
            sub = [(CLEAN, p, m) for p, m in divide(rng, 0, c["L"], n)] + \
                  [(CORRUPTED, p, m) for p, m in divide(rng, 0, c["L"], rng.randint(1, 32 - n))]
            rng.shuffle(sub)
            calls.append(dict(c, k=sub[:rng.randint(1, len(sub))]))
    res = harness(calls)
    for c, r in zip(calls, res):
        check(c, r)
    assert sum(r["tiles"] > 0 for r in res) > 1000
    for i in range(0, len(calls), 3):  # the same problem and queries: the same chunks and the same workspace
        assert len({(r["unit"], r["bytes"]) for r in res[i:i + 3]}) == 1


def test_ragged_shards_are_cut_like_whole_streams(harness):
    """Eight shards of 380 rows, four of 528 and four of 816: none of them a multiple of 128."""
    for L, M, H, KV, D, shards in [(2660, 20, 56, 8, 128, 7), (2112, 16, 16, 16, 64, 4), (3264, 16, 24, 8, 128, 4)]:
        n, cut = L // shards, 0
        base = dict(batch=1, L=L, M=M, H=H, KV=KV, D=D, f32=0, intra=0, hilo=0, window=0, table=[],
                    q=[(CORRUPTED, 0, n)])
        for rank in range(shards):
            c = dict(base, q=[(CORRUPTED, rank * n, n)])
            whole, parts = harness([dict(c, k=[(CORRUPTED, rank * n, n), (CLEAN, 0, L)]),
                                    dict(c, k=[(CORRUPTED, rank * n, n)] + [(CLEAN, s * n, n) for s in range(shards)])])
            check(c, whole)
            check(c, parts)
            assert (whole["tiles"] > 0) == (parts["tiles"] > 0) == (whole["unit"] > 0), (L, rank)
            cut += whole["tiles"] > 0
        assert cut > 0, L


def test_overlapping_ranges_stay_whole(harness):
    c = dict(batch=1, L=2040, M=24, H=32, KV=8, D=128, f32=0, intra=0, hilo=0, window=0, table=[],
             q=[(CORRUPTED, 0, 2040), (CLEAN, 0, 2040)])
    twice, once = harness([dict(c, k=[(CLEAN, 0, 1000), (CLEAN, 999, 1041)]),
                           dict(c, k=[(CLEAN, 0, 1000), (CORRUPTED, 999, 1041), (CLEAN, 1000, 0), (CLEAN, 1000, 40)])])
    assert once["tiles"] > 0 and twice["tiles"] == 0 and all(ch == 1 for *_, ch, _ in twice["ranges"])


def test_the_size_query_holds_the_plan(harness):
    if not os.path.exists(bd.library_path):
        pytest.skip("library not built")
    rng = random.Random(5)
    calls = [dict(draw(rng), table=[]) for _ in range(200)]
    for c, r in zip(calls, harness(calls)):
        p = bd.make_problem(c["batch"], c["L"], c["M"], c["H"], c["KV"], c["D"], bd.F32 if c["f32"] else bd.BF16,
                            clean_intra=c["intra"], hilo=c["hilo"], window=c["window"])
        n = bd.attn_bwd_workspace_bytes(p, [bd.Range(*x) for x in c["q"]])
        assert n == r["stats"] + (r["bytes"] if r["unit"] else 0), c


def test_workgroups_per_cu_are_those_of_the_kernels(harness):
    """The planner's side-by-side workgroups against the registers and LDS of the kernels as built."""
    text = listing("bwd_dkdv.hip")
    if text is None:
        pytest.skip("hipcc not available")
    seen = 0
    for name, res in kernel_resources(text).items():
        m = re.search(r"dkdv_kernelILi(\d+)ELb(\d)ELb(\d)E", name)
        if not m:
            continue
        D, adaptive, rows = (int(x) for x in m.groups())
        waves_per_simd = 512 // (-(-res["vgpr_count"] // 8) * 8)  # a workgroup has one wave on each SIMD
        held = min(waves_per_simd, 160 * 1024 // res["group_segment_fixed_size"])
        c = dict(batch=1, L=256, M=16, H=3 if rows else 2, KV=1, D=D, f32=0, intra=0, hilo=15 if adaptive else 0,
                 window=0, table=[], q=[(CLEAN, 0, 256)], k=[(CLEAN, 0, 256)])
        assert harness([c])[0]["wgs_per_cu"] == held, (name, res)
        seen += 1
    assert seen == 8
