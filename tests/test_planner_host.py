"""The planner on the CPU, for every unit shape: the XCD-aware search finds
the cut of least cost, planning a call's work costs less than the call, and
jobs and batches take the kernel measured fastest at their sizes."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SQUARE, WIDE, NARROW, TILE, REGION = range(5)
OVERHEAD = {SQUARE: 8, WIDE: 16, NARROW: 8, TILE: 24, REGION: 40}


@pytest.fixture(scope="module")
def P(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("planner") / "libplanner_host.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "paper_2005_09481_amd", "csrc"),
                    os.path.join(ROOT, "tests", "planner_host.cpp"),
                    os.path.join(ROOT, "paper_2005_09481_amd", "csrc", "xeng_plan.cpp"), "-o", out],
                   check=True, capture_output=True)
    L = ctypes.CDLL(out)
    i32, i64, p32, p64 = ctypes.c_int32, ctypes.c_int64, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int64)
    L.host_plan.restype = i64
    L.host_plan.argtypes = [p32, p64, i32, i32, i32, i32, i32, i64, p64, i64]
    L.host_choose.argtypes = [i32, i64, i32, i32, p32]
    L.host_choose_batch.argtypes = [p32, p64, i32, i32]
    L.host_plan_us.restype = ctypes.c_double
    L.host_plan_us.argtypes = [i32, i64, i32, i32, i32]
    return L


def plan(P, jobs, wgs, shape, min_stages=4, xcd=False, cap=0):
    """Rows (job, i, j, t0, t1, atomic, workgroup), or None."""
    n = (ctypes.c_int32 * len(jobs))(*[j[0] for j in jobs])
    t = (ctypes.c_int64 * len(jobs))(*[j[1] for j in jobs])
    args = (n, t, len(jobs), wgs, min_stages, shape, int(xcd), cap)
    count = P.host_plan(*args, None, 0)
    if count < 0:
        return None
    out = np.zeros((max(count, 1), 7), dtype=np.int64)
    assert P.host_plan(*args, out.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), count) == count
    return out[:count]


def units_of(n, shape):
    nt, nr = -(-n // 128), -(-n // 64)
    if shape == NARROW:
        return [(0, 0)]
    if shape == REGION:
        return [(i, j) for i in range(nr) for j in range(i, nr)]
    if shape == WIDE:
        return [(i, j) for i in range(nt) for j in range(i // 2, (nt + 1) // 2)]
    return [(i, j) for i in range(nt) for j in range(i, nt)]


def stage_cost(i, j, n, shape):
    """Sixteenths of a stage: 13 for a wide window with one tile outside the triangle."""
    nt = -(-n // 128)
    return 13 if shape == WIDE and (i <= 2 * j < nt) != (i <= 2 * j + 1 < nt) else 16


def workgroup_costs(pieces, n, shape):
    cost = {}
    for _, i, j, t0, t1, _, w in pieces.tolist():
        cost[w] = cost.get(w, 0) + -(-(t1 - t0) // 64) * stage_cost(i, j, n, shape) + 16 * OVERHEAD[shape]
    return cost


def tails_fit(tails, wgs, budget, ovh):
    """Whether the tails (stage cost, stages) fill at most `wgs` workgroups of `budget`, in order."""
    k, left = 0, budget
    for wc, r in tails:
        while r > 0:
            if left - ovh < wc:
                k, left = k + 1, budget
                if k >= wgs:
                    return False
            take = min(r, (left - ovh) // wc)
            r, left = r - take, left - take * wc - ovh
    return True


def least_cost(n, t, wgs, shape):
    """The smallest largest workgroup cost of any cut into segments and tails."""
    ns, ovh = -(-t // 64), OVERHEAD[shape]
    order = sorted(units_of(n, shape), key=lambda u: sum(((u[0] >> k) & 1) << (2 * k + 1) |
                                                         (((2 if shape == WIDE else 1) * u[1] >> k) & 1) << (2 * k)
                                                         for k in range(16)))
    wc = [stage_cost(i, j, n, shape) for i, j in order]
    mean = -(-ns * sum(wc) // (16 * wgs))
    best = None
    for L in range(max(32, mean - ovh), min(mean + 4 * ovh, 1023, ns - 1) + 1):
        seg = [min(ns, 1023, max(1, L * 16 // c)) for c in wc]
        full = [ns // s for s in seg]
        tails = [(c, ns - f * s) for c, f, s in zip(wc, full, seg) if ns > f * s]
        rest = wgs - sum(full)
        if rest < 0 or (tails and rest == 0):
            continue
        cost = max(s * c + 16 * ovh for s, c in zip(seg, wc))
        if tails:
            lo, hi = 16 * ovh + 16, 16 * ovh * len(tails) + sum(c * r for c, r in tails)
            while lo < hi:
                mid = (lo + hi) // 2
                if tails_fit(tails, rest, mid, 16 * ovh):
                    hi = mid
                else:
                    lo = mid + 1
            cost = max(cost, lo)
        best = cost if best is None else min(best, cost)
    return best


@pytest.mark.parametrize("n,t,wgs,shape", [
    (512, 30000, 256, REGION), (300, 32768, 240, REGION), (768, 12000, 256, REGION), (1024, 5000, 256, REGION),
    (768, 65536, 256, TILE), (1000, 32768, 256, TILE), (2048, 5000, 256, TILE), (1100, 20000, 128, TILE),
    (2048, 32768, 256, WIDE), (2000, 9000, 256, WIDE), (1536, 30000, 256, WIDE), (1000, 32768, 512, SQUARE),
])
def test_xcd_search_finds_the_least_cost(P, n, t, wgs, shape):
    pieces = plan(P, [(n, t)], wgs, shape, xcd=True)
    want = least_cost(n, t, wgs, shape)
    if want is None:
        assert pieces is None
    else:
        # (a unit's last stage may be partial: it costs a whole one)
        assert max(workgroup_costs(pieces, n, shape).values()) == want


@pytest.mark.parametrize("n,t,shape", [(512, 30000, REGION), (1024, 12000, REGION), (1536, 30000, TILE),
                                       (2048, 5000, TILE), (2048, 30000, WIDE), (3072, 65536, WIDE)])
def test_planning_takes_less_than_the_call(P, n, t, shape):
    # a call with new sizes plans its work on the host first; these take 20 to
    # 100 us where the calls themselves take 30 us and more
    assert P.host_plan_us(n, t, 256, shape, 30) < 400


@pytest.mark.parametrize("n,t,shape", [(3840, 4096, WIDE), (1408, 8192, REGION), (1408, 49152, REGION),
                                       (2816, 8192, TILE), (1296, 4096, REGION), (2048, 32768, WIDE),
                                       (1024, 16384, REGION), (1000, 32768, TILE)])
def test_xcd_plan_is_never_far_behind_the_linear_one(P, n, t, shape):
    # with few workgroups left for the tails of many units it would be: the
    # linear order is then taken
    pieces, linear = plan(P, [(n, t)], 256, shape, xcd=True), plan(P, [(n, t)], 256, shape)
    if pieces is not None:
        cost, want = workgroup_costs(pieces, n, shape), workgroup_costs(linear, n, shape)
        assert max(cost.values()) <= max(want.values()) + 16 * OVERHEAD[shape]


def choose(P, n, t, cus=256, min_stages=4):
    wgs = ctypes.c_int32()
    return P.host_choose(n, t, cus, min_stages, ctypes.byref(wgs)), wgs.value


@pytest.mark.parametrize("n,t,shape,wgs", [
    # measured on both sides of each line (see choose_dma)
    (512, 8192, REGION, 0), (1024, 16384, REGION, 0), (1024, 49152, TILE, 0), (1536, 256, TILE, 78), (1536, 2048, REGION, 0),
    (1408, 4096, REGION, 253), (1408, 8192, REGION, 253), (1408, 16384, REGION, 253), (1408, 49152, TILE, 0),
    (2048, 512, TILE, 136), (2048, 1536, TILE, 136), (2048, 2048, TILE, 136), (2048, 16384, TILE, 0),
    (2048, 32768, WIDE, 0), (3072, 512, WIDE, 156), (3072, 20000, WIDE, 0),
    (4096, 1, WIDE, 0), (4096, 64, WIDE, 0), (4096, 1024, TILE, 0), (4096, 4096, TILE, 0), (4096, 20000, WIDE, 0),
    (5008, 64, WIDE, 0), (5008, 512, WIDE, 0), (5008, 20000, WIDE, 0), (6000, 2048, WIDE, 0), (6000, 12000, WIDE, 0),
    (8192, 64, WIDE, 0), (8192, 12000, WIDE, 0),
])
def test_single_jobs_take_the_measured_kernel(P, n, t, shape, wgs):
    assert choose(P, n, t) == (shape, wgs)


def test_minimum_piece_length_limits_cuts_not_the_kernels(P):
    # a job of more units than compute units is never left to one kernel alone
    for min_stages in (1, 4, 64, 1 << 20):
        assert choose(P, 4096, 64, min_stages=min_stages)[0] == WIDE
        assert choose(P, 2048, 512, min_stages=min_stages) == (TILE, 136)


@pytest.mark.parametrize("jobs,n,t,shape", [(4, 512, 3000, REGION), (4, 512, 20000, TILE), (16, 256, 3000, REGION),
                                            (16, 256, 12000, TILE), (16, 256, 32768, TILE), (2, 640, 12000, REGION),
                                            (2, 640, 32768, TILE), (8, 1024, 4096, TILE), (8, 2048, 4096, WIDE)])
def test_batches_take_the_measured_kernel(P, jobs, n, t, shape):
    assert P.host_choose_batch((ctypes.c_int32 * jobs)(*[n] * jobs), (ctypes.c_int64 * jobs)(*[t] * jobs), jobs,
                               256) == shape


def assert_covers_once(pieces, jobs, shape, wgs, cap=0, gaps=False):
    """Every unit x sample of every job once, in runs of whole stages of at
    most `cap` (by default the longest for which the kernel's int32 sums stay
    exact); shared units, and only those, flushed with atomics; the workgroups
    in order from 0, without gaps but in XCD plans (where some places on the
    last XCD stay empty)."""
    cap = cap or (16383 if shape == SQUARE else 1023)
    runs = {}
    for job, i, j, t0, t1, atomic, _ in pieces.tolist():
        runs.setdefault((job, i, j), []).append((t0, t1, atomic))
    assert set(runs) == {(k, i, j) for k, (n, t) in enumerate(jobs) if t > 0 for i, j in units_of(n, shape)}
    for (job, _, _), r in runs.items():
        r.sort()
        assert [a for a, _, _ in r] + [jobs[job][1]] == [0] + [b for _, b, _ in r]
        assert all(a % 64 == 0 and 0 < b - a <= 64 * cap for a, b, _ in r)
        assert all(atomic == (len(r) > 1) for _, _, atomic in r)
    assert np.all(np.diff(pieces[:, 6]) >= 0) and pieces[0, 6] >= 0 and pieces[-1, 6] < wgs
    assert gaps or pieces[-1, 6] + 1 == len(set(pieces[:, 6].tolist()))


SHAPES = [SQUARE, WIDE, NARROW, TILE, REGION]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("seed", range(6))
def test_plans_cover_every_unit_once(P, shape, seed):
    rng = np.random.default_rng(100 * seed + shape)
    for _ in range(25):
        # batches with empty jobs among them, on whole chips and on a few units
        jobs = [(int(rng.integers(1, 65 if shape == NARROW else 1500)), int(rng.choice([0, 1, 63, 64, 65, rng.integers(1, 9000)])))
                for _ in range(int(rng.integers(1, 7)))]
        if not any(t for _, t in jobs):
            continue
        wgs, min_stages, cap = int(rng.choice([8, 240, 256, 512])), int(rng.choice([1, 4, 32])), int(rng.choice([0, 0, 5, 100]))
        pieces = plan(P, jobs, wgs, shape, min_stages, cap=cap)
        assert_covers_once(pieces, jobs, shape, wgs, cap)


@pytest.mark.parametrize("shape", SHAPES)
def test_long_jobs_stay_below_the_piece_limit(P, shape):
    # one unit's samples past the longest piece, on one workgroup and on all
    for t in (64 * 1023, 64 * 1023 + 1, 64 * 3000 - 7):
        for wgs in (1, 256):
            assert_covers_once(plan(P, [(64, t)], wgs, shape), [(64, t)], shape, wgs)


@pytest.mark.parametrize("shape", [SQUARE, WIDE, TILE, REGION])
@pytest.mark.parametrize("seed", range(4))
def test_xcd_plans_cover_every_unit_once(P, shape, seed):
    rng = np.random.default_rng(1000 + 10 * seed + shape)
    found = 0
    for _ in range(40):
        job = (int(rng.integers(65, 3000)), int(rng.integers(2000, 70000)))
        wgs, cap = int(rng.choice([64, 240, 256, 512])), int(rng.choice([0, 0, 200]))
        pieces = plan(P, [job], wgs, shape, xcd=True, cap=cap)
        if pieces is not None:
            found += 1
            assert_covers_once(pieces, [job], shape, wgs, cap, gaps=True)
    assert found
