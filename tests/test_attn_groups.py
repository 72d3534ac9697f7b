"""The cut of a batch into workgroups of the resident attention kernel (csrc/attn_groups.h): host arithmetic, compiled here."""
import ctypes
import subprocess
import time

import numpy as np
import pytest

from paper_2511_12934_amd import build

CSRC = build.CSRC
TILE, LOAD = 4, 6


# the same search by bisection in 64-bit integers, what the plan's time is measured against
BISECTION = """
#include <algorithm>
#include <cstdint>
static int bisection(int n, const int32_t *t, const int32_t *k, int cu, int m, int32_t *g)
{
    long cost = 0;
    for (int i = 0; i < n; ++i) cost += (long)t[i] * (k[i] + %d);
    auto count = [&](long w) {
        int sum = 0;
        for (int i = 0; i < n; ++i) {
            const long room = std::max(w - %dL * k[i], 1L);
            g[i] = (int)std::min(((long)t[i] * (k[i] + %d) + room - 1) / room, ((long)t[i] + m - 1) / m);
            sum += g[i];
        }
        return sum;
    };
    long lo = std::max(cost / cu, 1L), hi = lo;
    while (count(hi) > cu) lo = hi, hi += hi / 2 + %d;
    while (hi - lo > 1 + hi / 64) {
        const long mid = (lo + hi) / 2;
        (count(mid) > cu ? lo : hi) = mid;
    }
    return count(hi);
}
""" % (TILE, LOAD, TILE, LOAD)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_groups")
    (d / "plan.cpp").write_text(BISECTION + '#include "attn_groups.h"\n'
                                'static_assert(aif::GROUP_TILE == %d && aif::GROUP_LOAD == %d, "");\n' % (TILE, LOAD) +
                                'extern "C" int plan(int n, const int32_t *t, const int32_t *k, int cu, int m, int32_t *g)\n'
                                '{ return aif::plan_group_counts(n, t, k, cu, m, g); }\n'
                                'extern "C" void plans(int n, const int32_t *t, const int32_t *k, int cu, int m, int32_t *g)\n'
                                '{ for (int i = 0; i < 20; ++i) aif::plan_group_counts(n, t, k, cu, m, g); }\n'
                                'extern "C" void bisections(int n, const int32_t *t, const int32_t *k, int cu, int m, int32_t *g)\n'
                                '{ for (int i = 0; i < 20; ++i) bisection(n, t, k, cu, m, g); }\n'
                                'extern "C" int user_tiles(int n, const int32_t *t, int cu, int dh)\n'
                                '{ return aif::groups_min_tiles(n, t, aif::GROUP_MIN_TILES, aif::user_fine_groups(cu, dh)); }\n')
    so = str(d / "plan.so")
    subprocess.check_call([build.HIPCC, "-x", "c++", "-O3", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", so])
    lib = ctypes.CDLL(so)
    f = lib.plan
    f.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]

    def run(tiles, keys, n_cu, min_tiles):
        t, k = np.asarray(tiles, np.int32), np.asarray(keys, np.int32)
        g = np.full(t.size, -1, np.int32)
        return f(t.size, t.ctypes.data, k.ctypes.data, n_cu, min_tiles, g.ctypes.data), g.astype(np.int64)
    run.plans, run.bisections, run.user_tiles = lib.plans, lib.bisections, lib.user_tiles
    return run


def best_groups(tiles, keys, n_cu, min_tiles):
    """The smallest whole cost w for which one group a unit is enough, by bisection in exact integers, and the groups it gives."""
    t, k = tiles.astype(object), keys.astype(object)

    def groups(w):
        return [min(-(-a * (b + TILE) // max(w - LOAD * b, 1)), -(-a // min_tiles)) for a, b in zip(t, k)]
    lo, hi = 0, int(max(a * (b + TILE) + LOAD * b for a, b in zip(t, k)))
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if sum(groups(mid)) > n_cu else (lo, mid)
    return hi, np.array(groups(hi), np.float64)


@pytest.mark.parametrize("longest", [1, 5, 40, 700, 70_000, 1 << 26])       # tiles; the last is a list of 2^31 candidates
@pytest.mark.parametrize("min_tiles", [4, 12])
def test_groups_are_within_bounds_and_of_like_cost(plan, longest, min_tiles):
    rng = np.random.default_rng(longest + min_tiles)
    for n in (1, 2, 15, 16, 63, 128, 255, 256):
        for n_cu in (256, max(n, 104), n):
            for _ in range(4):
                tiles = np.maximum(1, (longest * rng.random(n) ** rng.choice([0.0, 1.0, 3.0])).astype(np.int64))
                keys = rng.integers(0, 39, n)
                total, g = plan(tiles, keys, n_cu, min_tiles)
                assert total == g.sum() <= n_cu and g.min() >= 1
                assert np.all(g <= -(-tiles // min_tiles))
                # The costliest group (tiles in proportion).  Where min_tiles bounds a request's groups they are the best
                # plan's; the others cost at most the w that the search ended with, and its bracket, which the least w lies in, is
                # 1 + w / 64 wide (and 2^-20 for the sums in floats).
                def worst(groups):
                    return float(np.max(tiles * (keys + TILE) / groups + LOAD * keys))
                w, best = best_groups(tiles, keys, n_cu, min_tiles)
                assert worst(g) <= max(worst(best), (w + 1) * 64 / 63) * (1 + 2.0 ** -20), (n, n_cu)


def test_the_host_waits_little_for_the_plan(plan):
    """256 requests: the search is on the way to the first launch.  The integer bisection takes five to seven times as long as the
    plan; a third of its time is allowed, both in turn in the same process."""
    r = np.arange(256)
    tiles = np.ascontiguousarray((10_000 - 7_500 * ((r * 0.618) % 1.0)) / 32, np.int32)
    keys, g = np.ascontiguousarray(16 - r % 10, np.int32), np.zeros(256, np.int32)
    args = [256, *(ctypes.c_void_p(a.ctypes.data) for a in (tiles, keys)), 256, 4, ctypes.c_void_p(g.ctypes.data)]
    best = {}
    for _ in range(200):
        for name in ("plans", "bisections"):
            f = getattr(plan, name)
            t0 = time.perf_counter()
            f(*args)
            best[name] = min(best.get(name, 1e9), time.perf_counter() - t0)
    assert best["plans"] < best["bisections"] / 3, best


@pytest.mark.parametrize("d_head, users, tiles, want", [(64, 8, 16, 4), (64, 40, 16, 4), (64, 41, 16, 12), (64, 64, 16, 12), (64, 160, 1, 4), (64, 161, 1, 12),
                                                        (64, 53, 9, 4), (64, 54, 9, 12), (32, 64, 16, 4), (32, 65, 16, 12)])
def test_user_network_cuts_into_fours_while_they_are_few(plan, d_head, users, tiles, want):
    t = np.full(users, tiles, np.int32)
    assert plan.user_tiles(users, ctypes.c_void_p(t.ctypes.data), 256, d_head) == want
