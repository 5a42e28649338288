"""The autotuner and the resident loop: a loop that gives up while it is timed has
not run its iterations, so it must not win (a query without a finite distance
ends it in its first step), and the block size and candidate loop are tuned for
the launches also where the loop applies, and no load is timed that a grid
cannot have.  A registration under the chosen
schedule takes at most 1.6 times the best of all schedules."""
import time

import numpy as np
import pytest

from paper_2512_04996_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import FORM_HANDED_OVER, FORM_LOOP, FORM_STEPS  # noqa: E402
from paper_2512_04996_amd.api import autotune_cache_clear, build_grid, build_grid_fixed, prof_enable, prof_read, prof_reset  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def grid(n):
    P = synth.config("paper_room_226k")
    rng = np.random.default_rng(n)
    q = P.q[:, rng.permutation(P.q.shape[1])[:n]]
    p = P.p[:, rng.permutation(P.p.shape[1])[:n * 9 // 10]].copy()
    return build_grid_fixed(dev(q), P.meta["grid_origin"], P.voxel, P.meta["grid_dims"], P.rings).dilate(P.rings), p


def test_a_loop_that_gives_up_does_not_win():
    g, p = grid(60000)
    p[0, 100] = 3e19          # finite; its squared distances are not
    P = dev(p)

    def best():
        t = []
        for _ in range(4):
            t0 = time.perf_counter()
            g.register(P, 1)
            t.append(time.perf_counter() - t0)
        return min(t)

    autotune_cache_clear()
    g.autotune(P, searches_per_plan=30)
    chosen, tuned = g.schedule, best()
    assert g.last_form in (FORM_HANDED_OVER, FORM_STEPS)
    swept = []
    for block in (128, 256):
        for lanes in (1, 2, 4, 8):
            for mode in (0, 1):
                g.set_schedule(block, lanes, True, 128, mode)
                swept.append((best(), block, lanes, mode))
    assert tuned < 1.6 * min(swept)[0], (chosen, tuned, sorted(swept)[:4])


def test_no_listed_queries_are_timed_where_none_are_listed():
    # a fine grid lists no query with a finite distance: tuning a large source
    # takes some 90 registrations' time; with a listed load it took 1100
    P = synth.room_pair(seed=8, n=700000, m=600000, voxel=0.03, rings=2, iters=30)
    g = build_grid(dev(P.q), P.voxel, P.rings).dilate(P.rings)
    p = dev(P.p)
    autotune_cache_clear()
    t0 = time.perf_counter()
    g.autotune(p, searches_per_plan=30)
    tuning = time.perf_counter() - t0
    once = []
    for _ in range(4):
        t0 = time.perf_counter()
        g.register(p, 30)
        once.append(time.perf_counter() - t0)
    assert tuning < 300 * min(once), (tuning, once)


def test_the_launches_are_tuned_where_the_loop_applies():
    g, p = grid(20000)
    P = dev(p)
    autotune_cache_clear()
    g.autotune(P, searches_per_plan=30)
    chosen = g.schedule
    g.register(P, 5)
    assert g.last_form == FORM_LOOP

    def search_ms():
        prof_reset()
        prof_enable(True)
        try:
            for _ in range(3):
                g.register(P, 8, use_graph=False)
            n, ms = prof_read("nns_local")
        finally:
            prof_enable(False)
            prof_reset()
        return ms / n

    tuned = search_ms()
    swept = []
    for block in (128, 256, 512):
        for mode in (0, 1):
            g.set_schedule(block, chosen["lanes_per_query"], chosen["sort_source"], 128, mode)
            swept.append((search_ms(), block, mode))
    assert tuned < 1.25 * min(swept)[0], (chosen, tuned, sorted(swept))
