"""Global searches among crowded voxels (hundreds to thousands of points each),
whose first cube the tree search drops and whose voxels it takes nearest first:
correspondences against the oracle bit for bit, from queries one voxel off, far
inside the grid and outside it, with targets at equal distances; in the
correspondence search, the launch-per-step search and the resident loop; a wave
whose queries use up its budget and go to the exhaustive search; and the
overflowed blocks of the direct layout, whose time is bounded by a multiple of
the segmented layout's."""
import time

import numpy as np
import pytest

import oracle
from paper_2512_04996_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import FORM_STEPS  # noqa: E402
from paper_2512_04996_amd.api import build_grid_fixed, prof_enable, prof_reset  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def clouds(dims, counts, m, copies, seed):
    """Voxels of the given counts scattered over the grid, one in each corner brick first."""
    rng = np.random.default_rng(seed)
    D = np.array(dims)
    vox = np.stack([rng.integers(0, d, len(counts)) for d in D])
    q = np.concatenate([v[:, None] + rng.uniform(0.01, 0.99, (3, c)) for v, c in zip(vox.T, counts)], 1)
    q = q[:, rng.permutation(q.shape[1])]
    if copies:
        q[:, ::3] = q[:, 1::3][:, :1]
        q[:, 1::7] = np.floor(q[:, 1::7]) + 0.5     # many targets at each of a few places
    near = q[:, rng.integers(0, q.shape[1], m)] + rng.choice([-1.3, 1.3, 0.0, 2.2], (3, m))
    far = rng.uniform(-0.6, 1.6, (3, m)) * D[:, None]
    p = np.where(rng.random(m) < 0.5, near, far)
    return q.astype(np.float32), p.astype(np.float32)


def registered(g, p, step, **kw):
    prof_enable(step)   # with timing on: one launch per step
    try:
        return g.register(p, 1, correspondences=True, **kw)
    finally:
        prof_enable(False)
        prof_reset()


@pytest.mark.parametrize("dims", [(3, 4, 4), (16, 16, 16), (70, 5, 9)])
@pytest.mark.parametrize("counts", [(380, 385, 390), (700,) * 12, (3000, 1, 5, 2000, 97, 96), (20000, 900, 400)])
@pytest.mark.parametrize("copies", [False, True])
def test_crowded_voxels_far_and_near(dims, counts, copies):
    q, p = clouds(dims, counts, 2000, copies, sum(counts) + dims[0])
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 1.0, dims, 1).dilate(0)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 1.0, dims), 0)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    assert rF > 100
    P = dev(p)
    for lanes in (1, 4, 8):
        g.set_schedule(128, lanes, lanes == 4, 64)
        idx, d2, fb = g.nns(P, IDENT)
        got = [(idx, d2, int(fb.cpu()[0]))]
        for step in (False, True):
            r = registered(g, P, step)
            got.append((r.nn_idx, r.nn_d2, int(r.fallbacks[0][0])))
        for i, d, f in got:
            assert np.array_equal(i.cpu().numpy(), ridx), lanes
            assert np.array_equal(d.cpu().numpy().view(np.uint32), rd2.view(np.uint32)) and f == rF


def test_a_wave_past_its_budget_lists_its_queries():
    rng = np.random.default_rng(2)
    n, m = 300000, 640     # 64 queries of a wave, each with 300,000 points to look at
    q = np.concatenate([rng.uniform(3.01, 3.99, (3, n)), rng.uniform(0.1, 15.9, (3, 50))], 1).astype(np.float32)
    p = (rng.uniform(-0.2, 0.2, (3, m)) + np.array([[3.5], [3.5], [7.0]])).astype(np.float32)
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 1.0, (16, 16, 16), 1).dilate(0)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 1.0, (16, 16, 16)), 0)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    for lanes in (1, 8):
        g.set_schedule(128, lanes, False, 64)
        runs = [registered(g, dev(p), step) for step in (False, True)]
        for r in runs:
            assert np.array_equal(r.nn_idx.cpu().numpy(), ridx) and int(r.fallbacks[0][0]) == rF
            assert np.array_equal(r.nn_d2.cpu().numpy().view(np.uint32), rd2.view(np.uint32))
        # the listed queries' moments are added after the others': the last bits differ
        np.testing.assert_allclose(runs[0].Rt, runs[1].Rt, rtol=0, atol=1e-10)
        np.testing.assert_allclose(runs[0].rmse[0], runs[1].rmse[0], rtol=1e-12)


def test_few_far_queries_of_a_large_source_are_listed():
    rng = np.random.default_rng(9)
    n, m = 120000, 140000     # more queries than the resident loop takes at four lanes
    q = rng.uniform(0, 4, (3, n)).astype(np.float32)
    p = q[:, rng.integers(0, n, m)] + rng.normal(0, 0.01, (3, m))
    p[2, 5000:5100] += 9.0
    p = p.astype(np.float32)
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 0.5, (8, 8, 8), 1).dilate(1)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 0.5, (8, 8, 8)), 1)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    for lanes in (4, 8):
        g.set_schedule(128, lanes, True, 64)
        r = g.register(dev(p), 1, correspondences=True)
        assert g.last_form == FORM_STEPS and int(r.fallbacks[0][0]) == rF
        assert np.array_equal(r.nn_idx.cpu().numpy(), ridx)
        assert np.array_equal(r.nn_d2.cpu().numpy().view(np.uint32), rd2.view(np.uint32))
        runs = [g.register(dev(p), 5) for _ in range(3)]
        assert all(np.array_equal(x.Rt, runs[0].Rt) for x in runs)


def test_overflowed_blocks_cost_a_bounded_multiple():
    P = synth.config("paper_room_226k")
    g = build_grid_fixed(dev(P.q), P.meta["grid_origin"], P.voxel, P.meta["grid_dims"], P.rings).dilate(P.rings)
    g.build_direct(65536)
    p = dev(P.p)

    def best(**kw):
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            r = g.register(p, 10, **kw)
            t.append(time.perf_counter() - t0)
        return min(t), r

    seg, _ = best()
    direct, r = best(layout="direct")
    g.free_direct()
    assert r.fallbacks[0][0] > 5000
    # measured 6 (60 when a wave scanned a cube of voxels for each query)
    assert direct < 20 * seg, (direct, seg)
