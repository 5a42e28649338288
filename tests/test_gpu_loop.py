"""The resident loop against the launch-per-step form, bit for bit.

A registration runs in one launch where its source's units (16 wave records of
64 / lanes queries) fit the device's blocks; with kernel timing on it runs one
search, fold and solve launch per step.  Both have the same arithmetic in the
same order, so poses, RMSE, counters and correspondences are equal without a
tolerance.  Sources: one, a few and just over a unit's queries, the last unit
a single query, units past one gather (256) and past the blocks of the device
(two units a block), and past what the loop takes; batches with empty pairs,
one-unit pairs and larger ones; queries without a local candidate; the stop
rule; and degenerate sums, where the loop hands over."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched, prof_enable, prof_reset  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def both(g, p, ms, K, **kw):
    """register() as one launch, and as one launch per step."""
    one = g.register(dev(p), K, m_per_pair=ms, correspondences=True, **kw)
    prof_enable(True)
    try:
        step = g.register(dev(p), K, m_per_pair=ms, correspondences=True, **kw)
    finally:
        prof_enable(False)
        prof_reset()
    return one, step


def same(a, b):
    assert np.array_equal(a.Rt, b.Rt) and np.array_equal(a.iters, b.iters)
    assert np.array_equal(a.degenerate, b.degenerate) and a.status == b.status
    for x, y in ((a.rmse, b.rmse), (a.fallbacks, b.fallbacks), (a.candidates, b.candidates),
                 (a.dilated_lookups, b.dilated_lookups)):
        assert all(np.array_equal(u, v) for u, v in zip(x, y))
    assert torch.equal(a.nn_idx, b.nn_idx) and torch.equal(a.nn_d2.view(torch.int32), b.nn_d2.view(torch.int32))


def cloud(rng, n, m, spread=0.02):
    """A bumpy surface, and moved samples of it (some far off, in no voxel's reach)."""
    u = rng.uniform(0, 1, (2, n))
    q = np.stack([u[0], u[1], 0.2 * np.sin(7 * u[0]) * np.cos(5 * u[1])])
    p = q[:, rng.integers(0, n, m)] + rng.normal(0, spread / 4, (3, m))
    far = rng.random(m) < 0.02
    p[:, far] += rng.normal(0, 0.3, (3, int(far.sum())))
    a = 0.02
    R = np.array([[np.cos(a), -np.sin(a), 0], [np.sin(a), np.cos(a), 0], [0, 0, 1]])
    return q.astype(np.float32), (R @ p + np.array([[0.004], [-0.003], [0.006]])).astype(np.float32)


def unit(lanes):
    return 16 * 64 // lanes


SINGLE = [(lanes, units, extra) for lanes in (1, 2, 4, 8) for units, extra in ((0, 1), (0, 63), (1, 0), (1, 1), (5, -1))]
SINGLE += [(8, 256, 0), (8, 256, 1), (8, 300, 17), (8, 512, 0), (8, 513, 0), (1, 257, -3)]


@pytest.mark.parametrize("lanes,units,extra", SINGLE)
def test_units_of_one_pair(lanes, units, extra):
    m = unit(lanes) * units + extra
    q, p = cloud(np.random.default_rng(m + lanes), 20000, m)
    g = build_grid_batched(dev(q), [q.shape[1]], [0.03], 2).dilate(2)
    for sort in (True, False):
        g.set_schedule(256, lanes, sort, 64)
        for early in (False, True):
            same(*both(g, p, [m], 6, early_stop=early, rmse_eps=1e-4))


@pytest.mark.parametrize("lanes", [1, 4, 8])
@pytest.mark.parametrize("ms", [(0, 1, 0), (700, 0, 64, 1025, 40000), (300,) * 40 + (90000,), (20000,) * 20])
def test_batches(lanes, ms):
    rng = np.random.default_rng(len(ms) + lanes)
    qs, ps = zip(*(cloud(rng, 3000, m) for m in ms))
    g = build_grid_batched(dev(np.concatenate(qs, 1)), [3000] * len(ms), [0.05] * len(ms), 2).dilate(2)
    g.set_schedule(128, lanes, lanes != 4, 64)
    for early in (False, True):
        same(*both(g, np.concatenate(ps, 1), list(ms), 8, early_stop=early, rmse_eps=1e-4))


@pytest.mark.parametrize("kind", ["one_place", "line", "plane", "turned"])
@pytest.mark.parametrize("m", [3, 5000])
def test_sums_that_do_not_pin_the_rotation(kind, m):
    rng = np.random.default_rng(m)
    q, _ = cloud(rng, 4000, 10)
    p = rng.uniform(0.2, 0.8, (3, m)).astype(np.float32)
    if kind == "one_place":
        p[:] = np.array([[0.5], [0.4], [0.0]])
    elif kind == "line":
        p[1:] = 0.4
    elif kind == "plane":
        p[2] = 0.0
        q[2] = 0.0
    else:
        p = (1.0 - q[:, rng.integers(0, 4000, m)]).astype(np.float32)
    g = build_grid_batched(dev(q), [4000], [0.05], 2).dilate(2)
    same(*both(g, p, [m], 5))
    same(*both(g, p, [m], 5, Rt0=np.array([-1.0, 0, 0, 0, -1, 0, 0, 0, 1, 1, 1, 0])))


def test_calls_that_follow_one_another():
    """Messages of an earlier call, with other sizes, are never taken for this one's."""
    rng = np.random.default_rng(3)
    q, p = cloud(rng, 20000, 30000)
    g = build_grid_batched(dev(q), [20000], [0.03], 2).dilate(2)
    for m, lanes, K in ((30000, 4, 7), (30000, 8, 1), (500, 4, 9), (30000, 1, 3), (0, 4, 2), (129, 8, 4)):
        g.set_schedule(256, lanes, True, 64)
        same(*both(g, p[:, :m], [m], K))
