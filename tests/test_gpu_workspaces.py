"""A grid whose workspaces are laid out again in place (another voxel count,
source size or number of iterations) gives what a fresh grid gives, bit for
bit: shapes that grow, shrink by more than four times and come back, pairs of
a batch that swap their shapes (the total stays), sources that grow and
shrink, more iterations than before, the exhaustive search's words in between,
and the single steps (rebuild, dilate, register, nns) as the joined call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def clouds(rng, ns, ms, scales):
    q = [rng.uniform(0, 1, (3, n)) * np.array([[1.0], [s], [0.3]]) for n, s in zip(ns, scales)]
    p = [x[:, rng.integers(0, x.shape[1], m)] + rng.normal(0, 0.02, (3, m)) for x, m in zip(q, ms)]
    return dev(np.concatenate(q, 1)), dev(np.concatenate(p, 1))


@pytest.mark.parametrize("joined", [True, False])
@pytest.mark.parametrize("ns", [(4000,), (3000, 1500)])
def test_layouts_in_turn(joined, ns):
    rng = np.random.default_rng(len(ns) + joined)
    B = len(ns)
    steps = [((1.0, 3.0), (500, 700), 5), ((3.0, 1.0), (500, 700), 5), ((40.0, 20.0), (500, 700), 5),
             ((0.2, 0.3), (500, 700), 5), ((1.0, 3.0), (9000, 0), 5), ((2.0, 2.5), (9000, 0), 40),
             ((2.0, 2.5), (60, 90), 3), ((1.0, 3.0), (500, 700), 5)]
    g = None
    for scales, ms, K in steps:
        ms = [max(m, 1) for m in ms[:B]] if B == 1 else list(ms)
        q, p = clouds(rng, ns, ms, scales)
        if g is None:
            g = build_grid_batched(q, list(ns), [0.05] * B, 2).dilate(2)
        kw = dict(m_per_pair=ms, correspondences=True)
        if joined:
            res = g.rebuild_register(q, 2, p, K, **kw)
        else:
            g.rebuild(q).dilate(2)
            res = g.register(p, K, **kw)
        fresh = build_grid_batched(q, list(ns), [0.05] * B, 2).dilate(2)
        ref = fresh.register(p, K, **kw)
        pose = np.tile(IDENT, B)
        for got, want in ((res, ref), (g.register(p, 2, global_only=True, **kw),
                                       fresh.register(p, 2, global_only=True, **kw)),
                          (g.register(p, K, early_stop=True, use_graph=False, **kw),
                           fresh.register(p, K, early_stop=True, use_graph=False, **kw))):
            assert np.array_equal(got.Rt, want.Rt) and np.array_equal(got.iters, want.iters)
            assert all(np.array_equal(a, b) for a, b in zip(got.rmse, want.rmse))
            assert torch.equal(got.nn_idx, want.nn_idx) and torch.equal(got.nn_d2, want.nn_d2)
        for a, b in zip(g.nns(p, pose, m_per_pair=ms), fresh.nns(p, pose, m_per_pair=ms)):
            assert torch.equal(a, b)
        for b in range(B):
            for a, w in zip(g.export(b), fresh.export(b)):
                assert np.array_equal(np.asarray(a), np.asarray(w))
        fresh.free()
