"""GPU parity of the exact global search on the occupancy pyramid (a 64-ary
tree of 4 x 4 x 4 cells over the voxels): grids whose axes end at, one before
and one past whole cells of each level (4, 16, 64 voxels), grids of at most
4^3 voxels (no pyramid), flat and line-shaped grids, rows with more points
than a lane scans alone, and queries near, far and outside.  Indices, float32
distances and global-search counts equal the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched, build_grid_fixed  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)
DIMS = [(1, 1, 1), (4, 4, 4), (5, 4, 3), (16, 16, 16), (17, 15, 16), (63, 64, 65), (257, 1, 1), (1, 300, 2),
        (70, 5, 66), (1030, 3, 1)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def clouds(seed, dims, n, m, lumps):
    """Targets in clusters of a few voxels (most voxels stay empty), queries over the grid and around it."""
    rng = np.random.default_rng(seed)
    D = np.array(dims, np.float64)
    c = rng.uniform(0, 1, (lumps, 3)) * D
    q = c[rng.integers(0, lumps, n)] + rng.normal(0, 0.3, (n, 3))
    q = np.clip(q, 0.01, D - 0.01)
    p = np.concatenate([rng.uniform(-0.1, 1.1, (m // 2, 3)) * D, q[rng.integers(0, n, m - m // 2)] +
                        rng.normal(0, 3.0, (m - m // 2, 3))])
    p[:8] = np.array([(i & 1, (i >> 1) & 1, i >> 2) for i in range(8)]) * D * 3 - D   # far corners
    return q.T.astype(np.float32), p.T.astype(np.float32)


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("rings,n,lumps", [(0, 3000, 5), (2, 700, 40)])
def test_every_depth_and_edge(dims, rings, n, lumps):
    q, p = clouds(sum(dims) + rings, dims, n, 1500, lumps)
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 1.0, dims, rings).dilate(rings)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 1.0, dims), rings)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    for lanes in (1, 4):
        g.set_schedule(128, lanes, lanes == 4, 64)
        idx, d2, fb = g.nns(dev(p), IDENT)
        assert int(fb.cpu()[0]) == rF
        assert np.array_equal(idx.cpu().numpy(), ridx)
        assert np.array_equal(d2.cpu().numpy().view(np.uint32), rd2.view(np.uint32))
    assert rF > 0


def test_every_pair_of_a_batch_has_its_own_pyramid():
    rng = np.random.default_rng(5)
    qs = [rng.uniform(0, s, (3, n)).astype(np.float32) for s, n in ((1.0, 50), (9.0, 900), (40.0, 3000))]
    ps = [(q[:, rng.integers(0, q.shape[1], 700)] + rng.normal(0, 2.0, (3, 700))).astype(np.float32) for q in qs]
    g = build_grid_batched(dev(np.concatenate(qs, 1)), [q.shape[1] for q in qs], [0.5, 0.4, 0.7], 1).dilate(1)
    idx, d2, fb = g.nns(dev(np.concatenate(ps, 1)), np.tile(IDENT, 3), m_per_pair=[700] * 3)
    idx, d2 = idx.cpu().numpy().reshape(3, 700), d2.cpu().numpy().reshape(3, 700)
    for b, (q, p, v) in enumerate(zip(qs, ps, (0.5, 0.4, 0.7))):
        og = oracle.dilate(oracle.build_grid(q, v, 1), 1)
        ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
        assert rF > 0 and int(fb.cpu()[b]) == rF
        assert np.array_equal(idx[b], ridx) and np.array_equal(d2[b].view(np.uint32), rd2.view(np.uint32))
