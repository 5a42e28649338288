"""Crowded voxels: the scan of a whole wave (8 lanes a query) against the
oracle's correspondences and the query-by-query scan, bit for bit.  Voxels of
one below, at and one past the count it starts from (64), its four loads (256)
and several rounds; targets that occur several times (equal distances, where
it hands over); waves whose queries look into one voxel and into many (source
order), some beside voxels of a few points or with no candidate at all; in the
launch-per-step search and in the resident loop."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_fixed, prof_enable, prof_reset  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("counts", [(63, 64, 65, 3), (255, 256, 257, 1), (191, 1, 64, 320), (511, 513, 1300, 6),
                                    (5000, 7, 63, 70)])
@pytest.mark.parametrize("copies", [False, True])
@pytest.mark.parametrize("m", [1, 8, 999, 20000])
def test_crowded_voxels(counts, copies, m):
    rng = np.random.default_rng(sum(counts) + m)
    cell = rng.permutation(27)[:len(counts)]
    q = np.concatenate([np.array([[v % 3], [v // 3 % 3], [v // 9]]) + rng.uniform(0.01, 0.99, (3, c))
                        for v, c in zip(cell, counts)], 1).astype(np.float32)
    q = q[:, rng.permutation(q.shape[1])]
    if copies:
        q[:, ::2] = q[:, 1::2][:, :q[:, ::2].shape[1]] if q.shape[1] % 2 == 0 else q[:, ::2]
        q[:, :: 5] = q[:, :1]
    p = (q[:, rng.integers(0, q.shape[1], m)] + rng.normal(0, 0.05, (3, m))).astype(np.float32)
    p[:, ::17] = rng.uniform(-1, 4, (3, len(range(0, m, 17))))
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 1.0, (3, 3, 3), 1).dilate(1)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 1.0, (3, 3, 3)), 1)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    res = []
    for sort in (True, False):
        for step, mode in ((True, 0), (True, 1), (False, 1)):
            g.set_schedule(128, 8, sort, 64, search_mode=mode)
            prof_enable(step)   # with timing on: one launch per step
            try:
                one = g.register(dev(p), 1, correspondences=True)
                res.append((sort, g.register(dev(p), 4)))
            finally:
                prof_enable(False)
                prof_reset()
            assert np.array_equal(one.nn_idx.cpu().numpy(), ridx), (sort, step, mode)
            assert np.array_equal(one.nn_d2.cpu().numpy().view(np.uint32), rd2.view(np.uint32)), (sort, step, mode)
            assert one.fallbacks[0][0] == rF
    for sort in (True, False):
        runs = [r for s, r in res if s == sort]
        for r in runs[1:]:
            assert np.array_equal(r.Rt, runs[0].Rt) and np.array_equal(r.rmse[0], runs[0].rmse[0])
            assert np.array_equal(r.candidates[0], runs[0].candidates[0])
