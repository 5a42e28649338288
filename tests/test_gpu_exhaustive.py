"""The exhaustive registration's correspondences against the oracle's exact
nearest targets (a grid of one voxel), bit for bit: target counts at, one
below and one past a chunk (32) and a staged tile (512), source counts around
a block (256), a block of four queries a thread (1024) and the size from which
that form is taken (16384), equal distances in different chunks and splits
(the lowest index wins), and batches of uneven pairs with an empty one."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def exact(q, p):
    idx, d2, _, _ = oracle.nns(oracle.build_grid_fixed(q, (-10.0, -10.0, -10.0), 20.0, (1, 1, 1)), q, p, IDENT)
    return idx, d2.view(np.uint32)


@pytest.mark.parametrize("ns,ms", [((n,), (m,)) for n in (1, 31, 32, 33, 511, 513, 9001) for m in (1, 255, 257, 1025)] +
                         [((700,), (16383,)), ((700,), (16384,)), ((5000,), (17409,)), ((97,), (40000,)),
                          ((40, 3000, 1, 900), (700, 0, 5, 2049)), ((33, 2000, 512), (9000, 1, 8000))])
@pytest.mark.parametrize("copies", [False, True])
def test_correspondences(ns, ms, copies):
    rng = np.random.default_rng(sum(ns) + sum(ms))
    qs = [rng.uniform(-1, 1, (3, n)).astype(np.float32) for n in ns]
    if copies:   # every target several times over, far apart in the list
        qs = [q[:, rng.integers(0, max(1, q.shape[1] // 7), q.shape[1])] for q in qs]
    ps = [rng.uniform(-1.5, 1.5, (3, m)).astype(np.float32) for m in ms]
    g = build_grid_batched(dev(np.concatenate(qs, 1)), list(ns), [0.5] * len(ns), 1).dilate(1)
    for K in (1, 2):   # the words of an earlier iteration are not taken for this one's
        res = g.register(dev(np.concatenate(ps, 1)), K, m_per_pair=list(ms), global_only=True, correspondences=True)
    one = g.register(dev(np.concatenate(ps, 1)), 1, m_per_pair=list(ms), global_only=True, correspondences=True)
    idx, d2 = one.nn_idx.cpu().numpy(), one.nn_d2.cpu().numpy().view(np.uint32)
    at = 0
    for b, (q, p, m) in enumerate(zip(qs, ps, ms)):
        if m == 0:
            continue
        ridx, rd2 = exact(q, p)
        assert np.array_equal(idx[at:at + m], ridx) and np.array_equal(d2[at:at + m], rd2)
        assert one.fallbacks[b][0] == m and one.candidates[b][0] == 0
        assert list(res.fallbacks[b]) == [m] * len(res.fallbacks[b])
        # rmse: float64 sums of the float32 squared distances, exact to the order of m roundings
        want = np.sqrt(rd2.view(np.float32).astype(np.float64).sum() / m)
        np.testing.assert_allclose(one.rmse[b][0], want, rtol=2.3e-16 * (m + 4), atol=0)
        at += m
