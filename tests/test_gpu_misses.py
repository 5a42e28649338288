"""Correspondences whose queries miss: the search's masks and the launch that
resolves them, against the oracle bit for bit.  Every number of lanes per query
and block size, source sizes around a wave, a block and one block's share of
masks; no query, a few and all of them missing; batches with empty pairs; both
entry points; queries so far off that no distance is finite (target 0,
infinitely far); and more masks than the launch takes in one round."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched, build_grid_fixed  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def case(seed, n, m, share):
    rng = np.random.default_rng(seed)
    q = rng.uniform(0, 10, (3, n)) * np.array([[1.0], [1.0], [0.1]])
    p = q[:, rng.integers(0, n, m)] + rng.normal(0, 0.05, (3, m))
    far = np.sort(rng.permutation(m)[:int(round(share * m))])
    p[2, far] += rng.uniform(2.0, 9.0, far.size)
    return q.astype(np.float32), p.astype(np.float32)


@pytest.mark.parametrize("m", [1, 63, 64, 65, 511, 513, 6000])
@pytest.mark.parametrize("share", [0.0, 0.05, 1.0])
def test_masks(m, share):
    q, p = case(m, 3000, m, share)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 0.5, (21, 21, 21)), 1)
    ridx, rd2, rF, _ = oracle.nns(og, q, p, IDENT)
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 0.5, (21, 21, 21), 1).dilate(1)
    for block, lanes in ((128, 1), (128, 8), (256, 2), (512, 4), (512, 8)):
        g.set_schedule(block, lanes, lanes != 2, 64)
        idx, d2, fb = g.nns(dev(p), IDENT)
        i2 = torch.full((m,), -7, dtype=torch.int32, device="cuda")
        e2 = torch.zeros(m, device="cuda")
        f2 = torch.zeros(1, dtype=torch.int32, device="cuda")
        g.nns_noalloc(dev(p), IDENT, i2, e2, f2)
        for a, b, f in ((idx, d2, fb), (i2, e2, f2)):
            assert np.array_equal(a.cpu().numpy(), ridx) and int(f.cpu()[0]) == rF
            assert np.array_equal(b.cpu().numpy().view(np.uint32), rd2.view(np.uint32))


@pytest.mark.parametrize("ms", [(0, 5, 700), (900, 0, 1300, 64)])
def test_batches(ms):
    qs, ps = zip(*(case(7 + k, 800 + 100 * k, max(m, 1), 0.3) for k, m in enumerate(ms)))
    ps = [p[:, :m] for p, m in zip(ps, ms)]
    g = build_grid_batched(dev(np.concatenate(qs, 1)), [q.shape[1] for q in qs], [0.5] * len(ms), 1).dilate(1)
    idx, d2, fb = g.nns(dev(np.concatenate(ps, 1)), np.tile(IDENT, len(ms)), m_per_pair=list(ms))
    at = 0
    for b, (q, p, m) in enumerate(zip(qs, ps, ms)):
        ridx, rd2, rF, _ = oracle.nns(oracle.dilate(oracle.build_grid(q, 0.5, 1), 1), q, p, IDENT) if m else (0, 0, 0, 0)
        assert int(fb.cpu()[b]) == rF
        if m:
            assert np.array_equal(idx[at:at + m].cpu().numpy(), ridx)
            assert np.array_equal(d2[at:at + m].cpu().numpy().view(np.uint32), rd2.view(np.uint32))
        at += m


def test_no_finite_distance():
    q, p = case(3, 500, 200, 0.1)
    p[0, ::9] = 3e19     # the square overflows float32
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 0.5, (21, 21, 21), 1).dilate(1)
    idx, d2, fb = g.nns(dev(p), IDENT)
    assert (idx.cpu().numpy()[::9] == 0).all() and np.isinf(d2.cpu().numpy()[::9]).all()
    rest = np.arange(200) % 9 != 0
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 0.5, (21, 21, 21)), 1)
    ridx, rd2, _, _ = oracle.nns(og, q, np.ascontiguousarray(p[:, rest]), IDENT)
    assert np.array_equal(idx.cpu().numpy()[rest], ridx)
    assert np.array_equal(d2.cpu().numpy()[rest].view(np.uint32), rd2.view(np.uint32))


def test_more_masks_than_a_round():
    q, p = case(5, 2000, 2000, 0.02)
    p = np.tile(p, (1, 850))     # 1.7M queries, 8 to a wave: 212,500 masks
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 0.5, (21, 21, 21), 1).dilate(1)
    g.set_schedule(128, 8, True, 64)
    idx, d2, fb = g.nns(dev(p), IDENT)
    og = oracle.dilate(oracle.build_grid_fixed(q, (0.0, 0.0, 0.0), 0.5, (21, 21, 21)), 1)
    ridx, rd2, rF, _ = oracle.nns(og, q, np.ascontiguousarray(p[:, :2000]), IDENT)
    assert int(fb.cpu()[0]) == 850 * rF
    assert (idx.view(850, 2000) == torch.from_numpy(ridx).cuda()).all()
    assert (d2.view(850, 2000) == torch.from_numpy(rd2).cuda()).all()
