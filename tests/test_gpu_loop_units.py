"""Blocks of the resident loop that take two units in turn, against the
launch-per-step form bit for bit: no query without a candidate, and such
queries in the first units only, in the second only, in both and scattered,
so that a block's units take the two paths (with and without global searches)
in either order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd.api import build_grid_batched, prof_enable, prof_reset  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("lanes", [1, 4, 8])
@pytest.mark.parametrize("units,extra", [(257, 0), (300, -5), (512, 0)])
@pytest.mark.parametrize("where", ["none", "first", "second", "both", "scattered"])
def test_two_units_a_block(lanes, units, extra, where):
    rng = np.random.default_rng(units + lanes)
    m = 16 * 64 // lanes * units + extra
    u = rng.uniform(0, 1, (2, 20000))
    q = np.stack([u[0], u[1], 0.2 * np.sin(7 * u[0]) * np.cos(5 * u[1])])
    p = q[:, rng.integers(0, 20000, m)] + rng.normal(0, 0.002, (3, m)) + np.array([[0.004], [-0.003], [0.005]])
    # query t of the source order is in record t // (64 / lanes), record r in
    # unit r mod U, unit u the second one of a block from half the units on
    unit = np.arange(m) * lanes // 64 % units
    late = unit >= -(-units // 2)
    far = {"none": np.zeros(m, bool), "first": ~late, "second": late, "both": late | ~late,
           "scattered": rng.random(m) < 0.3}[where] & (rng.random(m) < 0.02)
    p[2, far] += rng.uniform(0.2, 0.4, int(far.sum()))
    g = build_grid_batched(dev(q), [20000], [0.03], 2).dilate(2)
    g.set_schedule(256, lanes, False, 64)
    kw = dict(m_per_pair=[m], correspondences=True)
    one = g.register(dev(p), 4, **kw)
    prof_enable(True)   # with timing on: one launch per step
    try:
        step = g.register(dev(p), 4, **kw)
    finally:
        prof_enable(False)
        prof_reset()
    assert (one.fallbacks[0][0] > 0) == bool(far.any())
    assert np.array_equal(one.Rt, step.Rt) and np.array_equal(one.rmse[0], step.rmse[0])
    assert np.array_equal(one.fallbacks[0], step.fallbacks[0])
    assert np.array_equal(one.candidates[0], step.candidates[0])
    assert torch.equal(one.nn_idx, step.nn_idx) and torch.equal(one.nn_d2.view(torch.int32), step.nn_d2.view(torch.int32))
