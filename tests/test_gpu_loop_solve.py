"""Sums that the resident loop's refinement does not solve stay in the loop:
near-planar and mirrored clouds, turns of more than 90 degrees, and targets on a
line or in one place (the pose is kept).  Results equal the launch-per-step
form's bit for bit, and no registration hands over and starts again."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import FORM_LOOP, FORM_STEPS  # noqa: E402
from paper_2512_04996_amd.api import build_grid_batched, prof_enable, prof_reset  # noqa: E402

TURN = np.array([-1.0, 0, 0, 0, -1, 0, 0, 0, 1, 1, 1, 0])


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def clouds(kind, n, m):
    rng = np.random.default_rng(n + m)
    u = rng.uniform(0, 1, (2, n))
    z = 0.2 * np.sin(7 * u[0]) * np.cos(5 * u[1])
    q = np.stack([u[0], u[1], {"plane": 0 * z, "thin": 1e-4 * z, "line": 0 * z}.get(kind, z)])
    if kind == "line":
        q[1] = 0.4
    p = q[:, rng.integers(0, n, m)]
    if kind in ("turned", "mirrored", "bumpy"):
        p = p + rng.normal(0, 0.002, (3, m))
    if kind == "mirrored":
        p[0] = 1.0 - p[0]
    if kind == "one_place":
        p = np.tile(p[:, :1], (1, m))
    return q, p + np.array([[0.004], [-0.003], [0.0]])


@pytest.mark.parametrize("kinds", [("plane",), ("thin",), ("line",), ("one_place",), ("turned",), ("mirrored",),
                                   ("bumpy", "plane", "line", "turned")])
@pytest.mark.parametrize("m", [1, 700, 30000])
def test_loop_solves_what_the_refinement_does_not(kinds, m):
    qs, ps = zip(*(clouds(k, 4000, m) for k in kinds))
    B = len(kinds)
    g = build_grid_batched(dev(np.concatenate(qs, 1)), [4000] * B, [0.05] * B, 2).dilate(2)
    g.set_schedule(128, 2, True, 64)
    rt = np.concatenate([TURN if k == "turned" else np.eye(3, 4).reshape(12)[[0, 1, 2, 4, 5, 6, 8, 9, 10, 3, 7, 11]]
                         for k in kinds])
    p = dev(np.concatenate(ps, 1))
    kw = dict(m_per_pair=[m] * B, Rt0=rt, correspondences=True)
    one = g.register(p, 6, **kw)
    assert g.last_form == FORM_LOOP
    prof_enable(True)
    try:
        step = g.register(p, 6, **kw)
    finally:
        prof_enable(False)
        prof_reset()
    assert g.last_form == FORM_STEPS
    assert np.array_equal(one.Rt, step.Rt) and one.status == step.status
    assert np.array_equal(one.degenerate, step.degenerate) and np.array_equal(one.iters, step.iters)
    for x, y in ((one.rmse, step.rmse), (one.fallbacks, step.fallbacks), (one.candidates, step.candidates)):
        assert all(np.array_equal(a, b) for a, b in zip(x, y))
    assert torch.equal(one.nn_idx, step.nn_idx) and torch.equal(one.nn_d2.view(torch.int32), step.nn_d2.view(torch.int32))
    for k, d in zip(kinds, one.degenerate):
        if m == 1 or k in ("line", "one_place"):
            assert d == 6, (k, d)
