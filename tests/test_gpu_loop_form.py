"""Which form a registration takes: the resident loop for every source whose
units (16 wave records) are at most two per block of the device (one on a grid
of 4 points a voxel or more), launches per step past that and for the forms that have no loop, and a hand-over for queries
without a finite distance.  The comparisons of the two forms rest on this."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import (FORM_HANDED_OVER, FORM_LOOP, FORM_NONE, FORM_STEPS,  # noqa: E402
                                       VicpError)
from paper_2512_04996_amd.api import build_grid_batched, build_grid_fixed, prof_enable, prof_reset  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def cloud(n, m):
    rng = np.random.default_rng(n + m)
    u = rng.uniform(0, 1, (2, n))
    q = np.stack([u[0], u[1], 0.2 * np.sin(7 * u[0]) * np.cos(5 * u[1])])
    return q, q[:, rng.integers(0, n, m)] + rng.normal(0, 0.004, (3, m))


def grid(q, ms):
    B = len(ms)
    return build_grid_batched(dev(np.tile(q, B)), [q.shape[1]] * B, [0.05] * B, 2).dilate(2)


@pytest.mark.parametrize("lanes", [1, 2, 4, 8])
@pytest.mark.parametrize("sort", [True, False])
def test_single_pair_by_units(lanes, sort):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    unit = 16 * 64 // lanes
    most = min(2 * cus, 512)
    q, p = cloud(5000, most * unit + 1)
    g = grid(q, [1])
    assert g.last_form == FORM_NONE
    g.set_schedule(256, lanes, sort, 64)
    for m, form in ((64, FORM_LOOP), (5 * unit, FORM_LOOP), (cus * unit, FORM_LOOP), (cus * unit + 1, FORM_LOOP),
                    (most * unit, FORM_LOOP), (most * unit + 1, FORM_STEPS)):
        g.register(dev(p[:, :m]), 2, m_per_pair=[m])
        assert g.last_form == form, (m, lanes)
    g.register(dev(p[:, :0]), 2, m_per_pair=[0])
    assert g.last_form == FORM_NONE


@pytest.mark.parametrize("ms,form", [((0, 64, 0), FORM_LOOP), ((700, 0, 64, 1025, 40000), FORM_LOOP),
                                     ((300,) * 40 + (90000,), FORM_LOOP), ((60000,) * 20, FORM_STEPS)])
def test_batches(ms, form):
    q, _ = cloud(3000, 1)
    p = np.concatenate([cloud(3000, m)[1] for m in ms], 1)
    g = grid(q, ms)
    g.register(dev(p), 3, m_per_pair=list(ms))
    assert g.last_form == form


@pytest.mark.parametrize("n,crowded", [(4 * 4096 - 1, False), (4 * 4096, True)])
def test_crowded_grids_take_one_unit_a_block(n, crowded):
    cus = min(torch.cuda.get_device_properties(0).multi_processor_count, 512)
    rng = np.random.default_rng(n)
    q = rng.uniform(0, 16, (3, n))
    g = build_grid_fixed(dev(q), (0.0, 0.0, 0.0), 1.0, (16, 16, 16), 2).dilate(2)
    g.set_schedule(256, 8, True, 64)
    for m, form in ((128 * cus, FORM_LOOP), (128 * cus + 1, FORM_STEPS if crowded else FORM_LOOP)):
        p = q[:, rng.integers(0, n, m)] + rng.normal(0, 0.1, (3, m))
        g.register(dev(p), 2)
        assert g.last_form == form, m


def test_forms_without_a_loop_and_hand_over():
    q, p = cloud(4000, 3000)
    g = grid(q, [3000]).build_direct(4096)
    for kw, form in (({}, FORM_LOOP), ({"use_graph": False}, FORM_LOOP), ({"early_stop": True}, FORM_LOOP),
                     ({"global_only": True}, FORM_STEPS), ({"layout": "direct"}, FORM_STEPS)):
        g.register(dev(p), 3, **kw)
        assert g.last_form == form, kw
    prof_enable(True)
    try:
        g.register(dev(p), 3)
    finally:
        prof_enable(False)
        prof_reset()
    assert g.last_form == FORM_STEPS
    g.rebuild_register(dev(q), 2, dev(p), 3)
    assert g.last_form == FORM_LOOP
    far = p.copy()
    far[0, 5] = 3e19          # finite, but its squared distances are not
    g.register(dev(far), 3)
    assert g.last_form == FORM_HANDED_OVER
    far[0, 5] = np.nan
    with pytest.raises(VicpError):
        g.register(dev(far), 3)
    assert g.last_form == FORM_HANDED_OVER
    g.register(dev(p), 3)
    assert g.last_form == FORM_LOOP
