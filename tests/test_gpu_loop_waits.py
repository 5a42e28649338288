"""Registrations whose loop blocks do not all meet: a stream that may use only a
part of the compute units runs launches per step from the start, and a loop whose
wait is over (its limits set to nothing, so that the first wait ends it) hands
over, after which the grid leaves the loop out for 32 registrations and then
takes it again.  Results are the loop's bit for bit, and no call waits a second."""
import ctypes
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import FORM_HANDED_OVER, FORM_LOOP, FORM_STEPS, lib  # noqa: E402
from paper_2512_04996_amd.api import build_grid_batched  # noqa: E402

REST = 32


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def case(ms):
    rng = np.random.default_rng(sum(ms))
    u = rng.uniform(0, 1, (2, 4000))
    q = np.stack([u[0], u[1], 0.2 * np.sin(7 * u[0]) * np.cos(5 * u[1])])
    p = np.concatenate([q[:, rng.integers(0, 4000, m)] + rng.normal(0, 0.004, (3, m)) for m in ms], 1)
    B = len(ms)
    return build_grid_batched(dev(np.tile(q, B)), [4000] * B, [0.05] * B, 2).dilate(2), dev(p)


def equal(a, b):
    return (np.array_equal(a.Rt, b.Rt) and all(np.array_equal(x, y) for x, y in zip(a.rmse, b.rmse)) and
            torch.equal(a.nn_idx, b.nn_idx) and torch.equal(a.nn_d2, b.nn_d2))


def waits(g, arrive, patience):
    f = lib().vicp_test_loop_waits
    f.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint64]
    assert f(g.handle, arrive, patience) == 0


@pytest.mark.parametrize("ms", [(20000,), (9000, 3000, 700)])
def test_a_wait_that_is_over_hands_over_and_rests(ms):
    g, p = case(ms)
    kw = dict(m_per_pair=list(ms), correspondences=True)
    ref = g.register(p, 5, **kw)
    assert g.last_form == FORM_LOOP
    waits(g, 0, 0)
    t0 = time.perf_counter()
    got = g.register(p, 5, **kw)
    assert time.perf_counter() - t0 < 0.5
    assert g.last_form == FORM_HANDED_OVER and equal(got, ref)
    waits(g, 200000, 100000000)
    for k in range(REST):
        got = g.register(p, 5, **kw)
        assert g.last_form == FORM_STEPS and (k % 16 or equal(got, ref))
    for _ in range(3):
        got = g.register(p, 5, **kw)
        assert g.last_form == FORM_LOOP and equal(got, ref)


def test_a_stream_of_some_compute_units_runs_steps():
    # the runtime this process already uses
    path = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
    hip = ctypes.CDLL(path.pop())
    g, p = case((20000,))
    ref = g.register(p, 5, correspondences=True)
    assert g.last_form == FORM_LOOP
    torch.cuda.synchronize()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    words = (cus + 31) // 32
    mask = (ctypes.c_uint32 * words)(*[0x0000FFFF] * words)     # half of each word's
    s = ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(s), ctypes.c_uint32(words), mask) == 0
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(s.value)):
            for _ in range(2):
                t0 = time.perf_counter()
                got = g.register(p, 5, correspondences=True)
                torch.cuda.current_stream().synchronize()
                assert time.perf_counter() - t0 < 0.5
                assert g.last_form == FORM_STEPS and equal(got, ref)
    finally:
        torch.cuda.synchronize()
        hip.hipStreamDestroy(s)
    with torch.cuda.stream(torch.cuda.Stream()):
        got = g.register(p, 5, correspondences=True)
        assert g.last_form == FORM_LOOP and equal(got, ref)
