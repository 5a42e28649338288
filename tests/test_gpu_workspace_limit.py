"""A workspace that grows takes an eighth more than it needs, but where the
allocator has only what it needs the grid takes that: through an allocator that
refuses larger requests, the rebuild and the registration succeed and give what a
fresh grid gives; one that refuses the need itself is out of memory."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import ERR_OOM, VicpError, check, lib  # noqa: E402
from paper_2512_04996_amd.api import Grid, _ptrs, _stream, build_grid  # noqa: E402

ALLOC = C.CFUNCTYPE(C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p)
FREE = C.CFUNCTYPE(None, C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p)


class Allocator(C.Structure):
    _fields_ = [("alloc", ALLOC), ("free", FREE), ("user", C.c_void_p)]


class Limited:
    """Device memory in torch tensors, requests above `limit` refused."""

    def __init__(self):
        self.limit, self.asked, self.held = None, [], {}
        self.struct = Allocator(ALLOC(self.alloc), FREE(self.free), None)

    def alloc(self, n, stream, user):
        self.asked.append(n)
        if self.limit is not None and n > self.limit:
            return None
        t = torch.empty(n, dtype=torch.uint8, device="cuda")
        self.held[t.data_ptr()] = t
        return t.data_ptr()

    def free(self, p, n, stream, user):
        torch.cuda.synchronize()
        del self.held[p]


def grid(q, voxel, rings, mem):
    h = C.c_void_p()
    qx, qy, qz = _ptrs(q)
    check(lib().vicp_build_grid(qx, qy, qz, q.shape[1], C.c_float(voxel), rings, C.cast(C.pointer(mem.struct), C.c_void_p),
                                _stream(), C.byref(h)), "vicp_build_grid")
    return Grid(h, q, [q.shape[1]], [voxel], rings)


def clouds(scale):
    rng = np.random.default_rng(7)
    q = rng.uniform(0, scale, (3, 3000)).astype(np.float32)
    p = q[:, rng.integers(0, 3000, 2000)] + rng.normal(0, 0.01, (3, 2000)).astype(np.float32)
    return torch.from_numpy(q).cuda(), torch.from_numpy(p.astype(np.float32)).cuda()


def run(g, q, p):
    g.rebuild(q).dilate(2)
    return g.register(p, 4, correspondences=True)


def test_growth_takes_what_there_is():
    small, large = clouds(1.0), clouds(2.0)
    mem = Limited()
    g = grid(small[0], 0.05, 2, mem)
    run(g, *small)
    mem.asked.clear()
    run(g, *large)
    growth = list(mem.asked)            # each its need and an eighth of it
    assert growth and all(n > (1 << 16) for n in growth)
    g.free()
    assert not mem.held
    ref = build_grid(large[0], 0.05, 2)
    want = run(ref, *large)
    mem = Limited()
    g = grid(small[0], 0.05, 2, mem)
    run(g, *small)
    mem.limit = max(n * 8 // 9 + 256 for n in growth)
    got = run(g, *large)
    assert np.array_equal(got.Rt, want.Rt) and torch.equal(got.nn_idx, want.nn_idx)
    assert max(n for n in mem.asked) > mem.limit      # it asked for more first
    g.free()
    mem = Limited()
    g = grid(small[0], 0.05, 2, mem)
    run(g, *small)
    mem.limit = min(n * 8 // 9 - 4096 for n in growth)
    with pytest.raises(VicpError) as e:
        run(g, *large)
    assert e.value.code == ERR_OOM
    g.free()
    assert not mem.held
