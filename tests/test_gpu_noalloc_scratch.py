"""The allocation-free search at the ends of its fixed array: the most source
points, and one search block fewer, under the schedules with the most search
blocks and the most waves, with misses; equal to vicp_nns bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2512_04996_amd._lib import NOALLOC_MAX_QUERIES  # noqa: E402
from paper_2512_04996_amd.api import build_grid  # noqa: E402

IDENT = np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], np.float32)


@pytest.mark.parametrize("m", [NOALLOC_MAX_QUERIES, NOALLOC_MAX_QUERIES - 15, 1])
def test_ends_of_the_array(m):
    rng = np.random.default_rng(m)
    q = rng.uniform(0, 1, (3, 5000)).astype(np.float32)
    p = rng.uniform(-0.02, 1.02, (3, m)).astype(np.float32)
    g = build_grid(torch.from_numpy(q).cuda(), 0.05, 1).dilate(1)
    P = torch.from_numpy(p).cuda()
    for block, lanes in ((128, 8), (512, 8), (256, 1)):
        g.set_schedule(block, lanes, False, 64)
        idx, d2, fb = g.nns(P, IDENT)
        out = (torch.full((m,), -7, dtype=torch.int32, device="cuda"), torch.zeros(m, device="cuda"),
               torch.zeros(1, dtype=torch.int32, device="cuda"))
        g.nns_noalloc(P, IDENT, *out)
        assert torch.equal(idx, out[0]) and torch.equal(d2.view(torch.int32), out[1].view(torch.int32))
        assert torch.equal(fb, out[2])
