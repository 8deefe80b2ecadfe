"""FFT tiles chosen by a launch's size (a plan neither tuned nor set) against the
2^12-element tiles that its reported schedule sets: the same bits, on both sides
of every line of the rule (tiles of 2^13 per launch: first pass radix 2^9 160,
2^8 8192; middle 1024; last 2^9 128, 2^8 768, 2^7 1536), for the rows, the
gradient, a band and sources sharing their times.  No tolerance: the same
operations on each element, in another grouping."""
import numpy as np
import pytest

from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


def _points(nc, n, span, seed):
    import torch
    rng = np.random.default_rng(seed)
    t = np.concatenate([np.sort(rng.uniform(0, span, n)) for _ in range(nc)])
    x = np.sin(2 * np.pi * 0.31 * t) + rng.normal(size=t.size)
    s = rng.uniform(0.5, 2.0, t.size)
    return np.arange(nc + 1) * n, [torch.from_numpy(v).cuda() for v in (t, x, s)]


# (log2 bins, H, curves): two passes [9,9], [9,8], [8,8], [8,7], [7,7] below and
# above their lines, three passes [7,7,7] and [8,8,8].
@pytest.mark.parametrize("lf,H,nc", [(16, 2, 1), (16, 3, 3), (15, 3, 3), (14, 3, 24),
                                     (13, 3, 40), (12, 3, 200), (18, 1, 1), (19, 3, 2),
                                     (22, 3, 1)])
def test_rows(lf, H, nc):
    import torch
    note(f"launch tiles 2^{lf} bins H={H} curves={nc}")
    off, a = _points(nc, 300, 60.0, lf + H + nc)
    plan = F.Plan(off, 2.0 ** (lf - 12), H, 1 << lf, precision="mixed")
    d, _, fl = plan.search(*a)
    plan.set_schedule(plan.info())
    e, _, fk = plan.search(*a)
    torch.cuda.synchronize()
    assert torch.equal(d.view(torch.int32), e.view(torch.int32)) and torch.equal(fl, fk)


def test_gradient_band_and_shared_times():
    import torch
    note("launch tiles: gradient, band, shared times")
    off, a = _points(2, 400, 50.0, 7)
    one = [v[:400].contiguous() for v in a]
    src = torch.from_numpy(np.random.default_rng(3).normal(size=(40, 400))).cuda()
    scale = torch.linspace(0.5, 2.0, 40, dtype=torch.float64, device="cuda")
    out = []
    for fix in (False, True):
        keep = F.Plan(off, 40.0, 3, 1 << 19, precision="mixed", keep_for_backward=True)
        band = F.Plan(off, 40.0, 3, 1 << 19, precision="mixed", first_bin=1 << 17)
        multi = F.Plan([0, 400], 10.0, 3, 1 << 16, precision="mixed")
        if fix:
            for p in (keep, band, multi):
                p.set_schedule(p.info())
        d, _, _ = keep.search(*a)
        g = torch.zeros_like(d)
        g[:, :, 1000::4099] = 1.0
        gx, gs = keep.backward(*a, g)[:2]
        b, _, _ = band.search(*a)
        m, _, _ = multi.search_multi(one[0], one[2], src, scale)
        torch.cuda.synchronize()
        out.append((d, gx, gs, b, m))
    for u, v in zip(*out):
        assert torch.isfinite(u).any()
        assert u.cpu().numpy().tobytes() == v.cpu().numpy().tobytes()
