"""Fine search at the edges of its split of the points: odd counts (points are
summed in pairs), one chunk and less, chunk remainders, more chunks than the
adding kernel takes at a time, curves of different chunk counts in one call, and
trial counts that leave lanes of the last wave idle.  Rows against the oracle,
relative with a floor of 2H'.  Tolerance: the phases' and sums' FP64 rounding, a
few eps times sqrt(n) <= 96, times condition numbers kept below 1e4, is below
1e-9 with room."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(41,), (64, 65, 129), (1023, 1024, 1025), (2049, 300),
                                   (8 * 1024 + 1, 9 * 1024)])
@pytest.mark.parametrize("H,K,R", [(1, 3, 7), (4, 2, 33), (8, 1, 64)])
def test_point_splits(sizes, H, K, R):
    import torch
    note(f"fine search sizes={sizes} H={H} K={K} R={R}")
    rng = np.random.default_rng(sum(sizes) + H)
    off = np.concatenate([[0], np.cumsum(sizes)])
    t = np.concatenate([np.sort(rng.uniform(0, 50.0, n)) for n in sizes])
    s = rng.uniform(0.5, 1.5, t.size)
    x = 3.0 + np.sin(2 * np.pi * 0.7 * t) + s * rng.normal(size=t.size)
    plan = F.Plan(off, 2.0, H, 1 << 13, precision="fp64")
    dev = [torch.from_numpy(v).cuda() for v in (t, x, s)]
    centres = rng.uniform(0.3, 1.9, (len(sizes), K))
    hw = 0.01
    rows = plan.fine_search(*dev, torch.from_numpy(centres).cuda(), R=R, half_width=hw,
                            want_rows=True)["rows"].cpu().numpy()
    torch.cuda.synchronize()
    for c, (a, b) in enumerate(zip(off[:-1], off[1:])):
        for j in range(K):
            pick = np.unique([0, R // 2, R - 1])
            fr = centres[c, j] + hw * (2.0 * pick / (R - 1) - 1.0)
            ref = ora.dchi2(t[a:b], x[a:b], s[a:b], fr, H)
            gate = ora.gate_mask(ref, fr, 1e4)
            assert gate.all()
            e = ora.rel_err(rows[c, j][pick].T, ref["dchi2"])
            assert e.max() <= 1e-9, (c, j, e.max())
