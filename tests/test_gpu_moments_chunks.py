"""Moments of curves of one chunk (written by the reducing kernel itself) and of
more (combined by a second one): chi2_0 and the flags of empty, one-point, short,
full and one-point-more chunks, alone and beside each other.  Tolerance: FP64
sums of at most 2049 positive terms, n eps < 1e-12."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1,), (255,), (257, 0, 3), (1023, 1024), (1025,), (2049, 1, 5)])
def test_chi2_0(sizes):
    import torch
    note(f"moments sizes={sizes}")
    rng = np.random.default_rng(len(sizes) + sizes[0])
    off = np.concatenate([[0], np.cumsum(sizes)])
    t = np.concatenate([np.sort(rng.uniform(0, 50.0, n)) for n in sizes])
    s = rng.uniform(0.5, 1.5, t.size)
    x = 7.0 + rng.normal(size=t.size)
    plan = F.Plan(off, 2.0, 1, 1 << 11, precision="fp64")
    _, c0, fl = plan.search(*[torch.from_numpy(v).cuda() for v in (t, x, s)])
    c0, fl = c0.cpu().numpy(), fl.cpu().numpy()
    for c, (a, b) in enumerate(zip(off[:-1], off[1:])):
        if a == b:
            assert np.isnan(c0[c]) and (fl[c] & 0x80).all()
            continue
        ref = ora.moments(t[a:b], x[a:b], s[a:b])["chi2_0"]
        assert abs(c0[c] - ref) <= 1e-12 * max(ref, 1.0)
