"""Overlapped waves of exactly half the buffers' capacity: the two waves' grids
fill the grid region, and the tile table of every wave takes the table region
from its start.  Curves whose harmonics reach the end of the covered grid
periods write the table to its last entry; the rows, chi2_0 and flags are the
one-stream search's bit for bit, repeated."""
import numpy as np
import pytest

from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note
from tests.test_gpu_fused import same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("curves,H,log_nf,laps", [(2, 1, 10, 1), (2, 3, 10, 1), (40, 2, 11, 1),
                                                  (4, 3, 11, 3), (24, 5, 12, 1)])
def test_half_capacity_waves_match_one_stream(curves, H, log_nf, laps):
    import torch
    rng = np.random.default_rng(curves + H)
    nf, span, n = 2 ** log_nf, 10.0, 300
    # harmonic 2H ends 20 cells before the end of the last period
    L = 4 * nf
    f_max = (laps * L - 20.0) / L * nf / (2 * H * span)
    t = np.concatenate([np.r_[0.0, np.sort(rng.uniform(0, span, n - 2)), span] for _ in range(curves)])
    x, s = rng.normal(size=t.size), rng.uniform(0.5, 1.5, t.size)
    dev = [torch.from_numpy(v).cuda() for v in (t, x, s)]
    off = np.arange(curves + 1) * n
    outs = []
    for two in (False, True):
        plan = F.Plan(off, f_max, H, nf, precision="mixed", t_span=[span] * curves, two_streams=two)
        info = plan.info()
        assert info["curves_per_wave"] == curves
        plan.set_schedule(dict(info, curves_per_wave=curves // 2))
        for rep in range(3 if two else 1):
            note(f"half-capacity waves: {curves} curves, H {H}, two streams {two}, run {rep}")
            d, c0, fl = plan.search(*dev)
            torch.cuda.synchronize()
            outs.append([v.cpu() for v in (d, c0, fl)])
        plan.close()
    assert np.isfinite(outs[0][0][:, :, 1:].double().numpy()).all()
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert same_bits(a, b)
