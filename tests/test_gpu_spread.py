"""The spreading sums every cell in point order, whatever strips the grid is cut
into: identical bit for bit to the spreading fused into the first FFT pass (a
thread per row segment, written independently), on strips of 32 cells (few
curves) and of 128 (eight curves of 2^18 cells), with points on and beside the
strips' edges, many points in one cell, one point, phases that wrap around the
grid, and every kind of kernel (floor gridding, the narrowest, odd, the widest);
and against the oracle."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note, sample_bins
from tests.test_gpu_fused import same_bits

pytestmark = pytest.mark.gpu


def _curve(rng, kind, span, cell):
    """Times of one curve on [0, span], sigma and data."""
    if kind == "edges":  # on and one ulp beside multiples of 32 and 128 cells
        t = np.arange(0.0, span, 32 * cell)[:400]
        t = np.concatenate([t, np.nextafter(t, span), t + 0.5 * cell])
    elif kind == "dense":  # hundreds of points in a few cells, then a gap
        t = np.concatenate([rng.uniform(0, 3 * cell, 700), rng.uniform(0.6 * span, span, 40), [span]])
    elif kind == "one":
        t = np.array([0.3 * span])
    else:
        t = rng.uniform(0.0, span, 350)
    t = np.sort(t)
    s = rng.uniform(0.05, 0.3, t.shape[0])
    return t, np.sin(2 * np.pi * t * 37.3 / span) + s * rng.standard_normal(t.shape[0]), s


@pytest.mark.parametrize("log_nf,curves,width,wrap,precision", [
    (12, 4, 0, False, "mixed"), (12, 4, 1, False, "mixed"), (12, 4, 4, True, "mixed"),
    (12, 4, 7, False, "fp64"), (12, 4, 16, True, "fp64"), (16, 8, 0, False, "mixed"),
    (16, 8, 16, True, "mixed"), (16, 8, 0, True, "fp64")])
def test_strips_identical_to_fused_and_match_the_oracle(log_nf, curves, width, wrap, precision):
    import torch
    nf, H, f_max = 1 << log_nf, 3, 10.0
    # harmonic 2H spans 0.85 or 1.7 grid periods
    span = (1.7 if wrap else 0.85) * nf / (2 * H * f_max)
    rng = np.random.default_rng(log_nf + width)
    kinds = ["edges", "dense", "one", "plain"] * (curves // 4)
    per = [_curve(rng, k, span, span / ((1.7 if wrap else 0.85) * 4 * nf)) for k in kinds]
    off = np.concatenate([[0], np.cumsum([len(c[0]) for c in per])])
    t, x, s = (torch.from_numpy(np.concatenate([c[i] for c in per])).cuda() for i in range(3))
    outs = []
    for fused in (False, True):
        note(f"strips 2^{log_nf} x {curves} w {width} wrap {wrap} {precision} fused {fused}")
        plan = F.Plan(off, f_max, H, nf, precision=precision, kernel_width=width, fused_spread=fused)
        d, c0, fl = plan.search(t, x, s)
        torch.cuda.synchronize()
        outs.append((d.cpu(), c0.cpu(), fl.cpu()))
        plan.close()
    for u, v in zip(*outs):
        assert same_bits(u, v)
    if width in (0, 16):
        bins = sample_bins(nf, 60, 9)
        fr = bins * (f_max / nf)
        kmax, tol = (1e2, 1e-5) if precision == "mixed" else (1e6, 1e-8)
        for c in (1, 3):
            ref = ora.dchi2(*per[c], fr, H)
            gate = ora.gate_mask(ref, fr, kmax)
            err = ora.rel_err(outs[0][0][c].double().numpy()[:, bins], ref["dchi2"])[:, gate]
            assert err.size == 0 or err.max() <= tol
