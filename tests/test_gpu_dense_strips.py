"""Strips that hold many points are spread with a lane per cell: 64-cell blocks of
harmonic 1 around every count at which that is decided (48 points of both
components, 1000 or 1500 of one) and at which points are staged anew (384), with
points on cells, on cell edges and in a single cell, and the other harmonics'
blocks stretched over more.  The cells, hence all results, are those of the
spreading fused into the first FFT pass and of the persistent search, bit for bit,
and agree with the oracle."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note, sample_bins
from tests.test_gpu_fused import same_bits

pytestmark = pytest.mark.gpu

NF = 2 ** 12
L = 4 * NF
COUNTS = [23, 24, 25, 47, 48, 49, 1, 0, 191, 192, 193, 383, 384, 385, 767, 768, 769, 3, 499, 501,
          749, 751, 999, 1001, 1499, 1501, 2100]


def _curve(rng, counts, kinds, cells):
    """Times in units of harmonic 1's cells, `counts` points in every 64 cells, spread over `cells`."""
    step = max(64, (int(cells) - 64) // max(1, len(counts) - 1) // 64 * 64)
    per = []
    for b, n in enumerate(counts):
        kind = kinds[b % len(kinds)]
        if kind == "cells":
            at = rng.integers(0, 64, n).astype(float)
        elif kind == "halves":
            at = rng.integers(0, 128, n) * 0.5
        elif kind == "one":
            at = 17.0 + 1e-3 * rng.uniform(0, 1, n)
        else:
            at = rng.uniform(0, 64, n)
        per.append(b * step + at)
    t = np.sort(np.concatenate([[0.0]] + per))
    s = rng.uniform(0.05, 0.3, t.size)
    return t, 0.02 * np.sin(t * 0.11) + s * rng.standard_normal(t.size), s


@pytest.mark.parametrize("H,width,wrap,precision", [
    (3, 0, False, "mixed"), (4, 0, True, "mixed"), (3, 1, False, "mixed"), (3, 7, False, "mixed"),
    (1, 9, True, "fp64"), (2, 4, False, "fp64"), (3, 16, True, "fp64"), (2, 0, False, "fp64")])
def test_dense_strips_identical_to_fused_and_match_the_oracle(H, width, wrap, precision):
    import torch
    rng = np.random.default_rng(100 * H + width)
    f_max = float(NF)  # one cell of harmonic 1 is 1 / L of a time unit
    cells = (1.7 if wrap else 0.85) * L / (2 * H)  # harmonic 2H ends past or within one period
    kinds = [["any"], ["cells", "any", "halves"], ["one", "any"]]
    per = [_curve(rng, list(rng.permutation(COUNTS)) if i else COUNTS, kinds[i % 3], cells)
           for i in range(3)]
    per.append(tuple(v[:40] for v in _curve(rng, [40], ["any"], 64)))  # one that stays sparse
    per = [(t / L, x, s) for t, x, s in per]
    off = np.concatenate([[0], np.cumsum([len(c[0]) for c in per])])
    dev = [torch.from_numpy(np.concatenate([c[i] for c in per])).cuda() for i in range(3)]
    outs = []
    for mode in ("staged", "fused_spread", "persistent"):
        if mode == "persistent" and precision == "fp64":
            continue  # mixed plans only
        note(f"dense strips H {H} w {width} wrap {wrap} {precision} {mode}")
        kw = {} if mode == "staged" else {mode: True}
        plan = F.Plan(off, f_max, H, NF, precision=precision, kernel_width=width, **kw)
        assert all(plan.info()[k] for k in kw)
        d, c0, fl = plan.search(*dev)
        torch.cuda.synchronize()
        outs.append([v.cpu() for v in (d, c0, fl)])
        plan.close()
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert same_bits(a, b)
    if width in (0, 16):
        bins = sample_bins(NF, 40, 9)
        fr = bins * (f_max / NF)
        kmax, tol = (1e2, 1e-5) if precision == "mixed" else (1e6, 1e-8)
        for c in (0, 1):
            ref = ora.dchi2(*per[c], fr, H)
            gate = ora.gate_mask(ref, fr, kmax)
            err = ora.rel_err(outs[0][0][c].double().numpy()[:, bins], ref["dchi2"])[:, gate]
            assert err.size == 0 or err.max() <= tol, err.max()


def test_dense_curves_spend_little_on_the_spreading():
    """400 curves of 640 points on 2^10 bins, six points a cell in the first harmonic:
    with strips alone the spreading took three times what the moments, the FFT and
    the solve take together (a tile of 1024 cells per workgroup: half as much again):
    less than 2.4 times, the fastest of eight."""
    import torch
    nf, H, n, nc, span = 2 ** 10, 4, 640, 400, 100.0
    rng = np.random.default_rng(1)
    t = np.sort(rng.uniform(0.0, span, (nc, n)), axis=1).ravel()
    dev = [torch.from_numpy(v).cuda() for v in (t, rng.normal(size=n * nc), np.ones(n * nc))]
    plan = F.Plan(np.arange(nc + 1) * n, 0.2 * nf / (2 * H * span), H, nf, precision="mixed")
    note("dense strips: spreading time of 400 curves")
    plan.search(*dev)
    best = {}
    for _ in range(8):
        plan.profile(True)
        plan.search(*dev)
        for stage, (ms, _) in plan.profile_read().items():
            best[stage] = min(best.get(stage, ms), ms)
        plan.profile(False)
    plan.close()
    spread = best.pop("spread")
    assert spread < 2.4 * sum(best.values()), (spread, best)
