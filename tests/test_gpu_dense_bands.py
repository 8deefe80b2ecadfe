"""Band plans' dense strips are spread with a lane per cell, two runs of 64 cells a
wave: blocks of harmonic 1 around every count at which that is decided (48 points of
a wave's four strips, 2000 or 3000) and at which points are staged anew (384).  A
curve searched alone (strips of 32, by cells) and among 1500 curves of few points
(strips of 128) has the same bits, and agrees with the oracle."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note, sample_bins
from tests.test_gpu_dense_strips import COUNTS, _curve
from tests.test_gpu_fused import same_bits

pytestmark = pytest.mark.gpu

NF = 2 ** 12
L = 2 * NF  # a band plan's complex grids
BAND_COUNTS = COUNTS + [1101, 1999, 2001, 2999, 3001]


@pytest.mark.parametrize("H,width,wrap,precision", [
    (2, 0, False, "mixed"), (3, 0, True, "mixed"), (2, 5, False, "mixed"), (1, 7, True, "mixed"),
    (1, 9, True, "fp64"), (2, 4, False, "fp64"), (2, 16, True, "fp64"), (1, 0, False, "fp64")])
def test_dense_band_strips_identical_to_sparse_batch_and_match_the_oracle(H, width, wrap,
                                                                          precision):
    import torch
    rng = np.random.default_rng(10 * H + width)
    cells = (1.7 if wrap else 0.85) * L / (2 * H)  # harmonic 2H ends past or within one period
    kinds = (["any"], ["cells", "any", "halves"], ["one", "any"])[H - 1]
    t, x, s = _curve(rng, [int(c) for c in rng.permutation(BAND_COUNTS)], kinds, cells)
    few = [np.sort(rng.uniform(0.0, cells, 8)) for _ in range(1500)]
    per = [(t / L, x, s)] + [(f / L, rng.normal(size=8), np.ones(8)) for f in few]
    rows = []
    for curves in (per[:1], per):
        note(f"dense bands H {H} w {width} wrap {wrap} {precision}, {len(curves)} curves")
        off = np.concatenate([[0], np.cumsum([len(c[0]) for c in curves])])
        dev = [torch.from_numpy(np.concatenate([c[i] for c in curves])).cuda() for i in range(3)]
        plan = F.Plan(off, float(NF), H, NF, precision=precision, kernel_width=width,
                      first_bin=NF)
        d, c0, fl = plan.search(*dev)
        torch.cuda.synchronize()
        rows.append([v[:1].cpu() for v in (d, c0, fl)])
        plan.close()
    for a, b in zip(*rows):
        assert same_bits(a, b)
    if width in (0, 16):
        kk = sample_bins(NF, 40, 9, k_min=0)
        fr = NF + kk.astype(float)
        kmax, tol = (1e2, 1e-5) if precision == "mixed" else (1e6, 1e-8)
        ref = ora.dchi2(*per[0], fr, H)
        gate = ora.gate_mask(ref, fr, kmax)
        err = ora.rel_err(rows[0][0][0].double().numpy()[:, kk], ref["dchi2"])[:, gate]
        assert err.size == 0 or err.max() <= tol, err.max()


def test_dense_bands_spend_little_on_the_spreading():
    """300 curves of 3000 points, H = 5, a band of 2^13 bins, nineteen points a cell in
    the first harmonic: by strips alone the spreading took 2.9 times what the moments,
    the FFT and the solve take together (by a tile of 1024 cells per workgroup 1.2
    times): less than 2.2 times, the fastest of eight."""
    import torch
    nf, H, n, nc, span = 2 ** 13, 5, 3000, 300, 100.0
    rng = np.random.default_rng(1)
    t = np.sort(rng.uniform(0.0, span, (nc, n)), axis=1).ravel()
    dev = [torch.from_numpy(v).cuda() for v in (t, rng.normal(size=n * nc), np.ones(n * nc))]
    plan = F.Plan(np.arange(nc + 1) * n, 0.1 * nf / (2 * H * span), H, nf, precision="mixed",
                  first_bin=nf)
    note("dense bands: spreading time of 300 curves")
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
    assert spread < 2.2 * sum(best.values()), (spread, best)
