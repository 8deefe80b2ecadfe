"""Curves with observing gaps: the strip table's entries across a gap all belong
to the point after it and are stored by its whole wave.  Gaps of a few to hundreds
of strips (each harmonic stretches them), owned by the first and last lanes of a
wave, by a wave of the table's second workgroup, and running past a grid period,
against the oracle; the persistent search bit for bit against the staged one;
and the spreading of a gapped curve takes about as long as that of an even one."""
import numpy as np
import pytest

from oracle import fchi2_oracle as ora
from paper_0901_1913_amd import fchi2 as F
from tests.gpu_util import note, sample_bins
from tests.test_gpu_fused import same_bits

pytestmark = pytest.mark.gpu

NF, H, SPAN = 2 ** 12, 3, 50.0
TOL = {"fp64": (1e6, 1e-8), "mixed": (1e2, 1e-5)}  # gate and bound of the parity tests


def _curve(rng, owner, gap, n=600):
    """n points over SPAN, an empty stretch of `gap` SPANs before point `owner`."""
    t = np.sort(rng.uniform(0.0, SPAN * (1 - gap), n))
    t[0], t[-1] = 0.0, SPAN * (1 - gap)
    t[owner:] += gap * SPAN
    s = rng.uniform(0.05, 0.2, n)
    return t, 0.3 * np.sin(2 * np.pi * t * 11.0 / SPAN) + s * rng.standard_normal(n), s


@pytest.mark.parametrize("fill,precision", [(0.9, "fp64"), (2.7, "fp64"), (0.9, "mixed")])
def test_gapped_curves_match_the_oracle(fill, precision):
    import torch
    rng = np.random.default_rng(17)
    f_max = fill * NF / (2 * H * SPAN)
    # in strips of harmonic 1 (of 128 or 32 cells): fractions of one to half the span
    gaps = [(1, 0.02), (63, 0.05), (64, 0.11), (65, 0.2), (255, 0.3), (256, 0.5), (320, 0.21), (599, 0.45)]
    per = [_curve(rng, o, g) for o, g in gaps]
    off = np.concatenate([[0], np.cumsum([len(c[0]) for c in per])])
    t, x, s = (torch.from_numpy(np.concatenate([c[i] for c in per])).cuda() for i in range(3))
    bins = sample_bins(NF, 80, 3)
    fr = bins * (f_max / NF)
    outs = []
    for persistent in ((False, True) if precision == "mixed" else (False,)):
        note(f"gaps: fill {fill} {precision} persistent {persistent}")
        plan = F.Plan(off, f_max, H, NF, precision=precision, t_span=[SPAN] * len(per),
                      persistent=persistent)
        assert plan.info()["persistent"] == int(persistent)
        d, c0, fl = plan.search(t, x, s)
        torch.cuda.synchronize()
        outs.append([v.cpu() for v in (d, c0, fl)])
        plan.close()
    for u, v in zip(outs[0], outs[-1]):
        assert same_bits(u, v)
    kmax, tol = TOL[precision]
    for c, curve in enumerate(per):
        ref = ora.dchi2(*curve, fr, H)
        gate = ora.gate_mask(ref, fr, kmax)
        err = ora.rel_err(outs[0][0][c].double().numpy()[:, bins], ref["dchi2"])[:, gate]
        assert err.size and err.max() <= tol, (gaps[c], err.max())


def test_a_gap_does_not_slow_the_spreading():
    """300 points on 2^22 bins, a third of the span empty or none (one lane storing
    the gap's entries takes seven times as long as the even curve): less than 2.5
    times, the fastest of eight."""
    import torch
    nf, n = 2 ** 22, 300
    rng = np.random.default_rng(5)
    ms = []
    for gap in (0.0, 1.0 / 3.0):
        t, x, s = _curve(rng, n // 2, gap, n)
        dev = [torch.from_numpy(v).cuda() for v in (t, x, s)]
        plan = F.Plan([0, n], 0.9 * nf / (2 * H * SPAN), H, nf, precision="mixed", t_span=[SPAN])
        note(f"gaps: spreading time, gap {gap:.2f}")
        plan.search(*dev)
        best = np.inf
        for _ in range(8):
            plan.profile(True)
            plan.search(*dev)
            best = min(best, plan.profile_read()["spread"][0])
            plan.profile(False)
        ms.append(best)
        plan.close()
    assert ms[1] < 2.5 * ms[0], ms
