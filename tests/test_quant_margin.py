"""The 16-bit prefilter's grant for its FP32 arithmetic (no GPU needed)."""
import numpy as np
import pytest

from paper_2607_17481_amd import synth

F = np.float32


@pytest.mark.parametrize("kind", ["ecg", "walk", "far", "spikes"])
@pytest.mark.parametrize("m", [16, 100, 575, 2048])
def test_fp32_evaluation_stays_within_its_grant(kind, m):
    """Of delta = (2^-16 (1 + 1e-4) + 2^-21) max|t - c| / sigma a window, the second
    term covers the FP32 factors and the FP32 evaluation of a difference: counted
    out, six units of 2^-24 on one side and seven on the other of the eight that
    it grants each."""
    rng = np.random.default_rng(m)
    t = synth.ecg_like(9000, 3) if kind in ("ecg", "spikes") else np.cumsum(rng.standard_normal(9000))
    if kind == "far":
        t = t * 1e-3 + 1e6
    if kind == "spikes":
        t[rng.choice(9000, 20)] += 1e3
    at = rng.choice(len(t) - m + 1, 200, replace=False)
    w = np.stack([t[a:a + m] for a in at])
    mu, isg = w.mean(1)[:, None], 1.0 / w.std(1)[:, None]
    c = 0.5 * t.min() + 0.5 * t.max()
    h = max(t.max() - c, c - t.min())
    x = np.rint((w - c) / h * 32767.0)
    a, z = (h * isg / 32767.0).astype(F), ((c - mu) * isg).astype(F)
    i, j = slice(0, None, 2), slice(1, None, 2)
    b = z[i] - z[j]                                                # FP32
    # fused products and sums: exact in FP64, rounded once
    inner = (-x[j] * a[j].astype(np.float64) + b.astype(np.float64)).astype(F)
    e = (x[i] * a[i].astype(np.float64) + inner.astype(np.float64)).astype(F)
    # the same of the quantized samples without rounding
    q = (x * h / 32767.0 + (c - mu)) * isg
    err = np.abs(e.astype(np.float64) - (q[i] - q[j]))
    unit = 2.0 ** -24 * h
    assert (err <= unit * (6.0 * isg[i] + 7.0 * isg[j]) * (1 + 1e-4)).all()
    assert (err <= 2.0 ** -21 * h * (isg[i] + isg[j])).all()
