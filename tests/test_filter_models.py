"""The threshold join's fp16 filter and the 16-bit prefilter of exact
distances, modelled in numpy from their definitions: neither may reject a pair
within the threshold, whatever the scale of the series."""
import numpy as np
import pytest

from paper_2607_17481_amd import synth


def windows(t, m, count, rng):
    i = rng.choice(len(t) - m + 1, count, replace=False)
    x = np.stack([t[a:a + m] for a in i])
    return x, x.mean(1), x.std(1)


def series(kind, rng):
    if kind == "ecg":
        return synth.ecg_like(6000, 3)
    t = np.cumsum(rng.standard_normal(6000))
    return t * 1e-3 + 1e6 if kind == "far" else t


@pytest.mark.parametrize("kind", ["ecg", "walk", "far"])
@pytest.mark.parametrize("m", [3, 17, 64, 65, 250])
def test_quantized_sum_never_rejects(kind, m):
    """S >= (thr + sqrt(m) (delta_i + delta_j))^2 (1 + 2e-4) implies d > thr,
    for thr at the pair's own distance (the tightest case)."""
    rng = np.random.default_rng(m)
    t = series(kind, rng)
    x, mu, sg = windows(t, m, 120, rng)
    c = 0.5 * t.min() + 0.5 * t.max()
    half = max(t.max() - c, c - t.min()) * (1 + 1e-12)
    q = np.rint((x - c) / half * 32767.0).astype(np.int16)
    f = np.float32
    a = (half / sg / 32767.0).astype(f)
    b = ((c - mu) / sg).astype(f)
    delta = (2.0 ** -16 * (1 + 1e-4) + 2.0 ** -21) * half / sg
    z = (x - mu[:, None]) / sg[:, None]
    for i in range(0, 120, 2):
        d = np.sqrt(((z[i] - z[i + 1]) ** 2).sum())
        e = q[i].astype(f) * a[i] - q[i + 1].astype(f) * a[i + 1] + f(b[i] - b[i + 1])
        s = float((e * e).sum(dtype=f))
        lim = (d + np.sqrt(m) * (delta[i] + delta[i + 1])) ** 2 * (1 + 2e-4)
        assert s < lim, (kind, m, i)


@pytest.mark.parametrize("m", [12, 100, 400, 2048])
def test_fp16_vectors_never_reject(m):
    """<G_q, G_c> + v >= 0.5 |G_c|^2 for every pair whose true features lie
    within Tr, with the filter term v split over two fp16 slots of scale c."""
    rng = np.random.default_rng(m)
    nmax = m / np.sqrt(2.0) * 1.01 + 1.0
    c = 1.0
    while 32768.0 * c < 2.5 * (0.5 * m * m * 1.03 + 2.0 * m + 2.0):
        c *= 2.0
    for spread in (1e-5, 1e-3, 0.05, 0.5):
        F = rng.standard_normal((2, 200, 30)) * np.geomspace(1.0, 1e-3, 30)
        F[1] = F[0] + spread * rng.standard_normal((200, 30))
        F *= (m / np.sqrt(2.0)) * rng.uniform(0.05, 0.99, (1, 200, 1)) / np.linalg.norm(F, axis=2, keepdims=True)
        G = np.where(np.abs(F) < 2.0 ** -14, 0.0, F).astype(np.float16).astype(np.float64)
        e = np.linalg.norm(G - F, axis=2)
        Tr = np.linalg.norm(F[0] - F[1], axis=1)          # the pair's own radius
        n2 = (G ** 2).sum(2)
        R = (Tr + e[0] + e.max()) * (1 + 1e-9)
        v = 0.5 * (R * R * (1 + 1e-9) - n2[0].astype(np.float32) * (1 - 2.0 ** -23))
        v += 1.6e-5 * nmax * np.sqrt(n2[0]) + 1e-30
        v += 2.0 ** -22 * (np.abs(v) + nmax * nmax)
        v += 5e-6 * np.abs(v) + 2.0 ** -12 * c
        x = np.clip(v / c, -60000.0, 60000.0).astype(np.float32)
        hi = x.astype(np.float16).astype(np.float32)
        lo = x - hi
        hi = np.where(np.abs(hi) < 2.0 ** -14, 0.0, hi)
        lo = np.where(np.abs(lo) < 2.0 ** -14, 0.0, lo).astype(np.float16).astype(np.float32)
        acc = np.zeros(200, dtype=np.float32)             # FP32 sums, in order
        for k in range(30):
            acc += (G[0, :, k] * G[1, :, k]).astype(np.float32)
        acc += (hi * np.float32(c)).astype(np.float32)
        acc += (lo * np.float32(c)).astype(np.float32)
        term = (0.5 * n2[1].astype(np.float32) * (1 - 2.0 ** -23)).astype(np.float32)
        assert np.all(acc >= term), (m, spread)
