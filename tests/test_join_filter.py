"""The threshold join's filter as its tiles compute it: FP32 accumulators that
start at minus the candidate's Gram term, take the 32 products of the fp16
operands (the last two carry the query's term) and keep a pair iff their sign is
clear.  Modelled in numpy around the library's own term (its margins are in
there), at pairs that lie exactly on the threshold."""
import numpy as np
import pytest

F = np.float32


def on_the_threshold(m, spread, norm, rng, pairs=400):
    """fp16 vectors of norm about norm * m / sqrt 2, `spread` of that apart, and
    the metadata of windows whose true features are just Tr apart: the errors e'
    lie along the difference, so R = |G_q - G_c|."""
    from paper_2607_17481_amd import pmp
    L = pmp.lib()
    G = rng.standard_normal((2, pairs, 30)) * np.geomspace(1.0, 1e-2, 30)
    G[0] *= norm * m / np.sqrt(2.0) / np.linalg.norm(G[0], axis=1, keepdims=True)
    G[1] = G[0] + spread * m / np.sqrt(60.0) * rng.standard_normal((pairs, 30))
    G = np.where(np.abs(G) < 2.0 ** -14, 0.0, G).astype(np.float16).astype(np.float64)
    d = np.linalg.norm(G[0] - G[1], axis=1)
    e = (0.2 * d).astype(F).astype(np.float64)
    n2 = (G ** 2).sum(2)
    gn = (np.sqrt(n2[0]) * (1 + 1e-12)).astype(F) * F(1 + 2.4e-7)
    v = np.array([L.pmp_join_filter_term(m, d[x] - 2 * e[x], F(n2[0, x]), F(e[x]), gn[x], F(e[x]))
                  for x in range(pairs)])
    bare = 0.5 * (d * d - n2[0])                   # the same without a margin
    return L, G, n2, v, bare


def keeps(L, m, G, n2, v, order):
    """Which pairs the accumulators keep, their products added in `order`."""
    c = F(L.pmp_join_scale(m))
    x = np.clip(v / float(c), -60000.0, 60000.0).astype(F)
    hi = x.astype(np.float16).astype(F)
    lo = x - hi
    hi = np.where(np.abs(hi) < F(2.0 ** -14), F(0), hi)
    lo = np.where(np.abs(lo) < F(2.0 ** -14), F(0), lo).astype(np.float16).astype(F)
    q = np.concatenate([G[0].astype(F), hi[:, None], lo[:, None]], axis=1)
    k = np.concatenate([G[1].astype(F), np.full((len(v), 2), c, F)], axis=1)
    term = (0.5 * n2[1].astype(F).astype(np.float64) * (1.0 - 2.0 ** -23)).astype(F)
    acc = F(0) - np.abs(term)
    for s in order:
        acc = (acc + (q[:, s] * k[:, s]).astype(F)).astype(F)
    return ~np.signbit(acc)


ORDERS = [np.arange(32), np.arange(32)[::-1], np.concatenate([np.arange(30, 32), np.arange(30)])]


@pytest.mark.parametrize("m", [3, 12, 100, 400, 2048])
@pytest.mark.parametrize("spread", [0.0, 1e-4, 1e-2, 0.3])
@pytest.mark.parametrize("norm", [0.05, 0.7, 1.0])
def test_pairs_on_the_threshold_are_kept(m, spread, norm):
    """Norms up to the largest |F| = m / sqrt 2 at radii down to 0, where the
    start value dominates the rounding."""
    L, G, n2, v, _ = on_the_threshold(m, spread, norm, np.random.default_rng(m))
    for order in ORDERS:
        assert keeps(L, m, G, n2, v, order).all()


@pytest.mark.parametrize("m", [100, 400, 2048])
def test_the_margin_is_needed(m):
    """The same pairs without the term's margins, or with them subtracted: the
    model rejects some, so the test above can fail."""
    L, G, n2, v, bare = on_the_threshold(m, 1e-2, 1.0, np.random.default_rng(m))
    assert (v > bare).all()
    assert not all(keeps(L, m, G, n2, bare, order).all() for order in ORDERS)
    assert not keeps(L, m, G, n2, 2.0 * bare - v, ORDERS[0]).any()


@pytest.mark.parametrize("m", [3, 100, 2048])
def test_filter_still_rejects(m):
    """Pairs well past the threshold are rejected: half their distance as the
    radius."""
    from paper_2607_17481_amd import pmp
    L, G, n2, _, _ = on_the_threshold(m, 0.3, 0.7, np.random.default_rng(m))
    d = np.linalg.norm(G[0] - G[1], axis=1)
    v = np.array([L.pmp_join_filter_term(m, 0.5 * d[x], F(n2[0, x]), F(1e-3), F(np.sqrt(n2[0, x])), F(1e-3))
                  for x in range(len(d))])
    assert pmp.lib() is L
    assert not keeps(L, m, G, n2, v, ORDERS[0]).any()
