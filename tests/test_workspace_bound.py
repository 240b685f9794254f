"""The workspace bound (no GPU needed)."""
import pytest


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("stride,sieve", [(16, 0), (1, 8)])
def test_bound_never_falls_as_requests_grow(precision, stride, sieve):
    """A workspace of a size that a request is said to need holds every smaller
    request: one buffer for the largest serves them all.  Over the sizes where
    the buffers' rules change (2^20 cells: 20,634 samples at 51 lengths)."""
    from paper_2607_17481_amd import pmp
    o = pmp.options(precision=precision, anchor_stride=stride, sieve_width=sieve)

    def rising(sizes):
        got = [(pmp.workspace_bytes(*s[:3], k=s[3], opts=o), s) for s in sizes]
        assert all(b for b, _ in got)
        for (a, s), (b, r) in zip(got, got[1:]):
            assert a <= b, (s, a, r, b)

    rising([(n, 50, 100, 20) for n in range(20_000, 24_000, 7)])
    rising([(n, 50, 100, 20) for n in range(200, 200_000, 331)])
    rising([(int(100 * 1.13 ** x), 50, 50, 20) for x in range(100)])
    rising([(30_000, 50, hi, 20) for hi in range(50, 130)])
    rising([(21_000, 50, 100, k) for k in (1, 2, 20, 128, 129, 500)])
