"""Host rules that size and place launches (no GPU needed)."""
import pytest


@pytest.mark.parametrize("queries", [1, 8, 8192, 8193, 32768, 32769, 1 << 19, (1 << 19) + 1,
                                     1 << 23, 5 * 10**8, (1 << 29) + 1, (1 << 31) - 1])
def test_probe_launches_stay_below_the_limit(queries):
    """A launch takes fewer than 2^32 work-items.  At eight lanes a query one
    launch of more than 2^29 queries (11 million samples, 51 lengths, every
    length an anchor) would have more."""
    from paper_2607_17481_amd import pmp
    items = pmp.lib().pmp_probe_work_items(queries)
    assert 0 < items < 1 << 32
    assert items >= 8 * min(queries, 1 << 20)
