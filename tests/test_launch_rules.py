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


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 64, 65, 100, 128, 129, 500, 1023, 1024, 1025,
                               5000])
def test_join_blocks_are_placed_over_the_chip(n):
    """Every block of a join launch is taken by one workgroup; workgroups go to
    the eight XCDs in turn and write to the segment of their number mod 64: a
    launch uses every XCD it has blocks for, evenly, up to 64 blocks have a
    segment each, and neighbours stay together on an XCD."""
    from paper_2607_17481_amd import pmp
    L = pmp.lib()
    groups = L.pmp_join_workgroups(n)
    at = {}
    for w in range(groups):
        b = L.pmp_join_block_of(n, w)
        assert -1 <= b < n
        if b >= 0:
            assert b not in at
            at[b] = w
    assert len(at) == n and groups < n + 8 * 128
    load = [0] * 8
    for w in at.values():
        load[w % 8] += 1
    run = min(128, -(-n // 8))
    assert max(load) - min(load) <= run and max(load) <= -(-n // (8 * run)) * run
    assert sum(x > 0 for x in load) == min(8, -(-n // run))
    segments = {w % 64 for w in at.values()}
    if n <= 64:
        assert len(segments) == n
    else:
        assert len(segments) > 48
    same = sum(at[b] % 8 == at[b + 1] % 8 for b in range(n - 1))
    assert same == n - 1 - (n - 1) // run
