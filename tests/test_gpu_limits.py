"""Calls at the edges of what one launch, one buffer or one allocation holds."""
import ctypes as C

import numpy as np
import pytest

from paper_2607_17481_amd import synth
from tests import parity
from tests.test_gpu_parity import PRECS, gpu, run, ws  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def test_probe_in_pieces(gpu):  # noqa: F811
    """A probe of more blocks than one launch takes (2^20, of eight queries):
    every length an anchor, so that the lengths after the first have 9 million
    queries; the same answer as with one anchor beside the first."""
    t = synth.ecg_like(600_000, 4)
    lo, hi, excl = 100, 115, 100
    own = gpu.Workspace("cuda:0")
    runs = [run(gpu, own, t, lo, hi, excl, 10, budget=4, anchor_stride=s) for s in (16, 1)]
    assert runs[1][1]["probe_queries"] - runs[1][1]["indexed_cells"] // 16 > 8 << 20
    assert runs[0][0] == runs[1][0]


def test_stream_probe_in_pieces(gpu, oracle):  # noqa: F811
    """A batch of more windows (51 anchors of 1,300) than one launch of the
    search takes (2^16), at a budget that takes in every earlier window: the
    profile of the last anchors, whose windows the second launch has, is exact."""
    lo, hi, batch, n = 20, 70, 1300, 3900
    t = np.cumsum(np.random.default_rng(batch).standard_normal(n))
    opts = gpu.options(gamma=1, anchor_stride=1)
    with gpu.Stream(n, lo, hi, 5, batch, budget=n, batch=batch, opts=opts) as s:
        s.append(t)
        s.flush()
        st = s.info()
        assert st["anchors"] == 51 and st["dropped"] == 0
        rows = {m: s.profile(m - lo)[0] for m in (lo, 69, 70)}
    for m, P in rows.items():
        ref = oracle.profile(t, m, batch)[0]
        assert len(P) == len(ref)
        for q, (a, b) in enumerate(zip(P, ref)):
            assert parity.dist_close(float(a), float(b)), (m, q, a, b)


@pytest.mark.parametrize("scale", [1e155, 1e-170])
@pytest.mark.parametrize("k", [1, 20])
def test_deviation_out_of_range_is_an_argument_error(gpu, ws, k, scale):  # noqa: F811
    """Windows whose variance overflows (or underflows) are refused as an
    argument error, also where their one-pass distances are far above every
    distance that the selection's keys tell apart."""
    rng = np.random.default_rng(6)
    t = scale * (np.sin(np.arange(3000) * (2 * np.pi / 60)) + 1e-5 * rng.standard_normal(3000))
    with pytest.raises(gpu.PMPError) as e:
        run(gpu, ws, t, 60, 64, 30, k)
    assert e.value.code == gpu.PMP_EINVAL


def test_kept_memory_is_given_back_when_an_allocation_fails(gpu):  # noqa: F811
    """pmp_open keeps a block of device memory.  A stream session, its exact
    query and a server give it back when there is no memory left for them, and
    go on; without a block to give back they fail."""
    import torch
    t = np.cumsum(np.random.default_rng(9).standard_normal(30_000))
    args = (32, 82, 5, 32)
    fail = gpu.lib().pmp_debug_fail_allocs
    block = gpu.workspace_bytes(len(t), 32, 82, 5)
    assert 400 << 20 < block < 1 << 30
    st = gpu.Stream(3000, *args)
    st.append(t[:3000])

    def free():
        return torch.cuda.mem_get_info(0)[0]

    calls = [lambda: gpu.Stream(3000, *args).close(), lambda: gpu.Server(0, 64 << 20, 1).close(),
             st.exact]
    for call in calls:
        gpu.open_host(t, *args, 16)
        a = free()
        fail(1)
        call()
        fail(0)
        assert free() - a > block // 2
    for call in calls[:2] + [lambda: gpu.open_host(t, *args, 16)]:
        fail(1)
        with pytest.raises(gpu.PMPError):
            call()
        fail(0)
    st.close()


def test_stream_batches_share_buffers_only_while_small(gpu):  # noqa: F811
    """The per-window buffers of a session follow its batch: a key, the margins,
    the list and the improvements of one batch, not of sixteen, once a batch
    fills a launch."""
    n, lo, budget = 60_000, 100, 1
    opts = gpu.options(gamma=8)
    held = []
    for batch in (20_000, 40_000):
        with gpu.Stream(n, lo, lo, 5, batch, budget=budget, batch=batch, opts=opts) as s:
            held.append(s.info()["device_bytes"])
    per_window = 8 * budget * 16 + 4 + 24 * 4 + 8
    assert held[1] - held[0] <= 20_000 * per_window + 4096


def join_blocks(gpu):  # noqa: F811
    again, in_place = C.c_int64(), C.c_int64()
    gpu.lib().pmp_debug_join_blocks(C.byref(again), C.byref(in_place))
    return again.value, in_place.value


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,lo,hi,fewest,most,shared", [
    # a few blocks, each with a segment of its own from the start: taken again
    # for nothing, then in place with many wavefronts to each
    (900, 40, 42, 1, 60, False),
    # forty blocks a segment, and more of them in place than half the wavefronts
    # of that launch: one wavefront each
    (6000, 30, 90, 1100, 10**9, True),
])
def test_overflowed_join_blocks(gpu, ws, oracle, n, lo, hi, fewest, most, shared, prec):  # noqa: F811
    """Blocks of the join that find their segment of the pair buffer full.  With
    one pair a segment they are verified in place; with room for a quarter of
    all pairs a segment holds several blocks' but not its forty's: those that
    overflowed are done when they are taken again."""
    excl, k = 20, 20
    t = np.cumsum(np.random.default_rng(n).standard_normal(n))
    rows = oracle.pan_profile_v2(t, range(lo, hi + 1), excl)
    join_blocks(gpu)
    res, st = run(gpu, ws, t, lo, hi, excl, k, precision=PRECS[prec])
    assert join_blocks(gpu) == (0, 0)
    ok, msg = parity.check_topk(res, rows, k, oracle, t, excl=excl)
    assert ok, msg
    dbg = gpu.Debug()
    dbg.size = C.sizeof(gpu.Debug)
    seen = []
    for cap in (1, st["join_candidates"] // 4):
        dbg.join_pair_cap = cap
        got, _ = run(gpu, ws, t, lo, hi, excl, k, debug=dbg, precision=PRECS[prec])
        assert got == res
        seen.append(join_blocks(gpu))
        print(cap, seen[-1])
    assert fewest <= seen[0][1] <= most
    if shared:
        assert seen[1][0] > seen[1][1]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("stride", [1, 16])
@pytest.mark.parametrize("fill", [1e9, 1e17, 1e18, 1e20, 1e25, 1e36, 1e100])
def test_windows_behind_a_fill_value(gpu, ws, oracle, fill, stride, prec):  # noqa: F811
    """A huge sample (a fill value of missing data) leaves the sliding DFT of the
    windows after it, up to the end of their segment of 64, with errors far
    above the features themselves, as their records' bounds say.  The best pairs
    lie just there: the certificate has to find them, whatever the value."""
    n, lo, hi, excl, k = 3000, 32, 33, 16, 3
    rng = np.random.default_rng(11)
    t = rng.standard_normal(n)
    # windows 1002 .. 1023, the last of the segment at 960, are near copies
    t[1002:1055] = t[2102:2155] + 0.02 * rng.standard_normal(53)
    t[1000] = fill
    rows = oracle.pan_profile(t, range(lo, hi + 1), excl)
    res, _ = run(gpu, ws, t, lo, hi, excl, k, budget=1, precision=PRECS[prec], anchor_stride=stride)
    assert {x.i // 100 for x in res} <= {10, 21} and res[0].dist < 0.5
    ok, msg = parity.check_topk(res, rows, k, oracle, t, excl=excl)
    assert ok, msg
