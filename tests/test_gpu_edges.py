"""GPU kernels at the sizes where their tiling changes: tile and block edges,
remainders, the smallest and largest of a range (against the CPU oracle; the
bars of test_gpu_parity.py)."""
import numpy as np
import pytest

from paper_2607_17481_amd import synth
from tests import parity
from tests.test_gpu_parity import PRECS, gpu, run, ws  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def check(gpu, ws, oracle, t, lo, hi, excl, k=20, **opt):  # noqa: F811
    rows = oracle.pan_profile(t, range(lo, hi + 1), excl)
    res, st = run(gpu, ws, t, lo, hi, excl, k, **opt)
    ok, msg = parity.check_topk(res, rows, k, oracle, t, excl=excl)
    assert ok, msg
    return st


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("repeat", [False, True])
@pytest.mark.parametrize("windows", [31, 127, 128, 129, 513, 1025])
def test_join_blocks(gpu, ws, oracle, windows, repeat, prec):  # noqa: F811
    """The threshold join's blocks of 128 queries and tiles of 32 candidates:
    one below, at and above a block; with an exact repeat (cells at 0 are not
    queries, so a block also scans the candidates before its first query) and
    without (it skips them)."""
    lo, hi, excl = 12, 14, 6
    n = windows + lo - 1
    t = np.cumsum(np.random.default_rng(windows).standard_normal(n))
    if repeat:
        t[n - 16:n - 1] = t[2:17] + 3.0
    check(gpu, ws, oracle, t, lo, hi, excl, precision=PRECS[prec], anchor_stride=2)


@pytest.mark.parametrize("prec", ["fp64", "bf16"])
@pytest.mark.parametrize("windows", [2, 7, 8, 9, 17, 64, 65])
def test_probe_groups(gpu, ws, oracle, windows, prec):  # noqa: F811
    """The probe's wavefronts of eight queries with eight lanes each: fewer
    queries than one wavefront takes, one below, at and above a multiple; flat
    stretches keep the windows of a wavefront apart (they are then read from
    the series, not from the staged copy)."""
    lo, hi, excl = 8, 9, 1
    n = windows + lo - 1
    t = np.random.default_rng(windows).standard_normal(n)
    check(gpu, ws, oracle, t, lo, hi, excl, k=5, precision=PRECS[prec])
    gaps = np.concatenate([np.concatenate([t, np.full(200, t[-1])]), t * 0.5 + 1.0])
    check(gpu, ws, oracle, gaps, lo, hi, excl, k=5, precision=PRECS[prec])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("windows", [8192, 8193, 32768, 32769])
def test_probe_teams(gpu, ws, oracle, windows, prec):  # noqa: F811
    """The probe's 64, 32 and 16 lanes per query: at and one past the largest
    launch of the first two."""
    m, excl = 8, 4
    t = np.random.default_rng(windows).standard_normal(windows + m - 1)
    check(gpu, ws, oracle, t, m, m, excl, precision=PRECS[prec])


@pytest.mark.parametrize("stride", [1, 16])
@pytest.mark.parametrize("lo", [3, 4, 17])
@pytest.mark.parametrize("windows", [5, 1023, 1024, 1026, 2049])
def test_moment_quads(gpu, ws, oracle, windows, lo, stride):  # noqa: F811
    """Moments of four windows a thread: windows of 3 samples and of every
    remainder, the last window in each place of its quad and tile, and flat
    stretches that leave one to three windows of a quad."""
    t = np.random.default_rng(windows + lo).standard_normal(windows + lo + 2)
    for a, w in ((37, lo), (90, lo + 1), (151, lo + 5), (700, 2 * lo + 3)):
        t[a:a + w] = t[a:a + 1] if a < len(t) else 0.0
    check(gpu, ws, oracle, t, lo, lo + 3, lo, k=5, anchor_stride=stride)


@pytest.mark.parametrize("lengths", [255, 256, 257, 600])
def test_many_lengths(gpu, ws, oracle, lengths):  # noqa: F811
    """Tables of more lengths than one launch's arguments or one block of
    lengths hold."""
    lo, excl = 8, 20
    t = np.cumsum(np.random.default_rng(lengths).standard_normal(lengths + 60))
    check(gpu, ws, oracle, t, lo, lo + lengths - 1, excl)


_LARGE_ROWS: dict = {}


@pytest.mark.parametrize("prec,stride", [("fp64", 16), ("fp32", 16), ("fp64", 1)])
@pytest.mark.parametrize("kind", ["ecg", "walk", "far", "tiny"])
def test_prefiltered_requests(gpu, ws, oracle, kind, prec, stride):  # noqa: F811
    """Requests of more than 2^20 windows, whose exact distances stand behind
    the 16-bit prefilter: a noisy series (nearly every pair ends there), a
    random walk (window spreads far below the series' range, so most pairs
    pass by it), the noisy series on a far offset and scaled by 2^-400."""
    if kind == "walk":
        t = np.cumsum(np.random.default_rng(4).standard_normal(27001))
    else:
        t = synth.ecg_like(27001, 9)
        if kind == "far":
            t = t * 3.0 + 1e5
    lo, hi, excl = 61, 100, 50
    ref = "ecg" if kind == "tiny" else kind       # an exact scaling keeps every distance
    if ref not in _LARGE_ROWS:
        _LARGE_ROWS[ref] = oracle.pan_profile_v2(t, range(lo, hi + 1), excl)
    if kind == "tiny":
        t = t * 2.0 ** -400
    res, st = run(gpu, ws, t, lo, hi, excl, precision=PRECS[prec], anchor_stride=stride)
    assert st["indexed_cells"] > 1 << 20
    ok, msg = parity.check_topk(res, _LARGE_ROWS[ref], 20, oracle, t, excl=excl)
    assert ok, msg


@pytest.mark.parametrize("lo,hi,k", [(8, 9, 1), (8, 9, 128), (8, 9, 129), (110, 111, 128),
                                     (111, 112, 128)])
@pytest.mark.parametrize("kind", ["walk", "tied", "short"])
def test_selection_forms(gpu, ws, oracle, kind, lo, hi, k):  # noqa: F811
    """The greedy on the device and, for more than 128 motifs or 14336 cells, on
    the host; distances that differ, that fall on a few equal values (a series
    of two levels) and fewer cells than motifs."""
    rng = np.random.default_rng(k + hi)
    n = 3000 if kind != "short" else 2 * hi
    t = np.cumsum(rng.standard_normal(n))
    if kind == "tied":
        t = np.sign(rng.standard_normal(n))
    check(gpu, ws, oracle, t, lo, hi, 5, k=k)


@pytest.mark.parametrize("n,lo,hi", [(2055, 8, 8), (2056, 8, 8), (16383, 16, 17), (16384, 16, 17),
                                     (20000, 41, 70)])
def test_scan_and_sort_sizes(gpu, ws, oracle, n, lo, hi):  # noqa: F811
    """Scans of one block (to 16384 entries) and of three kernels; sorts of one
    full tile and one key more, of several blocks that the histogram's last
    block scans, and of more than those (the join's 599,000 keys)."""
    t = np.cumsum(np.random.default_rng(n).standard_normal(n))
    rows = oracle.pan_profile_v2(t, range(lo, hi + 1), lo)
    res, _ = run(gpu, ws, t, lo, hi, lo)
    ok, msg = parity.check_topk(res, rows, 20, oracle, t, excl=lo)
    assert ok, msg


@pytest.mark.parametrize("kind", ["walk", "noise", "flat", "few"])
def test_width_matches_the_host(gpu, ws, kind):  # noqa: F811
    """The spectral width chosen on the device equals the host's: smooth and
    white series, constant windows among the samples, fewer windows than
    samples."""
    rng = np.random.default_rng(5)
    t = rng.standard_normal(3000)
    if kind != "noise":
        t = np.cumsum(t)
    if kind == "flat":
        t[500:1500] = 0.1
    if kind == "few":
        t = t[:150]
    _, st = run(gpu, ws, t, 20, 100, 10, 5)
    assert st["K"] == gpu.calibrate_width(t, 20, 100)


@pytest.mark.parametrize("batch,n", [(64, 5000), (63, 700), (1300, 5200)])
def test_stream_every_pair(gpu, oracle, batch, n):  # noqa: F811
    """A budget that takes in every earlier window: the profile is then exact.
    Turns of 64 candidates with remainders, merges in one block and of more
    entries than it holds (4096), and batches of more windows than it has
    threads (1024)."""
    m, excl = 32, batch
    t = np.cumsum(np.random.default_rng(batch).standard_normal(n))
    with gpu.Stream(n, m, m, 5, excl, budget=n, batch=batch, opts=gpu.options(gamma=1)) as s:
        s.append(t)
        s.flush()
        assert s.info()["dropped"] == 0
        P, _ = s.profile(0)
    ref = oracle.profile(t, m, excl)[0]
    assert len(P) == len(ref)
    for q, (a, b) in enumerate(zip(P, ref)):
        assert parity.dist_close(float(a), float(b)), (q, a, b)


def test_open_memory_is_reused(gpu, oracle):  # noqa: F811
    """pmp_open calls of growing, shrinking and equal sizes, overlapping ones
    from several threads, and after pmp_trim: every answer is the same as
    with fresh memory."""
    from concurrent.futures import ThreadPoolExecutor
    series = {n: np.cumsum(np.random.default_rng(n).standard_normal(n)) for n in (300, 2000, 900)}
    want = {n: oracle.topk(oracle.pan_profile(t, range(16, 25), 8), 5) for n, t in series.items()}

    def one(n):
        res = gpu.open_host(series[n], 16, 24, 5, 8)
        ok, msg = parity.canonical_equal(res, want[n])
        assert ok, (n, msg)

    for n in (300, 2000, 900, 900, 300):
        one(n)
    with ThreadPoolExecutor(4) as ex:
        list(ex.map(one, [300, 2000, 900, 2000] * 3))
    gpu.trim()
    gpu.trim()
    one(900)
