"""Calls at the edges of what one launch, one buffer or one allocation holds."""
import pytest

from paper_2607_17481_amd import synth
from tests.test_gpu_parity import gpu, run  # noqa: F401  (fixtures)

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
