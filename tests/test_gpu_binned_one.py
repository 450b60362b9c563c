"""Binned passes of one workgroup per CU against the gather layout, where their
registers and LDS run out: blocks of more entries than a lane's first groups
and than the indices kept in LDS, more rows than a lane loads ahead, long links
(summed in fixed point in FP32), links and streams without entries.  FP32 sums
are exact in FP64 (or in fixed point): bit equality; FP64 sums differ in their
order only (1e-12 over a short run)."""
import numpy as np
import pytest

from paper_2509_10722_amd import instances as I
from tests.gpu_util import host, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import (PMP_LAYOUT_BINNED, PMP_LAYOUT_GATHER,  # noqa: E402
                                      Solver)


def _instance(m, n, lo, hi, long_streams=0, hot_links=0, seed=6):
    """Streams of lo..hi links; the first long_streams on every third link, the
    first hot_links on every second stream; the last links unused."""
    rng = np.random.default_rng(seed)
    link, stream = I.random_routes(rng, m - 2, rng.integers(lo, hi + 1, n))
    keep = stream != n - 1
    pairs = [np.stack([link[keep], stream[keep]], 1)]
    every3, every2 = np.arange(0, m - 2, 3), np.arange(0, n - 1, 2)
    if long_streams:
        pairs.append(np.stack([np.tile(every3, long_streams), np.repeat(np.arange(long_streams), every3.size)], 1))
    if hot_links:
        pairs.append(np.stack([np.repeat(np.arange(hot_links), every2.size), np.tile(every2, hot_links)], 1))
    pairs = np.unique(np.concatenate(pairs), axis=0)
    row_ptr, col_idx = I.csr_from_pairs(m, n, pairs[:, 0], pairs[:, 1])
    return I.Instance("one", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 3, n).astype(np.uint8), 0.0, 20.0)


CASES = [
    (15800, 1023, 2, 5, 4, 0),          # a stream block of 21000 entries: past the groups and the kept indices
    (3000, 30011, 1, 3, 0, 2),          # long links alone in their blocks
    (1100000, 20000, 3, 6, 0, 0),       # more than four rows a lane on the link side
    (20000, 540000, 1, 2, 0, 0),        # more than two on the stream side
    (300, 257, 1, 4, 0, 0),             # blocks of one or two rows
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("case", CASES)
def test_one_workgroup_passes(case, dtype):
    inst = _instance(*case)
    a = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_BINNED)
    b = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_GATHER)
    for k in (7, 23):                                # a checked pass after plain ones, and plain ones after it
        for s in (a, b):
            s.iterate(k)
        for p, q in zip(a.solution(), b.solution()):
            if dtype == torch.float32:
                assert torch.equal(p, q)
            else:
                assert rel(host(p), host(q)) <= 1e-12
        ra, rb = a.residuals(), b.residuals()
        assert abs(ra[0] - rb[0]) <= 1e-9 * abs(rb[0]) and abs(ra[1] - rb[1]) <= 1e-9 * abs(rb[1])
