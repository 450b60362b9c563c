"""Setup and pruning on the device at the sizes where their work units end:
checks of the pattern in units of 2048 entries, the transpose, the sampled link
blocks of the binned layout, and the row widths of the pruning kernels.  All
integer data: equality, and errors exactly where the definition has them."""
import numpy as np
import pytest

from oracle import prune as orc_prune
from paper_2509_10722_amd import instances as I
from tests.gpu_util import host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import (PMP_LAYOUT_BINNED, PMP_LAYOUT_GATHER,  # noqa: E402
                                      PMPError, Solver)


def _rows(m, n, lengths, seed=3):
    """Links with the given numbers of streams (distinct, ascending)."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n, int(k), replace=False)) for k in lengths]
    row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    col_idx = (np.concatenate(cols) if cols else np.zeros(0)).astype(np.int32)
    return I.Instance("s", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 2, n).astype(np.uint8), 0.0, 20.0)


def _with(inst, col_idx, row_ptr=None):
    return I.Instance("s", inst.m, inst.n, inst.row_ptr if row_ptr is None else row_ptr, col_idx, inst.c, inst.w,
                      inst.utility, inst.lo, inst.hi)


# (n, row lengths): units of one entry less, exactly one, one more; empty rows
# at the start, the end and around a unit's border; a row over several units
UNITS = [(3000, [2047]), (3000, [2048, 5]), (3000, [2049, 1]),
         (700, [0, 0, 600, 600, 600, 248, 0, 0, 0, 5, 0]),
         (9000, [3, 8500, 0, 1, 2000, 41, 0])]


@pytest.mark.parametrize("n,lengths", UNITS)
def test_pattern_units(n, lengths):
    inst = _rows(len(lengths), n, lengths)
    s = Solver(inst, dtype=torch.float64)
    s.iterate(5)
    _, lam, _ = s.solution()
    # path prices are R^T lambda: the transpose in order, to FP64 rounding
    lam, pi = host(lam), host(s.path_prices())
    ref = np.zeros(inst.n)
    row = np.repeat(np.arange(inst.m), lengths)
    np.add.at(ref, inst.col_idx, lam[row])
    assert np.abs(pi - ref).max() <= 2 ** -52 * inst.m * max(1.0, np.abs(ref).max())
    s.close()


@pytest.mark.parametrize("n,lengths", UNITS)
@pytest.mark.parametrize("where", ["first", "border", "last"])
def test_pattern_errors_at_unit_borders(n, lengths, where):
    good = _rows(len(lengths), n, lengths)
    nnz = int(good.row_ptr[-1])
    k = {"first": 1, "border": min(2048, nnz - 1), "last": nnz - 1}[where]
    inside = k not in set(int(p) for p in good.row_ptr)
    # an entry equal to the one before it: refused inside a row, and fine where
    # a row begins (descending columns across rows are the ordinary case)
    col = good.col_idx.copy()
    if inside:
        col[k] = col[k - 1]
        with pytest.raises(PMPError):
            Solver(_with(good, col), dtype=torch.float64)
    for bad in (-1, n):
        col = good.col_idx.copy()
        col[k] = bad
        with pytest.raises(PMPError):
            Solver(_with(good, col), dtype=torch.float64)
    ptr = good.row_ptr.copy()
    ptr[0] = 1                      # (nnz is the last pointer)
    with pytest.raises(PMPError):
        Solver(_with(good, good.col_idx, ptr), dtype=torch.float64)


@pytest.mark.parametrize("m,hot", [(65536, 0), (65537, 0), (131073, 0), (140001, 3000)])
def test_sampled_link_blocks(m, hot):
    """Link blocks cut at every step-th row from 65537 links on: FP32 sums are
    exact in FP64, so the binned iterates equal the gather layout's."""
    rng = np.random.default_rng(8)
    n = 30011
    link, stream = I.random_routes(rng, m - 5, rng.integers(6, 12, n))
    pairs = np.stack([link, stream], 1)
    if hot:                                   # dense rows: blocks of few rows
        extra = np.stack([np.repeat(np.arange(20), hot), np.tile(np.arange(hot), 20)], 1)
        pairs = np.unique(np.concatenate([pairs, extra]), axis=0)
    row_ptr, col_idx = I.csr_from_pairs(m, n, pairs[:, 0], pairs[:, 1])
    inst = I.Instance("s", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 2, n).astype(np.uint8), 0.0, 20.0)
    a = Solver(inst, dtype=torch.float32, layout=PMP_LAYOUT_BINNED)
    b = Solver(inst, dtype=torch.float32, layout=PMP_LAYOUT_GATHER)
    for s in (a, b):
        s.iterate(13)
    for p, q in zip(a.solution(), b.solution()):
        assert torch.equal(p, q)


@pytest.mark.parametrize("mean", [3, 40])
def test_prune_row_widths(mean):
    """Eight lanes a row and a wave a row, rows of 0, 1, 7, 8, 9, 63, 64, 65 and
    200 streams among them."""
    rng = np.random.default_rng(2)
    m, n = 500, 40000
    lengths = rng.integers(0, 2 * mean + 1, m)
    lengths[:9] = [0, 1, 7, 8, 9, 63, 64, 65, 200]
    inst = _rows(m, n, lengths)
    failed = (rng.random(m) < 0.1).astype(np.uint8)
    failed[:9] = 0
    s = Solver(inst, dtype=torch.float64)
    s.iterate(3)
    p, lmap, smap = s.prune(failed)
    ref = orc_prune.prune(inst, failed)
    got = p.instance
    for name in ("row_ptr", "col_idx", "utility"):
        assert np.array_equal(getattr(got, name).cpu().numpy(), ref[name]), name
    assert np.array_equal(lmap.cpu().numpy(), ref["link_map"])
    assert np.array_equal(smap.cpu().numpy(), ref["stream_map"])
