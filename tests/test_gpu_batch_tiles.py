"""Batch tiles whose entries are clustered by the gathered index: sides of
exactly 2^19 rows (the last to be clustered) and of one more, tiles of exactly
8192 entries and of a remainder, an instance without entries.  Iterates equal
the one-at-a-time gather solves bit for bit, as the sums keep their order."""
import numpy as np
import pytest

from paper_2509_10722_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import (PMP_LAYOUT_GATHER, BatchSolver, Solver)  # noqa: E402


def _random(m, n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    link, stream = I.random_routes(rng, m, rng.integers(lo, hi + 1, n))
    row_ptr, col_idx = I.csr_from_pairs(m, n, link, stream)
    return I.Instance("t", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 2, n).astype(np.uint8), 0.0, 20.0)


def _full(m, n, seed):
    """Every stream on every link: m n entries in tiles of whole rows."""
    rng = np.random.default_rng(seed)
    row_ptr = (np.arange(m + 1) * n).astype(np.int32)
    return I.Instance("f", m, n, row_ptr, np.tile(np.arange(n, dtype=np.int32), m), rng.uniform(50, 90, m),
                      rng.uniform(0.2, 2, n), rng.integers(0, 2, n).astype(np.uint8), 0.0, 20.0)


BATCHES = {
    "links at the limit": lambda: [_random(1 << 19, 900, 2, 9, 1), _random((1 << 19) + 1, 900, 2, 9, 2),
                                   _random(300, 2000, 1, 5, 3)],
    "streams at the limit": lambda: [_random(4000, 1 << 19, 1, 2, 4), _random(4000, (1 << 19) + 1, 1, 2, 5)],
    "full tiles": lambda: [_full(64, 128, 6), _full(65, 128, 7), _full(8, 1024, 8), _full(3, 1, 9),
                           I.Instance("e", 3, 2, np.zeros(4, np.int32), np.zeros(0, np.int32), np.ones(3),
                                      np.ones(2), np.zeros(2, np.uint8), 0.0, 20.0)],
}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name", list(BATCHES))
def test_clustered_tiles(name, dtype):
    insts = BATCHES[name]()
    K = 30
    b = BatchSolver(insts, dtype=dtype, eps_abs=0.0)
    for _ in range(2):                       # a second call continues on the same tables
        b.solve(K)
    for k, inst in enumerate(insts):
        s = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_GATHER, eps_abs=0.0, max_iter=K)
        for _ in range(2):
            s.solve()
        for p, q in zip(b.solution(k), s.solution()):
            assert torch.equal(p, q), (name, k)
        s.close()
    b.close()
