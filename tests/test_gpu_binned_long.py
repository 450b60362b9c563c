"""Binned passes with one block per CU on both sides and a long link among short
ones, up to where its block has more entries than a workgroup loads at once (the
link side then keeps the kernels that stream them through), against the gather
layout: FP32 sums are exact in FP64 or in fixed point, bit
equality; FP64 sums differ in their order only (1e-12 over a short run)."""
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


@pytest.mark.parametrize("hi", [20.0, float("inf")])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("hot", [4096, 4097, 30000])
def test_long_links_among_short(hot, dtype, hi):
    rng = np.random.default_rng(8)
    m, n = 20000, 60000
    link, stream = I.random_routes(rng, m, rng.integers(2, 6, n))
    # link m / 2: on streams 0 .. hot - 1 alone
    keep = link != m // 2
    pairs = np.concatenate([np.stack([link[keep], stream[keep]], 1),
                            np.stack([np.full(hot, m // 2), np.arange(hot)], 1)])
    pairs = np.unique(pairs, axis=0)
    row_ptr, col_idx = I.csr_from_pairs(m, n, pairs[:, 0], pairs[:, 1])
    assert int(np.diff(row_ptr).max()) == hot and np.diff(np.unique(pairs[:, 1])).max() == 1
    inst = I.Instance("l", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      np.zeros(n, np.uint8), 0.0, hi)
    a = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_BINNED)
    b = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_GATHER)
    for k in (7, 23):
        for s in (a, b):
            s.iterate(k)
        for p, q in zip(a.solution(), b.solution()):
            if dtype == torch.float32 and (hi < float("inf") or hot <= 4096):
                assert torch.equal(p, q)
            else:       # (without a box, FP64 sums of long rows of FP32 rates: rounded to FP32 after)
                assert rel(host(p), host(q)) <= (1e-12 if dtype == torch.float64 else 1e-6)
    a.close()
    b.close()
