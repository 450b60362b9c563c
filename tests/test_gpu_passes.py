"""Mid-sized instances under the automatic layout: what their passes return
beside the plain iterations of tests/test_gpu_staged.py."""
import numpy as np
import pytest

from paper_2509_10722_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import PMP_LAYOUT_GATHER, Solver  # noqa: E402


def _instance(m, n, lo, hi, seed=4):
    """All three utilities, unused links at the end."""
    rng = np.random.default_rng(seed)
    link, stream = I.random_routes(rng, m - 3, rng.integers(lo, hi + 1, n))
    row_ptr, col_idx = I.csr_from_pairs(m, n, link, stream)
    return I.Instance("p", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 3, n).astype(np.uint8), 0.0, 20.0)


@pytest.mark.parametrize("size", [(5001, 150001, 6, 12), (20003, 200007, 5, 11)])
def test_fp32_gradient_sums_in_fp64(size):
    """FP32 problems below 2^21 nonzeros gather ybar and Sbar in FP64 whatever
    passes their iterations take: the same gradient bit for bit."""
    inst = _instance(*size)
    assert 2 ** 20 <= inst.nnz < 2 ** 21
    out = []
    for kw in ({}, {"layout": PMP_LAYOUT_GATHER}):
        s = Solver(inst, dtype=torch.float32, adapt_every=0, **kw)
        s.iterate(5)
        for _ in range(2):
            J = s.forward_ckpt(100, 25)
            gc, gw = s.backward()
        out.append((J, gc.clone(), gw.clone(), s.views()["x"].clone()))
        s.close()
    assert out[0][0] == out[1][0]
    for p, q in zip(out[0][1:], out[1][1:]):
        assert torch.equal(p, q)
