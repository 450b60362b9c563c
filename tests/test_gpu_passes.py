"""Which passes an instance runs, and mid-sized instances under the automatic
layout beside the plain iterations of tests/test_gpu_staged.py: solves through
balancing steps and both stop rules, problems of binned size, gradients."""
import numpy as np
import pytest

from paper_2509_10722_amd import instances as I
from tests.test_gpu_staged import SIZES, _instance as _staged_instance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import PMP_LAYOUT_BINNED, PMP_LAYOUT_GATHER, Solver  # noqa: E402


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


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_passes_in_use(dtype):
    def passes(inst, **kw):
        s = Solver(inst, dtype=dtype, **kw)
        p = s.passes_in_use()
        s.close()
        return p

    for size in SIZES:      # the tables of the last are refused: a link on many streams
        inst = _staged_instance(*size)
        assert passes(inst) == ("gather" if size[4] else "staged")
        assert passes(inst, layout=PMP_LAYOUT_GATHER) == "gather"
        assert passes(inst, layout=PMP_LAYOUT_BINNED) == "binned"
    small = _instance(300, 900, 2, 6)
    assert passes(small) == passes(small, layout=PMP_LAYOUT_GATHER) == "on-chip"
    assert passes(small, layout=PMP_LAYOUT_BINNED) == "binned"
    assert passes(_instance(60000, 60000, 2, 6)) == "gather"        # past one XCD
    wide = _instance(400000, 400000, 5, 8)                          # past what staging pays for
    assert passes(wide) == ("binned" if dtype == torch.float32 else "gather")


def test_staged_of_binned_size_equals_both():
    """nnz >= 2^21 in FP32: the sizes ask for the binned layout, the staged
    passes run without its messages; the iterates equal both bit for bit."""
    inst = _instance(20000, 300000, 5, 11)
    assert inst.nnz >= 2 ** 21
    a = Solver(inst)
    assert a.passes_in_use() == "staged" and a.layout_in_use() == "binned"
    a.iterate(57)               # through a balancing step
    for layout in (PMP_LAYOUT_GATHER, PMP_LAYOUT_BINNED):
        b = Solver(inst, layout=layout)
        b.iterate(57)
        for k in ("x", "a", "b", "zs", "u"):
            assert torch.equal(a.views()[k], b.views()[k]), (layout, k)
        ra, rb = a.residuals(), b.residuals()
        assert abs(ra[0] - rb[0]) <= 1e-9 * rb[0] and abs(ra[1] - rb[1]) <= 1e-9 * rb[1]
        b.close()
    a.close()


def test_refused_tables_leave_the_binned_layout_whole():
    """The staged tables are built where the binned ones go when the pattern is
    too uneven for them."""
    inst = _staged_instance(20000, 300000, 5, 11, 3900)
    assert inst.nnz >= 2 ** 21
    a, b = Solver(inst), Solver(inst, layout=PMP_LAYOUT_GATHER)
    assert a.passes_in_use() == "binned" and b.passes_in_use() == "gather"
    for s in (a, b):
        s.iterate(57)
    for k in ("x", "a", "b", "zs", "u"):
        assert torch.equal(a.views()[k], b.views()[k]), k
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("rel", [0.0, 1e-3])
def test_staged_solve_stops_and_balances_like_gather(rel, dtype):
    """Whole solves in replayed graphs: the same checks, rho steps and end."""
    inst = _instance(5001, 150001, 6, 12)
    out = []
    for kw in ({}, {"layout": PMP_LAYOUT_GATHER}):
        s = Solver(inst, dtype=dtype, eps_abs=1e-2, eps_rel=rel, max_iter=3000, **kw)
        assert s.passes_in_use() == ("gather" if kw else "staged")
        res = s.solve()
        out.append((res, s.history(), [t.double().cpu() for t in s.solution()]))
        s.close()
    (ra, ha, xa), (rb, hb, xb) = out
    assert ra["iterations"] == rb["iterations"] and ra["converged"] and rb["converged"]
    # (the relative rule stops after its first rho step)
    assert ha.shape == hb.shape and np.unique(ha[:, 3]).size >= (2 if rel else 3)
    assert np.array_equal(ha[:, 0], hb[:, 0]) and np.allclose(ha, hb, rtol=1e-8, atol=0)
    for p, q in zip(xa, xb):
        # FP32 sums are exact in FP64; FP64 sums differ in their order
        assert float((p - q).norm()) <= (0.0 if dtype == torch.float32 else 1e-9) * float(q.norm())
