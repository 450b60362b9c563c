"""The passes that gather from LDS (mid-sized instances under the automatic
layout) against the gather layout asked for by name: FP32 sums are exact in
FP64, so the iterates are equal bit for bit; FP64 sums differ in their order
only (a few ulp an iteration, 1e-12 over a short run)."""
import ctypes

import numpy as np
import pytest

from paper_2509_10722_amd import instances as I
from tests.gpu_util import rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import (PMP_LAYOUT_AUTO, PMP_LAYOUT_GATHER, Solver,  # noqa: E402
                                      load_library, params_default)


def _instance(m, n, lo, hi, hot=0, seed=4):
    """All three utilities, unused links at the end, an empty route, link 0 on
    `hot` more streams."""
    rng = np.random.default_rng(seed)
    link, stream = I.random_routes(rng, m - 3, rng.integers(lo, hi + 1, n))
    keep = stream != n - 2
    pairs = np.stack([link[keep], stream[keep]], 1)
    if hot:
        pairs = np.unique(np.concatenate([pairs, np.stack([np.zeros(hot, np.int64), np.arange(hot)], 1)]), axis=0)
    row_ptr, col_idx = I.csr_from_pairs(m, n, pairs[:, 0], pairs[:, 1])
    return I.Instance("s", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 3, n).astype(np.uint8), 0.0, 20.0)


def _planned(s):
    """Whether the sizes alone ask for the staged tables (in the workspace)."""
    lib, out = load_library(), []
    for layout in (PMP_LAYOUT_AUTO, PMP_LAYOUT_GATHER):
        b = ctypes.c_size_t()
        prm = params_default(layout=layout)
        assert lib.pmp_workspace_size(ctypes.byref(s.problem), ctypes.byref(prm), ctypes.byref(b)) == 0
        out.append(b.value)
    return out[0] > out[1]


# odd sizes, one chunk and several, one workgroup a link block and several; a
# link on so many streams that the tables are refused and the gathers stay
SIZES = [(5001, 150001, 6, 12, 0), (20003, 200007, 5, 11, 0), (30000, 300001, 5, 8, 0),
         (5001, 150001, 6, 12, 3900)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("size", SIZES)
def test_staged_equals_gather(size, dtype):
    inst = _instance(*size)
    K = 23
    a = Solver(inst, dtype=dtype)
    b = Solver(inst, dtype=dtype, layout=PMP_LAYOUT_GATHER)
    assert _planned(a) and a.layout_in_use() == b.layout_in_use() == "gather"
    for s in (a, b):
        s.iterate(K)
    ra, rb = a.residuals(), b.residuals()
    va, vb = a.views(), b.views()
    for k in ("x", "a", "b", "zs", "u", "v"):
        if dtype == torch.float32:
            assert torch.equal(va[k], vb[k]), k
        else:
            assert float((va[k] - vb[k]).norm() / vb[k].norm()) <= 1e-12, k
    assert abs(ra[0] - rb[0]) <= 1e-10 * rb[0] and abs(ra[1] - rb[1]) <= 1e-10 * rb[1]
    # the same iterates every time
    c = Solver(inst, dtype=dtype)
    c.iterate(K)
    for k in ("x", "u"):
        assert torch.equal(va[k], c.views()[k]), k
    for s in (a, b, c):
        s.close()


@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2e-6), (torch.float64, 1e-11)])
def test_staged_gradient(dtype, tol):
    """Reverse mode: ybar and Sbar are staged in the problem's precision (FP32:
    rounded once per sum's addend, 2^-24 each, against FP64 gathers)."""
    inst = _instance(5001, 150001, 6, 12)
    out = []
    for layout in (PMP_LAYOUT_AUTO, PMP_LAYOUT_GATHER):
        s = Solver(inst, dtype=dtype, adapt_every=0, layout=layout)
        J = s.forward_ckpt(12, 5)
        gc, gw = s.backward()
        out.append((J, gc.cpu().numpy(), gw.cpu().numpy()))
        s.close()
    (Ja, ca, wa), (Jb, cb, wb) = out
    assert abs(Ja - Jb) <= 1e-12 * abs(Jb)
    assert rel(ca, cb) <= tol and rel(wa, wb) <= tol
