"""Iterations held on chip (small instances in the gather layout) against the
passes of that layout, which the reverse mode's forward run still takes: the
same sums in the same order, so the iterates are equal bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2509_10722_amd import instances as I
from tests.gpu_util import close, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import Solver  # noqa: E402


def _instance(m, n, lo, hi, hot=0, seed=3):
    """Random routes of lo..hi links over a third of utilities each, the last
    two links unused, an empty route, and link 0 on `hot` more streams."""
    rng = np.random.default_rng(seed)
    used = max(hi, m - 2)
    link, stream = I.random_routes(rng, used, rng.integers(lo, hi + 1, n))
    if n > 2:
        keep = stream != n - 2
        link, stream = link[keep], stream[keep]
    pairs = np.stack([link, stream], 1)
    if hot:
        pairs = np.unique(np.concatenate([pairs, np.stack([np.zeros(hot, np.int64), np.arange(hot)], 1)]), axis=0)
    row_ptr, col_idx = I.csr_from_pairs(m, n, pairs[:, 0], pairs[:, 1])
    return I.Instance("r", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 3, n).astype(np.uint8), 0.0, 20.0)


# one workgroup / several (1,024 rows each), four lanes a segment or one,
# tails of every length, segments past the 16 register slots, odd sizes
SIZES = [(3, 1, 1, 2, 0), (7, 5, 1, 4, 0), (200, 1000, 2, 8, 0), (1024, 1024, 5, 9, 0),
         (1025, 1024, 3, 7, 0), (300, 2049, 1, 6, 25), (2500, 257, 5, 40, 0),
         (5000, 3001, 13, 19, 30), (20000, 9999, 3, 12, 0)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("size", SIZES)
def test_on_chip_equals_passes(size, dtype):
    inst = _instance(*size)
    K = 23
    a = Solver(inst, dtype=dtype, adapt_every=0)
    b = Solver(inst, dtype=dtype, adapt_every=0)
    a.iterate(K)
    b.forward_ckpt(K, K)
    va, vb = a.views(), b.views()
    for k in ("x", "a", "b", "zs", "u", "v"):
        assert torch.equal(va[k], vb[k]), k
    a.close()
    b.close()


@pytest.mark.parametrize("m,n", [(200, 1000), (3000, 2500)])
def test_on_chip_solve_matches_oracle(m, n):
    """Stop rule, balancing and the relative rule's norms inside the launch."""
    inst = _instance(m, n, 2, 8)
    for rel in (0.0, 1e-3):
        s = Solver(inst, dtype=torch.float64, eps_rel=rel, max_iter=4000)
        res = s.solve()
        x, lam, slack = s.solution()
        o = oracle.run(inst, res["iterations"], history=True)
        assert close(host(x), o["x"], 64) and close(host(lam), o["lam"], 64)
        assert abs(res["r_norm"] - o["r_norm"]) <= 1e-6 * o["r_norm"]
        assert abs(res["s_norm"] - o["s_norm"]) <= 1e-6 * o["s_norm"]
        if rel:     # stops at the first check that meets the relative rule
            J = inst.nnz + inst.m
            k = np.arange(9, res["iterations"], 10)
            tr = 1e-4 * J ** 0.5 + rel * np.maximum(o["hist_pnorm"], o["hist_znorm"])[k]
            ts = 1e-4 * J ** 0.5 + rel * o["hist_unorm"][k]
            met = (o["hist_r"][k] < tr) & (o["hist_s"][k] < ts)
            assert res["converged"] and met[-1] and not met[:-1].any()
        s.close()


def test_group_not_formed_runs_alone():
    """The launch's own way out when no XCD collects the group: the word that
    records the group is set to "none" from the host, found by the barrier
    counts next to it, and the run by one workgroup gives the same iterates."""
    inst = _instance(2500, 2200, 2, 8)
    K = 7
    s = Solver(inst, dtype=torch.float32, adapt_every=0)
    s.iterate(K)
    torch.cuda.synchronize()
    w = s.workspace[: s.workspace.numel() // 4 * 4].view(torch.int32)
    E = 2 * K                       # two barriers an iteration
    hit = torch.nonzero((w[64:-64] == E) & (w[65:-63] == E) & (w[128:] == E) & (w[:-128] == 0))
    assert hit.numel() == 1
    win = int(hit) + 64 - 64        # the word a line before the barrier counts
    w[win] = 99
    s.iterate(K)
    ref = Solver(inst, dtype=torch.float32, adapt_every=0)
    ref.iterate(K)
    ref.iterate(K)
    assert int(w[win]) == 0         # cleared again for the next launch
    for k, v in s.views().items():
        assert torch.equal(v, ref.views()[k]), k
    assert abs(s.residuals()[0] - ref.residuals()[0]) <= 1e-9 * ref.residuals()[0]
    s.iterate(K)                    # a group again
    ref.iterate(K)
    assert torch.equal(s.views()["x"], ref.views()["x"])
    s.close()
    ref.close()
