"""The bounded waits among the workgroups of a small instance's on-chip
iterations, ended from the host through the words they meet on: every kernel
exits by itself, the failure is reported by each call that uses the iterate, and
pmp_set_state starts over."""
import numpy as np
import pytest

from paper_2509_10722_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2509_10722_amd.pmp import PMP_ERR_HIP, PMPError, Solver  # noqa: E402


def _instance(m, n, lo, hi, seed=3):
    rng = np.random.default_rng(seed)
    link, stream = I.random_routes(rng, m, rng.integers(lo, hi + 1, n))
    row_ptr, col_idx = I.csr_from_pairs(m, n, link, stream)
    return I.Instance("w", m, n, row_ptr, col_idx, rng.uniform(1, 50, m), rng.uniform(0.2, 2, n),
                      rng.integers(0, 3, n).astype(np.uint8), 0.0, 20.0)


def _meeting_words(s, K):
    """The workspace as words, and the index of the word that records the
    group after K iterations (two barriers each) without balancing: the
    workgroups' barrier counts stand a line (64 words) behind it, the launch's
    two lines, the flag of an expired wait three."""
    torch.cuda.synchronize()
    w = s.workspace[: s.workspace.numel() // 4 * 4].view(torch.int32)
    E = 2 * K
    hit = torch.nonzero((w[64:-64] == E) & (w[65:-63] == E) & (w[128:] == E) & (w[:-128] == 0))
    assert hit.numel() == 1
    return w, int(hit)


def _refused(call):
    with pytest.raises(PMPError) as e:
        call()
    assert e.value.status == PMP_ERR_HIP and "barrier" in str(e.value)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("queued", [True, False])
def test_expired_barrier_wait_is_reported_until_set_state(dtype, queued):
    inst = _instance(5000, 4500, 2, 8)
    s, ref = Solver(inst, dtype=dtype), Solver(inst, dtype=dtype)
    for t in (s, ref):
        t.iterate(30)
    st = s.get_state()
    w, win = _meeting_words(s, 30)
    w[win + 3 * 64] = 1         # the first poll that finds a workgroup missing ends the wait
    if queued:
        s.iterate(200)
        _refused(s.residuals)
    else:
        _refused(s.solve)
    failed = torch.zeros(inst.m, dtype=torch.uint8)
    failed[0] = 1
    for call in (s.residuals, s.solution, s.get_state, s.path_prices, s.history, s.solve,
                 lambda: s.iterate(5), lambda: s.prune(failed), lambda: s.forward_ckpt(4, 2),
                 lambda: s.time_kernels(3)):
        _refused(call)
    s.set_state(st)
    for t in (s, ref):
        t.iterate(70)
    for k, v in s.views().items():
        assert torch.equal(v, ref.views()[k]), k
    assert s.residuals() == ref.residuals()
    s.reset()
    ref.reset()
    assert s.solve() == ref.solve()
    s.close()
    ref.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("few", [1, 2, 4])
def test_fewer_workgroups_than_laid_out(few, dtype):
    """A launch whose workgroups do not meet goes on with those that have
    started (the word that records the group is set from the host: the first
    `few` on XCD 0): the same iterates, balancing and residuals, for that launch
    only."""
    inst = _instance(5000, 4500, 2, 8)
    s, ref = Solver(inst, dtype=dtype, eps_rel=1e-3), Solver(inst, dtype=dtype, eps_rel=1e-3)
    for t in (s, ref):
        t.iterate(30)
    w, win = _meeting_words(s, 30)
    w[win] = 99 + 8 * (few - 1)
    for k in (137, 20):                     # with balancing steps; then a whole group again
        for t in (s, ref):
            t.iterate(k)
        assert int(w[win]) == 0
        for name, v in s.views().items():
            assert torch.equal(v, ref.views()[name]), name
        a, b = s.history(), ref.history()
        assert a.shape == b.shape and np.array_equal(a[:, [0, 3]], b[:, [0, 3]])
        assert np.allclose(a, b, rtol=1e-9, atol=0)
    s.reset()
    w[win] = 99 + 8 * (few - 1)
    res, want = s.solve(), Solver(inst, dtype=dtype, eps_rel=1e-3).solve()
    assert res["iterations"] == want["iterations"] and res["converged"] == want["converged"]
    s.close()
    ref.close()


def test_long_queue_in_several_launches():
    """More iterations than a launch takes: no check where launches meet."""
    inst = _instance(2500, 2200, 2, 8)
    a, b = Solver(inst), Solver(inst)
    a.iterate(2525)
    for k in (1000, 1000, 525):
        b.iterate(k)
    for name, v in a.views().items():
        assert torch.equal(v, b.views()[name]), name
    assert a.residuals() == b.residuals() and a.residuals()[2] == 2525
    its = a.history()[:, 0]
    assert np.array_equal(its, np.append(np.arange(50, 2501, 50), 2525))
    c = Solver(inst, adapt_every=0)
    c.iterate(2525)
    assert np.array_equal(c.history()[:, 0], [2525])
    for t in (a, b, c):
        t.close()
