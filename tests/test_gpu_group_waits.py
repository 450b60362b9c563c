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
