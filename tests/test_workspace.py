"""Workspace sizes (CPU only: pmp_workspace_size reads the sizes alone)."""
import ctypes

import pytest

from paper_2509_10722_amd import pmp


def _bytes(m, n, nnz, dtype, layout):
    b = ctypes.c_size_t()
    prob = pmp.pmp_problem(m=m, n=n, nnz=nnz, dtype=dtype)
    prm = pmp.params_default(layout=layout)
    assert pmp.load_library().pmp_workspace_size(ctypes.byref(prob), ctypes.byref(prm), ctypes.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("m,n,nnz", [(100000, 500000, 5000000), (100000, 1000000, 7500000),
                                     (100000, 1000000, 100000000)])
def test_staged_tables_and_messages_share_their_place(m, n, nnz):
    """An FP32 instance of binned size whose passes may gather from LDS reserves
    the larger of the two sets of tables, not both: 12 bytes a nonzero and its tile
    offsets for the messages; at most 16 for the index words of two sides, and the
    lanes' rows and partial sums."""
    gather, binned, auto = (_bytes(m, n, nnz, pmp.PMP_F32, k) for k in (1, 2, 0))
    assert binned > gather + 12 * nnz
    assert binned <= auto <= max(binned, gather + 18 * nnz)
