"""Entry lists of every remainder modulo four, at every 4-byte alignment of the index and weight arrays."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_12093_amd import binding as B
from paper_2308_12093_amd import graphs as G
from tests._util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def shifted(t, by):
    """The same values in memory that starts `by` elements after a 16-byte boundary."""
    room = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    room[by:] = t
    return room[by:]


@pytest.mark.parametrize("f", [7, 16, 260])
@pytest.mark.parametrize("nnz", [1, 15, 16, 18, 1023, 2049, 8190])
def test_spmm(nnz, f):
    rng = np.random.default_rng(nnz + f)
    n = max(1, nnz // 5)
    rows = np.sort(rng.integers(0, n, nnz))
    rowptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(rows, minlength=n), out=rowptr[1:])
    col, val = rng.integers(0, n, nnz).astype(np.int32), rng.standard_normal(nnz).astype(np.float32)
    X = rng.standard_normal((n, f)).astype(np.float32)
    ref = np.zeros((n, f))
    np.add.at(ref, rows, val[:, None].astype(np.float64) * X[col])
    rp = dev(rowptr)
    for by in range(4):
        C = torch.empty(n, f, device="cuda")
        B.gnn_spmm_csr(n, nnz, rp, shifted(dev(col), by), shifted(dev(val), by), shifted(G.expand(n, rp, nnz), by), dev(X),
                       f, C, workspace=B.alloc(B.gnn_spmm_workspace_bytes(n, nnz, f)))
        assert_close(host(C), ref, f"shift {by}", tol=2e-6)


@pytest.mark.parametrize("f", [1, 7, 8, 47, 64, 300])
def test_spmm_without_a_bias_keeps_the_sign_of_zero(f):
    """One entry a row: the product, which underflows to -0 in every other row."""
    n = 1000
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    val = torch.full((n,), 1e-30, device="cuda")
    X = torch.full((n, f), 1e-30, device="cuda")
    X[::2] = -1e-30
    C = torch.empty(n, f, device="cuda")
    B.gnn_spmm_csr(n, n, ids, ids[:n].clone(), val, ids[:n].clone(), X, f, C, workspace=B.alloc(B.gnn_spmm_workspace_bytes(n, n, f)))
    assert bool((C == 0).all()) and bool(torch.signbit(C[::2]).all()) and not bool(torch.signbit(C[1::2]).any())
