"""General copies around the slice counts where a workgroup takes one, two,
three or four wavefronts (prepared products and solves), against the oracle bit
for bit."""

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from rpcg_workloads import CSRHost, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _spd(n, seed):
    """A random sparse diagonally dominant matrix: rows share no offsets."""
    rng = np.random.default_rng(seed)
    i, j = rng.integers(0, n, 6 * n), rng.integers(0, n, 6 * n)
    M = sp.coo_matrix((-rng.random(6 * n), (i, j)), shape=(n, n)).tocsr()
    M = M + M.T
    M.setdiag(0)
    M.eliminate_zeros()
    M = (M + sp.diags(1.0 - np.asarray(M.sum(1)).ravel())).tocsr()
    M.sort_indices()
    return CSRHost(n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data)


@pytest.mark.parametrize("n", [64 * 256, 64 * 256 + 1, 64 * 512, 64 * 512 + 1, 64 * 768 + 1, 64 * 1024 + 1])
def test_few_slices(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg as R
    A = _spd(n, n)
    C = R.CSR.from_host(A)
    x = uniform_pm1(n, n)
    ref = oracle.spmv(A, x)
    M = R.PreparedMatrix(C)
    y = M.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    M.close()
    assert np.array_equal(y.view(np.uint64), ref.view(np.uint64))
    want = oracle.pcg(A, ref, tol=0.0, maxit=4)
    for mode in ("exblas", "fpe"):
        got, info = R.pcg_solve(C, torch.from_numpy(ref).cuda(), mode=mode, tol=0.0, maxit=4, raise_on_error=False)
        assert info["iterations"] == want["iters"]
        assert np.array_equal(got.cpu().numpy().view(np.uint64), want["x"].view(np.uint64))
