"""The loss forms its products A u in the pass that checks the diagonals: a
matrix that the check refuses is refused as before, whatever its columns, and
a missing probe is an error."""

import numpy as np
import pytest

from rpcg_workloads import CSRHost, grf_diffusion_csr, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    return rpcg


def _setup(R, N, nu):
    net = R.LearnedPreconditioner(N, max_batch=2)
    A = grf_diffusion_csr(N, 5)[0]
    us = [[torch.from_numpy(uniform_pm1(10 * k + m, A.n)).cuda() for m in range(nu)] for k in range(2)]
    return net, A, us


@pytest.mark.parametrize("nu", [1, 2, 3, 4])
@pytest.mark.parametrize("col", [-1, 7 ** 3, 2 ** 31 - 1, -2 ** 31])
def test_columns_outside_the_matrix(R, nu, col):
    """One diagonal entry's column out of range: the diagonal is missing."""
    print(f"lp refusal nu {nu} col {col}", flush=True)
    net, A, us = _setup(R, 7, nu)
    c = A.col_idx.copy()
    c[A.row_ptr[100] + list(c[A.row_ptr[100]:A.row_ptr[101]]).index(100)] = col
    mats = [R.CSR.from_host(A), R.CSR.from_host(CSRHost(A.n, A.row_ptr, c, A.val))]
    for call in (lambda: net.loss_grad(mats, us), lambda: net.train_step(mats, us, lr=1e-3)):
        with pytest.raises(R.RpcgError) as e:
            call()
        assert e.value.status == R.ERR_NOT_SPD
    loss, _ = net.loss_grad([R.CSR.from_host(A)] * 2, us)
    assert np.isfinite(loss)
    net.close()


@pytest.mark.parametrize("nu", [2, 3])
def test_missing_probe(R, nu):
    net, A, us = _setup(R, 6, nu)
    us[1][0] = None
    with pytest.raises(R.RpcgError) as e:
        net.loss_grad([R.CSR.from_host(A)] * 2, us)
    assert e.value.status == R.ERR_INVALID
    bad = A.val.copy()
    bad[A.row_ptr[3]:A.row_ptr[4]] *= -1.0
    with pytest.raises(R.RpcgError) as e:
        net.loss_grad([R.CSR.from_host(A), R.CSR.from_host(CSRHost(A.n, A.row_ptr, A.col_idx, bad))], us)
    assert e.value.status == R.ERR_NOT_SPD
    net.close()
