"""The CSR product at the row counts where its workgroups change size, with
rows shorter and longer than a chunk's share, against the oracle bit for bit."""

import numpy as np
import pytest

import oracle
from rpcg_workloads import CSRHost, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _rows(n, mean, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 2 * mean + 1, n)
    lens[n // 2] = 3000  # longer than any chunk
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return CSRHost(n, rp, rng.integers(0, n, rp[-1]).astype(np.int32), rng.standard_normal(rp[-1]))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 65535, 65536, 131071, 131072, 393215, 393216])
@pytest.mark.parametrize("mean", [4, 40])
def test_spmv_rows(n, mean):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg as R
    A = _rows(n, mean, n + mean)
    x = uniform_pm1(n, n)
    y = R.spmv(R.CSR.from_host(A), torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(y.view(np.uint64), oracle.spmv(A, x).view(np.uint64))
