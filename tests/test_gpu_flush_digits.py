"""Solver dots whose terms span most of the exponent range inside every
wavefront (more digit blocks than a row of lanes holds), and infinities among
them, against the oracle, bit for bit."""

import numpy as np
import pytest

from rpcg_workloads import CSRHost

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _diagonal(n, seed):
    rng = np.random.default_rng(seed)
    return CSRHost(n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), 1.0 + rng.random(n))


@pytest.mark.parametrize("n", [1, 63, 130, 1003])
@pytest.mark.parametrize("span", [0, 40, 470])
@pytest.mark.parametrize("mode,p", [("exblas", 0), ("exblas", 2), ("exblas", 8), ("fpe", 0), ("fpe", 8)])
def test_wide_terms(R, n, span, mode, p):
    A = _diagonal(n, 3)
    rng = np.random.default_rng(n + span)
    b = rng.standard_normal(n) * 2.0 ** rng.integers(-span, span + 1, n)
    ref = oracle.pcg(A, b, tol=0.0, maxit=3)
    x, info = R.pcg_solve(R.CSR.from_host(A), torch.from_numpy(b).cuda(), mode=mode, tol=0.0, maxit=3, fpe_size=p,
                          raise_on_error=False)
    assert info["iterations"] == ref["iters"]
    assert np.array_equal(info["hist"].cpu().numpy() if hasattr(info["hist"], "cpu") else np.asarray(info["hist"]),
                          ref["hist"])
    assert np.array_equal(x.cpu().numpy().view(np.uint64), ref["x"].view(np.uint64))


@pytest.mark.parametrize("mode", ["exblas", "fpe"])
def test_overflow_is_reported(R, mode):
    A = _diagonal(200, 4)
    b = np.ones(200)
    b[77] = 1e300  # its square overflows: one term of one dot of the pair is not finite
    _, info = R.pcg_solve(R.CSR.from_host(A), torch.from_numpy(b).cuda(), mode=mode, maxit=3, raise_on_error=False)
    assert info["status"] == -6
