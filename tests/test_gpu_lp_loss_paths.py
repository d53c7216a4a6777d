"""The loss over every number of probe vectors that has a path of its own, on
grids whose cells do not fill a workgroup, with rows in descending order and with rows too
long for a workgroup to stage: loss and output gradient against the oracle, given
the network's outputs. Both sides hold every vector in binary64; the exponential of
the diagonal output differs in the last float32 bit at most (2^-23: loss
within 1e-6, gradient within 1e-5 of its largest entry)."""

import numpy as np
import pytest

from oracle import lpnet
from rpcg_workloads import CSRHost, grf_diffusion_csr, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _rows(A, kind):
    """The same operator: entries of a row reversed, or behind 40 explicit zeros."""
    if kind == "plain":
        return A
    ci, va, out = [], [], [0]
    for a, b in zip(A.row_ptr[:-1], A.row_ptr[1:]):
        c, v = A.col_idx[a:b], A.val[a:b]
        if kind == "reversed":
            c, v = c[::-1], v[::-1]
        else:
            c, v = np.concatenate([np.arange(40) % A.n, c]), np.concatenate([np.zeros(40), v])
        ci.append(c)
        va.append(v)
        out.append(out[-1] + len(c))
    return CSRHost(A.n, np.asarray(out, np.int32), np.concatenate(ci).astype(np.int32), np.concatenate(va))


@pytest.mark.parametrize("N,nu", [(2, 1), (5, 1), (3, 2), (7, 2), (2, 4), (7, 4), (33, 4), (5, 3), (5, 8), (6, 11)])
@pytest.mark.parametrize("kind", ["plain", "reversed", "long"])
def test_loss_paths(N, nu, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg as R
    rng = np.random.default_rng(N * 100 + nu)
    q = lpnet.split(lpnet.init_params(N).astype(np.float64))
    q["W3"] = rng.standard_normal(q["W3"].shape) * 0.05
    q["b3"] = rng.standard_normal(4) * 0.1
    net = R.LearnedPreconditioner(N, max_batch=2)
    net.set_params(lpnet.join(q).astype(np.float32))
    As = [grf_diffusion_csr(N, 70 + N + k)[0] for k in range(2)]
    mats = [R.CSR.from_host(_rows(A, kind)) for A in As]
    us = [[uniform_pm1(100 * k + m, A.n) for m in range(nu)] for k, A in enumerate(As)]
    loss, dout = net.loss_grad(mats, [[torch.from_numpy(u).cuda() for u in row] for row in us], eps=1e-3)
    o = net.forward(mats).cpu().numpy()
    net.close()
    L, dos = 0.0, []
    for k, A in enumerate(As):
        G, dgdo = lpnet.factor(A, N, o[k])
        Lk, dG = lpnet.loss_grad(A, G, us[k], 1e-3)
        L += Lk / 2
        dos.append(lpnet.do_from_dg(G, dG, dgdo, N).reshape(-1, 4) / 2)
    assert abs(loss - L) <= 1e-6 * abs(L)
    d = dout.cpu().numpy()
    for k in range(2):
        assert np.max(np.abs(d[k] - dos[k])) <= 1e-5 * np.max(np.abs(dos[k]))
