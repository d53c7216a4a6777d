"""GPU parity of the diagonal-aligned matrix copy (prepared products and
solves) against the oracle, bit for bit: slice remainders, constant and stored
values, records in and out of runs of three, rows that do not line up."""

import numpy as np
import pytest

from rpcg_workloads import CSRHost, band_csr, scale_first, stencil27_csr, stencil7_varcoef_csr, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _offsets_csr(n, offs, seed, const, drop=0.0):
    """Rows with entries at the given offsets, in the given order (which need
    not ascend and may repeat), entries outside the matrix and a share `drop` of
    the others left out; constant per offset or random values with zeros of
    both signs."""
    rng = np.random.default_rng(seed)
    cols = np.arange(n)[:, None] + np.asarray(offs)[None, :]
    keep = (cols >= 0) & (cols < n) & ((rng.random(cols.shape) >= drop) | (np.asarray(offs) == 0)[None, :])
    vals = np.broadcast_to(rng.standard_normal(len(offs)), cols.shape).copy() if const else rng.standard_normal(cols.shape)
    if not const:
        vals[rng.random(cols.shape) < 0.1] = -0.0
        vals[rng.random(cols.shape) < 0.1] = 0.0
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))])
    return CSRHost(n, rp.astype(np.int32), cols[keep].astype(np.int32), vals[keep])


def _var27(N, seed):
    A = stencil27_csr(N)
    rng = np.random.default_rng(seed)
    return CSRHost(A.n, A.row_ptr, A.col_idx, A.val * (1.0 + 0.1 * rng.random(A.val.size)))


def _long_row(n):
    """One row longer than the merge takes: the general copy."""
    m = 1500
    lens = np.full(n, 1)
    lens[n // 2] = m
    rp = np.concatenate([[0], np.cumsum(lens)])
    col = np.concatenate([np.arange(n // 2), np.arange(m), np.arange(n // 2 + 1, n)])
    return CSRHost(n, rp.astype(np.int32), col.astype(np.int32), np.random.default_rng(1).standard_normal(rp[-1]))


CASES = {
    "n1": lambda: _offsets_csr(1, [0], 1, True),
    "n127": lambda: _offsets_csr(127, [-1, 0, 1], 2, True),
    "n129": lambda: _offsets_csr(129, [-1, 0, 1], 3, False),
    "n255_five": lambda: _offsets_csr(255, [-2, -1, 0, 1, 2], 4, True),
    "far": lambda: _offsets_csr(4099, [-1500, -7, 0, 7, 1500], 5, False),
    "far_const": lambda: _offsets_csr(4099, [-4000, -7, 0, 7, 4000], 6, True),
    "unsorted": lambda: _offsets_csr(3001, [5, 0, -5, 0, 40], 7, False),
    "holes": lambda: _offsets_csr(5003, list(range(-6, 7)), 8, False, drop=0.1),
    "holes_const": lambda: _offsets_csr(5003, list(range(-6, 7)), 9, True, drop=0.1),
    "wide_band": lambda: band_csr(2053, 130),
    "band17": lambda: _offsets_csr(3333, list(range(-17, 18)), 10, False),
    "stencil27_odd": lambda: stencil27_csr(21),
    "stencil27_var": lambda: _var27(23, 3),
    "stencil7": lambda: stencil7_varcoef_csr(29, 4),
    "first_scaled": lambda: scale_first(band_csr(3001, 9), 2.0 ** 16),
    "long_row": lambda: _long_row(2000),
}


@pytest.mark.parametrize("case", CASES)
def test_prepared_product_bitexact(R, orc, case):
    print(f"diag {case}", flush=True)
    A = CASES[case]()
    x = uniform_pm1(11, A.n) * 7.0
    x[A.n // 3] = -0.0
    want = orc.spmv(A, x)
    M = R.PreparedMatrix(R.CSR.from_host(A))
    for k in range(2):
        got = M.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64)), k


def test_masked_rows_do_not_see_infinities(R, orc):
    """A row without an entry at a record's offset is not touched by what x holds there."""
    A = _offsets_csr(1030, [-64, -1, 0, 1, 64], 12, True, drop=0.2)
    x = uniform_pm1(13, A.n)
    x[500] = np.inf
    want = orc.spmv(A, x)
    got = R.PreparedMatrix(R.CSR.from_host(A)).spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    hit = np.zeros(A.n, bool)
    hit[np.repeat(np.arange(A.n), np.diff(A.row_ptr))[A.col_idx == 500]] = True
    assert np.array_equal(got[~hit].view(np.uint64), want[~hit].view(np.uint64))
    assert not np.isfinite(got[hit]).any()


@pytest.mark.parametrize("case", ["stencil27_odd", "stencil27_var", "stencil7", "first_scaled"])
@pytest.mark.parametrize("mode", ["exblas", "fpe"])
def test_solve_same_bits_in_both_layouts(R, orc, case, mode):
    """The aligned copy and the general one (no_col16) give the oracle's iterates."""
    print(f"diag solve {case} {mode}", flush=True)
    A = CASES[case]()
    if case == "stencil27_var":  # symmetric part of the perturbed operator is SPD but rows differ: make it diagonal dominant
        A.val[A.col_idx == np.repeat(np.arange(A.n), np.diff(A.row_ptr))] = 40.0
    b = orc.spmv(A, uniform_pm1(14, A.n))
    ref = orc.pcg(A, b, tol=1e-8, maxit=40)
    Ad, bd = R.CSR.from_host(A), torch.from_numpy(b).cuda()
    for kw in ({}, {"no_col16": 1}):
        x, info = R.pcg_solve(Ad, bd, mode=mode, tol=1e-8, maxit=40, raise_on_error=False, **kw)
        assert info["iterations"] == ref["iters"]
        assert np.array_equal(x.cpu().numpy().view(np.uint64), ref["x"].view(np.uint64))


def test_bad_columns_are_refused(R):
    A = stencil27_csr(12)
    for bad in (-1, A.n, 2 ** 31 - 1):
        col = A.col_idx.copy()
        col[1000] = bad
        with pytest.raises(R.RpcgError):
            R.PreparedMatrix(R.CSR.from_host(CSRHost(A.n, A.row_ptr, col, A.val)))
