"""Which copy a matrix gets, and parity with the oracle where it is the aligned
one: without the first the aligned kernels could go unused unnoticed, as the general
copy gives the same bits. Values that vary need enough slices to be held aligned,
so those cases have more than the 1280 slices of 128 rows that 256 CUs ask for at most."""

import numpy as np
import pytest

from rpcg_workloads import CSRHost, band_csr, stencil27_csr, stencil7_varcoef_csr, uniform_pm1
from test_gpu_diag import CASES as SMALL, _offsets_csr

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BIG = 170_000  # rows: 1329 slices


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _bits(a):
    return np.ascontiguousarray(a).view(np.uint64)


def _product(R, orc, A, layout):
    x = uniform_pm1(21, A.n) * 5.0
    x[A.n // 3] = -0.0
    M = R.PreparedMatrix(R.CSR.from_host(A))
    assert M.layout == layout
    got = M.spmv(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(_bits(got), _bits(orc.spmv(A, x)))


@pytest.mark.parametrize("case", ["n127", "n255_five", "far_const", "holes_const", "wide_band", "stencil27_odd"])
def test_constant_coefficients_are_aligned(R, orc, case):
    print(f"layout {case}", flush=True)
    _product(R, orc, SMALL[case](), "aligned")


@pytest.mark.parametrize("case", ["n1", "long_row"])
def test_general_copies(R, orc, case):
    print(f"layout {case}", flush=True)
    _product(R, orc, SMALL[case](), "col16")


@pytest.mark.parametrize("n,aligned", [(63, False), (64, True), (65, True), (127, True), (128, True), (129, True)])
def test_smallest_aligned(R, orc, n, aligned):
    """One record of one slice serves n entries: aligned from the records' half on."""
    _product(R, orc, _offsets_csr(n, [0], 1, True), "aligned" if aligned else "col16")


@pytest.mark.parametrize("case,layout", [("n129", "col16"), ("far", "col16"), ("unsorted", "col32"), ("holes", "col16"),
                                         ("band17", "col16"), ("stencil27_var", "col16"), ("stencil7", "col16"),
                                         ("first_scaled", "aligned")])
def test_few_slices_of_varying_values(R, orc, case, layout):
    """They are faster in the general copy; one slice in sixteen may vary among constant ones."""
    print(f"layout {case}", flush=True)
    _product(R, orc, SMALL[case](), layout)


@pytest.mark.parametrize("n,w,layout", [(1000, 249, "aligned"), (1000, 250, "col16"), (2053, 130, "aligned")])
def test_bands_against_the_size(R, orc, n, w, layout):
    _product(R, orc, band_csr(n, w), layout)


@pytest.mark.parametrize("entries", [3, 7, 9, 27])
def test_slices_that_varying_values_need(R, orc, entries):
    """Five a CU; half of that for rows of one batch of loads."""
    rows = 128 * 5 * torch.cuda.get_device_properties(0).multi_processor_count
    if entries <= 7:
        rows //= 2
    offs = [7 * (k - entries // 2) for k in range(entries)]
    for n, layout in ((rows, "aligned"), (rows - 128, "col16")):
        _product(R, orc, _offsets_csr(n, offs, 9, False), layout)
        _product(R, orc, _offsets_csr(n, offs, 9, True), "aligned")


def _big(kind):
    if kind == "stencil7":
        return stencil7_varcoef_csr(56, 4)  # 175 616 rows
    if kind == "stencil27":
        A = stencil27_csr(56)
        return CSRHost(A.n, A.row_ptr, A.col_idx, A.val * (1.0 + 0.1 * np.random.default_rng(3).random(A.val.size)))
    offs, drop = {"tri": ([-1, 0, 1], 0.0), "far": ([-1500, -7, 0, 7, 1500], 0.0), "unsorted": ([5, 0, -5, 0, 40], 0.0),
                  "holes": (list(range(-6, 7)), 0.1), "band17": (list(range(-17, 18)), 0.0)}[kind]
    return _offsets_csr(BIG + {"tri": 1, "far": 127, "unsorted": 64, "holes": 77, "band17": 126}[kind], offs, 8, False, drop)


@pytest.mark.parametrize("kind", ["tri", "far", "unsorted", "holes", "band17", "stencil7", "stencil27"])
def test_varying_values_aligned(R, orc, kind):
    print(f"layout big {kind}", flush=True)
    _product(R, orc, _big(kind), "aligned")


@pytest.mark.parametrize("mode", ["exblas", "fpe"])
@pytest.mark.parametrize("kind", ["stencil7", "stencil27"])
def test_solves_over_varying_values(R, orc, kind, mode):
    A = _big(kind)
    if kind == "stencil27":  # rows differ: make it diagonally dominant
        A.val[A.col_idx == np.repeat(np.arange(A.n), np.diff(A.row_ptr))] = 40.0
    b = orc.spmv(A, uniform_pm1(14, A.n))
    ref = orc.pcg(A, b, tol=1e-8, maxit=6)
    Ad, bd = R.CSR.from_host(A), torch.from_numpy(b).cuda()
    for kw in ({}, {"no_col16": 1}):
        x, info = R.pcg_solve(Ad, bd, mode=mode, tol=1e-8, maxit=6, raise_on_error=False, **kw)
        assert info["iterations"] == ref["iters"]
        assert np.array_equal(_bits(x.cpu().numpy()), _bits(ref["x"]))


def test_binary32_and_refinement_over_varying_values(R, orc):
    A = _big("stencil7")
    b = orc.spmv(A, uniform_pm1(15, A.n))
    b32 = b.astype(np.float32)
    ref = orc.pcg_f32(A, b32, tol=1e-6, maxit=5)
    x, info = R.pcg_solve_f32(R.CSR.from_host(A, dtype=torch.float32), torch.from_numpy(b32).cuda(), tol=1e-6, maxit=5,
                              raise_on_error=False)
    assert info["iterations"] == ref["iters"]
    assert np.array_equal(x.cpu().numpy().view(np.uint32), ref["x"].view(np.uint32))
    ref = orc.ir(A, b, tol=1e-10, maxit_out=2, maxit_in=5)
    x, info = R.ir_solve(R.CSR.from_host(A), torch.from_numpy(b).cuda(), maxit=2, maxit_inner=5, raise_on_error=False)
    assert info["outer"] == 2
    assert np.array_equal(_bits(x.cpu().numpy()), _bits(ref["x"]))


def test_batch_over_varying_values(R, orc):
    """1312 slices in all, 540 without the largest systems: aligned and general give each system's own bits."""
    systems = [stencil7_varcoef_csr(N, 90 + N) for N in (40, 3, 17)]  # 500, 1, 39 slices
    systems += [stencil7_varcoef_csr(N, 7) for N in (41, 31)]         # 539, 233
    bs = [orc.spmv(A, uniform_pm1(30 + k, A.n)) for k, A in enumerate(systems)]
    refs = [orc.pcg(A, b, tol=1e-9, maxit=12) for A, b in zip(systems, bs)]
    for keep in (5, 3):
        for mode in ("exblas", "fpe"):
            B = R.Batch([R.CSR.from_host(A) for A in systems[:keep]], mode=mode, tol=1e-9, maxit=12)
            xs, infos, _ = B.solve([torch.from_numpy(b).cuda() for b in bs[:keep]], raise_on_error=False)
            for x, i, r in zip(xs, infos, refs):
                assert i["iterations"] == r["iters"]
                assert np.array_equal(_bits(x.cpu().numpy()), _bits(r["x"]))
            B.close()


def test_layout_of_nothing(R):
    assert R.lib().rpcg_smat_layout(None) == R.ERR_INVALID
