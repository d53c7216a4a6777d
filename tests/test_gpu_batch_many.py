"""Batches of many small systems, empty ones among them: the pass over the row
pointers serves all systems in one launch, and a system's dots have as many accumulator copies
as its size can use. Every system against the oracle; a malformed one is refused."""

import numpy as np
import pytest

from rpcg_workloads import CSRHost, stencil7_varcoef_csr, uniform_pm1

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _empty():
    return CSRHost(0, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0))


def _systems(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for k in range(count):
        N = int(rng.integers(0, 6))
        out.append(_empty() if N == 0 else stencil7_varcoef_csr(N, seed + k))
    return out


def _check(R, orc, systems, mode, **tuning):
    bs = [uniform_pm1(700 + k, A.n) for k, A in enumerate(systems)]
    refs = [orc.pcg(A, b, tol=1e-9, maxit=300) if A.n else None for A, b in zip(systems, bs)]
    B = R.Batch([R.CSR.from_host(A) for A in systems], mode=mode, tol=1e-9, maxit=300)
    if tuning:
        B.set_tuning(**tuning)
    for _ in range(2):
        xs, infos, _ = B.solve([torch.from_numpy(b).cuda() for b in bs], raise_on_error=False)
        for k, (x, i, r) in enumerate(zip(xs, infos, refs)):
            if r is None:
                assert i["iterations"] == 0 and i["status"] == 0
                continue
            assert i["iterations"] == r["iters"], k
            assert np.array_equal(i["hist"].numpy().view(np.uint64), r["hist"].view(np.uint64)), k
            assert np.array_equal(x.cpu().numpy().view(np.uint64), r["x"].view(np.uint64)), k
    B.close()


@pytest.mark.parametrize("mode", ["exblas", "fpe"])
@pytest.mark.parametrize("count", [1, 7, 300, 1400])
def test_many_small_systems(R, orc, count, mode):
    """1400 systems are held aligned (a slice each), fewer in the general copy."""
    print(f"batch of {count} {mode}", flush=True)
    _check(R, orc, _systems(count, 50 + count), mode)


@pytest.mark.parametrize("tile", [1, 3])
def test_more_runs_than_accumulator_copies(R, orc, tile):
    """A tile per slice: many runs of a system add to the same copies."""
    systems = [stencil7_varcoef_csr(N, 60 + N) for N in (9, 16, 21, 5)]
    _check(R, orc, systems, "exblas", policy=1, tile_slices=tile, grid_size=64, block_size=64)
    _check(R, orc, systems, "fpe", policy=0, grid_size=400, block_size=256)


@pytest.mark.parametrize("where", [0, 57, 99])
def test_malformed_row_pointers_are_refused(R, where):
    systems = [A for A in _systems(300, 9) if A.n > 8][:100]
    A = systems[where]
    for k, v in ((0, 1), (A.n, A.row_ptr[-1] - 1), (A.n // 2, A.row_ptr[-1] + 5), (A.n // 2, -3)):
        rp = A.row_ptr.copy()
        rp[k] = v
        mats = [R.CSR.from_host(S) for S in systems]
        mats[where] = R.CSR(A.n, torch.from_numpy(rp).cuda(), mats[where].col_idx, mats[where].val)
        with pytest.raises(R.RpcgError) as e:
            R.Batch(mats)
        assert e.value.status == R.ERR_INVALID
