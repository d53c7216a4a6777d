"""GPU parity of the one-launch dot at the edges of its launch shapes (one
workgroup, one and two levels of tickets, short and odd lengths, vectors at
8-byte alignment), of the digit-wise wavefront flush over the exponent range,
and of calls that follow each other on one context."""

import numpy as np
import pytest

from rpcg_workloads import exdot_narrow, exdot_wide

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _bits(v):
    return np.float64(v).view(np.uint64)


@pytest.mark.parametrize("n", [0, 1, 2, 3, 63, 2047, 2049, 8191, 8193, 12289, 70001, 300007, 1050001])
@pytest.mark.parametrize("mode", ["exblas", "fpe"])
def test_lengths_and_alignment(R, orc, n, mode):
    for x, y in (exdot_narrow(n + 1, n), exdot_wide(n + 2, n)):
        want = orc.exdot(x, y)
        for sx, sy in ((0, 0), (1, 0), (1, 1)):  # offsets in elements: 16- and 8-byte aligned starts
            X = torch.zeros(n + sx + 1, dtype=torch.float64, device="cuda")[sx:sx + n]
            Y = torch.zeros(n + sy + 1, dtype=torch.float64, device="cuda")[sy:sy + n]
            X.copy_(torch.from_numpy(x))
            Y.copy_(torch.from_numpy(y))
            out, info = R.exdot(X, Y, mode=mode)
            assert _bits(out.item()) == _bits(want) and info["status"] == 0


@pytest.mark.parametrize("grid", [1, 2, 7, 8, 9, 64, 65, 71, 300])
def test_ticket_levels(R, orc, grid):
    x, y = exdot_narrow(77, 40_011)
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    want = orc.exdot(x, y)
    for mode in ("exblas", "fpe"):
        for block in (64, 256):
            out, info = R.exdot(X, Y, mode=mode, grid_size=grid, block_size=block)
            assert _bits(out.item()) == _bits(want) and info["grid_size"] == grid
    a = R.exdot(X, Y, mode="plain", grid_size=grid, block_size=64)[0].item()
    assert a == R.exdot(X, Y, mode="plain", grid_size=grid, block_size=64)[0].item()
    assert abs(a - want) <= 40_011 * 2.0 ** -53 * np.abs(x * y).sum()


@pytest.mark.parametrize("scale", [-530, -500, -300, 0, 300, 500, 505, 508])
def test_flush_over_the_exponent_range(R, orc, scale):
    """Products around 2^(2 scale), the top and the bottom of the exact domain included."""
    rng = np.random.default_rng(600 + scale)
    n = 4099
    lo = -480 if scale < -480 else scale  # |x y| >= 2^-969
    x = np.ldexp(rng.random(n) + 0.5, lo) * rng.choice([-1.0, 1.0], n)
    y = np.ldexp(rng.random(n) + 0.5, lo) * rng.choice([-1.0, 1.0], n)
    want = orc.exdot(x, y)
    for mode in ("exblas", "fpe"):
        for grid in (1, 5):
            out, info = R.exdot(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), mode=mode, grid_size=grid)
            assert info["status"] == 0
            assert _bits(out.item()) == _bits(want), (mode, grid)


def test_calls_in_a_row(R, orc):
    """More calls than the context has blocks, asynchronous ones and ones with
    a record mixed, an error among them: each starts from an empty block."""
    x, y = exdot_wide(5, 30_001)
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    bad = X.clone()
    bad[17] = float("inf")
    want = orc.exdot(x, y)
    outs = []
    for k in range(40):
        if k % 9 == 4:
            with pytest.raises(R.RpcgError):
                R.exdot(bad, Y)
        out, info = R.exdot(X, Y, mode=("exblas", "fpe")[k % 2], sync=k % 3 == 0, grid_size=(0, 3, 90)[k % 3] or None)
        outs.append(out)
    digits = R.exdot_partial(X, Y)
    for out in outs:
        assert _bits(out.item()) == _bits(want)
    assert _bits(R.acc_round(digits).item()) == _bits(want)


def test_result_is_in_place_when_the_call_returns(R, orc):
    """With a record the call waits: another stream may read the result at once."""
    x, y = exdot_narrow(9, 200_003)
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    want = orc.exdot(x, y)
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    for _ in range(20):
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        R.exdot(X, Y, out=out)
        with torch.cuda.stream(other):
            got = out.clone()
        other.synchronize()
        assert _bits(got.item()) == _bits(want)
