"""FPE mode of the standalone dot: the record counts what an expansion could not
hold, and nothing else. Eight terms hold about 424 bits, so products over 150
binades leave no remainder, with the fallback as without it; and a lane that
has not ended its first measurement window counts the same either way."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    rpcg.context(0)
    return rpcg


def _spread(n, span, seed):
    """Vectors whose products spread over about `span` binades."""
    rng = np.random.default_rng(seed)
    e = rng.integers(0, span // 2 + 1, n) - span // 4
    return np.ldexp(1.0 + rng.random(n), e), np.ldexp(1.0 + rng.random(n), e) * rng.choice([-1.0, 1.0], n)


def _dot(R, x, y, noalloc, **kw):
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    if not noalloc:
        out, info = R.exdot(X, Y, mode="fpe", **kw)
        return out, info
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    return out, R.exdot_noalloc(X, Y, out, mode="fpe", **kw)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n", [100, 5000, 70_001, 1_000_003])
def test_eight_terms_hold_150_binades(R, orc, n, noalloc):
    x, y = _spread(n, 150, n)
    want = np.float64(orc.exdot(x, y)).view(np.uint64)
    for fallback in (1, 0):
        out, info = _dot(R, x, y, noalloc, fpe_size=8, fpe_fallback=fallback)
        assert np.float64(out.item()).view(np.uint64) == want
        assert (info["fpe_escapes"], info["fallbacks"], info["status"]) == (0, 0, 0), fallback


@pytest.mark.parametrize("n", [100, 5000])
@pytest.mark.parametrize("span", [140, 200, 300])
def test_short_dots_count_the_same_with_the_fallback(R, n, span):
    """Fewer than 32 products a lane: no lane has measured itself yet."""
    x, y = _spread(n, span, span + n)
    kept = _dot(R, x, y, False, fpe_size=4, fpe_fallback=1)[1]
    dropped = _dot(R, x, y, False, fpe_size=4, fpe_fallback=0)[1]
    assert kept["fpe_escapes"] == dropped["fpe_escapes"] > 0
    assert kept["fallbacks"] == 1 and kept["status"] == 0 and dropped["status"] == 2  # expansions inexact


@pytest.mark.parametrize("n", [1 << 23, (1 << 24) + 1, 1 << 26])
def test_one_workgroup_per_cu(R, orc, n):
    """Up to 2^27 pairs a second workgroup per CU costs more merges and windows than it hides latency."""
    x = torch.ones(n, dtype=torch.float64, device="cuda")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    out, info = R.exdot(x, x, mode="fpe")
    assert out.item() == n and info["grid_size"] == cus and info["fpe_escapes"] == 0
