"""What a dot with a record promises when it returns: the work enqueued on its
stream before has been done and the host sees its results, without any further wait."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [100, 9001, 300_007])
def test_earlier_work_is_in_place(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg as R
    s = torch.cuda.Stream()
    host = torch.zeros(1 << 20, dtype=torch.float64, pin_memory=True)
    x = torch.ones(n, dtype=torch.float64, device="cuda")
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for k in range(1, 12):
            v = torch.full((1 << 20,), float(k), dtype=torch.float64, device="cuda")
            for _ in range(k):
                v = v + 1.0
            host.copy_(v, non_blocking=True)
            _, info = R.exdot(x, x, out=out)
            seen = host.numpy()
            assert (seen[::4099] == 2.0 * k).all() and seen[-1] == 2.0 * k
            assert info["status"] == 0
            x += 1.0 / 1024.0
    s.synchronize()
    assert np.isfinite(out.item())
