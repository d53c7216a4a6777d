"""A new context is ready for every stream: its first dots run on a stream that
does not wait for the default stream, while that one is still busy with the work
that was ahead of the context's own initialisation."""

import ctypes

import numpy as np
import pytest

from rpcg_workloads import exdot_wide

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_first_dots_of_a_context_on_a_side_stream(orc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_07282_amd import rpcg
    L = rpcg.lib()
    x, y = exdot_wide(3, 50_021)
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    want = np.float64(orc.exdot(x, y)).view(np.uint64)
    busy = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    for mode in ("exblas", "fpe"):
        outs = torch.zeros(40, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        for _ in range(20):
            busy = (busy @ busy).clamp(-1, 1)
        h = ctypes.c_void_p()
        assert L.rpcg_create(ctypes.byref(h), X.device.index or 0) == 0
        with torch.cuda.stream(side):
            for k in range(40):
                assert L.rpcg_exdot(h, rpcg.MODES[mode], x.size, X.data_ptr(), Y.data_ptr(), outs[k:].data_ptr(), None,
                                    None, side.cuda_stream) == 0
        side.synchronize()
        got = outs.cpu().numpy().view(np.uint64)
        torch.cuda.synchronize()
        L.rpcg_destroy(h)
        assert (got == want).all()
