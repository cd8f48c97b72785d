"""Calls at the edges of the rules that choose a kernel."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# FP64 buffers at 4-byte boundaries (a caller's byte arithmetic): only the
# one-cell kernels take them, with the result that aligned buffers give
@pytest.mark.parametrize("shape", [(9, 95, 512), (60, 96, 130)])
def test_varcoef_buffers_off_the_element(shape):
    import torch
    import paper_2303_08365_amd as st
    lib, rng, n = st.library(), np.random.default_rng(91), int(np.prod(shape))
    plan = st.varcoef_plan(shape, "f64")
    fields = [rng.random(shape), 0.5 + rng.random(shape), rng.random(shape)]
    steps, every = 5, 3

    def run(off):
        bufs = [torch.zeros(8 * n + 8, dtype=torch.uint8, device="cuda") for _ in range(9)]  # u, k, lambda, work, grad, 2 checkpoints, 2 states
        seg = torch.zeros(16 * n + 8, dtype=torch.uint8, device="cuda")
        for b, f in zip(bufs, fields):
            b[off:off + 8 * n].copy_(torch.from_numpy(f.reshape(-1).view(np.uint8)))
        u, k, lam, work, grad, c0, c1 = (b.data_ptr() + off for b in bufs[:7])
        ck = (ctypes.c_void_p * 2)(c0, c1)
        print(f"varcoef {shape} buffers at +{off}", flush=True)
        assert lib.stencil_run_ckpt(plan._h, u, work, k, 0.1, steps, every, ck, None) == 0
        assert lib.stencil_adjoint_run(plan._h, k, 0.1, None, ck, every, steps, lam, grad, seg.data_ptr() + off, work, None) == 0
        torch.cuda.synchronize()
        return [b[off:off + 8 * n].cpu().numpy().view(np.float64) for b in (bufs[0], bufs[2], bufs[4], bufs[5], bufs[6])]

    for a, b in zip(run(4), run(0)):
        assert np.array_equal(a, b)
