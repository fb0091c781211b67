"""The launch that places the inputs of the launch-per-step recurrent form: each side of the line between its two
workgroup sizes, ragged sizes, and recurrences without inputs.  Needs a GPU."""
import numpy as np
import pytest
import torch

from oracle import pivot_oracle as O
from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL

import gpu_util as G
from test_gpu_chain import FREE_RUN_GATE
from test_gpu_lstm_units import _problem

pytestmark = pytest.mark.gpu


# groups of 16 bytes of one step's input, all batch rows: 192 and 208 (fp32), 120 and 132 (fp16)
@pytest.mark.parametrize("H,I,batch,wdtype", [(48, 16, 12, WL.F32), (48, 16, 13, WL.F32), (64, 32, 10, WL.F16), (64, 32, 11, WL.F16), (31, 6, 1, WL.F32),
                                               (33, 1, 3, WL.F16), (500, 77, 9, WL.F16), (300, 80, 64, WL.F32),
                                               (64, 0, 1, WL.F32), (64, 0, 5, WL.F16), (61, 0, 40, WL.F32), (200, 0, 40, WL.F16)])
@pytest.mark.parametrize("steps", [1, 3])
def test_inputs_of_launches_per_step(H, I, batch, wdtype, steps):
    lp = _problem(H, I, steps, batch, 16, 32, wdtype, 0.4)
    p = lp.fc
    Wd = O.dense_masked_natural(p.Wp, p.tile_mask, p.prow, p.pcol, p.bh, p.bw)
    h_ref, c_ref, _ = O.oracle_lstm(Wd, p.bias, lp.xs, lp.h0, lp.c0, H, state_dtype=np.float16 if wdtype == WL.F16 else np.float32)
    plan = G.dev_plan(p, flags=B.PIVOT_PLAN_LSTM_LAUNCH_PER_STEP)
    try:
        # NaN around the inputs, and in their place where there are none
        xs = torch.full((lp.xs.size + 64,), float("nan"), dtype=G.tdtype(p), device="cuda")
        xs[32:32 + lp.xs.size] = torch.from_numpy(lp.xs).cuda().view(-1)
        n = B.pivot_lstm_workspace_bytes(plan, H, I, steps, batch)
        ws = torch.full((n + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        st = torch.cuda.current_stream().cuda_stream
        res = []
        B.pivot_workspace_init(ws.data_ptr(), n, st)
        for _ in range(2):
            h, c = torch.from_numpy(lp.h0).cuda(), torch.from_numpy(lp.c0).cuda()
            B.pivot_lstm_run(plan, H, I, xs[32:].data_ptr(), h.data_ptr(), c.data_ptr(), None, steps, batch, ws.data_ptr(), n, st)
            assert B.pivot_lstm_status(plan, steps, batch, ws.data_ptr(), st) == 0
            res.append((h.cpu().numpy(), c.cpu().numpy()))
        assert np.abs(res[0][0] - h_ref).max() < FREE_RUN_GATE and np.abs(res[0][1] - c_ref).max() < FREE_RUN_GATE
        assert res[0][0].tobytes() == res[1][0].tobytes() and res[0][1].tobytes() == res[1][1].tobytes()
        assert bool((ws[n:] == 0xFF).all())
    finally:
        B.pivot_fc_plan_destroy(plan)
