"""The matrix-core kernel that gathers its fragments from a copy of the rows of x in LDS: rows of any alignment, up to the
longest (4096 columns, one 16-byte piece more where they are not aligned), with values beyond them that must not count.
Needs a GPU."""
import numpy as np
import pytest
import torch

from oracle import pivot_oracle as O
from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL

import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,bh,bw,batch", [(100, 4096, 16, 32, 16), (70, 4095, 64, 16, 5), (64, 4089, 32, 16, 13), (33, 1, 16, 64, 7), (40, 9, 16, 32, 16),
                                               (1000, 4090, 16, 32, 64), (200, 4095, 64, 16, 33), (300, 4000, 64, 64, 47)])   # several launch rows, the last one short
def test_rows_of_any_alignment(M, K, bh, bw, batch):
    p = WL.gen_fc(M, K, bh, bw, 0.6 if batch <= 16 else 0.35, seed=5, wdtype=WL.F16, batch=batch, act=WL.ACT_NONE)
    y_ref, D = O.oracle_fc(p.Wp, p.tile_mask, p.prow, p.pcol, p.bias, p.x, bh, bw, p.act, return_scale=True)
    plan = G.dev_plan(p)
    try:
        assert "fc_mfma_xrow_kernel" in B.pivot_fc_kernel_name(plan, batch)
        ws = G.workspace(max(256, B.pivot_fc_workspace_bytes(plan, batch)))
        st = torch.cuda.current_stream().cuda_stream
        for ldx in (K, K + 1, K + 7, K + 8):
            for off in (0, 1, 4, 7):
                print("K %d ldx %d offset %d" % (K, ldx, off), flush=True)
                buf = torch.full((16 + off + batch * ldx,), float("nan"), dtype=torch.float16, device="cuda")
                x = buf[8 + off:8 + off + batch * ldx].view(batch, ldx)
                x[:, :K] = torch.from_numpy(p.x).cuda()
                y = torch.full((batch, M), float("nan"), device="cuda")
                B.pivot_fc_run(plan, x.data_ptr(), ldx, y.data_ptr(), M, batch, ws.data_ptr(), ws.numel(), st)
                assert O.max_scaled_error(y.cpu().numpy(), y_ref, D) <= G.TOL[p.wdtype], (ldx, off)
    finally:
        B.pivot_fc_plan_destroy(plan)
