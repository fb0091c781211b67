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


@pytest.mark.parametrize("M,K,bh,bw,batch", [(100, 4096, 16, 32, 16), (90, 2048, 16, 32, 16), (60, 2047, 32, 32, 16), (70, 2056, 64, 64, 9), (500, 600, 32, 16, 29), (70, 4095, 64, 16, 5), (64, 4089, 32, 16, 13), (2100, 33, 16, 64, 13), (4200, 9, 16, 32, 7),
                                               (1000, 4090, 16, 32, 64), (200, 4095, 64, 16, 33), (300, 4000, 64, 64, 47)])   # several launch rows, the last one short
def test_rows_of_any_alignment(M, K, bh, bw, batch):
    p = WL.gen_fc(M, K, bh, bw, 0.6 if batch <= 16 else 0.3, seed=5, wdtype=WL.F16, batch=batch, act=WL.ACT_NONE)
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


@pytest.mark.parametrize("M,K,bh,bw,frac,batch", [(300, 3000, 16, 32, 0.1, 8), (300, 3001, 64, 16, 0.08, 12), (400, 891, 16, 32, 0.4, 16), (200, 2100, 32, 64, 0.1, 33)])
def test_layers_that_stay_with_the_other_lds_form(M, K, bh, bw, frac, batch):
    # long rows of which little is staged, and short rows that are no whole vectors
    p = WL.gen_fc(M, K, bh, bw, frac, seed=8, wdtype=WL.F16, batch=batch, act=WL.ACT_RELU)
    plan = G.dev_plan(p)
    try:
        assert "fc_mfma_lds_kernel" in B.pivot_fc_kernel_name(plan, batch)
    finally:
        B.pivot_fc_plan_destroy(plan)
    G.check_fc(p)
