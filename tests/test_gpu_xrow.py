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
                                               (1000, 4090, 16, 32, 64), (200, 4095, 64, 16, 33), (300, 4000, 64, 64, 47),   # several launch rows, the last one short
                                               (90, 2048, 16, 32, 64), (90, 1999, 16, 32, 61), (300, 1999, 32, 16, 60), (70, 2047, 16, 64, 64)])   # short rows of any alignment: where the other LDS form does not fit
def test_rows_of_any_alignment(M, K, bh, bw, batch, row_slices=0):
    p = WL.gen_fc(M, K, bh, bw, 0.6 if batch <= 16 else 0.3, seed=5, wdtype=WL.F16, batch=batch, act=WL.ACT_NONE)
    y_ref, D = O.oracle_fc(p.Wp, p.tile_mask, p.prow, p.pcol, p.bias, p.x, bh, bw, p.act, return_scale=True)
    plan = G.dev_plan(p, row_slices=row_slices)
    try:
        # (few columns in rows that are no whole vectors: the other LDS form)
        assert ("fc_mfma_xrow_kernel" if K > 64 else "fc_mfma_lds_kernel") in B.pivot_fc_kernel_name(plan, batch)
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


@pytest.mark.parametrize("M,K,bh,batch", [(300, 1999, 32, 60), (200, 2041, 64, 64)])
def test_rows_of_any_alignment_whole_row_blocks(M, K, bh, batch):
    # 32x32x16 matrix instructions: slices of 32 and 64 rows of 16-column tiles
    test_rows_of_any_alignment(M, K, bh, 16, batch, row_slices=1)


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


@pytest.mark.parametrize("M,K,bh,bw,chunk,batch", [(200, 1024, 32, 32, 8, 6), (200, 1024, 32, 32, 8, 15), (130, 600, 64, 16, 10, 24), (100, 1024, 16, 64, 5, 17)])
def test_split_block_rows_whose_x_is_not_aligned(M, K, bh, bw, chunk, batch):
    # counters and partial sums are those of the aligned rows' form, also where other rows take the one with launch rows
    # of 8; both leave the counters at zero, and nothing behind the workspace is touched
    p = WL.gen_fc(M, K, bh, bw, 0.7, seed=9, wdtype=WL.F16, batch=batch, act=WL.ACT_NONE)
    y_ref, D = O.oracle_fc(p.Wp, p.tile_mask, p.prow, p.pcol, p.bias, p.x, bh, bw, p.act, return_scale=True)
    plan = G.dev_plan(p, chunk_tiles=chunk)
    try:
        assert "fc_mfma_xrow_kernel" in B.pivot_fc_kernel_name(plan, batch)
        n = B.pivot_fc_workspace_bytes(plan, batch)
        ws = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        st = torch.cuda.current_stream().cuda_stream
        B.pivot_workspace_init(ws.data_ptr(), n, st)
        for off, ldx in ((0, K), (0, K + 8), (3, K), (0, K), (1, K + 5)):
            print("%dx%d batch %d ldx %d offset %d" % (M, K, batch, ldx, off), flush=True)
            buf = torch.full((off + batch * ldx + 8,), float("nan"), dtype=torch.float16, device="cuda")
            x = buf[off:off + batch * ldx].view(batch, ldx)
            x[:, :K] = torch.from_numpy(p.x).cuda()
            for run in (lambda y: B.pivot_fc_run(plan, x.data_ptr(), ldx, y.data_ptr(), M, batch, ws.data_ptr(), n, st),
                        lambda y: B.pivot_fc_run_static(plan, x.data_ptr(), ldx, y.data_ptr(), M, batch, st)):
                y = torch.full((batch, M), float("nan"), device="cuda")
                run(y)
                assert O.max_scaled_error(y.cpu().numpy(), y_ref, D) <= G.TOL[p.wdtype], (ldx, off)
        assert bool((ws[n:] == 0x5A).all())
    finally:
        B.pivot_fc_plan_destroy(plan)
