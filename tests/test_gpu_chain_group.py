"""Chains small enough for one workgroup per batch row against the CPU oracle, at
the edges of what that form takes.  Needs a GPU."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL

import gpu_util as G
from test_gpu_chain import _check_chain, _run_chain

pytestmark = pytest.mark.gpu


def _in_one_workgroup(probs):
    """Whether a run takes the form: it leaves the other one-launch form's launch counters (4096 bytes in front of
    the status word) alone."""
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    plans = [G.dev_plan(p) for p in probs]
    mlp = B.pivot_mlp_plan(plans, 0)
    try:
        st = torch.cuda.current_stream().cuda_stream
        xd = torch.from_numpy(probs[0].x).cuda()
        yd = torch.empty((1, probs[-1].M), dtype=torch.float32, device="cuda")
        ws = G.workspace(B.pivot_mlp_workspace_bytes(mlp, 1))
        B.pivot_mlp_run(mlp, xd.data_ptr(), probs[0].K, yd.data_ptr(), probs[-1].M, 1, ws.data_ptr(), ws.numel(), st)
        torch.cuda.synchronize()
        counters = (ctypes.c_uint32 * 1024)()
        assert hip.hipMemcpy(counters, ctypes.c_void_p(B.pivot_mlp_status_word(mlp) - 4096), 4096, 2) == 0
        assert ("mlp_group_kernel" in B.pivot_mlp_kernel_name(mlp, 1)) == (not any(counters))
        return not any(counters)
    finally:
        B.pivot_mlp_plan_destroy(mlp)
        for h in plans:
            B.pivot_fc_plan_destroy(h)


# (tile height, width, sizes, kept): tiles of fewer rows than a wave-load covers (several tiles a load), of one and of several
# wave-loads; ragged sizes; inputs beyond 1024 columns; 2 to 5 layers; units that take turns on the wavefronts
@pytest.mark.parametrize("bh,bw,dims,kept,taken", [
    (16, 16, (256, 256, 256, 256), 1 / 16, True), (16, 16, (100, 90, 50), 0.3, True), (8, 16, (61, 75, 33), 0.4, True),
    (32, 32, (97, 130, 40), 0.3, True), (64, 64, (130, 70, 65), 0.4, None), (8, 64, (260, 72, 40, 24), 0.3, True),
    (64, 16, (150, 64, 64), 0.2, None), (16, 32, (3001, 40, 40, 19), 0.03, True), (16, 16, (2049, 40, 19), 0.02, False), (16, 16, (1025, 300, 10), 0.03, True),
    (16, 16, (17, 500, 33, 20), 0.1, True), (16, 16, (64, 48, 48, 48, 48, 20), 0.4, True),
    (16, 16, (512, 512, 512, 512), 1 / 16, True), (32, 32, (300, 300, 300, 300, 300), 0.15, None),
    (32, 32, (1024, 1024, 1024), 0.2, False)])
@pytest.mark.parametrize("eliminated", [False, True])
@pytest.mark.parametrize("wdtype", [WL.F32, WL.F16])
def test_chain_in_one_workgroup(wdtype, eliminated, bh, bw, dims, kept, taken):
    probs = WL.config4(seed=51 + bh + len(dims), dims=dims, eliminated=eliminated, bh=bh, bw=bw, frac=kept, wdtype=wdtype)
    _check_chain(probs, want_one_launch=True, repeats=3)
    _check_chain(probs, flags=B.PIVOT_MLP_KEEP_FINAL_BLOCK_ORDER, want_one_launch=True)
    if taken is not None:
        assert _in_one_workgroup(probs) == taken


@pytest.mark.parametrize("wdtype", [WL.F32, WL.F16])
def test_empty_block_rows_and_infinite_inputs(wdtype):
    # a layer without kept tiles, a block row without any; an infinite input reaches the rows that read it and no
    # other (padding of a wave-load meets no x), as with a launch per layer
    probs = WL.config4(seed=52, dims=(80, 90, 70, 33), bh=16, bw=16, frac=0.3, wdtype=wdtype)
    probs[0].tile_mask[1, :] = 0
    probs[2].tile_mask[:] = 0
    assert _in_one_workgroup(probs)
    _check_chain(probs, want_one_launch=True)
    probs = WL.config4(seed=53, dims=(80, 90, 70), bh=16, bw=16, frac=0.2, wdtype=wdtype)
    assert _in_one_workgroup(probs)
    probs[0].x[0, 5] = np.inf
    one = _run_chain(probs, want_one_launch=True)
    per_layer = _run_chain(probs, flags=B.PIVOT_MLP_LAUNCH_PER_LAYER, want_one_launch=False)
    for special in (np.isnan, np.isposinf, np.isneginf):
        assert (special(one) == special(per_layer)).all()
    assert not np.isfinite(one).all() and np.isfinite(one).any()


@pytest.mark.parametrize("batch", [2, 17, 64])
@pytest.mark.parametrize("wdtype", [WL.F32, WL.F16])
def test_batch_rows_equal_single_runs(wdtype, batch):
    # a workgroup per batch row: row for row the bits of runs of one, whatever lies between the rows of x and y
    probs = WL.config4(seed=54, batch=batch, dims=(203, 130, 75), bh=16, bw=16, frac=0.15, wdtype=wdtype)
    _check_chain(probs, want_one_launch=True)
    # three layers of 13-16 wave-loads a wavefront (fp32): from batch 2 on, at batch 1 in many workgroups that wait
    three = WL.config4(seed=55, batch=batch, dims=(600, 400, 200, 100), bh=64, bw=64, frac=0.1, wdtype=wdtype)
    _check_chain(three, want_one_launch=True, form="mlp_group_kernel<%s, 64, %d>" % (("float", 16) if wdtype == WL.F32 else ("_Float16", 8)))
    plans = [G.dev_plan(p) for p in three]
    mlp = B.pivot_mlp_plan(plans, 0)
    try:
        assert ("mlp_persist_kernel" if wdtype == WL.F32 else "mlp_group_kernel") in B.pivot_mlp_kernel_name(mlp, 1)
        for bad in (0, 65):
            with pytest.raises(B.PivotError):
                B.pivot_mlp_kernel_name(mlp, bad)
    finally:
        B.pivot_mlp_plan_destroy(mlp)
        for h in plans:
            B.pivot_fc_plan_destroy(h)
    plans = [G.dev_plan(p) for p in probs]
    mlp = B.pivot_mlp_plan(plans, 0)
    try:
        st = torch.cuda.current_stream().cuda_stream
        K, M, ldx, ldy = probs[0].K, probs[-1].M, probs[0].K + 3, probs[-1].M + 5
        x = torch.full((batch, ldx), float("nan")).to(torch.from_numpy(probs[0].x).dtype)
        x[:, :K] = torch.from_numpy(probs[0].x)
        xd = x.cuda()
        yd = torch.full((batch, ldy), 7.0, dtype=torch.float32, device="cuda")
        one = torch.zeros(batch, M, dtype=torch.float32, device="cuda")
        ws = G.workspace(B.pivot_mlp_workspace_bytes(mlp, batch))
        B.pivot_mlp_run(mlp, xd.data_ptr(), ldx, yd.data_ptr(), ldy, batch, ws.data_ptr(), ws.numel(), st)
        for b in range(batch):
            B.pivot_mlp_run(mlp, xd[b].data_ptr(), ldx, one[b].data_ptr(), M, 1, ws.data_ptr(), ws.numel(), st)
        torch.cuda.synchronize()
        assert torch.equal(yd[:, :M], one) and bool((yd[:, M:] == 7.0).all())
    finally:
        B.pivot_mlp_plan_destroy(mlp)
        for h in plans:
            B.pivot_fc_plan_destroy(h)


@pytest.mark.parametrize("batch,shift", [(2, 0), (8, 0), (64, 0), (8, 700)])
def test_outputs_stored_over_the_inputs(batch, shift):
    # several batch rows whose y lies in the memory of x: every row is read before any is overwritten, as with a
    # launch per layer (whose bits these are: the one-workgroup form is not taken)
    probs = WL.config4(seed=56, batch=batch, dims=(256, 200, 144), bh=16, bw=16, frac=0.15)
    plans = [G.dev_plan(p) for p in probs]
    res = []
    for flags, shared in ((0, True), (B.PIVOT_MLP_LAUNCH_PER_LAYER, False)):
        mlp = B.pivot_mlp_plan(plans, flags)
        try:
            st = torch.cuda.current_stream().cuda_stream
            K, M = probs[0].K, probs[-1].M
            buf = torch.zeros(batch * K + shift + batch * M, dtype=torch.float32, device="cuda")
            x = buf[:batch * K].view(batch, K)
            x.copy_(torch.from_numpy(probs[0].x))
            y = buf[shift:shift + batch * M].view(batch, M) if shared else torch.empty(batch, M, device="cuda")
            ws = G.workspace(B.pivot_mlp_workspace_bytes(mlp, batch))
            B.pivot_mlp_run(mlp, x.data_ptr(), K, y.data_ptr(), M, batch, ws.data_ptr(), ws.numel(), st)
            torch.cuda.synchronize()
            res.append(y.clone())
        finally:
            B.pivot_mlp_plan_destroy(mlp)
    for h in plans:
        B.pivot_fc_plan_destroy(h)
    assert torch.equal(res[0], res[1])
