"""Parity of the batched matrix-core kernel (x in fragment order) and of the
two ways its input is made, at the sizes where they can go wrong: every tile
shape, odd tile counts, ragged sides, each side of a block of 16 batch rows,
split and empty block rows, rows of x too long or not aligned for the copy.
Needs a GPU.  Bounds: those of gpu_util (fp32 sums of n <= 16384 products,
worst case n * 2^-24 = 1e-3 of |W||x| and typically sqrt(n) * 2^-24 = 8e-6, here
measured below 1e-7; fp16 products are exact in fp32, so the same holds)."""
import numpy as np
import pytest
import torch

from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL

import gpu_util as G
from oracle import pivot_oracle as O
from test_gpu_chain import _check_chain, _run_chain

pytestmark = pytest.mark.gpu

SHAPES = [(bh, bw) for bh in (8, 16, 32, 64) for bw in (8, 16, 32, 64)]


@pytest.mark.parametrize("wdtype", [WL.F32, WL.F16])
@pytest.mark.parametrize("bh,bw", SHAPES)
def test_every_tile_shape_behind_a_boundary(bh, bw, wdtype):
    # a layer fed by another one in a launch of its own takes this kernel from batch 2 on, whatever its size
    for i, (batch, chunk) in enumerate([(2, 0), (15, 3), (16, 0), (17, 1), (33, 2), (64, 0)]):
        probs = WL.config4(seed=70 + i, batch=batch, dims=(100, 5 * bw + 3, 3 * bh - 1), bh=bh, bw=bw, frac=0.7, wdtype=wdtype,
                           eliminated=bool(i % 2))
        if i >= 4:
            probs[1].tile_mask[0, :] = 0            # an empty block row
        err, _ = _check_chain(probs, chunk_tiles=chunk, flags=B.PIVOT_MLP_LAUNCH_PER_LAYER)
        print("%s %dx%d batch %d: %.3g" % (wdtype, bh, bw, batch, err), flush=True)
        assert err <= 1e-5 or wdtype == WL.F16


@pytest.mark.parametrize("K,M,bh,bw,frac", [(3000, 200, 32, 32, 0.5), (3000, 100, 8, 32, 0.6), (2300, 70, 64, 16, 0.9), (400, 300, 16, 64, 0.5)])
def test_fp32_behind_a_boundary_few_batch_rows(K, M, bh, bw, frac):
    # batch 2-8: the vector kernel where work items are few and long, the batched one otherwise, on each side of the
    # batches where the choice changes; intermediates in rows or in fragment order
    for i, batch in enumerate((2, 3, 4, 5, 8, 9)):
        probs = WL.config4(seed=60 + i, batch=batch, dims=(50, K, M), bh=bh, bw=bw, frac=frac, eliminated=bool(i % 2))
        err, _ = _check_chain(probs, flags=B.PIVOT_MLP_LAUNCH_PER_LAYER)
        print("%d -> %d %dx%d batch %d: %.3g" % (K, M, bh, bw, batch, err), flush=True)
        assert err <= 1e-5


@pytest.mark.parametrize("wdtype,M,K,bh,bw,batch,frac", [
    (WL.F32, 2048, 2048, 32, 32, 3, 1.0),        # the smallest batch; every wavefront runs several rounds
    (WL.F32, 1000, 1501, 8, 8, 64, 0.8),         # stacked tiles, a ragged last column, all four batch blocks
    (WL.F32, 600, 2300, 64, 64, 37, 0.9),
    (WL.F32, 500, 30000, 16, 16, 17, 0.12),
    (WL.F16, 64, 16390, 8, 8, 64, 1.0),          # items of 768 tiles; rows of x copied into LDS
    (WL.F16, 200, 33000, 64, 32, 20, 0.5),       # rows of x too long for the copy
    (WL.F16, 100, 32768, 32, 32, 20, 0.2),       # the longest that is copied
    (WL.F16, 100, 32761, 32, 32, 20, 0.2),
    (WL.F16, 64, 32769, 16, 32, 9, 0.2),
    (WL.F16, 4096, 4100, 32, 32, 40, 0.2),
])
def test_natural_input(wdtype, M, K, bh, bw, batch, frac):
    p = WL.gen_fc(M, K, bh, bw, frac, seed=81, wdtype=wdtype, batch=batch, act=WL.ACT_RELU)
    plan = G.dev_plan(p)
    try:
        assert "fc_frag_kernel" in B.pivot_fc_kernel_name(plan, batch)
        st = torch.cuda.current_stream().cuda_stream
        y_ref, D = G.oracle_of(p)
        ws = G.workspace(B.pivot_fc_workspace_bytes(plan, batch))
        for off, ldx in ((0, K), (1, K + 3)):       # aligned, densely packed rows; and rows that are neither
            ws[B.pivot_fc_workspace_bytes(plan, batch) // 2:].fill_(0xFF)      # scratch of x and partial sums: NaN patterns
            G.B.pivot_workspace_init(ws.data_ptr(), ws.numel() // 2 // 4 * 4, st)
            buf = torch.full((batch * ldx + 8,), float("nan"), dtype=G.tdtype(p), device="cuda")
            rows = buf[off:off + batch * ldx].view(batch, ldx)
            rows[:, :K] = torch.from_numpy(p.x).cuda()
            y = torch.full((batch, M), float("nan"), device="cuda")
            B.pivot_fc_run(plan, rows.data_ptr(), ldx, y.data_ptr(), M, batch, ws.data_ptr(), ws.numel(), st)
            torch.cuda.synchronize()
            err = G.O.max_scaled_error(y.cpu().numpy().astype(np.float64), y_ref, D)
            print("%s %dx%d batch %d offset %d: %.3g" % (wdtype, M, K, batch, off, err), flush=True)
            assert err <= 1e-5
    finally:
        B.pivot_fc_plan_destroy(plan)


@pytest.mark.parametrize("wdtype", [WL.F32, WL.F16])
@pytest.mark.parametrize("bh,bw", SHAPES)
def test_infinities_reach_the_rows_of_their_tiles_and_stay_infinite(bh, bw, wdtype):
    # Tiles are taken in groups (up to 8 of them), whose last is filled up with copies of the item's last tile: an
    # infinity in that tile's x must not meet the copies' zero weights.  The first layer's bias puts the infinity
    # into one column of the second one's input, each time in another block row's last tile, behind which every
    # number of tiles from 1 to 11 occurs; with ReLU a NaN would be stored as 0.
    for i, (batch, act) in enumerate([(2, WL.ACT_RELU), (17, WL.ACT_NONE), (40, WL.ACT_RELU)]):
        probs = WL.config4(seed=90 + i, batch=batch, dims=(60, 11 * bw - 3, 11 * bh - 1), bh=bh, bw=bw, frac=0.7, wdtype=wdtype)
        p = probs[1]
        p.act = act
        p.tile_mask[:] = 0
        for br in range(11):
            p.tile_mask[br, np.random.default_rng(br).permutation(11)[:br + 1]] = 1
        br = (3, 4, 8)[i]
        c = int(np.flatnonzero(p.tile_mask[br])[-1]) * bw + 2
        j = int(p.pcol[c])
        probs[0].bias[j] = np.inf
        y = _run_chain(probs, flags=B.PIVOT_MLP_LAUNCH_PER_LAYER)
        h, _ = G.oracle_of(probs[0])
        h = h.astype(np.float16 if wdtype == WL.F16 else np.float32).astype(np.float64)
        assert np.isinf(h[:, j]).all() and np.isfinite(np.delete(h, j, axis=1)).all()
        kept = O.unpivot_weights(np.ascontiguousarray(O.expand_tile_mask(p.tile_mask, bh, bw, p.M, p.K)[:p.M, :p.K]), p.prow, p.pcol) != 0
        W = O.unpivot_weights(p.Wp, p.prow, p.pcol).astype(np.float64)
        W[~kept] = 0.0
        rows = kept[:, j]
        ref, D = O.fc_dense(W, np.where(np.isinf(h), 0.0, h), p.bias, act), O.error_scale(W, np.where(np.isinf(h), 0.0, h), p.bias)
        assert rows.any() and not rows.all() and (W[rows, j] != 0).all()
        want = np.where(W[rows, j] > 0, np.inf, 0.0 if act == WL.ACT_RELU else -np.inf)
        print("%s %dx%d batch %d: %d rows" % (wdtype, bh, bw, batch, rows.sum()), flush=True)
        assert np.array_equal(y[:, rows], np.broadcast_to(want, (batch, rows.sum())))
        assert O.max_scaled_error(y[:, ~rows], ref[:, ~rows], D[:, ~rows]) <= G.TOL[wdtype]


def test_static_scratch_takes_plans_whose_runs_need_few_counters():
    # 1040 split block rows: 16 launch rows of 4 batch rows would need more counters than the built-in scratch holds,
    # but no run of this plan takes that form while the copy of x fits
    p = WL.gen_fc(16640, 1088, 16, 32, 1.0, seed=83, wdtype=WL.F16, batch=40)
    plan = G.dev_plan(p, chunk_tiles=32)
    try:
        st = torch.cuda.current_stream().cuda_stream
        y_ref, D = G.oracle_of(p)
        for batch in (1, 40):
            xd, y = torch.from_numpy(p.x[:batch]).cuda(), torch.full((batch, p.M), float("nan"), device="cuda")
            B.pivot_fc_run_static(plan, xd.data_ptr(), p.K, y.data_ptr(), p.M, batch, st)
            torch.cuda.synchronize()
            assert G.O.max_scaled_error(y.cpu().numpy().astype(np.float64), y_ref[:batch], D[:batch]) <= 1e-5
    finally:
        B.pivot_fc_plan_destroy(plan)


def test_static_scratch_takes_shorter_launch_rows_where_long_ones_do_not_fit():
    # 3658 pieces of 16 rows: partial sums of one launch row of 64 batch rows are 15 MB, of three of 16 rows 11.2 MB, and
    # the nine launch rows of the kernel without a copy of x need too many counters.  Whole numbers: every order of
    # summation gives the same bits
    M, K, batch = 29264, 2112, 33
    rng = np.random.default_rng(84)
    W = np.ascontiguousarray(np.tile(rng.integers(-2, 3, (77, K)).astype(np.float16), (M // 77 + 1, 1))[:M])
    x = torch.from_numpy(rng.integers(-2, 3, (batch, K)).astype(np.float16)).cuda()
    ident = lambda n: np.arange(n, dtype=np.int32)
    plan = B.pivot_fc_plan(M, K, 16, 32, B.PIVOT_F16, W, B.PIVOT_W_PIVOTED, np.ones((M // 16, K // 32), np.uint8), ident(M), ident(K),
                           None, chunk_tiles=33, device=0)
    try:
        y = torch.full((batch, M), float("nan"), device="cuda")
        B.pivot_fc_run_static(plan, x.data_ptr(), K, y.data_ptr(), M, batch, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(y, x.float() @ torch.from_numpy(W).cuda().float().t())
    finally:
        B.pivot_fc_plan_destroy(plan)


def test_static_scratch_takes_many_pieces_of_short_rows():
    # 6400 pieces of 32 rows: partial sums of a launch row of 16 batch rows are 13 MB, of 8, which layers of so many work
    # items take at this batch, 6.6 MB.  Whole numbers: every order of summation gives the same bits
    M, K, batch = 12800, 2048, 6
    rng = np.random.default_rng(85)
    W = np.ascontiguousarray(np.tile(rng.integers(-2, 3, (77, K)).astype(np.float16), (M // 77 + 1, 1))[:M])
    x = torch.from_numpy(rng.integers(-2, 3, (batch, K)).astype(np.float16)).cuda()
    ident = lambda n: np.arange(n, dtype=np.int32)
    plan = B.pivot_fc_plan(M, K, 32, 32, B.PIVOT_F16, W, B.PIVOT_W_PIVOTED, np.ones((M // 32, K // 32), np.uint8), ident(M), ident(K),
                           None, chunk_tiles=4, device=0)
    try:
        y = torch.full((batch, M), float("nan"), device="cuda")
        B.pivot_fc_run_static(plan, x.data_ptr(), K, y.data_ptr(), M, batch, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(y, x.float() @ torch.from_numpy(W).cuda().float().t())
    finally:
        B.pivot_fc_plan_destroy(plan)


def test_static_scratch_without_room_for_the_copy():
    # 64 rows of 50000 fp32 columns are 12.8 MB, more than the built-in scratch holds: the kernels that need no copy run
    p = WL.gen_fc(96, 50000, 32, 32, 0.9, seed=82, batch=64)
    plan = G.dev_plan(p)
    try:
        assert "fc_frag_kernel" in B.pivot_fc_kernel_name(plan, 64)
        st = torch.cuda.current_stream().cuda_stream
        xd, y = torch.from_numpy(p.x).cuda(), torch.full((64, p.M), float("nan"), device="cuda")
        B.pivot_fc_run_static(plan, xd.data_ptr(), p.K, y.data_ptr(), p.M, 64, st)
        torch.cuda.synchronize()
        y_ref, D = G.oracle_of(p)
        assert G.O.max_scaled_error(y.cpu().numpy().astype(np.float64), y_ref, D) <= 1e-5
    finally:
        B.pivot_fc_plan_destroy(plan)
