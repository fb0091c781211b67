"""The one-launch recurrent form whose workgroups own whole units: every
instantiation, ragged sizes, both weight types and several tile shapes against
the CPU oracle, and infinities and NaNs against the launch-per-step form.
Needs a GPU."""
import numpy as np
import pytest
import torch

from oracle import pivot_oracle as O
from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL

import gpu_util as G
from test_gpu_chain import FREE_RUN_GATE, _lstm_gpu

pytestmark = pytest.mark.gpu


def _problem(H, I, steps, batch, bh, bw, wdtype, frac, seed=11):
    rng = np.random.default_rng(seed)
    fc = WL.gen_fc(4 * H, H + I, bh, bw, frac, seed, mask="uniform", wdtype=wdtype, batch=batch, act=WL.ACT_NONE, rng=rng, draw_x=False)
    td = np.float16 if wdtype == WL.F16 else np.float32
    xs = rng.standard_normal((steps, batch, I)).astype(td)
    h0 = (0.5 * rng.standard_normal((batch, H))).astype(np.float32)
    c0 = rng.standard_normal((batch, H)).astype(np.float32)
    return WL.LSTMProblem(fc, H, I, xs, h0, c0)


# (H, I, batch, bh, bw, dtype) and the form it takes on 256 compute units: every instantiation of both types; one or two
# buffers of sums; up to eight teams, the last one short; H and I no multiples of anything (the copy of x), at the edges
# of a k-step and the largest of a form
CASES = [((64, 32, 1, 16, 32, "f16"), "2, 8, 1, true> teams 1 sums 2"), ((65, 33, 8, 8, 8, "f16"), "2, 8, 1, true> teams 1 sums 2"),
         ((31, 1, 3, 16, 16, "f16"), "2, 8, 1, true> teams 1 sums 2"), ((512, 256, 8, 64, 64, "f16"), "2, 8, 1, true> teams 1 sums 2"),
         ((1100, 40, 2, 16, 32, "f16"), "2, 16, 1, true> teams 1 sums 2"), ((2048, 8, 7, 16, 32, "f16"), "2, 16, 1, true> teams 1 sums 2"),
         ((513, 33, 12, 32, 16, "f16"), "2, 8, 1, false> teams 1 sums 2"), ((1024, 1024, 16, 16, 64, "f16"), "2, 8, 1, false> teams 1 sums 1"),
         ((400, 24, 40, 16, 64, "f16"), "4, 8, 1, false> teams 3 sums 2"), ((1000, 500, 32, 16, 32, "f16"), "2, 8, 2, false> teams 1 sums 2"),
         ((900, 1000, 30, 8, 16, "f16"), "2, 8, 2, false> teams 1 sums 1"), ((200, 96, 64, 16, 32, "f16"), "2, 8, 1, false> teams 4 sums 2"),
         ((70, 13, 5, 8, 16, "f32"), "2, 8, 1, true> teams 1 sums 2"), ((256, 128, 8, 16, 32, "f32"), "2, 8, 1, true> teams 1 sums 2"),
         ((700, 4, 3, 32, 8, "f32"), "2, 16, 1, true> teams 1 sums 2"), ((1000, 500, 8, 16, 32, "f32"), "2, 16, 1, true> teams 1 sums 2"),
         ((400, 24, 12, 16, 32, "f32"), "2, 8, 1, true> teams 2 sums 2"), ((250, 60, 20, 64, 64, "f32"), "2, 8, 1, true> teams 3 sums 2"),
         ((300, 300, 48, 8, 8, "f32"), "2, 8, 1, false> teams 3 sums 2"), ((512, 200, 64, 16, 32, "f32"), "4, 8, 1, false> teams 4 sums 1"),
         ((512, 300, 64, 32, 32, "f32"), "2, 8, 2, false> teams 2 sums 2"), ((512, 400, 64, 16, 16, "f32"), "2, 8, 2, false> teams 2 sums 1")]


def _check_form(plan, steps, batch, form):
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert B.pivot_lstm_kernel_name(plan, steps, batch).endswith(form)
    assert B.pivot_lstm_kernel_name(plan, steps, batch).startswith("lstm_units_kernel<")


@pytest.mark.parametrize("sizes,form", CASES)
def test_sequence_against_the_oracle(sizes, form):
    H, I, batch, bh, bw, dtype = sizes
    # fp32 sums of fp16 or fp32 products in another order, sigmoids of fp32: the free-run gate of the other forms
    wdtype = WL.F16 if dtype == "f16" else WL.F32
    lp = _problem(H, I, 5, batch, bh, bw, wdtype, 0.3)
    p = lp.fc
    Wd = O.dense_masked_natural(p.Wp, p.tile_mask, p.prow, p.pcol, p.bh, p.bw)
    h_ref, c_ref, _ = O.oracle_lstm(Wd, p.bias, lp.xs, lp.h0, lp.c0, H, state_dtype=np.float16 if dtype == "f16" else np.float32)
    plan = G.dev_plan(p, flags=B.PIVOT_PLAN_LSTM_ONE_LAUNCH_ALWAYS)
    try:
        _check_form(plan, 5, batch, form)
        h, c, z = _lstm_gpu(lp, plan, lp.xs, lp.h0, lp.c0)
        assert np.abs(h - h_ref).max() < FREE_RUN_GATE and np.abs(c - c_ref).max() < FREE_RUN_GATE
        assert np.isfinite(z).all()
        h2, c2, z2 = _lstm_gpu(lp, plan, lp.xs, lp.h0, lp.c0)
        assert np.array_equal(h, h2) and np.array_equal(c, c2) and np.array_equal(z, z2)
    finally:
        B.pivot_fc_plan_destroy(plan)


# (one team, eight teams, two batch blocks per team; the form that exchanges gate sums, its last workgroup with 11 tiles)
@pytest.mark.parametrize("H,I,batch,dtype,frac", [(300, 96, 3, "f32", 0.3), (200, 96, 64, "f16", 0.3), (1000, 500, 32, "f16", 0.3),
                                                  (512, 1100, 8, "f16", 0.313)])
def test_a_run_that_gives_up_can_be_taken_back(H, I, batch, dtype, frac):
    # the last workgroup is missing: those of its team give up after 2^18 polls (every kernel exits by itself), the other
    # teams are through and have written their h and c by then
    lp = _problem(H, I, 6, batch, 16, 32, WL.F16 if dtype == "f16" else WL.F32, frac, seed=6)
    st = torch.cuda.current_stream().cuda_stream
    xs, h, c = torch.from_numpy(lp.xs).cuda(), torch.from_numpy(lp.h0).cuda(), torch.from_numpy(lp.c0).cuda()

    def run(flags, h, c):
        plan = G.dev_plan(lp.fc, flags=flags)
        try:
            ws = G.workspace(B.pivot_lstm_workspace_bytes(plan, H, I, 6, batch))
            B.pivot_lstm_run(plan, H, I, xs.data_ptr(), h.data_ptr(), c.data_ptr(), None, 6, batch, ws.data_ptr(), ws.numel(), st)
            B.pivot_lstm_restore(plan, 6, batch, ws.data_ptr(), h.data_ptr(), c.data_ptr(), st)
            return B.pivot_lstm_status(plan, 6, batch, ws.data_ptr(), st)
        finally:
            B.pivot_fc_plan_destroy(plan)
    for _ in range(2):
        assert run(B.PIVOT_PLAN_LSTM_GIVE_UP, h, c) == 1
        assert np.array_equal(h.cpu().numpy(), lp.h0) and np.array_equal(c.cpu().numpy(), lp.c0)     # put back
    h2, c2 = h.clone(), c.clone()
    assert run(0, h, c) == 0 and run(B.PIVOT_PLAN_LSTM_LAUNCH_PER_STEP, h2, c2) == 0        # the caller can run it again
    assert (h - h2).abs().max() < 2e-3 and (c - c2).abs().max() < 4e-3


def test_four_streams_at_once():
    # half the compute units' worth of workgroups each, half a compute unit per workgroup: four launches, as many as a
    # process has hardware queues, are resident together and wait for none of the others
    lp = _problem(1024, 96, 40, 32, 16, 32, WL.F16, 0.1, seed=9)
    plan = G.dev_plan(lp.fc)
    try:
        xs = torch.from_numpy(lp.xs).cuda()
        nws = B.pivot_lstm_workspace_bytes(plan, 1024, 96, 40, 32)
        jobs = [(torch.cuda.Stream(), torch.from_numpy(lp.h0).cuda(), torch.from_numpy(lp.c0).cuda(), G.workspace(nws)) for _ in range(5)]
        torch.cuda.synchronize()

        def enqueue(job):
            s, h, c, ws = job
            B.pivot_lstm_run(plan, 1024, 96, xs.data_ptr(), h.data_ptr(), c.data_ptr(), None, 40, 32, ws.data_ptr(), ws.numel(), s.cuda_stream)
        for _ in range(4):                               # the state goes on from run to run
            for job in jobs[:4]:
                enqueue(job)
        torch.cuda.synchronize()
        for _ in range(4):
            enqueue(jobs[4])                             # alone
            torch.cuda.synchronize()
        for s, h, c, ws in jobs:
            assert B.pivot_lstm_status(plan, 40, 32, ws.data_ptr(), s.cuda_stream) == 0
            assert torch.equal(h, jobs[4][1]) and torch.equal(c, jobs[4][2])
    finally:
        B.pivot_fc_plan_destroy(plan)


@pytest.mark.parametrize("sizes,form", [((96, 40, 3, "f16"), "2, 8, 1, true> teams 1 sums 2"), ((96, 40, 3, "f32"), "2, 8, 1, true> teams 1 sums 2"),
                                        ((400, 24, 40, "f16"), "4, 8, 1, false> teams 3 sums 2"), ((512, 200, 64, "f32"), "4, 8, 1, false> teams 4 sums 1"),
                                        ((900, 1000, 30, "f16"), "2, 8, 2, false> teams 1 sums 1"), ((512, 300, 64, "f32"), "2, 8, 2, false> teams 2 sums 2"),
                                        ((1024, 1000, 16, "f16"), "2, 8, 1, false> teams 1 sums 1")])
@pytest.mark.parametrize("what", ["inf x", "nan x", "inf h", "nan h"])
def test_infinities_and_nans_reach_the_rows_of_kept_tiles_only(sizes, form, what):
    # columns outside the kept tiles are zeros in this form's dense rows; a product with an infinity must not count
    H, I, batch, dtype = sizes
    wdtype = WL.F16 if dtype == "f16" else WL.F32
    lp = _problem(H, I, 4, batch, 16, 32, wdtype, 0.25, seed=4)
    bad = np.inf if what.startswith("inf") else np.nan
    if what.endswith("x"):
        lp.xs[1, batch - 1, 7], lp.xs[2, 0, I - 1] = bad, -bad
    else:
        lp.h0[1, 5] = bad
    res = []
    for flags in (B.PIVOT_PLAN_LSTM_ONE_LAUNCH_ALWAYS, B.PIVOT_PLAN_LSTM_LAUNCH_PER_STEP):
        plan = G.dev_plan(lp.fc, flags=flags)
        try:
            if flags == B.PIVOT_PLAN_LSTM_ONE_LAUNCH_ALWAYS:
                _check_form(plan, 4, batch, form)
            # the step that meets the value, and a few behind it
            res.append([_lstm_gpu(lp, plan, lp.xs[:n], lp.h0, lp.c0) for n in (1, 2, 4)])
        finally:
            B.pivot_fc_plan_destroy(plan)
    for one, per in zip(*res):
        for a, b in zip(one, per):
            assert np.array_equal(np.isnan(a), np.isnan(b))
            fin = np.isfinite(b)
            assert np.array_equal(a[~fin & ~np.isnan(b)], b[~fin & ~np.isnan(b)])
            assert np.abs(a[fin] - b[fin]).max() < 20 * FREE_RUN_GATE if fin.any() else True
