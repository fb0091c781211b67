"""Performance cases: the calls that programs built on this library make, from
a layer of a few KB to matrices of hundreds of MB, each through the binding's
entry points as a program calls them (plan, workspace and buffers made once,
one run call per pass).

Three kinds of call: one layer (``pivot_fc_run``), a chain of layers
(``pivot_mlp_run``) and a recurrent sequence (``pivot_lstm_run``).  Plans are
BRC, the layout of every workload here; the other two layouts exist for the
layout study.  Batches go from one request to 64 (the most a call takes), both
weight types, tile sides 8 to 64, ragged sizes among them.  Inputs are drawn
from the seed alone with the distributions of ``workloads.py``; the weights
come from the GPU's generator, which is quicker than numpy's.
"""
import math

import numpy as np
import torch

from paper_1712_01084_amd import binding as B
from paper_1712_01084_amd import workloads as WL


def _layer(M, K, bh, bw, kept, mask, dtype, batch, act=1, name=None):
    c = dict(kind="layer", M=M, K=K, bh=bh, bw=bw, kept=kept, mask=mask, dtype=dtype, batch=batch, act=act)
    return dict(c, name=name) if name else c


def _chain(dims, bh, bw, kept, dtype, batch, eliminated=False, mask="balanced", name=None):
    c = dict(kind="chain", dims="-".join(str(d) for d in dims), bh=bh, bw=bw, kept=kept, mask=mask, dtype=dtype,
             batch=batch, eliminated=eliminated)
    return dict(c, name=name) if name else c


def _recurrent(H, I, steps, bh, bw, kept, mask, dtype, batch, name=None):
    c = dict(kind="recurrent", H=H, I=I, steps=steps, bh=bh, bw=bw, kept=kept, mask=mask, dtype=dtype, batch=batch)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one request to three small block-diagonal layers of the paper's grid (256 at 6.25 %: 16 blocks of
        # 16x16): the smallest call, where launches and latencies are everything
        _chain((256, 256, 256, 256), 16, 16, 0.0625, "f32", 1, mask="blockdiag", name="chain 256x3 f32 b1"),
        # one request to the AlexNet fc6 shape at the fullest fill-in of the paper's grid
        _layer(4096, 9216, 32, 32, 0.25, "balanced", "f32", 1, name="layer 4096x9216 f32 b1"),
        # sixteen requests served together, fp32, sizes that fit no tile
        _layer(3999, 9203, 32, 32, 0.10, "uniform", "f32", 16, name="layer 3999x9203 f32 b16"),
        # four and sixteen requests to the 4096 fp16 layer with tall narrow tiles
        _layer(4096, 4096, 64, 16, 0.50, "uniform", "f16", 4, act=0, name="layer 4096 f16 b4"),
        _layer(4096, 4096, 64, 16, 0.25, "uniform", "f16", 16, act=0, name="layer 4096 f16 b16"),
        # a full batch through a classifier layer of ragged sizes
        _layer(1000, 4090, 16, 32, 0.25, "uniform", "f16", 64, act=0, name="layer 1000x4090 f16 b64"),
        # one request to the largest matrix: bandwidth and nothing else
        _layer(16384, 16384, 64, 64, 0.25, "uniform", "f16", 1, name="layer 16384 f16 b1"),
        # the VGG classifier, one image at a time, and a batch of 32 in fp16
        _chain((25088, 4096, 4096, 1000), 32, 32, 0.10, "f32", 1, name="chain vgg f32 b1"),
        _chain((25088, 4096, 4096, 1000), 32, 32, 0.10, "f16", 32, name="chain vgg f16 b32"),
        # the LSTM: a whole sequence; one step per call with the state carried on, as a decoder that feeds its
        # output back calls it; and a larger batch of short sequences
        _recurrent(2048, 1024, 256, 16, 32, 0.125, "zipf", "f16", 8, name="lstm 256 steps f16 b8"),
        _recurrent(2048, 1024, 1, 16, 32, 0.125, "zipf", "f16", 8, name="lstm 1 step f16 b8"),
        _recurrent(1024, 512, 32, 16, 32, 0.125, "balanced", "f16", 32, name="lstm 32 steps f16 b32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, most):
    return 1 if rng.random() < 0.35 else _log(rng, 2, most)


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "chain", "recurrent"))
    dtype = rng.choice(("f32", "f16"))
    kept = round(math.exp(rng.uniform(math.log(0.05), math.log(0.5))), 4)
    if kind == "layer":
        M, K = _log(rng, 64, 12000), _log(rng, 64, 12000)
        if rng.random() < 0.15:
            kept = 1.0
        # no more weights than the largest listed layer keeps
        kept = min(kept, round(6.0e7 / (M * K), 4))
        return _layer(M, K, rng.choice((8, 16, 32, 64)), rng.choice((8, 16, 32, 64)), kept,
                      rng.choice(("uniform", "balanced", "zipf")), dtype, _batch(rng, 64), act=rng.choice((0, 1)))
    if kind == "chain":
        dims = [_log(rng, 200, 20000)] + [_log(rng, 200, 5000) for _ in range(rng.choice((2, 3)))]
        return _chain(dims, rng.choice((16, 32, 64)), rng.choice((16, 32, 64)), min(kept, 0.25), dtype, _batch(rng, 64),
                      eliminated=rng.random() < 0.5)
    return _recurrent(_log(rng, 64, 2048), _log(rng, 32, 1024), _log(rng, 1, 100), rng.choice((16, 16, 32)), 32,
                      min(kept, 0.25), rng.choice(("balanced", "zipf", "uniform")), dtype, rng.choice((1, 2, 4, 8, 16, 32)))


# ------------------------------------------------------------------ inputs

def _wd(case):
    return B.PIVOT_F32 if case["dtype"] == "f32" else B.PIVOT_F16


def _td(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float16


def _es(case):
    return 4 if case["dtype"] == "f32" else 2


def _grid(case, M, K):
    return -(-M // case["bh"]), -(-K // case["bw"])


def _mask(rng, case, M, K):
    nbr, nbc = _grid(case, M, K)
    if case["mask"] == "blockdiag":
        return WL.mask_block_diagonal(nbr)
    if case["mask"] == "balanced":
        return WL.mask_balanced(rng, nbr, nbc, case["kept"])
    if case["mask"] == "zipf":
        return WL.mask_zipf(rng, nbr, nbc, max(case["kept"], 1.0 / nbc))
    return WL.mask_uniform(rng, nbr, nbc, case["kept"])


def _tiles(case, M, K):
    """How many tiles _mask keeps (the count does not depend on the seed)."""
    nbr, nbc = _grid(case, M, K)
    if case["mask"] == "blockdiag":
        return nbr
    if case["mask"] == "balanced":
        return nbr * min(nbc, WL.balanced_row_count(case["kept"], nbc))
    if case["mask"] == "zipf":
        return int(round(max(case["kept"], 1.0 / nbc) * nbr * nbc))
    return int(round(case["kept"] * nbr * nbc))


class _State:
    """What a program keeps between calls: plans, workspace, buffers."""

    def __init__(self, case, seed):
        self.case = case
        self.rng = np.random.default_rng(seed)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.stream = torch.cuda.current_stream().cuda_stream
        self.plans, self.mlp = [], None

    def __del__(self):
        if self.mlp is not None:
            B.pivot_mlp_plan_destroy(self.mlp)
        for p in self.plans:
            B.pivot_fc_plan_destroy(p)

    def normal(self, *shape, sigma=1.0):
        return torch.randn(*shape, generator=self.gen, device="cuda").mul_(sigma)

    def plan(self, M, K, act, pcol=None):
        """One pruned layer: weights N(0, 1/K) in block space, bias N(0, 0.1^2), random permutations."""
        c = self.case
        W = self.normal(M, K, sigma=K ** -0.5).to(_td(c)).cpu().numpy()
        prow = self.rng.permutation(M).astype(np.int32)
        pcol = self.rng.permutation(K).astype(np.int32) if pcol is None else pcol
        bias = self.normal(M, sigma=0.1).cpu().numpy()
        self.plans.append(B.pivot_fc_plan(M, K, c["bh"], c["bw"], _wd(c), W, B.PIVOT_W_PIVOTED, _mask(self.rng, c, M, K),
                                          prow, pcol, bias, act=act, device=0))
        return self.plans[-1], prow

    def workspace(self, nbytes):
        self.nws = max(nbytes, 256)
        self.ws = torch.empty(self.nws, dtype=torch.uint8, device="cuda")
        B.pivot_workspace_init(self.ws.data_ptr(), self.nws, self.stream)


def _prepare_layer(case, seed):
    s = _State(case, seed)
    M, K, batch = case["M"], case["K"], case["batch"]
    p, _ = s.plan(M, K, case["act"])
    s.x = s.normal(batch, K).to(_td(case))
    if case["act"]:
        s.x.clamp_(min=0)                 # a layer with ReLU follows one with ReLU
    s.y = torch.zeros(batch, M, device="cuda")
    s.workspace(B.pivot_fc_workspace_bytes(p, batch))
    return s


def _run_layer(s):
    c = s.case
    B.pivot_fc_run(s.plans[0], s.x.data_ptr(), c["K"], s.y.data_ptr(), c["M"], c["batch"], s.ws.data_ptr(), s.nws, s.stream)
    return s.y


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _prepare_chain(case, seed):
    s = _State(case, seed)
    dims, batch, prow = _dims(case), case["batch"], None
    for l in range(len(dims) - 1):
        act = B.PIVOT_ACT_RELU if l + 2 < len(dims) else B.PIVOT_ACT_NONE
        _, prow = s.plan(dims[l + 1], dims[l], act, pcol=prow if case["eliminated"] else None)
    s.mlp = B.pivot_mlp_plan(s.plans)
    s.x = s.normal(batch, dims[0]).clamp_(min=0).to(_td(case))
    s.y = torch.zeros(batch, dims[-1], device="cuda")
    s.dims = dims
    s.workspace(B.pivot_mlp_workspace_bytes(s.mlp, batch))
    return s


def _run_chain(s):
    B.pivot_mlp_run(s.mlp, s.x.data_ptr(), s.dims[0], s.y.data_ptr(), s.dims[-1], s.case["batch"], s.ws.data_ptr(), s.nws,
                    s.stream)
    return s.y


def _prepare_recurrent(case, seed):
    s = _State(case, seed)
    H, I, steps, batch = case["H"], case["I"], case["steps"], case["batch"]
    p, _ = s.plan(4 * H, H + I, B.PIVOT_ACT_NONE)
    s.xs = s.normal(steps, batch, I).to(_td(case))
    s.h, s.c = torch.zeros(batch, H, device="cuda"), torch.zeros(batch, H, device="cuda")
    s.workspace(B.pivot_lstm_workspace_bytes(p, H, I, steps, batch))
    return s


def _run_recurrent(s):
    c = s.case
    if c["steps"] > 1:                    # a new sequence; a single step carries the state of the one before on
        s.h.zero_()
        s.c.zero_()
    B.pivot_lstm_run(s.plans[0], c["H"], c["I"], s.xs.data_ptr(), s.h.data_ptr(), s.c.data_ptr(), None, c["steps"],
                     c["batch"], s.ws.data_ptr(), s.nws, s.stream)
    return s.h, s.c


def prepare(case, seed):
    return {"layer": _prepare_layer, "chain": _prepare_chain, "recurrent": _prepare_recurrent}[case["kind"]](case, seed)


def run(state):
    return {"layer": _run_layer, "chain": _run_chain, "recurrent": _run_recurrent}[state.case["kind"]](state)


# ---------------------------------------------------------------- the floor

def _layer_bytes(case, M, K):
    """Kept tiles, their block columns, both permutations and the bias."""
    T = _tiles(case, M, K)
    return T * case["bh"] * case["bw"] * _es(case) + 4 * T + 4 * (_grid(case, M, K)[0] + 1) + 4 * K + 8 * M


def _layer_flops(case, M, K):
    return 2 * _tiles(case, M, K) * case["bh"] * case["bw"] * case["batch"]


def work(case):
    b, es = case["batch"], _es(case)
    if case["kind"] == "layer":
        M, K = case["M"], case["K"]
        return {"bytes": _layer_bytes(case, M, K) + b * (K * es + M * 4), "flops": _layer_flops(case, M, K)}
    if case["kind"] == "chain":
        d = _dims(case)
        return {"bytes": sum(_layer_bytes(case, m, k) for k, m in zip(d, d[1:])) + b * (d[0] * es + d[-1] * 4),
                "flops": sum(_layer_flops(case, m, k) for k, m in zip(d, d[1:]))}
    H, I, steps = case["H"], case["I"], case["steps"]
    # the weights once for the sequence, every input, the state in and out
    return {"bytes": _layer_bytes(case, 4 * H, H + I) + steps * b * I * es + 16 * b * H,
            "flops": steps * (_layer_flops(case, 4 * H, H + I) + 30 * b * H)}


def tolerance(case):
    """About four times what was measured between fp32 sums in another order and float64: single layers and
    fp32 chains 4e-7 (largest element 2.7e-6).  Where fp16 values stand between the sums (chains of fp16
    layers, the recurrent state) an element on a rounding boundary may round the other way: 1e-5 (2.4e-4).
    An fp32 recurrence adds the error of its exponentials."""
    if case["kind"] == "layer" or (case["kind"] == "chain" and case["dtype"] == "f32"):
        return {"rel": 1.5e-6, "max": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 4e-5, "max": 1e-3}
