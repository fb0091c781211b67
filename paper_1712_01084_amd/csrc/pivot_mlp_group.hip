// A chain of at most 256 KB of weights in ONE workgroup per batch row.  The
// one-launch form over many workgroups (pivot_mlp_persist.hip) pays a
// device-wide exchange of about 1.8 us per boundary, a launch per layer, which
// larger batches of larger chains take, an empty launch's turnaround and a
// trip; here a boundary is an LDS barrier.  Batch rows meet only in the
// caches: each has a compute unit of its own, which reads the weights at the
// rate it would read them alone.
//
// The chain plan holds the tile values once more, in the order in which the
// sixteen wavefronts take them: slot k of wavefront w is the 1 KB at
// (16 k + w) KB, beside it, per lane, where its piece of the input stands in
// LDS, where its output goes, and the bias.  No address depends on another
// load: the first eight slots (up to 128 KB, the whole of most chains) and up
// to 1024 elements of x are requested at kernel start and come in one trip; a
// later slot is requested when the one eight before it is consumed, further x
// in turns of 1024 with a trip each.  Then an LDS gather of x and one LDS
// barrier per layer.  A wavefront takes
// whole units (the rows of one wave-load of a block row), so no sums cross
// wavefronts; layer ends fall on the same slot in all of them.  Intermediates
// of fp16 chains are rounded to fp16 once, like those of the other forms.
//
// What bounds it: the launch and one trip to memory; beyond about 64 KB the rate of one compute unit.  Us per run in
// replayed graphs, many workgroups / one: 256-256-256-256 block-diagonal 16x16 fp32 (48 KB) 6.1 / 2.65 (eager calls 6.2 /
// 3.7, the host's), eight such layers (128 KB) 13.0 / 4.9; 512-512-512-512 fp16 6 % kept (96 KB) 6.5 / 4.2, 512-512-512
// 32x32 fp16 10 % (128 KB) 4.9 / 4.15, 200-200-200 fp16 4.8 / 2.45.  Of several batch rows, a launch per layer / this form,
// batch 2, 8, 64: the first 6.9 / 2.8, 7.3 / 2.8, 7.9 / 2.9 (eager calls 13.5 / 3.9), the 128 KB fp16 chain 5.5 / 4.4, 6.1 /
// 4.5, 6.7 / 4.7, 500-500-500 64x64 fp16 10 % 4.86 / 4.87, 7.6 / 4.95, 6.5 / 5.0.
#include <algorithm>
#include <cstring>

#include "pivot_fc_kernels.h"

namespace pivot {

namespace {

constexpr int kGroupNW = 16;                    // wavefronts of the workgroup
constexpr int kGroupNT = kGroupNW * 64;
constexpr size_t kGroupLds = 60 * 1024;
enum { kSlotEnd = 1, kSlotRelu = 2, kSlotLast = 4 };    // flags of a slot; from bit 8 on: lanes between the tiles of a wave-load

// q_layer_ends: bit k set = a layer ends with slot k.  q_k0 = columns of x | padded << 16; q_act_vecs: 16-byte pieces of LDS in
// front of the natural-order x (the layers' inputs in block order, one behind the other, the first one the chain's).
// The arguments that the first loads need come first (preloaded).
template <typename WT, int BW, int NS>
__global__ void __launch_bounds__(kGroupNT) mlp_group_kernel(const int4* __restrict__ p_meta, const char* __restrict__ p_vals,
                                                             const WT* __restrict__ p_x, const int32_t* __restrict__ p_pcol,
                                                             long long q_ldx, int q_k0, int q_act_vecs, uint32_t q_layer_ends,
                                                             float* __restrict__ p_y, long long q_ldy) {
    using V = typename Elem<WT>::vec;
    constexpr int VEC = Elem<WT>::VEC, LPR = BW / VEC;
    extern __shared__ __align__(16) char smem[];
    WT* act = reinterpret_cast<WT*>(smem);
    WT* xn = act + (size_t)q_act_vecs * VEC;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = q_k0 & 0xFFFF, kpad = (int)((uint32_t)q_k0 >> 16);
    p_x += (long long)blockIdx.x * q_ldx;
    p_y += (long long)blockIdx.x * q_ldy;

    // x first: the first thing that is waited for
    const WT x0 = p_x[tid < K ? tid : K - 1];
    const int src0 = p_pcol[tid < kpad ? tid : kpad - 1];
    // Eight slots are in flight (their registers); a later one is asked for when the one eight before it is consumed.
    constexpr int NF = NS < 8 ? NS : 8;
    int4 m[NF];
    V w[NF];
    auto ask = [&](int k) {
        const int at = (k * kGroupNW + wave) * 64 + lane;
        m[k % NF] = p_meta[at];
        w[k % NF] = load16<V>(p_vals + (size_t)at * 16);
    };
    #pragma unroll
    for (int k = 0; k < NF; ++k) ask(k);
    __builtin_amdgcn_sched_barrier(0);                  // every load above is issued before anything below waits
    // padding columns of the later layers' inputs are never stored to
    for (int i = kpad / VEC + tid; i < q_act_vecs; i += kGroupNT) reinterpret_cast<V*>(act)[i] = V(0);
    if (tid < K) xn[tid] = x0;
    for (int i = tid + kGroupNT; i < K; i += kGroupNT) xn[i] = p_x[i];
    lds_barrier();
    if (tid < kpad) act[tid] = src0 >= 0 ? xn[src0] : WT(0);
    for (int i = tid + kGroupNT; i < kpad; i += kGroupNT) {
        const int s = p_pcol[i];
        act[i] = s >= 0 ? xn[s] : WT(0);
    }
    lds_barrier();

    float acc = 0.f;
    #pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int4 mk = m[k % NF];
        const V xv = *reinterpret_cast<const V*>(act + (mk.x > 0 ? mk.x : 0));
        acc = dot_vec(w[k % NF], mk.x >= 0 ? xv : V(0), acc);
        if (k + NF < NS) {
            ask(k + NF);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int f = __builtin_amdgcn_readfirstlane(mk.w);
        if (f & kSlotEnd) {
            float v = group_sum<LPR>(acc);
            for (int o = f >> 8; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
            v = apply_act(v + __int_as_float(mk.z), (f & kSlotRelu) ? 1 : 0);
            if (mk.y >= 0) {
                if (f & kSlotLast) p_y[mk.y] = v;
                else act[mk.y] = WT(v);
            }
            acc = 0.f;
        }
        if ((q_layer_ends >> k) & 1u) lds_barrier();
    }
}

using GroupLaunch = void (*)(const ChainGroup&, const void*, int64_t, const int32_t*, float*, int64_t, int, hipStream_t);
template <typename WT, int BW, int NS>
void launch_group_t(const ChainGroup& g, const void* x, int64_t ldx, const int32_t* pcol_pad, float* y, int64_t ldy, int batch, hipStream_t st) {
    hipLaunchKernelGGL((mlp_group_kernel<WT, BW, NS>), dim3(batch), dim3(kGroupNT), g.smem, st,
                       reinterpret_cast<const int4*>(g.dev_meta), reinterpret_cast<const char*>(g.dev_vals),
                       reinterpret_cast<const WT*>(x), pcol_pad, (long long)ldx, (int)((uint32_t)g.K | ((uint32_t)g.K_pad << 16)),
                       g.act_vecs, g.layer_ends, y, (long long)ldy);
}
template <typename WT, int BW>
GroupLaunch group_launch_of(int ns) {
    switch (ns) {
        case 3: return launch_group_t<WT, BW, 3>;
        case 4: return launch_group_t<WT, BW, 4>;
        case 6: return launch_group_t<WT, BW, 6>;
        case 8: return launch_group_t<WT, BW, 8>;
        case 12: return launch_group_t<WT, BW, 12>;
        default: return launch_group_t<WT, BW, 16>;
    }
}

}  // namespace

// Lays a chain out for one workgroup if it is one that the form takes.  `dst[l]`: block-space row of layer l -> position in the
// next layer's block-order input, -1 = not stored; keep: the last layer's outputs stay in block order.
bool chain_group_build(const std::vector<const HostPlan*>& layers, const std::vector<std::vector<int32_t>>& dst, bool keep, ChainGroup& g) {
    const int Lc = (int)layers.size();
    const HostPlan& f = *layers[0];
    const int wdtype = f.d.wdtype, bw = f.d.bw, es = elem_size(wdtype), vec = 16 / es;
    if (bw != 16 && bw != 32 && bw != 64) return false;
    // A longer x is copied in turns of 1024 elements, a trip each; every boundary saves about 1.8 us (us, many workgroups /
    // one, two fp16 layers: 2000-200-200 4.6 / 4.3, 4000-200-200 4.3 / 4.8).
    if (f.K_pad > 2048 * (Lc - 1)) return false;
    const int lpr = bw / vec, rpw = 64 / lpr;
    size_t act = 0;
    std::vector<int> act_off;
    for (const HostPlan* hp : layers) {
        if (hp->d.wdtype != wdtype || hp->d.bw != bw || hp->d.layout != PIVOT_BRC) return false;
        act_off.push_back((int)act);
        act += hp->K_pad;
        if ((act + f.d.K) * es > kGroupLds) return false;
    }
    // Every four slots beyond 8 cost 0.6-0.9 us (a compute unit's 64 bytes a clock), every boundary of the forms it replaces
    // 1.2-1.8 at batch 1 and 2.2 beyond.  Us, batch 1 / 8, the other forms and this one: two layers, 12 slots, 640x3 16x16 fp16
    // 10 % 5.1, 5.2 / 5.4, 5.3, 800x3 5 % 5.2, 6.1 / 5.4, 6.3, 512x3 32x32 fp32 10 % 5.1, 6.0 / 5.4, 6.1; three layers, 9-12
    // slots, 512x4 16x16 fp32 6 % 6.4, 5.0 / 7.7, 5.2, 784-128-64-10 32x32 fp16 40 % 5.8, 5.7 / 7.9, 5.8; 13-16 slots,
    // 600-400-200-100 64x64 fp32 10 % 5.7, 6.05 / 8.0, 6.2; four layers, 300x5 32x32 fp16 15 % 8.0, 5.9 / 11.0, 6.0.
    const int most = Lc == 2 ? 8 : kChainGroupSlots;
    // units of a layer: the rows of one wave-load of a block row (all of it where the tile has fewer), to the least loaded
    // wavefront, longest first
    struct Unit { int br, piece, loads, wave, pos; };
    std::vector<std::vector<Unit>> units(Lc);
    std::vector<int> first(Lc + 1, 0);
    for (int l = 0; l < Lc; ++l) {
        const HostPlan& hp = *layers[l];
        const int tpl = hp.d.bh >= rpw ? 1 : rpw / hp.d.bh, pieces = hp.d.bh >= rpw ? hp.d.bh / rpw : 1;
        if ((long long)hp.nbr * pieces > (long long)kGroupNW * kChainGroupSlots) return false;
        for (int br = 0; br < hp.nbr; ++br) {
            const int loads = std::max(1, (hp.row_ptr[br + 1] - hp.row_ptr[br] + tpl - 1) / tpl);
            for (int p = 0; p < pieces; ++p) units[l].push_back({br, p, loads, 0, 0});
        }
        std::stable_sort(units[l].begin(), units[l].end(), [](const Unit& a, const Unit& b) { return a.loads > b.loads; });
        int load[kGroupNW] = {};
        for (Unit& u : units[l]) {
            u.wave = (int)(std::min_element(load, load + kGroupNW) - load);
            u.pos = load[u.wave];
            load[u.wave] += u.loads;
        }
        first[l + 1] = first[l] + *std::max_element(load, load + kGroupNW);
        if (first[l + 1] > most) return false;
    }
    const int used = first[Lc];
    g.nslots = used <= 3 ? 3 : (used <= 4 ? 4 : (used <= 6 ? 6 : (used <= 8 ? 8 : (used <= 12 ? 12 : 16))));
    g.batch_from = Lc == 3 && used > 12 ? 2 : 1;
    g.layer_ends = 0;
    for (int l = 0; l + 1 < Lc; ++l) g.layer_ends |= 1u << (first[l + 1] - 1);      // (nothing reads the last layer's outputs)
    g.meta.assign((size_t)g.nslots * kGroupNT * 4, 0);
    g.vals.assign((size_t)g.nslots * kGroupNT * 16, 0);
    for (size_t i = 0; i < (size_t)g.nslots * kGroupNT; ++i) { g.meta[4 * i] = -1; g.meta[4 * i + 1] = -1; }
    for (int l = 0; l < Lc; ++l) {
        const HostPlan& hp = *layers[l];
        const bool last = l + 1 == Lc;
        const int bh = hp.d.bh, tpl = bh >= rpw ? 1 : rpw / bh;
        for (const Unit& u : units[l]) {
            const int t0 = hp.row_ptr[u.br], t1 = hp.row_ptr[u.br + 1];
            for (int i = 0; i < u.loads; ++i) {
                const size_t slot = ((size_t)(first[l] + u.pos + i) * kGroupNW + u.wave) * 64;
                const bool end = i + 1 == u.loads;
                const int flags = end ? kSlotEnd | (hp.d.act == PIVOT_ACT_RELU ? kSlotRelu : 0) | (last ? kSlotLast : 0) |
                                        (tpl > 1 ? bh * lpr : 64) << 8 : 0;
                for (int lane = 0; lane < 64; ++lane) {
                    int32_t* m = &g.meta[(slot + lane) * 4];
                    const int s = lane / lpr, cg = lane % lpr;
                    const int row = tpl > 1 ? s % bh : u.piece * rpw + s;
                    const int t = t0 + i * tpl + (tpl > 1 ? s / bh : 0);
                    m[3] = flags;
                    if (t < t1) {
                        m[0] = act_off[l] + hp.col_idx[t] * bw + cg * vec;
                        memcpy(&g.vals[(slot + lane) * 16], &hp.vals[(((size_t)t * bh + row) * bw + (size_t)cg * vec) * es], 16);
                    }
                    if (end && cg == 0 && s < (tpl > 1 ? bh : rpw)) {
                        const int R = u.br * bh + row;
                        const int to = !last ? dst[l][R] : (keep ? (R < hp.d.M ? R : -1) : hp.prow_pad[R]);
                        m[1] = to < 0 ? -1 : (last ? to : act_off[l + 1] + to);
                        memcpy(&m[2], &hp.bias_p[R], 4);
                    }
                }
            }
        }
    }
    g.K = f.d.K; g.K_pad = f.K_pad; g.act_vecs = (int)(act / vec);
    g.smem = act * es + align_up((size_t)f.d.K * es, 16);
    g.wdtype = wdtype; g.bw = bw;
    return true;
}

int launch_chain_group(const ChainGroup& g, const void* x, int64_t ldx, const int32_t* pcol_pad, float* y, int64_t ldy, int batch, void* stream) {
    GroupLaunch run = nullptr;
    if (g.wdtype == PIVOT_F32) run = g.bw == 16 ? group_launch_of<float, 16>(g.nslots) : (g.bw == 32 ? group_launch_of<float, 32>(g.nslots) : group_launch_of<float, 64>(g.nslots));
    else run = g.bw == 16 ? group_launch_of<_Float16, 16>(g.nslots) : (g.bw == 32 ? group_launch_of<_Float16, 32>(g.nslots) : group_launch_of<_Float16, 64>(g.nslots));
    run(g, x, ldx, pcol_pad, y, ldy, batch, reinterpret_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

}  // namespace pivot
