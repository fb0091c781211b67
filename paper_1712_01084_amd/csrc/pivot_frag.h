// Batched layer kernel on the matrix cores, both weight types and every tile
// shape: x comes in fragment order, the weights stream once per launch row of
// up to 64 batch rows.
//
// Fragment order of a [batch][K_pad] input in block order: groups of 16 bytes
// (VEC = 8 fp16 or 4 fp32 consecutive columns of one batch row), group-major,
// the batch rows of a group side by side: element (b, c) at
// ((c / VEC) * batch + b) * VEC + c % VEC.  A lane's B fragment (VEC
// consecutive k of one batch row) is then one 16-byte load, and the sixteen
// lanes that hold the same k of sixteen batch rows read contiguous memory.
// The order is written by gather_frag_kernel (natural-order x), by the
// epilogue of the layer before (chains) or by the recurrent cell.
//
// A step covers SK = 4 * VEC columns: v_mfma_f32_16x16x32_f16, or four
// v_mfma_f32_16x16x4_f32 whose k indices are permuted alike in A and B (lane l
// supplies columns VEC*(l/16).. of row l%16, element e of its fragment goes
// to the e-th instruction).  Wider tiles take several steps; of narrower ones
// several consecutive tiles of the block row make a step.  Tiles of 8 rows are
// stacked in pairs: rows 0-7 of A come from one set of tiles, rows 8-15 from
// the next, each set meets its own B fragments in an accumulator of its own,
// and the halves that belong together are added at the end; the loads stay
// whole, half the (idle) matrix work is thrown away.
//
// What bounds it: the memory pipeline of a compute unit, which takes the weights once and, per row slice, the x
// of the block row (batch / rows of the slice times the bytes of the weights); fp32 from batch 32 on also the matrix
// cores (64 batch rows of 8192x8192 at 25 % kept: 15 us of MFMA at the rate this card reaches).  8192x8192, 25 %
// kept, 32x32 tiles, the whole call with the copy of x: fp32 (67 MB) batch 16 18.5 us (the vector kernel 55.5), fp16
// (34 MB) batch 16 12.2 us (LDS-fed 15.7) and batch 64 17.6 us.
#pragma once

#include "pivot_fc_kernels.h"

namespace pivot {

// Registers that hold the block columns of a wavefront's tiles: an item of a device plan has at most 48 KB / (bw * 4
// rows * element size) tiles (max_chunk_tiles), 768 of the narrowest, of which four wavefronts hold 248 each.
constexpr int frag_cols(int bw, int vec) { return bw == 8 && vec == 8 ? 4 : 2; }

template <typename WT> struct FragMfma;
template <> struct FragMfma<_Float16> {
    static constexpr int NE = 1;                        // instructions per fragment
    __device__ static __forceinline__ f32x4 run(const f16x8& a, const f16x8& b, const f32x4& c, int) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct FragMfma<float> {
    static constexpr int NE = 4;
    __device__ static __forceinline__ f32x4 run(const f32x4& a, const f32x4& b, const f32x4& c, int e) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    }
};

// BH: rows of this launch's slice (8, 16 or 32), NBT: blocks of 16 batch rows per launch row, NW: wavefronts (2 or 4).
template <typename WT, int BH, int BW, int NBT, int NW>
__global__ void __launch_bounds__(NW * 64) fc_frag_kernel(PIVOT_GEMV_PARAMS, FcTail a) {
    using V = typename Elem<WT>::vec;
    using MF = FragMfma<WT>;
    constexpr int VEC = Elem<WT>::VEC;
    constexpr int NT = NW * 64;
    constexpr int SK  = 4 * VEC;                        // columns per step
    constexpr int TPS = BW < SK ? SK / BW : 1;          // tiles per step (narrow tiles)
    constexpr int KS  = BW < SK ? 1 : BW / SK;          // steps per tile (wide tiles)
    constexpr int LPT = BW < SK ? BW / VEC : 4;         // lane groups of 16 that share a tile
    constexpr int RS  = BH < 16 ? 2 : 1;                // sets of tiles stacked in the 16 rows of A
    constexpr int RB  = BH < 16 ? 1 : BH / 16;          // row blocks
    constexpr int RT  = BH < 16 ? BH : 16;              // rows of A that come from one tile
    constexpr int TPG = TPS * RS;                       // tiles per group (what a wavefront consumes together)
    // Steps in flight: 8 KB of weights per wavefront or more (4 KB for stacked tiles and 64 batch rows), in at most 40
    // fragments (160 registers)
    constexpr int U   = (RB + RS * NBT) * 8 <= (RB < 2 ? 40 : 32) ? 8 : 4;
    constexpr int NC  = frag_cols(BW, VEC);             // registers of block columns per lane
    constexpr int NB  = 16 * NBT, N = BH * NB;
    static_assert(U % KS == 0, "steps in flight are whole tiles");

    extern __shared__ __align__(16) char smem[];
    __shared__ int s_flag;
    float* red = reinterpret_cast<float*>(smem);        // NW * N floats

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = blockIdx.y * NB, slice = blockIdx.z;
    const int q_uniform_parts = q_ct_parts >> 16, q_uniform_ct = q_uniform_parts > 0 ? (q_ct_parts & 0xFFFF) : 0;
    const int q_bh_full = q_misc & 0x7F, q_batch = (q_misc >> 7) & 0x7F;
    const Chunk ck = load_chunk(q_uniform_ct, q_uniform_parts, p_chunks);
    const int br = ck.br, tile_begin = ck.tile_begin, ntiles = ck.ntiles;
    const int row0 = br * q_bh_full + slice * BH;
    const int tile_elems = q_bh_full * BW;

    const int li = lane & 15, lg = lane >> 4;           // A row / B column, k group
    const int kc = TPS > 1 ? lg % LPT : lg;             // 16-byte piece of the tile row
    const int ts = TPS > 1 ? lg / LPT : 0;              // tile of the step
    const int ta = (RS == 2 ? (li >> 3) * TPS : 0) + ts; // tile of the group this lane's A rows come from

    const int tmax = ntiles > 0 ? ntiles - 1 : 0;
    const int ngroups = (ntiles + TPG - 1) / TPG;
    const int nmine = ngroups > wave ? (ngroups - wave + NW - 1) / NW : 0;   // groups wave, wave + NW, ...
    const int imax = nmine > 0 ? nmine - 1 : 0;
    const int nsteps = nmine * KS;

    // Block columns of the wavefront's tiles, one per lane, fetched together (the launcher sees to it that NC
    // registers hold them): the address of a B fragment then depends on no further load.
    int cv[NC];
    #pragma unroll
    for (int h = 0; h < NC; ++h) {
        const int q = h * 64 + lane;
        const int t = (wave + (q / TPG) * NW) * TPG + q % TPG;
        cv[h] = p_idx[tile_begin + (t < tmax ? t : tmax)];
    }
    // the lane's B columns; past the last batch row it repeats that row (its sums are never stored)
    uint32_t xoff[NBT];
    #pragma unroll
    for (int nb = 0; nb < NBT; ++nb) {
        const int b = b0 + nb * 16 + li;
        xoff[nb] = (uint32_t)(kc * q_batch + (b < q_batch ? b : q_batch - 1)) * 16u;
    }
    const uint32_t tile_x = (uint32_t)(BW / VEC) * (uint32_t)q_batch * 16u;   // bytes of x per block column
    const uint32_t step_x = 4u * (uint32_t)q_batch * 16u;                     // ... per step inside a tile
    const WT* vbase = reinterpret_cast<const WT*>(p_vals) + (size_t)tile_begin * tile_elems
                      + (size_t)slice * BH * BW + (li % RT) * BW + kc * VEC;

    V w[U][RB], xv[U][RS][NBT];
    // loads are unconditional: groups past the wavefront's last repeat it
    auto fill_w = [&](int u, int s) {
        const int i = s / KS < imax ? s / KS : imax;
        const int tile = (wave + i * NW) * TPG + ta;
        const WT* p = vbase + (size_t)(tile < tmax ? tile : tmax) * tile_elems + (u % KS) * SK;
        #pragma unroll
        for (int rb = 0; rb < RB; ++rb) w[u][rb] = load16<V>(p + rb * 16 * BW);
    };
    auto fill_x = [&](int u, int s) {
        const int i = s / KS < imax ? s / KS : imax;
        #pragma unroll
        for (int rs = 0; rs < RS; ++rs) {
            const int q = i * TPG + rs * TPS + ts;
            int c;
            if constexpr (TPS == 1) {
                const int qs = __builtin_amdgcn_readfirstlane(q);
                c = __builtin_amdgcn_readlane(qs < 64 ? cv[0] : cv[1], qs & 63);
            } else {
                c = __builtin_amdgcn_ds_bpermute((q & 63) * 4, cv[0]);
                #pragma unroll
                for (int h = 1; h < NC; ++h) {
                    const int ch = __builtin_amdgcn_ds_bpermute((q & 63) * 4, cv[h]);
                    c = q < h * 64 ? c : ch;
                }
            }
            const char* xp = reinterpret_cast<const char*>(p_x) + ((uint32_t)c * tile_x + (u % KS) * step_x);
            #pragma unroll
            for (int nb = 0; nb < NBT; ++nb) xv[u][rs][nb] = load16<V>(xp + xoff[nb]);
        }
    };
    // the first weights depend on nothing but the descriptor; x, whose addresses need the block columns, behind them
    #pragma unroll
    for (int u = 0; u < U; ++u) fill_w(u, u);
    __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
    for (int u = 0; u < U; ++u) fill_x(u, u);
    RowPre<BH, N, NT> rp;
    rp.load(p_bias, p_scatter, row0, tid);
    __builtin_amdgcn_sched_barrier(0);                  // every load above is issued before anything below waits

    f32x4 acc[RB][RS][NBT];
    #pragma unroll
    for (int rb = 0; rb < RB; ++rb)
        #pragma unroll
        for (int rs = 0; rs < RS; ++rs)
            #pragma unroll
            for (int nb = 0; nb < NBT; ++nb) acc[rb][rs][nb] = f32x4(0);
    // Tiles that the last, incomplete group does not have: neither the weights nor the x loaded in their place may
    // count (zero weights alone are not enough: 0 times an infinity is a NaN).
    auto clear_missing = [&](int u, int s) {
        if constexpr (TPG > 1) {
            const int t0 = (wave + (s / KS) * NW) * TPG;
            #pragma unroll
            for (int rb = 0; rb < RB; ++rb) w[u][rb] = t0 + ta < ntiles ? w[u][rb] : V(0);
            #pragma unroll
            for (int rs = 0; rs < RS; ++rs)
                #pragma unroll
                for (int nb = 0; nb < NBT; ++nb) xv[u][rs][nb] = t0 + rs * TPS + ts < ntiles ? xv[u][rs][nb] : V(0);
        }
    };
    auto consume = [&](int u) {
        #pragma unroll
        for (int e = 0; e < MF::NE; ++e)
            #pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                #pragma unroll
                for (int rs = 0; rs < RS; ++rs)
                    #pragma unroll
                    for (int nb = 0; nb < NBT; ++nb)
                        acc[rb][rs][nb] = MF::run(w[u][rb], xv[u][rs][nb], acc[rb][rs][nb], e);
    };
    int s0 = 0;
    for (; s0 + U < nsteps; s0 += U) {
        #pragma unroll
        for (int u = 0; u < U; ++u) {
            consume(u);                                 // (never a group the wavefront ends with)
            fill_w(u, s0 + u + U);
            fill_x(u, s0 + u + U);
            __builtin_amdgcn_sched_barrier(0);          // a slot is refilled as soon as it is consumed
        }
    }
    // The masks only in the wavefront that has the incomplete group (in all of them: up to 1 us a call), chosen per
    // step for stacked tiles and once for the others (the other way round 0.2-0.4 us slower).
    const bool incomplete = TPG > 1 && (wave + imax * NW) * TPG + TPG > ntiles;
    if (RS == 2 || !incomplete) {
        #pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < nsteps) {
                if (RS == 2 && (wave + ((s0 + u) / KS) * NW) * TPG + TPG > ntiles) clear_missing(u, s0 + u);
                consume(u);
            }
    } else {
        #pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < nsteps) {
                clear_missing(u, s0 + u);
                consume(u);
            }
    }

    // Every wavefront's sums go to LDS, the epilogue adds them.  Accumulator element v of lane l is
    // C[row 4(l/16)+v][batch column l%16]; of stacked tiles rows 8-15 of the second set (lanes 32-63) belong to
    // rows 0-7.
    if constexpr (RS == 2) {
        #pragma unroll
        for (int nb = 0; nb < NBT; ++nb)
            #pragma unroll
            for (int v = 0; v < 4; ++v) acc[0][0][nb][v] += __shfl_xor(acc[0][1][nb][v], 32, 64);
    }
    if (RS == 1 || lg < 2) {
        #pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            #pragma unroll
            for (int nb = 0; nb < NBT; ++nb)
                *reinterpret_cast<f32x4*>(red + wave * N + (nb * 16 + li) * BH + rb * 16 + lg * 4) = acc[rb][0][nb];
    }
    lds_barrier();
    finish_rows<BH, NB, NT, kEither>(a, red, NW, br, ck.slot, ck.first, ck.nparts, rp, b0, tid, &s_flag);
}

template <typename WT, int BH, int BW, int NBT>
static int launch_frag_t(const FcArgs& a, int nw, dim3 grid, hipStream_t st) {
    const size_t smem = (size_t)nw * BH * 16 * NBT * 4;
    if (nw == 2) hipLaunchKernelGGL((fc_frag_kernel<WT, BH, BW, NBT, 2>), grid, dim3(128), smem, st, PIVOT_GEMV_ARGS(a), fc_tail(a));
    else         hipLaunchKernelGGL((fc_frag_kernel<WT, BH, BW, NBT, 4>), grid, dim3(256), smem, st, PIVOT_GEMV_ARGS(a), fc_tail(a));
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

// the instantiations of one slice height (one translation unit each)
template <typename WT, int BH>
static int launch_frag_w(const FcArgs& a, int bw, int nbt, int nw, dim3 grid, hipStream_t st) {
#define X(BW_)                                                                          \
    if (bw == BW_) {                                                                    \
        if (nbt == 1) return launch_frag_t<WT, BH, BW_, 1>(a, nw, grid, st);            \
        if (nbt == 2) return launch_frag_t<WT, BH, BW_, 2>(a, nw, grid, st);            \
        if (nbt == 4) return launch_frag_t<WT, BH, BW_, 4>(a, nw, grid, st);            \
    }
    X(8) X(16) X(32) X(64)
#undef X
    set_error("no batched matrix-core kernel for %dx%d row slices, %d batch blocks", BH, bw, nbt);
    return PIVOT_E_UNSUPPORTED;
}

}  // namespace pivot
