// The recurrent loop in one launch with ONE exchange per step: a workgroup owns
// whole units, that is all four gate rows of each, so the gate sums never leave
// it and h is the only thing that crosses workgroups.
//
// The gate rows of a unit lie in four unrelated block rows, so the rows of a
// workgroup share no tiles.  They are laid out densely instead: once per launch
// a workgroup scatters its 16*RB rows (kept tiles, zeros elsewhere) over the
// NATURAL columns [h | x] and holds them as MFMA A fragments, the h columns in
// registers, the x columns in LDS.  The zeros cost matrix work that is idle
// anyway (2048 units, 1024 inputs, 12.5 % kept: 32 rows x 3072 columns per
// workgroup, 0.3 us of MFMA a step) and buy three things: no index is followed
// inside the loop, every workgroup has the same work whatever the row lengths
// are, and x_t is read straight from the caller's array.
//
// A team of workgroups runs up to 16*NBT batch rows; teams are independent.
// Exchange: per step a buffer [group of VEC units][batch row][VEC] (VEC units are
// 16 bytes), pre-filled with a bit pattern no finite value has, the units of a
// workgroup contiguous: it writes whole lines, and a B fragment (VEC consecutive
// h of one batch row) is one 16-byte load of every lane.  A wavefront takes every
// fourth k-step, re-reads its fragments until no element is the pattern,
// multiplies, hands its sums to the cell threads through LDS (fixed order), and
// works on the x part of the next step while h is on its way.
//
// Zeros outside the kept tiles are only neutral for finite inputs.  A wavefront
// that meets an infinity or a NaN says so, and the workgroup computes that step
// from the tile lists instead (slow_step), where a column meets the rows of its
// kept tiles and no others.
//
// What bounds it: latency.  A step of 2048 units at batch 8 is 3.1 us: store to
// arrival 0.9, fragments 0.5, matrix work and hand-over 0.9, cell 0.6 (one wavefront
// per SIMD, dependent instructions).  Us for a sequence, the form that exchanges
// gate sums or a launch per step -> this one: 2048 units, 1024 inputs, fp16, 256
// steps, batch 8 1727 -> 790; 1024 units, 512 inputs, fp16, 32 steps, batch 32 237 ->
// 122; 1000 units, 500 inputs, fp32, 20 steps, batch 8 130 -> 111.  A workgroup uses
// at most half a compute unit and every wait is bounded like those of the kernel
// that exchanges gate sums.
#include <algorithm>
#include <atomic>
#include <cstdio>

#include "pivot_fc_kernels.h"
#include "pivot_frag.h"

namespace pivot {

namespace {

constexpr int kUW = 4;                      // wavefronts per workgroup
constexpr int kUT = kUW * 64;
static_assert(kUW == 4, "a wavefront sets up four rows of a block");
constexpr int kUX = 8;                      // k-steps of x per wavefront
constexpr size_t kULds = 80 * 1024 - 512;   // half a compute unit, less the static part
constexpr uint32_t kUSpinLimit = 1u << 18;

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct UnitArgs {
    const void*    vals;        // BRC tile values
    const int32_t* xidx;        // [T*bw] natural column of every kept tile's columns, -1 = padding
    const int32_t* row_ptr;     // [nbr+1]
    const int32_t* invprow;     // [4H]
    const float*   bias_p;
    const void*    xs;          // x_t: element (t, b, i) at t*xs_step + b*xs_row + i
    void*          hx;          // exchange buffers: step t at t*step_bytes, team k's part at k*team_bytes in it
    uint32_t*      ctl;         // [256] status
    float*         h;
    float*         c;
    float*         z_dbg;
    long long      xs_step;
    unsigned long long step_bytes, team_bytes;
    int xs_row, xgroups;        // xgroups: 16-byte groups of a row of xs
    int H, I, batch, steps, bt, wgs;    // bt: batch rows of a team; wgs: workgroups of a team
    int bh, bw, hsteps, xsteps, slots;
};

// v + (o of the lane that the data-parallel control CTRL names)
template <int CTRL>
__device__ __forceinline__ float dpp_add_from(float v, float o) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, o), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float usigm(float v) { return 1.0f / (1.0f + __expf(-v)); }

__device__ __forceinline__ uint32_t uld32(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void ust32(uint32_t* p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ bool unit_keep_waiting(uint32_t* ctl, uint32_t& spins) {
    __builtin_amdgcn_s_sleep(1);
    if ((++spins & 63u) != 0u) return true;
    if (uld32(ctl + 256) != 0u) return false;
    if (spins >= kUSpinLimit) { ust32(ctl + 256, 1u); return false; }
    return true;
}

// What crosses workgroups is a finite value, the mark (all bits set: not there yet), a NaN, which is always handed
// over as the bits just below the mark, or an infinite h_0.  So one unsigned maximum over the words read tells the
// mark (all ones) and NaNs (an exponent of all ones behind a sign bit); only in step 0 infinities are looked for.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
template <typename WT> struct Pattern;
template <> struct Pattern<_Float16> {
    using Top = u16x2;
    __device__ static __forceinline__ void top(Top& t, uint32_t w) { t = __builtin_elementwise_max(t, __builtin_bit_cast(u16x2, w)); }
    __device__ static __forceinline__ bool mark(const Top& t) { return t.x == 0xFFFFu || t.y == 0xFFFFu; }
    __device__ static __forceinline__ bool odd(const Top& t) { return t.x >= 0xFC00u || t.y >= 0xFC00u; }
    static constexpr uint32_t kMagnitude = 0x7FFF7FFFu;
    __device__ static __forceinline__ bool odd_magnitude(const Top& t) { return t.x >= 0x7C00u || t.y >= 0x7C00u; }
    __device__ static __forceinline__ uint32_t bits(float v) { return v == v ? (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)v) : 0xFFFEu; }
};
template <> struct Pattern<float> {
    using Top = uint32_t;
    __device__ static __forceinline__ void top(Top& t, uint32_t w) { t = t > w ? t : w; }
    __device__ static __forceinline__ bool mark(const Top& t) { return t == 0xFFFFFFFFu; }
    __device__ static __forceinline__ bool odd(const Top& t) { return t >= 0xFF800000u; }
    static constexpr uint32_t kMagnitude = 0x7FFFFFFFu;
    __device__ static __forceinline__ bool odd_magnitude(const Top& t) { return t >= 0x7F800000u; }
    __device__ static __forceinline__ uint32_t bits(float v) { return v == v ? __float_as_uint(v) : 0xFFFFFFFEu; }
};
template <typename WT, uint32_t MASK = 0xFFFFFFFFu>
__device__ __forceinline__ void take_top(typename Pattern<WT>::Top& t, const u32x4& v) {
    #pragma unroll
    for (int k = 0; k < 4; ++k) Pattern<WT>::top(t, v[k] & MASK);
}

// A step with infinities or NaNs among its inputs: the gate sums of the workgroup's rows from the tile lists, a
// wavefront per row, into the first wavefront's sums; the other wavefronts' sums become zero.
template <typename WT, int RB>
__device__ void slow_step(const UnitArgs& a, const WT* hbuf, const WT* xt, int unit0, int nb, float* red) {
    constexpr int U = 4 * RB, SHIFT = sizeof(WT) == 2 ? 3 : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < kUW * a.bt * 16 * RB; i += kUT) red[i] = 0.f;
    __syncthreads();
    for (int row = wave; row < 16 * RB; row += kUW) {
        const int uu = row >> 2, j = unit0 + uu;
        if (j >= a.H) continue;
        const int R = a.invprow[(row & 3) * a.H + j], br = R / a.bh, rr = R - br * a.bh;
        const int e0 = a.row_ptr[br] * a.bw, e1 = a.row_ptr[br + 1] * a.bw;
        for (int b = 0; b < nb; ++b) {
            float sum = 0.f;
            for (int e = e0 + lane; e < e1; e += 64) {
                const int n = a.xidx[e], t = e / a.bw;
                if (n < 0) continue;
                const float w = (float)reinterpret_cast<const WT*>(a.vals)[((size_t)t * a.bh + rr) * a.bw + (e - t * a.bw)];
                float in;
                if (n >= a.H) in = (float)xt[(long long)b * a.xs_row + (n - a.H)];
                else {
                    const size_t o = frag_index(b, n, a.bt, SHIFT);
                    if constexpr (sizeof(WT) == 2) {
                        const uint32_t word = uld32(reinterpret_cast<const uint32_t*>(hbuf) + (o >> 1));
                        in = (float)__builtin_bit_cast(_Float16, (unsigned short)((o & 1) ? word >> 16 : word & 0xFFFFu));
                    } else in = __uint_as_float(uld32(reinterpret_cast<const uint32_t*>(hbuf) + o));
                }
                sum = fmaf(w, in, sum);
            }
            sum = group_sum<64>(sum);
            if (lane == 0) red[((size_t)b * U + (uu ^ (b & (U - 1)))) * 4 + (row & 3)] = sum;
        }
    }
    __syncthreads();
}

// RB: blocks of 16 gate rows (4 units each), HS: k-steps of h per wavefront, NBT: blocks of 16 batch rows.
// PAIR (teams of up to 8 rows): the lanes of batch columns 8-15 hold the fragments of the wavefront's next k-step
// instead of copies; each k-step has accumulators of its own, of which one half is meant, and half as many loads,
// registers and checks are needed for the same matrix work.
template <typename WT, int RB, int HS, int NBT, bool PAIR>
__global__ void __launch_bounds__(kUT, 2) lstm_units_kernel(UnitArgs a) {
    using V = typename Elem<WT>::vec;
    using MF = FragMfma<WT>;
    using PT = Pattern<WT>;
    constexpr int VEC = Elem<WT>::VEC, SK = 4 * VEC, U = 4 * RB;
    constexpr int SHIFT = sizeof(WT) == 2 ? 3 : 2;
    constexpr int PS = PAIR ? 2 : 1;                    // k-steps per fragment
    static_assert(!PAIR || NBT == 1, "a pair fills the 16 batch columns");
    extern __shared__ __align__(16) char smem[];
    __shared__ __align__(16) float s_bias[U * 4];
    __shared__ int s_flag[2][2];                        // [step parity]: {a wait gave up, an input is not finite}, = step + 1
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = blockIdx.x / a.wgs, unit0 = (blockIdx.x - team * a.wgs) * U;
    const int b0 = team * a.bt, nb = a.batch - b0 < a.bt ? a.batch - b0 : a.bt;
    const int li = lane & 15, lg = lane >> 4;
    V* xw = reinterpret_cast<V*>(smem);                 // [xsteps][RB][64] A fragments of the x columns
    float* red0 = reinterpret_cast<float*>(smem + (size_t)a.xsteps * RB * 1024);   // [slots][wavefront][bt][U, swizzled][4 gates]
    const int red_slot = kUW * a.bt * U * 4;

    // ---- weights: rows of the plan's tiles -> dense A fragments over natural columns --------------------------
    if (tid < 4) s_flag[tid >> 1][tid & 1] = 0;
    // lane l of every wavefront knows gate row l: its tiles and its row inside them
    int my_e0 = 0, my_e1 = 0, my_rr = 0;
    if (lane < 16 * RB && unit0 + (lane >> 2) < a.H) {
        const int R = a.invprow[(lane & 3) * a.H + unit0 + (lane >> 2)];
        const int br = R / a.bh;
        my_rr = R - br * a.bh;
        my_e0 = a.row_ptr[br]; my_e1 = a.row_ptr[br + 1];
    }
    // Scatters the columns that `place` accepts of the wavefront's four rows of a 16-row block.  The rows' tiles make
    // one list, of which a lane takes VEC consecutive columns of a tile at a time and four such pieces together, so
    // that a pass over typical rows costs one trip to memory and a long row shares its trips (2048 units, 1024 inputs,
    // rows by a Zipf law: 32 steps at batch 1 184.6 us with a row at a time, 155.4 with four rows side by side; 4 steps
    // at batch 8 63.8 us with four rows side by side, 55.2 with one list).
    const int vpt = a.bw / VEC;                         // vectors per tile row
    auto scatter_rows = [&](int block, auto&& place) {
        int t0[4], rr[4], end[4];
        #pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = block * 16 + wave + k * kUW;
            t0[k] = __builtin_amdgcn_readlane(my_e0, row);
            rr[k] = __builtin_amdgcn_readlane(my_rr, row);
            end[k] = (__builtin_amdgcn_readlane(my_e1, row) - t0[k]) * vpt + (k > 0 ? end[k - 1] : 0);
        }
        #pragma unroll 1
        for (int q0 = 0; q0 < end[3]; q0 += 256) {
            V v[4];
            int32_t xi[4][VEC];
            int rk[4];
            #pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u * 64 + lane;
                // past the end: the first piece of some tile, not used
                const bool have = q < end[3];
                const int k = have ? (q >= end[0]) + (q >= end[1]) + (q >= end[2]) : 0;
                const int at = have ? q - (k == 0 ? 0 : (k == 1 ? end[0] : (k == 2 ? end[1] : end[2]))) : 0;
                const int tk = k == 0 ? t0[0] : (k == 1 ? t0[1] : (k == 2 ? t0[2] : t0[3]));
                const int rrk = k == 0 ? rr[0] : (k == 1 ? rr[1] : (k == 2 ? rr[2] : rr[3]));
                const int tl = at / vpt, cg = (at - tl * vpt) * VEC;
                const int t = have ? tk + tl : 0;
                rk[u] = have ? wave + k * kUW : -1;
                v[u] = load16<V>(reinterpret_cast<const WT*>(a.vals) + ((size_t)t * a.bh + rrk) * a.bw + cg);
                #pragma unroll
                for (int e = 0; e < VEC; ++e) xi[u][e] = a.xidx[(size_t)t * a.bw + cg + e];
            }
            #pragma unroll
            for (int u = 0; u < 4; ++u)
                #pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (rk[u] >= 0 && xi[u][e] >= 0) place(rk[u], xi[u][e], v[u][e]);
        }
    };
    // where column k of row r of a 16-row block lies in a list of A fragments
    auto frag_pos = [&](int k, int r, int blocks, int rb) {
        const int ks = k / SK, kr = k - ks * SK;
        return (((ks * blocks + rb) * 64) + (kr / VEC) * 16 + r) * VEC + kr % VEC;
    };
    const int hsteps = a.hsteps, xsteps = a.xsteps;
    const int nh = hsteps > wave ? (hsteps - wave + kUW - 1) / kUW : 0;     // k-steps wave, wave + 4, ...
    const int nx = xsteps > wave ? (xsteps - wave + kUW - 1) / kUW : 0;
    V w[HS][RB];
    #pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        __syncthreads();
        for (int i = tid; i < hsteps * 64; i += kUT) xw[i] = V(0);
        __syncthreads();
        scatter_rows(rb, [&](int r, int n, WT v) { if (n < a.H) reinterpret_cast<WT*>(smem)[frag_pos(n, r, 1, 0)] = v; });
        __syncthreads();
        #pragma unroll
        for (int i = 0; i < HS; ++i) w[i][rb] = i < nh ? xw[(wave + i * kUW) * 64 + lane] : V(0);
    }
    __syncthreads();
    for (int i = tid; i < xsteps * RB * 64; i += kUT) xw[i] = V(0);
    __syncthreads();
    if (xsteps > 0) {
        #pragma unroll 1
        for (int rb = 0; rb < RB; ++rb)
            scatter_rows(rb, [&](int r, int n, WT v) { if (n >= a.H) reinterpret_cast<WT*>(smem)[frag_pos(n - a.H, r, RB, rb)] = v; });
    }

    // ---- cell threads: (unit, batch row), the VEC units of a group side by side -------------------------------
    const int ce = tid % VEC, cb = (tid / VEC) % a.bt, cu = tid / (VEC * a.bt) * VEC + ce;
    const bool cell_wave = wave * 64 < U * a.bt;        // uniform over the wavefront
    const bool has = cu < U && unit0 + cu < a.H && cb < nb;
    if (tid < U * 4) s_bias[tid] = unit0 + (tid >> 2) < a.H ? a.bias_p[a.invprow[(tid & 3) * a.H + unit0 + (tid >> 2)]] : 0.f;
    const int state = has ? (b0 + cb) * a.H + unit0 + cu : 0;
    float c_state = has ? a.c[state] : 0.f;
    const int red_at = (cb * U + (cu ^ (cb & (U - 1)))) * 4;
    const int red_wr = ((wave * a.bt + li) * U + (lg ^ (li & (U - 1)))) * 4;   // unit lg of batch row li, see below
    const int h_at = (int)frag_index(cb, unit0 + cu, a.bt, SHIFT);   // its place in the exchange buffer

    // ---- addresses of the B fragments; rows past the last repeat it (their sums are never read) -----------------
    int hoff[NBT], xrow[NBT];
    #pragma unroll
    for (int n = 0; n < NBT; ++n) {
        const int col = PAIR ? li & 7 : n * 16 + li, b = col < nb ? col : nb - 1;
        hoff[n] = (((wave + (PAIR ? li >> 3 : 0) * kUW) * 4 + lg) * a.bt + b) * 16;
        xrow[n] = b * a.xs_row;
    }
    // a word per lane: k-step lane/4 of the wavefront, group lane%4 of it, last batch row
    const int probe = ((wave + (nh > 0 ? (lane >> 2) % nh : 0) * kUW) * 4 + (lane & 3)) * a.bt * 16 + (nb - 1) * 16 + 12;
    const int hstep = kUW * 4 * a.bt * 16;              // bytes from one k-step of the wavefront to its next
    u32x4 xv[kUX / PS][NBT];
    auto load_x = [&](int t) {
        const WT* xt = reinterpret_cast<const WT*>(a.xs) + (size_t)t * a.xs_step + (long long)b0 * a.xs_row;
        #pragma unroll
        for (int i = 0; i < kUX / PS; ++i) {
            const int grp = (wave + (i * PS + (PAIR ? li >> 3 : 0)) * kUW) * 4 + lg;
            #pragma unroll
            for (int n = 0; n < NBT; ++n) {
                xv[i][n] = u32x4(0);
                if (i * PS < nx && grp < a.xgroups) xv[i][n] = load16<u32x4>(xt + xrow[n] + grp * VEC);
            }
        }
    };
    load_x(0);
    __syncthreads();                                    // x weights are in LDS

    for (int t = 0; t < a.steps; ++t) {
        const int stamp = t + 1;
        // addresses are made from these anew in every step: kept in registers across the loop they cost 30
        int xl = lane * (int)sizeof(V), wl = red_wr, rl = red_at;
        asm volatile("" : "+v"(xl), "+v"(wl), "+v"(rl));
        int* flag = s_flag[t & 1];
        char* hbase = reinterpret_cast<char*>(a.hx) + (size_t)t * a.step_bytes + (size_t)team * a.team_bytes;
        bool dead = false;

        // x part: while h is on its way
        f32x4 acc[PS][RB][NBT];
        #pragma unroll
        for (int p = 0; p < PS; ++p)
            #pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                #pragma unroll
                for (int n = 0; n < NBT; ++n) acc[p][rb][n] = f32x4(0);
        typename PT::Top xtop{};
        #pragma unroll
        for (int i = 0; i < kUX; ++i) {
            if (i >= nx) continue;                      // wave-uniform
            if (i % PS == 0)
                #pragma unroll
                for (int n = 0; n < NBT; ++n) take_top<WT, PT::kMagnitude>(xtop, xv[i / PS][n]);
            #pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const V wv = *reinterpret_cast<const V*>(smem + ((wave + i * kUW) * RB + rb) * 1024 + xl);
                #pragma unroll
                for (int n = 0; n < NBT; ++n)
                    #pragma unroll
                    for (int e = 0; e < MF::NE; ++e) acc[i % PS][rb][n] = MF::run(wv, __builtin_bit_cast(V, xv[i / PS][n]), acc[i % PS][rb][n], e);
            }
        }
        bool odd = PT::odd_magnitude(xtop);

        // h part: 16-byte device-coherent loads (volatile: a poll must not be merged with the one before)
        {
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(hbase, 0, (int)a.team_bytes, 0x00027000);
            constexpr int kCoherent = (int)(16u | (1u << 31));
            u32x4 hv[HS / PS][NBT];
            uint32_t spins = 0;
            if (nh > 0) {
                // The fragments, all at once (past the last k-step the loads are out of the buffer's range and give
                // zero).  Whoever comes early first polls one word of every producer until none is the mark; the cell
                // threads come latest and read at once.  Where something is still missing, both again.
                for (bool early = !cell_wave;; early = true) {
                    while (early) {
                        typename PT::Top top{};
                        PT::top(top, __builtin_amdgcn_raw_buffer_load_b32(rs, probe, 0, kCoherent));
                        if (!__any(PT::mark(top))) break;
                        if (!unit_keep_waiting(a.ctl, spins)) { dead = true; break; }
                    }
                    int hl[NBT];
                    #pragma unroll
                    for (int n = 0; n < NBT; ++n) { hl[n] = hoff[n]; asm volatile("" : "+v"(hl[n])); }
                    #pragma unroll
                    for (int i = 0; i < HS / PS; ++i)
                        #pragma unroll
                        for (int n = 0; n < NBT; ++n) hv[i][n] = __builtin_amdgcn_raw_buffer_load_b128(rs, hl[n] + i * PS * hstep, 0, kCoherent);
                    typename PT::Top top{};
                    #pragma unroll
                    for (int i = 0; i < HS / PS; ++i)
                        #pragma unroll
                        for (int n = 0; n < NBT; ++n) take_top<WT>(top, hv[i][n]);
                    if (__any(PT::mark(top)) && !dead) {
                        dead = !unit_keep_waiting(a.ctl, spins);
                        continue;
                    }
                    odd |= PT::odd(top);
                    break;
                }
                if (t == 0) {                           // the caller's h_0 may be infinite
                    typename PT::Top top{};
                    #pragma unroll
                    for (int i = 0; i < HS / PS; ++i)
                        #pragma unroll
                        for (int n = 0; n < NBT; ++n) take_top<WT, PT::kMagnitude>(top, hv[i][n]);
                    odd |= PT::odd_magnitude(top);
                }
                #pragma unroll
                for (int i = 0; i < HS; ++i)
                    #pragma unroll
                    for (int e = 0; e < MF::NE; ++e)
                        #pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
                            #pragma unroll
                            for (int n = 0; n < NBT; ++n)
                                acc[i % PS][rb][n] = MF::run(w[i][rb], __builtin_bit_cast(V, hv[i / PS][n]), acc[i % PS][rb][n], e);
            }
        }
        if (t + 1 < a.steps) load_x(t + 1);
        if (a.slots == 1 && t > 0) lds_barrier();       // the cell threads have read the sums of the step before
        float* red = red0 + (a.slots == 2 && (t & 1) ? red_slot : 0);
        // accumulator element v of lane l: gate v of unit rb*4 + l/16, batch row l%16
        #pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            #pragma unroll
            for (int n = 0; n < NBT; ++n) {
                const int col = n * 16 + li;
                f32x4 sum = acc[0][rb][n];
                if constexpr (PAIR) {                   // columns 8-15 of the odd k-steps
                    #pragma unroll
                    for (int v = 0; v < 4; ++v) sum[v] = dpp_add_from<0x128>(sum[v], acc[PS - 1][rb][n][v]);
                }
                if (col < a.bt)
                    *reinterpret_cast<f32x4*>(red + n * 16 * U * 4 + (wl ^ (rb * 16))) = sum;
            }
        if (dead && lane == 0) flag[0] = stamp;
        if (__any(odd) && lane == 0) flag[1] = stamp;
        lds_barrier();
        const bool stop = __builtin_amdgcn_readfirstlane(flag[0]) == stamp, slow = __builtin_amdgcn_readfirstlane(flag[1]) == stamp;
        if (stop) return;                               // the same in every wavefront: the flags of a parity change two barriers later
        if (slow)
            slow_step<WT, RB>(a, reinterpret_cast<const WT*>(hbase), reinterpret_cast<const WT*>(a.xs) + (size_t)t * a.xs_step + (long long)b0 * a.xs_row,
                              unit0, nb, red);
        if (cell_wave) {
            f32x4 z = f32x4(0);
            float h_state = 0.f;
            if (has) {
                #pragma unroll
                for (int k = 0; k < kUW; ++k) z += *reinterpret_cast<const f32x4*>(red + k * a.bt * U * 4 + rl);
                #pragma unroll
                for (int q = 0; q < 4; ++q) z[q] += s_bias[cu * 4 + q];
                c_state = usigm(z[1]) * c_state + usigm(z[0]) * tanhf(z[2]);
                h_state = usigm(z[3]) * tanhf(c_state);
            }
            if (t + 1 < a.steps) {
                char* nbase = hbase + a.step_bytes;
                const uint32_t bits = has ? PT::bits(h_state) : 0u;
                if constexpr (sizeof(WT) == 2) {
                    const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits, 0xB1, 0xF, 0xF, false);   // the next unit, 0 past the last
                    if (has && (ce & 1) == 0) ust32(reinterpret_cast<uint32_t*>(nbase) + (h_at >> 1), bits | (other << 16));
                } else {
                    if (has) ust32(reinterpret_cast<uint32_t*>(nbase) + h_at, bits);
                }
            } else if (has) {
                a.c[state] = c_state;
                a.h[state] = h_state;
                if (a.z_dbg) {
                    float* zd = a.z_dbg + (size_t)(b0 + cb) * 4 * a.H + unit0 + cu;
                    #pragma unroll
                    for (int q = 0; q < 4; ++q) zd[q * a.H] = z[q];
                }
            }
        }
    }
}

// Exchange buffers: h_0 in step 0, the mark in every later step, zero past the last unit; clears the control words and
// saves h_0 and c_0.  Where the caller's rows are not whole aligned 16-byte groups, also a zero-padded copy of them.
template <typename WT>
__global__ void __launch_bounds__(256) lstm_units_prepare_kernel(const WT* __restrict__ xs, const float* __restrict__ h0, const float* __restrict__ c0, float* __restrict__ saved, char* __restrict__ hx, char* __restrict__ xc,
                                                                 uint32_t* __restrict__ ctl, int H, int I, int batch, int bt, int hgroups, int xcgroups,
                                                                 int teams, int steps) {
    constexpr int VEC = Elem<WT>::VEC;
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int k = threadIdx.x; k < (int)kLstmCtlBytes / 4; k += 256) ctl[k] = 0u;
    const int first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
    // spread over all workgroups: by those of the first step alone it cost up to 2 us
    const int n = batch * H, all = stride * gridDim.y;
    for (int i = blockIdx.y * stride + first; i < n; i += all) { saved[i] = h0[i]; saved[n + i] = c0[i]; }
    const int per_team = hgroups * bt, per_step = per_team * teams, per_x = xcgroups * batch;
    for (int t = blockIdx.y; t < steps; t += gridDim.y) {
        for (int i = first; i < per_step; i += stride) {
            const int k = i / per_team, q = i - k * per_team, g = q / bt;
            const int b = k * bt + (q - g * bt);
            u32x4 v;
            #pragma unroll
            for (int word = 0; word < 4; ++word) {
                uint32_t u = 0;
                #pragma unroll
                for (int s = 0; s < VEC / 4; ++s) {
                    const int j = g * VEC + word * (VEC / 4) + s;
                    uint32_t bits = 0;
                    if (j < H) {
                        if (t > 0) bits = VEC == 8 ? 0xFFFFu : 0xFFFFFFFFu;
                        else if (b < batch) bits = Pattern<WT>::bits(h0[(size_t)b * H + j]);
                    }
                    u |= bits << (16 * s);
                }
                v[word] = u;
            }
            reinterpret_cast<u32x4*>(hx)[(size_t)t * per_step + i] = v;
        }
        for (int i = first; i < per_x; i += stride) {
            const int b = i / xcgroups, c = (i - b * xcgroups) * VEC;
            const WT* row = xs + ((size_t)t * batch + b) * I;
            typename Elem<WT>::vec v;
            #pragma unroll
            for (int e = 0; e < VEC; ++e) v[e] = c + e < I ? row[c + e] : WT(0);
            reinterpret_cast<typename Elem<WT>::vec*>(xc)[(size_t)t * per_x + i] = v;
        }
    }
}

struct UnitForm { int rb, hs, nbt; bool pair; };
// In order of preference.  Few gate rows per workgroup keep a step's matrix work short; more of them, or more batch
// rows per team, need fewer workgroups.
constexpr int kNForms = 5;
constexpr UnitForm kForms[kNForms] = {{2, 8, 1, true}, {2, 16, 1, true}, {2, 8, 1, false}, {4, 8, 1, false}, {2, 8, 2, false}};

using UnitKernel = void (*)(UnitArgs);
template <typename WT>
UnitKernel units_kernel(int form) {
    switch (form) {
        case 0: return lstm_units_kernel<WT, 2, 8, 1, true>;
        case 1: return lstm_units_kernel<WT, 2, 16, 1, true>;
        case 2: return lstm_units_kernel<WT, 2, 8, 1, false>;
        case 3: return lstm_units_kernel<WT, 4, 8, 1, false>;
        default: return lstm_units_kernel<WT, 2, 8, 2, false>;
    }
}

struct UnitShape { int form, teams, bt, wgs, hsteps, xsteps, slots; size_t smem; };

// Compute units of a device, or 0; makes the LDS of the kernels available and checks that two workgroups of each fit
// a compute unit.  Asked once per device.
int units_device(int device) {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> known[kMaxDevices];         // 0 unknown, -1 unusable, else compute units
    if (device < 0 || device >= kMaxDevices) return 0;
    std::atomic<int>& k = known[device];
    if (const int v = k.load(std::memory_order_acquire)) return v > 0 ? v : 0;
    int prev = -1, cus = 0;
    if (hipGetDevice(&prev) != hipSuccess) { (void)hipGetLastError(); return 0; }
    if (prev != device && hipSetDevice(device) != hipSuccess) { (void)hipGetLastError(); return 0; }
    bool ok = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0;
    for (int wd : {PIVOT_F32, PIVOT_F16})
        for (int f = 0; ok && f < kNForms; ++f) {
            int per_cu = 0;
            const void* fn = reinterpret_cast<const void*>(wd == PIVOT_F32 ? units_kernel<float>(f) : units_kernel<_Float16>(f));
            ok = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kULds) == hipSuccess &&
                 hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kUT, kULds) == hipSuccess && per_cu >= 2;
        }
    if (!ok) (void)hipGetLastError();
    if (prev != device) (void)hipSetDevice(prev);
    k.store(ok ? cus : -1, std::memory_order_release);
    return ok ? cus : 0;
}

// Whether form f takes the sizes, and how.
bool units_form(int wdtype, int H, int I, int batch, int f, UnitShape* out) {
    const int sk = 64 / elem_size(wdtype);
    const UnitForm& F = kForms[f];
    UnitShape& s = *out;
    s.form = f;
    s.hsteps = (H + sk - 1) / sk; s.xsteps = (I + sk - 1) / sk;
    if (s.hsteps > F.hs * kUW || s.xsteps > kUX * kUW) return false;
    const int rows = F.pair ? 8 : 16 * F.nbt;
    s.teams = (batch + rows - 1) / rows;
    s.bt = (batch + s.teams - 1) / s.teams;
    s.teams = (batch + s.bt - 1) / s.bt;
    s.wgs = (H + 4 * F.rb - 1) / (4 * F.rb);
    const size_t xw = (size_t)s.xsteps * F.rb * 1024, red = (size_t)kUW * s.bt * F.rb * 16 * 4;
    s.slots = xw + 2 * red <= kULds ? 2 : 1;
    s.smem = std::max((size_t)s.hsteps * 1024, xw + s.slots * red);
    return s.smem <= kULds;
}

// The first form that takes the sizes with at most `limit` workgroups.
bool units_shape(const HostPlan& hp, int H, int I, int batch, int limit, UnitShape* out) {
    for (int f = 0; f < kNForms; ++f)
        if (units_form(hp.d.wdtype, H, I, batch, f, out) && (long long)out->teams * out->wgs <= limit) return true;
    return false;
}

// A workgroup takes at most half a compute unit.  Launches on different streams that hold part of the device and wait
// for the rest would wait for each other, so the grid is such that as many launches as a process has hardware queues
// (4) are resident together: half the compute units.  Plans that the form exchanging gate sums takes may use them all
// (two launches fit; of that form's one or two).
bool pick(const HostPlan& hp, int H, int I, int batch, int device, UnitShape* s) {
    if (hp.d.layout != PIVOT_BRC || hp.T < 1 || H < 1 || I < 0) return false;
    const int cus = units_device(device);
    if (cus < 2) return false;
    const bool all = lstm_persist_supported(hp, H, batch, device, nullptr, nullptr);
    return units_shape(hp, H, I, batch, all ? cus : cus / 2, s);
}

size_t units_hx_step(const UnitShape& s) { return (size_t)s.hsteps * 4 * s.bt * s.teams * 16; }
size_t units_xc_step(const UnitShape& s, int batch) { return (size_t)s.xsteps * 4 * batch * 16; }

template <typename WT>
int launch_units_t(const LstmPersistLaunch& P, const UnitShape& s) {
    const HostPlan& hp = *P.hp;
    hipStream_t st = reinterpret_cast<hipStream_t>(P.stream);
    constexpr int VEC = Elem<WT>::VEC;
    const bool direct = P.I % VEC == 0 && (reinterpret_cast<uintptr_t>(P.xs) & 15) == 0;
    char* hx = reinterpret_cast<char*>(P.xg);
    char* xc = hx + units_hx_step(s) * P.steps;
    const int hgroups = s.hsteps * 4, xcgroups = direct ? 0 : s.xsteps * 4;
    const int per_step = std::max(hgroups * s.bt * s.teams, xcgroups * P.batch);
    const dim3 blocks((per_step + 255) / 256, std::min(P.steps, 1024));
    hipLaunchKernelGGL(lstm_units_prepare_kernel<WT>, blocks, dim3(256), 0, st, reinterpret_cast<const WT*>(P.xs), P.h, P.c, P.saved, hx, xc, P.ctl,
                       P.H, P.I, P.batch, s.bt, hgroups, xcgroups, s.teams, P.steps);
    HIP_TRY(hipGetLastError());
    UnitArgs a;
    a.vals = P.vals; a.xidx = P.xidx; a.row_ptr = P.row_ptr; a.invprow = P.invprow; a.bias_p = P.bias_p;
    a.xs = direct ? P.xs : xc; a.hx = hx; a.ctl = P.ctl; a.h = P.h; a.c = P.c; a.z_dbg = P.z_dbg;
    a.xs_row = direct ? P.I : xcgroups * VEC; a.xs_step = (long long)P.batch * a.xs_row; a.xgroups = a.xs_row / VEC;
    a.step_bytes = units_hx_step(s); a.team_bytes = a.step_bytes / s.teams;
    a.H = P.H; a.I = P.I; a.batch = P.batch; a.steps = P.steps; a.bt = s.bt; a.wgs = s.wgs;
    a.bh = hp.d.bh; a.bw = hp.d.bw; a.hsteps = s.hsteps; a.xsteps = s.xsteps; a.slots = s.slots;
    const int grid = s.teams * s.wgs;
    hipLaunchKernelGGL(units_kernel<WT>(s.form), dim3(P.give_up && grid > 1 ? grid - 1 : grid), dim3(kUT), s.smem, st, a);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

}  // namespace

bool lstm_units_supported(const HostPlan& hp, int H, int I, int batch, int device) {
    UnitShape s;
    return pick(hp, H, I, batch, device, &s);
}

std::string lstm_units_name(const HostPlan& hp, int H, int I, int batch, int device) {
    UnitShape s;
    if (!pick(hp, H, I, batch, device, &s)) return "";
    const UnitForm& F = kForms[s.form];
    char buf[128];
    snprintf(buf, sizeof buf, "lstm_units_kernel<%s, %d, %d, %d, %s> teams %d sums %d", hp.d.wdtype == PIVOT_F32 ? "float" : "_Float16", F.rb, F.hs, F.nbt,
             F.pair ? "true" : "false", s.teams, s.slots);
    return buf;
}

// Before the first step a wavefront goes through the tiles of its rows, 256 pieces of 16 bytes at a time, twice.  Us for
// 4 / 6 / 8 / 12 steps, this form against the launches it replaces (the other one-launch form or one per step):
// 2048 units, 1024 inputs, batch 8, equal rows (48 pieces) 33.6 / 39.5 / 44.6 / 56.0 against 42.8 / 55.6 / 68.1 / 93.5,
// Zipf rows (the longest 384 pieces) 55.2 / 60.8 / 66.7 / 77.7 against 45.4 / 58.7 / 72.4 / 99.1.
int lstm_units_min_steps(const HostPlan& hp) {
    return (long long)hp.max_row_tiles * hp.d.bw * elem_size(hp.d.wdtype) / 16 <= 128 ? 4 : 8;
}

size_t lstm_units_step_bytes(const HostPlan& hp, int batch) {
    // the same on every device and for a host-only plan: the largest of the forms that take the sizes
    const int H = hp.d.M / 4, I = hp.d.K - H;
    if (hp.d.layout != PIVOT_BRC || hp.T < 1 || (hp.d.flags & PIVOT_PLAN_LSTM_LAUNCH_PER_STEP) || H < 1 || 4 * H != hp.d.M || I < 0) return 0;
    size_t most = 0;
    for (int f = 0; f < kNForms; ++f) {
        UnitShape s;
        if (units_form(hp.d.wdtype, H, I, batch, f, &s)) most = std::max(most, units_hx_step(s) + units_xc_step(s, batch));
    }
    return most;
}

int launch_lstm_units(const LstmPersistLaunch& P) {
    UnitShape s;
    if (!pick(*P.hp, P.H, P.I, P.batch, P.device, &s)) {
        set_error("internal: one-exchange recurrent kernel not available for this plan");
        return PIVOT_E_UNSUPPORTED;
    }
    return P.hp->d.wdtype == PIVOT_F32 ? launch_units_t<float>(P, s) : launch_units_t<_Float16>(P, s);
}

}  // namespace pivot
