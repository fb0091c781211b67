// Utility kernels around the layer kernels: workspace clearing, the empty
// kernel used to measure the launch floor, the pre-gather of x for the
// matrix-core path, the dense comparator and the LSTM cell.
#include "pivot_fc_kernels.h"

namespace pivot {

// ---------------------------------------------------------------------------
// x in natural order -> fragment order (pivot_frag.h): the group fetch through
// P_col, once per launch instead of once per kept tile.
// gather_frag_kernel: a workgroup copies ONE row of x into LDS, whole, with
// coalesced loads, and makes one segment of its groups from there; gathered
// straight from memory every element moves a line of its own.  The segment is
// the fastest grid dimension and a multiple of 8 of them are launched, so the
// workgroups that write the batch rows of one group, 16 bytes of a line each,
// share an XCD (round-robin over workgroups) and its L2 makes whole lines of
// them.
// gather_frag_far_kernel: rows too long for LDS.  A workgroup makes 32 groups
// for eight batch rows; half a wavefront takes one batch row, and the groups
// change places through LDS so that they are stored as whole 128-byte lines.
// ---------------------------------------------------------------------------
template <typename WT>
struct GroupIdx {
    int4 s4[Elem<WT>::VEC / 4];
    __device__ __forceinline__ void load(const int32_t* pcol_pad, int g) {
        #pragma unroll
        for (int q = 0; q < Elem<WT>::VEC / 4; ++q) s4[q] = reinterpret_cast<const int4*>(pcol_pad + (size_t)g * Elem<WT>::VEC)[q];
    }
    __device__ __forceinline__ typename Elem<WT>::vec gather(const WT* row) const {
        constexpr int VEC = Elem<WT>::VEC;
        int src[VEC];
        #pragma unroll
        for (int q = 0; q < VEC / 4; ++q) { src[4 * q] = s4[q].x; src[4 * q + 1] = s4[q].y; src[4 * q + 2] = s4[q].z; src[4 * q + 3] = s4[q].w; }
        typename Elem<WT>::vec v;
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = row[src[e] > 0 ? src[e] : 0];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = src[e] >= 0 ? v[e] : WT(0);
        return v;
    }
};

template <typename WT>
__global__ void __launch_bounds__(512) gather_frag_kernel(const int32_t* __restrict__ pcol_pad, const WT* __restrict__ x,
                                                          WT* __restrict__ xg, long long ldx, int K, int ngroups, int batch, int seg_groups) {
    using V = typename Elem<WT>::vec;
    constexpr int VEC = Elem<WT>::VEC, NT = 512;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, b = blockIdx.y;
    // whole aligned 16-byte pieces, from the one that holds the row's first element to the one that holds its last
    const WT* xr = x + (long long)b * ldx;
    const int shift = (int)(reinterpret_cast<uintptr_t>(xr) & 15) / (int)sizeof(WT);
    const int nvec = (shift + K + VEC - 1) / VEC;
    const V* xv = reinterpret_cast<const V*>(xr - shift);
    const int g0 = blockIdx.x * seg_groups, g1 = g0 + seg_groups < ngroups ? g0 + seg_groups : ngroups;
    GroupIdx<WT> gi;
    gi.load(pcol_pad, g0 + tid < g1 ? g0 + tid : 0);
    // straight into LDS: no register waits for another piece (kept in registers behind a test per piece, the compiler
    // waited for the second piece before it asked for the third)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    #pragma unroll
    for (int u = 0; u < 9; ++u) {                       // 64 KB by 512 threads (and one piece): the whole row at once
        const int i = u * NT + tid;
        if (i < nvec)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xv + i),
                                             (__attribute__((address_space(3))) void*)(smem + (u * NT + wave * 64) * 16), 16, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const WT* row = reinterpret_cast<const WT*>(smem) + shift;
    for (int g = g0 + tid; g < g1; g += NT) {
        if (g != g0 + tid) gi.load(pcol_pad, g);
        reinterpret_cast<V*>(xg)[(size_t)g * batch + b] = gi.gather(row);
    }
}

template <typename WT>
__global__ void __launch_bounds__(256) gather_frag_far_kernel(const int32_t* __restrict__ pcol_pad, const WT* __restrict__ x,
                                                              WT* __restrict__ xg, long long ldx, int ngroups, int batch) {
    using V = typename Elem<WT>::vec;
    __shared__ V s_v[32][9];
    const int tid = threadIdx.x;
    const int g0 = blockIdx.x * 32, b0 = blockIdx.y * 8;
    {
        const int gl = tid & 31, bl = tid >> 5;
        const int g = g0 + gl < ngroups ? g0 + gl : ngroups - 1, b = b0 + bl < batch ? b0 + bl : batch - 1;
        GroupIdx<WT> gi;
        gi.load(pcol_pad, g);
        s_v[gl][bl] = gi.gather(x + (long long)b * ldx);
    }
    __syncthreads();
    const int gl = tid >> 3, bl = tid & 7;
    if (g0 + gl < ngroups && b0 + bl < batch) reinterpret_cast<V*>(xg)[(size_t)(g0 + gl) * batch + b0 + bl] = s_v[gl][bl];
}

template <typename WT>
static int launch_gather_frag_t(const WT* x, int64_t ldx, const int32_t* pcol_pad, WT* xg, int K, int K_pad, int batch, hipStream_t st) {
    const int ngroups = K_pad / Elem<WT>::VEC;
    const size_t smem = gather_row_lds(reinterpret_cast<uintptr_t>(x), ldx, K, sizeof(WT));
    // The copy pays for long fp16 inputs of many elements (us per call of a layer with 1000 outputs, 16x32 tiles, 25 %
    // kept, copied / direct: 2048 columns, batch 64 6.1 / 5.9; 3000, 64 6.5 / 7.1; 4090, 64 7.6 / 8.2; 4096, 32 6.0 / 6.2;
    // 9216, 16 7.0 / 7.4; 12000, 17 8.3 / 9.1; 25088, 8 10.0 / 10.3; with 4096 outputs, 32x32 tiles: 2048, 64 9.1 / 9.2;
    // 4096, 32 7.8 / 8.5; 8000, 32 9.8 / 10.3).  Of fp32 rows a line holds half as many elements and the copy is twice as
    // long: 9216 columns, batch 16 8.4 / 6.9 and 64 12.7 / 10.6, always slower.  To the longest row that fits, aligned or
    // not: 32768, 32x32 tiles, 10 %, batch 64 13.3 / 17.4, 32 unaligned 9.6 / 12.1.
    if (sizeof(WT) == 2 && smem > 0 && K >= 3000 && (size_t)batch * K >= 128 * 1024) {
        const int segs = 8;
        if (smem > 64 * 1024)                           // (unaligned rows of 32761 to 32768 columns)
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(gather_frag_kernel<WT>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        hipLaunchKernelGGL(gather_frag_kernel<WT>, dim3(segs, batch), dim3(512), smem, st, pcol_pad, x, xg, (long long)ldx, K, ngroups, batch, (ngroups + segs - 1) / segs);
    } else {
        hipLaunchKernelGGL(gather_frag_far_kernel<WT>, dim3((ngroups + 31) / 32, (batch + 7) / 8), dim3(256), 0, st, pcol_pad, x, xg, (long long)ldx, ngroups, batch);
    }
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

int launch_gather_frag(const void* x, int64_t ldx, const int32_t* pcol_pad, void* xg, int K, int K_pad, int batch,
                       int wdtype, void* stream) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (wdtype == PIVOT_F16) return launch_gather_frag_t<_Float16>((const _Float16*)x, ldx, pcol_pad, (_Float16*)xg, K, K_pad, batch, st);
    return launch_gather_frag_t<float>((const float*)x, ldx, pcol_pad, (float*)xg, K, K_pad, batch, st);
}

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
__global__ void fill_zero_kernel(uint32_t* p, size_t nwords) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < nwords; i += stride) p[i] = 0u;
}

__global__ void null_kernel() {}

int launch_null(void* stream) {
    hipLaunchKernelGGL(null_kernel, dim3(1), dim3(64), 0, reinterpret_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

// Reads `npieces` KB once: wavefront w reads pieces [w*per, (w+1)*per), 16 bytes per lane and piece, eight
// pieces in flight, adds everything up and stores one float per wavefront.  Nothing but the read: what one
// launch of the layer kernel cannot beat for the same number of bytes.
__global__ void __launch_bounds__(512) stream_read_kernel(const f32x4* __restrict__ base, int npieces, int per_wave,
                                                           float* __restrict__ out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gw = blockIdx.x * (blockDim.x >> 6) + wave;
    const int last = npieces > 0 ? npieces - 1 : 0;
    float acc = 0.f;
    for (int k0 = 0; k0 < per_wave; k0 += 8) {
        f32x4 w[8];
        #pragma unroll
        for (int u = 0; u < 8; ++u) {
            int piece = gw * per_wave + k0 + u;
            piece = piece < last ? piece : last;
            w[u] = base[(size_t)piece * 64 + lane];
        }
        #pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u < per_wave && gw * per_wave + k0 + u < npieces) acc += w[u].x + w[u].y + w[u].z + w[u].w;
    }
    acc = group_sum<64>(acc);
    if (lane == 0) out[gw] = acc;
}

int launch_stream_read(const void* buf, size_t bytes, float* out, void* stream) {
    const int G = 256, W = 8;
    const int npieces = (int)(bytes / 1024);
    if (npieces < 1) { set_error("stream read needs at least 1 KB"); return PIVOT_E_SHAPE; }
    const int per_wave = (npieces + G * W - 1) / (G * W);
    hipLaunchKernelGGL(stream_read_kernel, dim3(G), dim3(W * 64), 0, reinterpret_cast<hipStream_t>(stream),
                       reinterpret_cast<const f32x4*>(buf), npieces, per_wave, out);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

// ---------------------------------------------------------------------------
// What one trip between two workgroups costs (see pivot_exchange_probe_run).
// Scratch: [8 int64 results][pad to 1 KB][256 words: XCD + 1 of every workgroup][flag words, one per 256-byte line].
// Every wait is bounded; a workgroup that gives up reports -1 and its partner runs into its own bound.
// ---------------------------------------------------------------------------
constexpr int kProbeMaxWg = 256;
constexpr unsigned kProbeMaxSpin = 1u << 20;
constexpr int kProbeTabOff = 1024, kProbeFlagOff = 4096;          // bytes

template <int SCOPE>
__device__ bool probe_bounce(unsigned* a2b, unsigned* b2a, bool is_a, int rounds) {
    for (int i = 1; i <= rounds; ++i) {
        const unsigned v = (unsigned)i;
        unsigned spins = 0;
        if (is_a) {
            __hip_atomic_store(a2b, v, __ATOMIC_RELAXED, SCOPE);
            while (__hip_atomic_load(b2a, __ATOMIC_RELAXED, SCOPE) != v) { if (++spins > kProbeMaxSpin) return false; }
        } else {
            while (__hip_atomic_load(a2b, __ATOMIC_RELAXED, SCOPE) != v) { if (++spins > kProbeMaxSpin) return false; }
            __hip_atomic_store(b2a, v, __ATOMIC_RELAXED, SCOPE);
        }
    }
    return true;
}

// plain stores (the L1 writes through to the XCD's L2), polls that invalidate the L1 first
__device__ bool probe_bounce_l2(unsigned* a2b, unsigned* b2a, bool is_a, int rounds) {
    volatile unsigned* va = a2b;
    volatile unsigned* vb = b2a;
    for (int i = 1; i <= rounds; ++i) {
        const unsigned v = (unsigned)i;
        unsigned spins = 0;
        if (is_a) {
            *va = v;
            for (;;) { asm volatile("buffer_inv sc0" ::: "memory"); if (*vb == v) break; if (++spins > kProbeMaxSpin) return false; }
        } else {
            for (;;) { asm volatile("buffer_inv sc0" ::: "memory"); if (*va == v) break; if (++spins > kProbeMaxSpin) return false; }
            *vb = v;
        }
    }
    return true;
}

__global__ void __launch_bounds__(64) exchange_probe_kernel(char* scratch, int nwg, int rounds) {
    extern __shared__ char one_per_cu[];                // sized so that a compute unit holds one workgroup
    long long* out = reinterpret_cast<long long*>(scratch);
    unsigned* tab = reinterpret_cast<unsigned*>(scratch + kProbeTabOff);
    unsigned* f = reinterpret_cast<unsigned*>(scratch + kProbeFlagOff);
    const int wg = blockIdx.x;
    if (threadIdx.x != 0) return;
    unsigned xcc = 0;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    xcc &= 0xFu;
    __hip_atomic_store(tab + wg, xcc + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // wait (bounded) until every workgroup has published, then pick the partners: the first workgroup on
    // workgroup 0's XCD and the first on another one (every workgroup computes the same two)
    bool all = false;
    for (unsigned spin = 0; spin < 4096u && !all; ++spin) {
        all = true;
        for (int i = 0; i < nwg; ++i)
            if (__hip_atomic_load(tab + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) { all = false; break; }
    }
    int pb = -1, pc = -1;
    if (all) {
        const unsigned x0 = __hip_atomic_load(tab + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int i = 1; i < nwg; ++i) {
            const unsigned xi = __hip_atomic_load(tab + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (pb < 0 && xi == x0) pb = i;
            if (pc < 0 && xi != x0) pc = i;
        }
    }
    if (!all || pb < 0 || pc < 0) { if (wg == 0) out[0] = -1; return; }
    if (wg != 0 && wg != pb && wg != pc) return;
    const bool is_a = wg == 0;
    if (wg == 0 || wg == pb) {
        long long t0 = wall_clock64();
        bool ok = probe_bounce<__HIP_MEMORY_SCOPE_AGENT>(f + 0, f + 64, is_a, rounds);
        long long t1 = wall_clock64();
        if (is_a) { out[1] = ok ? t1 - t0 : -1; out[4] = pb; }
        t0 = wall_clock64();
        ok = probe_bounce<__HIP_MEMORY_SCOPE_WORKGROUP>(f + 128, f + 192, is_a, rounds);
        t1 = wall_clock64();
        if (is_a) out[2] = ok ? t1 - t0 : -1;
        t0 = wall_clock64();
        ok = probe_bounce_l2(f + 256, f + 320, is_a, rounds);
        t1 = wall_clock64();
        if (is_a) out[6] = ok ? t1 - t0 : -1;
    }
    if (wg == 0 || wg == pc) {
        const long long t0 = wall_clock64();
        const bool ok = probe_bounce<__HIP_MEMORY_SCOPE_AGENT>(f + 384, f + 448, is_a, rounds);
        const long long t1 = wall_clock64();
        if (is_a) { out[3] = ok ? t1 - t0 : -1; out[5] = pc; }
    }
    if (is_a) out[0] = 1;
}

int launch_exchange_probe(void* scratch, int rounds, void* stream) {
    int dev = 0, cus = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int nwg = cus < kProbeMaxWg ? cus : kProbeMaxWg;
    if (nwg < 2) { set_error("the probe needs at least two compute units"); return PIVOT_E_UNSUPPORTED; }
    // 96 KB of LDS per workgroup: no two on one compute unit, so all of them are resident at once
    const size_t smem = 96 * 1024;
    static bool allowed[16] = {};
    if (!allowed[dev & 15]) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&exchange_probe_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        allowed[dev & 15] = true;
    }
    int rc = launch_fill_zero(scratch, PIVOT_PROBE_SCRATCH_BYTES, stream);
    if (rc != PIVOT_OK) return rc;
    hipLaunchKernelGGL(exchange_probe_kernel, dim3(nwg), dim3(64), smem, reinterpret_cast<hipStream_t>(stream),
                       reinterpret_cast<char*>(scratch), nwg, rounds);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

int launch_fill_zero(void* dev, size_t bytes, void* stream) {
    if (bytes == 0) return PIVOT_OK;
    if (bytes % 4 != 0 || (reinterpret_cast<uintptr_t>(dev) % 4) != 0) { set_error("fill needs 4-byte alignment"); return PIVOT_E_SHAPE; }
    size_t nwords = bytes / 4;
    int blocks = (int)((nwords + 255) / 256 > 2048 ? 2048 : (nwords + 255) / 256);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, reinterpret_cast<hipStream_t>(stream),
                       reinterpret_cast<uint32_t*>(dev), nwords);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

// ---------------------------------------------------------------------------
// dense comparator: y = act(W x + b), W streamed once, one wave per R rows,
// UN steps of the row loop in flight.  At batch 1 two rows per wavefront and 8
// steps (4096x9216 fp32 cold: 27.7 us = 5.5 TB/s; four rows and 2 steps, half
// the wavefronts per compute unit, 32.7 us; one row and 8 steps 28.0 us).
// ---------------------------------------------------------------------------
template <typename WT, int NB, int R, int UN>
__global__ void __launch_bounds__(256) dense_kernel(const WT* W, int M, int K, const WT* x, long long ldx,
                                                    const float* bias, float* y, long long ldy, int batch, int act) {
    using V = typename Elem<WT>::vec;
    constexpr int VEC = Elem<WT>::VEC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = (blockIdx.x * 4 + wave) * R;
    if (row0 >= M) return;
    float acc[R][NB];
    #pragma unroll
    for (int r = 0; r < R; ++r)
        #pragma unroll
        for (int b = 0; b < NB; ++b) acc[r][b] = 0.f;
    const WT* wrow[R];
    #pragma unroll
    for (int r = 0; r < R; ++r) wrow[r] = W + (size_t)((row0 + r < M) ? row0 + r : M - 1) * K;
    #pragma unroll UN
    for (int k = lane * VEC; k < K; k += 64 * VEC) {
        V wv[R];
        #pragma unroll
        for (int r = 0; r < R; ++r) wv[r] = load16<V>(wrow[r] + k);
        #pragma unroll
        for (int b = 0; b < NB; ++b) {
            const V xv = (b < batch) ? load16<V>(x + (size_t)b * ldx + k) : V(0);
            #pragma unroll
            for (int r = 0; r < R; ++r) acc[r][b] = dot_vec(wv[r], xv, acc[r][b]);
        }
    }
    #pragma unroll
    for (int r = 0; r < R; ++r)
        #pragma unroll
        for (int b = 0; b < NB; ++b) {
            float v = group_sum<64>(acc[r][b]);
            if (lane == 0 && row0 + r < M && b < batch)
                y[(size_t)b * ldy + row0 + r] = apply_act(v + (bias ? bias[row0 + r] : 0.f), act);
        }
}

template <typename WT, int NB, int R, int UN>
static int launch_dense_t(const void* W, int M, int K, const void* x, int64_t ldx, const float* bias,
                          void* y, int64_t ldy, int batch, int act, hipStream_t st) {
    int rows_per_block = 4 * R;
    dim3 grid((M + rows_per_block - 1) / rows_per_block);
    hipLaunchKernelGGL((dense_kernel<WT, NB, R, UN>), grid, dim3(256), 0, st, (const WT*)W, M, K, (const WT*)x,
                       (long long)ldx, bias, (float*)y, (long long)ldy, batch, act);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

int launch_dense(const void* W, int wdtype, int M, int K, const void* x, int64_t ldx, const float* bias,
                 void* y, int64_t ldy, int batch, int act, void* stream) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int vec = (wdtype == PIVOT_F32) ? 4 : 8;
    if (K % vec != 0 || ldx % vec != 0) { set_error("dense comparator needs K and ldx to be multiples of %d", vec); return PIVOT_E_UNSUPPORTED; }
    if (batch < 1 || batch > 16) { set_error("dense comparator supports batch 1..16"); return PIVOT_E_UNSUPPORTED; }
    // from 512 MB on the form with four rows per wavefront is the faster one again (16384x16384 fp32: 178 us against 193)
    const bool huge = (size_t)M * (size_t)K * (size_t)(wdtype == PIVOT_F32 ? 4 : 2) >= ((size_t)512 << 20);
    if (wdtype == PIVOT_F32) {
        if (batch == 1 && huge) return launch_dense_t<float, 1, 4, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
        if (batch == 1) return launch_dense_t<float, 1, 2, 8>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
        if (batch <= 4) return launch_dense_t<float, 4, 2, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
        return launch_dense_t<float, 16, 1, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
    }
    if (batch == 1 && huge) return launch_dense_t<_Float16, 1, 4, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
    if (batch == 1) return launch_dense_t<_Float16, 1, 2, 8>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
    if (batch <= 4) return launch_dense_t<_Float16, 4, 2, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
    return launch_dense_t<_Float16, 16, 1, 2>(W, M, K, x, ldx, bias, y, ldy, batch, act, st);
}

// ---------------------------------------------------------------------------
// generic sparse comparator: y = act(A x + b) with A in plain CSR (the kind of
// routine a pruned layer is usually handed to; Section 5.1 compares against
// one).  L lanes share a row; L is the power of two nearest the mean row length.
// ---------------------------------------------------------------------------
template <typename WT, int L>
__global__ void __launch_bounds__(256) csr_spmv_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                       const WT* __restrict__ val, const WT* __restrict__ x,
                                                       const float* __restrict__ bias, float* __restrict__ y, int M, int act) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = gid / L, sub = gid % L;
    const bool ok = row < M;
    const int b = ok ? row_ptr[row] : 0, e = ok ? row_ptr[row + 1] : 0;
    float acc = 0.f;
    for (int k = b + sub; k < e; k += L) acc = fmaf((float)val[k], (float)x[col[k]], acc);
    acc = group_sum<L>(acc);
    if (ok && sub == 0) y[row] = apply_act(acc + (bias ? bias[row] : 0.f), act);
}

template <typename WT>
static int launch_csr_t(const int32_t* row_ptr, const int32_t* col, const void* val, int M, int64_t nnz, const void* x,
                        const float* bias, float* y, int act, hipStream_t st) {
    const double mean = M > 0 ? (double)nnz / M : 0;
    int L = 1;
    while (L < 64 && L * 1.5 < mean) L *= 2;
#define CSR_CASE(L_)                                                                                                     \
    case L_: hipLaunchKernelGGL((csr_spmv_kernel<WT, L_>), dim3((unsigned)(((size_t)M * L_ + 255) / 256)), dim3(256), 0, \
                                st, row_ptr, col, (const WT*)val, (const WT*)x, bias, y, M, act); break;
    switch (L) { CSR_CASE(1) CSR_CASE(2) CSR_CASE(4) CSR_CASE(8) CSR_CASE(16) CSR_CASE(32) default: CSR_CASE(64) }
#undef CSR_CASE
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

int launch_csr(const int32_t* row_ptr, const int32_t* col, const void* val, int wdtype, int M, int64_t nnz, const void* x,
               const float* bias, float* y, int act, void* stream) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (wdtype == PIVOT_F32) return launch_csr_t<float>(row_ptr, col, val, M, nnz, x, bias, y, act, st);
    return launch_csr_t<_Float16>(row_ptr, col, val, M, nnz, x, bias, y, act, st);
}

// ---------------------------------------------------------------------------
// LSTM cell around the pruned gate matrix (gate order i,f,g,o).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float sigmoidf_(float v) { return 1.0f / (1.0f + __expf(-v)); }

// Few arguments: beyond 112 bytes of them a launch costs the host 0.07-0.7 us more (FcTail).
// flags: batch | fp16 << 8 | fragment order << 9.
constexpr int lstm_flags(int batch, int wdtype, int frag) { return batch | (wdtype == PIVOT_F16 ? 256 : 0) | (frag ? 512 : 0); }

__global__ void __launch_bounds__(256) lstm_cell_kernel(const float* __restrict__ z_all, const int32_t* __restrict__ invpcol,
                                                        float* __restrict__ h_all, float* __restrict__ c_all, void* __restrict__ xg_next,
                                                        float* __restrict__ z_dbg, int H, int K_pad, int flags) {
    const int batch = flags & 0xFF;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= batch * H) return;
    const int b = idx / H, j = idx - b * H;
    // the layer kernel scattered the gate pre-activations into natural order: coalesced reads here
    const float* z = z_all + (size_t)b * 4 * H;
    const float zi = z[j];
    const float zf = z[H + j];
    const float zg = z[2 * H + j];
    const float zo = z[3 * H + j];
    const int dstc = xg_next ? invpcol[j] : 0;
    const float c = sigmoidf_(zf) * c_all[idx] + sigmoidf_(zi) * tanhf(zg);
    const float h = sigmoidf_(zo) * tanhf(c);
    c_all[idx] = c;
    h_all[idx] = h;
    if (xg_next) {
        // boundary fusion (Section 4.2.1 applied to the recurrence): h_t goes straight to its
        // block-order position in the next step's input
        const int shift = (flags & 256) ? 3 : 2;
        const size_t o = (flags & 512) ? frag_index(b, dstc, batch, shift) : (size_t)b * K_pad + dstc;
        if (flags & 256) reinterpret_cast<_Float16*>(xg_next)[o] = (_Float16)h;
        else             reinterpret_cast<float*>(xg_next)[o] = h;
    }
    if (z_dbg) {
        float* zd = z_dbg + (size_t)b * 4 * H;
        zd[j] = zi; zd[H + j] = zf; zd[2 * H + j] = zg; zd[3 * H + j] = zo;
    }
}

int launch_lstm_cell(const LstmCellLaunch& L) {
    int n = L.batch * L.H;
    hipLaunchKernelGGL(lstm_cell_kernel, dim3((n + 255) / 256), dim3(256), 0, reinterpret_cast<hipStream_t>(L.stream),
                       L.z, L.invpcol, L.h, L.c, L.xg_next, L.z_dbg, L.H, L.K_pad, lstm_flags(L.batch, L.wdtype, L.frag));
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

// Block-order inputs of all steps for the launch-per-step form, in one launch: x_t and h_0 in place, zero in the
// padding columns and wherever a later h_t will land; clears the control words too.  A thread makes one 16-byte
// group of one batch row; blockIdx.y is the step.
// What bounds it: the launch and two dependent trips, the group's sources and their values.  All values are asked for
// together, of fp16 rows x and (in the first step) h for every element, whichever it needs: behind a branch per element
// they came one trip after the other (2048 units, 1024 inputs, fp16, batch 8: 5.8 -> 2.6 us).  NT: threads a workgroup.
// One wavefront, for the few groups there are, but for those that one workgroup of four covers: the launch behind it
// then waits for one XCD (a single step, us, one wavefront / four: fp32, 80 to 192 groups of all rows 6.4-6.8 / 5.8-6.2;
// fp16, 72 to 80 6.6-7.0 / 6.2-6.5, 136 to 192 7.0-7.2 / 7.0-7.5, 256 6.9 / 7.5; 512 and more, fp32 7.6-9.7 / 7.8-10.2,
// fp16 6.6-8.2 / 7.3-9.7).
template <typename WT, int NT>
__global__ void __launch_bounds__(NT) lstm_inputs_kernel(const int32_t* __restrict__ pcol_pad, const WT* __restrict__ xs,
                                                         const float* __restrict__ h0, WT* __restrict__ xg, uint32_t* __restrict__ ctl,
                                                         unsigned step_vecs, int H, int I, int K_pad, int flags) {
    using V = typename Elem<WT>::vec;
    constexpr int VEC = Elem<WT>::VEC;
    const int batch = flags & 0xFF, ngroups = K_pad / VEC;
    const int i = blockIdx.x * NT + threadIdx.x, t = blockIdx.y;
    if (t == 0)                                         // (shared out: by one workgroup alone 0.1 us)
        for (int k = i; k < (int)kLstmCtlBytes / 4; k += (ngroups * batch + NT - 1) / NT * NT) ctl[k] = 0u;
    if (i >= ngroups * batch) return;
    const bool frag = (flags & 512) != 0;
    const int g = frag ? i / batch : i % ngroups, b = frag ? i % batch : i / ngroups;
    GroupIdx<WT> gi;
    gi.load(pcol_pad, g);
    const int* src = reinterpret_cast<const int*>(gi.s4);
    // (without inputs there is no row of x to read from: any readable place will do)
    const WT* x = I > 0 ? xs + ((size_t)t * batch + b) * I : reinterpret_cast<const WT*>(h0);
    const float* h = h0 + (size_t)b * H;
    V v;
    if constexpr (sizeof(WT) == 4) {                    // one load: from x or from h
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = *(src[e] >= H ? x + (src[e] - H) : h + (src[e] >= 0 ? src[e] : 0));
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = src[e] >= (t == 0 ? 0 : H) ? v[e] : WT(0);
    } else {
        WT xv[VEC];
        float hv[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) xv[e] = x[src[e] > H ? src[e] - H : 0];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) hv[e] = 0.f;
        if (t == 0) {
            #pragma unroll
            for (int e = 0; e < VEC; ++e) hv[e] = h[src[e] >= 0 && src[e] < H ? src[e] : 0];
        }
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = src[e] >= H ? xv[e] : (src[e] >= 0 ? (WT)hv[e] : WT(0));
    }
    reinterpret_cast<V*>(xg)[(size_t)t * step_vecs + i] = v;
}

__global__ void __launch_bounds__(256) lstm_restore_kernel(const uint32_t* __restrict__ ctl, const float* __restrict__ saved, float* __restrict__ h,
                                                           float* __restrict__ c, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n || ctl[256] == 0u) return;
    h[i] = saved[i];
    c[i] = saved[n + i];
}

int launch_lstm_restore(const uint32_t* ctl, const float* saved, float* h, float* c, int n, void* stream) {
    hipLaunchKernelGGL(lstm_restore_kernel, dim3((n + 255) / 256), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), ctl, saved, h, c, n);
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

template <typename WT, int NT>
static void launch_lstm_inputs_t(const LstmInputsLaunch& L, int groups, hipStream_t st) {
    hipLaunchKernelGGL((lstm_inputs_kernel<WT, NT>), dim3((unsigned)((groups + NT - 1) / NT), L.steps), dim3(NT), 0, st, L.pcol_pad, (const WT*)L.xs, L.h0, (WT*)L.xg,
                       L.ctl, (unsigned)(L.xg_step_bytes / 16), L.H, L.I, L.K_pad, lstm_flags(L.batch, L.wdtype, L.frag));
}

int launch_lstm_inputs(const LstmInputsLaunch& L) {
    hipStream_t st = reinterpret_cast<hipStream_t>(L.stream);
    const int groups = L.K_pad * elem_size(L.wdtype) / 16 * L.batch;
    if (L.wdtype == PIVOT_F16) {
        if (groups <= 128) launch_lstm_inputs_t<_Float16, 256>(L, groups, st);
        else               launch_lstm_inputs_t<_Float16, 64>(L, groups, st);
    } else {
        if (groups <= 192) launch_lstm_inputs_t<float, 256>(L, groups, st);
        else               launch_lstm_inputs_t<float, 64>(L, groups, st);
    }
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

}  // namespace pivot
