// Matrix-core layer kernel whose B fragments are gathered from a copy of x in LDS (fp16 weights, batch 5..64):
// instantiations and dispatch.
#include "pivot_fc_kernels.h"

namespace pivot {

template <int KIND, int BH, int BW, int XV, bool CHAIN>
static int launch_c(const FcArgs& a, dim3 grid, size_t smem, hipStream_t st) {
    // more than 64 KB of dynamic LDS per workgroup has to be allowed per kernel and device
    static size_t allowed[16] = {};
    const auto kernel = CHAIN ? fc_mfma_xrow_chain_kernel<KIND, BH, BW, XV> : fc_mfma_xrow_kernel<KIND, BH, BW, XV>;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    size_t& have = allowed[dev & 15];
    if (smem > 64 * 1024 && smem > have) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        have = smem;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(8 * 64), smem, st, PIVOT_GEMV_ARGS(a), fc_tail(a));
    HIP_TRY(hipGetLastError());
    return PIVOT_OK;
}

template <int KIND, int BH, int BW>
static int launch_t(const FcArgs& a, dim3 grid, size_t smem, hipStream_t st) {
    const bool short_rows = xrow_xv(a.xn_vecs) == 4;
    if (a.out_form & kOutFrag) return short_rows ? launch_c<KIND, BH, BW, 4, true>(a, grid, smem, st) : launch_c<KIND, BH, BW, 8, true>(a, grid, smem, st);
    return short_rows ? launch_c<KIND, BH, BW, 4, false>(a, grid, smem, st) : launch_c<KIND, BH, BW, 8, false>(a, grid, smem, st);
}

int launch_mfma_xrow_f16(const FcArgs& a, int kind, int bhs, int bw, dim3 grid, size_t smem, hipStream_t st) {
#define X(BH_, BW_)                                                                                        \
    if (bhs == BH_ && bw == BW_) {                                                                         \
        if constexpr (BW_ % 32 == 0 && BH_ % 16 == 0) { if (kind == 0) return launch_t<0, BH_, BW_>(a, grid, smem, st); } \
        if constexpr (BH_ % 32 == 0 && BW_ == 16)     { if (kind == 1) return launch_t<1, BH_, BW_>(a, grid, smem, st); } \
        if constexpr (BH_ == 16 && BW_ == 16)          { if (kind == 2) return launch_t<2, BH_, BW_>(a, grid, smem, st); } \
    }
    PIVOT_SHAPES(X)
#undef X
    set_error("no matrix-core kernel (kind %d) for %dx%d row slices", kind, bhs, bw);
    return PIVOT_E_UNSUPPORTED;
}

}  // namespace pivot
