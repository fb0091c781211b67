// Vector-ALU layer kernels, fp16 weights: instantiations and dispatch.
#include "pivot_gemv.h"

namespace pivot {

int launch_gemv_f16(const FcArgs& a, int bhs, int bw, int nb, int nw, int xres, dim3 grid, size_t smem, hipStream_t st) {
#define X(BH_, BW_) if (bhs == BH_ && bw == BW_) return launch_nb<_Float16, BH_, BW_>(a, nb, nw, xres, grid, smem, st);
    PIVOT_SHAPES(X)
#undef X
    set_error("no vector kernel for %dx%d row slices", bhs, bw);
    return PIVOT_E_UNSUPPORTED;
}

}  // namespace pivot
