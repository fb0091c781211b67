// Batched matrix-core layer kernel, fp32 weights, slices of 32 rows: instantiations.
#include "pivot_frag.h"

namespace pivot {

int launch_frag_f32_32(const FcArgs& a, int bw, int nbt, int nw, dim3 grid, hipStream_t st) {
    return launch_frag_w<float, 32>(a, bw, nbt, nw, grid, st);
}

}  // namespace pivot
