// Batched matrix-core layer kernel, fp16 weights, slices of 16 rows: instantiations.
#include "pivot_frag.h"

namespace pivot {

int launch_frag_f16_16(const FcArgs& a, int bw, int nbt, int nw, dim3 grid, hipStream_t st) {
    return launch_frag_w<_Float16, 16>(a, bw, nbt, nw, grid, st);
}

}  // namespace pivot
