// i8 MFMA GEMM, tile 64x64 with 4 waves and a deep ring: all epilogue instantiations of this shape.
#include "q8_gemm_kernel.h"

namespace q8 {

int launch_tile_64x64_w4(const int8_t* xq, const int8_t* wq, int M, int N, int K, int group_m, const Epilogue& ep,
                       hipStream_t st)
{
    return launch_tile<64, 64, 2, 2, 5>(xq, wq, M, N, K, group_m, ep, st);
}

}  // namespace q8
