// i8 MFMA GEMM, tile 192x128, stage buffers and workgroups per compute unit as given: all epilogue instantiations of this shape.
#include "q8_gemm_ring_kernel.h"

namespace q8 {

int launch_ring_192x128_s1(const int8_t* xq, const int8_t* wq, int M, int N, int K, int group_m, int by_xcd, const Epilogue& ep, hipStream_t st)
{
    return launch_ring<192, 128, 2, 2, 1, 3>(xq, wq, M, N, K, group_m, by_xcd, ep, st);
}

}  // namespace q8
