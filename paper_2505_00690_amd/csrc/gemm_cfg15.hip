// BF16 GEMM tile configuration S3_64x128_W2x4 (64 x 128 tile, eight waves of 32x32; two workgroups share a CU),
// small-tile main loop with three K tiles in flight, instantiated for BF16 and
// e4m3 weights.  One translation unit per configuration so the build compiles
// them in parallel.
#include "gemm_kernels.hpp"

namespace vl {

hipError_t gemm_launch_cfg15(const bf16_t* A, int lda, const void* B, int ldb, bool b_fp8,
                               int M, int N, int K, int op, const EpiArgs& e, hipStream_t s) {
  if (b_fp8)
    return launch_bf16_dl<64, 128, 2, 4, true, 2, 3, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
  return launch_bf16_dl<64, 128, 2, 4, false, 2, 3, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
}

}  // namespace vl
