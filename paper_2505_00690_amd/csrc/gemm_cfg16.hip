// BF16 GEMM tile configuration S4_128x128_W2x4 (128 x 128 tile, eight waves of 64x32),
// small-tile main loop with four K tiles in flight, instantiated for BF16 and
// e4m3 weights.  One translation unit per configuration so the build compiles
// them in parallel.
#include "gemm_kernels.hpp"

namespace vl {

hipError_t gemm_launch_cfg16(const bf16_t* A, int lda, const void* B, int ldb, bool b_fp8,
                               int M, int N, int K, int op, const EpiArgs& e, hipStream_t s) {
  if (b_fp8)
    return launch_bf16_dl<128, 128, 2, 4, true, 2, 4, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
  return launch_bf16_dl<128, 128, 2, 4, false, 2, 4, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
}

}  // namespace vl
