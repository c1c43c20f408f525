// BF16 GEMM tile configuration S4_64x32_W2x1 (64 x 32 tile, two waves of 32x32; three workgroups share a CU.  For
// products of a few hundred tiles or fewer, where the time is the chain of
// K steps of one tile),
// small-tile main loop with four K tiles in flight, instantiated for BF16 and
// e4m3 weights.  One translation unit per configuration so the build compiles
// them in parallel.
#include "gemm_kernels.hpp"

namespace vl {

hipError_t gemm_launch_cfg13(const bf16_t* A, int lda, const void* B, int ldb, bool b_fp8,
                               int M, int N, int K, int op, const EpiArgs& e, hipStream_t s) {
  if (b_fp8)
    return launch_bf16_dl<64, 32, 2, 1, true, 2, 4, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
  return launch_bf16_dl<64, 32, 2, 1, false, 2, 4, LOOP_SMALL>(A, lda, B, ldb, M, N, K, op, e, s);
}

}  // namespace vl
