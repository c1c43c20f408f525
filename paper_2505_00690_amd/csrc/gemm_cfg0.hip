// BF16 GEMM tile configuration DL_256x256_W2x4 (256 x 256 tile, 8 waves, 128x64 outputs per wave;
// phased main loop where K is long), instantiated for BF16 and e4m3 weights.  One translation unit per
// configuration so the build compiles them in parallel.
#include "gemm_kernels.hpp"

namespace vl {

hipError_t gemm_launch_cfg0(const bf16_t* A, int lda, const void* B, int ldb, bool b_fp8,
                               int M, int N, int K, int op, const EpiArgs& e, hipStream_t s) {
  if (b_fp8)
    return launch_bf16_dl<256, 256, 2, 4, true, 2, 2, LOOP_PHASED>(A, lda, B, ldb, M, N, K, op, e, s);
  return launch_bf16_dl<256, 256, 2, 4, false, 2, 2, LOOP_PHASED>(A, lda, B, ldb, M, N, K, op, e, s);
}

}  // namespace vl
