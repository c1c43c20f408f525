// MXFP8 GEMM tile configuration MX_64x64_W2x2 (64 x 64 tile, 2 x 2 waves,
// three K tiles in the ring, two workgroups per CU).
// One translation unit per configuration so the build compiles them in
// parallel.
#include "gemm_mx.hpp"

namespace vl {

hipError_t gemm_mx_launch_cfg18(const uint8_t* A, const uint8_t* SA, const uint8_t* B,
                               const uint8_t* SB, int M, int N, int K, int op, const EpiArgs& e,
                               hipStream_t s) {
  return launch_mx<64, 64, 2, 2, 3>(A, SA, B, SB, M, N, K, op, e, s);
}

}  // namespace vl
