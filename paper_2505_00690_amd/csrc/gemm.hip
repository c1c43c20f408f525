// Dense contractions C[M,N] = A[M,K] . B[N,K]^T with fused epilogues: the
// configuration table, the tile heuristics and the launchers, plus the FP32
// kernels.
//
// BF16 path (kernels in gemm_kernels.hpp): v_mfma_f32_32x32x16_bf16 on
// gfx950.  A workgroup owns a BM x BN output tile and walks K in steps of 64
// through a ring of two or three LDS stages filled by direct-to-LDS loads
// (buffer_load ... lds, 16 bytes per lane) issued one or two K steps ahead.
// LDS rows are 64 BF16 (128 B) whose eight 16-byte chunks are permuted by
// XOR with (r ^ (r >> 3)) & 7, so the operand reads of an MFMA are free of
// bank conflicts.  Output tiles are dealt XCD by XCD.  The epilogue stages
// each 32-row slab of a wave's tile through LDS and stores rows whole.  All
// configurations accumulate K in the same order, so they agree bitwise; the
// per-configuration instantiations live in gemm_cfg*.hip / gemm_mx_cfg*.hip.
//
// FP32: the large products are in gemm_f32.hip; here a few-rows kernel for
// the heads' small products (pooled rows or embeddings against the projection
// or the texts).
#include <algorithm>

#include "gemm_kernels.hpp"

namespace vl {

// ------------------------------------------------- BF16 GEMM configurations
hipError_t gemm_launch_cfg0(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg1(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg2(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg3(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg4(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg5(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg6(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg7(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg8(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                               const EpiArgs&, hipStream_t);

hipError_t gemm_launch_cfg13(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                                const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg14(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                                const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg15(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                                const EpiArgs&, hipStream_t);
hipError_t gemm_launch_cfg16(const bf16_t*, int, const void*, int, bool, int, int, int, int,
                                const EpiArgs&, hipStream_t);

// ------------------------------------------------ MXFP8 GEMM configurations
hipError_t gemm_mx_launch_cfg9(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                               int, int, int, int, const EpiArgs&, hipStream_t);
hipError_t gemm_mx_launch_cfg10(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                                int, int, int, int, const EpiArgs&, hipStream_t);
hipError_t gemm_mx_launch_cfg11(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                                int, int, int, int, const EpiArgs&, hipStream_t);
hipError_t gemm_mx_launch_cfg12(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                                int, int, int, int, const EpiArgs&, hipStream_t);

const char* gemm_cfg_name(int cfg) {
  static const char* names[N_GEMM_CFGS] = {"DL_256x256_W2x4", "DL_256x256_W4x2", "DL_256x256_W2x2", "DL_128x128_W2x2", "DL_256x128_W2x2", "DL_128x256_W2x2", "REG_128x128_W2x2", "DL_192x256_W2x4",
                                           "DL3_160x256_W1x8", "MX_160x256_W1x8", "MX_192x256_W2x4", "MX_128x256_W2x4", "MX_128x128_W2x2",
                                           "S4_64x32_W2x1", "S4_64x64_W2x2", "S3_64x128_W2x4", "S4_128x128_W2x4"};
  return cfg >= 0 && cfg < N_GEMM_CFGS ? names[cfg] : "unknown";
}

// Estimated time of a tile configuration, from what one workgroup costs: a
// launch takes base + (K / 64) max(lat, thr n) + epi n microseconds, n the
// workgroups per CU, rounded up.  lat is a K tile's time when a CU has one
// workgroup, thr its share of a full CU, epi a tile's prologue and epilogue.
struct GemmCost {
  int cfg, bm, bn;
  double base, lat, thr, epi;
};
static double gemm_cost(const GemmCost& c, int M, int N, int K) {
  const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
  const double n = (double)((tiles + 255) / 256);
  return c.base + K / 64 * std::max(c.lat, c.thr * n) + c.epi * n;
}

int gemm_cfg_heuristic(int M, int N, int K, bool b_fp8) {
  (void)b_fp8;
  // Fitted to every configuration's time over M = 20 .. 26 000 at the block
  // shapes of widths 384, 768 and 1024 (residual of the fit 7-14 %).  Over
  // those 228 products the configuration it picks takes 0.6 % longer than the
  // fastest on average (18 % at most); estimating rounds of the 128-row and
  // larger tiles alone, as before the small tiles, took 65 % longer (577 x
  // 1024 x 4096: 45.8 us as 40 tiles of 128 x 128, 15.2 us as 160 of 64 x 64).
  static const GemmCost cands[] = {{CFG_DL_256x256_W2x4, 256, 256, 0.0, 0.30, 1.09, 10.1},
                                   {CFG_DL_192x256_W2x4, 192, 256, 0.0, 0.30, 0.938, 8.07},
                                   {CFG_DL3_160x256_W1x8, 160, 256, 0.0, 0.0, 0.812, 7.18},
                                   {CFG_S4_128x128_W2x4, 128, 128, 0.45, 0.0, 0.423, 5.0},
                                   {CFG_S3_64x128_W2x4, 64, 128, 2.76, 0.28, 0.29, 1.4},
                                   {CFG_S4_64x64_W2x2, 64, 64, 3.1, 0.168, 0.164, 0.95},
                                   {CFG_S4_64x32_W2x1, 64, 32, 3.4, 0.141, 0.115, 0.52}};
  const GemmCost* best = cands;
  for (const GemmCost& c : cands)
    if (gemm_cost(c, M, N, K) < gemm_cost(*best, M, N, K)) best = &c;
  return best->cfg;
}

hipError_t gemm_bf16(const bf16_t* A, int lda, const void* B, int ldb, bool b_fp8, int M, int N,
                     int K, int op, int cfg, const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (b_fp8 && op == OP_PATCH) return hipErrorInvalidValue;
  if (!gemm_cfg_is_bf16(cfg)) cfg = gemm_cfg_heuristic(M, N, K, b_fp8);
  // The register-staged kernel has no producer side of the LayerNorm
  // folding, reads no device row count and has no GELU-backward form; its
  // direct-to-LDS counterpart gives the same bits.
  if (cfg == CFG_REG_128x128_W2x2 && (e.u_out || e.m_dev || op == OP_DGELU))
    cfg = CFG_DL_128x128_W2x2;
  switch (cfg) {
    case 0: return gemm_launch_cfg0(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 1: return gemm_launch_cfg1(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 2: return gemm_launch_cfg2(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 3: return gemm_launch_cfg3(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 4: return gemm_launch_cfg4(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 5: return gemm_launch_cfg5(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 6: return gemm_launch_cfg6(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 7: return gemm_launch_cfg7(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 8: return gemm_launch_cfg8(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 13: return gemm_launch_cfg13(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 14: return gemm_launch_cfg14(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 15: return gemm_launch_cfg15(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
    case 16: return gemm_launch_cfg16(A, lda, B, ldb, b_fp8, M, N, K, op, e, s);
  }
  return hipErrorInvalidValue;
}

int gemm_mx_cfg_heuristic(int M, int N, int K) {
  (void)K;
  // Same model as the BF16 heuristic, with the relative tile efficiencies
  // measured for the MXFP8 kernel on gfx950.
  struct C { int cfg, bm, bn; double eff; };
  static const C cands[] = {{CFG_MX_192x256_W2x4, 192, 256, 1.0},
                            {CFG_MX_160x256_W1x8, 160, 256, 0.95},
                            {CFG_MX_128x256_W2x4, 128, 256, 0.85},
                            {CFG_MX_128x128_W2x2, 128, 128, 0.6}};
  int best = CFG_MX_128x128_W2x2;
  double best_t = 1e300;
  for (const C& c : cands) {
    const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    const double t = (double)((tiles + 255) / 256) * (c.bm * c.bn) / (65536.0 * c.eff);
    if (t < best_t) { best_t = t; best = c.cfg; }
  }
  return best;
}

hipError_t gemm_mx(const uint8_t* A, const uint8_t* SA, const uint8_t* B, const uint8_t* SB,
                   int M, int N, int K, int op, int cfg, const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (K % 128 || N % 32) return hipErrorInvalidValue;
  if (!gemm_cfg_is_mx(cfg)) cfg = gemm_mx_cfg_heuristic(M, N, K);
  switch (cfg) {
    case CFG_MX_160x256_W1x8: return gemm_mx_launch_cfg9(A, SA, B, SB, M, N, K, op, e, s);
    case CFG_MX_192x256_W2x4: return gemm_mx_launch_cfg10(A, SA, B, SB, M, N, K, op, e, s);
    case CFG_MX_128x256_W2x4: return gemm_mx_launch_cfg11(A, SA, B, SB, M, N, K, op, e, s);
    case CFG_MX_128x128_W2x2: return gemm_mx_launch_cfg12(A, SA, B, SB, M, N, K, op, e, s);
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------ FP32 GEMM with few A rows
// The small products of the heads (logits of a few images against many
// texts, projections of pooled rows): A has few rows and B is the large
// operand, so 64x64 tiles leave most CUs idle.  A workgroup owns 8 rows of A
// (staged in LDS in K chunks) and 32 columns; thread (kq, column) sums its
// column's products with the 8 rows over the float4 chunks kq, kq + 8, kq +
// 16, ... of K, and the 8 partial sums of an output are added in kq order.
// Every output is computed the same way whatever M is, so a row's result does
// not depend on the other rows of the batch.
constexpr int FR_M = 8, FR_N = 32, FR_KQ = 8, FR_KC = 512;

template <int OP>
__global__ __launch_bounds__(256) void k_gemm_f32_rows(const float* __restrict__ A, int lda,
                                                       const float* __restrict__ B, int ldb,
                                                       int M, int N, int K, EpiArgs e) {
  constexpr int EPI = OpEpi<OP>::kind;
  __shared__ float4 sA[FR_M][FR_KC / 4];
  __shared__ float sP[FR_KQ][FR_M][FR_N + 1];
  const int tid = threadIdx.x;
  const int nl = tid & (FR_N - 1), kq = tid >> 5;
  const int nbn = (N + FR_N - 1) / FR_N;      // one-dimensional grid: no limit on M
  const int m0 = (int)(blockIdx.x / nbn) * FR_M, n0 = (int)(blockIdx.x % nbn) * FR_N;
  const float* brow = B + (size_t)min(n0 + nl, N - 1) * ldb;
  float acc[FR_M];
#pragma unroll
  for (int r = 0; r < FR_M; ++r) acc[r] = 0.f;
  constexpr int NB = FR_KC / 4 / FR_KQ;   // B chunks per thread and K chunk
  for (int k0 = 0; k0 < K; k0 += FR_KC) {
    const int nc = min(FR_KC, K - k0) / 4;   // float4 chunks in this K chunk
    // All of this thread's B loads of the K chunk are issued first, so their
    // latencies overlap one another and the A staging.
    float4 b[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = kq + FR_KQ * i;
      b[i] = c < nc ? *reinterpret_cast<const float4*>(brow + k0 + 4 * c)
                    : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();                          // readers of the previous chunk are done
    for (int i = tid; i < FR_M * nc; i += 256) {
      const int r = i / nc, c = i - r * nc;
      sA[r][c] = *reinterpret_cast<const float4*>(A + (size_t)min(m0 + r, M - 1) * lda + k0 + 4 * c);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = kq + FR_KQ * i;
      if (c >= nc) break;
#pragma unroll
      for (int r = 0; r < FR_M; ++r) {
        const float4 a = sA[r][c];
        acc[r] = fmaf(a.x, b[i].x, acc[r]);
        acc[r] = fmaf(a.y, b[i].y, acc[r]);
        acc[r] = fmaf(a.z, b[i].z, acc[r]);
        acc[r] = fmaf(a.w, b[i].w, acc[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < FR_M; ++r) sP[kq][r][nl] = acc[r];
  __syncthreads();
  if (tid >= FR_M * FR_N / 4) return;
  const int r = tid / (FR_N / 4), nq = (tid % (FR_N / 4)) * 4;
  const int m = m0 + r, n = n0 + nq;
  if (m >= M || n >= N) return;
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float t = sP[0][r][nq + j];
#pragma unroll
    for (int q = 1; q < FR_KQ; ++q) t += sP[q][r][nq + j];
    v[j] = t;
  }
  epi_store4<EPI, false>(e, m, n, v[0], v[1], v[2], v[3]);
}

hipError_t gemm_f32_rows(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                         int op, const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const int64_t blocks = (int64_t)((N + FR_N - 1) / FR_N) * ((M + FR_M - 1) / FR_M);
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  dim3 grid((unsigned)blocks), block(256);
#define VL_GEMM_CASE(OP)                                                                   \
  case OP:                                                                                 \
    hipLaunchKernelGGL(k_gemm_f32_rows<OP>, grid, block, 0, s, A, lda, B, ldb, M, N, K, e); \
    break;
  switch (op) {
    VL_GEMM_CASE(OP_QKV)
    VL_GEMM_CASE(OP_OPROJ)
    VL_GEMM_CASE(OP_FC1)
    VL_GEMM_CASE(OP_FC2)
    VL_GEMM_CASE(OP_LOGITS)
    default: return hipErrorInvalidValue;
  }
#undef VL_GEMM_CASE
  return hipGetLastError();
}

}  // namespace vl
