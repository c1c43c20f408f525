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
hipError_t gemm_mx_launch_cfg17(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                                int, int, int, int, const EpiArgs&, hipStream_t);
hipError_t gemm_mx_launch_cfg18(const uint8_t*, const uint8_t*, const uint8_t*, const uint8_t*,
                                int, int, int, int, const EpiArgs&, hipStream_t);

const char* gemm_cfg_name(int cfg) {
  static const char* names[N_GEMM_CFGS] = {"DL_256x256_W2x4", "DL_256x256_W4x2", "DL_256x256_W2x2", "DL_128x128_W2x2", "DL_256x128_W2x2", "DL_128x256_W2x2", "REG_128x128_W2x2", "DL_192x256_W2x4",
                                           "DL3_160x256_W1x8", "MX_160x256_W1x8", "MX_192x256_W2x4", "MX_128x256_W2x4", "MX_128x128_W2x4",
                                           "S4_64x32_W2x1", "S4_64x64_W2x2", "S3_64x128_W2x4", "S4_128x128_W2x4", "MX_64x128_W2x4", "MX_64x64_W2x2"};
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

// The same for MXFP8, by rounds: a full round of `wgs` workgroups per CU takes
// f + (K / 128) c microseconds, a last one of at most 256 workgroups f1 + (K /
// 128) c1 (for one workgroup per CU the two are the same).
int gemm_mx_cfg_heuristic(int M, int N, int K) {
  struct C { int cfg, bm, bn, wgs; double f, c, f1, c1; };
  // From every configuration's time at M = 65 .. 18 464 and the block shapes
  // of width 1024.  Rounds of the tiles of 128 rows and more alone, as before
  // the two small ones and the deeper rings, took up to twice as long (257 x
  // 1024 x 4096: 27.2 us as 24 tiles of 128 x 128 with two stages, 13.2 us as
  // 80 of 64 x 64; 577 x 3072 x 1024: 10.9, 7.0 as 240 of 64 x 128; 4616 x
  // 1024 x 4096: 38.6 with two stages of 128 x 256, 33.3 with three).
  static const C cands[] = {{CFG_MX_192x256_W2x4, 192, 256, 1, 7.3, 1.2, 7.3, 1.2},
                            {CFG_MX_160x256_W1x8, 160, 256, 1, 7.0, 1.15, 7.0, 1.15},
                            {CFG_MX_128x256_W2x4, 128, 256, 1, 6.9, 0.78, 6.9, 0.78},
                            {CFG_MX_128x128_W2x4, 128, 128, 1, 5.0, 0.54, 5.0, 0.54},
                            {CFG_MX_64x128_W2x4, 64, 128, 2, 5.2, 0.57, 3.6, 0.367},
                            {CFG_MX_64x64_W2x2, 64, 64, 2, 4.3, 0.39, 3.2, 0.31}};
  int best = -1;
  double best_t = 1e300;
  for (const C& c : cands) {
    const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    const long round = 256L * c.wgs, last = tiles % round, kt = K / 128;
    const double full = c.f + kt * c.c;
    const double t = tiles / round * full +
                     (last == 0 ? 0.0 : last <= 256 ? c.f1 + kt * c.c1 : full);
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
    case CFG_MX_128x128_W2x4: return gemm_mx_launch_cfg12(A, SA, B, SB, M, N, K, op, e, s);
    case CFG_MX_64x128_W2x4: return gemm_mx_launch_cfg17(A, SA, B, SB, M, N, K, op, e, s);
    case CFG_MX_64x64_W2x2: return gemm_mx_launch_cfg18(A, SA, B, SB, M, N, K, op, e, s);
  }
  return hipErrorInvalidValue;
}

// --------------------------------------------- FP32 GEMM of the heads' products
// The products of the heads (projections of pooled rows, logits of images
// against texts): one to a few thousand A rows, K of a few hundred.  A
// workgroup owns 16 RT x 16 RT outputs on v_mfma_f32_16x16x4_f32, whose result
// is the chain of its four products in k order.  Chain q of an output takes
// the float4 chunks q, q + 8, q + 16, ... of K, the 8 chains are added in q
// order, and wave w holds chains w and w + 4.  An output is computed the same
// way whatever M, N and RT are, so a row's result does not depend on the
// other rows of the batch.  256 K values of the tile's rows are one stage of
// LDS, streamed by direct-to-LDS loads of a whole 1 KB row each, NS stages in
// flight.  RT = 2 with two stages, and RT = 1 with four, take 133 KB: a
// workgroup to a CU.  RT = 1 with two lets two share it.  (Operands loaded
// straight into registers need 16-byte pieces of 16 rows per instruction:
// scores of 1000 x 1000 over K = 512 took 39 us against 26; the vector-ALU
// kernel before this one, with the same sums, 58 us.)
constexpr int FR_KC = 256;                    // K values per stage
constexpr int FR_LD = FR_KC + 4;              // LDS row: rows 4 banks apart
template <int OP, int RT, int NS>
__global__ __launch_bounds__(256) void k_gemm_f32_rows(const float* __restrict__ A, int lda,
                                                       const float* __restrict__ B, int ldb,
                                                       int M, int N, int K, EpiArgs e) {
  constexpr int EPI = OpEpi<OP>::kind;
  constexpr int T = 16 * RT;                  // tile side
  constexpr int LPW = T / 2;                  // rows (loads) per wave and stage
  static_assert(NS >= 2 && NS <= 4, "stages");
  __shared__ __attribute__((aligned(16))) float smem[NS * 2 * T * FR_LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nbn = (N + T - 1) / T;            // one-dimensional grid: no limit on M
  const int m0 = (int)(blockIdx.x / nbn) * T, n0 = (int)(blockIdx.x % nbn) * T;
  // Rows past M or N repeat the last one; K values past K read as zero (past
  // the row's buffer).
  const float* A0 = A + (size_t)m0 * lda;
  const float* B0 = B + (size_t)n0 * ldb;
  const int ma = min(T, M - m0) - 1, nb = min(T, N - n0) - 1;
  const uint32_t lds0 = lds_offset(smem);
  auto issue = [&](int st, int ch) {
    const int v = (FR_KC * ch + 4 * lane) * 4;
#pragma unroll
    for (int j = 0; j < LPW / 2; ++j) {
      const int row = wave + 4 * j;
      const uint32_t lo = lds0 + (st * 2 * T + row) * FR_LD * 4;
      dma16(buffer_rsrc(A0 + (size_t)min(row, ma) * lda, (uint64_t)K * 4), lo, v, 0);
      dma16(buffer_rsrc(B0 + (size_t)min(row, nb) * ldb, (uint64_t)K * 4), lo + T * FR_LD * 4, v,
            0);
    }
  };
  f32x4 acc[2][RT][RT];                       // chains w, w + 4
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < RT; ++c) acc[h][r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nch = (K + FR_KC - 1) / FR_KC;
  for (int i = 0; i < NS && i < nch; ++i) issue(i, i);
  const int i = lane & 15, k = lane >> 4;
  int st = 0;
  for (int ch = 0; ch < nch; ++ch) {
    switch (min(NS - 1, nch - 1 - ch)) {      // stages still on their way
      case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LPW) : "memory"); break;
      case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPW) : "memory"); break;
      case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW) : "memory"); break;
      default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    lds_barrier();
    // Lane (i, k): component k of chunk wave + 4 x of row i.
    const float* sa = smem + (st * 2 * T + i) * FR_LD + 4 * wave + k;
    const float* sb = sa + T * FR_LD;
#pragma unroll
    for (int x = 0; x < FR_KC / 16; ++x) {
      float a[RT], b[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        a[r] = sa[r * 16 * FR_LD + 16 * x];
        b[r] = sb[r * 16 * FR_LD + 16 * x];
      }
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < RT; ++c)
          acc[x & 1][r][c] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[c], acc[x & 1][r][c], 0, 0, 0);
    }
    if (ch + NS < nch) {
      lds_barrier();                          // every wave has read the stage
      issue(st, ch + NS);
    }
    st = st + 1 == NS ? 0 : st + 1;
  }
  lds_barrier();
  // C layout: lane (column i, k), register q: row 4 k + q.
  float (*sP)[T][T + 1] = reinterpret_cast<float(*)[T][T + 1]>(smem);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < RT; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          sP[wave + 4 * h][16 * r + 4 * k + q][16 * c + i] = acc[h][r][c][q];
  __syncthreads();
  if (tid >= T * T / 4) return;
  const int r = tid / (T / 4), nq = (tid % (T / 4)) * 4;
  const int m = m0 + r, n = n0 + nq;
  if (m >= M || n >= N) return;
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float t = sP[0][r][nq + j];
#pragma unroll
    for (int q = 1; q < 8; ++q) t += sP[q][r][nq + j];
    v[j] = t;
  }
  epi_store4<EPI, false>(e, m, n, v[0], v[1], v[2], v[3]);
}

hipError_t gemm_f32_rows(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                         int op, const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  // 16 x 16 tiles as long as they are one round.  Beyond that 32 x 32 tiles,
  // which read each operand half as often; but up to 16 rows half of such a
  // tile is padding, and small tiles, two workgroups to a CU, are faster (1 x
  // 20 000 over K = 512: 14.9 us in 32 x 32 tiles, 13.5 in 16 x 16 with four
  // stages, 9.7 so, the copy rate; 11.3 on the vector ALU.  16 x 8000: 5.6, 5.7,
  // 4.2; 24 x 8000: 5.7 in 32 x 32, 7.1 in 16 x 16).
  auto tiles = [&](int t) { return (int64_t)((N + t - 1) / t) * ((M + t - 1) / t); };
  const bool one_round = tiles(16) <= 256, small = one_round || M <= 16;
  const int64_t blocks = tiles(small ? 16 : 32);
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  dim3 grid((unsigned)blocks), block(256);
  auto launch = [&](auto k) {
    hipLaunchKernelGGL(k, grid, block, 0, s, A, lda, B, ldb, M, N, K, e);
  };
#define VL_GEMM_CASE(OP)                              \
  case OP:                                            \
    if (one_round) launch(k_gemm_f32_rows<OP, 1, 4>); \
    else if (small) launch(k_gemm_f32_rows<OP, 1, 2>); \
    else launch(k_gemm_f32_rows<OP, 2, 2>);           \
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
