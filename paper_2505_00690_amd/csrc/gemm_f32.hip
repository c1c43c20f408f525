// FP32 contraction C[M,N] = A[M,K] . B[N,K]^T with the fused epilogues, on the
// FP32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// That instruction adds its four products one after the other, each as a
// fused multiply-add in FP32 (checked against an fmaf chain on the hardware,
// subnormal products included), so a chain of them over ascending K gives
// exactly the bits of an fmaf loop over k, whatever the tile: the result does
// not depend on the batch size.  The matrix cores do 256 FLOP per clock and
// CU in FP32, twice what unpacked FMAs reach.
#include "gemm_kernels.hpp"

namespace vl {

constexpr int F32_BK = 32;   // K values per LDS tile: rows of 128 bytes, as the BF16 tiles

// One workgroup owns 16 TM rows of A and 64 columns: four waves side by side,
// 16 TM x 16 outputs each.  MFMA-bound (32 cycles per instruction against one
// or two 4-byte LDS reads), so the tile is chosen by how its count fills 256
// CUs; a ring of F32_ST K tiles arrives by direct-to-LDS loads, and the
// fragments of a whole K tile are read one tile ahead of their MFMAs.  Lane
// (l16, q) holds row l16, k = 4s + q of step s; B rows are the MFMA's first
// operand, so a lane ends with four consecutive columns of one row of C.
// Measured (MI355X; a 64 x 64 tile of FMAs before): 1576 x 768 x 3072 186 -> 86
// us (87 TFLOP/s), 1576 x 3072 x 768 114 -> 85 us, 1024 x 768 x 1024 58 -> 25 us;
// the matrix pipe is busy 60-70 % of the time.
// K tiles in the ring: as many as let two workgroups share a CU's LDS.
constexpr int f32_stages(int tm) {
  const int st = 80 * 1024 / ((16 * tm + 64) * 128);
  return st > 6 ? 6 : st;
}

template <int TM, int OP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 4))) void k_gemm_f32(
    const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb, int M, int N,
    int K, int gm, int gn, EpiArgs e) {
  constexpr int EPI = OpEpi<OP>::kind;
  constexpr int BM = 16 * TM, BN = 64;
  constexpr int F32_ST = f32_stages(TM);
  constexpr int GA = BM / 8, IA = (GA + 3) / 4;   // 8-row load groups of A; per wave
  __shared__ __attribute__((aligned(1024))) char sA[F32_ST][BM * 128];
  __shared__ __attribute__((aligned(1024))) char sB[F32_ST][BN * 128];
  int tm_, tn_;
  xcd_tile(gm, gn, 8, &tm_, &tn_);
  const int m0 = tm_ * BM, n0 = tn_ * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const i32x4 ra = buffer_rsrc(A + (size_t)m0 * lda, (uint64_t)min(M - m0, BM) * lda * 4);
  const i32x4 rb = buffer_rsrc(B + (size_t)n0 * ldb, (uint64_t)min(N - n0, BN) * ldb * 4);
  // Chunk s of tile row r sits at s ^ ((r >> 1) & 7): 16 rows read at one
  // chunk hit all 64 banks, and rows 16 apart are permuted alike, so the
  // reads of a step differ by immediates (two to an instruction).
  const int lrow = lane >> 3;
  const uint32_t ldsA = lds_offset(&sA[0][0]), ldsB = lds_offset(&sB[0][0]);
  // All of a wave's row groups have its parity, hence one chunk pattern.  (A
  // last K tile of 16 columns also fetches what follows them, up to the
  // buffer's end: never read.)
  const int chunk = (((lane & 7) ^ (lane >> 4)) ^ ((wave & 1) << 2)) << 4;
  const int av = lrow * lda * 4 + chunk, bv = lrow * ldb * 4 + chunk;
  const bool all_a = GA % 4 == 0 || wave < GA % 4;   // else one load fewer
  auto issue = [&](int buf, int kt) {
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int grp = wave + 4 * i;
      if (i + 1 < IA || all_a)
        dma16_rows(ra, ldsA + buf * BM * 128 + grp * 1024, av, grp * 8 * lda * 4, kt * 128);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int grp = wave + 4 * i;
      dma16_rows(rb, ldsB + buf * BN * 128 + grp * 1024, bv, grp * 8 * ldb * 4, kt * 128);
    }
  };
  // All but the youngest F32_ST - 2 tiles' loads have landed.
  auto wait_steady = [&]() {
    if (all_a) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((F32_ST - 2) * (IA + 2)) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((F32_ST - 2) * (IA + 1)) : "memory");
  };
  f32x4 acc[TM];
#pragma unroll
  for (int b = 0; b < TM; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int l16 = lane & 15, q = lane >> 4;
  const int pA = l16 * 128 + ((l16 >> 1) << 4) + 4 * q;
  const int pB = pA + 16 * wave * 128;
  auto ldfrag = [&](float (&fa)[8][TM], float (&fb)[8], int buf) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      fb[s] = *reinterpret_cast<const float*>(sB[buf] + (pB ^ (s << 4)));
#pragma unroll
      for (int b = 0; b < TM; ++b)
        fa[s][b] = *reinterpret_cast<const float*>(sA[buf] + (pA ^ (s << 4)) + b * 2048);
    }
  };
  const int KT = (K + F32_BK - 1) / F32_BK;
  float fa[2][8][TM], fb[2][8];
  for (int i = 0; i < F32_ST && i < KT; ++i) issue(i, i);
  if (KT >= F32_ST - 1) wait_steady();   // tile 0 (and 1)
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
  ldfrag(fa[0], fb[0], 0);
  int cur = 0;
  auto mma = [&](auto buf, int s) {
    constexpr int f = decltype(buf)::value;
#pragma unroll
    for (int b = 0; b < TM; ++b)
      acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[f][s], fa[f][s][b], acc[b], 0, 0, 0);
  };
  auto step = [&](auto buf, int kt) {
    constexpr int f = decltype(buf)::value;
    const int nxt = cur + 1 == F32_ST ? 0 : cur + 1;
    // Tile kt + 1 must have landed; at the barrier every wave has tile kt in
    // registers, so its stage takes tile kt + F32_ST.
    if (kt + F32_ST <= KT) wait_steady();
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (kt + F32_ST < KT) issue(cur, kt + F32_ST);
    ldfrag(fa[f ^ 1], fb[f ^ 1], nxt);
#pragma unroll
    for (int s = 0; s < 8; ++s) mma(buf, s);
    // The next tile's reads (R instructions) ride between these MFMAs: the
    // matrix pipe would drain while a run of reads issues, and issued all at
    // once they exceed the LDS counter's range, so the MFMAs would wait for
    // them.
    constexpr int R = 8 * ((TM + 1) / 2 + 1), MM = 8 * TM;
    constexpr int PER = (R + MM - 1) / MM, NG = (R + PER - 1) / PER;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);
    }
    if (MM > NG) __builtin_amdgcn_sched_group_barrier(0x008, MM - NG, 0);
    cur = nxt;
  };
  const int full = K / F32_BK;
  int kt = 0;
  for (; kt + 1 < full; kt += 2) {
    step(std::integral_constant<int, 0>(), kt);
    step(std::integral_constant<int, 1>(), kt + 1);
  }
  // The odd tile, and a last one of 16 columns (its fragments are read).
  if (kt < full) {
    step(std::integral_constant<int, 0>(), kt);
    if (K & 16)
#pragma unroll
      for (int s = 0; s < 4; ++s) mma(std::integral_constant<int, 1>(), s);
  } else if (K & 16) {
#pragma unroll
    for (int s = 0; s < 4; ++s) mma(std::integral_constant<int, 0>(), s);
  }
  const int n = n0 + 16 * wave + 4 * q;
  if (n >= N) return;
#pragma unroll
  for (int b = 0; b < TM; ++b) {
    const int m = m0 + 16 * b + l16;
    if (m < M) epi_store4<EPI, false>(e, m, n, acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
  }
}

template <int TM>
static hipError_t launch_f32(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                             int op, const EpiArgs& e, hipStream_t s) {
  const int gm = (M + 16 * TM - 1) / (16 * TM), gn = (N + 63) / 64;
  dim3 grid(gm * gn), block(256);
#define VL_GEMM_CASE(OP)                                                                      \
  case OP:                                                                                    \
    hipLaunchKernelGGL((k_gemm_f32<TM, OP>), grid, block, 0, s, A, lda, B, ldb, M, N, K, gm,  \
                       gn, e);                                                                \
    break;
  switch (op) {
    VL_GEMM_CASE(OP_PATCH)
    VL_GEMM_CASE(OP_QKV)
    VL_GEMM_CASE(OP_OPROJ)
    VL_GEMM_CASE(OP_FC1)
    VL_GEMM_CASE(OP_FC2)
    VL_GEMM_CASE(OP_LOGITS)
    VL_GEMM_CASE(OP_FC1_PRE)
    default: return hipErrorInvalidValue;
  }
#undef VL_GEMM_CASE
  return hipGetLastError();
}

hipError_t gemm_f32(const float* A, int lda, const float* B, int ldb, int M, int N, int K,
                    int op, const EpiArgs& e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (K % 16) return hipErrorInvalidValue;
  // The matrix cores are the bound, and the workgroups of a CU share them: a
  // launch takes the fullest CU's rows, ceil(tiles / 256) x TM, plus about
  // half a row block per workgroup for its loads and epilogue.
  static const int tms[] = {8, 6, 5, 4, 3, 2, 1};
  int best = 8;
  double best_t = 1e300;
  for (int tm : tms) {
    const long tiles = (long)((M + 16 * tm - 1) / (16 * tm)) * ((N + 63) / 64);
    const double t = (double)((tiles + 255) / 256) * (tm + 0.5);
    if (t < best_t) { best_t = t; best = tm; }
  }
  switch (best) {
    case 8: return launch_f32<8>(A, lda, B, ldb, M, N, K, op, e, s);
    case 6: return launch_f32<6>(A, lda, B, ldb, M, N, K, op, e, s);
    case 5: return launch_f32<5>(A, lda, B, ldb, M, N, K, op, e, s);
    case 4: return launch_f32<4>(A, lda, B, ldb, M, N, K, op, e, s);
    case 3: return launch_f32<3>(A, lda, B, ldb, M, N, K, op, e, s);
    case 2: return launch_f32<2>(A, lda, B, ldb, M, N, K, op, e, s);
    default: return launch_f32<1>(A, lda, B, ldb, M, N, K, op, e, s);
  }
}

}  // namespace vl
