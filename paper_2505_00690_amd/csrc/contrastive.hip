// Contrastive losses of matched (image, text) batches and their gradients,
// FP32: logits l_ij = scale <e_i, t_j> + bias, then
//   softmax head (CLIP, Radford et al. 2021, Sec. 2.3): the mean of the
//     image->text and text->image cross-entropies with the matching pair as
//     the target,
//   sigmoid head (SigLIP, Zhai et al. 2023, Eq. 1): -(1/n) sum_ij log
//     sigmoid(z_ij l_ij), z_ij = +1 on the diagonal and -1 elsewhere.
// dL/dl (G) is formed element-wise from the logits and the row / column
// log-sum-exps; the embedding gradients are the GEMMs scale * G T and
// scale * G^T E.
#include <mutex>

#include "kernels.hpp"

namespace vl {

// The logits are walked in 64 x 64 tiles, one per workgroup (thread t: row t /
// 4, the 16 columns from 16 (t % 4)), so a matrix of n^2 logits fills the chip
// in both directions: 1024 pairs are 256 workgroups, where one workgroup per 64
// columns left 240 CUs idle (97 us for the column sums alone; parts, merge and
// gradient now take 20 us together).  Latency and launches bound them: 4 MB of
// logits are read twice.
constexpr int CT = 64;

// Maximum and sum of exponentials (relative to that maximum) of 16 values and
// the three other threads of the row.  A NaN makes the sum NaN, also where it
// is the only value in range (the maximum, which skips NaN, is -inf then).
__device__ __forceinline__ float2 lse_part(const float (&v)[16]) {
  float mx = v[0];
#pragma unroll
  for (int j = 1; j < 16; ++j) mx = fmaxf(mx, v[j]);
  mx = xor_op<1>(mx, MaxOp());
  mx = xor_op<2>(mx, MaxOp());
  float s = 0.f;
  // (no value in range, or none above -inf: 0)
#pragma unroll
  for (int j = 0; j < 16; ++j) s += mx == -INFINITY && v[j] == mx ? 0.f : expf(v[j] - mx);
  s = xor_op<1>(s, AddOp());
  s = xor_op<2>(s, AddOp());
  return make_float2(mx, s);
}

// out [cols, ld_out] = in [rows, cols]^T, zero-filled past `rows` up to
// ld_out columns: one 32 x 32 tile (tx, ty) through LDS.
__device__ __forceinline__ void transpose_tile(const float* __restrict__ in, int rows, int cols,
                                               float* __restrict__ out, int ld_out, int tx, int ty,
                                               float (*t)[33]) {
  const int r0 = ty * 32, c0 = tx * 32;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;   // 32 x 8
  for (int k = y; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + x;
    t[k][x] = (r < rows && c < cols) ? in[(size_t)r * cols + c] : 0.f;
  }
  __syncthreads();
  for (int k = y; k < 32; k += 8) {
    const int c = c0 + k, r = r0 + x;   // out row c, column r
    if (c < cols && r < ld_out) out[(size_t)c * ld_out + r] = t[x][k];
  }
}

// Workgroups below nt^2: the (max, sum) of each row and column of logit tile
// (ti, tj), rowp[tj][i] and colp[ti][j].  The others: the transposes Tt, Et
// [dim, ld] of the embeddings that the gradient GEMMs read (they do not
// depend on the logits and ride along).
__global__ __launch_bounds__(256) void k_lse_parts(const float* __restrict__ L, int n, int ld,
                                                   int nt, float2* __restrict__ rowp,
                                                   float2* __restrict__ colp,
                                                   const float* __restrict__ E,
                                                   const float* __restrict__ T, int dim,
                                                   float* __restrict__ Et,
                                                   float* __restrict__ Tt) {
  __shared__ float t[CT][CT + 1];
  const int tid = threadIdx.x, r = tid >> 2, c0 = (tid & 3) * 16;
  int b = blockIdx.x - nt * nt;
  if (b >= 0) {
    const int ntx = (dim + 31) / 32, nty = (ld + 31) / 32;
    const bool second = b >= ntx * nty;
    if (second) b -= ntx * nty;
    transpose_tile(second ? E : T, n, dim, second ? Et : Tt, ld, b % ntx, b / ntx,
                   reinterpret_cast<float(*)[33]>(&t[0][0]));
    return;
  }
  const int ti = blockIdx.x / nt, tj = blockIdx.x % nt;
  const int i = ti * CT + r, j0 = tj * CT + c0;
  float v[16];
  const float* row = L + (size_t)min(i, n - 1) * ld;
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = -INFINITY;
#pragma unroll
  for (int k = 0; k < 16; k += 4)
    if (i < n && j0 + k < n) {   // ld is a multiple of 16: whole groups are in the row
      const float4 x = *reinterpret_cast<const float4*>(row + j0 + k);
      const float xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j0 + k + e < n) v[k + e] = xs[e];
    }
#pragma unroll
  for (int k = 0; k < 16; ++k) t[r][c0 + k] = v[k];
  const float2 rp = lse_part(v);
  if (i < n && (tid & 3) == 0) rowp[(size_t)tj * n + i] = rp;
  __syncthreads();
  // the same thread layout over the transposed tile
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = t[c0 + k][r];
  const float2 cp = lse_part(v);
  const int j = tj * CT + r;
  if (j < n && (tid & 3) == 0) colp[(size_t)ti * n + j] = cp;
}

// Log-sum-exps from the tiles' parts, in a fixed order: rows (blockIdx.y = 0;
// also the diagonal logits, which the gradient kernel overwrites) and columns.
__global__ __launch_bounds__(256) void k_lse_merge(const float2* __restrict__ rowp,
                                                   const float2* __restrict__ colp, int n, int nt,
                                                   const float* __restrict__ L, int ld,
                                                   float* __restrict__ rlse,
                                                   float* __restrict__ clse,
                                                   float* __restrict__ diag) {
  __shared__ float2 sm[4][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + l;
  const float2* p = (blockIdx.y ? colp : rowp) + min(i, n - 1);
  float mx = -INFINITY, s = 0.f;
  for (int k0 = w; k0 < nt; k0 += 16) {   // wave w: parts w, w + 4, ..., four loads at once
    float2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = k0 + 4 * u < nt ? p[(size_t)(k0 + 4 * u) * n] : make_float2(-INFINITY, 0.f);
    const float m = fmaxf(mx, fmaxf(fmaxf(v[0].x, v[1].x), fmaxf(v[2].x, v[3].x)));
    if (m > -INFINITY) {
      s *= expf(mx - m);
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u].y * expf(v[u].x - m);
    } else {   // sums of 0, or NaN
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u].y;
    }
    mx = m;
  }
  sm[w][l] = make_float2(mx, s);
  __syncthreads();
  if (w != 0 || i >= n) return;
  const float m = fmaxf(fmaxf(sm[0][l].x, sm[1][l].x), fmaxf(sm[2][l].x, sm[3][l].x));
  s = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) s += sm[u][l].y * expf(sm[u][l].x - m);
  (blockIdx.y ? clse : rlse)[i] = m + logf(s);
  if (blockIdx.y == 0) diag[i] = L[(size_t)i * ld + i];
}

// G = dL/dl of logit tiles, in place over L (columns n .. ld-1 set to zero:
// they are the K padding of the gradient GEMMs) and transposed into Gt [n,
// ld] (zero-padded likewise), plus the workgroup's terms (loss, sum g (l -
// bias), sum g) in part[3 blockIdx.x ..].  A workgroup walks `per` column
// tiles of one row of tiles.
//
// Softmax head: g = ((p - d) + (q - d)) / 2n with p, q the row and column
// softmax and d the identity.  Every row of p - d and every column of q - d
// sums to zero, so sum g l is formed as sum ((p - d)(l - rlse_i) + (q - d)(l -
// clse_j)) / 2n, whose terms are smaller.
__global__ __launch_bounds__(256) void k_contrastive_grad(float* __restrict__ L, int n, int ld,
                                                          int nt, int per, int head, float bias,
                                                          const float* __restrict__ rlse,
                                                          const float* __restrict__ clse,
                                                          float* __restrict__ Gt,
                                                          float* __restrict__ part) {
  __shared__ float t[CT][CT + 1];
  __shared__ float red[4];
  const int tid = threadIdx.x, r = tid >> 2, c0 = (tid & 3) * 16;
  const int groups = (nt + per - 1) / per;
  const int ti = blockIdx.x / groups, tj0 = blockIdx.x % groups * per;
  const int i = ti * CT + r;
  const float inv_n = 1.f / (float)n;
  const float rl = i < n ? rlse[i] : 0.f;
  float sl = 0.f, sg = 0.f, s0 = 0.f;
  for (int tj = tj0; tj < min(tj0 + per, nt); ++tj) {
    if (tj > tj0) __syncthreads();   // readers of the previous tile are done
    const int j0 = tj * CT + c0;
    float* row = L + (size_t)i * ld;
#pragma unroll
    for (int k = 0; k < 16; k += 4) {
      float g[4] = {0.f, 0.f, 0.f, 0.f};
      const bool in = i < n && j0 + k < ld;
      if (in) {
        const float4 x = *reinterpret_cast<const float4*>(row + j0 + k);
        const float xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = j0 + k + e;
          if (j >= n) continue;
          const float l = xs[e];
          if (head == 0) {
            const float d = j == i ? 1.f : 0.f, cl = clse[j];
            const float p = expf(l - rl) - d, q = expf(l - cl) - d;
            g[e] = 0.5f * inv_n * (p + q);
            sg += 0.5f * inv_n * (p * (l - rl) + q * (l - cl));
          } else {
            const float z = j == i ? 1.f : -1.f;
            const float u = -z * l;                 // loss term softplus(u)
            sl += u > 0.f ? u + log1pf(expf(-u)) : log1pf(expf(u));
            g[e] = -z * inv_n / (1.f + expf(-u));   // -z sigmoid(u) / n
            sg += g[e] * (l - bias);
            s0 += g[e];
          }
        }
        *reinterpret_cast<float4*>(row + j0 + k) = make_float4(g[0], g[1], g[2], g[3]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) t[r][c0 + k + e] = g[e];
    }
    __syncthreads();
    const int j = tj * CT + r;       // row of Gt
    if (j < n) {
#pragma unroll
      for (int k = 0; k < 16; k += 4) {
        const int ic = ti * CT + c0 + k;
        if (ic < ld)
          *reinterpret_cast<float4*>(Gt + (size_t)j * ld + ic) =
              make_float4(t[c0 + k][r], t[c0 + k + 1][r], t[c0 + k + 2][r], t[c0 + k + 3][r]);
      }
    }
  }
  auto sum = [](float a, float b) { return a + b; };
  sl = block_reduce(sl, red, sum);
  sg = block_reduce(sg, red, sum);
  s0 = block_reduce(s0, red, sum);
  if (tid == 0) {
    part[3 * blockIdx.x + 0] = sl;
    part[3 * blockIdx.x + 1] = sg;
    part[3 * blockIdx.x + 2] = s0;
  }
}

// Fixed-order reduction of the workgroups' terms into loss, dL/dscale,
// dL/dbias.
__global__ __launch_bounds__(256) void k_contrastive_reduce(const float* __restrict__ part, int np,
                                                            const float* __restrict__ rlse,
                                                            const float* __restrict__ clse,
                                                            const float* __restrict__ diag, int n,
                                                            int head, float scale,
                                                            float* __restrict__ loss,
                                                            float* __restrict__ dsb) {
  __shared__ float red[4];
  float sl = 0.f, sg = 0.f, s0 = 0.f;
  if (head == 0)
    for (int i = threadIdx.x; i < n; i += 256) sl += (rlse[i] - diag[i]) + (clse[i] - diag[i]);
  for (int i = threadIdx.x; i < np; i += 256) {
    sl += part[3 * i];
    sg += part[3 * i + 1];
    s0 += part[3 * i + 2];
  }
  auto sum = [](float a, float b) { return a + b; };
  sl = block_reduce(sl, red, sum);
  sg = block_reduce(sg, red, sum);
  s0 = block_reduce(s0, red, sum);
  if (threadIdx.x == 0) {
    loss[0] = head == 0 ? 0.5f * sl / (float)n : sl / (float)n;
    dsb[0] = sg / scale;
    dsb[1] = head == 0 ? 0.f : s0;
  }
}

size_t contrastive_workspace_bytes(int n, int dim) {
  const size_t n16 = (size_t)(n + 15) / 16 * 16;
  auto a = [](size_t b) { return (b + 255) / 256 * 256; };
  return a(4 * (size_t)n * n16) * 2 + a(4 * (size_t)dim * n16) * 2 + a(4 * (size_t)n) * 3 +
         a(12 * (size_t)n);
}

hipError_t contrastive_loss(const float* E, const float* Tx, int n, int dim, int head,
                            float scale, float bias, float* loss, float* dE, float* dT,
                            float* dsb, void* ws, hipStream_t s) {
  const int n16 = (n + 15) / 16 * 16;
  auto a = [](size_t b) { return (b + 255) / 256 * 256; };
  char* w = static_cast<char*>(ws);
  float* L = reinterpret_cast<float*>(w);                 w += a(4 * (size_t)n * n16);
  float* Gt = reinterpret_cast<float*>(w);                w += a(4 * (size_t)n * n16);
  float* Tt = reinterpret_cast<float*>(w);                w += a(4 * (size_t)dim * n16);
  float* Et = reinterpret_cast<float*>(w);                w += a(4 * (size_t)dim * n16);
  float* rlse = reinterpret_cast<float*>(w);              w += a(4 * (size_t)n);
  float* clse = reinterpret_cast<float*>(w);              w += a(4 * (size_t)n);
  float* diag = reinterpret_cast<float*>(w);              w += a(4 * (size_t)n);
  float* part = reinterpret_cast<float*>(w);
  hipError_t err;
  // logits [n, n16] (the GEMM writes whole 4-column groups, so up to three
  // columns past n; every reader stops at n, and the gradient kernel zeroes
  // the padding)
  EpiArgs e;
  e.out = L; e.ldo = n16; e.alpha = scale; e.beta = bias;
  // One kernel for every n, so a pair's logit is the same chain of fused
  // multiply-adds in every batch (the heads' kernel, with eight chains, is 3 us
  // faster up to 512 pairs, 34 against 37; but other last bits of the logits,
  // some 1e-7 of the gradients here, come out of a training step's BF16
  // backward as 4e-4 of its weight gradients).
  err = gemm_f32(E, dim, Tx, dim, n, n, dim, OP_LOGITS, e, s);
  if (err != hipSuccess) return err;
  const int nt = (n + CT - 1) / CT;
  // The tiles' row and column parts wait in Gt's place (2 nt n pairs, at most a
  // quarter of it and 16 n bytes more), which the gradient kernel fills later.
  float2* rowp = reinterpret_cast<float2*>(Gt);
  float2* colp = rowp + (size_t)nt * n;
  const int64_t lse_blocks = (int64_t)nt * nt + 2 * (int64_t)((dim + 31) / 32) * ((n16 + 31) / 32);
  if (lse_blocks > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_lse_parts, dim3((unsigned)lse_blocks), dim3(256), 0, s, L, n, n16, nt, rowp,
                     colp, E, Tx, dim, Et, Tt);
  hipLaunchKernelGGL(k_lse_merge, dim3((n + 63) / 64, 2), dim3(256), 0, s, rowp, colp, n, nt, L,
                     n16, rlse, clse, diag);
  // One term triple per workgroup, n triples at most (the workspace's share):
  // one column tile per workgroup up to about 4096 pairs.
  int per = 1;
  while ((int64_t)nt * ((nt + per - 1) / per) > n) ++per;
  const int gb = nt * ((nt + per - 1) / per);
  hipLaunchKernelGGL(k_contrastive_grad, dim3(gb), dim3(256), 0, s, L, n, n16, nt, per, head, bias,
                     rlse, clse, Gt, part);
  hipLaunchKernelGGL(k_contrastive_reduce, dim3(1), dim3(256), 0, s, part, gb, rlse, clse, diag, n,
                     head, scale, loss, dsb);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  // dE = scale * G T : A = G [n, n16], B = T^T [dim, n16]
  EpiArgs ge;
  ge.out = dE; ge.ldo = dim; ge.alpha = scale; ge.beta = 0.f;
  if ((err = gemm_f32(L, n16, Tt, n16, n, dim, n16, OP_LOGITS, ge, s)) != hipSuccess) return err;
  // dT = scale * G^T E : A = G^T [n, n16], B = E^T [dim, n16]
  EpiArgs gt;
  gt.out = dT; gt.ldo = dim; gt.alpha = scale; gt.beta = 0.f;
  return gemm_f32(Gt, n16, Et, n16, n, dim, n16, OP_LOGITS, gt, s);
}

// Scratch of the allocation-free contrastive entry point: a file-scope
// device array, one copy per GPU, alive until the process ends.  Host code
// never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol); it asks the runtime for the array's device
// address once per device, with that device current, and uses that address.
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

}  // namespace vl
