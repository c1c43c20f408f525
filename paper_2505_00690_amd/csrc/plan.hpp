// Host-side planning of an encode call: how a packed batch of images (or
// token sequences) is cut into parts, which attention work items and
// descriptors the kernels read, and where every activation buffer sits in
// the caller's workspace.  Plain C++ (no device code or HIP calls), so it
// also builds on its own for host-only checks.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "batch.hpp"

namespace vl {

constexpr size_t kAlign = 256;     // workspace and region alignment
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

constexpr int kMaxTokens = 1025;   // 32 x 32 patches + class token
constexpr int kAttnQ = 128;        // queries per attention work item
constexpr int kResMinTokens = 128; // K/V-resident attention: more tokens than one work item
constexpr int kResMaxTiles = 10;   //   and at most 10 key tiles of 64 (the 160 KB of LDS)
constexpr int kMaxItems = 65535;   // images / texts per call (grid y of the gather kernels)
constexpr int64_t kSplitMinTokens = 4096;  // two-part batches from this many tokens
constexpr int64_t kMaxBatchTokens = int64_t(1) << 24;

// The streamed attention work items (blocks of `step` rows) of the n sequences
// seq[] (indices into imgs), most key tiles first, so that the last workgroups
// to start are short ones.  The kernel gives each XCD a contiguous range of
// the (head, item) pairs; where `heads` is no multiple of the 8 XCDs these cut
// a head's items, so the order is then dealt round-robin into runs of equal
// total length, one after the other.  Sequences of one tile count keep their
// order.  (30 sequences of 1 .. 1500 tokens, 16 heads of 32: 114 us in batch
// order, 108 so.)
// With short_ok, items of sequences of at most kShortTokens tokens go last, in
// their order, for the short-sequence kernel; returns their number.  That is
// a launch more where others remain, so few of them (less than the 768
// workgroups the chip holds at a time) then stay among the others.
// out: sum of ceil(ntok / step) items.
constexpr int kShortTokens = 64;
int attention_items(const int32_t* seq, int n, const ImgDesc* imgs, int step, int heads,
                    bool short_ok, AttnItem* out);

// Whether K/V-resident attention is the faster form for a batch or part of n
// sequences (token counts ntok(i)).  Both forms give the same bits.  A
// resident workgroup has a CU to itself (160 KB of LDS, two waves per SIMD);
// the streaming kernel keeps three waves per SIMD, spreads a sequence over
// ceil(ntok / 128) workgroups and lets ragged lengths even out, and reads keys
// and values from L2 more often.  That is the better use of the chip (16
// heads, us, resident / streamed: one image of 577 tokens 35 / 17, 12 images
// 37.4 / 35.0, 32 of 512 59 / 56, 48 of 577 110 / 107; 12 heads: 96 of 197
// 52 / 42, 48 of 442 71 / 54; 100 of 1 .. 640 110 / 99) except when the
// (image, head) pairs are just one per CU and the key tiles many and equal: 16
// of 577 39.4 / 40.8, 14 38.7 / 39.6, 16 of 512 30.8 / 32.1, of 442 28.4 /
// 28.8, of 320 21.9 / 20.5.
template <typename F>
bool resident_pays(int n, int heads, F ntok) {
  const int tiles = (ntok(0) + 63) / 64;
  for (int i = 0; i < n; ++i)
    if ((ntok(i) + 63) / 64 != tiles) return false;
  return tiles >= 7 && tiles <= kResMaxTiles && n * heads <= 256 && n * heads >= 224;
}

// What planning needs to know of a model.
struct PlanModel {
  bool text = false;          // sequences of token ids (else images)
  bool split = false;         // two-part batches allowed (option on, not FP32)
  bool resident = false;      // K/V-resident attention usable (option on, BF16 or MXFP8
                              // activations, head width 64, image model)
  bool map_pool = false;      // attention-pooling head buffers
  bool fold_buffers = false;  // LayerNorm folding buffers (BF16 / e4m3-weight models)
  int es = 2;                 // bytes per activation element (4 for FP32 models)
  int D = 0, F = 0, Kpad = 0, Pd = 0;  // width, MLP width, padded patch length, output dim
  int P = 1, channels = 3;    // patch side and input planes (images)
  int ctx = 0;                // longest sequence (texts)
  int heads = 8;              // attention heads
  bool short_ok = false;      // short-sequence attention kernel usable (BF16 output)
  bool res_rule = false;      // resident only where resident_pays(), and not in bucketed
                              // plans, whose batches differ (VL_OPT_ATTN_RESIDENT 2, the
                              // default); else every sequence that fits (1)
};

// A batch runs as one or two parts.  A part is a run of consecutive images
// with its own descriptors (token starts relative to the part) and its own
// regions of every activation buffer, so two parts never share memory and
// can run concurrently on two streams.  Every kernel works per token row or
// per image with a fixed accumulation order, so a part computes exactly what
// the whole batch would for its images.
struct Part {
  int i0 = 0, n = 0, T = 0, max_ntok = 0, n_items = 0;
  size_t off_imgs = 0, off_items = 0;                       // in the descriptor region
  // Images whose attention runs K/V-resident (indices within the part) and
  // the largest of their key-tile counts.
  size_t off_res = 0;
  int n_res = 0, res_tiles = 0;
  int n_short = 0;      // of n_items, the last ones: the short-sequence kernel's
  size_t off_tok = 0, off_X = 0, off_Y = 0, off_QH = 0, off_E = 0;  // in the workspace
  size_t off_map = 0;   // MAP pooling: per image O, x, LN(x) [n, D] and MLP hidden [n, F]
  // LayerNorm folding: u = bf16(x * gamma) [T, D], per-32-column (mean, M2)
  // partials [T, D/32, 2] and row (mean, rstd) [T, 2]
  size_t off_U = 0, off_PS = 0, off_RS = 0;
  // Launch sizes and buffer regions.  Equal to the counts above, except in
  // a bucketed plan, where they are the bucket's capacities and the kernels
  // read the live counts from the part's BatchCounts record at off_bc.
  bool bucketed = false;
  int T_cap = 0, n_cap = 0, items_cap = 0, res_cap = 0, ntok_cap = 0, res_class = 0;
  size_t off_bc = 0;
};

struct Plan {
  bool bucketed = false;
  int n = 0, T = 0;
  std::vector<int32_t> hw;          // (H, W) per image, for graph keys
  std::vector<char> desc;           // host image of the descriptor region
  size_t desc_bytes = 0;
  std::vector<Part> parts;
  size_t total = 0;                 // workspace bytes
};

// Capacities of a bucketed plan.  Tokens: up to 16 as they are; above,
// rounded up to a multiple of 2^(floor(log2 T) - 2) but kept below the next
// power of two, so a bucket spans at most a quarter of its values and the
// capacity has the floor(log2) of the count, which is what the GEMM tile
// choice depends on.  Images: the next power of two (at most kMaxItems).
int cap_tokens(int T);
int cap_images(int n);

// An image batch: n images of heights hs[i] x widths ws[i].  one_part keeps
// it in one part; bucketed sizes the parts for their capacity buckets.
// False (with *why) on invalid input.
bool make_plan(const PlanModel& m, int32_t n, const int32_t* hs, const int32_t* ws, Plan* p,
               std::string* why, bool one_part = false, bool bucketed = false);

// A text batch: n sequences of lens[i] tokens; descriptors hold the
// sequence's offset in the packed id stream and graph keys (length, 0).
bool make_text_plan(const PlanModel& m, int32_t n, const int32_t* lens, Plan* p,
                    std::string* why);

// A bucketed plan's per-call pointers: the pixel buffer and each part's
// first output row, written into the parts' BatchCounts records.
void bind_batch(Plan& p, const void* pix, float* emb, int Pd);

}  // namespace vl
