// Host check of encode plans made with the options that the library sets for
// its models (head counts, short-sequence kernel, resident attention off /
// forced / by rule): every query block of every sequence once, streamed,
// short or resident; short ones last and only where they go apart; resident
// ones exactly where the option or the rule says; capacities cover counts.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>

#include "plan.hpp"

using namespace vl;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

int main() {
  std::mt19937 rng(11);
  auto uni = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
  int n_plans = 0, n_short_parts = 0, n_mixed_short = 0, n_rule = 0, n_forced = 0;
  for (int t = 0; t < 3000; ++t) {
    const int kind = t % 5;   // BF16 images, head width 64; FP32; MXFP8; texts; head width 32
    PlanModel m;
    m.heads = kind == 4 ? 24 : 4 * uni(1, 4);
    m.D = kind == 4 ? 768 : 64 * m.heads;
    m.F = 4 * m.D; m.Kpad = 640; m.Pd = 512; m.P = 16; m.channels = 3; m.ctx = 77;
    m.text = kind == 3;
    m.es = kind == 1 ? 4 : 2;
    m.split = kind != 1 && uni(0, 1);
    m.fold_buffers = kind == 0 || kind == 3 || kind == 4;
    m.short_ok = kind == 0 || kind == 3 || kind == 4;
    const int option = uni(0, 2);   // VL_OPT_ATTN_RESIDENT
    m.res_rule = option == 2;
    m.resident = option != 0 && (kind == 0 || kind == 2);
    const bool equal = uni(0, 1), bucketed = kind == 0 && uni(0, 2) == 0;
    // (a third of the equal batches around the rule's pair and tile counts)
    const bool near = equal && !m.text && uni(0, 2) == 0;
    const int n = near     ? uni(std::max(1, 210 / m.heads), 270 / m.heads)
                  : m.text ? uni(1, 400)
                  : uni(0, 4) ? uni(1, 24) : uni(25, 300);
    std::vector<int32_t> h(n), w(n);
    const int small = uni(0, 2);    // small images: at most 64 tokens
    const int eh = 16 * uni(near ? 19 : 1, 25), ew = 16 * uni(near ? 19 : 1, 25);
    for (int i = 0; i < n; ++i) {
      const int hi = small == 0 || (small == 1 && uni(0, 1)) ? 7 : 25;
      h[i] = m.text ? uni(1, 77) : equal ? eh : 16 * uni(1, hi);
      w[i] = m.text ? 0 : equal ? ew : 16 * uni(1, hi);
    }
    Plan p;
    std::string why;
    CHECK(m.text ? make_text_plan(m, n, h.data(), &p, &why)
                 : make_plan(m, n, h.data(), w.data(), &p, &why, uni(0, 3) == 0, bucketed));
    ++n_plans;
    int images = 0;
    for (const Part& q : p.parts) {
      auto img = [&](int i) {
        ImgDesc d;
        std::memcpy(&d, p.desc.data() + q.off_imgs + sizeof d * i, sizeof d);
        return d;
      };
      CHECK(q.i0 == images && q.n > 0 && q.n <= q.n_cap);
      images += q.n;
      CHECK(q.n_short >= 0 && q.n_short <= q.n_items && q.n_items <= q.items_cap);
      CHECK(q.n_res <= q.res_cap && q.res_tiles <= q.res_class);
      CHECK(p.desc_bytes >= q.off_items + sizeof(AttnItem) * q.items_cap &&
            p.desc_bytes >= q.off_res + sizeof(int32_t) * q.res_cap);
      // what the resident option or its rule takes
      const bool pays =
          m.resident && m.res_rule && !bucketed && resident_pays(q.n, m.heads, [&](int i) { return img(i).ntok; });
      std::vector<int> res;
      int tiles = 0, fit = 0, streamed = 0;
      for (int i = 0; i < q.n; ++i) {
        const int nt = img(i).ntok;
        if (m.resident && (!m.res_rule || pays) && nt > kResMinTokens && nt <= 64 * kResMaxTiles) {
          res.push_back(i);
          tiles = std::max(tiles, (nt + 63) / 64);
        } else {
          streamed += 1;
          fit += nt <= kShortTokens;
        }
      }
      CHECK(q.n_res == (int)res.size() && q.res_tiles == tiles);
      CHECK(!pays || q.n_res == q.n);
      std::map<std::pair<int, int>, int> seen;
      for (int k = 0; k < q.n_res; ++k) {
        int32_t i;
        std::memcpy(&i, p.desc.data() + q.off_res + 4 * k, 4);
        CHECK(i == res[k]);
        for (int q0 = 0; q0 < img(i).ntok; q0 += kAttnQ) seen[{i, q0}]++;
      }
      const bool apart = m.short_ok && !bucketed && (fit == streamed || fit * m.heads >= 768);
      CHECK(q.n_short == (apart ? fit : 0));
      for (int k = 0; k < q.n_items; ++k) {
        AttnItem it;
        std::memcpy(&it, p.desc.data() + q.off_items + sizeof it * k, sizeof it);
        CHECK(it.img >= 0 && it.img < q.n && it.q0 >= 0 && it.q0 < img(it.img).ntok);
        if (k >= q.n_items - q.n_short) CHECK(img(it.img).ntok <= kShortTokens && it.q0 == 0);
        else if (apart) CHECK(img(it.img).ntok > kShortTokens);
        seen[{it.img, it.q0}]++;
      }
      size_t want = 0;
      for (int i = 0; i < q.n; ++i) want += (img(i).ntok + kAttnQ - 1) / kAttnQ;
      CHECK(seen.size() == want);
      for (const auto& s : seen) CHECK(s.second == 1);
      n_short_parts += q.n_short > 0;
      n_mixed_short += q.n_short > 0 && q.n_short < q.n_items;
      n_rule += pays;
      n_forced += q.n_res > 0 && !m.res_rule;
    }
    CHECK(images == n);
  }
  std::printf("ok plans=%d short=%d mixed=%d rule=%d forced=%d\n", n_plans, n_short_parts,
              n_mixed_short, n_rule, n_forced);
}
