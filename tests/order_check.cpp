// Host checks of attention work order and of the resident rule (plan.hpp):
// every item once, most key tiles first inside each run, runs of balanced
// length, equal tile counts untouched, short sequences last where they go
// apart; plans with the rule cover every query block once.
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
  std::mt19937 rng(7);
  int resident_parts = 0;
  for (int t = 0; t < 600; ++t) {
    const int heads = 1 + (int)(rng() % 64), n = 1 + (int)(rng() % 60);
    std::vector<ImgDesc> imgs(n);
    std::vector<AttnItem> items;
    const int one = t % 3 == 0 ? 1 + (int)(rng() % 900) : 0;
    for (int i = 0; i < n; ++i) {
      std::memset(&imgs[i], 0, sizeof imgs[i]);
      imgs[i].ntok = one ? one : 1 + (int)(rng() % (t % 5 ? 900 : 90));
      for (int q0 = 0; q0 < imgs[i].ntok; q0 += kAttnQ) items.push_back(AttnItem{i, q0});
    }
    const bool short_ok = t & 1;
    std::vector<int32_t> seq(n);
    for (int i = 0; i < n; ++i) seq[i] = i;
    std::vector<AttnItem> a(items.size());
    const int n_short =
        attention_items(seq.data(), n, imgs.data(), kAttnQ, heads, short_ok, a.data());
    auto key = [](const AttnItem& x) { return std::make_pair(x.img, x.q0); };
    std::map<std::pair<int, int>, int> seen;
    for (const auto& x : a) seen[key(x)]++;
    CHECK(a.size() == items.size() && seen.size() == items.size());
    int fit = 0;
    for (const auto& x : items) fit += short_ok && imgs[x.img].ntok <= kShortTokens;
    const bool apart = fit == (int)items.size() || fit * heads >= 768;
    CHECK(n_short == (apart ? fit : 0));
    for (int k = 0; k < n_short; ++k) {
      const AttnItem x = a[a.size() - n_short + k];
      CHECK(imgs[x.img].ntok <= kShortTokens);
      if (k) CHECK(key(a[a.size() - n_short + k - 1]) < key(x));
    }
    a.resize(a.size() - n_short);
    if (a.empty()) continue;
    for (size_t i = 0; n_short && i < items.size();)
      if (imgs[items[i].img].ntok <= kShortTokens) items.erase(items.begin() + i);
      else ++i;
    bool same = true;
    auto tiles = [&](const AttnItem& x) { return (imgs[x.img].ntok + 63) / 64; };
    for (const auto& x : a) same = same && tiles(x) == tiles(a[0]);
    if (same) {
      for (size_t i = 0; i < a.size(); ++i) CHECK(key(a[i]) == key(items[i]));
      continue;
    }
    const size_t runs = heads % 8 == 0 ? 1 : heads % 4 == 0 ? 2 : heads % 2 == 0 ? 4 : 8;
    size_t p = 0;
    long lo = -1, hi = 0;
    for (size_t k = 0; k < runs; ++k) {
      const size_t cnt = a.size() / runs + (k < a.size() % runs ? 1 : 0);
      long sum = 0;
      for (size_t i = 0; i < cnt; ++i) {
        const int len = tiles(a[p + i]);
        if (i) CHECK(len <= tiles(a[p + i - 1]));
        sum += len;
      }
      p += cnt;
      lo = lo < 0 ? sum : std::min(lo, sum);
      hi = std::max(hi, sum);
    }
    CHECK(hi - lo <= 15);   // dealt round-robin: runs differ by at most the longest
  }
  for (int t = 0; t < 400; ++t) {
    PlanModel m;
    m.resident = m.res_rule = true;
    m.split = t & 1;
    m.D = 768; m.F = 3072; m.Kpad = 768; m.Pd = 512; m.P = 16;
    m.heads = 4 * (1 + (int)(rng() % 5));
    const int n = 1 + (int)(rng() % 70), px = 16 * (18 + (int)(rng() % 9));
    std::vector<int32_t> hw(n, px);
    if (t % 4 == 0) hw[rng() % n] = 224;
    for (int bucketed = 0; bucketed < 2; ++bucketed) {
      Plan p;
      std::string why;
      CHECK(make_plan(m, n, hw.data(), hw.data(), &p, &why, false, bucketed != 0));
      for (const Part& q : p.parts) {
        std::map<std::pair<int, int>, int> seen;
        auto at = [&](size_t off) { return p.desc.data() + off; };
        for (int j = 0; j < q.n_items; ++j) {
          AttnItem it;
          std::memcpy(&it, at(q.off_items + sizeof it * j), sizeof it);
          seen[{it.img, it.q0}]++;
        }
        for (int j = 0; j < q.n_res; ++j) {
          int32_t i;
          std::memcpy(&i, at(q.off_res + 4 * j), 4);
          ImgDesc d;
          std::memcpy(&d, at(q.off_imgs + sizeof d * i), sizeof d);
          for (int q0 = 0; q0 < d.ntok; q0 += kAttnQ) seen[{i, q0}]++;
        }
        size_t want = 0;
        for (int i = 0; i < q.n; ++i) {
          ImgDesc d;
          std::memcpy(&d, at(q.off_imgs + sizeof d * i), sizeof d);
          want += (d.ntok + kAttnQ - 1) / kAttnQ;
        }
        CHECK(seen.size() == want);
        for (const auto& s : seen) CHECK(s.second == 1);
        CHECK(!bucketed || (q.n_res == 0 && q.res_cap == 0));
        if (q.n_res) {
          ++resident_parts;
          CHECK(q.n_res == q.n && q.n_items == 0 && q.res_tiles >= 7 && q.n * m.heads <= 256 &&
                q.n * m.heads >= 224);
        }
      }
    }
  }
  CHECK(resident_parts > 5);
  std::printf("ok\n");
}
