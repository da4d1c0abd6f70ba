// CPU model of how cc_lds's two workgroups go over one stretch of the offset
// tables: on every table, whatever it holds, each graph has exactly one taker,
// and a group's entries can be indexed with; and of the shares of a batch's work
// that its workgroups get.  Prints OK.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "lds_rules.hpp"

namespace {

constexpr int kCap = 65536, kPairs = 1 << 30, kGroup = 512;

bool check(const std::vector<int64_t>& voff, const std::vector<int64_t>& eoff, int heavy) {
  const int G = (int)voff.size() - 1;
  std::vector<int> takers(G, 0);
  for (const bool take_heavy : {true, false}) {
    for (int ga = 0; ga < G;) {
      const int k = std::min(G - ga, kGroup);
      std::vector<int> sv(k + 1), se(k + 1);
      for (int i = 0; i <= k; ++i) {
        sv[i] = pj::table_entry((int64_t)((uint64_t)voff[ga + i] - (uint64_t)voff[ga]));
        se[i] = pj::table_entry((int64_t)((uint64_t)eoff[ga + i] - (uint64_t)eoff[ga]));
      }
      int heavy_at = k, past = k;
      for (int i = k - 1; i >= 0; --i) {
        if (!(pj::entry_fits(sv[i], sv[i + 1], kCap) && pj::entry_fits(se[i], se[i + 1], kPairs)))
          past = i;
        if (se[i + 1] - se[i] > heavy) heavy_at = i;
      }
      const pj::TableStep next = pj::table_step(heavy_at, past, take_heavy);
      if (next.count < 1 || next.count > k) return false;
      if (next.ours)
        for (int i = 0; i < next.count; ++i) {
          ++takers[ga + i];
          if (past > 0 && (sv[i + 1] < sv[i] || sv[i + 1] > kCap || se[i + 1] < se[i])) return false;
        }
      ga += next.count;
    }
  }
  return std::all_of(takers.begin(), takers.end(), [](int t) { return t == 1; });
}

// The work of every workgroup (0.75 ns a vertex, 0.5 a pair, 6 a graph) is within
// its share and the largest graph it may end with.
bool shares(const std::vector<int64_t>& voff, const std::vector<int64_t>& eoff) {
  const int64_t G = (int64_t)voff.size() - 1, n = voff.back(), m = eoff.back();
  constexpr int kCus = 256;
  const int64_t bin = pj::graph_bin(n, m, G, kCus);
  const auto key = [&](int64_t g) { return pj::graph_key(voff[g], eoff[g], g); };
  const auto cost = [&](int64_t a, int64_t b) {
    return 0.75 * (double)(voff[b] - voff[a]) + 0.5 * (double)(eoff[b] - eoff[a]) + 6.0 * (double)(b - a);
  };
  double largest = 0;
  for (int64_t g = 0; g < G; ++g) largest = std::max(largest, cost(g, g + 1));
  const double share = std::max(cost(0, G) / (2 * kCus), 2048.0);
  const int64_t bins = key(G) / bin + 1;
  if (bins > 8 * kCus + n / 2048) return false;
  int64_t at = 0;
  for (int64_t b = 0; b < bins; ++b) {
    int64_t end = at;
    while (end < G && (b == bins - 1 || key(end) < (b + 1) * bin)) ++end;
    if (cost(at, end) > 2 * share + largest) return false;
    at = end;
  }
  return at == G;
}

bool all_shares() {
  const auto table = [](std::vector<int64_t> sizes) {
    std::vector<int64_t> off{0};
    for (const int64_t s : sizes) off.push_back(off.back() + s);
    return off;
  };
  const auto same = [](size_t count, int64_t size) { return std::vector<int64_t>(count, size); };
  std::vector<int64_t> crowd = same(1000000, 0);  // empty graphs before others
  crowd.insert(crowd.end(), 1000, 100);
  return shares(table(same(20, 100)), table(same(20, 1000000))) &&       // small and dense
         shares(table(same(1000, 20)), table(same(1000, 50000))) &&
         shares(table(same(500000, 1)), table(same(500000, 1))) &&
         shares(table(crowd), table(crowd)) && shares(table(same(3, 1000)), table(same(3, 1500))) &&
         shares(table(same(1024, 11000)), table(same(1024, 50000))) &&
         shares(table(same(5, 65536)), table(same(5, 0)));
}

// The largest size of a table, where it is more than kSmallInstance.
bool largest() {
  std::mt19937_64 rng(3);
  for (int run = 0; run < 2000; ++run) {
    const int64_t count = 1 + (int64_t)(rng() % 700);
    const uint64_t size = 1 + rng() % (run % 2 ? 40 : 4000);
    std::vector<int64_t> off{0};
    for (int64_t i = 0; i < count; ++i)
      off.push_back(off.back() + (int64_t)(rng() % 100 ? rng() % size : 50 * size));
    int64_t most = 0;
    for (int64_t i = 0; i < count; ++i) most = std::max(most, off[i + 1] - off[i]);
    const int64_t got = pj::largest_instance(off.data(), count);
    if (got > most || (got < most && most > pj::kSmallInstance)) return false;
    off.back() = -5;
    if (pj::largest_instance(off.data(), count) != INT64_MAX) return false;
  }
  return true;
}

}  // namespace

int main() {
  if (!largest()) return printf("largest\n"), 1;
  if (!all_shares()) return printf("shares\n"), 1;
  std::mt19937_64 rng(7);
  const auto below = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
  // 3 * 10^9 pairs: a heavy graph behind more than 2^31 pairs of light ones
  {
    std::vector<int64_t> voff{0}, eoff{0};
    for (int g = 0; g < 520; ++g) {
      voff.push_back(voff.back() + 100);
      eoff.push_back(eoff.back() + (g == 450 ? 10'000'000 : 5'500'000));
    }
    if (!check(voff, eoff, (int)(eoff.back() / 512))) return printf("many pairs\n"), 1;
  }
  for (int run = 0; run < 3000; ++run) {
    const int G = 1 + (int)below(1500);
    std::vector<int64_t> voff{0}, eoff{0};
    const int64_t v = 1 + below(run % 3 ? 300 : 60'000), e = 1 + below(run % 5 ? 500 : 20'000'000);
    for (int g = 0; g < G; ++g) {
      voff.push_back(voff.back() + below(v));
      eoff.push_back(eoff.back() + below(below(9) ? e : 9 * e));
    }
    const int heavy = (int)std::min<int64_t>(kPairs, eoff.back() / 512);
    if (run % 2)  // entries of any value
      for (int64_t i = below(9); i > 0; --i) {
        auto& off = below(2) ? voff : eoff;
        off[(size_t)below(G + 1)] = below(3) ? below(2 * off.back() + 2) : (int64_t)rng();
      }
    if (!check(voff, eoff, heavy)) return printf("run %d\n", run), 1;
  }
  printf("OK\n");
  return 0;
}
