// CPU model of lr_lds's jumping rounds and of its rule for one whole list: a
// workgroup's waves advance in any order between two barriers, the 64 lanes of
// a wave together.  Arguments: nodes, threads of the workgroup, shape, runs.
// Prints how many of the runs were taken for one list.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "lds_rules.hpp"

namespace {

std::mt19937_64 rng(12345);

int below(int n) { return (int)(rng() % (uint64_t)n); }

// Successors of a list through a random permutation, and what its tail does.
std::vector<int> make(int n, const char* shape) {
  std::vector<int> at(n), succ(n);
  for (int i = 0; i < n; ++i) at[i] = i;
  if (!strcmp(shape, "descending")) {  // a cycle of 2^k nodes, next to each other
    int cycle = 2;
    while (cycle * 2 < n) cycle *= 2;
    for (int i = 0; i < n; ++i) succ[i] = i == 0 ? cycle - 1 : i - 1;
    return succ;
  }
  for (int i = n - 1; i > 0; --i) std::swap(at[i], at[below(i + 1)]);
  for (int i = 0; i + 1 < n; ++i) succ[at[i]] = at[i + 1];
  int& last = succ[at[n - 1]];
  if (!strcmp(shape, "valid")) last = -1;
  else if (!strcmp(shape, "circle")) last = at[0];
  else last = at[below(n - 1)];  // "back": into the middle
  return succ;
}

bool accepted(const std::vector<int>& succ, int threads) {
  const int n = (int)succ.size(), kWave = 64, waves = threads / kWave;
  const int rows = (n + threads - 1) / threads;
  std::vector<uint32_t> word(n), mine(n);
  for (int j = 0; j < n; ++j)
    word[j] = mine[j] = succ[j] < 0 || succ[j] == j ? pj::list_tail_word(j) : pj::list_word(succ[j]);
  std::vector<int> row(waves), order;
  for (int span = 1; span < n; span *= 2) {
    std::fill(row.begin(), row.end(), 0);
    // every wave's rows in order, the waves in any order and at any pace
    order.clear();
    for (int w = 0; w < waves; ++w) order.insert(order.end(), rows, w);
    if (below(4) != 0)
      for (int i = (int)order.size() - 1; i > 0; --i) std::swap(order[i], order[below(i + 1)]);
    for (int w : order) {
      const int j0 = (w * rows + row[w]++) * kWave;
      uint32_t next[64];
      for (int l = 0; l < kWave && j0 + l < n; ++l)
        next[l] = pj::list_jump(mine[j0 + l], word[pj::list_target(mine[j0 + l])]);
      for (int l = 0; l < kWave && j0 + l < n; ++l) word[j0 + l] = mine[j0 + l] = next[l];
    }
  }
  for (int j = 0; j < n; ++j)
    if (pj::list_whole(mine[j], n)) return true;
  return false;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  const int n = atoi(argv[1]), threads = atoi(argv[2]), runs = atoi(argv[4]);
  int taken = 0;
  for (int r = 0; r < runs; ++r) taken += accepted(make(n, argv[3]), threads);
  printf("%d\n", taken);
  return 0;
}
