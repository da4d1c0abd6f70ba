// Checks of record_plan.hpp: strips stay within 32 bits and the memory within
// its limit at any size, and a group's strips suffice for lists laid out at
// random.  Prints OK.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "record_plan.hpp"

namespace {

std::mt19937_64 rng(11);
int64_t below(int64_t n) { return (int64_t)(rng() % (uint64_t)n); }

int fail(const char* what) {
  printf("%s\n", what);
  return 1;
}

int sizes() {
  // 3.1 * 10^8 lists of one node and one of 20000: eight strips a list, before
  for (const int64_t L : {int64_t(1000), int64_t(1000000), int64_t(310000000), int64_t(1) << 30})
    for (const int64_t avg : {1, 2, 5, 10, 100, 10000})
      for (const int log2B : {1, 5, 6, 16})
        for (const int64_t strip : {72, 136})
          for (const int64_t max_walk : {16, 1024}) {
            const int64_t n0 = L * avg + 20000;
            if (n0 >= INT32_MAX) continue;
            const int64_t heads = pj::record_heads(nullptr, L, n0, log2B);
            const int64_t slabs =
                pj::kXcds * pj::record_batch_slabs(n0, heads, 1 << 15, log2B, max_walk, 128);
            if (slabs <= 0) return fail("slabs");
            if (!pj::record_fits(slabs, strip, 8 * n0, n0)) continue;
            if (slabs * pj::kSlab >= INT32_MAX) return fail("strip numbers");
            if (slabs * pj::kSlab * strip + 8 * n0 >
                pj::kRecordBytesPerNode * n0 + pj::kRecordBytesFree)
              return fail("bytes");
          }
  // what it is for: lists of a hundred nodes and more beside long ones
  for (const int64_t n0 : {int64_t(1) << 20, int64_t(1) << 26, int64_t(430000000)}) {
    const int64_t slabs = pj::kXcds * pj::record_batch_slabs(n0, n0 / 800, 1 << 20, 5, 1024, 128);
    if (!pj::record_fits(slabs, 72, 4 * n0, n0)) return fail("ordinary batch");
  }
  return 0;
}

int one_batch() {
  const int log2B = 1 + (int)below(5), max_walk = 16 * (1 + (int)below(4));
  std::vector<int64_t> off{0};
  const int64_t L = 1 + below(3000);
  const int64_t crowd = below(L);  // short lists from here on, half of the time
  for (int64_t l = 0; l < L; ++l)
    off.push_back(off.back() + (below(40) == 0 && l < crowd ? below(9000) : below(4)));
  const int64_t n0 = off.back();
  if (n0 == 0) return 0;
  int64_t longest = 0;
  std::vector<int64_t> next(n0, -1), head(L, -1);
  for (int64_t l = 0; l < L; ++l) {
    const int64_t size = off[l + 1] - off[l];
    longest = std::max(longest, size);
    std::vector<int64_t> at(size);
    for (int64_t i = 0; i < size; ++i) at[i] = off[l] + i;
    for (int64_t i = size - 1; i > 0; --i) std::swap(at[i], at[below(i + 1)]);
    for (int64_t i = 0; i + 1 < size; ++i) next[at[i]] = at[i + 1];
    if (size) head[l] = at[0];
  }
  const pj::RecordChunks c = pj::record_chunks(n0, log2B);
  std::vector<int64_t> splitter(c.blocks);
  std::vector<char> is(n0, 0);
  for (int64_t b = 0; b < c.blocks; ++b) {
    const int64_t lo = b << log2B;
    is[splitter[b] = lo + below(std::min<int64_t>(n0 - lo, 1 << log2B))] = 1;
  }
  const auto strips = [&](int64_t x) {
    int64_t count = 0, len = 0;
    for (;;) {
      if (len++ % pj::kStrip == 0) ++count;
      if (len == max_walk) len = 0;
      x = next[x];
      if (x < 0 || is[x]) return count;
    }
  };
  const int64_t chunk_nodes = int64_t(pj::kWalkChunk) << log2B;
  for (int known = 0; known < 2; ++known) {
    const int64_t heads = pj::record_heads(known ? off.data() : nullptr, L, n0, log2B);
    const int64_t slabs = pj::record_batch_slabs(n0, heads, longest, log2B, max_walk, 4);
    for (int g = 0; g < pj::kXcds; ++g) {
      const int64_t lo = pj::record_group_chunk(c.chunks, g) * pj::kWalkChunk;
      const int64_t hi =
          std::min(c.blocks, pj::record_group_chunk(c.chunks, g + 1) * pj::kWalkChunk);
      int64_t used = 0, starts = 0;
      for (int64_t b = lo; b < hi; ++b) used += strips(splitter[b]);
      for (int64_t l = 0; l < L; ++l) {
        const int64_t chunk = off[l] / chunk_nodes;
        if (head[l] < 0 || chunk < pj::record_group_chunk(c.chunks, g) ||
            chunk >= pj::record_group_chunk(c.chunks, g + 1))
          continue;
        ++starts;
        if (!is[head[l]]) used += strips(head[l]);
      }
      if (starts > heads) return fail("heads");
      if (used > (slabs - 2 * 4) * pj::kSlab) return fail("strips of a group");
    }
  }
  return 0;
}

}  // namespace

int main() {
  if (sizes()) return 1;
  for (int run = 0; run < 1500; ++run)
    if (one_batch()) return 1;
  printf("OK\n");
  return 0;
}
