// Rules of the LDS solvers in a form that a build for the CPU can include: the
// tests model the kernels with them.
#pragma once

#include <stdint.h>

#ifdef __HIP__
#include <hip/hip_runtime.h>
#define PJ_RULE __host__ __device__ __forceinline__
#else
#define PJ_RULE inline
#endif

namespace pj {

// -------------------------------------------- groups of instances in LDS
// Workgroup b takes the lists whose key lies in its block of `bin`: the nodes and
// the lists before them, so that it has at most `bin` nodes' starts and at most
// `bin` lists, also where thousands of empty ones lie together.
PJ_RULE int64_t list_key(int64_t off, int64_t l) { return off + l; }

// Graphs likewise, by a key of the work before them: a vertex 1 (0.75 ns of a
// workgroup's time), a pair 1/2, and a graph 8, as tiny ones cost that much.
PJ_RULE int64_t graph_key(int64_t voff, int64_t eoff, int64_t g) { return voff + eoff / 2 + 8 * g; }

// Keys of one workgroup: half a compute unit's share of all, but no less than 2048
// and no more than go with 32768 vertices.
PJ_RULE int64_t graph_bin(int64_t n, int64_t m, int64_t graphs, int cus) {
  const int64_t all = graph_key(n, m, graphs);
  const int64_t share = all / (2 * cus), most = 32768 * (all / (n > 0 ? n : 1));
  const int64_t bin = share < 2048 ? 2048 : share;
  return bin < most ? bin : most;
}

// Size of the largest instance of a host's table (INT64_MAX where it is seen to
// decrease).  Sizes up to kSmallInstance are not told apart: 64 instances that
// are no more together are looked at as one, as a pass over a table of 10^6 graphs
// takes as long as its solve.
constexpr int64_t kSmallInstance = 2048;
inline int64_t largest_instance(const int64_t* off, int64_t count) {
  constexpr int64_t kStep = 64;
  int64_t most = 0;
  for (int64_t g = 0; g < count; g += kStep) {
    const int64_t end = g + kStep < count ? g + kStep : count;
    const int64_t all = off[end] - off[g];
    if (all >= 0 && all <= kSmallInstance) continue;
    for (int64_t i = g; i < end; ++i) {
      const int64_t size = off[i + 1] - off[i];
      if (size < 0) return INT64_MAX;
      if (size > most) most = size;
    }
  }
  return most;
}

// Of its instances a workgroup takes the ones that fit LDS together, and again.
// The table is the device's: it may hold anything, so only a run of entries that
// each fit after the one before may be indexed with.  An entry relative to the
// group's first: what no table of this size can hold does not fit.
PJ_RULE int table_entry(int64_t d) { return d < 0 || d > INT32_MAX ? INT32_MAX : (int)d; }
PJ_RULE bool entry_fits(int before, int entry, int cap) { return entry >= before && entry <= cap; }

// Graphs with many pairs (heavy ones) go to workgroups of their own, so two
// workgroups go over one stretch of the table: each takes or passes over the
// next instances, the heavy ones one at a time, the others a group at a time.
// Of k instances `heavy_at` is the first heavy one and `past` the first that does
// not fit (k: none).  Whether an instance is heavy is only asked of those before
// `past` and of the first, whose size does not depend on where the group
// starts; so both workgroups answer alike, and every instance has one taker.
struct TableStep {
  int count;  // instances gone over
  bool ours;
};
PJ_RULE TableStep table_step(int heavy_at, int past, bool take_heavy) {
  const bool heavy = heavy_at == 0;
  const int group = heavy_at < past ? heavy_at : past;
  return {heavy || group == 0 ? 1 : group, heavy == take_heavy};
}

// ------------------------------------------------ pointer jumping (lr_lds)
// A node's word holds (distance << 16 | tail mark | node) of the node it has
// jumped to.  A tail points to itself at distance 0 and carries the mark; a
// jump copies the mark with the node, so a marked word has reached a tail of the
// input, and one that has not (its path ends in a cycle, whatever its distance
// has grown or wrapped to) never gets it.  The path to a tail passes no node
// twice, so a marked distance is exact and below kListNodes; it is size - 1 for
// some node exactly if that node's path is the whole list.
constexpr int kListNodes = 1 << 14;
constexpr uint32_t kListTail = kListNodes;

PJ_RULE uint32_t list_tail_word(int node) { return kListTail | (uint32_t)node; }
PJ_RULE uint32_t list_word(int next) { return 1u << 16 | (uint32_t)next; }
PJ_RULE int list_target(uint32_t word) { return (int)(word & (kListNodes - 1)); }
PJ_RULE int list_distance(uint32_t word) { return (int)(word >> 16); }

// The word after a jump to the target of `mine`, whose word is `there`.  After k
// jumps a node up to 2^k - 1 steps from its tail has the mark.
PJ_RULE uint32_t list_jump(uint32_t mine, uint32_t there) {
  return ((mine >> 16) + (there >> 16)) << 16 | (there & 0xffff);
}

PJ_RULE bool list_whole(uint32_t word, int size) {
  return (word & kListTail) != 0 && list_distance(word) == size - 1;
}

}  // namespace pj
