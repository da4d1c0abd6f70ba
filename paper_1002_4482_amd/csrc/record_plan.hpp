// Sizes of the recorded walk (lr_walk_rec), in a form that a build for the CPU
// can include: the tests check them at sizes that no test allocates.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace pj {

constexpr int kStrip = 16;       // nodes of a strip
constexpr int kSlab = 256;       // strips of a slab
constexpr int kXcds = 8;
constexpr int kWalkChunk = 64;   // splitter blocks (items) a wave takes at a time

// A batch's nodes are walked in kXcds groups of consecutive chunks.
struct RecordChunks {
  int64_t blocks, chunks;
};
inline RecordChunks record_chunks(int64_t n0, int log2B) {
  RecordChunks c;
  c.blocks = (n0 + (int64_t(1) << log2B) - 1) >> log2B;
  c.chunks = (c.blocks + kWalkChunk - 1) / kWalkChunk;
  return c;
}
constexpr int64_t record_group_chunk(int64_t chunks, int group) { return chunks * group / kXcds; }

// Most lists with nodes that start in one group: counted in the host's table
// (non-decreasing, L + 1 entries), or, without one (a captured call may be
// replayed with other lists of the same total), as many as there can be.
inline int64_t record_heads(const int64_t* off, int64_t L, int64_t n0, int log2B) {
  const RecordChunks c = record_chunks(n0, log2B);
  const int64_t chunk_nodes = int64_t(kWalkChunk) << log2B;
  int64_t most = 0, below = 0;
  for (int g = 0; g < kXcds; ++g) {
    const int64_t lo = record_group_chunk(c.chunks, g), hi = record_group_chunk(c.chunks, g + 1);
    int64_t lists = L;
    if (off) {
      const int64_t upto =
          g == kXcds - 1 ? L : std::lower_bound(off, off + L, hi * chunk_nodes) - off;
      lists = upto - below;
      below = upto;
    }
    most = std::max(most, std::min(lists, (hi - lo) * chunk_nodes));
  }
  return most;
}

// Slabs of one group: of the strips of `nodes` nodes in `pieces` sublist pieces,
// each of which ends in one partly filled strip at most, and for every wave one
// partly filled and one unused slab.
inline int64_t record_slabs(int64_t nodes, int64_t pieces, int64_t waves) {
  return (nodes / kStrip + pieces) / kSlab + 1 + 2 * waves;
}

// Slabs of each group of a batch.  The sublists that start in a group's chunks
// stay in the lists that do, so they hold its nodes and two lists at most -- of
// the longest size a captured call may be replayed with, the next power of two --
// and never more than all.
inline int64_t record_batch_slabs(int64_t n0, int64_t heads, int64_t longest, int log2B,
                                  int64_t max_walk, int64_t waves) {
  const RecordChunks c = record_chunks(n0, log2B);
  const int64_t statics = (c.chunks / kXcds + 1) * kWalkChunk;
  const int64_t nodes = std::min(n0, (statics << log2B) + 2 * longest);
  return record_slabs(nodes, statics + heads + nodes / max_walk + 64, waves);
}

// Strips are numbered in 32 bits, and the walk in place needs none of the
// memory: batches whose lists would waste it (many short ones in one place beside
// a long one) stay there.
constexpr int64_t kRecordBytesPerNode = 32;
constexpr int64_t kRecordBytesFree = int64_t(256) << 20;

inline bool record_fits(int64_t slabs, int64_t strip_bytes, int64_t ent_bytes, int64_t n0) {
  const int64_t limit = kRecordBytesPerNode * n0 + kRecordBytesFree;
  return slabs < (int64_t(1) << 31) / kSlab && ent_bytes <= limit &&
         slabs * kSlab <= (limit - ent_bytes) / strip_bytes;
}

}  // namespace pj
