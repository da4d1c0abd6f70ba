// List ranking on gfx950: Wyllie pointer jumping and the random-splitter
// (sparse ruling set) method with recursive ranking of the splitter list.
//
// One code path serves a single list and a batch of lists: a single list is
// a batch with L = 1.  Global node ids run over the concatenation; the
// successors of level 0 are local to their list.
//
// Ruling set, per level l (Section 3.2, "Parallel Random Splitter"):
//   * splitters: one node per block of 2^log2B consecutive ids, at an offset
//     drawn by a counter-based hash (so "is y a splitter" is arithmetic, with
//     no mark array), plus one virtual splitter per list standing at its head;
//   * walk (the paper's RS3): persistent lanes take splitters from a work
//     counter and follow successors until the next splitter or the tail,
//     writing (sublist id, weight before the node) per node and
//     (next splitter, sublist weight) per splitter.  A walk longer than
//     max_walk nodes is cut and the cut node becomes a new splitter, which
//     bounds every loop even on malformed input;
//   * the splitter lists (one per input list, head = its virtual splitter)
//     form level l+1, weighted by sublist length, and are ranked the same way
//     (the recursion replacing the paper's single-block RS4) until a level is
//     small enough for one workgroup, which ranks it in LDS (lr_base_walk, or
//     the paper's single-kernel Wyllie for many lists, lr_base_lds);
//   * expand (the paper's RS5): rank[x] = rank of its splitter + its weight
//     offset, a coalesced pass per level.
// Long lists that are not local, and large batches of shorter ones, record
// level 0's walks instead of writing over the nodes, and deal the records to
// the ranks (lr_walk_rec, lr_bin, lr_place).  Lists that fit LDS are ranked
// there by one kernel (lr_lds, lr_one_lds).
// The rank counted here is the distance from the head; the paper's RS5
// subtracts from the splitter rank because it counts toward the tail.
#include <algorithm>
#include <cmath>
#include <vector>

#include "lds_rules.hpp"
#include "pj_internal.hpp"
#include "record_plan.hpp"

namespace pj {
namespace {

constexpr int kMaxCutoff = 16384;
constexpr int kBaseThreads = 1024;
constexpr int kPerThread = kMaxCutoff / kBaseThreads;

struct LevelCtl {
  int32_t n;     // nodes at this level (level 0: written by init)
  int32_t r;     // static splitters of this level (written by its walk)
  int32_t dyn;   // cut points requested at this level (may exceed the cap)
  int32_t work;  // work counter of the persistent walk
};

struct LrCtl {
  LevelCtl lv[PJ_MAX_LEVELS + 2];
  int32_t err;
  int32_t pad;
  unsigned long long base_total;  // total weight seen by the base ranking
  unsigned long long near;        // single list: successors within kNear ids
};

// A successor within kNear ids of its node counts as local (see lr_walk).
constexpr int kNear = 64;

// Most successors are not local: level 0 takes the far spacing, where the plan
// has one.
__device__ __forceinline__ bool far_chosen(const LrCtl* ctl, int N) {
  return 2ull * ctl->near <= (unsigned long long)N;
}

// Node count of level `level` >= 1: static + virtual + granted cut points of
// the level below.
__device__ __forceinline__ int level_nodes(const LrCtl* ctl, int level, int L, int cap_prev) {
  if (level == 0) return ctl->lv[0].n;
  const LevelCtl& p = ctl->lv[level - 1];
  return p.r + L + min(p.dyn, cap_prev);
}

__device__ __forceinline__ uint32_t splitter_offset(uint32_t block, uint32_t seed, uint32_t bsize) {
  uint32_t h = mix32(block * 0x9E3779B9u ^ seed);
  return (uint32_t)(((uint64_t)h * bsize) >> 32);
}

// Is id y the static splitter of its block?
__device__ __forceinline__ bool is_static(int y, int N, int log2B, uint32_t seed) {
  int b = y >> log2B;
  int start = b << log2B;
  int bsize = min(1 << log2B, N - start);
  return (uint32_t)(y - start) == splitter_offset((uint32_t)b, seed, (uint32_t)bsize);
}

// What a walk needs to know of a node's successor y (a global id), worked out
// once by the head-find pass so that a step of the walk is a read and a sign
// test: y, with the sign bit set if y is a static splitter.  A tail is -1.
// Weighted calls get {code, weight} pairs.
constexpr int kNoCopy = 0, kPlainCopy = 1, kCodedCopy = 2, kPairCopy = 3;

__device__ __forceinline__ int step_code(int y, int N, int log2B, uint32_t seed) {
  return is_static(y, N, log2B, seed) ? y | INT32_MIN : y;
}

__device__ __forceinline__ void store_pair(int2* p, int a, int b) { *p = make_int2(a, b); }

// Recorded walk (see lr_walk_rec; its sizes are in record_plan.hpp).
constexpr int kBinShift = 15;
constexpr int kBinNodes = 1 << kBinShift;  // 128 KiB of ranks in LDS
constexpr int kWordLongest = 1 << 20;      // (see lr_bin)
constexpr int kBinShiftMin = 12;
constexpr int kTileSlabs = 4;
constexpr int kTileThreads = kTileSlabs * kSlab;
constexpr int kTileBins = 2048;

struct RecCtl {
  int32_t taken[kXcds];      // slabs taken of each group's
};

struct RecArgs {
  RecCtl* ctl;
  int4* strips;         // kStrip node ids (-1: none) per strip
  int4* before;         // weighted: weight of the sublist before each of them
  int2* head;           // {sublist id, offset of the strip's first node} per strip
  int32_t* used;        // strips used of each slab
  int32_t* chunk_list;  // a batch: first list of each chunk
  int32_t* cursor;      // entries of each bin
  void* ent;            // a bin's entries, one per node
  int bin_shift;        // nodes of a bin, as a shift
  int group_slabs;      // slabs of a group (an XCD of a batch; all of one list)
  int log2B;            // splitter spacing
  int if_far;           // only if the head-find pass found the list not local
};

// Where the first four nodes of a strip are, the next four kSlab words on: a
// slab holds those of its strips side by side, so that the lanes of a wave move
// whole lines (4096 lists of 2^6..2^20 nodes, strip after strip: walk 4280 us,
// lr_bin 1300; side by side 4165 and 1240).
__device__ __forceinline__ int64_t strip_word(int strip) {
  return (int64_t)(strip / kSlab) * (kSlab * kStrip / 4) + strip % kSlab;
}

// ------------------------------------------------------------------ init
__global__ void lr_init(LrCtl* ctl, int n0, unsigned long long* lsum, int32_t* ltails,
                        int32_t* lerr, int L, int64_t* off_single, RecArgs rec, int nbins) {
  int tid = blockIdx.x * blockDim.x + threadIdx.x;
  int stride = gridDim.x * blockDim.x;
  int32_t* c = reinterpret_cast<int32_t*>(ctl);
  for (int i = tid; i < (int)(sizeof(LrCtl) / 4); i += stride) c[i] = 0;
  for (int i = tid; i < L; i += stride) {
    lsum[i] = 0ull;
    ltails[i] = 0;
    lerr[i] = 0;
  }
  if (rec.ctl && tid < (int)(sizeof(RecCtl) / 4)) reinterpret_cast<int32_t*>(rec.ctl)[tid] = 0;
  for (int i = tid; i < nbins; i += stride) rec.cursor[i] = 0;
  if (tid == 0) {
    ctl->lv[0].n = n0;
    if (off_single) {
      off_single[0] = 0;
      off_single[1] = n0;
    }
  }
}

// ------------------------------------------------------------- head find
// Head of each list by the index-sum identity: the nodes with a predecessor
// are exactly the non-tail successors, so
//   head = size(size-1)/2 - sum of non-tail successors.
// The same coalesced pass counts tails and flags out-of-range successors.
template <int kCopy>
__global__ void __launch_bounds__(256) lr_headfind_single(const int32_t* succ, int n,
                                                          int32_t* copy,
                                                          const int32_t* __restrict__ weight,
                                                          int2* __restrict__ pair, int log2B,
                                                          uint32_t seed,
                                                          unsigned long long* lsum,
                                                          int32_t* ltails, int32_t* lerr,
                                                          unsigned long long* lnear) {
  unsigned long long acc = 0;
  int tails = 0, bad = 0, near = 0;
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int stride = gridDim.x * blockDim.x;
  const bool vec = ((reinterpret_cast<uintptr_t>(succ) | reinterpret_cast<uintptr_t>(copy) |
                     reinterpret_cast<uintptr_t>(weight)) & 15) == 0;
  const int n4 = vec ? (n >> 2) : 0;
  const int4* s4 = reinterpret_cast<const int4*>(succ);
  const auto one = [&](int s, int i) {  // counts node i, returns its code
    const bool tail = (s == -1) | (s == i);
    const bool range = (unsigned)s < (unsigned)n;
    tails += tail;
    bad |= (!tail & !range);
    acc += (!tail & range) ? (unsigned long long)s : 0ull;
    near += (!tail & range) & ((unsigned)(s - i + kNear) <= 2u * kNear);
    return kCopy < kCodedCopy ? s : (tail | !range) ? -1 : step_code(s, n, log2B, seed);
  };
  for (int q = tid; q < n4; q += stride) {
    int4 v = s4[q];
    const int i = q << 2;
    v.x = one(v.x, i);
    v.y = one(v.y, i + 1);
    v.z = one(v.z, i + 2);
    v.w = one(v.w, i + 3);
    if (kCopy == kPairCopy) {
      const int4 u = reinterpret_cast<const int4*>(weight)[q];
      reinterpret_cast<int4*>(pair)[2 * q] = make_int4(v.x, u.x, v.y, u.y);
      reinterpret_cast<int4*>(pair)[2 * q + 1] = make_int4(v.z, u.z, v.w, u.w);
    } else if (kCopy != kNoCopy) {
      reinterpret_cast<int4*>(copy)[q] = v;
    }
  }
  for (int i = (n4 << 2) + tid; i < n; i += stride) {
    const int v = one(succ[i], i);
    if (kCopy == kPairCopy) pair[i] = make_int2(v, weight[i]);
    else if (kCopy != kNoCopy) copy[i] = v;
  }
  acc = wave_sum(acc);
  tails = wave_sum(tails);
  bad = wave_sum(bad);
  near = wave_sum(near);
  // one atomic per workgroup: atomics on a single address serialise
  __shared__ unsigned long long s_acc[256 / kWave];
  __shared__ int s_tails[256 / kWave], s_bad[256 / kWave], s_near[256 / kWave];
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) {
    s_acc[w] = acc;
    s_tails[w] = tails;
    s_bad[w] = bad;
    s_near[w] = near;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x / kWave); ++i) {
      acc += s_acc[i];
      tails += s_tails[i];
      bad += s_bad[i];
      near += s_near[i];
    }
    if (acc) atomicAdd(lsum, acc);
    if (tails) atomicAdd(ltails, tails);
    if (bad) atomicOr(lerr, kErrRange);
    if (near && lnear) atomicAdd(lnear, (unsigned long long)near);
  }
}

// Batched form: each wave owns chunks of 64*kChunk consecutive positions and
// tracks the owning list while it advances.  Its sums go to the list's words
// when it leaves the list, so a wave takes four chunks where there are enough
// (headfind_grid): with one each, the atomics of a few long lists serialise (8
// lists of 1.4 M nodes: 150 us, 60 us with several).
constexpr int kHfChunk = 16;
template <int kCopy>
__global__ void __launch_bounds__(256) lr_headfind_batched(const int32_t* succ,
                                                           const int64_t* __restrict__ off, int L,
                                                           int n, int32_t* copy,
                                                           const int32_t* __restrict__ weight,
                                                           int2* __restrict__ pair, int log2B,
                                                           uint32_t seed,
                                                           unsigned long long* lsum,
                                                           int32_t* ltails, int32_t* lerr) {
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int nwaves = (gridDim.x * blockDim.x) / kWave;
  const int lane = lane_id();
  const int chunk = kWave * kHfChunk;
  // each wave owns a contiguous run of chunks: one search of the offset
  // table per wave, then every lane follows the list boundaries forward
  const int64_t nchunks = ((int64_t)n + chunk - 1) / chunk;
  const int64_t per = (nchunks + nwaves - 1) / nwaves;
  const int64_t ci0 = (int64_t)wave * per;
  const int64_t ci1 = ci0 + per < nchunks ? ci0 + per : nchunks;
  if (ci0 >= ci1) return;
  int l = find_instance(off, L, ci0 * chunk);
  int64_t lbase = off[l], lend = off[l + 1];
  unsigned long long acc = 0;
  int tails = 0;
  for (int64_t ci = ci0; ci < ci1; ++ci) {
    const int64_t c0 = ci * chunk;
    // all loads (and the copy) of the chunk first: the flushes below hold
    // atomics that would otherwise keep each load waiting for the last
    int sv[kHfChunk];
#pragma unroll
    for (int t = 0; t < kHfChunk; ++t) {
      const int64_t g = c0 + t * kWave + lane;
      sv[t] = g < n ? succ[g] : 0;
    }
    if (kCopy == kPlainCopy) {
#pragma unroll
      for (int t = 0; t < kHfChunk; ++t) {
        const int64_t g = c0 + t * kWave + lane;
        if (g < n) copy[g] = sv[t];
      }
    }
    for (int t = 0; t < kHfChunk; ++t) {
      int64_t g = c0 + t * kWave + lane;
      if (g >= n) break;
      if (g >= lend) {  // moved into a later list: flush
        if (acc) atomicAdd(&lsum[l], acc);
        if (tails) atomicAdd(&ltails[l], tails);
        acc = 0;
        tails = 0;
        l = find_from(off, L, l, g);  // (past thousands of empty ones at a time)
        lbase = off[l];
        lend = off[l + 1];
      }
      const int s = sv[t];
      int x = (int)(g - lbase);
      int size = (int)(lend - lbase);
      bool tail = (s == -1) | (s == x);
      bool range = (unsigned)s < (unsigned)size;
      tails += tail;
      if (!tail & !range) atomicOr(&lerr[l], kErrRange);
      acc += (!tail & range) ? (unsigned long long)s : 0ull;
      if (kCopy >= kCodedCopy) {
        const int code = (tail | !range) ? -1 : step_code((int)lbase + s, n, log2B, seed);
        if (kCopy == kPairCopy) pair[g] = make_int2(code, weight[g]);
        else copy[g] = code;
      }
    }
  }
  // wave-combine when the whole wave ended in one list
  const int l0 = __shfl(l, 0);
  if (__ballot(l != l0) == 0) {
    acc = wave_sum(acc);
    tails = wave_sum(tails);
    if (lane == 0) {
      if (acc) atomicAdd(&lsum[l], acc);
      if (tails) atomicAdd(&ltails[l], tails);
    }
  } else {
    if (acc) atomicAdd(&lsum[l], acc);
    if (tails) atomicAdd(&ltails[l], tails);
  }
}

// ------------------------------------------------------------------ walk
struct WalkArgs {
  const int32_t* succ0;              // level 0: local successors
  const int32_t* weight0;            // level 0, weighted call: node weights (unpacked form)
  const int2* link_in;               // level >= 1: {next, weight} per node
  const int64_t* off;                // level 0: list offsets (L+1)
  const unsigned long long* lsum;    // level 0: head-find sums
  const int32_t* ltails;             // level 0: tail counts
  int32_t* lerr;                     // per-list error bits
  int2* state;                       // {sublist id, weight before node} per node
  int32_t* work;                     // level 0 packed form: successor copy, overwritten
                                     // in place by (sublist id << kbits | offset)
  int2* link_out;                    // {next splitter, sublist weight} per splitter
  LrCtl* ctl;
  int L;
  int level;
  int log2B;
  int log2B_far; // level 0, single list, > 0: the block size used instead of
                 // 2^log2B when fewer than half the successors are local,
  int kbits_far; // with these offset bits and cut length
  int max_walk_far;
  int max_walk;
  int cap;       // cut points this level may create
  int cap_prev;  // cut points the level below could create
  int kbits;     // level 0 packed form: bits of the in-sublist offset
  uint32_t seed;
  int if_near;   // only if the successors are local (the recorded walk took the others)
};

// kPacked (level 0): the successors are read from a.work, a copy made by the
// head-find pass, and each visited slot is overwritten with the node's packed
// state.  The read and the write then touch the same cache line, which costs
// far less than a write to a second random line.
constexpr int kWalkBurst = 16;

// kPaired (level 0, weighted calls): the state array holds {step code, weight}
// pairs, made by the head-find pass, and a visited one {-2 - sublist id, weight
// before the node}: one random line per node instead of three for successor,
// weight and state (walk of 2^26 random nodes 5.66 -> 2.58 ms in place, 1.59
// recorded).  A visited state is told from a code by its sign and size, which
// the host makes sure of.
template <bool kLevel0, bool kBatched, bool kPacked, bool kPaired = false>
__global__ void __launch_bounds__(1024) lr_walk(WalkArgs a) {
  LrCtl* ctl = a.ctl;
  const int N = level_nodes(ctl, a.level, a.L, a.cap_prev);
  // Splitter spacing for level 0 of a single list chosen on the device from
  // the head-find pass: when most successors are local (sequential-like
  // layouts), the lanes of a wave walk neighbouring sublists and share cache
  // lines, and short sublists (spacing 2^log2B) pay; when they are random,
  // every step is its own line and fewer, longer sublists (2^log2B_far) make
  // the final scatter's splitter-rank gathers hit in L2.  The plan is sized
  // for the smaller spacing.
  const bool far =
      kLevel0 && a.log2B_far > 0 && far_chosen(ctl, N);
  if (kLevel0 && far && a.if_near) return;
  const int log2B = far ? a.log2B_far : a.log2B;
  const int kbits = far ? a.kbits_far : a.kbits;
  const int max_walk = far ? a.max_walk_far : a.max_walk;
  // One list, packed: the work array holds step codes, made for the far spacing
  // when there is one.
  constexpr bool kCoded = kPaired || (kLevel0 && !kBatched && kPacked);
  const bool coded = a.log2B_far == 0 || far;
  const int r = (int)(((int64_t)N + (1 << log2B) - 1) >> log2B);
  const int head_base = kLevel0 ? 0 : ctl->lv[a.level - 1].r;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->lv[a.level].r = r;
  const int items = r + a.L;
  int* dyn = &ctl->lv[a.level].dyn;
  const uint32_t seed = a.seed;
  // Work distribution.  One list, and the recursion levels: each workgroup
  // owns a contiguous range of items (static splitters, then the virtual
  // splitters at the list heads) and hands them to its lanes through an LDS
  // counter.  A batch's level 0 (kChunks): its thousands of list heads come
  // last and would all fall to the last workgroups, so each wave walks
  // chunks of kWalkChunk items instead, first the chunk of its own index,
  // then chunks taken from a device-wide counter with one atomic per chunk
  // (4096 lists of 2^6..2^20 nodes: 17.1 -> 15.7 ms for the walk; for one
  // list the counter costs more than it balances: the sequential 2^26 list,
  // 8 M sublists, 0.6 -> 1.5 ms).  A counter hit at every refill of every
  // wave would serialise at the memory side.
  constexpr bool kChunks = kLevel0 && kBatched;
  __shared__ int wg_next;
  int wg_hi = items;
  if (!kChunks) {
    const int per = (int)(((int64_t)items + gridDim.x - 1) / gridDim.x);
    const int wg_lo = min(items, (int)((int64_t)blockIdx.x * per));
    wg_hi = min(items, wg_lo + per);
    if (threadIdx.x == 0) wg_next = wg_lo;
    __syncthreads();
  }
  const int nwaves = (int)(((int64_t)gridDim.x * blockDim.x) / kWave);
  const int wave_id = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave);
  int chunk_lo = (int)min<int64_t>(items, (int64_t)wave_id * kWalkChunk);
  int chunk_hi = (int)min<int64_t>(items, (int64_t)chunk_lo + kWalkChunk);
  bool drained = false;  // the device-wide counter has passed the last item
  int* counter = &ctl->lv[a.level].work;
  const int64_t dyn_base = (int64_t)nwaves * kWalkChunk;

  int sid = -1;       // sublist being walked, -1 = idle
  int x = 0;          // current node
  int k = 0;          // weight of the sublist before x
  int steps = 0;
  int64_t base = 0;   // level 0: first id of the lane's list
  int size = N;       // level 0: size of the lane's list
  int lid = 0;        // level 0: list index
  bool retired = false;
  int errbits = 0;
  // what a node's step needs: {successor or code, weight}
  const auto fetch = [&](int at) {
    if (kPaired) return a.state[at];
    if (kLevel0 && kPacked) return make_int2(a.work[at], 1);
    if (kLevel0) return make_int2(a.succ0[at], a.weight0 ? a.weight0[at] : 1);
    return a.link_in[at];
  };
  int2 in = make_int2(-1, 0);  // of node x

  while (true) {
    const bool need = (sid < 0) & !retired;
    const uint64_t needm = __ballot(need);
    if (needm) {
      int first, avail;
      if (kChunks) {
        if (chunk_lo >= chunk_hi && !drained) {  // the wave's chunk is used up
          int got = 0;
          if (lane_id() == 0) got = atomicAdd(counter, kWalkChunk);
          got = __shfl(got, 0);
          const int64_t lo = dyn_base + got;
          drained = lo >= items;
          chunk_lo = drained ? items : (int)lo;
          chunk_hi = drained ? items : (int)min<int64_t>(items, lo + kWalkChunk);
        }
        first = chunk_lo;
        avail = chunk_hi - chunk_lo;
        chunk_lo += min(avail, __popcll(needm));
      } else {
        const int leader = __builtin_ctzll(needm);
        int f = 0;
        if (lane_id() == leader) f = atomicAdd(&wg_next, __popcll(needm));
        first = __shfl(f, leader);
        avail = max(0, wg_hi - first);
      }
      // lanes past the end of the chunk (or range) wait for the next chunk,
      // or retire once there is none
      const int rank_in = lanes_below(needm);
      if (need && rank_in >= avail) {
        retired = kChunks ? drained : true;
      } else if (need) {
        const int item = first + rank_in;
        if (item < r) {  // static splitter
          const int start = item << log2B;
          const int bsize = min(1 << log2B, N - start);
          x = start + (int)splitter_offset((uint32_t)item, seed, (uint32_t)bsize);
          if (kLevel0 && kBatched && !kCoded) {
            lid = find_instance(a.off, a.L, x);
            base = a.off[lid];
            size = (int)(a.off[lid + 1] - base);
          }
          sid = item;
          k = 0;
          steps = 0;
        } else {  // virtual splitter standing at the head of list l
          const int l = item - r;
          int h;
          bool ok = true;
          if (kLevel0) {
            if (kBatched) {
              base = a.off[l];
              size = (int)(a.off[l + 1] - base);
            } else {
              base = 0;
              size = N;
            }
            lid = l;
            if (size == 0) {
              ok = false;  // empty list: a weightless one-node list above
            } else {
              const unsigned long long tri =
                  (unsigned long long)size * (unsigned long long)(size - 1) / 2ull;
              const long long hl = (long long)(tri - a.lsum[l]);
              if (a.ltails[l] != 1 || hl < 0 || hl >= size) {
                atomicOr(&a.lerr[l], a.ltails[l] != 1 ? kErrTails : kErrHead);
                ok = false;
              }
              h = (int)(base + hl);
            }
          } else {
            h = head_base + l;
            if (h >= N) {
              errbits |= kErrBase;
              ok = false;
            }
          }
          if (!ok) {
            store_pair(&a.link_out[item], -1, 0);
          } else if (is_static(h, N, log2B, seed)) {
            store_pair(&a.link_out[item], h >> log2B, 0);
          } else {
            x = h;
            sid = item;
            k = 0;
            steps = 0;
          }
        }
      }
    }
    if (need && sid >= 0) {
      in = fetch(x);
      // waited for here, or the loop below would wait for its stores as well
      asm volatile("" : "+v"(in.x), "+v"(in.y));
    }
    if (__ballot(!retired) == 0) break;
    // Up to kWalkBurst steps before looking for new work: when the steps hit
    // in cache (local layouts) the work-distribution code, not memory, would
    // otherwise set the pace; random layouts do not notice either way.
    for (int rep = 0; rep < kWalkBurst && sid >= 0; ++rep) {
      int y = in.x, w = in.y;
      bool tail;
      bool stop = false;  // y is a static splitter
      bool seen = false;  // (paired) a walk has been here: a malformed input
      if (kPaired) {
        seen = in.x < -1 && in.x >= INT32_MIN + N;
        tail = in.x == -1 || seen;
        y = in.x & INT32_MAX;
        if (seen) w = 0;
        if (seen) errbits |= kErrBase;
        stop = coded ? in.x < 0 : is_static(y, N, log2B, seed);
      } else if (kCoded) {
        tail = in.x == -1;
        y = in.x & INT32_MAX;
        if (!tail && y >= N) {  // a state: a malformed input led here twice
          errbits |= kErrRange;
          tail = true;
        }
        stop = coded ? in.x < 0 : is_static(y, N, log2B, seed);
      } else if (kLevel0) {
        const int s = in.x;
        const int xl = (int)(x - base);
        tail = (s == -1) | (s == xl);
        if (!tail && (unsigned)s >= (unsigned)size) {
          atomicOr(&a.lerr[lid], kErrRange);
          tail = true;
        }
        y = (int)(base + s);
      } else {
        tail = in.x == -1;
        if (!tail && (unsigned)in.x >= (unsigned)N) {
          errbits |= kErrBase;
          tail = true;
        }
      }
      if (!kCoded) stop = is_static(y, N, log2B, seed);
      // The next load before this node's store: a load is only waited for
      // together with the stores issued before it (2^20 random nodes, whose
      // longest sublist of about 90 steps sets the time: walks of 61 + 32 us,
      // 67 + 36 the other way round).
      if (!tail && !stop) in = fetch(y);
      if (kLevel0 && kPacked) a.work[x] = (sid << kbits) | k;
      else if (!seen) store_pair(&a.state[x], kPaired ? -2 - sid : sid, k);
      k += w;
      x = y;
      if (tail) {
        store_pair(&a.link_out[sid], -1, k);
        sid = -1;
      } else if (stop) {
        store_pair(&a.link_out[sid], y >> log2B, k);
        sid = -1;
      } else if (++steps >= max_walk) {
        const int t = atomicAdd(dyn, 1);
        if (t >= a.cap) {
          errbits |= kErrOverflow;
          store_pair(&a.link_out[sid], -1, k);
          sid = -1;
        } else {
          const int nid = r + a.L + t;
          store_pair(&a.link_out[sid], nid, k);
          sid = nid;
          k = 0;
          steps = 0;
        }
      }
    }
  }
  if (errbits) atomicOr(&ctl->err, errbits);
}

// ------------------------------------------------------ recorded walk
// Level 0 where in-place states do not pay.  The walk (lr_walk_rec) only reads
// the successors and records the nodes it meets, in strips of kStrip
// consecutive nodes of one sublist; lr_bin deals the recorded nodes, with
// their ranks, to bins of kBinNodes consecutive ids, and lr_place puts a bin's
// ranks in order in LDS and writes them.  Writing the state over each successor
// (lr_walk) makes every step a write of a 32-byte sector besides the read of a
// 128-byte line, and its random reads alone run 1.65 times as fast (2^26 random
// nodes: 1.21 ms against 1.99); what is recorded moves in whole lines.
//
// A batch whose lists each fit an XCD's L2 gains more.  Workgroup ids are dealt
// round-robin over the XCDs, and each XCD takes chunks of consecutive splitter
// blocks (and heads of lists, see lr_rec_chunks) from its own eighth
// of the nodes in order, so the lists its lanes walk at one time are a few
// neighbours, which stay in its L2.  Nothing but the hit rate depends on the
// mapping.  256 lists of 2^18 nodes, following successors: 69 G nodes/s over
// all XCDs, 220 G/s list by list.
//
// Strips are handed out in slabs of kSlab per wave, in order from one counter
// per group: the XCD of a batch, so that lr_bin finds slabs of neighbouring
// lists together, or all waves of one list.  A wave holds one slab ahead, so
// it never waits for the counter.
// First list of every chunk of kWalkChunk splitter blocks (a batch).  The heads of
// the lists that start in a group are dealt to its chunks in equal numbers, in
// order: about those of the chunk's own nodes where lists are spread evenly, and
// no more than that where many short or empty ones lie together, which one wave
// would take 64 at a time (1000 lists of 2^16 nodes and 4 * 10^6 empty ones in one
// place: 142 ms by place, 4.0 like this).
__global__ void __launch_bounds__(256) lr_rec_chunks(const int64_t* __restrict__ off, int L,
                                                     int nchunks, int log2_chunk,
                                                     int32_t* __restrict__ chunk_list) {
  const auto lists_below = [&](int64_t chunk) {  // lists that start before a chunk
    if (chunk >= nchunks) return L;
    int lo = 0, hi = L;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (off[mid] < chunk << log2_chunk) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  for (int c = blockIdx.x * 256 + threadIdx.x; c <= nchunks; c += gridDim.x * 256) {
    int g = 0;  // the chunk's group
    while (g < kXcds - 1 && c >= record_group_chunk(nchunks, g + 1)) ++g;
    const int64_t first = record_group_chunk(nchunks, g), end = record_group_chunk(nchunks, g + 1);
    const int64_t la = lists_below(first), lb = lists_below(end);
    chunk_list[c] = c >= end ? (int)lb : (int)(la + (lb - la) * (c - first) / (end - first));
  }
}

template <bool kBatched, bool kPaired>
__global__ void __launch_bounds__(256) lr_walk_rec(WalkArgs a, RecArgs rec) {
  LrCtl* ctl = a.ctl;
  const int N = ctl->lv[0].n;
  if (!kBatched && rec.if_far && !far_chosen(ctl, N)) return;
  const int log2B = rec.log2B;
  const uint32_t seed = a.seed;
  const int r = (int)(((int64_t)N + (1 << log2B) - 1) >> log2B);
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->lv[0].r = r;
  int* dyn = &ctl->lv[0].dyn;
  const int nchunks = (r + kWalkChunk - 1) / kWalkChunk;
  const int home = blockIdx.x % kXcds;
  // the wave's chunks: every waves-th of its XCD's range
  const int waves = gridDim.x / kXcds * (256 / kWave);
  const int range_hi = (int)record_group_chunk(nchunks, home + 1);
  int chunk = (int)record_group_chunk(nchunks, home) + blockIdx.x / kXcds * (256 / kWave) +
              threadIdx.x / kWave;
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  // the current chunk: static splitters first .. first + statics - 1, then the
  // heads of the lists la .. la + heads - 1; next of them to be taken
  int first = 0, statics = 0, la = 0, heads = 0, next = 0;
  int slab = -1, cursor = kSlab;    // the wave's slab and the strips used of it
  const int group = kBatched ? home : 0;
  int ahead_slab = 0;               // in lane 0: the group's slab taken ahead
  if (lane_id() == 0) ahead_slab = atomicAdd(&rec.ctl->taken[group], 1);
  int ahead_la = 0, ahead_lb = 0;   // lists of the next chunk, read early
  if (kBatched && chunk < range_hi) {
    ahead_la = rec.chunk_list[chunk];
    ahead_lb = rec.chunk_list[chunk + 1];
  }

  int sid = -1, x = 0, k = 0, steps = 0;
  int errbits = 0;
  for (;;) {
    for (;;) {
      const bool idle = sid < 0;
      const uint64_t idle_mask = __ballot(idle);
      if (idle_mask == 0) break;
      if (next >= statics + heads) {  // the chunk is used up
        if (chunk >= range_hi) break;
        first = chunk * kWalkChunk;
        statics = min(kWalkChunk, r - first);
        next = 0;
        if (kBatched) {
          la = __builtin_amdgcn_readfirstlane(ahead_la);
          heads = __builtin_amdgcn_readfirstlane(ahead_lb) - la;
        } else {
          heads = chunk == 0 ? 1 : 0;
        }
        chunk += waves;
        if (kBatched && chunk < range_hi) {
          ahead_la = rec.chunk_list[chunk];
          ahead_lb = rec.chunk_list[chunk + 1];
        }
      }
      const int item = next + lanes_below(idle_mask);
      const int end = statics + heads;
      next = min(end, next + (int)__popcll(idle_mask));
      if (idle && item < statics) {
        const int block = first + item;
        const int start = block << log2B;
        x = start + (int)splitter_offset((uint32_t)block, seed,
                                         (uint32_t)min(1 << log2B, N - start));
        sid = block;
        k = steps = 0;
      } else if (idle && item < end) {  // the virtual splitter at a list's head
        const int l = la + item - statics;
        const int64_t base = kBatched ? a.off[l] : 0;
        const int size = kBatched ? (int)(a.off[l + 1] - base) : N;
        if (size == 0) {
          store_pair(&a.link_out[r + l], -1, 0);
        } else {
          const unsigned long long tri =
              (unsigned long long)size * (unsigned long long)(size - 1) / 2ull;
          const long long h = (long long)(tri - a.lsum[l]);
          if (a.ltails[l] != 1 || h < 0 || h >= size) {
            atomicOr(&a.lerr[l], a.ltails[l] != 1 ? kErrTails : kErrHead);
            store_pair(&a.link_out[r + l], -1, 0);
          } else if (is_static((int)(base + h), N, log2B, seed)) {
            store_pair(&a.link_out[r + l], (int)(base + h) >> log2B, 0);
          } else {
            x = (int)(base + h);
            sid = r + l;
            k = steps = 0;
          }
        }
      }
    }
    // kStrip steps, kept in registers
    const uint64_t walking = __ballot(sid >= 0);
    if (walking == 0) break;  // nothing left to take either
    const bool walks = sid >= 0;
    const int k0 = k;
    bool over = !walks;
    int node[kStrip], before[kStrip];
#pragma unroll
    for (int t = 0; t < kStrip; ++t) {
      node[t] = over ? -1 : x;
      before[t] = k;
      if (!over) {
        if (kPaired) {
          const int2 in = a.state[x];
          x = in.x;
          k += in.y;
        } else {
          x = a.work[x];
          ++k;
        }
        ++steps;
        over = x < 0;
      }
    }
    if (walks && over)  // at a tail or the next static splitter
      store_pair(&a.link_out[sid], x == -1 ? -1 : (x & INT32_MAX) >> log2B, k);
    // the strips of the walking lanes; those past the slab's end go to a new one
    const int count = (int)__popcll(walking);
    const int mine = cursor + lanes_below(walking);
    int strip = mine < kSlab ? slab * kSlab + mine : -1;
    if (cursor + count > kSlab) {
      const int fresh = __builtin_amdgcn_readfirstlane(ahead_slab);
      if (lane_id() == 0) {
        if (slab >= 0) rec.used[slab] = kSlab;
        ahead_slab = atomicAdd(&rec.ctl->taken[group], 1);
      }
      slab = fresh < rec.group_slabs ? group * rec.group_slabs + fresh : -1;
      if (strip < 0 && slab >= 0) strip = slab * kSlab + (mine - kSlab);
      cursor -= kSlab;
      if (slab < 0) cursor = kSlab - count;  // no slab: only a malformed input gets here
    }
    cursor += count;
    if (walks) {
      if (strip >= 0) {
        int4* const to = rec.strips + strip_word(strip);
        int4* const to_before = rec.before + strip_word(strip);
#pragma unroll
        for (int t = 0; t < kStrip / 4; ++t)
          to[t * kSlab] =
              make_int4(node[4 * t], node[4 * t + 1], node[4 * t + 2], node[4 * t + 3]);
        if (kPaired)
#pragma unroll
          for (int t = 0; t < kStrip / 4; ++t)
            to_before[t * kSlab] =
                make_int4(before[4 * t], before[4 * t + 1], before[4 * t + 2], before[4 * t + 3]);
        rec.head[strip] = make_int2(sid, k0);
      } else {
        errbits |= kErrOverflow;
        if (!over) store_pair(&a.link_out[sid], -1, k);
        over = true;
      }
      if (!over && steps >= a.max_walk) {  // cut: the node reached becomes a splitter
        const int t = atomicAdd(dyn, 1);
        if (t >= a.cap) {
          errbits |= kErrOverflow;
          store_pair(&a.link_out[sid], -1, k);
          over = true;
        } else {
          const int nid = r + a.L + t;
          store_pair(&a.link_out[sid], nid, k);
          sid = nid;
          k = 0;
          steps = 0;
        }
      }
      if (over) sid = -1;
    }
  }
  if (lane_id() == 0) {
    if (slab >= 0) rec.used[slab] = cursor;
    if (ahead_slab < rec.group_slabs) rec.used[group * rec.group_slabs + ahead_slab] = 0;
  }
  if (errbits) atomicOr(&ctl->err, errbits);
}

// Deals the recorded nodes to bins: an entry of node and rank for every node,
// where rank = rank of the strip's sublist + place in it.  A bin's region of
// `ent` holds one entry per node of the bin, which a valid input fills exactly.
// A tile of kTileSlabs slabs, a strip a thread, is sorted by bin in LDS, so that
// its entries reach a bin as one run.  kTileBins bins from the tile's lowest on
// are sorted; entries past them (slabs of distant lists in one tile) go to
// their bins one by one.
//
// kWord: the entry is one word, rank << bin_shift | node's place in the bin.
// Batches of lists of up to kWordLongest nodes take it, with bins of
// 2^(32 - bits of the longest list's ranks) nodes.  lr_bin and lr_place move 4
// bytes a node for the strips, 4 for the ranks and twice the entry, so the word
// instead of a {node, rank} pair takes them from 1400 + 1264 us to 1310 + 629
// (4096 lists of 2^6..2^20 nodes).  Beyond kWordLongest the bins are so small
// that kTileBins of them no longer cover the lists of a tile (100 lists of
// 2^17..2^20.9 nodes, 21 bits: lr_bin 217 us with pairs, 920 with words); one
// list's ranks take up to 26 bits, and weights 32.
template <bool kBatched, bool kToTail, bool kPaired, bool kWord = false>
__global__ void __launch_bounds__(kTileThreads) lr_bin(RecArgs rec,
                                                       const int32_t* __restrict__ srank,
                                                       const int64_t* __restrict__ off, int L,
                                                       int cap_here, LrCtl* ctl) {
  using Entry = std::conditional_t<kWord, uint32_t, uint2>;
  __shared__ Entry ent[kTileThreads * kStrip];
  __shared__ uint16_t bin_of[kWord ? kTileThreads * kStrip : 1];
  Entry* const out = static_cast<Entry*>(rec.ent);
  const int shift = kWord ? rec.bin_shift : kBinShift;
  const int bin_nodes = 1 << shift;
  const auto entry = [&](int node, int rank) {
    if constexpr (kWord) return (uint32_t)rank << shift | (uint32_t)(node & (bin_nodes - 1));
    else return make_uint2((unsigned)node, (unsigned)rank);
  };
  __shared__ int hist[kTileBins], start[kTileBins];
  __shared__ int wsum[kTileThreads / kWave];
  __shared__ int low, total;
  const int N = ctl->lv[0].n;
  if (!kBatched && rec.if_far && !far_chosen(ctl, N)) return;
  const int Nup = level_nodes(ctl, 1, L, cap_here);
  const int tid = threadIdx.x;
  const int groups = kBatched ? kXcds : 1;
  const int group = blockIdx.x % groups;
  const int taken = min(rec.ctl->taken[group], rec.group_slabs);
  bool bad = false;
  // the thread's strip of the tile at i0, read one tile ahead
  int ahead[kStrip], ahead_strip = 0;
  int2 ahead_head = make_int2(-1, 0);
  const auto fetch = [&](int i0) {
    ahead_head = make_int2(-1, 0);
    const int i = i0 + tid / kSlab;
    if (i < taken) {
      const int slab = group * rec.group_slabs + i;
      if (tid % kSlab < rec.used[slab]) {
        const int strip = slab * kSlab + tid % kSlab;
        ahead_head = rec.head[strip];
        const int4* const from = rec.strips + strip_word(strip);
        ahead_strip = strip;
#pragma unroll
        for (int t = 0; t < kStrip / 4; ++t) {
          const int4 v = from[t * kSlab];
          ahead[4 * t] = v.x;
          ahead[4 * t + 1] = v.y;
          ahead[4 * t + 2] = v.z;
          ahead[4 * t + 3] = v.w;
        }
      }
    }
  };
  const int step = gridDim.x / groups * kTileSlabs;
  const int begin = blockIdx.x / groups * kTileSlabs;
  if (begin < taken) fetch(begin);
  for (int i0 = begin; i0 < taken; i0 += step) {
    int node[kStrip], pos[kStrip], place[kStrip];  // place: in the sublist
    const int2 h = ahead_head;
    const bool have = h.x >= 0;
    const bool known = (unsigned)h.x < (unsigned)Nup;
    bad |= have && !known;
#pragma unroll
    for (int t = 0; t < kStrip; ++t) {
      node[t] = known ? ahead[t] : -1;
      if (!kPaired) place[t] = kToTail ? -t : t;
    }
    if (kPaired) {  // (not read a tile ahead: the registers do not last)
      const int4* const from = rec.before + strip_word(ahead_strip);
#pragma unroll
      for (int t = 0; t < kStrip / 4; ++t) {
        const int4 v = have ? from[t * kSlab] : make_int4(0, 0, 0, 0);
        place[4 * t] = v.x;
        place[4 * t + 1] = v.y;
        place[4 * t + 2] = v.z;
        place[4 * t + 3] = v.w;
      }
    }
    int value = known ? srank[h.x] + (kPaired ? 0 : h.y) : 0;
    if (kToTail && known) {
      int size = N;
      if (kBatched) {
        const int l = find_instance(off, L, node[0]);
        size = (int)(off[l + 1] - off[l]);
      }
      value = size - 1 - value;
    }
    if (i0 + step < taken) fetch(i0 + step);
    if (tid == 0) low = INT32_MAX;
    for (int b = tid; b < kTileBins; b += kTileThreads) hist[b] = 0;
    __syncthreads();
    int lo = 0;  // (one list has kTileBins bins at most)
    if (kBatched) {
      int least = INT32_MAX;
#pragma unroll
      for (int t = 0; t < kStrip; ++t)
        if (node[t] >= 0) least = min(least, node[t] >> shift);
      least = wave_min(least);
      if (lane_id() == 0) atomicMin(&low, least);
      __syncthreads();
      lo = low;
    }
#pragma unroll
    for (int t = 0; t < kStrip; ++t) {
      pos[t] = -1;
      if (node[t] >= 0) {
        const int b = (node[t] >> shift) - lo;
        if (b < kTileBins) {
          pos[t] = atomicAdd(&hist[b], 1);
        } else {
          const int at = atomicAdd(&rec.cursor[b + lo], 1);
          if (at < bin_nodes)
            out[((int64_t)(b + lo) << shift) + at] = entry(node[t], value + place[t]);
        }
      }
    }
    __syncthreads();
    // The bins' regions are asked for here and needed after the sort (lanes on
    // consecutive cursors).
    constexpr int kPer = kTileBins / kTileThreads;
    int to[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int b = tid + q * kTileThreads, c = hist[b];
      to[q] = 0;
      if (c) to[q] = atomicAdd(&rec.cursor[lo + b], c);
    }
    // exclusive prefix of the counts, kPer bins a thread
    int cnt[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      cnt[q] = hist[tid * kPer + q];
      sum += cnt[q];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int u = __shfl_up(incl, o, kWave);
      if (lane_id() >= o) incl += u;
    }
    if (lane_id() == kWave - 1) wsum[tid / kWave] = incl;
    __syncthreads();
    int excl = incl - sum;
    for (int w = 0; w < tid / kWave; ++w) excl += wsum[w];
    if (tid == kTileThreads - 1) total = excl + sum;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int b = tid * kPer + q;
      start[b] = excl;
      excl += cnt[q];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kStrip; ++t)
      if (pos[t] >= 0) {
        const int b = (node[t] >> shift) - lo;
        const int e = start[b] + pos[t];
        ent[e] = entry(node[t], value + place[t]);
        if (kWord) bin_of[e] = (uint16_t)b;
      }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {  // hist: from place in the tile to place in the bin
      const int b = tid + q * kTileThreads;
      hist[b] = to[q] - start[b];
    }
    __syncthreads();
    for (int e = tid; e < total; e += kTileThreads) {
      const Entry v = ent[e];
      int b;
      if constexpr (kWord) b = bin_of[e];
      else b = (int)(v.x >> shift) - lo;
      const int at = e + hist[b];
      if (at < bin_nodes) out[((int64_t)(lo + b) << shift) + at] = v;
    }
    __syncthreads();  // hist, start and ent are reused by the next tile
  }
  if (__ballot(bad) && lane_id() == 0) atomicOr(&ctl->err, kErrTotal);
}

// Ranks put in order in LDS and written, kBinNodes at a time (one bin or
// several).
template <bool kWord>
__global__ void __launch_bounds__(kTileThreads) lr_place(RecArgs rec, int32_t* __restrict__ rank,
                                                         LrCtl* ctl) {
  __shared__ int32_t out[kBinNodes];
  __shared__ int filled[kBinNodes >> kBinShiftMin];
  using Entry = std::conditional_t<kWord, uint32_t, uint2>;
  const int N = ctl->lv[0].n;
  if (rec.if_far && !far_chosen(ctl, N)) return;
  const int shift = kWord ? rec.bin_shift : kBinShift;
  const int nparts = (int)(((int64_t)N + kBinNodes - 1) >> kBinShift);
  for (int p = blockIdx.x; p < nparts; p += gridDim.x) {
    const int64_t v0 = (int64_t)p << kBinShift;
    const int size = (int)min<int64_t>(kBinNodes, N - v0);
    const int bins = (size + (1 << shift) - 1) >> shift;
    if ((int)threadIdx.x < bins) {
      const int b = threadIdx.x;
      const int f = rec.cursor[(v0 >> shift) + b];
      filled[b] = f;
      if (f != min(1 << shift, size - (b << shift))) atomicOr(&ctl->err, kErrTotal);
    }
    __syncthreads();
    const Entry* e = static_cast<const Entry*>(rec.ent) + v0;
    constexpr int kIn = kWord ? 16 : 8;  // entries in flight per thread
    for (int q0 = threadIdx.x; q0 < size; q0 += kIn * kTileThreads) {
      Entry v[kIn];
#pragma unroll
      for (int u = 0; u < kIn; ++u) {
        const int q = q0 + u * kTileThreads;
        if (q < size) v[u] = e[q];
      }
#pragma unroll
      for (int u = 0; u < kIn; ++u) {
        const int q = q0 + u * kTileThreads;
        const int place = q & ((1 << shift) - 1);
        if (q >= size || place >= filled[q >> shift]) continue;
        if constexpr (kWord)
          out[q - place + (v[u] & ((1u << shift) - 1))] = (int)(v[u] >> shift);
        else
          out[v[u].x & (kBinNodes - 1)] = (int)v[u].y;
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < size; q += kTileThreads) rank[v0 + q] = out[q];
    __syncthreads();
  }
}

// ------------------------------------------------- caller-chosen splitters
// Level 0 of one list with the splitters chosen by the caller (Section 3.2's
// random-versus-even comparison).  "Is y a splitter" is then no longer
// arithmetic: lr_mark_splitters overwrites each splitter's slot of the
// successor copy with the mark -(2 + splitter index) and keeps the
// successor it replaced, and the walk learns that it reached a splitter from
// the word it reads at the next node anyway.  Distinct ids leave exactly one
// mark per splitter; a repeated id or one out of range raises kErrSplitter.
__global__ void __launch_bounds__(256) lr_mark_splitters(int32_t* __restrict__ work,
                                                         const int32_t* __restrict__ splitters,
                                                         int r, int n, int32_t* __restrict__ ssucc,
                                                         int32_t* lerr) {
  bool bad = false;
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < r; s += gridDim.x * blockDim.x) {
    const int x = splitters[s];
    int old = -1;
    if ((unsigned)x >= (unsigned)n) {
      bad = true;
    } else {
      old = atomicExch(&work[x], -(2 + s));
      bad |= old <= -2;  // a second mark of one node
    }
    ssucc[s] = old;
  }
  if (__ballot(bad) && lane_id() == 0) atomicOr(lerr, kErrSplitter);
}

// The level-0 walk over marked splitters (one list, packed state).  A lane
// holds the node x it has reached and x's successor word sx, read one step
// earlier: it writes x's packed state over sx's slot, then reads the word of
// the successor, which tells whether that node is a splitter (a mark) or
// gives the next successor.  A splitter's own slot keeps its mark, which is
// its state (its sublist, offset 0) for the final scatter: the walker that
// arrives from its predecessor may read the mark at any time during the
// kernel.  Work distribution and cuts as in lr_walk.
__global__ void __launch_bounds__(1024) lr_walk_marked(WalkArgs a,
                                                       const int32_t* __restrict__ splitters,
                                                       const int32_t* __restrict__ ssucc, int r) {
  LrCtl* ctl = a.ctl;
  const int N = ctl->lv[0].n;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->lv[0].r = r;
  const int items = r + 1;  // chosen splitters, then the virtual one at the head
  int* dyn = &ctl->lv[0].dyn;
  __shared__ int wg_next;
  const int per = (int)(((int64_t)items + gridDim.x - 1) / gridDim.x);
  const int wg_lo = min(items, (int)((int64_t)blockIdx.x * per));
  const int wg_hi = min(items, wg_lo + per);
  if (threadIdx.x == 0) wg_next = wg_lo;
  __syncthreads();

  int sid = -1, x = 0, sx = 0, k = 0, steps = 0;
  bool at_mark = false;  // x is a chosen splitter: its slot keeps the mark
  bool retired = false;
  int errbits = 0;
  while (true) {
    const bool need = (sid < 0) & !retired;
    const uint64_t needm = __ballot(need);
    if (needm) {
      const int leader = __builtin_ctzll(needm);
      int first = 0;
      if (lane_id() == leader) first = atomicAdd(&wg_next, __popcll(needm));
      first = __shfl(first, leader);
      if (need) {
        const int item = first + lanes_below(needm);
        if (item >= wg_hi) {
          retired = true;
        } else if (item < r) {  // a chosen splitter
          const int y = splitters[item];
          if ((unsigned)y >= (unsigned)N) {  // reported by the marking pass
            store_pair(&a.link_out[item], -1, 0);
          } else {
            sid = item;
            x = y;
            sx = ssucc[item];
            k = 0;
            steps = 0;
            at_mark = true;
          }
        } else {  // the virtual splitter at the head
          const unsigned long long tri =
              (unsigned long long)N * (unsigned long long)(N - 1) / 2ull;
          const long long h = (long long)(tri - a.lsum[0]);
          if (a.ltails[0] != 1 || h < 0 || h >= N) {
            atomicOr(&a.lerr[0], a.ltails[0] != 1 ? kErrTails : kErrHead);
            store_pair(&a.link_out[item], -1, 0);
          } else {
            const int v = a.work[(int)h];
            if (v <= -2) {  // the head is a chosen splitter itself
              store_pair(&a.link_out[item], -(v + 2), 0);
            } else {
              sid = item;
              x = (int)h;
              sx = v;
              k = 0;
              steps = 0;
              at_mark = false;
            }
          }
        }
      }
    }
    if (__ballot(!retired) == 0) break;
    for (int rep = 0; rep < kWalkBurst && sid >= 0; ++rep) {
      bool tail = (sx == -1) | (sx == x);
      if (!tail && (unsigned)sx >= (unsigned)N) {
        atomicOr(&a.lerr[0], kErrRange);
        tail = true;
      }
      if (!at_mark) a.work[x] = (sid << a.kbits) | k;
      at_mark = false;
      ++k;
      if (tail) {
        store_pair(&a.link_out[sid], -1, k);
        sid = -1;
        continue;
      }
      const int y = sx;
      const int v = a.work[y];
      if (v <= -2) {
        // (an index past the level's nodes only comes from a malformed input
        // word, which the head-find pass has reported; level 1 bounds it)
        store_pair(&a.link_out[sid], -(v + 2), k);
        sid = -1;
      } else if (++steps >= a.max_walk) {
        const int t = atomicAdd(dyn, 1);
        if (t >= a.cap) {
          errbits |= kErrOverflow;
          store_pair(&a.link_out[sid], -1, k);
          sid = -1;
        } else {
          const int nid = r + 1 + t;
          store_pair(&a.link_out[sid], nid, k);
          sid = nid;
          k = 0;
          steps = 0;
          x = y;
          sx = v;
        }
      } else {
        x = y;
        sx = v;
      }
    }
  }
  if (errbits) atomicOr(&ctl->err, errbits);
}

// Longest level-0 sublist (stats only): the largest weight among the level-1
// nodes, which for unit weights is the node count of each sublist piece.
__global__ void __launch_bounds__(256) lr_sublist_max(const int2* __restrict__ link,
                                                      const LrCtl* ctl, int L, int cap0,
                                                      int32_t* out) {
  const int N1 = level_nodes(ctl, 1, L, cap0);
  int mx = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N1; j += gridDim.x * blockDim.x)
    mx = max(mx, link[j].y);
  mx = -wave_min(-mx);
  if (lane_id() == 0 && mx > 0) atomicMax(out, mx);
}

// ------------------------------------------------------------ base: LDS
// Ranks a weighted forest of at most kMaxCutoff nodes in one workgroup:
// predecessor links are built in LDS, then pointer jumping along them sums
// the weights of all earlier nodes (exclusive prefix from each head).  The
// heads must be exactly the ids head_base .. head_base + L - 1.
__global__ void __launch_bounds__(kBaseThreads) lr_base_lds(const int2* __restrict__ link,
                                                            int32_t* __restrict__ srank,
                                                            LrCtl* ctl, int level, int L,
                                                            int cap_prev) {
  __shared__ int lnk[kMaxCutoff];
  __shared__ int pre[kMaxCutoff];
  __shared__ int nheads;
  __shared__ int bad;
  __shared__ unsigned long long total;
  const int N = level_nodes(ctl, level, L, cap_prev);
  const int head_base = ctl->lv[level - 1].r;
  const int tid = threadIdx.x;
  if (tid == 0) {
    nheads = 0;
    bad = 0;
    total = 0ull;
  }
  if (N > kMaxCutoff) {
    if (tid == 0) atomicOr(&ctl->err, kErrBase);
    return;
  }
  for (int j = tid; j < N; j += kBaseThreads) lnk[j] = -1;
  __syncthreads();
  // All global loads of a phase are issued before any is used: one
  // workgroup alone cannot hide their latency otherwise.
  unsigned long long mytotal = 0;
  {
    int2 in[kPerThread];
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      in[t] = j < N ? link[j] : make_int2(-1, 0);
    }
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      if (j >= N) continue;
      mytotal += (unsigned)in[t].y;
      if (in[t].x >= 0 && in[t].x < N) {
        if (atomicExch(&lnk[in[t].x], j) != -1) bad = 1;
      } else if (in[t].x != -1) {
        bad = 1;
      }
    }
  }
  __syncthreads();
  int myheads = 0;
  {
    int pw[kPerThread];
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      const int p = j < N ? lnk[j] : -1;
      pw[t] = p >= 0 ? link[p].y : 0;
      if (j < N && p < 0) {
        ++myheads;
        if (j < head_base || j >= head_base + L) bad = 1;
      }
    }
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      if (j < N) pre[j] = pw[t];
    }
  }
  if (myheads) atomicAdd(&nheads, myheads);
  mytotal = wave_sum(mytotal);
  if (lane_id() == 0 && mytotal) atomicAdd(&total, mytotal);
  __syncthreads();
  int rounds = 0;
  while ((1 << rounds) < N) ++rounds;
  int pa[kPerThread], la[kPerThread];
  for (int it = 0; it < rounds; ++it) {
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      la[t] = -1;
      pa[t] = 0;
      if (j < N) {
        const int p = lnk[j];
        if (p >= 0) {
          pa[t] = pre[p];
          la[t] = lnk[p];
        } else {
          la[t] = -2;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      if (j < N && la[t] != -2) {
        pre[j] += pa[t];
        lnk[j] = la[t];
      }
    }
    __syncthreads();
  }
  for (int j = tid; j < N; j += kBaseThreads) {
    if (lnk[j] != -1) bad = 1;
    srank[j] = pre[j];
  }
  __syncthreads();
  if (tid == 0) {
    if (bad || nheads != L) atomicOr(&ctl->err, kErrBase);
    ctl->base_total = total;
  }
}

// The same for a few lists (at most kBaseLists), by the ruling set once more,
// inside LDS: one splitter per block of 4 or 8 ids and the heads; a thread walks
// its splitters' sublists, the splitters are ranked by pointer jumping, and a
// node gets its splitter's rank + its offset.  Jumping over all nodes takes
// ceil(log2 N) rounds of two LDS accesses a node, which set its time (12500
// nodes: 52 us, 35 with one splitter per 4 ids); here a node costs three
// accesses, and only a quarter or an eighth of the nodes jump.
//
// One workgroup runs it, so latency and its instruction count bound it: every
// phase issues its reads before it uses one, a walk reads its next node before
// it marks the last, each wave has its own share of the walks instead of a
// counter, and a wave skips the rows it has no part in (12500 nodes: 35 -> 21.7
// us, 8194: 29 -> 20).  A second workgroup of the same XCD reads the level into
// their L2 meanwhile, as one CU alone reads 9 bytes a clock from beyond it (2 us
// of 12500 nodes).  Blocks of 8 take more steps a walk and half the jumps (calls,
// blocks of 4 and of 8: one list of 5000 nodes 14.8 and 15.2 us, 7000 15.3 and
// 16.1, 9000 17.7 and 16.3, 10240 18.6 both, 12000 20.9 and 18.9, 16384 24.7 and
// 22.2; as bases, lists of 100003, 120000, 2^20 and 2^22 nodes 62.3 and 61.8, 64.2
// and 61.0, 125.6 and 126.1, 263.3 and 262.2).
//
// word[x]: {weight, next (| kStop)} at first; {offset, splitter | kSeen} once a walk has
// passed x; of a splitter {weight of its sublist, next splitter} after its walk
// and {weight of the sublists before it, ancestor} while jumping.
constexpr int kBaseBlock4 = 10240;  // blocks of 4 up to this many nodes
constexpr int kBaseLists = 1024;
constexpr int kEarlyRows = 2;
constexpr int kSeen = 1 << 30;
constexpr int kStop = 1 << 29;  // the next node is a splitter
constexpr int kEnd = kStop - 1;  // no next node (with kStop in a node's word)
constexpr unsigned long long kNoPred = ~0ull;

__device__ __forceinline__ unsigned long long pack_w(int hi, uint32_t lo) {
  return (unsigned long long)(unsigned)hi << 32 | lo;
}

// The splitter of block b (in the last block it may lie past the nodes: then
// there is none).
__device__ __forceinline__ int base_splitter(int b, int log2b) {
  return (b << log2b) + (int)(((unsigned)b % 65536 * 0x9E3779u >> 20) & ((1u << log2b) - 1));
}

// A node's first word; heads are ids head_base .. head_base + L - 1.
__device__ __forceinline__ unsigned long long base_word(int to, bool end, int weight, int log2b,
                                                        int head_base, int L) {
  const bool stop = end | ((unsigned)(to - head_base) < (unsigned)L) |
                    (base_splitter(to >> log2b, log2b) == to);
  return pack_w(weight, (end ? kEnd : to) | (stop ? kStop : 0));
}

// Ranks the N nodes whose first words lie in word[] (before a barrier) and
// hands each to emit(node, rank).  word[kMaxCutoff] is taken for their splitter
// by lanes without one.  Returns whether this thread saw that they are no L
// lists from those heads.
template <class Emit>
__device__ __forceinline__ int base_rank(unsigned long long* word, int N, int log2b, int head_base,
                                         int L, Emit emit) {
  const int tid = threadIdx.x;
  // the wave's first row entry: rows it has no part in are skipped as a whole
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  const auto is_head = [&](int x) { return (unsigned)(x - head_base) < (unsigned)L; };
  int bad = 0;
  __syncthreads();
  const int blocks = (N + (1 << log2b) - 1) >> log2b;
  // Walks: a lane takes a splitter, follows its successors to the next one and
  // leaves {sublist weight, next splitter or kEnd} in the splitter's word,
  // which no other walk reads.  (A branch leads to a node walked already, and a
  // cycle without a splitter to its own first node: either ends the walk.)
  {
    const int slots = blocks + L;
    constexpr int kWaves = kBaseThreads / kWave;
    const int per = (slots + kWaves - 1) / kWaves;
    int next = wave0 / kWave * per;
    const int last = min(slots, next + per);
    int own = -1, x = 0, acc = 0;
    unsigned long long w = 0;
    for (;;) {
      const uint64_t idle = __ballot(own < 0);
      if (idle && next < last) {
        const int slot = next + lanes_below(idle);
        next += (int)__popcll(idle);
        if (own < 0 && slot < last) {
          const int at = slot < blocks ? base_splitter(slot, log2b) : head_base + slot - blocks;
          // (a head may be its block's splitter)
          if (slot < blocks ? at < N : base_splitter(at >> log2b, log2b) != at) {
            own = x = at;
            acc = 0;
            w = word[x];
          }
        }
      } else if (idle == ~0ull) {
        break;
      }
#pragma unroll
      for (int rep = 0; rep < 4; ++rep)
        if (own >= 0) {
          const int to = (int)(uint32_t)w;
          const bool end = to & (kSeen | kStop);
          const unsigned long long mark = pack_w(acc, (uint32_t)(own | kSeen));
          const int at = x;
          acc += (int)(w >> 32);
          x = end ? own : to;
          w = word[x];
          word[at] = mark;
          if (end) {
            word[own] = pack_w(acc, (to & kSeen) ? kEnd : to & ~kStop);
            bad |= to & kSeen;
            own = -1;
          }
        }
    }
  }
  __syncthreads();
  // the thread's splitters: one per row of blocks, then one head
  constexpr int kRows =
      (std::max(kBaseBlock4 / 4, kMaxCutoff / 8) + kBaseThreads - 1) / kBaseThreads + 1;
  constexpr int kNone = kMaxCutoff;
  int mine[kRows];
  unsigned long long at[kRows];
  const auto row = [&](int t) {
    return t < kRows - 1 ? t * kBaseThreads + wave0 < blocks : wave0 < L;
  };
#pragma unroll
  for (int t = 0; t < kRows; ++t)
    if (row(t)) {
      const int b = tid + t * kBaseThreads, h = head_base + tid;
      const int x = t < kRows - 1 ? base_splitter(b, log2b) : h;
      const bool is = t < kRows - 1 ? b < blocks && x < N
                                    : tid < L && base_splitter(h >> log2b, log2b) != h;
      mine[t] = is ? x : kNone;
      at[t] = is ? word[x] : pack_w(0, kEnd);
    }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kRows; ++t)
    if (row(t))
      word[mine[t]] = is_head(mine[t]) || mine[t] == kNone ? pack_w(0, (uint32_t)mine[t]) : kNoPred;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kRows; ++t)
    if (row(t) && (uint32_t)at[t] != kEnd)
      bad |= atomicExch(&word[(uint32_t)at[t]],
                        pack_w((int)(at[t] >> 32), (uint32_t)mine[t])) != kNoPred;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kRows; ++t)
    if (row(t)) at[t] = word[mine[t]];
  // (a malformed forest may leave splitters without predecessor: they jump
  // nowhere)
#pragma unroll
  for (int t = 0; t < kRows; ++t)
    if (row(t) && at[t] == kNoPred) {
      bad = 1;  // a head that is no list's
      word[mine[t]] = at[t] = pack_w(0, (uint32_t)mine[t]);
    }
  __syncthreads();
  for (int span = 1; span < blocks + L; span *= 2) {
    unsigned long long up[kRows];
#pragma unroll
    for (int t = 0; t < kRows; ++t)
      if (row(t)) up[t] = word[(uint32_t)at[t]];
#pragma unroll
    for (int t = 0; t < kRows; ++t)
      if (row(t) && (uint32_t)up[t] != (uint32_t)at[t]) {
        at[t] = pack_w((int)(at[t] >> 32) + (int)(up[t] >> 32), (uint32_t)up[t]);
        word[mine[t]] = at[t];
      }
    __syncthreads();
  }
  unsigned long long w[kPerThread], of[kPerThread];
#pragma unroll
  for (int t = 0; t < kPerThread; ++t)
    if (t * kBaseThreads + wave0 < N) w[t] = word[tid + t * kBaseThreads];
#pragma unroll
  for (int t = 0; t < kPerThread; ++t)
    if (t * kBaseThreads + wave0 < N) {
      of[t] = w[t];
      if ((uint32_t)w[t] & kSeen) of[t] = word[(uint32_t)w[t] ^ kSeen];
      else w[t] = 0;
    }
  // (the word of a node that no walk came by leads to no head: the next node,
  // kStop added to a head, or kEnd)
#pragma unroll
  for (int t = 0; t < kPerThread; ++t) {
    const int j = tid + t * kBaseThreads;
    if (j >= N) continue;
    bad |= !is_head((int)(uint32_t)of[t]);
    emit(j, (int)(of[t] >> 32) + (int)(w[t] >> 32));
  }
  return bad;
}

// Reads one node per 128-byte line, to have them in this XCD's L2.
template <class T>
__device__ __forceinline__ void read_ahead(const T* p, int n) {
  constexpr int kPerLine = 128 / sizeof(T);
  int any = 0;
  for (int j = threadIdx.x * kPerLine; j < n; j += kPerLine * kBaseThreads)
    any |= *reinterpret_cast<const int*>(p + j);
  asm volatile("" ::"v"(any));  // that the loads are kept
}

// `bound` nodes may be read of link, whatever the level's node count.
__global__ void __launch_bounds__(kBaseThreads) lr_base_walk(const int2* __restrict__ link,
                                                             int32_t* __restrict__ srank,
                                                             LrCtl* ctl, int level, int L,
                                                             int cap_prev, int bound) {
  if (blockIdx.x > 0) {
    if (blockIdx.x % kXcds == 0)
      read_ahead(link, min(bound, level_nodes(ctl, level, L, cap_prev)));
    return;
  }
  __shared__ unsigned long long word[kMaxCutoff + 1];
  __shared__ unsigned long long total;
  const int tid = threadIdx.x;
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  int2 in[kPerThread];  // the first rows while the node count is on its way
  const auto read = [&](int t, int limit) {
    const int j = tid + t * kBaseThreads;
    in[t] = j < limit ? link[j] : make_int2(-1, 0);
  };
#pragma unroll
  for (int t = 0; t < kEarlyRows; ++t) read(t, bound);
  const int N = level_nodes(ctl, level, L, cap_prev);
#pragma unroll
  for (int t = kEarlyRows; t < kPerThread; ++t) read(t, min(N, bound));
  const int head_base = ctl->lv[level - 1].r;
  if (tid == 0) total = 0ull;
  if (N > min(kMaxCutoff, bound) || head_base + L > N) {
    if (tid == 0) atomicOr(&ctl->err, kErrBase);
    return;
  }
  const int log2b = N <= kBaseBlock4 ? 2 : 3;
  int bad = 0;
  unsigned long long mytotal = 0;
#pragma unroll
  for (int t = 0; t < kPerThread; ++t)
    if (t * kBaseThreads + wave0 < N) {
      const int j = tid + t * kBaseThreads;
      const int to = j < N ? in[t].x : -1;
      const int weight = j < N ? in[t].y : 0;
      const bool end = (unsigned)to >= (unsigned)N;
      bad |= end & (to != -1);
      mytotal += (unsigned)weight;
      word[j] = base_word(to, end, weight, log2b, head_base, L);
    }
  bad |= base_rank(word, N, log2b, head_base, L, [&](int j, int rank) { srank[j] = rank; });
  mytotal = wave_sum(mytotal);
  if (lane_id() == 0 && mytotal) atomicAdd(&total, mytotal);
  if (bad) atomicOr(&ctl->err, kErrBase);
  __syncthreads();
  if (tid == 0) ctl->base_total = total;
}

// One whole list of at most kMaxCutoff nodes, weighted or not, in the same way
// and in one kernel: the head is what the sum of the successors leaves out.
// succ is read before any rank is written (in place allowed).  Bound as
// lr_base_walk is, and by the call itself below 2000 nodes.  Unweighted lists of
// up to kOneList nodes are left to lr_lds, whose jumps need no head and no walks
// (a call of 2000 nodes 11.9 us here, 10.4 there; 4096: 12.8 both; 6000: 14.3
// and 15.5; 16384: 21.1 and 28.1).  Weighted lists took a kernel to clear two
// words and one that jumped over every node with weights and links apart: 28 us
// for 100 to 2000 nodes, 71.5 for 16383, and here 10.8 to 11.8, and 21.2.
constexpr int kOneList = 4096;

__global__ void __launch_bounds__(kBaseThreads) lr_one_lds(const int32_t* succ,
                                                           const int32_t* __restrict__ weight,
                                                           int n, int to_tail, int32_t* rank,
                                                           int32_t* lerr, int32_t* status) {
  if (blockIdx.x > 0) {
    if (blockIdx.x % kXcds == 0) {
      read_ahead(succ, n);
      if (weight) read_ahead(weight, n);
    }
    return;
  }
  __shared__ unsigned long long word[kMaxCutoff + 1];
  __shared__ unsigned long long sum;
  __shared__ int tails, wrong;
  const int tid = threadIdx.x;
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  int to[kPerThread], w[kPerThread];
#pragma unroll
  for (int t = 0; t < kPerThread; ++t) {
    const int j = tid + t * kBaseThreads;
    to[t] = j < n ? succ[j] : -1;
    w[t] = j < n ? weight ? weight[j] : 1 : 0;
  }
  if (tid == 0) {
    sum = 0;
    tails = wrong = 0;
  }
  __syncthreads();
  {
    unsigned long long mine = 0;
    int ends = 0, bad = 0;
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      if (to[t] == j) to[t] = -1;
      ends += j < n && to[t] == -1;
      bad |= to[t] < -1 || to[t] >= n;
      mine += to[t] > 0 ? to[t] : 0;
    }
    mine = wave_sum(mine);
    ends = wave_sum(ends);
    if (lane_id() == 0) {
      atomicAdd(&sum, mine);
      atomicAdd(&tails, ends);
    }
    if (bad) wrong = 1;
  }
  __syncthreads();
  const long long head = (long long)n * (n - 1) / 2 - (long long)sum;
  int bad = tails != 1 || wrong || head < 0 || head >= n;
  if (!bad) {
    const int log2b = n <= kBaseBlock4 ? 2 : 3;
#pragma unroll
    for (int t = 0; t < kPerThread; ++t)
      if (t * kBaseThreads + wave0 < n)
        word[tid + t * kBaseThreads] =
            base_word(to[t], to[t] == -1, w[t], log2b, (int)head, 1);
    bad = base_rank(word, n, log2b, (int)head, 1,
                    [&](int j, int r) { rank[j] = to_tail ? n - 1 - r : r; });
    if (bad) wrong = 1;
  }
  __syncthreads();
  if (tid == 0) {
    const bool ok = tails == 1 && !wrong && head >= 0 && head < n;
    if (status) status[0] = ok ? PJ_OK : PJ_EBADLIST;
    if (lerr) lerr[0] = ok ? 0 : kErrBase;
  }
}

// ---------------------------------------------------- base: device-wide
// The same predecessor pointer jumping for forests too large for one
// workgroup, one launch per round; (prefix, link) pairs are packed into one
// 64-bit word so a gather reads a consistent pair.
__device__ __forceinline__ unsigned long long pack_pl(int prefix, int lnk) {
  return ((unsigned long long)(unsigned)prefix << 32) | (unsigned)lnk;
}

__global__ void wide_clear(int32_t* lnk, const LrCtl* ctl, int level, int L, int cap_prev) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x)
    lnk[j] = -1;
}

__global__ void wide_pred(const int2* __restrict__ link, int32_t* lnk, LrCtl* ctl, int level,
                          int L, int cap_prev) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  int bad = 0;
  unsigned long long tot = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const int2 in = link[j];
    tot += (unsigned)in.y;
    if (in.x >= 0 && in.x < N) {
      if (atomicExch(&lnk[in.x], j) != -1) bad = 1;
    } else if (in.x != -1) {
      bad = 1;
    }
  }
  tot = wave_sum(tot);
  if (lane_id() == 0 && tot) atomicAdd(&ctl->base_total, tot);
  if (bad) atomicOr(&ctl->err, kErrBase);
}

__global__ void wide_init(const int2* __restrict__ link, const int32_t* __restrict__ lnk,
                          unsigned long long* pl, LrCtl* ctl, int level, int L, int cap_prev) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  const int head_base = ctl->lv[level - 1].r;
  int bad = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const int p = lnk[j];
    if (p < 0 && (j < head_base || j >= head_base + L)) bad = 1;
    pl[j] = pack_pl(p >= 0 ? link[p].y : 0, p);
  }
  if (bad) atomicOr(&ctl->err, kErrBase);
}

__global__ void wide_jump(unsigned long long* pl, const LrCtl* ctl, int level, int L,
                          int cap_prev) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const unsigned long long v = pl[j];
    const int p = (int)(unsigned)v;
    if (p < 0) continue;
    const unsigned long long q = pl[p];
    const int pre = (int)(v >> 32) + (int)(q >> 32);
    pl[j] = pack_pl(pre, (int)(unsigned)q);
  }
}

__global__ void wide_final(const unsigned long long* __restrict__ pl, int32_t* srank, LrCtl* ctl,
                           int level, int L, int cap_prev) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  int bad = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const unsigned long long v = pl[j];
    if ((int)(unsigned)v != -1) bad = 1;
    srank[j] = (int)(v >> 32);
  }
  if (bad) atomicOr(&ctl->err, kErrBase);
}

// ---------------------------------------------------------------- expand
// rank of node x = rank of its splitter + weight before x in its sublist.
__global__ void __launch_bounds__(256) lr_expand(const int2* __restrict__ state,
                                                 const int32_t* __restrict__ srank_up,
                                                 int32_t* __restrict__ out, LrCtl* ctl, int level,
                                                 int L, int cap_prev, int cap_here) {
  const int N = level_nodes(ctl, level, L, cap_prev);
  const int Nup = level_nodes(ctl, level + 1, L, cap_here);
  int bad = 0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < N; j += gridDim.x * blockDim.x) {
    const int2 s = state[j];
    int v = 0;
    if ((unsigned)s.x < (unsigned)Nup) v = srank_up[s.x] + s.y;
    else bad = 1;
    out[j] = v;
  }
  if (bad) atomicOr(&ctl->err, kErrTotal);
}

// Level 0: write the output ranks (from the head, or to the tail).
constexpr int kExpandPer = 4;
template <bool kBatched, bool kToTail, bool kPacked>
__global__ void __launch_bounds__(256) lr_expand0(const int2* __restrict__ state,
                                                  const int32_t* __restrict__ srank_up,
                                                  int32_t* rank,
                                                  const int64_t* __restrict__ off, LrCtl* ctl,
                                                  int L, int cap_here, int kbits_near,
                                                  int kbits_far, int if_near) {
  const int N = ctl->lv[0].n;
  if (if_near && far_chosen(ctl, N)) return;
  // the walk's choice of packing (see lr_walk), from the same count
  const int kbits = kbits_far > 0 && far_chosen(ctl, N) ? kbits_far : kbits_near;
  const int Nup = level_nodes(ctl, 1, L, cap_here);
  int bad = 0;
  // kExpandPer nodes per thread per pass, loads first: the splitter-rank
  // gathers of one thread are in flight together.  The packed words are read
  // once and overwritten, so they are streamed past the cache (nontemporal)
  // and the gathered splitter ranks keep it.
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j0 < N;
       j0 += kExpandPer * stride) {
    int2 s[kExpandPer];
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) {
      const int64_t j = j0 + u * stride;
      s[u] = make_int2(-1, 0);
      if (j < N) {
        if (kPacked) {
          // a packed (sublist, offset) word, or the mark -(2 + splitter) that
          // a caller-chosen splitter keeps (its sublist, offset 0)
          const int w = __builtin_nontemporal_load(&rank[j]);
          s[u] = w >= 0 ? make_int2((int)((unsigned)w >> kbits), w & ((1 << kbits) - 1))
                        : make_int2(-(w + 2), 0);
        } else {
          s[u] = state[j];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) {
      const int64_t j = j0 + u * stride;
      if (j >= N) break;
      int v = 0;
      if ((unsigned)s[u].x < (unsigned)Nup) v = srank_up[s[u].x] + s[u].y;
      else bad = 1;
      if (kToTail) {
        int size = N;
        if (kBatched) {
          const int l = find_instance(off, L, j);
          size = (int)(off[l + 1] - off[l]);
        }
        v = size - 1 - v;
      }
      __builtin_nontemporal_store(v, &rank[j]);
    }
  }
  if (bad) atomicOr(&ctl->err, kErrTotal);
}

// Level 0 of a paired walk: rank = rank of the sublist + weight before the node.
// A pair no walk came by (a cycle beside the list) is reported.
__global__ void __launch_bounds__(256) lr_expand0_paired(const int2* __restrict__ state,
                                                         const int32_t* __restrict__ srank_up,
                                                         int32_t* __restrict__ rank, LrCtl* ctl,
                                                         int L, int cap_here, int if_near) {
  const int N = ctl->lv[0].n;
  if (if_near && far_chosen(ctl, N)) return;
  const int Nup = level_nodes(ctl, 1, L, cap_here);
  int bad = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j0 < N;
       j0 += kExpandPer * stride) {
    int2 s[kExpandPer];
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) {
      const int64_t j = j0 + u * stride;
      s[u] = j < N ? state[j] : make_int2(-1, 0);
    }
#pragma unroll
    for (int u = 0; u < kExpandPer; ++u) {
      const int64_t j = j0 + u * stride;
      if (j >= N) break;
      const int sid = -2 - s[u].x;
      const bool ok = s[u].x < -1 && s[u].x >= INT32_MIN + N && sid < Nup;
      rank[j] = ok ? srank_up[sid] + s[u].y : 0;
      bad |= !ok;
    }
  }
  if (bad) atomicOr(&ctl->err, kErrTotal);
}

// ------------------------------------------------ per-node batched passes
// Calls f(g, l, base, size) for every node g of a batch, with l its list.
// Each wave owns a contiguous run of chunks of kWave * kListedPer nodes: one
// search of the offset table per wave, then every lane follows the list
// boundaries forward (a search per node costs a chain of dependent loads).
// Lanes of a wave touch consecutive nodes, so accesses stay coalesced.
constexpr int kListedPer = 16;
template <class F>
__device__ __forceinline__ void for_each_listed(const int64_t* __restrict__ off, int L, int64_t n,
                                                F f) {
  constexpr int64_t kChunk = kWave * kListedPer;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int nwaves = (gridDim.x * blockDim.x) / kWave;
  const int lane = lane_id();
  const int64_t nchunks = (n + kChunk - 1) / kChunk;
  const int64_t per = (nchunks + nwaves - 1) / nwaves;
  const int64_t ci0 = (int64_t)wave * per;
  const int64_t ci1 = ci0 + per < nchunks ? ci0 + per : nchunks;
  if (ci0 >= ci1) return;
  int l = find_instance(off, L, ci0 * kChunk);
  int64_t base = off[l], end = off[l + 1];
  for (int64_t ci = ci0; ci < ci1; ++ci)
    for (int t = 0; t < kListedPer; ++t) {
      const int64_t g = ci * kChunk + t * kWave + lane;
      if (g >= n) break;
      while (g >= end) {  // later lists (empty ones skipped)
        ++l;
        base = end;
        end = off[l + 1];
      }
      f(g, l, base, (int)(end - base));
    }
}

// --------------------------------------------------------------- Wyllie
// Pointer jumping (Section 3.1) on packed (distance to tail, next) pairs:
// one 64-bit read of the node's own pair, one 64-bit gather of its next's
// pair, one 64-bit write.  Updating in place is safe: a gather that sees a
// pair already advanced in this round still holds a consistent
// (distance, next) relation, only a longer jump.
__device__ __forceinline__ unsigned long long pack_dn(int dist, int next) {
  return ((unsigned long long)(unsigned)dist << 32) | (unsigned)next;
}

template <bool kBatched>
__global__ void __launch_bounds__(1024) wy_init(const int32_t* __restrict__ succ,
                                                const int64_t* __restrict__ off, int L, int n,
                                                unsigned long long* __restrict__ pair,
                                                int32_t* lerr) {
  auto one = [&](int64_t g, int l, int64_t base, int size) {
    const int s = succ[g];
    const int xl = (int)(g - base);
    bool tail = (s == -1) | (s == xl);
    if (!tail && (unsigned)s >= (unsigned)size) {
      atomicOr(&lerr[l], kErrRange);
      tail = true;
    }
    pair[g] = tail ? pack_dn(0, -1) : pack_dn(1, (int)(base + s));
  };
  if (kBatched) {
    for_each_listed(off, L, n, one);
  } else {
    const int stride = gridDim.x * blockDim.x;
    for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += stride) one(g, 0, 0, n);
  }
}

__global__ void __launch_bounds__(1024) wy_jump(unsigned long long* __restrict__ pair, int n) {
  const int stride = gridDim.x * blockDim.x;
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += stride) {
    const unsigned long long v = pair[g];
    const int nx = (int)(unsigned)v;
    if (nx < 0) continue;
    const unsigned long long q = pair[nx];
    pair[g] = pack_dn((int)(v >> 32) + (int)(q >> 32), (int)(unsigned)q);
  }
}

template <bool kBatched, bool kToTail>
__global__ void __launch_bounds__(1024) wy_final(const unsigned long long* __restrict__ pair,
                                                 const int64_t* __restrict__ off, int L, int n,
                                                 int32_t* __restrict__ rank, int32_t* lerr) {
  auto one = [&](int64_t g, int l, int64_t, int size) {
    const unsigned long long v = pair[g];
    const int dist = (int)(v >> 32);
    if ((int)(unsigned)v != -1) atomicOr(&lerr[l], kErrBase);
    rank[g] = kToTail ? dist : size - 1 - dist;
  };
  if (kBatched) {
    for_each_listed(off, L, n, one);
  } else {
    const int stride = gridDim.x * blockDim.x;
    for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += stride) one(g, 0, 0, n);
  }
}

// ------------------------------------------------- one workgroup's lists
// Lists short enough for LDS: a workgroup reads its lists' successors once,
// ranks them by pointer jumping in LDS and writes the ranks, one kernel in all.
// A node's word (lds_rules.hpp) holds the distance to the node it has jumped to
// and that node, so a jump is one LDS read and one write.  Jumping in place is
// safe: whatever version of a word a jump reads is a true distance (modulo 2^16
// on the way round a cycle).  A list is one list exactly if no successor is out of
// range and some node is size - 1 steps away from a tail; the words tell that
// by a mark that only a tail hands out, as distances round a cycle may take any
// value.
//
// A workgroup takes the lists of its block of `bin` keys (nodes and lists, see
// list_key), up to kSubLists lists and kCap nodes at a time.  Bound by LDS accesses
// (ceil(log2 of the longest list) jumps a node) and, for one short list, by the
// launch.  20000 lists of 2^3..2^10 nodes: 341 us on the sublist walks, 49 us
// here; one list of 4096 nodes took 32 us a call with links and sums apart and a
// kernel before it, and 12.6 us; of 16384 nodes 72 and 29 us.
constexpr int kSubLists = 1024;

template <int kCap, int kThreads>
__global__ void __launch_bounds__(kThreads) lr_lds(const int32_t* succ, int n,
                                                   const int64_t* __restrict__ off, int L,
                                                   int bin, int to_tail, int32_t* rank,
                                                   int32_t* lerr, int32_t* status) {
  static_assert(kCap <= kListNodes, "a node fits its word");
  constexpr int kRows = kCap / kThreads;
  __shared__ uint32_t word[kCap];
  __shared__ int so[kSubLists + 1];
  __shared__ uint32_t whole[kSubLists / 32], bad[kSubLists / 32];
  __shared__ int longest, past;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = lane_id();
  int64_t l0 = 0, l1 = 1;
  if (off) {
    const auto key = [&](int64_t l) { return list_key(off[l], l); };
    l0 = blockIdx.x == 0 ? 0 : count_below<kThreads>(L, (int64_t)blockIdx.x * bin, key);
    l1 = blockIdx.x == gridDim.x - 1
             ? L : count_below<kThreads>(L, (int64_t)(blockIdx.x + 1) * bin, key);
  }
  for (int64_t la = l0; la < l1;) {
    int k = (int)min<int64_t>(l1 - la, kSubLists);
    const int64_t v0 = off ? off[la] : 0;
    __syncthreads();  // the last lists' tables and words are done with
    for (int i = tid; i <= k; i += kThreads) {
      so[i] = table_entry((off ? off[la + i] : i * (int64_t)n) - v0);
    }
    if (tid < kSubLists / 32) whole[tid] = bad[tid] = 0;
    if (tid == 0) {
      longest = 1;
      past = k;
    }
    __syncthreads();
    for (int i = tid; i < k; i += kThreads)
      if (!entry_fits(so[i], so[i + 1], kCap)) atomicMin(&past, i);
    __syncthreads();
    const int fit = past;  // lists of the group that fit LDS together
    const int take = max(fit, 1);
    const int nv = so[take];
    if (fit == 0 || v0 < 0 || v0 > n - nv) {  // not the table the host planned with
      for (int i = tid; i < take; i += kThreads) {
        if (status) status[la + i] = PJ_EBADLIST;
        if (lerr) lerr[la + i] = kErrRange;
      }
      la += take;
      continue;
    }
    k = take;
    int most = 1;
    for (int i = tid; i < k; i += kThreads) most = max(most, so[i + 1] - so[i]);
    most = -wave_min(-most);
    if (lane == 0) atomicMax(&longest, most);
    // a wave owns rows of 64 consecutive nodes, so it looks a list up once and
    // follows the boundaries forward
    const int rows = (nv + kThreads - 1) / kThreads;
    const int j0 = wave * rows * kWave + lane;
    uint32_t mine[kRows];
#pragma unroll
    for (int t = 0; t < kRows; ++t)
      if (t < rows && j0 + t * kWave < nv) mine[t] = (uint32_t)succ[v0 + j0 + t * kWave];
    int l = k > 1 && j0 < nv ? lds_find(so, k, j0) : 0;
#pragma unroll
    for (int t = 0; t < kRows; ++t) {
      const int j = j0 + t * kWave;
      if (t < rows && j < nv) {
        while (l < k - 1 && so[l + 1] <= j) ++l;
        const int base = so[l], size = min(so[l + 1], nv) - base;
        const int s = (int)mine[t];
        const bool tail = (s == -1) | (s == j - base);
        const bool range = s >= 0 && s < size;
        if (!tail && !range) atomicOr(&bad[l >> 5], 1u << (l & 31));
        mine[t] = tail || !range ? list_tail_word(j) : list_word(base + s);
        word[j] = mine[t];
      }
    }
    __syncthreads();
    for (int span = 1; span < longest; span *= 2) {
#pragma unroll
      for (int t = 0; t < kRows; ++t) {
        const int j = j0 + t * kWave;
        if (t < rows && j < nv) {
          const uint32_t next = list_jump(mine[t], word[list_target(mine[t])]);
          if (next != mine[t]) word[j] = mine[t] = next;
        }
      }
      __syncthreads();
    }
    l = k > 1 && j0 < nv ? lds_find(so, k, j0) : 0;
#pragma unroll
    for (int t = 0; t < kRows; ++t) {
      const int j = j0 + t * kWave;
      if (t < rows && j < nv) {
        while (l < k - 1 && so[l + 1] <= j) ++l;
        const int size = so[l + 1] - so[l], d = list_distance(mine[t]);
        if (list_whole(mine[t], size)) atomicOr(&whole[l >> 5], 1u << (l & 31));
        rank[v0 + j] = to_tail ? d : size - 1 - d;
      }
    }
    if (status || lerr) {
      __syncthreads();
      for (int i = tid; i < k; i += kThreads) {
        const bool ok = so[i + 1] == so[i] || ((whole[i >> 5] & ~bad[i >> 5]) >> (i & 31) & 1);
        if (status) status[la + i] = ok ? PJ_OK : PJ_EBADLIST;
        if (lerr) lerr[la + i] = ok ? 0 : kErrBase;
      }
    }
    la += k;
  }
}

// Weighted batches: a whole batch of at most kMaxCutoff nodes in one workgroup,
// predecessor links in LDS and pointer jumping along them, a node's own term
// being its predecessor's weight.  succ is read before any rank is written (in
// place allowed).
__global__ void __launch_bounds__(kBaseThreads) lr_small_weighted(
    const int32_t* succ, const int32_t* __restrict__ weight, const int64_t* __restrict__ off,
    int L, int n, int32_t* rank, int32_t* ltails, int32_t* lerr) {
  __shared__ int lnk[kMaxCutoff];
  __shared__ int pre[kMaxCutoff];
  const int tid = threadIdx.x;
  for (int j = tid; j < n; j += kBaseThreads) lnk[j] = -1;
  __syncthreads();
  // Thread t reads the kPerThread consecutive ids from t * kPerThread, all
  // loads first, and follows the list boundaries forward (one search of the
  // offset table per thread).
  const int j0 = tid * kPerThread;
  if (j0 < n) {
    int sv[kPerThread];
    if (j0 + kPerThread <= n && (reinterpret_cast<uintptr_t>(succ) & 15) == 0) {
      const int4* s4 = reinterpret_cast<const int4*>(succ + j0);
#pragma unroll
      for (int q = 0; q < kPerThread / 4; ++q) {
        const int4 v = s4[q];
        sv[4 * q] = v.x;
        sv[4 * q + 1] = v.y;
        sv[4 * q + 2] = v.z;
        sv[4 * q + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int t = 0; t < kPerThread; ++t) sv[t] = j0 + t < n ? succ[j0 + t] : -1;
    }
    int l = find_instance(off, L, j0);
    int base = (int)off[l], end = (int)off[l + 1];
    for (int t = 0; t < kPerThread; ++t) {
      const int j = j0 + t;
      if (j >= n) break;
      while (j >= end) {
        ++l;
        base = end;
        end = (int)off[l + 1];
      }
      const int s = sv[t];
      const bool tail = (s == -1) | (s == j - base);
      if (tail) {
        atomicAdd(&ltails[l], 1);
      } else if ((unsigned)s >= (unsigned)(end - base)) {
        atomicOr(&lerr[l], kErrRange);
      } else if (atomicExch(&lnk[base + s], j) != -1) {
        atomicOr(&lerr[l], kErrBase);
      }
    }
  }
  __syncthreads();
  for (int j = tid; j < n; j += kBaseThreads) {
    const int p = lnk[j];
    pre[j] = p >= 0 ? weight[p] : 0;
  }
  __syncthreads();
  int rounds = 0;
  while ((1 << rounds) < n) ++rounds;
  int pa[kPerThread], la[kPerThread];
  for (int it = 0; it < rounds; ++it) {
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      la[t] = -2;
      pa[t] = 0;
      if (j < n) {
        const int p = lnk[j];
        if (p >= 0) {
          pa[t] = pre[p];
          la[t] = lnk[p];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int j = tid + t * kBaseThreads;
      if (j < n && la[t] != -2) {
        pre[j] += pa[t];
        lnk[j] = la[t];
      }
    }
    __syncthreads();
  }
  if (j0 < n) {
    int l = find_instance(off, L, j0);
    int end = (int)off[l + 1];
    for (int t = 0; t < kPerThread; ++t) {
      const int j = j0 + t;
      if (j >= n) break;
      while (j >= end) {
        ++l;
        end = (int)off[l + 1];
      }
      if (lnk[j] != -1) atomicOr(&lerr[l], kErrBase);
      rank[j] = pre[j];
    }
  }
}

// ------------------------------------------------------------ full check
// Complete check of the output (validate = 1): per list, ranks are a
// permutation of 0..size-1 and rank[succ[i]] = rank[i] + 1 off the tail.
__global__ void chk_clear(int32_t* cnt, int n) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x)
    cnt[j] = 0;
}

template <bool kBatched>
__global__ void chk_count(const int32_t* __restrict__ succ, const int32_t* __restrict__ rank,
                          const int64_t* __restrict__ off, int L, int n, int to_tail,
                          int32_t* cnt, int32_t* lerr) {
  auto one = [&](int64_t g, int l, int64_t base, int size) {
    int r = rank[g];
    if (to_tail) r = size - 1 - r;
    if ((unsigned)r >= (unsigned)size) {
      atomicOr(&lerr[l], kErrCheck);
      return;
    }
    atomicAdd(&cnt[base + r], 1);
    const int s = succ[g];
    const int xl = (int)(g - base);
    if (s == -1 || s == xl) return;
    if ((unsigned)s >= (unsigned)size) {
      atomicOr(&lerr[l], kErrCheck);
      return;
    }
    int rs = rank[base + s];
    if (to_tail) rs = size - 1 - rs;
    if (rs != r + 1) atomicOr(&lerr[l], kErrCheck);
  };
  // a grid-stride sweep, not for_each_listed: all waves then work in one
  // window of the batch, whose ranks the random gathers above find in cache
  // (contiguous runs per wave were slower: 27.7 against 17.6 ms on 4096 lists)
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += gridDim.x * blockDim.x) {
    if (kBatched) {
      const int l = find_instance(off, L, g);
      one(g, l, off[l], (int)(off[l + 1] - off[l]));
    } else {
      one(g, 0, 0, n);
    }
  }
}

template <bool kBatched>
__global__ void chk_perm(const int32_t* __restrict__ cnt, const int64_t* __restrict__ off, int L,
                         int n, int32_t* lerr) {
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += gridDim.x * blockDim.x) {
    if (cnt[g] != 1) {
      const int l = kBatched ? find_instance(off, L, g) : 0;
      atomicOr(&lerr[l], kErrCheck);
    }
  }
}

// Weighted calls with a status: the level sums are weights, not node counts,
// so the coverage check by the base total does not apply.  Instead every
// state word starts as "no sublist", and an expansion that meets one (a node
// no walk reached: a cycle beside the list) reports it.
__global__ void __launch_bounds__(256) lr_state_clear(int2* __restrict__ state, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    state[i] = make_int2(-1, 0);
}

// ---------------------------------------------------------------- status
__global__ void lr_status(const LrCtl* ctl, const int32_t* lerr, const int32_t* ltails,
                          const int64_t* off, int L, int n0, int check_total, int check_tails,
                          int32_t* status) {
  const bool global_bad = ctl && (ctl->err != 0 ||
                                  (check_total && ctl->base_total != (unsigned long long)n0));
  for (int l = blockIdx.x * blockDim.x + threadIdx.x; l < L; l += gridDim.x * blockDim.x) {
    const int64_t size = off[l + 1] - off[l];
    bool bad = global_bad || lerr[l] != 0;
    if (check_tails && size > 0 && ltails[l] != 1) bad = true;
    status[l] = (lerr[l] & kErrSplitter) ? PJ_EINVAL : bad ? PJ_EBADLIST : PJ_OK;
  }
}

// ------------------------------------------------------------------ host
inline int ilog2(int v) {
  int r = 0;
  while ((1 << r) < v) ++r;
  return r;
}

inline int grid_for(int64_t n, int block, int cap) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

// Workgroups of the batched head find: four chunks a wave, but no fewer than
// two workgroups per CU while every wave has a chunk.
inline int headfind_grid(int64_t n, int cap) {
  const int64_t per = kHfChunk * kWave * (256 / kWave);  // nodes of a workgroup's chunks
  const int64_t least = std::min<int64_t>(n / per + 1, 512);
  return (int)std::min<int64_t>(cap, std::max(least, n / (4 * per) + 1));
}

struct Plan {
  int algo = PJ_ALGO_RULING_SET;
  bool small = false;      // every list ranked in LDS
  int levels = 0;          // walk levels
  int base_kind = 1;       // 1 LDS, 2 device-wide
  int64_t bound[PJ_MAX_LEVELS + 2] = {};
  int log2B[PJ_MAX_LEVELS + 1] = {};
  int cap[PJ_MAX_LEVELS + 1] = {};
  int wide_rounds = 0;
  int wy_rounds = 0;
  bool paired = false;     // weighted: {step code, weight} pairs at level 0
  bool packed = false;     // level 0 state packed into the output buffer
  int kbits = 0;           // offset bits of the packed state
  int max_walk0 = 0;       // cut length at level 0
  int log2B_far = 0;       // > 0: level 0 may pick this on the device (see lr_walk),
  int kbits_far = 0;       // with these offset bits (packed form)
  int max_walk_far = 0;    // and this cut length
  int rec_grid = 0, rec_log2B = 0, rec_chunks = 0, rec_bins = 0, group_slabs = 0;
  int bin_shift = 0;       // and deals them to bins of this size (see lr_bin),
  bool word = false;       // in entries of one word
  int max_slabs = 0;       // > 0: level 0 records its walks (see lr_walk_rec)
  int64_t chosen = 0;      // > 0: level 0 uses this many caller-chosen splitters
};

// rank may be succ itself (in place: the successors are overwritten by the
// ranks, the way Section 3.2 reuses the device successor array for the
// output); any other overlap is rejected.  The full output check reads succ
// after the ranks are written, so it needs two arrays.
inline int check_alias(const int32_t* succ, const int32_t* rank, int64_t n, bool validate) {
  if (n <= 0) return PJ_OK;
  const uintptr_t s0 = (uintptr_t)succ, r0 = (uintptr_t)rank;
  const uintptr_t bytes = (uintptr_t)n * sizeof(int32_t);
  if (s0 == r0) return validate ? PJ_EINVAL : PJ_OK;
  if (s0 < r0 + bytes && r0 < s0 + bytes) return PJ_EINVAL;
  return PJ_OK;
}

inline int bits_for(int64_t v) {  // bits to hold values 0..v-1
  int b = 0;
  while ((int64_t(1) << b) < v) ++b;
  return b;
}

// chosen > 0: level 0 has that many caller-chosen splitters (never the
// one-workgroup path, so that they are used).
Plan make_plan(int64_t n0, int64_t L, int64_t max_size, const pj_opts& o, bool weighted,
               int64_t chosen) {
  // weighted calls need the separate (sublist, offset) state: an offset is then
  // a weight sum, not a step count
  const bool pack = !weighted && o.level0_state != PJ_STATE_SEPARATE;
  Plan p;
  p.algo = o.algo == PJ_ALGO_WYLLIE ? PJ_ALGO_WYLLIE : PJ_ALGO_RULING_SET;
  p.bound[0] = n0;
  if (p.algo == PJ_ALGO_WYLLIE) {
    p.wy_rounds = ilog2((int)std::max<int64_t>(max_size, 1));
    return p;
  }
  p.chosen = chosen;
  // One workgroup's lists: the whole input, or (unweighted) every list of a
  // batch up to the cutoff.  The latter looks at ceil(log2) of the longest list
  // only, which the key of a captured batch holds.
  int64_t longest = 1;
  while (longest < max_size) longest *= 2;
  if (chosen == 0 && (n0 <= o.cutoff || (!weighted && longest <= o.cutoff))) {
    p.small = true;
    return p;
  }
  int lv = 0;
  for (;;) {
    const int64_t b = p.bound[lv];
    if (lv > 0) {
      if (b <= o.cutoff) {
        p.base_kind = 1;
        break;
      }
      if (lv >= PJ_MAX_LEVELS || b * 4 > p.bound[lv - 1] * 3) {
        p.base_kind = 2;
        p.wide_rounds = ilog2((int)b);
        break;
      }
    }
    const int spacing = lv == 0 ? o.spacing : o.spacing_up;
    p.log2B[lv] = ilog2(std::max(2, spacing));
    const int64_t r = lv == 0 && chosen > 0 ? chosen
                                            : (b + (1ll << p.log2B[lv]) - 1) >> p.log2B[lv];
    int mw = o.max_walk;
    if (lv == 0) {
      // Pack (sublist id, offset) into 31 bits when the id space allows an
      // offset of at least 4 bits; the cut length then bounds the offset.
      p.packed = false;
      for (int kb = bits_for(mw); pack && kb >= 4; --kb) {
        const int mwk = std::min(mw, 1 << kb);
        const int64_t ids = r + L + b / mwk + 64;
        if (bits_for(ids) + kb <= 31) {
          p.packed = true;
          p.kbits = kb;
          mw = mwk;
          break;
        }
      }
      p.max_walk0 = mw;
    }
    p.cap[lv] = (int)(b / mw + 64);
    p.bound[lv + 1] = r + L + p.cap[lv];
    ++lv;
  }
  p.levels = lv;
  // (a visited state -2 - sublist id must not reach down to a splitter's code)
  p.paired = weighted && p.bound[1] + n0 + 2 < (int64_t(1) << 31);
  return p;
}

// Completes a plan made for level-0 spacing kLocalSpacing with the far
// alternative (see lr_walk): its packing and cut length.  The far sublist ids
// are fewer, so the offset may take more bits; the cut length may only grow,
// which keeps the planned cut-point capacity sufficient.
void add_far_spacing(Plan& p, int64_t n0, int64_t L, int far, int max_walk) {
  if (far <= 0 || p.levels < 1 || p.algo != PJ_ALGO_RULING_SET || p.chosen > 0) return;
  const int lg = ilog2(far);
  const int64_t r = (n0 + (1ll << lg) - 1) >> lg;
  if (!p.packed) {
    p.log2B_far = lg;
    p.max_walk_far = p.max_walk0;
    return;
  }
  for (int kb = bits_for(max_walk); kb >= 4; --kb) {
    const int mwk = std::min(max_walk, 1 << kb);
    if (mwk < p.max_walk0) break;
    if (bits_for(r + L + n0 / mwk + 64) + kb <= 31) {
      p.log2B_far = lg;
      p.kbits_far = kb;
      p.max_walk_far = mwk;
      return;
    }
  }
}

// The plan with level 0 recorded (see lr_walk_rec), where that suits the input.
//   * one list, from 11 M nodes on (9 M: 488 us in place, 524 recorded; 12 M: 600
//     and 567; 2^26: 3140 and 2340), up to the nodes that kTileBins bins hold,
//     and only if the head-find pass finds it not local;
//   * a batch of 2^20 nodes or more (1.4 M: 194 and 176 us) whose lists stay
//     near one L2.
// Strips are 16 nodes long, so sublists are 32 nodes long at least (8.4 M nodes
// in 200 lists: 387 us with 8, 334 with 32), and with 32 a batch walks as fast
// as with 64 for fewer of its nodes in flight.  Few lanes walk at one time (two
// workgroups a CU for one list, whose reads run at 55 G/s from 128 lanes a CU
// on; one for a batch, which holds the lists walked at one time to an L2).
constexpr int64_t kRecordList = int64_t(11) << 20;
constexpr int64_t kRecordBatch = int64_t(1) << 20;
constexpr int64_t kRecordLongest = int64_t(1) << 21;
constexpr int kRecordSpacing = 32;

//
// h_off: the host's table where the call runs on these very lists, else nullptr.
bool recorded_plan(const Plan& in_place, int64_t n0, int64_t L, int64_t max_size,
                   const int64_t* h_off, bool single, bool weighted, const pj_opts& o,
                   bool spacing_given, Plan* out) {
  const Plan& q = in_place;
  if (weighted != q.paired || q.algo != PJ_ALGO_RULING_SET || q.small || q.chosen > 0 ||
      (o.level0_state == PJ_STATE_SEPARATE && !weighted) || o.max_walk % kStrip != 0)
    return false;
  if (single ? !(q.packed || q.paired) || n0 < kRecordList || n0 > (int64_t)kTileBins * kBinNodes
             : n0 < kRecordBatch || max_size > kRecordLongest)
    return false;
  Plan p = in_place;
  if (!single && !spacing_given && o.spacing < kRecordSpacing) {
    pj_opts wide = o;
    wide.spacing = kRecordSpacing;
    p = make_plan(n0, L, max_size, wide, weighted, 0);
  }
  if (p.log2B_far > 0) p.log2B_far = std::max(p.log2B_far, ilog2(kRecordSpacing));
  p.rec_grid = device_info().cus * (single ? 2 : 1) / kXcds * kXcds;
  p.rec_log2B = p.log2B_far > 0 ? p.log2B_far : p.log2B[0];
  const RecordChunks chunks = record_chunks(n0, p.rec_log2B);
  const int64_t waves = p.rec_grid / (single ? 1 : kXcds) * (256 / kWave);
  p.rec_chunks = (int)chunks.chunks;
  p.word = !single && !weighted && max_size <= kWordLongest;
  p.bin_shift = p.word ? std::min(kBinShift, 32 - bits_for(max_size)) : kBinShift;
  p.rec_bins = (int)((n0 + (1ll << p.bin_shift) - 1) >> p.bin_shift);
  int64_t slabs = 0;
  if (single) {
    slabs = record_slabs(n0, chunks.blocks + kWalkChunk + 1 + n0 / o.max_walk + 64, waves);
  } else {
    const int64_t longest = h_off ? max_size : 1ll << bits_for(max_size);
    slabs = record_batch_slabs(n0, record_heads(h_off, L, n0, p.rec_log2B), longest, p.rec_log2B,
                               o.max_walk, waves);
    if (!record_fits(kXcds * slabs, 4 * kStrip * (weighted ? 2 : 1) + 8,
                     ((int64_t)p.rec_bins << p.bin_shift) * (p.word ? 4 : 8), n0))
      return false;
  }
  p.group_slabs = (int)slabs;
  p.max_slabs = (int)(slabs * (single ? 1 : kXcds));
  *out = p;
  return true;
}

struct Buffers {
  LrCtl* ctl = nullptr;
  unsigned long long* lsum = nullptr;
  int32_t* ltails = nullptr;
  int32_t* lerr = nullptr;
  int64_t* off1 = nullptr;            // {0, n} for the single-list call
  int2* state[PJ_MAX_LEVELS + 1] = {};
  int2* link[PJ_MAX_LEVELS + 2] = {};  // link[l] = input of level l (l >= 1)
  int32_t* srank[PJ_MAX_LEVELS + 2] = {};
  int32_t* wide_lnk = nullptr;
  unsigned long long* wide_pl = nullptr;
  unsigned long long* wy_pair = nullptr;
  int32_t* chk = nullptr;
  int32_t* status_tmp = nullptr;
  int32_t* ssucc = nullptr;           // successors of caller-chosen splitters
  RecArgs rec = {};
  int32_t* sub_max = nullptr;         // stats: longest level-0 sublist
};

// Carve (or, with ws == nullptr, just count) the buffers a plan needs.
size_t carve(const Plan& p, int64_t L, bool single, bool validate, bool want_status,
             Workspace* ws, Buffers* b) {
  size_t bytes = 0;
  auto take = [&](auto*& ptr, size_t count) {
    using T = std::remove_pointer_t<std::remove_reference_t<decltype(ptr)>>;
    bytes += ws_bytes(count, sizeof(T));
    if (ws) ptr = ws->take<T>(count);
  };
  take(b->ctl, 1);
  take(b->lsum, (size_t)std::max<int64_t>(L, 1));
  take(b->ltails, (size_t)std::max<int64_t>(L, 1));
  take(b->lerr, (size_t)std::max<int64_t>(L, 1));
  if (single) take(b->off1, 2);
  if (validate) take(b->chk, (size_t)p.bound[0]);
  if (want_status) take(b->status_tmp, (size_t)std::max<int64_t>(L, 1));
  if (p.algo == PJ_ALGO_WYLLIE) {
    take(b->wy_pair, (size_t)p.bound[0]);
    return bytes;
  }
  if (p.small) return bytes;
  take(b->sub_max, 1);
  if (p.max_slabs > 0) {
    const size_t slabs = (size_t)p.max_slabs;
    take(b->rec.ctl, 1);
    take(b->rec.strips, slabs * kSlab * kStrip / 4);
    take(b->rec.head, slabs * kSlab);
    take(b->rec.used, slabs);
    if (!single) take(b->rec.chunk_list, (size_t)p.rec_chunks + 1);
    take(b->rec.cursor, (size_t)p.rec_bins);
    uint32_t* ent = nullptr;
    take(ent, ((size_t)p.rec_bins << p.bin_shift) * (p.word ? 1 : 2));
    b->rec.ent = ent;
    b->rec.bin_shift = p.bin_shift;
    if (p.paired) {
      take(b->rec.before, slabs * kSlab * kStrip / 4);
      b->state[0] = reinterpret_cast<int2*>(b->rec.ent);  // read before the bins are filled
    }
    b->rec.group_slabs = p.group_slabs;
    b->rec.log2B = p.rec_log2B;
    b->rec.if_far = p.log2B_far > 0 ? 1 : 0;
  }
  if (p.chosen > 0) take(b->ssucc, (size_t)p.chosen);
  for (int l = 0; l < p.levels; ++l) {
    if (l > 0 || !(p.packed || (p.max_slabs > 0 && (p.paired || p.log2B_far == 0)))) take(b->state[l], (size_t)p.bound[l]);
    take(b->link[l + 1], (size_t)p.bound[l + 1]);
    take(b->srank[l + 1], (size_t)p.bound[l + 1]);
  }
  if (p.base_kind == 2) {
    take(b->wide_lnk, (size_t)p.bound[p.levels]);
    take(b->wide_pl, (size_t)p.bound[p.levels]);
  }
  return bytes;
}

// Lists ranked in LDS (see lr_lds).  The smaller instance lets eight workgroups
// share a CU.  A workgroup's block of nodes leaves room for the longest list to
// run over its end, or, for lists over half the capacity, is half the capacity.
// One list of more than kOneList nodes, or weighted, goes to lr_one_lds.
int launch_lds(const int32_t* succ, const int32_t* weight, int64_t n, int64_t max_size,
               const int64_t* d_off, int64_t L, int32_t* rank, int to_tail, int32_t* lerr,
               int32_t* status, hipStream_t stream) {
  if (!d_off && (weight || n > kOneList)) {
    hipLaunchKernelGGL(lr_one_lds, dim3(kXcds + 1), dim3(kBaseThreads), 0, stream, succ, weight,
                       (int)n, to_tail, rank, lerr, status);
    PJ_HIP(hipGetLastError());
    return PJ_OK;
  }
  constexpr int kSmallCap = 4096;
  const bool small = d_off && max_size <= kSmallCap;
  const int cap = small ? kSmallCap : kMaxCutoff;
  const int bin = (int)std::max<int64_t>(cap / 2, cap - max_size);
  const auto k = small ? lr_lds<kSmallCap, 256> : lr_lds<kMaxCutoff, kBaseThreads>;
  hipLaunchKernelGGL(k, dim3(d_off ? (unsigned)((n + L) / bin + 1) : 1), dim3(small ? 256 : kBaseThreads),
                     0, stream, succ, (int)n, d_off, (int)L, bin, to_tail, rank, lerr, status);
  PJ_HIP(hipGetLastError());
  return PJ_OK;
}

}  // namespace

int list_rank_impl(const int32_t* succ, const int64_t* d_off, int64_t L, const int64_t* h_off,
                   int64_t n_single, int32_t* rank, const pj_opts* user, hipStream_t stream,
                   const int32_t* weight) {
  const bool single = d_off == nullptr;
  if (L < 0) return PJ_EINVAL;
  if (single) L = 1;
  if (L > INT32_MAX / 2) return PJ_EINVAL;
  pj_opts o = resolved_opts(user);
  if (o.spacing > 65536 || o.spacing_up > 65536) return PJ_EINVAL;
  if (user && user->stats) {
    *user->stats = pj_stats{};
    user->stats->status = PJ_OK;
  }

  // total nodes and the largest list, from the host's view of the offsets
  int64_t n0 = 0, max_size = 0;
  std::vector<int64_t> hbuf;
  const int64_t* ho = single ? nullptr : h_off;
  if (single) {
    n0 = n_single;
    max_size = n0;
  } else {
    if (L == 0) return PJ_OK;
    if (!ho) {
      hbuf.resize((size_t)L + 1);
      PJ_HIP(hipMemcpyAsync(hbuf.data(), d_off, sizeof(int64_t) * (L + 1),
                            hipMemcpyDeviceToHost, stream));
      PJ_HIP(hipStreamSynchronize(stream));
      ho = hbuf.data();
    }
    if (ho[0] != 0) return PJ_EINVAL;
    for (int64_t l = 0; l < L; ++l) {
      const int64_t s = ho[l + 1] - ho[l];
      if (s < 0) return PJ_EINVAL;
      max_size = std::max(max_size, s);
    }
    n0 = ho[L];
  }
  if (n0 < 0 || n0 >= INT32_MAX) return PJ_EINVAL;
  if (n0 > 0 && (!succ || !rank)) return PJ_EINVAL;
  PJ_TRY(check_alias(succ, rank, n0, o.validate != 0));
  if (weight) {
    // weighted ranks are exclusive prefix sums from the head by the ruling
    // set; the to-tail form and the full check (a permutation test) do not
    // apply
    if (o.algo == PJ_ALGO_WYLLIE || o.to_tail || o.validate) return PJ_EINVAL;
    const uintptr_t w0 = (uintptr_t)weight, r0 = (uintptr_t)rank;
    const uintptr_t bytes = (uintptr_t)n0 * sizeof(int32_t);
    if (n0 > 0 && w0 < r0 + bytes && r0 < w0 + bytes) return PJ_EINVAL;
  }
  const bool want_status = o.validate && !o.d_status;
  if (n0 == 0 && !o.d_status) return PJ_OK;
  if (o.level0_state != PJ_STATE_AUTO && o.level0_state != PJ_STATE_SEPARATE) return PJ_EINVAL;
  // caller-chosen level-0 splitters: one unweighted list, ruling set, the
  // packed state (the marks live in the successor copy)
  const int64_t chosen = o.d_splitters && n0 > 0 ? o.n_splitters : 0;
  if (o.d_splitters && n0 > 0 &&
      (!single || weight || o.algo == PJ_ALGO_WYLLIE || o.level0_state == PJ_STATE_SEPARATE ||
       o.n_splitters < 1 || o.n_splitters > n0))
    return PJ_EINVAL;

  int far_spacing = 0;
  bool spacing_given = false;
  {  // ruling-set parameters left at zero come from the tune cache, if tuned
    pj_opts raw;
    pj_opts_init(&raw);
    if (user) raw = *user;
    apply_tuned(raw, n0, L);
    far_spacing = level0_spacing(raw.spacing, n0, single, &o.spacing);
    spacing_given = raw.spacing > 0;
    o.spacing_up = raw.spacing_up > 0 ? raw.spacing_up : o.spacing_up;
    o.cutoff = raw.cutoff > 0 ? std::min(std::max(raw.cutoff, 64), 16384) : o.cutoff;
    o.max_walk = raw.max_walk > 0 ? std::max(raw.max_walk, 16) : o.max_walk;
    if (raw.block > 0) o.block = std::min(1024, (raw.block + 63) / 64 * 64);
  }
  Plan p = make_plan(n0, L, max_size, o, weight != nullptr, chosen);
  if (chosen > 0 && !p.packed) return PJ_EINVAL;  // too many splitters for the packed state
  add_far_spacing(p, n0, L, far_spacing, o.max_walk);
  Buffers b;
  size_t need = carve(p, L, single, o.validate != 0, want_status, nullptr, &b);
  if (p.small && (!weight || single) && n0 > 0 && !o.validate && !(user && user->stats)) {
    // one kernel, which also writes the statuses: no workspace, no init
    if (o.workspace && o.workspace_bytes < need) return PJ_EINVAL;
    return launch_lds(succ, weight, n0, max_size, d_off, L, rank, o.to_tail, nullptr, o.d_status,
                      stream);
  }
  Workspace ws;
  // the recorded walk where its strips fit the caller's workspace or the pool
  bool recorded = false;
  Plan pr;
  if (recorded_plan(p, n0, L, max_size, ho && !capturing(stream) ? ho : nullptr, single,
                    weight != nullptr, o, spacing_given, &pr)) {
    const size_t more = carve(pr, L, single, o.validate != 0, want_status, nullptr, &b);
    if (!o.workspace || o.workspace_bytes >= more)
      recorded = workspace_acquire(ws, more, &o, stream) == PJ_OK;
    if (!recorded) (void)hipGetLastError();  // no memory for it: in place
  }
  if (recorded) p = pr;
  else PJ_TRY(workspace_acquire(ws, need, &o, stream));
  b = Buffers{};
  carve(p, L, single, o.validate != 0, want_status, &ws, &b);
  const int64_t* off = single ? b.off1 : d_off;
  int32_t* status = o.d_status ? o.d_status : b.status_tmp;

  PhaseTimer tm;
  pj_stats* st = user ? user->stats : nullptr;
  PJ_TRY(tm.begin(st != nullptr, stream));

  const int n = (int)n0;
  const int Li = (int)L;
  const int blk = o.block;
  const int cus = device_info().cus;
  const int gcap = cus * 16;

  hipLaunchKernelGGL(lr_init, dim3(grid_for(std::max<int64_t>(L, 64), 256, 1024)), dim3(256), 0,
                     stream, b.ctl, n, b.lsum, b.ltails, b.lerr, Li, b.off1,
                     b.rec, recorded ? p.rec_bins : 0);
  PJ_HIP(hipGetLastError());
  tm.mark("init");

  bool check_total = false, check_tails = false;
  if (n0 > 0 && p.algo == PJ_ALGO_WYLLIE) {
    if (o.validate || o.d_status) {
      if (single)
        hipLaunchKernelGGL(lr_headfind_single<kNoCopy>, dim3(grid_for(n / 4 + 1, 256, 1024)),
                           dim3(256), 0, stream, succ, n, nullptr, nullptr, nullptr, 0, 0u, b.lsum,
                           b.ltails, b.lerr, nullptr);
      else
        hipLaunchKernelGGL(lr_headfind_batched<kNoCopy>,
                           dim3(headfind_grid(n, gcap)), dim3(256), 0,
                           stream, succ, off, Li, n, nullptr, nullptr, nullptr, 0, 0u, b.lsum, b.ltails,
                           b.lerr);
      check_tails = true;
      tm.mark("headfind");
    }
    const int g = grid_for(n, blk, gcap);
    if (single)
      hipLaunchKernelGGL(wy_init<false>, dim3(g), dim3(blk), 0, stream, succ, off, Li, n,
                         b.wy_pair, b.lerr);
    else
      hipLaunchKernelGGL(wy_init<true>, dim3(g), dim3(blk), 0, stream, succ, off, Li, n,
                         b.wy_pair, b.lerr);
    tm.mark("wyllie_init");
    for (int it = 0; it < p.wy_rounds; ++it)
      hipLaunchKernelGGL(wy_jump, dim3(g), dim3(blk), 0, stream, b.wy_pair, n);
    tm.mark("wyllie_jump");
    if (single) {
      if (o.to_tail)
        hipLaunchKernelGGL((wy_final<false, true>), dim3(g), dim3(blk), 0, stream, b.wy_pair, off,
                           Li, n, rank, b.lerr);
      else
        hipLaunchKernelGGL((wy_final<false, false>), dim3(g), dim3(blk), 0, stream, b.wy_pair,
                           off, Li, n, rank, b.lerr);
    } else {
      if (o.to_tail)
        hipLaunchKernelGGL((wy_final<true, true>), dim3(g), dim3(blk), 0, stream, b.wy_pair, off,
                           Li, n, rank, b.lerr);
      else
        hipLaunchKernelGGL((wy_final<true, false>), dim3(g), dim3(blk), 0, stream, b.wy_pair,
                           off, Li, n, rank, b.lerr);
    }
    tm.mark("wyllie_final");
  } else if (n0 > 0 && p.small) {
    if (weight && !single) {
      hipLaunchKernelGGL(lr_small_weighted, dim3(1), dim3(kBaseThreads), 0, stream, succ, weight,
                         off, Li, n, rank, b.ltails, b.lerr);
      check_tails = true;
    } else {
      PJ_TRY(launch_lds(succ, weight, n0, max_size, d_off, L, rank, o.to_tail, b.lerr, nullptr,
                        stream));
    }
    tm.mark("small");
  } else if (n0 > 0) {
    // level 0 head find (and, in the packed form, the successor copy, which
    // in place is already there)
    int32_t* copy = !weight && (p.packed || recorded) ? rank : nullptr;
    // weighted: successor and weight side by side where the state goes
    int2* pair = weight && p.paired ? b.state[0] : nullptr;
    const bool copy_succ = copy && (const void*)succ != (const void*)rank;
    if (single) {
      auto k = pair ? lr_headfind_single<kPairCopy>
               : copy && p.chosen == 0 ? lr_headfind_single<kCodedCopy>
               : copy_succ ? lr_headfind_single<kPlainCopy> : lr_headfind_single<kNoCopy>;
      // (a workgroup ends in up to four atomics on the same words: 2^20 nodes
      // take 18.9 us with 1024 workgroups and 11.5 us with 256)
      hipLaunchKernelGGL(k, dim3(grid_for(n / 4 + 1, 256, n <= 1 << 22 ? 256 : 1024)), dim3(256),
                         0, stream, succ, n, copy, weight, pair,
                         p.log2B_far > 0 ? p.log2B_far : p.log2B[0], level_seed(o.seed, 0),
                         b.lsum, b.ltails, b.lerr, &b.ctl->near);
    } else {
      auto k = pair ? lr_headfind_batched<kPairCopy>
                        : recorded ? lr_headfind_batched<kCodedCopy>
                        : copy_succ ? lr_headfind_batched<kPlainCopy>
                                    : lr_headfind_batched<kNoCopy>;
      hipLaunchKernelGGL(k, dim3(headfind_grid(n, gcap)), dim3(256), 0,
                         stream, succ, off, Li, n, copy, weight, pair, p.log2B[0],
                         level_seed(o.seed, 0), b.lsum, b.ltails, b.lerr);
    }
    PJ_HIP(hipGetLastError());
    if (p.chosen > 0) {
      hipLaunchKernelGGL(lr_mark_splitters, dim3(grid_for(p.chosen, 256, gcap)), dim3(256), 0,
                         stream, copy, o.d_splitters, (int)p.chosen, n, b.ssucc, b.lerr);
      PJ_HIP(hipGetLastError());
    }
    tm.mark("headfind");
    check_total = weight == nullptr;
    if (weight && status)
      for (int lv = pair ? 1 : 0; lv < p.levels; ++lv)
        hipLaunchKernelGGL(lr_state_clear, dim3(grid_for(p.bound[lv], 256, gcap)), dim3(256), 0,
                           stream, b.state[lv], p.bound[lv]);
    check_tails = true;
    // walks, level by level
    for (int lv = 0; lv < p.levels; ++lv) {
      WalkArgs a{};
      a.succ0 = succ;
      a.weight0 = weight;
      a.link_in = b.link[lv];
      a.off = off;
      a.lsum = b.lsum;
      a.ltails = b.ltails;
      a.lerr = b.lerr;
      a.state = b.state[lv];
      a.work = copy;
      a.link_out = b.link[lv + 1];
      a.ctl = b.ctl;
      a.L = Li;
      a.level = lv;
      a.log2B = p.log2B[lv];
      a.log2B_far = lv == 0 && single ? p.log2B_far : 0;
      a.kbits_far = p.kbits_far;
      a.max_walk_far = p.max_walk_far;
      a.max_walk = lv == 0 ? p.max_walk0 : o.max_walk;
      a.cap = p.cap[lv];
      a.cap_prev = lv > 0 ? p.cap[lv - 1] : 0;
      a.kbits = p.kbits;
      a.seed = level_seed(o.seed, lv);
      void (*kfn)(WalkArgs);
      if (lv > 0) kfn = lr_walk<false, false, false>;
      else if (pair) kfn = single ? lr_walk<true, false, false, true> : lr_walk<true, true, false, true>;
      else if (single) kfn = p.packed ? lr_walk<true, false, true> : lr_walk<true, false, false>;
      else kfn = p.packed ? lr_walk<true, true, true> : lr_walk<true, true, false>;
      if (lv == 0 && recorded) {
        WalkArgs ra = a;
        ra.max_walk = o.max_walk;
        if (!single)
          hipLaunchKernelGGL(lr_rec_chunks, dim3(grid_for(p.rec_chunks + 1, 256, gcap)), dim3(256),
                             0, stream, off, Li, p.rec_chunks, p.rec_log2B + 6, b.rec.chunk_list);
        const auto walk = pair ? (single ? lr_walk_rec<false, true> : lr_walk_rec<true, true>)
                               : (single ? lr_walk_rec<false, false> : lr_walk_rec<true, false>);
        hipLaunchKernelGGL(walk, dim3(p.rec_grid), dim3(256), 0, stream, ra, b.rec);
        PJ_HIP(hipGetLastError());
        if (!b.rec.if_far) {
          tm.mark("walk0");
          continue;
        }
        a.if_near = 1;
      }
      const bool marked = lv == 0 && p.chosen > 0;
      const int64_t items =
          marked ? p.chosen + 1 : ((p.bound[lv] + (1ll << a.log2B) - 1) >> a.log2B) + L;
      // workgroup size o.block (tunable): it sets how many lanes share one
      // LDS work counter and contiguous range of splitters
      int g = marked ? persistent_grid((const void*)lr_walk_marked, blk, 0)
                     : persistent_grid((const void*)kfn, blk, 0);
      g = (int)std::min<int64_t>(g, (items + blk - 1) / blk);
      if (g < 1) g = 1;
      if (marked)
        hipLaunchKernelGGL(lr_walk_marked, dim3(g), dim3(blk), 0, stream, a, o.d_splitters,
                           (const int32_t*)b.ssucc, (int)p.chosen);
      else
        hipLaunchKernelGGL(kfn, dim3(g), dim3(blk), 0, stream, a);
      PJ_HIP(hipGetLastError());
      tm.mark(lv == 0 ? "walk0" : "walk_up");
    }
    // base ranking of the top level
    const int top = p.levels;
    const int cap_prev = p.cap[top - 1];
    if (p.base_kind == 1) {
      if (L <= kBaseLists)
        hipLaunchKernelGGL(lr_base_walk, dim3(kXcds + 1), dim3(kBaseThreads), 0, stream, b.link[top],
                           b.srank[top], b.ctl, top, Li, cap_prev, (int)p.bound[top]);
      else
        hipLaunchKernelGGL(lr_base_lds, dim3(1), dim3(kBaseThreads), 0, stream, b.link[top],
                           b.srank[top], b.ctl, top, Li, cap_prev);
    } else {
      const int g = grid_for(p.bound[top], 256, gcap);
      hipLaunchKernelGGL(wide_clear, dim3(g), dim3(256), 0, stream, b.wide_lnk, b.ctl, top, Li,
                         cap_prev);
      hipLaunchKernelGGL(wide_pred, dim3(g), dim3(256), 0, stream, b.link[top], b.wide_lnk, b.ctl,
                         top, Li, cap_prev);
      hipLaunchKernelGGL(wide_init, dim3(g), dim3(256), 0, stream, b.link[top], b.wide_lnk,
                         b.wide_pl, b.ctl, top, Li, cap_prev);
      for (int it = 0; it < p.wide_rounds; ++it)
        hipLaunchKernelGGL(wide_jump, dim3(g), dim3(256), 0, stream, b.wide_pl, b.ctl, top, Li,
                           cap_prev);
      hipLaunchKernelGGL(wide_final, dim3(g), dim3(256), 0, stream, b.wide_pl, b.srank[top],
                         b.ctl, top, Li, cap_prev);
    }
    PJ_HIP(hipGetLastError());
    tm.mark("base");
    // expand back down
    for (int lv = top - 1; lv >= 1; --lv) {
      const int g = grid_for(p.bound[lv], 256, gcap);
      hipLaunchKernelGGL(lr_expand, dim3(g), dim3(256), 0, stream, b.state[lv], b.srank[lv + 1],
                         b.srank[lv], b.ctl, lv, Li, p.cap[lv - 1], p.cap[lv]);
    }
    tm.mark("expand_up");
    const int g0 = grid_for(n, 256, gcap);
    void (*ex0)(const int2*, const int32_t*, int32_t*, const int64_t*, LrCtl*, int, int, int, int,
                int);
    if (single) {
      if (o.to_tail) ex0 = p.packed ? lr_expand0<false, true, true> : lr_expand0<false, true, false>;
      else ex0 = p.packed ? lr_expand0<false, false, true> : lr_expand0<false, false, false>;
    } else {
      if (o.to_tail) ex0 = p.packed ? lr_expand0<true, true, true> : lr_expand0<true, true, false>;
      else ex0 = p.packed ? lr_expand0<true, false, true> : lr_expand0<true, false, false>;
    }
    if (recorded) {
      const auto bin =
          pair ? (single ? lr_bin<false, false, true> : lr_bin<true, false, true>)
          : single ? (o.to_tail ? lr_bin<false, true, false> : lr_bin<false, false, false>)
          : p.word ? (o.to_tail ? lr_bin<true, true, false, true> : lr_bin<true, false, false, true>)
                   : (o.to_tail ? lr_bin<true, true, false> : lr_bin<true, false, false>);
      const int cus = device_info().cus;
      hipLaunchKernelGGL(bin, dim3(cus / kXcds * kXcds), dim3(kTileThreads), 0, stream, b.rec,
                         (const int32_t*)b.srank[1], off, Li, p.cap[0], b.ctl);
      tm.mark("bin");
      hipLaunchKernelGGL(p.word ? lr_place<true> : lr_place<false>,
                         dim3((unsigned)std::min<int64_t>((n0 + kBinNodes - 1) >> kBinShift, cus)), dim3(kTileThreads),
                         0, stream, b.rec, rank, b.ctl);
      tm.mark("place");
    }
    if (pair && (!recorded || b.rec.if_far))
      hipLaunchKernelGGL(lr_expand0_paired, dim3(g0), dim3(256), 0, stream, (const int2*)pair,
                         (const int32_t*)b.srank[1], rank, b.ctl, Li, p.cap[0], recorded ? 1 : 0);
    else if (!recorded || b.rec.if_far)
      hipLaunchKernelGGL(ex0, dim3(g0), dim3(256), 0, stream, b.state[0], b.srank[1], rank, off,
                         b.ctl, Li, p.cap[0], p.kbits, single ? p.kbits_far : 0,
                         recorded ? 1 : 0);
    PJ_HIP(hipGetLastError());
    tm.mark("expand0");
  }

  if (o.validate && n0 > 0) {
    const int g = grid_for(n, 256, gcap);
    hipLaunchKernelGGL(chk_clear, dim3(g), dim3(256), 0, stream, b.chk, n);
    if (single) {
      hipLaunchKernelGGL(chk_count<false>, dim3(g), dim3(256), 0, stream, succ, rank, off, Li, n,
                         o.to_tail, b.chk, b.lerr);
      hipLaunchKernelGGL(chk_perm<false>, dim3(g), dim3(256), 0, stream, b.chk, off, Li, n,
                         b.lerr);
    } else {
      hipLaunchKernelGGL(chk_count<true>, dim3(g), dim3(256), 0, stream, succ, rank, off, Li, n,
                         o.to_tail, b.chk, b.lerr);
      hipLaunchKernelGGL(chk_perm<true>, dim3(g), dim3(256), 0, stream, b.chk, off, Li, n,
                         b.lerr);
    }
    PJ_HIP(hipGetLastError());
    tm.mark("validate");
  }
  if (status) {
    hipLaunchKernelGGL(lr_status, dim3(grid_for(L, 256, 1024)), dim3(256), 0, stream,
                       p.algo == PJ_ALGO_RULING_SET && !p.small ? b.ctl : nullptr, b.lerr,
                       b.ltails, off, Li, n, check_total ? 1 : 0, check_tails ? 1 : 0, status);
    PJ_HIP(hipGetLastError());
  }

  int result = PJ_OK;
  if (want_status) {
    std::vector<int32_t> hs((size_t)L);
    PJ_HIP(hipMemcpyAsync(hs.data(), status, sizeof(int32_t) * L, hipMemcpyDeviceToHost, stream));
    PJ_HIP(hipStreamSynchronize(stream));
    for (int64_t l = 0; l < L; ++l)
      if (hs[l] != PJ_OK) {
        result = hs[l];
        break;
      }
  }
  if (st) {
    PJ_TRY(tm.finish(st));
    st->algo = p.algo;
    st->levels = p.levels;
    st->base_kind = p.small ? 0 : p.base_kind;
    int32_t hmax = 0;
    if (p.algo == PJ_ALGO_RULING_SET && !p.small && n0 > 0) {
      PJ_HIP(hipMemsetAsync(b.sub_max, 0, sizeof(int32_t), stream));
      hipLaunchKernelGGL(lr_sublist_max, dim3(grid_for(p.bound[1], 256, gcap)), dim3(256), 0,
                         stream, (const int2*)b.link[1], (const LrCtl*)b.ctl, Li, p.cap[0],
                         b.sub_max);
      PJ_HIP(hipGetLastError());
      PJ_HIP(hipMemcpyAsync(&hmax, b.sub_max, sizeof hmax, hipMemcpyDeviceToHost, stream));
    }
    LrCtl hc{};
    PJ_HIP(hipMemcpyAsync(&hc, b.ctl, sizeof hc, hipMemcpyDeviceToHost, stream));
    PJ_HIP(hipStreamSynchronize(stream));
    st->level_nodes[0] = n0;
    for (int l = 1; l <= p.levels && l <= PJ_MAX_LEVELS; ++l)
      st->level_nodes[l] = hc.lv[l - 1].r + L + std::min(hc.lv[l - 1].dyn, p.cap[l - 1]);
    if (p.levels > 0) {
      st->sublists0 = st->level_nodes[1];
      st->cuts0 = std::min(hc.lv[0].dyn, p.cap[0]);
      st->max_sublist0 = hmax;
    }
    if (p.algo == PJ_ALGO_WYLLIE) st->rounds = n0 > 0 ? p.wy_rounds : 0;
    st->status = result;
  }
  PJ_TRY(workspace_release(ws));
  return result;
}

// First-level splitter spacing when the caller leaves it at zero: about 2^20
// splitters, so the splitter ranks that the final scatter gathers (4 B each)
// stay near one XCD's 4 MiB L2, from 8 (short walks for small, latency-bound
// lists) up to 256 for one list (2^28 nodes: 14.5 ms at 256 against 15.9 at
// 64, measured; longer walks cost imbalance, a larger table costs L2
// misses) and up to 64 for a batch, whose many short lists end most walks
// early anyway.  One list of up to 25600 nodes takes 2 and of up to 60000 takes
// 4: its splitters still fit the base, whose time grows less than that of the
// longest walk falls (random lists at 8, 4 and 2: 17000 nodes 50, 41 and 37.5
// us, 25000 46, 41 and 40, 32000 46, 42 and 43, 55000 52 and 46; 85000, with one
// more level, 57.8 and 59.5; local lists of 32000 and 60000, whose walks share
// their lines, 30 and 34 at 8, 32 and 36 at 4).
int list_rank_default_spacing(int64_t n, bool single) {
  if (single && n <= 60000) return n <= 25600 ? 2 : 4;
  const int cap = single ? 256 : 64;
  int sp = 8;
  while (sp < cap && (n >> 20) > sp) sp *= 2;
  return sp;
}

// Level-0 spacing actually planned.  A caller's (or tuned) value is used as
// is.  Otherwise a single list of at least 2^22 nodes is planned with
// spacing kLocalSpacing and lets the walk switch to the size default on the
// device when its successors are not local (the returned far spacing);
// smaller lists and batches use the size default.
constexpr int kLocalSpacing = 8;
constexpr int64_t kAdaptiveMin = int64_t(1) << 22;

int level0_spacing(int requested, int64_t n0, bool single, int32_t* planned) {
  if (requested > 0) {
    *planned = requested;
    return 0;
  }
  const int dflt = list_rank_default_spacing(n0, single);
  if (single && n0 >= kAdaptiveMin && dflt != kLocalSpacing) {
    *planned = kLocalSpacing;
    return dflt;
  }
  *planned = dflt;
  return 0;
}

size_t list_rank_workspace(int64_t n0, int64_t L, const pj_opts* user, bool single,
                           bool weighted) {
  pj_opts raw;
  pj_opts_init(&raw);
  if (user) raw = *user;
  apply_tuned(raw, n0, L);
  (void)level0_spacing(raw.spacing, n0, single, &raw.spacing);
  pj_opts o = resolved_opts(&raw);
  const int64_t chosen = o.d_splitters && single && !weighted && n0 > 0
                             ? std::max<int64_t>(1, std::min(o.n_splitters, n0)) : 0;
  Plan p = make_plan(n0, L, n0, o, weighted, chosen);
  Buffers b;
  return carve(p, L, single, o.validate != 0, o.validate && !o.d_status, nullptr, &b);
}

// Workspace with which a batch of these sizes is recorded, if it is; else as
// list_rank_workspace.
size_t list_rank_graph_workspace(int64_t n0, int64_t L, int64_t max_size, const pj_opts* user) {
  pj_opts raw;
  pj_opts_init(&raw);
  if (user) raw = *user;
  apply_tuned(raw, n0, L);
  const bool spacing_given = raw.spacing > 0;
  (void)level0_spacing(raw.spacing, n0, false, &raw.spacing);
  const pj_opts o = resolved_opts(&raw);
  Plan p = make_plan(n0, L, max_size, o, false, 0), pr;
  Buffers b;
  const bool status = o.validate && !o.d_status;
  size_t bytes = list_rank_workspace(n0, L, user, false);
  if (recorded_plan(p, n0, L, max_size, nullptr, false, false, o, spacing_given, &pr))
    bytes = std::max(bytes, carve(pr, L, false, o.validate != 0, status, nullptr, &b));
  return bytes;
}

}  // namespace pj

extern "C" {

int pj_list_rank_ex(const int32_t* succ, int64_t n, int32_t* rank, const pj_opts* opts,
                    pj_stream_t stream) {
  if (n < 0) return PJ_EINVAL;
  return pj::list_rank_impl(succ, nullptr, 1, nullptr, n, rank, opts, (hipStream_t)stream);
}

int pj_list_rank(const int32_t* succ, int64_t n, int32_t* rank, pj_stream_t stream) {
  return pj_list_rank_ex(succ, n, rank, nullptr, stream);
}

int pj_list_rank_batched_ex(const int32_t* succ, const int64_t* offsets, int64_t L,
                            int32_t* rank, const pj_opts* opts, pj_stream_t stream) {
  if (!offsets || L < 0) return PJ_EINVAL;
  if (opts && opts->use_graph && !opts->stats && !(opts->validate && !opts->d_status) && L > 0) {
    std::vector<int64_t> hbuf;
    const int64_t* ho = opts->h_offsets;
    if (!ho) {
      hbuf.resize((size_t)L + 1);
      PJ_HIP(hipMemcpyAsync(hbuf.data(), offsets, sizeof(int64_t) * (L + 1),
                            hipMemcpyDeviceToHost, (hipStream_t)stream));
      PJ_HIP(hipStreamSynchronize((hipStream_t)stream));
      ho = hbuf.data();
    }
    if (ho[0] != 0 || ho[L] < 0 || ho[L] >= INT32_MAX) return PJ_EINVAL;
    for (int64_t l = 0; l < L; ++l)
      if (ho[l + 1] < ho[l]) return PJ_EINVAL;
    if (ho[L] > 0 && (!succ || !rank)) return PJ_EINVAL;
    PJ_TRY(pj::check_alias(succ, rank, ho[L], opts->validate != 0));
    return pj::graph_batched(succ, offsets, L, ho, rank, *opts, (hipStream_t)stream);
  }
  return pj::list_rank_impl(succ, offsets, L, opts ? opts->h_offsets : nullptr, 0, rank, opts,
                            (hipStream_t)stream);
}

int pj_list_rank_batched(const int32_t* succ, const int64_t* offsets, int64_t L, int32_t* rank,
                         pj_stream_t stream) {
  return pj_list_rank_batched_ex(succ, offsets, L, rank, nullptr, stream);
}

int pj_list_rank_weighted(const int32_t* succ, const int32_t* weight, int64_t n, int32_t* rank,
                          const pj_opts* opts, pj_stream_t stream) {
  if (n < 0 || (n > 0 && !weight)) return PJ_EINVAL;
  return pj::list_rank_impl(succ, nullptr, 1, nullptr, n, rank, opts, (hipStream_t)stream,
                            n > 0 ? weight : nullptr);
}

int pj_list_rank_weighted_batched(const int32_t* succ, const int32_t* weight,
                                  const int64_t* offsets, int64_t L, int32_t* rank,
                                  const pj_opts* opts, pj_stream_t stream) {
  if (!offsets || L < 0 || (L > 0 && !weight)) return PJ_EINVAL;
  return pj::list_rank_impl(succ, offsets, L, opts ? opts->h_offsets : nullptr, 0, rank, opts,
                            (hipStream_t)stream, weight);
}

size_t pj_list_rank_weighted_workspace_bytes(int64_t total_nodes, int64_t L,
                                             const pj_opts* opts) {
  if (total_nodes < 0 || L < 1) return 0;
  const size_t batched = pj::list_rank_workspace(total_nodes, L, opts, false, true);
  return L > 1 ? batched
               : std::max(batched, pj::list_rank_workspace(total_nodes, L, opts, true, true));
}

size_t pj_list_rank_workspace_bytes(int64_t total_nodes, int64_t L, const pj_opts* opts) {
  if (total_nodes < 0 || L < 1) return 0;
  // one list may go through either entry point: size for the larger layout
  const size_t batched = pj::list_rank_workspace(total_nodes, L, opts, false);
  return L > 1 ? batched
               : std::max(batched, pj::list_rank_workspace(total_nodes, L, opts, true));
}

}  // extern "C"
