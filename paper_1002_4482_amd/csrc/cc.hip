// Connected components on gfx950: hook and shortcut (Section 4, the family of
// the paper's SV-GPU) over a parent forest that only ever points to smaller
// ids, so the root a component ends with is its smallest vertex id and the
// flat forest is the label array.
//
// State: the parent array D (held in the caller's label buffer), D[v] <= v.
//   hook      a pair (u, v) climbs from the larger of its two nodes; when that
//             node is a root it is hooked onto the other node with a compare
//             and swap (D[x]: x -> y, y < x).  A node that is no root any more
//             never becomes one again, so every success joins two trees, and
//             a pair is finished when both nodes are the same: one pass over
//             the pairs settles connectivity, with no rounds and no host check.
//   shortcut  D[v] <- the root of v, one writer per word.
// SV's stars, stamps and stagnant hooks exist because its hooks are blind
// concurrent stores; a compare and swap needs none of them.  The hook is the
// published lock-free form of union-find by ids (Rem's algorithm; with compare and
// swap, Jayanti and Tarjan; on GPUs, ECL-CC by Jaiganesh and Burtscher), and joining
// a sample of the pairs first, so that most of the rest need only be looked at, is
// the idea of Afforest (Sutton, Ben-Nun and Barak).
//
// Large graphs run hook and shortcut kernels over the whole device (cc_hook,
// cc_flatten); graphs of at most kLdsVertices vertices are solved in the LDS
// of one workgroup each (cc_lds).
#include <algorithm>
#include <array>
#include <cstddef>
#include <map>
#include <mutex>
#include <vector>

#include "lds_rules.hpp"
#include "pj_internal.hpp"

namespace pj {
namespace {

constexpr int kFlatHops = 24;   // parent steps of a vertex in cc_flatten between its stores
constexpr int kFlatPer = 4;     // vertices of a thread in cc_flatten

constexpr int kClasses = 255;

struct CcCtl {
  int32_t err;
  int32_t steps;                // longest chain of parent steps of a shortcut, up to kFlatHops
  int32_t ordered;              // the ids follow the graph (sample_order)
  int32_t again;                // pairs were given up and are still to be joined
  int32_t redo;                 // joining them joined trees: one more shortcut
  int32_t classes;              // numbered parents (cc_class_pick), 0: not used
  int32_t parents[kClasses];
};

// Memory access discipline.  D is read and hooked by every workgroup of one
// kernel, on eight XCDs with an L2 each.
//   * Hooks are device-scope compare and swaps, performed at the coherent
//     level whatever the L2s hold: a swap that finds D[x] == x is the only one
//     that ever does, so no hook is lost and none happens twice.
//   * Reads are device-scope relaxed loads (same rate as plain ones here: 77
//     G/s on a 16 MiB array, 222 G/s on 2 MiB).  An old value is harmless: it is
//     an ancestor in the same tree, and a node mistaken for a root fails the
//     swap, which returns its parent.
//   * cc_hook's path halving stores (device-scope) replace the parent of a
//     node that has one by an ancestor.  Such a node is never swapped again, and
//     whichever of several stores lands last is an ancestor.
//   * The shortcut's stores are plain: each word has one writer in the kernel.

// Joins the trees of x and y.  Both only ever move to a parent, the larger
// first, so the loop ends after at most x + y steps even on stale values.
//
// After `halve` steps it halves the path.  In a large forest that starts late:
// the stores of a giant component's pairs go to the few nodes under its root and
// serialise there (2^20 pairs of a 2^22-vertex uniform graph on a quarter of the
// roots: 450 us from the 3rd step on, 240 us from the 16th); a small one is bound
// by the chain of reads instead (300000 vertices: 70 us against 79 us).
//
// Hooks may chain every vertex to the one before, and then a pair that meets the
// chain climbs as far as the graph is long, with nobody else on the way (a ring of
// 4 * 10^6 vertices in id order: 1.03 s, nearly all for the pair that closes it).
// So a pair is given up after `most` steps, and its chunk of pairs is marked and
// read again once a shortcut has flattened the chains (that ring: 0.43 ms).
//
// The lanes of a wave that hook the same root send one swap: the pairs of a hub
// with the largest id all meet at the hub's parent, and swaps on one word run at
// 88 M/s (a star of 4 * 10^6 vertices 3.26 ms, with one swap a wave 0.21).
constexpr int kHalveSmall = 3, kHalveLarge = 16;
constexpr int64_t kHalveSmallBelow = 1 << 20;
constexpr int kNever = INT32_MAX;

// Steps before the path is halved and before a pair is given up.  With random ids
// a few pairs of many millions take more than 24 (8 M in paths 720 us with 24, 697
// with 32 and 48).  Where ids follow the graph thousands may climb at once, and
// those that halve their paths meet at the same few nodes (a grid of 10^6 vertices,
// 300 wide, numbered row by row with ids from two halves in turn: swaps of 1.6 ms;
// without halving the whole solve takes 0.12).
struct Climb {
  int halve, most;
};
constexpr Climb kClimbSmall{kHalveSmall, 48}, kClimbLarge{kHalveLarge, 48};
constexpr Climb kClimbOrdered{kNever, 24};

enum Joined { kSame, kHooked, kLeft };

__device__ __forceinline__ Joined join(int32_t* D, int x, int y, int halve, int most) {
  for (int step = 1; x != y; ++step) {
    if (step > most) return kLeft;
    const int hi = max(x, y);
    y = min(x, y);
    x = hi;
    int p = load_coherent(&D[x]);
    if (p == x) {
      const int first = __builtin_amdgcn_readfirstlane(x);
      const bool swaps = x != first || lanes_below(__ballot(1)) == 0;
      if (swaps) p = atomicCAS(&D[x], x, y);
      const int got = __builtin_amdgcn_readfirstlane(p);
      const int to = __builtin_amdgcn_readfirstlane(y);
      if (!swaps) p = got == x ? to : got;
      else if (p == x) return kHooked;
    } else if (step > halve) {
      const int g = load_coherent(&D[p]);
      if (g != p) publish(&D[x], g);
      p = g;
    }
    x = p;
  }
  return kSame;
}

// Marks a chunk that holds pairs given up: for cc_hook_rest, which reads the
// others anyway, or for the last kernels.
constexpr int32_t kForRest = 1, kForLast = 2;

__device__ __forceinline__ void mark_left(int32_t* left, int64_t chunk, bool any, int32_t how,
                                          CcCtl* ctl) {
  if (__ballot(any) && lane_id() == 0) {
    publish(&left[chunk], how);
    if (how == kForLast) publish(&ctl->again, 1);
  }
}

// Whether the ids follow the graph: one workgroup counts, of 1024 sampled pairs,
// how many distances of ids differ (in steps of n / 2^14).  With random ids nearly
// all do; where paths, rings, grids or layers are numbered in order few do.
constexpr int kSamples = 1024;

__device__ __forceinline__ void sample_order(const int32_t* __restrict__ src,
                                             const int32_t* __restrict__ dst, int64_t m, int n,
                                             CcCtl* ctl) {
  constexpr int kSlots = 4 * kSamples;
  __shared__ int slot[kSlots], distinct;
  const int tid = threadIdx.x;
  unsigned away[kSamples / 256];
#pragma unroll
  for (int t = 0; t < kSamples / 256; ++t) {
    const uint32_t i = t * 256 + tid + 1;
    const int64_t e = (int64_t)(((uint64_t)mix32(i) << 20 ^ mix32(i + kSamples)) % (uint64_t)m);
    const unsigned d = (unsigned)src[e] - (unsigned)dst[e];
    away[t] = min(d, 0u - d) / (unsigned)max(1, n >> 14);  // (2^31 at most)
  }
  for (int i = tid; i < kSlots; i += 256) slot[i] = -1;
  if (tid == 0) distinct = 0;
  __syncthreads();
  int mine = 0;
#pragma unroll
  for (int t = 0; t < kSamples / 256; ++t)
    for (uint32_t h = mix32(away[t]);; ++h) {  // a quarter of the slots is taken at most
      const int old = atomicCAS(&slot[h % kSlots], -1, (int)away[t]);
      mine += old == -1;
      if (old == -1 || old == (int)away[t]) break;
    }
  atomicAdd(&distinct, mine);
  __syncthreads();
  if (tid == 0) ctl->ordered = distinct < kSamples * 7 / 8;
}

__global__ void __launch_bounds__(256) cc_init(int32_t* __restrict__ D, int n, CcCtl* ctl,
                                               int32_t* __restrict__ left, int64_t nchunks,
                                               const int32_t* __restrict__ src,
                                               const int32_t* __restrict__ dst, int64_t sampled) {
  if (sampled > 0 && blockIdx.x == gridDim.x - 1) {  // a workgroup more, of its own
    sample_order(src, dst, sampled, n, ctl);
    return;
  }
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int stride = (gridDim.x - (sampled > 0)) * blockDim.x;
  if (tid < (int)(offsetof(CcCtl, parents) / 4) &&
      !(sampled > 0 && tid == (int)(offsetof(CcCtl, ordered) / 4)))
    reinterpret_cast<int32_t*>(ctl)[tid] = 0;
  const int n4 = (reinterpret_cast<uintptr_t>(D) & 15) == 0 ? n >> 2 : 0;
  for (int q = tid; q < n4; q += stride)
    reinterpret_cast<int4*>(D)[q] = make_int4(4 * q, 4 * q + 1, 4 * q + 2, 4 * q + 3);
  for (int v = 4 * n4 + tid; v < n; v += stride) D[v] = v;
  for (int64_t c = tid; c < nchunks; c += stride) left[c] = 0;
}

// kPer rows of 256 pairs from row `row` on, loaded and range-checked: an id out
// of range makes the pair (0, 0).
template <int kPer>
__device__ __forceinline__ bool load_pairs(const int32_t* __restrict__ src,
                                           const int32_t* __restrict__ dst, int64_t m, int n,
                                           int64_t row, int (&x)[kPer], int (&y)[kPer]) {
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int64_t e = (row + t) * 256 + threadIdx.x;
    x[t] = e < m ? src[e] : 0;
    y[t] = e < m ? dst[e] : 0;
  }
  bool bad = false;
#pragma unroll
  for (int t = 0; t < kPer; ++t)
    if ((unsigned)x[t] >= (unsigned)n || (unsigned)y[t] >= (unsigned)n) {
      bad = true;
      x[t] = y[t] = 0;
    }
  return bad;
}

__device__ __forceinline__ void report(CcCtl* ctl, bool bad) {
  if (__ballot(bad) && lane_id() == 0) atomicOr(&ctl->err, kErrRange);
}

// First hooks, blind: every stride-th chunk's pairs store their smaller end as the
// larger end's parent, no read and no swap (85 G stores/s against 27 G swaps/s).
// One of the pairs of a vertex wins; the others join nothing yet, and all of them
// are read again.  A workgroup more than those samples the order of the ids.
constexpr int kHookPer = 8;

__global__ void __launch_bounds__(256) cc_hook_blind(const int32_t* __restrict__ src,
                                                     const int32_t* __restrict__ dst, int64_t m,
                                                     int n, int32_t* __restrict__ D,
                                                     int64_t stride, int64_t units,
                                                     const int32_t* only_if, CcCtl* ctl) {
  if (only_if && *only_if == 0) return;
  if (!only_if && blockIdx.x == gridDim.x - 1) {  // (cc_init has sampled otherwise)
    sample_order(src, dst, m, n, ctl);
    return;
  }
  const int64_t groups = gridDim.x - (only_if ? 0 : 1);
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units; i += groups) {
    int x[kHookPer], y[kHookPer];
    bad |= load_pairs(src, dst, m, n, i * stride * kHookPer, x, y);
#pragma unroll
    for (int t = 0; t < kHookPer; ++t)
      if (x[t] != y[t]) D[max(x[t], y[t])] = min(x[t], y[t]);
  }
  report(ctl, bad);
}

// Hooks the pairs of the chunks stride - 1, 2 * stride - 1, ..., and leaves those
// given up to the kernels that `how` says.
template <int kPer>
__global__ void __launch_bounds__(256) cc_hook(const int32_t* __restrict__ src,
                                               const int32_t* __restrict__ dst, int64_t m, int n,
                                               int32_t* D, int64_t stride, int64_t units,
                                               Climb climb, int32_t* left, int32_t how,
                                               CcCtl* ctl) {
  if (ctl->ordered) climb = kClimbOrdered;
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units; i += gridDim.x) {
    int x[kPer], y[kPer];
    constexpr int kParts = kHookPer / kPer;
    const int64_t c = (i / kParts + 1) * stride - 1;
    bad |= load_pairs(src, dst, m, n, c * kHookPer + i % kParts * kPer, x, y);
    bool any = false;
#pragma unroll
    for (int t = 0; t < kPer; ++t)
      any |= join(D, x[t], y[t], climb.halve, climb.most) == kLeft;
    mark_left(left, c, any, how, ctl);
  }
  report(ctl, bad);
}

// Classes: a byte per vertex that tells most pairs of one tree apart from the
// others without D.  The up to 255 parents that most of kClassSamples sampled
// vertices have are numbered 1..255; a vertex with such a parent gets its
// number, any other 0.  Two ends with the same number other than 0 have the
// same parent.  One workgroup picks the parents; with few of the samples
// covered (small trees everywhere) it picks none and the bytes are not used.
constexpr int kClassSamples = 8192;
constexpr int kClassTable = 16384;

__global__ void __launch_bounds__(1024) cc_class_pick(const int32_t* __restrict__ D, int n,
                                                      CcCtl* ctl) {
  __shared__ int key[kClassTable];
  __shared__ int count[kClassTable];
  __shared__ int hist[64], above, covered, picked;
  const int tid = threadIdx.x;
  for (int i = tid; i < kClassTable; i += 1024) {
    key[i] = -1;
    count[i] = 0;
  }
  if (tid < 64) hist[tid] = 0;
  if (tid == 0) above = covered = picked = 0;
  int p[kClassSamples / 1024];
#pragma unroll
  for (int t = 0; t < kClassSamples / 1024; ++t)
    p[t] = D[(int)((uint64_t)mix32(t * 1024 + tid + 1) * (uint32_t)n >> 32)];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kClassSamples / 1024; ++t) {
    uint32_t h = mix32((uint32_t)p[t]);
    for (;; ++h) {  // at most half the slots are ever taken
      const int old = atomicCAS(&key[h & (kClassTable - 1)], -1, p[t]);
      if (old == -1 || old == p[t]) break;
    }
    atomicAdd(&count[h & (kClassTable - 1)], 1);
  }
  __syncthreads();
  for (int i = tid; i < kClassTable; i += 1024)
    if (count[i]) atomicAdd(&hist[min(count[i], 63)], 1);
  __syncthreads();
  if (tid == 0) {  // parents sampled at least `above` times: at most kClasses
    int c = 63, sum = hist[63];
    while (c > 2 && sum + hist[c - 1] <= kClasses) sum += hist[--c];
    above = c;
  }
  __syncthreads();
  for (int i = tid; i < kClassTable; i += 1024)
    if (count[i] >= above) {
      const int at = atomicAdd(&picked, 1);
      if (at < kClasses) {  // (more than 255 parents of 63 samples: the first ones)
        ctl->parents[at] = key[i];
        atomicAdd(&covered, count[i]);
      }
    }
  __syncthreads();
  if (tid == 0)
    ctl->classes = covered >= kClassSamples * 7 / 10 ? min(picked, kClasses) : 0;
}

__global__ void __launch_bounds__(256) cc_class_fill(const int32_t* __restrict__ D, int n,
                                                     const CcCtl* ctl,
                                                     uint32_t* __restrict__ cls) {
  constexpr int kSlots = 1024;
  __shared__ int key[kSlots];
  __shared__ uint8_t num[kSlots];
  const int classes = ctl->classes;
  if (classes == 0) return;
  for (int i = threadIdx.x; i < kSlots; i += 256) key[i] = -1;
  __syncthreads();
  if ((int)threadIdx.x < classes) {
    const int p = ctl->parents[threadIdx.x];
    uint32_t h = mix32((uint32_t)p);
    while (atomicCAS(&key[h & (kSlots - 1)], -1, p) != -1) ++h;
    num[h & (kSlots - 1)] = (uint8_t)(threadIdx.x + 1);
  }
  __syncthreads();
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; 4 * q < n;
       q += (int64_t)gridDim.x * 256) {
    uint32_t word = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t v = 4 * q + t;
      const int p = v < n ? D[v] : -2;
      uint32_t h = mix32((uint32_t)p);
      int k = key[h & (kSlots - 1)];
      while (k != p && k != -1) k = key[++h & (kSlots - 1)];
      if (k == p) word |= (uint32_t)num[h & (kSlots - 1)] << 8 * t;
    }
    cls[q] = word;
  }
}

// Hooks the pairs of all the other chunks, and of the `swapped` ones where pairs
// were given up, most of which lie in one tree by now: two reads (of classes, or
// of D) settle those, the rest is gathered in LDS first so that the lanes of a wave
// climb together.
template <bool kClassed>
__device__ __forceinline__ void hook_rest(const int32_t* __restrict__ src,
                                          const int32_t* __restrict__ dst, int64_t m, int n,
                                          int32_t* D, const uint8_t* __restrict__ cls,
                                          int64_t stride, int64_t units, int64_t swapped,
                                          int32_t* left, CcCtl* ctl, int2* queue, int* queued) {
  const Climb climb = ctl->ordered ? kClimbOrdered : kClimbLarge;
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units + swapped; i += gridDim.x) {
    int64_t c = i / (stride - 1) * stride + i % (stride - 1);
    if (i >= units) {
      c = (i - units + 1) * stride - 1;
      if (left[c] == 0) continue;
    }
    int x[kHookPer], y[kHookPer];
    bad |= load_pairs(src, dst, m, n, c * kHookPer, x, y);
    if (threadIdx.x == 0) *queued = 0;
    int cx[kHookPer], cy[kHookPer];
#pragma unroll
    for (int t = 0; t < kHookPer; ++t) cx[t] = kClassed ? cls[x[t]] : load_coherent(&D[x[t]]);
#pragma unroll
    for (int t = 0; t < kHookPer; ++t) cy[t] = kClassed ? cls[y[t]] : load_coherent(&D[y[t]]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kHookPer; ++t) {
      const bool open = x[t] != y[t] && (cx[t] != cy[t] || (kClassed && cx[t] == 0));
      const uint64_t mk = __ballot(open);
      if (mk == 0) continue;
      int at = 0;
      if (lane_id() == 0) at = atomicAdd(queued, __popcll(mk));
      at = __shfl(at, 0);
      if (open)
        queue[at + lanes_below(mk)] = kClassed ? make_int2(x[t], y[t]) : make_int2(cx[t], cy[t]);
    }
    __syncthreads();
    const int total = *queued;
    bool any = false;
    for (int q = threadIdx.x; q < total; q += 256)
      any |= join(D, queue[q].x, queue[q].y, climb.halve, climb.most) == kLeft;
    mark_left(left, c, any, kForLast, ctl);
    __syncthreads();  // the queue is reused by the next chunk
  }
  report(ctl, bad);
}

__global__ void __launch_bounds__(256) cc_hook_rest(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst, int64_t m,
                                                    int n, int32_t* D,
                                                    const uint8_t* __restrict__ cls,
                                                    int64_t stride, int64_t units, int64_t swapped,
                                                    int32_t* left, CcCtl* ctl) {
  __shared__ int2 queue[256 * kHookPer];
  __shared__ int queued;
  if (cls && ctl->classes > 0)
    hook_rest<true>(src, dst, m, n, D, cls, stride, units, swapped, left, ctl, queue, &queued);
  else
    hook_rest<false>(src, dst, m, n, D, cls, stride, units, swapped, left, ctl, queue, &queued);
}

// The pairs still given up, on a flat forest, to the end.  Nearly always there are
// none.
__global__ void __launch_bounds__(256) cc_join_left(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst, int64_t m,
                                                    int n, int32_t* D, int64_t nchunks,
                                                    const int32_t* __restrict__ left, CcCtl* ctl) {
  if (ctl->again == 0) return;
  bool hooked = false;
  for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
    if (left[c] != kForLast) continue;
    int x[kHookPer], y[kHookPer];
    (void)load_pairs(src, dst, m, n, c * kHookPer, x, y);
#pragma unroll
    for (int t = 0; t < kHookPer; ++t)
      hooked |= join(D, x[t], y[t], kHalveSmall, kNever) == kHooked;
  }
  if (__ballot(hooked) && lane_id() == 0) publish(&ctl->redo, 1);
}

// Shortcut: D[v] <- its root, in one pass whatever the depth.  Hooks leave trees
// far less than kFlatHops deep, and then a vertex climbs to its root.  From a
// deeper one it publishes, every kFlatHops steps, how far it has come, so that
// the vertices under it skip those steps: a parent's id is smaller than its
// child's and vertices are taken in ascending order, so what is above a vertex
// is flat already or climbs at the same time, and the depth left is divided by
// kFlatHops + 1 while one vertex takes kFlatHops steps.  The order is the
// workgroups', each with a run of vertices: with a stride over the grid the
// first ones would reach vertices of workgroups that wait for them to end, and
// climb link by link (a path of 2^22 ids in order: 347 ms).  (Climbing stops at
// the root even if none of those stores is seen.)  Bound by the reads of parents;
// in passes of kFlatHops steps, most of which found nothing left, a launch each,
// three shortcuts of a solve took 68 us of 300000 vertices and 112 of 10^6, and
// take 36 and 46 here (whole solves 165 -> 130 and 296 -> 230 us).  Four vertices a
// thread, one by one: with two there is less above that is flat already (10^6
// 252 us), with six too few lanes in small graphs; only deep ones climb side by
// side (a path of 2^20 ids in order, doubled: 554 us, one by one 792).
//
// only_if: only if that word is not 0.  Nearly always it is, so the workgroups are
// larger: 8000 of 256 threads that end at once take 17 us.  (Fewer that take runs
// from a counter either wait for it, 2^22 vertices 160 us instead of 60, or take
// the next run ahead, and others then climb through the vertices of runs that are
// held and not begun: a path of 2^22 ids in order 137 ms.)
template <int kThreads>
__global__ void __launch_bounds__(kThreads) cc_flatten(int32_t* D, int n, const int32_t* only_if,
                                                       CcCtl* ctl) {
  if (only_if && *only_if == 0) return;
  const int64_t v0 = (int64_t)blockIdx.x * (kThreads * kFlatPer) + threadIdx.x;
  int most = 0;
  int up[kFlatPer];  // of the deep vertices: the ancestor reached
  bool deep = false;
#pragma unroll
  for (int t = 0; t < kFlatPer; ++t) {  // one by one: the later find flat trees above
    const int64_t v = v0 + t * kThreads;
    up[t] = -1;
    if (v >= n) continue;
    const int p0 = D[v];
    int p = p0, h = 0;
    for (; h < kFlatHops; ++h) {  // (plain reads: most lanes end at the same few roots)
      const int g = D[p];
      if (g == p) break;
      p = g;
    }
    most = max(most, h);
    if (h == kFlatHops) {
      publish(&D[v], p);
      up[t] = p;
      deep = true;
    } else if (p != p0) {
      D[v] = p;
    }
  }
  while (deep) {  // side by side
    bool left = true;
    for (int h = 0; h < kFlatHops && left; ++h) {
      int g[kFlatPer];
#pragma unroll
      for (int t = 0; t < kFlatPer; ++t) g[t] = up[t] >= 0 ? load_coherent(&D[up[t]]) : -1;
      left = false;
#pragma unroll
      for (int t = 0; t < kFlatPer; ++t) {
        left |= g[t] != up[t];
        up[t] = g[t];
      }
    }
#pragma unroll
    for (int t = 0; t < kFlatPer; ++t)
      if (up[t] >= 0) publish(&D[v0 + t * kThreads], up[t]);
    deep = left;
  }
  most = -wave_min(-most);
  if (lane_id() == 0 && most > 1 && load_coherent(&ctl->steps) < most) atomicMax(&ctl->steps, most);
}

// ------------------------------------------------- one workgroup's graphs
// Graphs whose parent arrays fit in LDS: one workgroup reads a graph's pairs,
// joins them in LDS and writes the labels, so a solve is one kernel whose only
// memory traffic is the input (a part of it twice) and the output.  Parents
// are 16 bits wide, two to a word: 65536 vertices take 128 of the 160 KiB.
// Bound by vector instructions and LDS accesses of the 16 waves that fit, and
// by the latency of the pair loads (two rows of chunks in flight, about 36 GB/s
// per CU).  1024 graphs of 2^8..2^16 vertices, 5.9 * 10^7 pairs: 2109 us on the
// device-wide path, 345 us here; 1000 vertices and 1500 pairs 65 and 14 us.
//
// A workgroup takes the graphs of its block of `bin` keys (graph_key: vertices,
// pairs and graphs), up to kSubGraphs graphs of kLdsVertices vertices in all at a
// time, so thousands of tiny graphs share a workgroup and a graph of any size up to
// that, or with many pairs, has one of its own (with blocks of vertices alone one workgroup
// took 20 graphs of 100 vertices and 10^6 pairs, 7.9 ms; 0.15 now).
constexpr int kLdsVertices = 65536;
constexpr int kLdsThreads = 1024;
constexpr int kSubGraphs = 512;
constexpr int kLdsPairs = 1 << 30;
constexpr int kLdsPer = 8;         // pairs a lane loads at a time
constexpr int kLdsPatience = 128;  // steps of a wave before it gives pairs up
constexpr int kLdsChunk = kWave * kLdsPer;

// Parent of x in `word`, which holds the parents of x & ~1 and x | 1.
__device__ __forceinline__ int half_of(uint32_t word, int x) { return word >> (x & 1) * 16 & 0xffff; }

__device__ __forceinline__ uint32_t lds_load(const uint32_t* par, int x) {
  return __hip_atomic_load(&par[x >> 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lds_store(uint32_t* par, int x, int p) {
  __hip_atomic_store(&reinterpret_cast<uint16_t*>(par)[x], (uint16_t)p, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A pair on its way through the LDS forest, one step of `join` at a time.  A
// node that is climbed from gets its grandparent as parent (path splitting),
// which the next step reads anyway.
struct LdsPair {
  int x = 0, y = 0, from = -1;  // from: the node x was climbed from

  __device__ __forceinline__ void step(uint32_t* par) {
    if (x == y) return;
    if (x < y) {
      const int t = x;
      x = y;
      y = t;
      from = -1;
    }
    const uint32_t word = lds_load(par, x);
    int p = half_of(word, x);
    if (p == x) {
      // a root: the swap covers both halves of the word, and when it loses to
      // a change of the other half the pair tries again next step
      const int sh = (x & 1) * 16;
      const uint32_t seen =
          atomicCAS(&par[x >> 1], word, (word & ~(0xffffu << sh)) | (uint32_t)y << sh);
      p = seen == word ? y : half_of(seen, x);
      if (p != x) from = -1;
      x = p;
    } else {
      if (from >= 0) lds_store(par, from, p);
      from = x;
      x = p;
    }
  }
};

// Shortcut of the LDS forest of nv vertices, D[v] <- D[D[v]] until nothing
// changes: a thread owns a word, the parents of two vertices, and all threads
// jump at once, so even a path as long as the forest takes few steps.  Returns
// the most jumps of a word; ends with a barrier.
__device__ __forceinline__ int lds_flatten(uint32_t* par, int nv) {
  int most = 0;
  for (int i = threadIdx.x; i < (nv + 1) / 2; i += kLdsThreads) {
    uint32_t word = par[i];
    for (int h = 0;; ++h) {
      const int p0 = word & 0xffff, p1 = word >> 16;
      const int g0 = half_of(lds_load(par, p0), p0), g1 = half_of(lds_load(par, p1), p1);
      if (g0 == p0 && g1 == p1) {
        most = max(most, h);
        break;
      }
      word = (uint32_t)g0 | (uint32_t)g1 << 16;
      __hip_atomic_store(&par[i], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  __syncthreads();
  return most;
}

// voff == nullptr: one graph of n vertices and m pairs.  The host has checked
// the tables it planned with; what the device's hold is checked here against
// n, m and kLdsVertices, and graphs that do not fit get PJ_EINVAL.
__global__ void __launch_bounds__(kLdsThreads) cc_lds(
    const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t m, int n,
    const int64_t* __restrict__ voff, const int64_t* __restrict__ eoff, int G, int64_t bin,
    int bins, int heavy, int32_t* __restrict__ label, int32_t* __restrict__ status, int32_t* deepest) {
  __shared__ uint32_t par[kLdsVertices / 2];
  __shared__ int sv[kSubGraphs + 1], se[kSubGraphs + 1];
  __shared__ uint32_t badbits[kSubGraphs / 32];
  constexpr int kWaves = kLdsThreads / kWave;
  __shared__ uint32_t queue[kWaves][kLdsChunk / 2];  // (x << 16 | y)
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = lane_id();
  __shared__ int first_heavy, past;  // first graph that is heavy, that does not fit
  __shared__ int gave_up;            // the last attempt at a part that gave pairs up
  int attempt = 0;
  if (tid == 0) gave_up = 0;
  // with a second set of `bins` workgroups, the first takes the heavy graphs
  const bool take_heavy = (int)gridDim.x > bins && (int)blockIdx.x < bins;
  const int block = (int)blockIdx.x % bins;
  int64_t g0 = 0, g1 = 1;
  if (voff) {
    const auto key = [&](int64_t g) { return graph_key(voff[g], eoff[g], g); };
    g0 = block == 0 ? 0 : count_below<kLdsThreads>(G, block * bin, key);
    g1 = block == bins - 1 ? G : count_below<kLdsThreads>(G, (block + 1) * bin, key);
  }
  int deep = 0;
  for (int64_t ga = g0; ga < g1;) {
    int k = (int)min<int64_t>(g1 - ga, kSubGraphs);
    const int64_t v0 = voff ? voff[ga] : 0, e0 = voff ? eoff[ga] : 0;
    __syncthreads();  // the last graphs' tables and parents are done with
    for (int i = tid; i <= k; i += kLdsThreads) {
      sv[i] = table_entry((voff ? voff[ga + i] : i * (int64_t)n) - v0);
      se[i] = table_entry((voff ? eoff[ga + i] : i * m) - e0);
    }
    if (tid < kSubGraphs / 32) badbits[tid] = 0;
    if (tid == 0) first_heavy = past = k;
    __syncthreads();
    if (tid < k) {
      if (!(entry_fits(sv[tid], sv[tid + 1], kLdsVertices) && entry_fits(se[tid], se[tid + 1], kLdsPairs)))
        atomicMin(&past, tid);
      if ((int)gridDim.x > bins && se[tid + 1] - se[tid] > heavy) atomicMin(&first_heavy, tid);
    }
    __syncthreads();
    const TableStep next = table_step(first_heavy, past, take_heavy);
    if (!next.ours) {
      ga += next.count;
      continue;
    }
    k = next.count;
    const int nv = sv[k], ne = se[k];
    if (past == 0 || v0 < 0 || v0 > n - nv || e0 < 0 || e0 > m - ne) {
      if (status)
        for (int i = tid; i < k; i += kLdsThreads) status[ga + i] = PJ_EINVAL;
      ga += k;
      continue;
    }
    for (int i = tid; i < (min(nv, kLdsVertices) + 1) / 2; i += kLdsThreads)
      par[i] = (uint32_t)(2 * i) | (uint32_t)(2 * i + 1) << 16;
    __syncthreads();
    // As for a large graph: blind hooks of about two pairs a vertex, joins of
    // half a pair a vertex, and then the rest, most of which lies in one tree
    // by then, each part on a flat forest: joins on trees that are still being
    // built climb long ways.  A wave gathers the pairs that are not in one
    // tree yet in a queue of its own, and its lanes take the next one as soon
    // as they are done with theirs.  Where joins chain one vertex to the next,
    // pairs climb as far as the graph is long: a wave that goes on for long gives
    // up the pairs it has, and the part is done again on a flat forest, with twice
    // the patience (a ring of 30000 vertices whose ids alternate between two
    // halves: 1190 us, 85 like this).
    const int nchunks = (int)(((int64_t)ne + kLdsChunk - 1) / kLdsChunk);
    const int ratio = ne / max(nv, 1);
    const int s1 = max(1, ratio / 2);
    const int s2 = max(2, 2 * ratio);
    uint32_t* const q = queue[wave];
    int patience = kLdsPatience;
    for (int part = 0; part < 3;) {
      // the part's chunks: 0, s1, ...; s2 - 1, 2 * s2 - 1, ...; all but those
      const int count = part == 0 ? (nchunks + s1 - 1) / s1
                                  : part == 1 ? nchunks / s2 : nchunks - nchunks / s2;
      if (count == 0) {  // uniform over the workgroup
        ++part;
        continue;
      }
      ++attempt;
      const auto chunk_of = [&](int i) {
        return part == 0 ? i * s1 : part == 1 ? (i + 1) * s2 - 1 : i + i / (s2 - 1);
      };
      int x[kLdsPer], y[kLdsPer];
      const auto load = [&](int i) {
        if (i >= count) return;
        const int64_t c0 = (int64_t)chunk_of(i) * kLdsChunk;
        const int32_t* const ps = src + e0 + c0;
        const int32_t* const pd = dst + e0 + c0;
        const int rest = (int)min<int64_t>(ne - c0, kLdsChunk);
#pragma unroll
        for (int t = 0; t < kLdsPer; ++t) {
          const int e = t * kWave + lane;
          x[t] = e < rest ? ps[e] : 0;
          y[t] = e < rest ? pd[e] : 0;
        }
      };
      LdsPair pair;
      int queued = 0;  // uniform over the wave
      const auto drain = [&](bool all) {
        for (int steps = 0;; ++steps) {
          if (steps >= patience) {
            if (__ballot(pair.x != pair.y) && lane == 0)
              __hip_atomic_store(&gave_up, attempt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            pair = LdsPair{};
            steps = 0;
          }
          if (queued > 0) {
            const bool idle = pair.x == pair.y;
            const uint64_t mk = __ballot(idle);
            const int at = queued - 1 - lanes_below(mk);
            if (idle && at >= 0) {
              const uint32_t v = q[at];
              pair = LdsPair{(int)(v >> 16), (int)(v & 0xffff), -1};
            }
            queued = max(0, queued - (int)__popcll(mk));
          } else if (!all || __ballot(pair.x != pair.y) == 0) {
            return;
          }
          pair.step(par);
        }
      };
      load(wave);
      int g = 0;
      for (int i = wave; i < count; i += kWaves) {
        const int c0 = chunk_of(i) * kLdsChunk;
        int a[kLdsPer], b[kLdsPer];
        // the graph of the chunk's first pair; chunks only move forward
        while (g < k - 1 && __builtin_amdgcn_readfirstlane(se[g + 1]) <= c0) ++g;
        if (c0 + kLdsChunk <= __builtin_amdgcn_readfirstlane(se[g + 1]) || g == k - 1) {
          const int base = __builtin_amdgcn_readfirstlane(sv[g]);
          const int end = min(__builtin_amdgcn_readfirstlane(sv[g + 1]), nv);
          const unsigned size = (unsigned)max(end - base, 0);
          bool bad = false;
#pragma unroll
          for (int t = 0; t < kLdsPer; ++t) {
            const bool ok = (unsigned)x[t] < size && (unsigned)y[t] < size;
            bad |= !ok && c0 + t * kWave + lane < ne;
            a[t] = ok ? base + x[t] : 0;
            b[t] = ok ? base + y[t] : 0;
          }
          if (bad) atomicOr(&badbits[g >> 5], 1u << (g & 31));
        } else {  // the chunk holds pairs of several graphs
          int own = g;
#pragma unroll
          for (int t = 0; t < kLdsPer; ++t) {
            const int e = c0 + t * kWave + lane;
            a[t] = b[t] = 0;
            if (e < ne) {
              own = find_from(se, k, own, e);
              const int base = sv[own], size = min(sv[own + 1], nv) - base;
              const bool ok = x[t] >= 0 && x[t] < size && y[t] >= 0 && y[t] < size;
              if (!ok) atomicOr(&badbits[own >> 5], 1u << (own & 31));
              a[t] = ok ? base + x[t] : 0;
              b[t] = ok ? base + y[t] : 0;
            }
          }
        }
        load(i + kWaves);  // the next chunk's pairs, while this one's are joined
        if (part == 0) {
#pragma unroll
          for (int t = 0; t < kLdsPer; ++t)
            if (a[t] != b[t]) lds_store(par, max(a[t], b[t]), min(a[t], b[t]));
          continue;
        }
#pragma unroll
        for (int t = 0; t < kLdsPer; ++t) {
          const uint32_t wa = lds_load(par, a[t]), wb = lds_load(par, b[t]);
          a[t] = half_of(wa, a[t]);
          b[t] = half_of(wb, b[t]);
        }
#pragma unroll
        for (int half = 0; half < kLdsPer; half += kLdsPer / 2) {
#pragma unroll
          for (int t = half; t < half + kLdsPer / 2; ++t) {
            const uint64_t mk = __ballot(a[t] != b[t]);
            if (a[t] != b[t]) q[queued + lanes_below(mk)] = (uint32_t)a[t] << 16 | (uint32_t)b[t];
            queued += (int)__popcll(mk);
          }
          drain(false);
        }
      }
      drain(true);
      __syncthreads();
      const bool again = gave_up == attempt;
      deep = max(deep, lds_flatten(par, nv));
      if (again) patience *= 2;
      else ++part;
    }
    int g = 0;
    for (int c0 = wave * kLdsChunk; c0 < nv; c0 += kWaves * kLdsChunk) {
      while (g < k - 1 && __builtin_amdgcn_readfirstlane(sv[g + 1]) <= c0) ++g;
      int own = g;
#pragma unroll
      for (int t = 0; t < kLdsPer; ++t) {
        const int v = c0 + t * kWave + lane;
        if (v >= nv) break;
        own = find_from(sv, k, own, v);
        label[v0 + v] = half_of(lds_load(par, v), v) - sv[own];
      }
    }
    if (status)
      for (int i = tid; i < k; i += kLdsThreads)
        status[ga + i] = badbits[i >> 5] >> (i & 31) & 1 ? PJ_EINVAL : PJ_OK;
    ga += k;
  }
  if (deepest) {
    deep = -wave_min(-deep);
    if (lane == 0 && deep > 0) atomicMax(deepest, deep);
  }
}

// ------------------------------------------------------- batches, general
// Batched: rewrite local pairs as global vertex ids (graph g's vertices start
// at voff[g]).  A pair whose ends leave its graph becomes a self-loop of
// vertex 0 and is charged to its graph.
__global__ void gerr_clear(int32_t* gerr, int G) {
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x)
    gerr[g] = 0;
}

__global__ void __launch_bounds__(256) cc_globalise(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst,
                                                    const int64_t* __restrict__ voff,
                                                    const int64_t* __restrict__ eoff, int G,
                                                    int64_t m, int32_t* __restrict__ gsrc,
                                                    int32_t* __restrict__ gdst,
                                                    int32_t* __restrict__ gerr) {
  // Each wave owns a contiguous run of chunks of kWave * kGlobPer pairs: one
  // search of the offset table per wave, then every lane follows the graph
  // boundaries forward.  A chunk's loads are all issued before use.
  constexpr int kGlobPer = 16;
  constexpr int64_t kChunk = kWave * kGlobPer;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int nwaves = (gridDim.x * blockDim.x) / kWave;
  const int lane = lane_id();
  const int64_t nchunks = (m + kChunk - 1) / kChunk;
  const int64_t per = (nchunks + nwaves - 1) / nwaves;
  const int64_t ci0 = (int64_t)wave * per;
  const int64_t ci1 = ci0 + per < nchunks ? ci0 + per : nchunks;
  if (ci0 >= ci1) return;
  int g = find_instance(eoff, G, ci0 * kChunk);
  int64_t gend = eoff[g + 1], base = voff[g], size = voff[g + 1] - base;
  for (int64_t ci = ci0; ci < ci1; ++ci) {
    int us[kGlobPer], vs[kGlobPer];
#pragma unroll
    for (int t = 0; t < kGlobPer; ++t) {
      const int64_t e = ci * kChunk + t * kWave + lane;
      us[t] = e < m ? src[e] : 0;
      vs[t] = e < m ? dst[e] : 0;
    }
    for (int t = 0; t < kGlobPer; ++t) {
      const int64_t e = ci * kChunk + t * kWave + lane;
      if (e >= m) break;
      while (e >= gend) {  // later graphs (empty ones skipped)
        ++g;
        gend = eoff[g + 1];
        base = voff[g];
        size = voff[g + 1] - base;
      }
      const bool ok = (unsigned)us[t] < (uint64_t)size && (unsigned)vs[t] < (uint64_t)size;
      gsrc[e] = ok ? (int)(base + us[t]) : 0;
      gdst[e] = ok ? (int)(base + vs[t]) : 0;
      if (!ok) publish(&gerr[g], 1);  // flags of other graphs share the line
    }
  }
}


// Batched, after the last shortcut: labels become local ids.
__global__ void __launch_bounds__(256) cc_localise(int32_t* __restrict__ label, int n,
                                                   const int64_t* __restrict__ voff, int G) {
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
    label[v] -= (int)voff[find_instance(voff, G, v)];
}

// Out-of-range pairs are charged to their own graph when the batch records
// them per graph (gerr).
__global__ void cc_status(const CcCtl* ctl, int G, const int32_t* gerr, int32_t* status) {
  const bool range = (ctl->err & kErrRange) != 0;
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x)
    status[g] = (gerr ? gerr[g] != 0 : range) ? PJ_EINVAL : PJ_OK;
}

// Sizes of a batch whose tables the host does not have: each workgroup writes
// {most vertices of a graph, most pairs of a graph} of its share and {vertices,
// pairs} of all to a place of its own (one workgroup alone reads 36 GB/s: 10^6
// graphs 0.25 ms); a table that decreases somewhere reports INT64_MAX vertices for
// the graph.
constexpr int kSizesBlocks = 16;
struct SizesOut {
  int64_t* at[kSizesBlocks];
};
__global__ void __launch_bounds__(1024) cc_sizes(const int64_t* __restrict__ voff,
                                                 const int64_t* __restrict__ eoff, int64_t G,
                                                 SizesOut to) {
  __shared__ int64_t wv[1024 / kWave], we[1024 / kWave];
  int64_t mv = 0, me = 0;
  for (int64_t g = (int64_t)blockIdx.x * 1024 + threadIdx.x; g < G; g += (int64_t)gridDim.x * 1024) {
    const int64_t dv = voff[g + 1] - voff[g], de = eoff[g + 1] - eoff[g];
    mv = max(mv, dv < 0 || de < 0 ? INT64_MAX : dv);
    me = max(me, de);
  }
  mv = -wave_min(-mv);
  me = -wave_min(-me);
  if (lane_id() == 0) {
    wv[threadIdx.x / kWave] = mv;
    we[threadIdx.x / kWave] = me;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 1024 / kWave; ++i) {
      mv = max(mv, wv[i]);
      me = max(me, we[i]);
    }
    int64_t* const out = to.at[blockIdx.x];
    out[0] = mv;
    out[1] = me;
    out[2] = voff[G];
    out[3] = eoff[G];
  }
}

inline int grid_for(int64_t n, int block, int cap) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

// Class bytes pay from where D is well past one XCD's 4 MiB L2 (its random reads
// then run at 77 G/s, those of a 4 MiB byte array at 190 G/s) and the pairs read
// through them are many: 2^22 vertices, 2^25 pairs, last part 828 us without and
// 515 us with them (planted components; 33 us to make them).
inline bool use_classes(int64_t n, int64_t m) { return n >= (3 << 19) && m >= 3 * n; }

// Sparse graphs from this size on are hooked blind first only if ids follow them.
constexpr int64_t kGatedFrom = 1 << 21;

inline int64_t hook_chunks(int64_t m) { return (m + 256 * kHookPer - 1) / (256 * kHookPer); }

struct CcBuffers {
  CcCtl* ctl = nullptr;
  uint32_t* cls = nullptr;               // class bytes, four to a word
  int32_t* left = nullptr;               // a mark per chunk of pairs (mark_left)
  int32_t* gsrc = nullptr;
  int32_t* gdst = nullptr;
  int32_t* gerr = nullptr;               // batched: per-graph out-of-range flag
  int32_t* status_tmp = nullptr;
};

size_t cc_carve(int64_t n, int64_t m, int64_t G, bool globalise, bool want_status, Workspace* ws,
                CcBuffers* b) {
  size_t bytes = 0;
  auto take = [&](auto*& ptr, size_t count) {
    using T = std::remove_pointer_t<std::remove_reference_t<decltype(ptr)>>;
    bytes += ws_bytes(count, sizeof(T));
    if (ws) ptr = ws->take<T>(count);
  };
  take(b->ctl, 1);
  if (use_classes(n, m)) take(b->cls, (size_t)((n + 3) / 4));
  take(b->left, (size_t)std::max<int64_t>(hook_chunks(m), 1));
  if (globalise) {
    take(b->gsrc, (size_t)std::max<int64_t>(m, 1));
    take(b->gdst, (size_t)std::max<int64_t>(m, 1));
    take(b->gerr, (size_t)std::max<int64_t>(G, 1));
  }
  if (want_status) take(b->status_tmp, (size_t)std::max<int64_t>(G, 1));
  return bytes;
}

// Sizes of one call, from the caller or the host's offset tables.
struct CcSizes {
  int64_t n = 0, m = 0, G = 1;
  int64_t max_n = 0, max_m = 0;  // largest graph (INT64_MAX: a table that decreases)
};

// One solve's launch state.  The steps only enqueue work; the eager call and
// the graph capture share them.
struct CcRun {
  CcSizes z;
  bool batched = false;
  const int64_t* d_voff = nullptr;
  const int64_t* d_eoff = nullptr;
  const int32_t* src = nullptr;
  const int32_t* dst = nullptr;
  int32_t* D = nullptr;         // parent array, in the caller's label buffer
  int32_t* status = nullptr;
  bool lds = false;             // every graph in one workgroup's LDS
  int64_t bin = 1;              // and the keys each workgroup answers for (graph_key)
  CcBuffers b;
  hipStream_t stream = nullptr;
  PhaseTimer* tm = nullptr;
};

// LDS or the whole device: microseconds of a workgroup with the largest graph or
// with a CU's share of all, and of the device-wide kernels' launches and
// dependent passes (few for forests, long climbs in sparse graphs with cycles,
// three parts otherwise), which then join 30000 pairs a microsecond, 75000 in
// smaller graphs.  Measured, LDS and device-wide, vertices / pairs: uniform 10000 /
// 20000 29 and 69, 20000 / 40000 48 and 80, 40000 / 80000 83 and 92, 60000 / 120000
// 122 and 85, 60000 / 80000 100 and 111, 60000 / 40000 70 and 60, 20000 / 100000 72
// and 80, 1000 / 300000 201 and 40 (1000 / 100000, still in LDS, 73 and 41); paths
// of 36000 58 and 60 (in order 55 and 48), of 60000 88 and 62; 1024 graphs of
// 2^8..2^16 vertices, 5.9 * 10^7 pairs, 344 us and 2.07 ms.
void cc_plan(CcRun& r) {
  const CcSizes& z = r.z;
  const int cus = device_info().cus;
  const double lds_us = 12 + 0.75e-3 * std::max((double)z.max_n, (z.n + 8.0 * z.G) / cus) +
                        0.5e-3 * std::max((double)z.max_m, (double)z.m / cus);
  const double device_us = (z.m <= z.n           ? 57
                            : 2 * z.m < 3 * z.n ? 110
                                                : 65 + 0.6e-3 * std::min<double>(z.n, kLdsVertices)) +
                           z.m / (z.n < kHalveSmallBelow ? 75000.0 : 30000.0);
  r.lds = z.n > 0 && z.max_n <= kLdsVertices && z.max_m <= kLdsPairs && lds_us <= device_us;
  r.bin = graph_bin(z.n, z.m, z.G, cus);
}

// Workgroups of cc_lds per set, the pairs that make a graph heavy (half a CU's
// share) and the sets: with more workgroups than CUs, a first set takes the
// heavy graphs, so that none of them starts last (1024 graphs of 2^8..2^16
// vertices: 410 us with one set, 341 us with two).
inline int cc_lds_bins(const CcRun& r) {
  return r.batched ? (int)(graph_key(r.z.n, r.z.m, r.z.G) / r.bin + 1) : 1;
}
inline int cc_lds_heavy(const CcRun& r) {
  return (int)std::min<int64_t>(kLdsPairs, r.z.m / (2 * device_info().cus));
}
inline int cc_lds_sets(const CcRun& r) {
  return cc_lds_bins(r) > device_info().cus && r.z.max_m > cc_lds_heavy(r) ? 2 : 1;
}

size_t cc_need(const CcRun& r, bool want_status, Workspace* ws, CcBuffers* b) {
  return cc_carve(r.z.n, r.z.m, r.z.G, r.batched && !r.lds, want_status, ws, b);
}

void mark(CcRun& r, const char* phase) {
  if (r.tm) r.tm->mark(phase);
}

// Enqueues the whole solve.
int cc_enqueue(CcRun& r) {
  const CcSizes& z = r.z;
  CcBuffers& b = r.b;
  hipStream_t stream = r.stream;
  const int n = (int)z.n;
  const int cus = device_info().cus;
  const int cap = cus * 16;
  const int gv = grid_for(z.n, 256, cap);
  if (r.lds) {
    int32_t* deepest = nullptr;
    if (r.tm && r.tm->on) {
      hipLaunchKernelGGL(cc_init, dim3(1), dim3(256), 0, stream, r.D, 0, b.ctl, nullptr,
                         0, nullptr, nullptr, 0);
      deepest = &b.ctl->steps;
    }
    const int bins = cc_lds_bins(r);
    hipLaunchKernelGGL(cc_lds, dim3(bins * cc_lds_sets(r)), dim3(kLdsThreads), 0, stream, r.src, r.dst,
                       z.m, n, r.d_voff, r.d_eoff, (int)z.G, r.bin, bins, cc_lds_heavy(r), r.D,
                       r.status, deepest);
    PJ_HIP(hipGetLastError());
    mark(r, "lds");
    return PJ_OK;
  }
  const int32_t* es = r.src;
  const int32_t* ed = r.dst;
  if (r.batched) {
    hipLaunchKernelGGL(gerr_clear, dim3(grid_for(z.G, 256, 1024)), dim3(256), 0, stream, b.gerr,
                       (int)z.G);
    if (z.m > 0) {
      hipLaunchKernelGGL(cc_globalise, dim3(grid_for(z.m, 256, cap)), dim3(256), 0, stream, r.src,
                         r.dst, r.d_voff, r.d_eoff, (int)z.G, z.m, b.gsrc, b.gdst, b.gerr);
      es = b.gsrc;
      ed = b.gdst;
    }
  }
  const int64_t nchunks = hook_chunks(z.m);
  const bool sparse = 2 * z.m < 3 * z.n, gated = sparse && z.n >= kGatedFrom;
  hipLaunchKernelGGL(cc_init, dim3(grid_for(z.n / 4, 256, cap) + gated), dim3(256), 0, stream,
                     r.D, n, b.ctl, b.left, nchunks, es, ed, gated ? z.m : 0);
  PJ_HIP(hipGetLastError());
  mark(r, "init");
  const auto flatten = [&](const int32_t* only_if = nullptr) {
    const int threads = only_if ? 1024 : 256;
    hipLaunchKernelGGL(only_if ? cc_flatten<1024> : cc_flatten<256>,
                       dim3(grid_for(z.n, threads * kFlatPer, INT32_MAX)), dim3(threads), 0, stream,
                       r.D, n, only_if, b.ctl);
    mark(r, "shortcut");
  };
  const auto hook_blind = [&](int64_t stride, const int32_t* only_if) {
    const int64_t units = (nchunks + stride - 1) / stride;
    const int groups = only_if ? grid_for(units, 1, 8 * cus) : grid_for(units, 1, cap) + 1;
    hipLaunchKernelGGL(cc_hook_blind, dim3(groups), dim3(256), 0, stream, es, ed, z.m, n, r.D,
                       stride, units, only_if, b.ctl);
    mark(r, "hook_blind");
  };
  if (z.m > 0) {
    const Climb climb = z.n < kHalveSmallBelow ? kClimbSmall : kClimbLarge;
    const auto hook = [&](int64_t stride, int64_t chunks) {
      // two pairs a thread where eight would leave CUs without work (200000
      // vertices in paths 73 us instead of 91); no more of them at once than
      // that in a graph with many pairs, whose joins meet at few roots (300000
      // vertices, 450000 pairs: 127 us with eight, 212 with two)
      const bool few = chunks < cus / (stride > 1 ? 4 : 2);
      const int64_t units = few ? chunks * (kHookPer / 2) : chunks;
      hipLaunchKernelGGL(few ? cc_hook<2> : cc_hook<kHookPer>, dim3(grid_for(units, 1, cap)),
                         dim3(256), 0, stream, es, ed, z.m, n, r.D, stride, units, climb, b.left,
                         stride > 1 ? kForRest : kForLast, b.ctl);
      mark(r, "hook");
    };
    if (sparse) {
      // Paths, trees and sparser: all pairs blind, a shortcut, and swaps.  Where the
      // ids follow the graph the first settles nearly all (10^6 vertices in rings
      // of 100 in order: 58 us, 364 with swaps alone).  With random ids almost
      // every pair joins two trees, so a large graph spares nothing by it: 64
      // paths, 8 M pairs, 700 us with swaps alone, 530 of them for the swaps and
      // the reads of both ends, which run at 27 and 63 G/s, and 790 with all three;
      // 10^6 vertices 179 and 176.
      hook_blind(1, gated ? &b.ctl->ordered : nullptr);
      flatten(gated ? &b.ctl->ordered : nullptr);
      hook(1, nchunks);
    } else {
      // Blind hooks of about two pairs a vertex, swaps of half a pair a vertex,
      // each on a flat forest, and the rest, most of which is settled by then.
      // Swapping all pairs at once climbs unfinished trees: 2^22 vertices and
      // 2^25 pairs 2480 us, in parts 950 us; 10^6 and 2.2 * 10^6 473 and 215.
      // Four chunks are hooked blind and two swapped, at least, of each graph: without
      // them the rest would all meet at few roots (1000 vertices and 10^7 pairs
      // 350 us, with them 80).
      const int64_t spread = std::max<int64_t>(1, nchunks / (4 * z.G));
      hook_blind(std::max<int64_t>(1, std::min(z.m / z.n / 2, spread)), nullptr);
      flatten();
      const int64_t stride = std::max<int64_t>(2, std::min(2 * (z.m / z.n), 2 * spread));
      const int64_t swapped = nchunks / stride;
      if (swapped > 0) {
        hook(stride, swapped);
        flatten();
      }
      if (b.cls) {
        hipLaunchKernelGGL(cc_class_pick, dim3(1), dim3(1024), 0, stream, (const int32_t*)r.D, n,
                           b.ctl);
        hipLaunchKernelGGL(cc_class_fill, dim3(grid_for(z.n / 4, 256, cap)), dim3(256), 0, stream,
                           (const int32_t*)r.D, n, (const CcCtl*)b.ctl, b.cls);
        mark(r, "classes");
      }
      hipLaunchKernelGGL(cc_hook_rest, dim3(grid_for(nchunks - swapped, 1, cap)), dim3(256), 0,
                         stream, es, ed, z.m, n, r.D, (const uint8_t*)b.cls, stride,
                         nchunks - swapped, swapped, b.left, b.ctl);
      mark(r, "hook_rest");
    }
    flatten();
    const int gl = grid_for(nchunks, 1, 4 * cus);
    hipLaunchKernelGGL(cc_join_left, dim3(gl), dim3(256), 0, stream, es, ed, z.m, n, r.D, nchunks,
                       (const int32_t*)b.left, b.ctl);
    mark(r, "hook_left");
    flatten(&b.ctl->redo);
  }
  if (r.batched && z.n > 0) {
    hipLaunchKernelGGL(cc_localise, dim3(gv), dim3(256), 0, stream, r.D, n, r.d_voff, (int)z.G);
    mark(r, "localise");
  }
  PJ_HIP(hipGetLastError());
  if (r.status && z.G > 0) {
    hipLaunchKernelGGL(cc_status, dim3(grid_for(z.G, 256, 1024)), dim3(256), 0, stream,
                       (const CcCtl*)b.ctl, (int)z.G,
                       r.batched ? (const int32_t*)b.gerr : nullptr, r.status);
    PJ_HIP(hipGetLastError());
  }
  return PJ_OK;
}

int cc_check_args(const int32_t* src, const int32_t* dst, int64_t n, int64_t m, int64_t G,
                  int32_t* label) {
  if (n < 0 || m < 0 || G < 0 || n >= INT32_MAX || m >= (int64_t(1) << 40)) return PJ_EINVAL;
  if (n > 0 && !label) return PJ_EINVAL;
  if (m > 0 && (!src || !dst)) return PJ_EINVAL;
  if (m > 0 && ((const void*)label == (const void*)src || (const void*)label == (const void*)dst))
    return PJ_EINVAL;
  if (m > 0 && n == 0) return PJ_EINVAL;
  return PJ_OK;
}

int cc_setup(CcRun& r, const int32_t* src, const int32_t* dst, const CcSizes& z,
             const int64_t* d_voff, const int64_t* d_eoff, int32_t* label, hipStream_t stream) {
  PJ_TRY(cc_check_args(src, dst, z.n, z.m, z.G, label));
  r.z = z;
  r.src = src;
  r.dst = dst;
  r.batched = d_voff != nullptr;
  r.d_voff = d_voff;
  r.d_eoff = d_eoff;
  r.D = label;
  r.stream = stream;
  cc_plan(r);
  return PJ_OK;
}

// validate without d_status: the first graph's status, read back.
int cc_read_status(const CcRun& r) {
  if (r.z.G <= 0) return PJ_OK;
  int32_t hs = 0;
  PJ_HIP(hipMemcpyAsync(&hs, r.status, sizeof hs, hipMemcpyDeviceToHost, r.stream));
  PJ_HIP(hipStreamSynchronize(r.stream));
  return hs;
}

int cc_impl(const int32_t* src, const int32_t* dst, const CcSizes& z, const int64_t* d_voff,
            const int64_t* d_eoff, int32_t* label, const pj_opts* user, hipStream_t stream) {
  CcRun r;
  PJ_TRY(cc_setup(r, src, dst, z, d_voff, d_eoff, label, stream));
  pj_opts o = resolved_opts(user);
  pj_stats* st = user ? user->stats : nullptr;
  if (st) *st = pj_stats{};
  const bool want_status = o.validate && !o.d_status;
  if (z.n == 0 && !o.d_status) return PJ_OK;

  // a workspace too small for the device-wide solve is refused on either path
  if (o.workspace &&
      o.workspace_bytes < cc_carve(z.n, z.m, z.G, r.batched, want_status, nullptr, &r.b))
    return PJ_EINVAL;
  Workspace ws;
  if (!r.lds || want_status || st) {  // the LDS solve itself needs no memory
    PJ_TRY(workspace_acquire(ws, cc_need(r, want_status, nullptr, &r.b), &o, stream));
    cc_need(r, want_status, &ws, &r.b);
  }
  r.status = o.d_status ? o.d_status : r.b.status_tmp;

  PhaseTimer tm;
  PJ_TRY(tm.begin(st != nullptr, stream));
  r.tm = &tm;
  PJ_TRY(cc_enqueue(r));
  int result = PJ_OK;
  if (want_status) result = cc_read_status(r);
  if (st) {
    PJ_TRY(tm.finish(st));
    st->algo = PJ_ALGO_SV;
    CcCtl hc{};
    PJ_HIP(hipMemcpyAsync(&hc, r.b.ctl, sizeof hc, hipMemcpyDeviceToHost, stream));
    PJ_HIP(hipStreamSynchronize(stream));
    st->rounds = 1 + hc.steps;
    st->level_nodes[0] = z.n;
    st->status = result;
  }
  PJ_TRY(workspace_release(ws));
  return result;
}

// ------------------------------------------------------------ graph replay
// A components solve captured once into a hipGraph and replayed.  The cache
// owns the workspace; the key holds every address and size the capture used,
// and the choice of path, which follows from the largest graph.
using CcGraphKey = std::array<int64_t, 13>;
struct CcGraphEntry {
  hipGraphExec_t exec = nullptr;
  void* ws = nullptr;
  size_t ws_bytes = 0;
  uint64_t last_used = 0;
};
std::mutex g_ccg_mu;
std::map<CcGraphKey, CcGraphEntry> g_ccg;
uint64_t g_ccg_clock = 0;
constexpr size_t kMaxCcGraphs = 8;
std::map<int, hipStream_t> g_ccg_capture;

void cc_graph_drop(CcGraphEntry& e) {
  if (e.exec) (void)hipGraphExecDestroy(e.exec);
  if (e.ws) (void)hipFree(e.ws);
  e = CcGraphEntry{};
}

int cc_graph(const int32_t* src, const int32_t* dst, const CcSizes& z, const int64_t* d_voff,
             const int64_t* d_eoff, int32_t* label, const pj_opts& o, hipStream_t stream) {
  CcRun r;
  PJ_TRY(cc_setup(r, src, dst, z, d_voff, d_eoff, label, stream));
  const bool want_status = o.validate && !o.d_status;
  if (z.n == 0 && !o.d_status) return PJ_OK;
  int dev = 0;
  PJ_HIP(hipGetDevice(&dev));
  const CcGraphKey key{dev,
                       (int64_t)(uintptr_t)src,
                       (int64_t)(uintptr_t)dst,
                       (int64_t)(uintptr_t)d_voff,
                       (int64_t)(uintptr_t)d_eoff,
                       (int64_t)(uintptr_t)label,
                       (int64_t)(uintptr_t)o.d_status,
                       z.G,
                       z.n,
                       z.m,
                       want_status ? 1 : 0,
                       r.lds ? 1 : 0,
                       r.lds ? cc_lds_sets(r) : 0};
  std::lock_guard<std::mutex> lk(g_ccg_mu);
  auto it = g_ccg.find(key);
  CcGraphEntry fresh;
  CcGraphEntry* e = nullptr;
  if (it != g_ccg.end()) {
    e = &it->second;
  } else {
    if (g_ccg.size() >= kMaxCcGraphs) {  // evict the least recently used
      auto lru = g_ccg.begin();
      for (auto j = g_ccg.begin(); j != g_ccg.end(); ++j)
        if (j->second.last_used < lru->second.last_used) lru = j;
      cc_graph_drop(lru->second);
      g_ccg.erase(lru);
    }
    fresh.ws_bytes = std::max<size_t>(cc_need(r, want_status, nullptr, &r.b), 256);
    PJ_HIP(hipMalloc(&fresh.ws, fresh.ws_bytes));
    e = &fresh;
  }
  Workspace ws;
  ws.base = static_cast<char*>(e->ws);
  ws.size = e->ws_bytes;
  cc_need(r, want_status, &ws, &r.b);
  r.status = o.d_status ? o.d_status : r.b.status_tmp;
  if (it == g_ccg.end()) {
    hipStream_t& cap = g_ccg_capture[dev];
    if (!cap && hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess) {
      cc_graph_drop(fresh);
      return PJ_EHIP;
    }
    r.stream = cap;
    hipGraph_t graph = nullptr;
    hipError_t he = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    int rc = he == hipSuccess ? PJ_OK : PJ_EHIP;
    if (rc == PJ_OK) rc = cc_enqueue(r);
    if (he == hipSuccess) he = hipStreamEndCapture(cap, &graph);
    if (rc == PJ_OK && he == hipSuccess)
      he = hipGraphInstantiate(&fresh.exec, graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
    if (rc != PJ_OK || he != hipSuccess) {
      cc_graph_drop(fresh);
      if (rc != PJ_OK) return rc;
      set_last_hip_error(he, "graph capture of components", __FILE__, __LINE__);
      return PJ_EHIP;
    }
    e = &g_ccg.emplace(key, fresh).first->second;
    r.stream = stream;
  }
  e->last_used = ++g_ccg_clock;
  PJ_HIP(hipGraphLaunch(e->exec, stream));
  return want_status ? cc_read_status(r) : PJ_OK;
}

// Sizes of a batch from the host's tables, or read from the device's.
int cc_batch_sizes(const int64_t* d_voff, const int64_t* d_eoff, int64_t G, const pj_opts* opts,
                   hipStream_t stream, CcSizes* z) {
  z->G = G;
  const int64_t* hv = opts ? opts->h_offsets : nullptr;
  const int64_t* he = opts ? opts->h_edge_offsets : nullptr;
  if (hv && he) {
    z->n = hv[G];
    z->m = he[G];
    z->max_n = largest_instance(hv, G);
    z->max_m = largest_instance(he, G);
    if (z->max_m == INT64_MAX) z->max_n = INT64_MAX;
    return PJ_OK;
  }
  std::array<PinnedWord, kSizesBlocks> pinned;  // 64 bytes each that the device can write
  SizesOut to = {};
  const int blocks = (int)std::min<int64_t>(kSizesBlocks, (G + 4095) / 4096);
  for (int b = 0; b < blocks; ++b) {
    to.at[b] = reinterpret_cast<int64_t*>(pinned[b].get());
    if (!to.at[b]) return PJ_ENOMEM;
  }
  hipLaunchKernelGGL(cc_sizes, dim3(blocks), dim3(1024), 0, stream, d_voff, d_eoff, G, to);
  PJ_HIP(hipGetLastError());
  PJ_HIP(hipStreamSynchronize(stream));
  for (int b = 0; b < blocks; ++b) {
    z->max_n = std::max(z->max_n, to.at[b][0]);
    z->max_m = std::max(z->max_m, to.at[b][1]);
  }
  z->n = to.at[0][2];
  z->m = to.at[0][3];
  return PJ_OK;
}

}  // namespace

void cc_graph_cache_clear() {
  std::lock_guard<std::mutex> lk(g_ccg_mu);
  (void)hipDeviceSynchronize();
  for (auto& kv : g_ccg) cc_graph_drop(kv.second);
  g_ccg.clear();
}

// Bytes reported to callers and charged to a server's budget: what the device-wide
// solve of a batch of these sizes takes, the most of any path.
size_t cc_workspace(int64_t n, int64_t m, int64_t G, const pj_opts* user) {
  const pj_opts o = resolved_opts(user);
  CcBuffers b;
  return cc_carve(n, m, G, true, o.validate && !o.d_status, nullptr, &b);
}

}  // namespace pj

extern "C" {

int pj_connected_components_ex(const int32_t* src, const int32_t* dst, int64_t n, int64_t m,
                               int32_t* label, const pj_opts* opts, pj_stream_t stream) {
  pj::CcSizes z;
  z.n = z.max_n = n;
  z.m = z.max_m = m;
  if (opts && opts->use_graph && !opts->stats)
    return pj::cc_graph(src, dst, z, nullptr, nullptr, label, *opts, (hipStream_t)stream);
  return pj::cc_impl(src, dst, z, nullptr, nullptr, label, opts, (hipStream_t)stream);
}

int pj_connected_components(const int32_t* src, const int32_t* dst, int64_t n, int64_t m,
                            int32_t* label, pj_stream_t stream) {
  return pj_connected_components_ex(src, dst, n, m, label, nullptr, stream);
}

int pj_connected_components_batched_ex(const int32_t* src, const int32_t* dst,
                                       const int64_t* vtx_off, const int64_t* edge_off,
                                       int64_t G, int32_t* label, const pj_opts* opts,
                                       pj_stream_t stream) {
  if (!vtx_off || !edge_off || G < 0) return PJ_EINVAL;
  if (G == 0) return PJ_OK;
  pj::CcSizes z;
  PJ_TRY(pj::cc_batch_sizes(vtx_off, edge_off, G, opts, (hipStream_t)stream, &z));
  if (opts && opts->use_graph && !opts->stats)
    return pj::cc_graph(src, dst, z, vtx_off, edge_off, label, *opts, (hipStream_t)stream);
  return pj::cc_impl(src, dst, z, vtx_off, edge_off, label, opts, (hipStream_t)stream);
}

int pj_connected_components_batched(const int32_t* src, const int32_t* dst,
                                    const int64_t* vtx_off, const int64_t* edge_off, int64_t G,
                                    int32_t* label, pj_stream_t stream) {
  return pj_connected_components_batched_ex(src, dst, vtx_off, edge_off, G, label, nullptr,
                                            stream);
}

size_t pj_cc_workspace_bytes(int64_t n, int64_t m, int64_t G, const pj_opts* opts) {
  if (n < 0 || m < 0 || G < 1) return 0;
  // one graph may go through either entry point: sized for the batched one
  return pj::cc_workspace(n, m, G, opts);
}

}  // extern "C"
