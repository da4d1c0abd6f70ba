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
// concurrent stores; a compare and swap needs none of them.
//
#include <algorithm>
#include <array>
#include <cmath>
#include <cstddef>
#include <map>
#include <mutex>
#include <vector>

#include "pj_internal.hpp"

namespace pj {
namespace {

constexpr int kFlatHops = 24;   // parent steps of one vertex in one shortcut pass
constexpr int kMaxFlat = 3 * 7; // shortcut passes: three times, and 25^7 > 2^31

constexpr int kClasses = 255;

struct CcCtl {
  int32_t err;
  int32_t steps;                // longest chain of parent steps of a shortcut pass
  int32_t more[kMaxFlat];       // shortcut pass i left vertices short of their root
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
// first, so the loop ends after at most x + y steps even on stale values;
// after `halve` steps it halves the path, which keeps long chains (paths whose
// ids follow their order) from being climbed link by link.  In a large forest
// that starts late: the stores of a giant component's pairs go to the few
// nodes under its root and serialise there (2^20 pairs of a 2^22-vertex uniform
// graph on a quarter of the roots: 450 us from the 3rd step on, 240 us from the
// 16th); a small one is bound by the chain of reads instead (300000 vertices:
// 70 us against 79 us).
constexpr int kHalveSmall = 3, kHalveLarge = 16;
constexpr int64_t kHalveSmallBelow = 1 << 20;

__device__ __forceinline__ void join(int32_t* D, int x, int y, int halve) {
  for (int step = 1; x != y; ++step) {
    const int hi = max(x, y);
    y = min(x, y);
    x = hi;
    int p = load_coherent(&D[x]);
    if (p == x) {
      p = atomicCAS(&D[x], x, y);
      if (p == x) return;
    } else if (step > halve) {
      const int g = load_coherent(&D[p]);
      if (g != p) publish(&D[x], g);
      p = g;
    }
    x = p;
  }
}

__global__ void __launch_bounds__(256) cc_init(int32_t* __restrict__ D, int n, CcCtl* ctl) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int stride = gridDim.x * blockDim.x;
  const int n4 = (reinterpret_cast<uintptr_t>(D) & 15) == 0 ? n >> 2 : 0;
  for (int q = tid; q < n4; q += stride)
    reinterpret_cast<int4*>(D)[q] = make_int4(4 * q, 4 * q + 1, 4 * q + 2, 4 * q + 3);
  for (int v = 4 * n4 + tid; v < n; v += stride) D[v] = v;
  if (tid < (int)(offsetof(CcCtl, parents) / 4)) reinterpret_cast<int32_t*>(ctl)[tid] = 0;
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

// First hooks of a graph with many pairs, blind: every stride-th chunk's pairs
// store their smaller end as the larger end's parent, no read and no swap (85
// G stores/s against 27 G swaps/s).  One of the pairs of a vertex wins; the
// others join nothing yet, and cc_hook_rest reads all of them again.
constexpr int kHookPer = 8;

__global__ void __launch_bounds__(256) cc_hook_blind(const int32_t* __restrict__ src,
                                                     const int32_t* __restrict__ dst, int64_t m,
                                                     int n, int32_t* __restrict__ D,
                                                     int64_t stride, int64_t units, CcCtl* ctl) {
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units; i += gridDim.x) {
    int x[kHookPer], y[kHookPer];
    bad |= load_pairs(src, dst, m, n, i * stride * kHookPer, x, y);
#pragma unroll
    for (int t = 0; t < kHookPer; ++t)
      if (x[t] != y[t]) D[max(x[t], y[t])] = min(x[t], y[t]);
  }
  report(ctl, bad);
}

// Hooks the pairs of the chunks stride - 1, 2 * stride - 1, ...
template <int kPer>
__global__ void __launch_bounds__(256) cc_hook(const int32_t* __restrict__ src,
                                               const int32_t* __restrict__ dst, int64_t m, int n,
                                               int32_t* D, int64_t stride, int64_t units,
                                               int halve, CcCtl* ctl) {
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units; i += gridDim.x) {
    int x[kPer], y[kPer];
    constexpr int kParts = kHookPer / kPer;
    const int64_t c = (i / kParts + 1) * stride - 1;
    bad |= load_pairs(src, dst, m, n, c * kHookPer + i % kParts * kPer, x, y);
#pragma unroll
    for (int t = 0; t < kPer; ++t) join(D, x[t], y[t], halve);
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

// Hooks the pairs of all the other chunks, most of which lie in one tree by
// now: two reads (of classes, or of D) settle those, the rest is gathered in
// LDS first so that the lanes of a wave climb together.
template <bool kClassed>
__device__ __forceinline__ void hook_rest(const int32_t* __restrict__ src,
                                          const int32_t* __restrict__ dst, int64_t m, int n,
                                          int32_t* D, const uint8_t* __restrict__ cls,
                                          int64_t stride, int64_t units, CcCtl* ctl, int2* queue,
                                          int* queued) {
  bool bad = false;
  for (int64_t i = blockIdx.x; i < units; i += gridDim.x) {
    int x[kHookPer], y[kHookPer];
    bad |= load_pairs(src, dst, m, n, (i / (stride - 1) * stride + i % (stride - 1)) * kHookPer, x, y);
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
    for (int q = threadIdx.x; q < total; q += 256) join(D, queue[q].x, queue[q].y, kHalveLarge);
    __syncthreads();  // the queue is reused by the next chunk
  }
  report(ctl, bad);
}

__global__ void __launch_bounds__(256) cc_hook_rest(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst, int64_t m,
                                                    int n, int32_t* D,
                                                    const uint8_t* __restrict__ cls,
                                                    int64_t stride, int64_t units, CcCtl* ctl) {
  __shared__ int2 queue[256 * kHookPer];
  __shared__ int queued;
  if (cls && ctl->classes > 0)
    hook_rest<true>(src, dst, m, n, D, cls, stride, units, ctl, queue, &queued);
  else
    hook_rest<false>(src, dst, m, n, D, cls, stride, units, ctl, queue, &queued);
}

// Shortcut: D[v] <- its root, or the ancestor kFlatHops + 1 steps up.  A pass
// divides the depth of every tree by kFlatHops + 1 at least (the reads return
// values no older than the kernel's start), so ceil(log25 n) passes flatten any
// forest; hooks leave depths far below 24, and a pass that leaves nothing over
// makes the later ones return at once.
__global__ void __launch_bounds__(256) cc_flatten(int32_t* D, int n, CcCtl* ctl, int pass,
                                                  int if_more) {
  if (if_more && ctl->more[pass - 1] == 0) return;
  const int stride = gridDim.x * blockDim.x;
  int most = 0;
  bool more = false;
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int p0 = D[v];
    int p = p0, h = 0;
    for (; h < kFlatHops; ++h) {
      const int g = D[p];
      if (g == p) break;
      p = g;
    }
    if (p != p0) D[v] = p;
    more |= h == kFlatHops;
    most = max(most, h);
  }
  most = -wave_min(-most);
  if (lane_id() == 0 && most > 1 && load_coherent(&ctl->steps) < most) atomicMax(&ctl->steps, most);
  raise_flag(&ctl->more[pass], more);
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

struct CcBuffers {
  CcCtl* ctl = nullptr;
  uint32_t* cls = nullptr;               // class bytes, four to a word
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
  CcBuffers b;
  hipStream_t stream = nullptr;
  PhaseTimer* tm = nullptr;
};

size_t cc_need(const CcRun& r, bool want_status, Workspace* ws, CcBuffers* b) {
  return cc_carve(r.z.n, r.z.m, r.z.G, r.batched, want_status, ws, b);
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
  const int cap = device_info().cus * 16;
  const int gv = grid_for(z.n, 256, cap);
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
  hipLaunchKernelGGL(cc_init, dim3(grid_for(z.n / 4, 256, cap)), dim3(256), 0, stream, r.D, n,
                     b.ctl);
  PJ_HIP(hipGetLastError());
  mark(r, "init");
  int pass = 0;
  int passes = 1;
  for (int64_t reach = kFlatHops + 1; reach < z.n; reach *= kFlatHops + 1) ++passes;
  // later passes mostly have nothing to do: a small grid returns sooner
  const auto flatten = [&] {
    for (int i = 0; i < passes; ++i, ++pass)
      hipLaunchKernelGGL(cc_flatten, dim3(i > 0 ? std::min(gv, cap / 4) : gv), dim3(256), 0,
                         stream, r.D, n, b.ctl, pass, i > 0 ? 1 : 0);
    mark(r, "shortcut");
  };
  if (z.m > 0) {
    const int64_t nchunks = (z.m + 256 * kHookPer - 1) / (256 * kHookPer);
    const int halve = z.n < kHalveSmallBelow ? kHalveSmall : kHalveLarge;
    const auto hook = [&](int64_t stride, int64_t chunks) {
      // two pairs a thread where eight would leave CUs without work (200000
      // vertices in paths 105 us instead of 125); no more of them at once than
      // that in a graph with many pairs, whose joins meet at few roots (300000
      // vertices, 450000 pairs: 155 us with eight, 240 with two)
      const bool few = chunks < device_info().cus / (stride > 1 ? 4 : 2);
      const int64_t units = few ? chunks * (kHookPer / 2) : chunks;
      hipLaunchKernelGGL(few ? cc_hook<2> : cc_hook<kHookPer>, dim3(grid_for(units, 1, cap)),
                         dim3(256), 0, stream, es, ed, z.m, n, r.D, stride, units, halve, b.ctl);
      mark(r, "hook");
    };
    if (2 * z.m < 3 * z.n) {
      // Paths, trees and sparser: almost every pair joins two trees, so nothing
      // is spared by parts (64 paths, 8 M pairs: 530 us for the swaps and the
      // reads of both ends, which run at 27 and 63 G/s).
      hook(1, nchunks);
    } else {
      // Blind hooks of about two pairs a vertex, swaps of half a pair a vertex,
      // each on a flat forest, and the rest, most of which is settled by then.
      // Swapping all pairs at once climbs unfinished trees: 2^22 vertices and
      // 2^25 pairs 1780 us, in parts 980 us; 10^6 and 2.2 * 10^6 530 and 280.
      const int64_t blind_stride = std::max<int64_t>(1, z.m / z.n / 2);
      const int64_t blind = (nchunks + blind_stride - 1) / blind_stride;
      hipLaunchKernelGGL(cc_hook_blind, dim3(grid_for(blind, 1, cap)), dim3(256), 0, stream, es,
                         ed, z.m, n, r.D, blind_stride, blind, b.ctl);
      mark(r, "hook_blind");
      flatten();
      const int64_t stride = std::max<int64_t>(2, 2 * (z.m / z.n));
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
                         nchunks - swapped, b.ctl);
      mark(r, "hook_rest");
    }
    flatten();
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

  Workspace ws;
  PJ_TRY(workspace_acquire(ws, cc_need(r, want_status, nullptr, &r.b), &o, stream));
  cc_need(r, want_status, &ws, &r.b);
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
using CcGraphKey = std::array<int64_t, 14>;
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
                       0,
                       0,
                       0};
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
    return PJ_OK;
  }
  int64_t tmp[2] = {0, 0};
  PJ_HIP(hipMemcpyAsync(&tmp[0], d_voff + G, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
  PJ_HIP(hipMemcpyAsync(&tmp[1], d_eoff + G, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
  PJ_HIP(hipStreamSynchronize(stream));
  z->n = tmp[0];
  z->m = tmp[1];
  return PJ_OK;
}

}  // namespace

void cc_graph_cache_clear() {
  std::lock_guard<std::mutex> lk(g_ccg_mu);
  (void)hipDeviceSynchronize();
  for (auto& kv : g_ccg) cc_graph_drop(kv.second);
  g_ccg.clear();
}

// Bytes reported to callers and charged to a server's budget.  The solve
// needs less; the figure is the one that budgets were made for (two stamps and
// a bit per vertex, two lists of pairs, the slices of their chunks, the flags
// of every round up to a bound, and a batch's pairs), so that a budget admits
// the requests it always did.
size_t cc_workspace(int64_t n, int64_t m, int64_t G, const pj_opts* user) {
  pj_opts o = resolved_opts(user);
  const bool status = o.validate && !o.d_status;
  CcBuffers b;
  const double lg = n > 1 ? std::floor(std::log((double)n) / std::log(1.5)) : 0.0;
  const size_t rounds = 4 * ((size_t)lg + 2) + 2;
  const size_t nn = (size_t)std::max<int64_t>(n, 1), mm = (size_t)std::max<int64_t>(m, 1);
  size_t bytes = ws_bytes(1, 8) + 2 * ws_bytes(nn, 4) + 2 * ws_bytes(rounds, 4) +
                 ws_bytes(rounds, 8) + ws_bytes(8 * rounds, 4) + ws_bytes((nn + 63) / 64, 8) +
                 2 * ws_bytes(mm, 8) + ws_bytes((mm + 2047) / 2048 * 9, 4) + 2 * ws_bytes(mm, 4) +
                 ws_bytes((size_t)std::max<int64_t>(G, 1), 4);
  if (status) bytes += ws_bytes((size_t)std::max<int64_t>(G, 1), 4);
  return std::max(bytes, cc_carve(n, m, G, true, status, nullptr, &b));
}

}  // namespace pj

extern "C" {

int pj_connected_components_ex(const int32_t* src, const int32_t* dst, int64_t n, int64_t m,
                               int32_t* label, const pj_opts* opts, pj_stream_t stream) {
  pj::CcSizes z;
  z.n = n;
  z.m = m;
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
