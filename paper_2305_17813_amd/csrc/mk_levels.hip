// Distance-only ("vanilla") traversals: BFS levels, level-synchronous and
// direction-optimizing, and SSSP distances by near-far relaxation (further down).
//
// The experimental section runs BFS in two variants: a vanilla one with 32-bit atomics that
// computes only distances, and the tree variant (64-bit <distance, parent> nodes) that the
// dynamic algorithms need; its static BFS is level-based.  This file is the vanilla variant:
// one u32 level per vertex, one level per step, and a byte per vertex for marks.  A step
// is either top-down (the frontier's out-arcs claim unreached vertices by CAS, or, when there are
// many, mark their bytes for a sweep over the vertices) or bottom-up (every unreached vertex scans its
// in-arcs, through the reverse view, for a vertex of the current level and stops at the
// first one).  A one-thread kernel picks the direction of each step on the device from the
// frontier's size and out-arc count against the number of unreached vertices, so the host
// only reads sizes back after 4, 8, 16 and 32 levels, then every 16.
//
// The rule is Beamer's direction optimization recast for slabs.  A top-down step reads a slab
// per frontier vertex and makes a random level read (and, for an unreached target, a CAS) per
// out-arc; a bottom-up step reads at least one slab per unreached vertex and a level per
// in-arc it scans until it meets the current level, and every bottom-up step also reads the
// level of every vertex.  Counting a slab as two random accesses, bottom-up is taken when
// 2 nf + mf > 6 nu + N / 2  (nf, mf: frontier vertices and out-arcs; nu: unreached
// vertices).  On a power-law graph the hub's neighbourhood passes this at once (few vertices,
// very many arcs).  On a road network the frontier has as few arcs per vertex as the
// unreached part and most unreached vertices find no parent, so bottom-up steps there cost
// more than top-down ones (measured); the N / 2 term keeps such a graph top-down.
#include <rocprim/device/device_scan.hpp>

#include <algorithm>

#include "mk_internal.h"

using namespace mk;

namespace {

constexpr uint32_t kLevelInf = 0xFFFFFFFFu;
constexpr uint32_t kChunk = kGroup;       // buckets of a multi-bucket vertex per work item
constexpr uint32_t kSyncFirst = 4, kSyncMax = 16;  // steps between size read-backs: 4, 4,
                                                    // then doubling while the traversal lasts

// How a step reaches vertices.  With few arcs the unreached neighbours are claimed by CAS, which go
// to memory at 5.7 G/s whatever else the step does.  Past N / kMarkShare arcs the step only sets a
// byte per neighbour, and a sweep over all vertices, 14 ps a vertex, collects what has a byte and
// no level: as much as the CAS of an N / 13th of the vertices, and on a road-like network about a
// quarter of the arcs reach something new (1,048,576 vertices, levels of up to 80,000 arcs: 1.69 ms
// with a share of 16, 1.23 with this one).  The great step of an R-MAT graph at scale 22: 456 us
// claiming, 365 marking and sweeping; 20 M reads of its 16 MB of levels brought 16 M lines into the
// L2s, the bytes mostly stay there.  A claiming step leaves the bytes alone: testing and setting them
// as well cost the road-like grid of 16.8 M vertices a line more per vertex (36 to 42 us a level).
//
// A traversal that may step bottom-up launches the sweep for every level anyway.  One that may not would
// launch it for nothing at most levels, so it marks and sweeps only on graphs of kSweepDense arcs a vertex,
// or of kSweepLeast vertices and 8 arcs a vertex, and claims on all others (with sweeps / without, us:
// 5,000 vertices, degree 150: 104 / 115, 100,000, degree 30: 180 / 199, R-MAT scale 16, edge factor 32: 201 /
// 219; 2^20 vertices, degree 8: 535 / 590, R-MAT scale 20, edge factor 16: 470 / 490; but edge factor 4: 362 /
// 336, scale 18, edge factors 4 and 8: 277 / 250, 250 / 238, 4,096 vertices of degree 4, 8 and 32: 325 / 283,
// 158 / 147, 89 / 83, grids of side 64: 455 / 350, 2,048: 1,620 / 1,437).
constexpr uint32_t kClaim = 0, kBottomUp = 1, kMark = 2, kMarkShare = 2;
constexpr uint32_t kSweepLeast = 1u << 20, kSweepDense = 24;

// Device counters of one call (in the caller's workspace).  Level L uses slot L mod 4.
struct LvCnt {
  uint32_t n[4];                // frontier sizes
  uint32_t nm[4];               // multi-bucket work items of the level's top-down step
  uint32_t mode, last;          // how the current step and the one before it reach vertices
  uint32_t bu_steps;            // bottom-up steps taken
  uint32_t reached;             // vertices reached before the current frontier, and its place in the
                                // queue: every vertex is queued once, frontier after frontier
  uint32_t pad[4];
  unsigned long long arcs[4];   // out-arcs of each frontier
};
static_assert(sizeof(LvCnt) <= 256, "counter block (and at most 64 pinned words of 8 bytes)");

// Every vertex unreached: no level, no mark.
__global__ void k_lv_fill(uint32_t* level, uint8_t* seen, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    level[v] = kLevelInf;
    seen[v] = 0;
  }
}

__global__ void k_lv_clear(LvCnt* c) {
  uint32_t* w = reinterpret_cast<uint32_t*>(c);
  for (uint32_t i = threadIdx.x; i < sizeof(LvCnt) / 4; i += blockDim.x) w[i] = 0;
}

__global__ void k_lv_seed(uint32_t* level, uint8_t* seen, uint32_t* q0, LvCnt* c, const uint32_t* deg,
                          uint32_t src) {
  if (threadIdx.x != 0) return;
  level[src] = 0;
  seen[src] = 1;
  q0[0] = src;
  c->n[0] = 1;
  c->arcs[0] = deg[src];
  c->mode = 0;
  c->reached = 0;
}

// Direction of level L's step, and the counters it fills.
__global__ void k_lv_decide(LvCnt* c, uint32_t L, uint32_t nv, bool allow_bu, bool sweeps) {
  if (threadIdx.x != 0) return;
  const uint32_t s = L & 3, nx = (L + 1) & 3;
  c->n[nx] = 0;
  c->arcs[nx] = 0;
  c->nm[s] = 0;
  const uint64_t nf = c->n[s], mf = c->arcs[s];
  if (L > 0) c->reached += c->n[(L - 1) & 3];
  const uint64_t nu = (uint64_t)nv - c->reached - nf;
  const uint32_t mode = allow_bu && nu > 0 && 2 * nf + mf > 6 * nu + nv / 2 ? kBottomUp
                        : sweeps && mf > nv / kMarkShare                     ? kMark
                                                                             : kClaim;
  c->last = L > 0 ? c->mode : kClaim;
  c->mode = mode;
  if (nf) c->bu_steps += mode == kBottomUp;
}

// Slab chains, sixteen to a group of 16 lanes: lane i holds the head of chain i (kInvalid: none)
// and the value that goes with it.  A round takes K of the group's chains one slab further, a
// word per lane: body(key words, live, values), where live[k] says that this lane's word of slab k
// holds a key.  `short0`: the head held by this lane has a word less (it names the extra heads).
//
// Every step below is bound by its instructions and by the rate at which a CU's address unit takes
// the lanes' lines.  A lane per slab reads 128 bytes as eight loads of 64 lines each and repeats the
// work on a word fifteen times under as many branches (160 registers, three waves on a SIMD); a
// group reads a slab as one line and does the work on its words once, at 54 to 121 registers.
// Distances at scale 22, the multi-bucket rounds of one run: 2.42 ms with a lane per slab, 2.20 with
// a group and eight slabs a round, 2.38 with four, 2.64 with two; marking prefers four (0.35 ms a
// run, 0.37 with eight).
constexpr int kRoundClaim = 4, kRoundRelax = 8;
template <int K, class Body>
__device__ inline void walk_chains(const DView& F, uint32_t head, uint32_t value, bool short0, Body body) {
  const int gl = glane(), g0 = lane64() - gl;
  uint32_t short_heads = (uint32_t)(__ballot(short0) >> g0) & 0xFFFFu;
  while (true) {
    const uint64_t all = __ballot(head != kInvalid);
    if (all == 0) break;
    uint32_t m = (uint32_t)(all >> g0) & 0xFFFFu;
    uint64_t w[K];
    uint32_t val[K], at[K];
    bool live[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      live[k] = m != 0;
      at[k] = m ? (uint32_t)__builtin_ctz(m) : 0u;
      m &= m - 1;
      const uint32_t t = __shfl(head, g0 + (int)at[k]);
      val[k] = __shfl(value, g0 + (int)at[k]);
      w[k] = live[k] ? slab_ptr(F, t)[gl] : kEmptyWord;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t next = __shfl((uint32_t)w[k], g0 + kKeysPerSlab);
      if (live[k] && gl == (int)at[k]) head = next;
      const int nd = kKeysPerSlab - (int)(short_heads >> at[k] & 1u);
      if (live[k]) short_heads &= ~(1u << at[k]);
      live[k] = live[k] && gl < nd && valid_key((uint32_t)w[k]);
    }
    body(w, live, val);
  }
}

// Append the words flagged in `found` (a bit per word) to the staged next frontier.
template <int K>
__device__ inline void push_found(WaveOut& o, uint32_t found, const uint64_t (&w)[K]) {
  bool any;
  uint32_t pos = wave_slots(o, (uint32_t)__popc(found), any);
  if (!any) return;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (found >> k & 1) o.buf[pos++] = (uint32_t)w[k];
}

// Block-wide exclusive prefix of k and one atomic per block on *ctr: this thread's first slot.
__device__ inline uint32_t block_reserve(uint32_t* ctr, uint32_t k, uint32_t* sh) {
  const int lane = lane64();
  const uint32_t w = threadIdx.x / 64;
  uint32_t incl = k;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t below = __shfl_up(incl, o);
    if (lane >= o) incl += below;
  }
  if (lane == 63) sh[w] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (uint32_t i = 0; i < kBlock / 64; ++i) {
      const uint32_t x = sh[i];
      sh[i] = total;
      total += x;
    }
    const uint32_t base = total ? atomicAdd(ctr, total) : 0u;
    for (uint32_t i = 0; i < kBlock / 64; ++i) sh[i] += base;
  }
  __syncthreads();
  const uint32_t first = sh[w] + incl - k;
  __syncthreads();
  return first;
}

// A step's frontier, 16 vertices to a group of lanes (four while there are groups to spare) and up
// to kTileRows a lane: the multi-bucket vertices of a block's tile become work items of 16 buckets,
// reserved by one atomic a tile (one a wave bounded the step: 37,000 on one address for 2.4 M
// vertices), then each(u) is called for the single-bucket ones, by whole waves (u = kInvalid:
// nothing).  `single`: no vertex of the graph has several buckets, so no count is read and no item made,
// and the step needs no second launch (the grid of side 1,024: 1.13 ms a run with both, 0.92 without).
constexpr uint32_t kTileRows = 4;
template <class Each>
__device__ inline void for_each_frontier(const DView& F, const uint32_t* fin, uint32_t n, bool single, uint32_t* nm,
                                         uint32_t* mu, uint32_t* mc, Each each) {
  __shared__ uint32_t sh[kBlock / 64];
  const uint32_t groups = gridDim.x * kGroupsPerBlock;
  const uint32_t per = n <= groups * kRoundClaim ? (uint32_t)kRoundClaim : (uint32_t)kGroup;
  const uint32_t rows = min(kTileRows, (n + groups * per - 1) / (groups * per));
  const uint32_t tile = kGroupsPerBlock * per * rows;
  for (uint32_t base = blockIdx.x * tile; base < n; base += gridDim.x * tile) {
    uint32_t u[kTileRows], nb[kTileRows], k = 0;
#pragma unroll
    for (uint32_t r = 0; r < kTileRows; ++r) {
      const uint32_t i = base + (r * kGroupsPerBlock + threadIdx.x / kGroup) * per + glane();
      u[r] = r < rows && (uint32_t)glane() < per && i < n ? fin[i] : kInvalid;
    }
    if (!single) {
#pragma unroll
      for (uint32_t r = 0; r < kTileRows; ++r) {
        nb[r] = u[r] != kInvalid ? F.nbk[u[r]] : 0u;
        k += nb[r] > 1 ? (nb[r] + kChunk - 1) / kChunk : 0u;
      }
      uint32_t pos = block_reserve(nm, k, sh);
#pragma unroll
      for (uint32_t r = 0; r < kTileRows; ++r) {
        if (nb[r] <= 1) continue;
        for (uint32_t j = 0; j * kChunk < nb[r]; ++j) {
          mu[pos] = u[r];
          mc[pos++] = j;
        }
        u[r] = kInvalid;
      }
    }
    for (uint32_t r = 0; r < rows; ++r) {
      const uint32_t x = r == 0 ? u[0] : r == 1 ? u[1] : r == 2 ? u[2] : u[3];
      each(x != kInvalid && F.deg[x] > 0 ? x : kInvalid);
    }
  }
}
static_assert(kTileRows == 4, "rows are picked by name");

// The work items of a step, one to a group of 16 lanes: each(u, head, short0) by whole waves, head
// being this lane's bucket of the item (kInvalid: none).
template <class Each>
__device__ inline void for_each_item(const DView& F, uint32_t nm, const uint32_t* mu, const uint32_t* mc, Each each) {
  for (uint32_t base = blockIdx.x * kGroupsPerBlock; base < nm; base += gridDim.x * kGroupsPerBlock) {
    const uint32_t it = base + threadIdx.x / kGroup;
    uint32_t u = kInvalid, head = kInvalid, b = 1;
    if (it < nm) {
      u = mu[it];
      b = mc[it] * kChunk + glane();
      const uint64_t* h = slab_ptr(F, u);
      const uint32_t nb = (uint32_t)(h[kKeysPerSlab] >> 32), xb = (uint32_t)h[kKeysPerSlab - 1];
      if (b < nb) head = b == 0 ? u : xb + b - 1;
    }
    each(u, head, b == 0);
  }
}

// Top-down on a round of slabs, claiming: every unreached neighbour gets level cur + 1 (the CAS
// winner pushes it and counts its out-arcs).
template <int K>
__device__ inline uint32_t claim_round(const uint64_t (&w)[K], const bool (&live)[K], uint32_t* level,
                                       const uint32_t* deg, uint32_t cur, unsigned long long& arcs) {
  uint32_t lv[K], dv[K], found = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) lv[k] = ld_u32(level + (live[k] ? (uint32_t)w[k] : 0u));
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint32_t v = (uint32_t)w[k];
    const bool open = live[k] && lv[k] == kLevelInf;
    lv[k] = dv[k] = 0;
    if (open) {
      lv[k] = atomicCAS(level + v, kLevelInf, cur + 1);
      dv[k] = deg[v];
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (lv[k] == kLevelInf) {
      found |= 1u << k;
      arcs += dv[k];
    }
  return found;
}

// Top-down on a round of slabs, marking: every neighbour's byte is set by plain stores, if it does
// not look set, and the sweep over the vertices afterwards finds those without a level.
template <int K>
__device__ inline void mark_round(const uint64_t (&w)[K], const bool (&live)[K], uint8_t* seen) {
  uint8_t sv[K];
#pragma unroll
  for (int k = 0; k < K; ++k) sv[k] = seen[live[k] ? (uint32_t)w[k] : 0u];
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (live[k] && !sv[k]) seen[(uint32_t)w[k]] = 1;
}

__device__ inline void block_add(unsigned long long* acc, unsigned long long v, unsigned long long* out) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(acc, v);
  __syncthreads();
  if (threadIdx.x == 0 && *acc) atomicAdd(out, *acc);
}

// Top-down step, single-bucket frontier vertices: a group of 16 lanes holds up to 16 vertices and
// reads their chains slab by slab (walk_chains).  A vertex with several buckets becomes ceil(nb / 16)
// work items for k_lv_td_multi.
__global__ void __launch_bounds__(kBlock) k_lv_td(DView F, LvCnt* c, uint32_t L, uint32_t* level,
                                                  uint8_t* seen, uint32_t* queue, uint32_t* mu_,
                                                  uint32_t* mc_, bool single) {
  const uint32_t s = L & 3;
  const uint32_t mode = c->mode;
  if (mode == kBottomUp) return;
  const uint32_t n = c->n[s];
  if (n == 0) return;
  const uint32_t* fin = queue + c->reached;
  __shared__ WaveStage S;
  __shared__ unsigned long long acc;
  WaveOut out = wave_out(S, queue + c->reached + n, &c->n[(L + 1) & 3]);
  if (threadIdx.x == 0) acc = 0;
  __syncthreads();
  unsigned long long arcs = 0;
  for_each_frontier(F, fin, n, single, &c->nm[s], mu_, mc_, [&](uint32_t u) {
    walk_chains<kRoundClaim>(F, u, 0u, false, [&](const auto& w, const auto& live, const auto&) {
      if (mode == kMark) mark_round(w, live, seen);
      else push_found(out, claim_round(w, live, level, F.deg, L, arcs), w);
    });
  });
  wave_out_close(out);
  block_add(&acc, arcs, &c->arcs[(L + 1) & 3]);
}

// Top-down step, multi-bucket frontier vertices: a 16-lane group per work item, whose 16 bucket
// chains it reads slab by slab.
__global__ void __launch_bounds__(kBlock) k_lv_td_multi(DView F, LvCnt* c, uint32_t L, uint32_t* level,
                                                        uint8_t* seen, uint32_t* queue, const uint32_t* mu_,
                                                        const uint32_t* mc_) {
  const uint32_t s = L & 3;
  const uint32_t mode = c->mode;
  if (mode == kBottomUp) return;
  const uint32_t nm = c->nm[s];
  if (nm == 0) return;
  __shared__ WaveStage S;
  __shared__ unsigned long long acc;
  WaveOut out = wave_out(S, queue + c->reached + c->n[s], &c->n[(L + 1) & 3]);
  if (threadIdx.x == 0) acc = 0;
  __syncthreads();
  unsigned long long arcs = 0;
  for_each_item(F, nm, mu_, mc_, [&](uint32_t, uint32_t head, bool short0) {
    walk_chains<kRoundClaim>(F, head, 0u, short0, [&](const auto& w, const auto& live, const auto&) {
      if (mode == kMark) mark_round(w, live, seen);
      else push_found(out, claim_round(w, live, level, F.deg, L, arcs), w);
    });
  });
  wave_out_close(out);
  block_add(&acc, arcs, &c->arcs[(L + 1) & 3]);
}

// Does some in-neighbour of v (reverse view) sit on level cur?  A lane walks v's buckets
// and stops at the first slab that holds one.  With `bytes` every vertex on level cur has its byte
// set, and the bytes say which levels to read.
__device__ inline bool has_parent_at(const DView& R, uint32_t v, const uint32_t* level, const uint8_t* seen,
                                     bool bytes, uint32_t cur) {
  Slab sl;
  load_slab(R, v, sl);
  const uint32_t nb = (uint32_t)(sl.w[15] >> 32);
  const uint32_t xb = nb > 1 ? (uint32_t)sl.w[14] : 0u;
  int nd = nb > 1 ? kKeysPerSlab - 1 : kKeysPerSlab;
  for (uint32_t b = 0; b < nb; ++b) {
    if (b > 0) {
      load_slab(R, xb + b - 1, sl);
      nd = kKeysPerSlab;
    }
    while (true) {
      bool hit = false;
      if (bytes) {
        uint8_t sv[kKeysPerSlab];
        load_of_keys<uint8_t>(seen, sl, live_words(sl, nd), (uint8_t)0, sv);
#pragma unroll
        for (int j = 0; j < kKeysPerSlab; ++j)
          if (!hit && sv[j]) hit = ld_u32(level + (uint32_t)sl.w[j]) == cur;
      } else {
        uint32_t lv[kKeysPerSlab];
        load_of_keys<uint32_t>(level, sl, live_words(sl, nd), kLevelInf, lv);
#pragma unroll
        for (int j = 0; j < kKeysPerSlab; ++j) hit |= lv[j] == cur;
      }
      if (hit) return true;
      const uint32_t t = (uint32_t)sl.w[15];
      if (t == kInvalid) break;
      load_slab(R, t, sl);
      nd = kKeysPerSlab;
    }
  }
  return false;
}

// Bottom-up step: every unreached vertex with in-arcs looks for a parent on level L.  Only
// the vertex's own lane writes its level, and no level changes to L during the step.  After a
// marking step the same sweep collects the vertices with a byte and no level.  (A block adds to two
// counters at its end; 8,192 blocks took 123 us for that at scale 22, these 2,048 take 55.)
__global__ void __launch_bounds__(kBlock) k_lv_bu(DView F, DView R, LvCnt* c, uint32_t L, uint32_t* level,
                                                  uint8_t* seen, uint32_t* queue, uint32_t nv) {
  const uint32_t s = L & 3;
  const uint32_t mode = c->mode;
  if (mode == kClaim || c->n[s] == 0) return;
  const bool bytes = c->last != kClaim;  // the frontier came from a sweep
  __shared__ WaveStage S;
  __shared__ unsigned long long acc;
  WaveOut out = wave_out(S, queue + c->reached + c->n[s], &c->n[(L + 1) & 3]);
  if (threadIdx.x == 0) acc = 0;
  __syncthreads();
  unsigned long long arcs = 0;
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t base = blockIdx.x * blockDim.x; base < nv; base += stride) {
    const uint32_t v = base + threadIdx.x;
    bool found = false;
    if (v < nv && ld_u32(level + v) == kLevelInf &&
        (mode == kMark ? seen[v] != 0 : R.deg[v] > 0 && has_parent_at(R, v, level, seen, bytes, L))) {
      level[v] = L + 1;
      seen[v] = 1;
      arcs += F.deg[v];
      found = true;
    }
    bool any;
    const uint32_t pos = wave_slots(out, found ? 1u : 0u, any);
    if (found) out.buf[pos] = v;
  }
  wave_out_close(out);
  block_add(&acc, arcs, &c->arcs[(L + 1) & 3]);
}

inline uint32_t blocks_for(uint64_t n, uint32_t cap) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + kBlock - 1) / kBlock, cap));
}

size_t levels_ws_bytes(const mk_graph* g) {
  return 256 + ((size_t)g->n * 4 + 256) + 2 * (levels_multi_cap(g) * 4 + 256) + ((size_t)g->n + 256) + 256;
}

// ----------------------------------------------------------------- tree nodes from levels
// <level, INVALID> for every reached vertex but the source (<0, source>); unreached ones
// get <INF, INVALID>.
__global__ void k_lv_tree_init(const uint32_t* level, uint64_t* D, uint32_t nv, uint32_t src) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t lv = level[v];
    D[v] = lv == kLevelInf ? kTreeNone : v == src ? (uint64_t)src : ((uint64_t)lv << 32) | kInvalid;
  }
}

// Reached vertices (other than the source) with more than kHeavyBuckets buckets in the
// reverse view, and their work items of kPrItem buckets.
constexpr uint32_t kPrItem = 4;
__global__ void k_lv_heavy(const uint32_t* nbk, const uint32_t* level, uint32_t nv, uint32_t src,
                           uint32_t* out, uint32_t* cnt) {
  __shared__ Stage S[1];
  stage_open(S[0], out, cnt);
  __syncthreads();
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t base = blockIdx.x * blockDim.x; base < nv; base += stride) {
    const uint32_t v = base + threadIdx.x;
    stage_push(S[0], v < nv && v != src && nbk[v] > kHeavyBuckets && level[v] != kLevelInf, v);
  }
  stage_close(S);
}

__global__ void k_lv_items(const uint32_t* nbk, const uint32_t* heavy, const uint32_t* nheavy, uint32_t* cnt) {
  const uint32_t nh = *nheavy;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < nh; j += gridDim.x * blockDim.x)
    cnt[j] = (nbk[heavy[j]] + kPrItem - 1) / kPrItem;
}

// Is u (distance du, arc weight w) a parent of a vertex at distance dv: du + w == dv, with
// the sum saturated below INF as the tree traversal does; BFS counts every arc as 1.
template <bool kUnit>
__device__ inline bool parent_arc(uint32_t du, uint64_t word, uint32_t dv) {
  if (du == kLevelInf) return false;
  const uint64_t w = kUnit ? 1ull : (word >> 32);
  return (uint32_t)min<uint64_t>((uint64_t)du + w, 0xFFFFFFFEull) == dv;
}

// Parent of every reached vertex: the smallest in-neighbour u with dist(u) + w(u, v) =
// dist(v) (the parent rule of the tree variant).  One lane per single-bucket vertex, a
// 16-lane group per vertex of 2 .. kHeavyBuckets buckets, and the heavy vertices' bucket
// items spread over every group, which fold their minima in with a 64-bit atomic minimum.
template <bool kUnit>
__global__ void __launch_bounds__(kBlock) k_lv_parents(DView R, const uint32_t* level, uint64_t* D, uint32_t nv,
                                                       uint32_t src, const uint32_t* heavy,
                                                       const uint32_t* nheavy, const uint32_t* hoff,
                                                       const uint32_t* hcnt) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    if (R.nbk[v] != 1 || v == src) continue;
    const uint32_t lv = level[v];
    if (lv == kLevelInf) continue;
    uint32_t best = kInvalid, t = v;
    Slab sl;
    while (true) {
      load_slab(R, t, sl);
      uint32_t lu[kKeysPerSlab];
      load_of_keys<uint32_t>(level, sl, live_words(sl, kKeysPerSlab), kLevelInf, lu);
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j)
        if (parent_arc<kUnit>(lu[j], sl.w[j], lv)) best = min(best, (uint32_t)sl.w[j]);
      t = (uint32_t)sl.w[15];
      if (t == kInvalid) break;
    }
    D[v] = ((uint64_t)lv << 32) | best;
  }
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  for (uint32_t v = g0; v < nv; v += ng) {
    const uint32_t nb = R.nbk[v];
    if (nb == 1 || nb > kHeavyBuckets || v == src) continue;
    const uint32_t lv = level[v];
    if (lv == kLevelInf) continue;
    uint64_t best = kTreeNone;
    for_each_slab(R, v, [&](uint64_t w, bool data) {
      const uint32_t u = (uint32_t)w;
      if (data && valid_key(u) && parent_arc<kUnit>(level[u], w, lv)) best = min(best, (uint64_t)u);
    });
    best = gmin_u64(best);
    if (glane() == 0) D[v] = ((uint64_t)lv << 32) | (uint32_t)best;
  }
  const uint32_t nh = *nheavy;
  if (nh == 0) return;
  const uint32_t items = hoff[nh - 1] + hcnt[nh - 1];
  for (uint32_t it = g0; it < items; it += ng) {
    uint32_t lo = 0, hi = nh;  // the last j with hoff[j] <= it
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (hoff[mid] <= it) lo = mid;
      else hi = mid;
    }
    const uint32_t v = heavy[lo];
    const uint32_t lv = level[v];
    const uint32_t b0 = (it - hoff[lo]) * kPrItem;
    uint64_t best = kTreeNone;
    for_each_bucket_range(R, v, b0, b0 + kPrItem, [&](uint64_t w, bool data) {
      const uint32_t u = (uint32_t)w;
      if (data && valid_key(u) && parent_arc<kUnit>(level[u], w, lv)) best = min(best, (uint64_t)u);
    });
    best = gmin_u64(best);
    if (glane() == 0 && best != kTreeNone) amin64(D + v, ((uint64_t)lv << 32) | best);
  }
}


// ----------------------------------------------------------------- distance-only SSSP
// The vanilla SSSP: one u32 distance per vertex relaxed by 32-bit atomic minimum, no
// parents.  Scheduling is near-far: a relaxed vertex whose new distance is below the band
// limit T joins the next near frontier, any other the far pile; when the near frontier runs
// dry, the far pile is split at T = (its smallest distance) + delta.  Every decision is made
// on the device, so the host only reads sizes back every few steps.  Any schedule reaches the
// same distances (label correcting), so the band width only changes the work.
struct DsCnt {
  uint32_t n[4];     // near frontier sizes by step mod 4
  uint32_t nm[4];    // multi-bucket work items by step mod 4
  uint32_t nfar[2];  // far pile sizes
  uint32_t fpar;     // index of the current far pile
  uint32_t T;        // band limit
  uint32_t band;     // band number (far-pile duplicate stamps)
  uint32_t fmin;     // smallest distance on the far pile (before a split)
  uint32_t done;     // blocks of the running split that have finished
  uint32_t dry;      // the last step left the near frontier empty: the far pile is to be split
  uint32_t pad[4];
};
static_assert(sizeof(DsCnt) <= 256, "counter block");

// A vertex's word holds its distance above the stamp of its last push, so that one 64-bit atomic
// minimum lowers the distance and says whether the vertex is queued already: near pushes are
// stamped kNear | step + 1, far ones with the band.  A distance below the band limit is on no far
// pile that the band will push to again, so one stamp serves both.  A minimum that only ties
// leaves the word alone: within a band a distance is always near or always far, and the stamps of
// each kind grow (a split stamps what it keeps).
//
// What a relaxation reads first is one byte per vertex, a distance that the vertex had, rounded up
// to kDsMant + 1 significant bits: an arc that does not beat it is dropped.  Four bytes a vertex
// brought 103 M lines into the L2s in a run at scale 22, the bytes bring half of that, and what
// they let through by rounding costs fewer atomics (10.8 M for all) than the second one that a stamp
// array takes (15.5 M).  The bytes are written without order among the lanes; any of them is a
// distance the vertex had, so none is too low.
//
// One run at scale 22: 4.0 ms with u32 distances, a stamp array for each queue and a lane per slab;
// 2.9 now.  What is left is slab reads: a round over most of the graph takes 0.9 ms for 20 M lines.
constexpr uint32_t kNear = 1u << 31;
constexpr int kDsMant = 3;
using DsByte = uint8_t;
constexpr DsByte kDsFar = 255;  // no distance yet: above every code

// d to its kDsMant + 1 leading bits, rounded down, as a code in the order of the values.
__device__ inline uint32_t ds_code(uint32_t d, uint32_t& exact) {
  const int e = max(0, 31 - __clz((int)(d | 1u)) - kDsMant);
  exact = (d & ((1u << e) - 1)) == 0;
  return ((uint32_t)e << kDsMant) + (d >> e);
}

__global__ void k_ds_fill(unsigned long long* word, DsByte* bound, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    word[v] = (unsigned long long)kLevelInf << 32;
    bound[v] = kDsFar;
  }
}

__global__ void k_ds_seed(unsigned long long* word, DsByte* bound, uint32_t* q0, DsCnt* c, uint32_t src,
                          uint32_t delta) {
  if (threadIdx.x != 0) return;
  word[src] = 0;
  bound[src] = 0;
  q0[0] = src;
  c->n[0] = 1;
  c->T = delta;
  c->band = 1;
  c->fmin = kLevelInf;
}

__global__ void k_ds_store(const unsigned long long* word, uint32_t* dist, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x)
    dist[v] = (uint32_t)(word[v] >> 32);
}

struct DsArgs {
  unsigned long long* word;
  DsByte* bound;
  uint32_t *far[2], *multi_v, *multi_c;
};

__device__ inline uint32_t ds_dist(const DsArgs& a, uint32_t v) {
  return ld_u32(reinterpret_cast<const uint32_t*>(a.word + v) + 1);
}

// Relax a round of slabs (val: the distances they are reached from): a neighbour whose distance
// drops goes to the near frontier (once per step, by the step stamp) or to the far pile (once per
// band).
template <int K>
__device__ inline void relax_round(const uint64_t (&w)[K], const bool (&live)[K],
                                   const uint32_t (&val)[K], const DsArgs& a, uint32_t step, uint32_t band,
                                   uint32_t T, uint32_t& near, uint32_t& far) {
  DsByte bv[K];
  unsigned long long old[K];
  uint32_t d[K], tried = 0, exact;
#pragma unroll
  for (int k = 0; k < K; ++k) bv[k] = a.bound[live[k] ? (uint32_t)w[k] : 0u];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    d[k] = (uint32_t)min<uint64_t>((uint64_t)val[k] + (w[k] >> 32), 0xFFFFFFFEull);
    old[k] = 0;
    if (live[k] && ds_code(d[k], exact) < bv[k]) {
      tried |= 1u << k;
      old[k] = atomicMin(a.word + (uint32_t)w[k], (unsigned long long)d[k] << 32 | (d[k] < T ? step : band));
    }
  }
  near = far = 0;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if ((tried >> k & 1) && d[k] < (uint32_t)(old[k] >> 32)) {
      const uint32_t code = ds_code(d[k], exact);
      a.bound[(uint32_t)w[k]] = (DsByte)(code + (exact ? 0u : 1u));
      if (d[k] < T) near |= (uint32_t)((uint32_t)old[k] != step) << k;
      else far |= (uint32_t)((uint32_t)old[k] != band) << k;
    }
}

__device__ inline void wave_min_to(uint32_t* out, uint32_t m) {
  for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0 && m != kLevelInf) atomicMin(out, m);
}

// Near step, single-bucket frontier vertices (up to 16 to a group of 16 lanes, which reads their
// chains slab by slab); others become 16-bucket items.
__global__ void __launch_bounds__(kBlock) k_ds_relax(DView F, DsCnt* c, uint32_t S, DsArgs a, const uint32_t* fin,
                                                     uint32_t* fout, bool single) {
  const uint32_t s = S & 3;
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // counters of the next step (unused in this one)
    c->n[(S + 2) & 3] = 0;
    c->nm[(S + 1) & 3] = 0;
  }
  const uint32_t n = c->n[s];
  if (n == 0) return;
  const uint32_t T = c->T, band = c->band, fp = c->fpar, step = kNear | (S + 1);
  __shared__ WaveStage St[2];
  WaveOut near = wave_out(St[0], fout, &c->n[(S + 1) & 3]);
  WaveOut far = wave_out(St[1], a.far[fp], &c->nfar[fp]);
  for_each_frontier(F, fin, n, single, &c->nm[s], a.multi_v, a.multi_c, [&](uint32_t u) {
    const uint32_t du = u != kInvalid ? ds_dist(a, u) : 0u;
    walk_chains<kRoundRelax>(F, u, du, false, [&](const auto& w, const auto& live, const auto& val) {
      uint32_t nr, fr;
      relax_round(w, live, val, a, step, band, T, nr, fr);
      push_found(near, nr, w);
      push_found(far, fr, w);
    });
  });
  wave_out_close(near);
  wave_out_close(far);
}

// Near step, multi-bucket frontier vertices: a 16-lane group per item, whose 16 bucket chains it
// reads slab by slab.
__global__ void __launch_bounds__(kBlock) k_ds_relax_multi(DView F, DsCnt* c, uint32_t S, DsArgs a,
                                                           uint32_t* fout) {
  const uint32_t s = S & 3;
  const uint32_t nm = c->nm[s];
  if (nm == 0) return;
  const uint32_t T = c->T, band = c->band, fp = c->fpar, step = kNear | (S + 1);
  __shared__ WaveStage St[2];
  WaveOut near = wave_out(St[0], fout, &c->n[(S + 1) & 3]);
  WaveOut far = wave_out(St[1], a.far[fp], &c->nfar[fp]);
  for_each_item(F, nm, a.multi_v, a.multi_c, [&](uint32_t u, uint32_t head, bool short0) {
    const uint32_t du = u != kInvalid ? ds_dist(a, u) : 0u;
    walk_chains<kRoundRelax>(F, head, du, short0, [&](const auto& w, const auto& live, const auto& val) {
      uint32_t nr, fr;
      relax_round(w, live, val, a, step, band, T, nr, fr);
      push_found(near, nr, w);
      push_found(far, fr, w);
    });
  });
  wave_out_close(near);
  wave_out_close(far);
}

// When a step leaves the near frontier empty: the smallest distance on the far pile at or past the
// band limit (a vertex below it has joined the near frontier since) ...  It also settles for the
// split whether the frontier is empty: the blocks of the split fill that frontier, so one that
// starts late would see it filled and leave out its share of the pile.
__global__ void k_ds_far_min(DsCnt* c, uint32_t S, DsArgs a) {
  const bool dry = c->n[(S + 1) & 3] == 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) c->dry = dry;
  if (!dry) return;
  const uint32_t fp = c->fpar, nf = c->nfar[fp], T = c->T;
  uint32_t m = kLevelInf;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nf; i += gridDim.x * blockDim.x) {
    const uint32_t d = ds_dist(a, a.far[fp][i]);
    if (d >= T) m = min(m, d);
  }
  wave_min_to(&c->fmin, m);
}

// ... and the split at T' = fmin + delta: those below T' start the next near frontier,
// the others move to the other pile, stamped with the next band.  The last block to finish
// commits the new band limit, band number and pile (no block waits for another).
__global__ void k_ds_split(DsCnt* c, uint32_t S, DsArgs a, uint32_t* fout, uint32_t delta) {
  if (!c->dry) return;
  const uint32_t fp = c->fpar, nf = c->nfar[fp];
  if (nf == 0) return;
  const uint32_t T2 = (uint32_t)min<uint64_t>((uint64_t)c->fmin + delta, 0xFFFFFFFFull);
  const uint32_t T = c->T, nb = c->band + 1;
  __shared__ Stage St[2];
  __shared__ bool last;
  stage_open(St[0], fout, &c->n[(S + 1) & 3]);
  stage_open(St[1], a.far[fp ^ 1], &c->nfar[fp ^ 1]);
  __syncthreads();
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t base = blockIdx.x * blockDim.x; base < nf; base += stride) {
    const uint32_t i = base + threadIdx.x;
    bool to_near = false, keep = false;
    uint32_t v = 0;
    if (i < nf) {
      v = a.far[fp][i];
      const uint32_t d = ds_dist(a, v);
      to_near = d >= T && d < T2;
      keep = d >= T2;
      if (keep) *reinterpret_cast<uint32_t*>(a.word + v) = nb;
    }
    stage_push(St[0], to_near, v);
    stage_push(St[1], keep, v);
  }
  stage_close(St);
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    last = atomicAdd(&c->done, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (last && threadIdx.x == 0) {
    __threadfence();
    c->T = T2;
    c->band = nb;
    c->nfar[fp] = 0;
    c->fpar = fp ^ 1;
    c->fmin = kLevelInf;
    c->done = 0;
  }
}

size_t dist_ws_bytes(const mk_graph* g) {
  return 256 + ((size_t)g->n * 8 + 256) + 4 * ((size_t)g->n * 4 + 256) + 2 * (levels_multi_cap(g) * 4 + 256) + 256;
}

}  // namespace

namespace mk {

size_t levels_multi_cap(const mk_graph* g) { return (size_t)g->n + g->view[VF].n_head / kChunk + 64; }

mk_status levels_run(mk_graph* g, uint32_t source, bool allow_bu, const LevelBufs& b, uint32_t* level,
                     uint64_t* pin, uint32_t* h_bottom_up_steps, hipStream_t stream) {
  const uint32_t N = g->n;
  LvCnt* c = reinterpret_cast<LvCnt*>(b.cnt);
  const DView F = g->view[VF].d;
  const DView R = g->view[VR].on ? g->view[VR].d : F;
  allow_bu = allow_bu && g->view[VR].on;
  const bool single = g->view[VF].n_head == N;
  const bool sweeps = allow_bu || g->m0 >= (uint64_t)(N >= kSweepLeast ? 8 : kSweepDense) * N;
  hipLaunchKernelGGL(k_lv_clear, dim3(1), dim3(64), 0, stream, c);
  hipLaunchKernelGGL(k_lv_fill, dim3(blocks_for(N, 4096)), dim3(kBlock), 0, stream, level, b.seen, N);
  hipLaunchKernelGGL(k_lv_seed, dim3(1), dim3(64), 0, stream, level, b.seen, b.q, c, F.deg, source);
  MK_LAUNCH(g, "k_lv_seed");
  uint64_t every = kSyncFirst, next_sync = kSyncFirst;
  for (uint32_t L = 0;; ++L) {
    hipLaunchKernelGGL(k_lv_decide, dim3(1), dim3(64), 0, stream, c, L, N, allow_bu, sweeps);
    hipLaunchKernelGGL(k_lv_td, dim3(blocks_for(N, 2048)), dim3(kBlock), 0, stream, F, c, L, level, b.seen,
                       b.q, b.multi_v, b.multi_c, single);
    if (!single)
      hipLaunchKernelGGL(k_lv_td_multi, dim3(2048), dim3(kBlock), 0, stream, F, c, L, level, b.seen, b.q,
                         b.multi_v, b.multi_c);
    if (sweeps)
      hipLaunchKernelGGL(k_lv_bu, dim3(blocks_for(N, 2048)), dim3(kBlock), 0, stream, F, R, c, L, level,
                         b.seen, b.q, N);
    MK_LAUNCH(g, "k_lv step");
    if (L + 1 == next_sync || L + 1 >= N) {
      if (next_sync >= 2 * kSyncFirst) every = std::min<uint64_t>(2 * every, kSyncMax);
      next_sync += every;
      read_back(c, pin, sizeof(LvCnt) / 4, stream);
      MK_HIP(g, hipStreamSynchronize(stream));
      if (reinterpret_cast<const volatile LvCnt*>(pin)->n[(L + 1) & 3] == 0 || L + 1 >= N) break;
    }
  }
  if (h_bottom_up_steps) *h_bottom_up_steps = reinterpret_cast<const volatile LvCnt*>(pin)->bu_steps;
  return MK_OK;
}

// Tree nodes <dist, smallest parent> from finished distances (BFS levels when kUnit).
template <bool kUnit>
mk_status tree_from_dist(mk_graph* g, uint32_t source, const uint32_t* dist, uint64_t* D, hipStream_t stream) {
  const uint32_t N = g->n;
  const DView R = g->view[VR].d;
  uint32_t* heavy = g->fq[2];
  uint32_t* hcnt = g->fq[3];
  uint32_t* hoff = g->fq[4];
  uint32_t* nh = reinterpret_cast<LvCnt*>(g->lv_cnt)->pad;
  hipLaunchKernelGGL(k_lv_clear, dim3(1), dim3(64), 0, stream, reinterpret_cast<LvCnt*>(g->lv_cnt));
  hipLaunchKernelGGL(k_lv_tree_init, dim3(blocks_for(N, 4096)), dim3(kBlock), 0, stream, dist, D, N, source);
  hipLaunchKernelGGL(k_lv_heavy, dim3(blocks_for(N, 4096)), dim3(kBlock), 0, stream, R.nbk, dist, N, source,
                     heavy, nh);
  hipLaunchKernelGGL(k_lv_items, dim3(blocks_for(N, 1024)), dim3(kBlock), 0, stream, R.nbk, heavy, nh, hcnt);
  size_t tb = g->scan_tmp_bytes;
  if (rocprim::exclusive_scan(g->scan_tmp, tb, hcnt, hoff, 0u, (size_t)N, rocprim::plus<uint32_t>(), stream) !=
      hipSuccess)
    return MK_ERR_HIP;
  hipLaunchKernelGGL(k_lv_parents<kUnit>, dim3(4096), dim3(kBlock), 0, stream, R, dist, D, N, source, heavy, nh,
                     hoff, hcnt);
  MK_LAUNCH(g, "k_lv_parents");
  return MK_OK;
}

mk_status bfs_tree_by_levels(mk_graph* g, uint32_t source, uint32_t* level, uint64_t* D, hipStream_t stream) {
  LevelBufs b;
  b.cnt = g->lv_cnt;
  b.q = g->fq[0];
  b.multi_v = g->lv_multi[0];
  b.multi_c = g->lv_multi[1];
  b.seen = reinterpret_cast<uint8_t*>(g->fq[1]);
  mk_status s = levels_run(g, source, true, b, level, g->h_pin, nullptr, stream);
  if (s != MK_OK) return s;
  return tree_from_dist<true>(g, source, level, D, stream);
}

// Every step either relaxes a non-empty near frontier or splits a non-empty far pile, and
// positive weights bound the number of distance drops, so the loop ends; the cap is a guard
// (and keeps the step stamps unique).
//
// The bounds (a byte per vertex) lie in `dist`, which takes the distances when they are final.
mk_status dist_run(mk_graph* g, uint32_t source, void* cnt, uint32_t* const q[2], DsArgs a,
                   uint32_t* dist, uint64_t* pin, hipStream_t stream) {
  a.bound = reinterpret_cast<DsByte*>(dist);
  const uint32_t N = g->n;
  DsCnt* c = reinterpret_cast<DsCnt*>(cnt);
  const DView F = g->view[VF].d;
  const uint32_t delta = std::max<uint32_t>(1u, g->sssp_delta);
  const bool single = g->view[VF].n_head == N;
  hipLaunchKernelGGL(k_lv_clear, dim3(1), dim3(64), 0, stream, reinterpret_cast<LvCnt*>(c));
  hipLaunchKernelGGL(k_ds_fill, dim3(blocks_for(N, 4096)), dim3(kBlock), 0, stream, a.word, a.bound, N);
  hipLaunchKernelGGL(k_ds_seed, dim3(1), dim3(64), 0, stream, a.word, a.bound, q[0], c, source, delta);
  MK_LAUNCH(g, "k_ds_seed");
  const uint64_t cap = std::min<uint64_t>(64ull * N + 1024, 1ull << 31);
  uint64_t every = kSyncFirst, next_sync = kSyncFirst;
  for (uint64_t S = 0;; ++S) {
    const uint32_t s32 = (uint32_t)S;
    uint32_t* fin = q[S & 1];
    uint32_t* fout = q[(S + 1) & 1];
    hipLaunchKernelGGL(k_ds_relax, dim3(blocks_for(N, 2048)), dim3(kBlock), 0, stream, F, c, s32, a, fin, fout,
                       single);
    if (!single)
      hipLaunchKernelGGL(k_ds_relax_multi, dim3(2048), dim3(kBlock), 0, stream, F, c, s32, a, fout);
    hipLaunchKernelGGL(k_ds_far_min, dim3(blocks_for(N, 1024)), dim3(kBlock), 0, stream, c, s32, a);
    hipLaunchKernelGGL(k_ds_split, dim3(blocks_for(N, 2048)), dim3(kBlock), 0, stream, c, s32, a, fout, delta);
    MK_LAUNCH(g, "k_ds step");
    if (S + 1 == next_sync) {
      if (next_sync >= 2 * kSyncFirst) every = std::min<uint64_t>(2 * every, kSyncMax);
      next_sync += every;
      read_back(c, pin, sizeof(DsCnt) / 4, stream);
      MK_HIP(g, hipStreamSynchronize(stream));
      const volatile DsCnt* h = reinterpret_cast<const volatile DsCnt*>(pin);
      if (h->n[(S + 1) & 3] == 0 && h->nfar[0] == 0 && h->nfar[1] == 0) break;
      if (S > cap) return MK_ERR_HIP;
    }
  }
  hipLaunchKernelGGL(k_ds_store, dim3(blocks_for(N, 4096)), dim3(kBlock), 0, stream, a.word, dist, N);
  MK_LAUNCH(g, "k_ds_store");
  return MK_OK;
}

mk_status sssp_tree_by_distances(mk_graph* g, uint32_t source, uint32_t* dist, uint64_t* D, hipStream_t stream) {
  uint32_t* q[2] = {g->fq[0], g->fq[1]};
  DsArgs a;
  a.word = reinterpret_cast<unsigned long long*>(D);  // the nodes are written afterwards
  a.far[0] = g->far[0];
  a.far[1] = g->far[1];
  a.multi_v = g->lv_multi[0];
  a.multi_c = g->lv_multi[1];
  mk_status s = dist_run(g, source, g->lv_cnt, q, a, dist, g->h_pin, stream);
  if (s != MK_OK) return s;
  return tree_from_dist<false>(g, source, dist, D, stream);
}

}  // namespace mk

extern "C" {

mk_status mk_bfs_levels(mk_graph* g, uint32_t source, uint32_t flags, void* d_ws, size_t ws_bytes,
                        uint32_t slot, uint32_t* d_level, uint32_t* h_bottom_up_steps, hipStream_t stream) {
  if (!g || !d_ws || !d_level || source >= g->n || slot >= kSlots || (flags & ~MK_BFS_TOP_DOWN_ONLY))
    return MK_ERR_INVALID_ARG;
  if (ws_bytes < levels_ws_bytes(g)) return MK_ERR_CAPACITY;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  if (!g->slot_pin[slot]) {
    if (hipHostMalloc((void**)&g->slot_pin[slot], 64 * sizeof(uint64_t), hipHostMallocDefault) != hipSuccess)
      return MK_ERR_HIP;
  }
  const uint32_t N = g->n;
  char* p = reinterpret_cast<char*>(((uintptr_t)d_ws + 255) & ~uintptr_t(255));
  auto take = [&](size_t bytes) {
    char* r = p;
    p += (bytes + 255) & ~size_t(255);
    return r;
  };
  LevelBufs b;
  b.cnt = take(256);
  b.q = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  b.multi_v = reinterpret_cast<uint32_t*>(take(levels_multi_cap(g) * 4));
  b.multi_c = reinterpret_cast<uint32_t*>(take(levels_multi_cap(g) * 4));
  b.seen = reinterpret_cast<uint8_t*>(take((size_t)N));
  return levels_run(g, source, !(flags & MK_BFS_TOP_DOWN_ONLY), b, d_level, g->slot_pin[slot],
                    h_bottom_up_steps, stream);
}

size_t mk_bfs_levels_workspace_bytes(const mk_graph* g) { return g ? levels_ws_bytes(g) : 0; }

mk_status mk_sssp_distances(mk_graph* g, uint32_t source, void* d_ws, size_t ws_bytes, uint32_t slot,
                            uint32_t* d_dist, hipStream_t stream) {
  if (!g || !d_ws || !d_dist || source >= g->n || slot >= kSlots) return MK_ERR_INVALID_ARG;
  if (ws_bytes < dist_ws_bytes(g)) return MK_ERR_CAPACITY;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  if (!g->slot_pin[slot]) {
    if (hipHostMalloc((void**)&g->slot_pin[slot], 64 * sizeof(uint64_t), hipHostMallocDefault) != hipSuccess)
      return MK_ERR_HIP;
  }
  const uint32_t N = g->n;
  char* p = reinterpret_cast<char*>(((uintptr_t)d_ws + 255) & ~uintptr_t(255));
  auto take = [&](size_t bytes) {
    char* r = p;
    p += (bytes + 255) & ~size_t(255);
    return r;
  };
  DsCnt* c = reinterpret_cast<DsCnt*>(take(256));
  uint32_t* q[2];
  q[0] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  q[1] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  DsArgs a;
  a.word = reinterpret_cast<unsigned long long*>(take((size_t)N * 8));
  a.far[0] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  a.far[1] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  a.multi_v = reinterpret_cast<uint32_t*>(take(levels_multi_cap(g) * 4));
  a.multi_c = reinterpret_cast<uint32_t*>(take(levels_multi_cap(g) * 4));
  return dist_run(g, source, c, q, a, d_dist, g->slot_pin[slot], stream);
}

size_t mk_sssp_distances_workspace_bytes(const mk_graph* g) { return g ? dist_ws_bytes(g) : 0; }

}  // extern "C"
