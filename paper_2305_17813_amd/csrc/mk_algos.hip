// Weakly connected components (section 4.4), PageRank (section 4.1) and triangle
// counting (section 4.3) over the slab views.
//
// All-vertex walks follow the paper's IterationScheme1 (one vertex per lane group); the
// few vertices with more than kHeavyBuckets buckets are walked by a whole block so that a
// power-law hub does not serialize one group.
#include <cstring>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mk_internal.h"

using namespace mk;

namespace {

constexpr uint32_t kWalkBlocks = 4096;
constexpr uint32_t kPrContribBlocks = 2048, kPrFinalBlocks = 512;
static_assert(kPrContribBlocks + kWalkBlocks + kPrFinalBlocks <= kPrParts, "PageRank partial sums");
constexpr uint32_t kPrChunk = 4;  // buckets per heavy-vertex work item
constexpr uint32_t kPrBatch = 8;  // head slabs a group loads at once in the PageRank kernels
constexpr int kPrSyncEvery = 4;

inline uint32_t blocks_for(uint64_t n, uint32_t cap = 4096) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + kBlock - 1) / kBlock, cap));
}

// Vertices of a view with more than kHeavyBuckets buckets (staged per block: they are
// sparse, and one counter atomic per wave that finds one would serialize).
__global__ void k_collect_heavy(const uint32_t* nbk, uint32_t nv, uint32_t* out, uint32_t* cnt) {
  __shared__ Stage S[1];
  stage_open(S[0], out, cnt);
  __syncthreads();
  const uint64_t lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; base < nv;
       base += stride) {
    const uint64_t v = base + lane;
    const bool heavy = v < nv && nbk[v] > kHeavyBuckets;
    stage_push(S[0], heavy, (uint32_t)v);
  }
  stage_close(S);
}

__global__ void k_zero_u32(uint32_t* p, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// ================================================================= union-find (WCC)
// Hooking rule: the larger root is hooked under the smaller one by CAS, so every parent
// pointer goes to a smaller id and the final root of a component is its minimum id.
__device__ inline uint32_t uf_find(uint32_t* P, uint32_t x) {
  while (true) {
    const uint32_t p = ld_u32(P + x);
    if (p == x) return x;
    const uint32_t gp = ld_u32(P + p);
    if (gp != p) __hip_atomic_store(P + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // halving
    x = gp;
  }
}

__device__ inline void uf_union(uint32_t* P, uint32_t a, uint32_t b) {
  while (true) {
    a = uf_find(P, a);
    b = uf_find(P, b);
    if (a == b) return;
    if (a < b) {
      const uint32_t t = a;
      a = b;
      b = t;
    }
    const uint32_t r = atomicCAS(P + a, a, b);  // hook the larger root under the smaller
    if (r == a) return;
    a = r;  // a was hooked meanwhile: continue from its true parent (a smaller id)
  }
}

// The same with another order: the hooked root is the one of larger uf_order.  Every parent pointer
// among roots then goes to a smaller order, whatever the ids, and chains stay short where
// neighbouring ids would make long ones (a row of a grid).  The root of a component is no
// longer its smallest id; k_wcc_min and k_wcc_label find that.
// uf_order is a bijection of the ids: the 32-bit finalizer of MurmurHash3 (Appleby).
__device__ inline uint32_t uf_order(uint32_t x) {
  x = (x ^ x >> 16) * 0x85EBCA6Bu;
  x = (x ^ x >> 13) * 0xC2B2AE35u;
  return x ^ x >> 16;
}
__device__ inline void uf_union_any(uint32_t* P, uint32_t a, uint32_t b) {
  while (true) {
    a = uf_find(P, a);
    b = uf_find(P, b);
    if (a == b) return;
    if (uf_order(a) < uf_order(b)) {
      const uint32_t t = a;
      a = b;
      b = t;
    }
    const uint32_t r = atomicCAS(P + a, a, b);
    if (r == a) return;
    a = r;  // a was hooked meanwhile: continue from its true parent
  }
}

__global__ void k_wcc_init(uint32_t* P, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) P[v] = v;
}

// Static WCC: union over every arc.  A neighbour whose parent already is u's root (as
// found once per vertex; a stale root only means an older member of the same component)
// is skipped without a union, and a lane issues the parent loads of a whole slab together.
__global__ void __launch_bounds__(kBlock) k_wcc_all(DView F, uint32_t* P, uint32_t nv,
                                                    const uint32_t* heavy, const uint32_t* nheavy, bool single) {
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  auto body = [&](uint32_t u, uint32_t ru, uint64_t x, bool data) {
    const uint32_t v = (uint32_t)x;
    if (data && valid_key(v) && ld_u32(P + v) != ru) uf_union(P, u, v);
  };
  // single-bucket vertices: one lane each
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < nv; u += gridDim.x * blockDim.x) {
    if (F.nbk[u] != 1 || F.deg[u] == 0) continue;
    const uint32_t ru = uf_find(P, u);
    Slab sl;
    uint32_t t = u;
    while (true) {
      load_slab(F, t, sl);
      uint32_t pv[kKeysPerSlab];
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j) {
        const uint32_t v = (uint32_t)sl.w[j];
        pv[j] = valid_key(v) ? ld_u32(P + v) : ru;
      }
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j)
        if (pv[j] != ru) uf_union(P, u, (uint32_t)sl.w[j]);
      t = (uint32_t)sl.w[15];
      if (t == kInvalid) break;
    }
  }
  if (single) return;  // no vertex has several buckets
  for (uint32_t u = g0; u < nv; u += ng) {
    const uint32_t nb = F.nbk[u];
    if (nb == 1 || nb > kHeavyBuckets || F.deg[u] == 0) continue;
    const uint32_t ru = uf_find(P, u);
    for_each_slab(F, u, [&](uint64_t x, bool data) { body(u, ru, x, data); });
  }
  const uint32_t nh = *nheavy, gib = threadIdx.x / kGroup;
  for (uint32_t j = blockIdx.x; j < nh; j += gridDim.x) {
    const uint32_t u = heavy[j];
    const uint32_t ru = uf_find(P, u);
    for_each_slab_strided(F, u, gib, kGroupsPerBlock, [&](uint64_t x, bool data) { body(u, ru, x, data); });
  }
}

// Before the all-arc walk of a static WCC: every vertex points at the smallest id among itself and
// the first four words of its primary slab, without atomics, and k_wcc_jump shortens the chains
// (four pointers per pass).  The walk then finds nearly every neighbour under the same root and
// unites the few trees that are left, where it used to unite every arc of a forest of single
// vertices: 3.25 ms on the 4096 x 4096 grid, 2.2 ms with it.  It pays where no vertex has several
// buckets, and on graphs of kHookLeast to kHookMost vertices, whose unions otherwise meet on few words
// (without / with it, us: R-MAT scale 16, edge factors 4 and 16: 256, 356 / 177, 256; scale 18: 640,
// 1,140 / 540, 650; scale 19: 1,070, 1,960 / 910, 1,380).  Smaller graphs only have more launches (scale
// 12: 78, 103 / 103, 134), on larger ones the passes cost more than they save (scale 20: 1,040, 1,220 /
// 1,330, 1,310; scale 22: 1,290, 2,220 / 1,250, 2,990; a million vertices, uniform, degree 8: 1,020 /
// 1,570).
constexpr uint32_t kHookLeast = 1u << 15, kHookMost = 1u << 19;
// vertices from which a recompute's walk has a lane for each again: no vertex of several buckets, and others
constexpr uint32_t kRootMost = 1u << 23, kRootMostMixed = 1u << 21;
constexpr uint32_t kWccHook = 4;
__device__ inline void first_words(const DView& V, uint32_t u, uint32_t (&v)[kWccHook]) {
  const uint4* q = reinterpret_cast<const uint4*>(slab_ptr(V, u));
  const uint4 a = q[0], b = q[1];
  v[0] = a.x;
  v[1] = a.z;
  v[2] = b.x;
  v[3] = b.z;
}

__global__ void __launch_bounds__(kBlock) k_wcc_hook_min(DView V, uint32_t* P, uint32_t nv) {
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < nv; u += gridDim.x * blockDim.x) {
    uint32_t best = u;
    if (V.deg[u]) {
      uint32_t v[kWccHook];
      first_words(V, u, v);
#pragma unroll
      for (uint32_t k = 0; k < kWccHook; ++k) best = min(best, v[k]);  // EMPTY and TOMBSTONE are larger
    }
    P[u] = best;
  }
}

constexpr int kWccJumps = 3;  // 2: 2.4 ms for hook, jumps and walk on the grid; 3: 2.2; 5: 2.3
__global__ void __launch_bounds__(kBlock) k_wcc_jump(uint32_t* P, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t p = ld_u32(P + v);
    if (p == v) continue;
    uint32_t r = p;
#pragma unroll
    for (int k = 0; k < 3; ++k) r = ld_u32(P + r);
    if (r != p) __hip_atomic_store(P + v, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Sampled static WCC (after the subgraph-sampling method of Sutton, Ben-Nun and Barak,
// "Optimizing parallel graph connectivity computation via subgraph sampling", IPDPS 2018), over
// the undirected view (both ends of an arc see it):
//   1. k_wcc_hook: every vertex points at the neighbour of highest degree among the first four
//      words of its primary slab (ties: smallest uf_order), if that ranks above itself.  No
//      atomics and no contention: the pointers climb towards the hubs.  On a power-law graph
//      this alone gathers nearly every vertex of the giant component under a few hubs.
//   2. k_wcc_link over the remaining roots: each unites with those four neighbours.
//   3. k_wcc_big: the most frequent root among kWccSamples vertices is taken as the largest
//      component.  If it holds less than half of the samples (a road network, where hooking makes
//      small trees), every vertex unites with its first two neighbours and the samples are
//      taken again.
//   4. k_wcc_rest: every vertex points at its root; those outside the largest component are
//      listed, and k_wcc_walk unites them with all their neighbours, so the arcs of the largest
//      component are not read.  An arc with an end outside it is united from that end; an arc
//      with both ends inside joins nothing new, so the partition is the plain one.
//   5. k_wcc_min, k_wcc_label: the smallest id of each component becomes its root and label.
// Uniting every vertex with two neighbours under the smaller id (instead of 1 and 2) took 1.1-1.3
// ms at R-MAT scale 22: half of those unions hook a hub's root, and their CASes meet on a few
// words.  With the walk of step 4 over every vertex, the recompute of R-MAT scale 22 as built took 1.6
// ms; it takes 0.38 (hooks 0.12, links 0.04 to 0.13, with the way the first words happen to lie, walk
// 0.11), and 0.9 to 1.1 after millions of uniform arcs, whose vertices hook less well.
constexpr uint32_t kWccLinks = 2;
constexpr uint32_t kWccSamples = 1024;

__global__ void __launch_bounds__(kBlock) k_wcc_hook(DView V, uint32_t* P, uint32_t* M, uint32_t nv) {
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < nv; u += gridDim.x * blockDim.x) {
    const uint32_t d = V.deg[u];
    uint32_t best = u, bd = d;
    if (d) {
      uint32_t v[kWccHook], dv[kWccHook];
      first_words(V, u, v);
#pragma unroll
      for (uint32_t k = 0; k < kWccHook; ++k) dv[k] = V.deg[valid_key(v[k]) ? v[k] : u];
#pragma unroll
      for (uint32_t k = 0; k < kWccHook; ++k)
        if (valid_key(v[k]) && (dv[k] > bd || (dv[k] == bd && uf_order(v[k]) < uf_order(best)))) {
          best = v[k];
          bd = dv[k];
        }
    }
    P[u] = best;
    M[u] = u;
  }
}

// Unite vertices with neighbours from their primary slabs' first words: the roots with all four
// (all == false), or, when the sample found no largest component (*enough == 0), every vertex
// with the first kWccLinks.
__global__ void __launch_bounds__(kBlock) k_wcc_link(DView V, uint32_t* P, uint32_t nv, bool all,
                                                     const uint32_t* enough) {
  if (all && *enough) return;
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < nv; u += gridDim.x * blockDim.x) {
    if ((!all && ld_u32(P + u) != u) || V.deg[u] == 0) continue;
    uint32_t v[kWccHook], linked = 0;
    first_words(V, u, v);
#pragma unroll
    for (uint32_t k = 0; k < kWccHook; ++k) {
      if (!valid_key(v[k]) || (all && linked == kWccLinks)) continue;
      uf_union_any(P, u, v[k]);
      ++linked;
    }
  }
}

__device__ inline uint32_t wcc_root(const uint32_t* P, uint32_t v) {
  uint32_t r = v;
  for (uint32_t p = ld_u32(P + r); p != r; p = ld_u32(P + r)) r = p;
  return r;
}

// One block of kWccSamples threads: the most frequent root among the sampled vertices into *big,
// and whether it holds at least half of them into *enough.  Samples are spread over the ids by a
// Weyl sequence and counted in an LDS table (two slots per sample, linear probing).  Vertices without
// arcs are in no component worth finding, and R-MAT graphs are full of them (more than half of scale
// 20 at edge factor 4): a thread takes the first of kWccTries vertices that has an arc, or no sample.
// One after the other, as a block has a whole CU's random reads to itself: 9.8 us without, 11.5 with two
// tries, 13 with three, 19 with four at once.  (A recompute with those vertices counted / left out, us:
// edge factor 2, scale 16: 71 / 55, 18: 93 / 74, 20: 177 / 130, 22: 313 / 282; edge factor 8, scale 20:
// 170 / 133, 22: 444 / 288.)
constexpr uint32_t kWccTries = 2;
__global__ void __launch_bounds__(kWccSamples) k_wcc_big(DView U, const uint32_t* P, uint32_t nv, uint32_t* big,
                                                         uint32_t* enough, bool again) {
  __shared__ uint32_t key[2 * kWccSamples], cnt[2 * kWccSamples];
  __shared__ unsigned long long best;
  if (again && *enough) return;
  for (uint32_t i = threadIdx.x; i < 2 * kWccSamples; i += kWccSamples) {
    key[i] = kInvalid;
    cnt[i] = 0;
  }
  if (threadIdx.x == 0) best = 0;
  uint32_t s = kInvalid;
  for (uint32_t k = 0; k < kWccTries && s == kInvalid; ++k) {
    const uint32_t v = (uint32_t)((threadIdx.x + k * kWccSamples) * 0x9E3779B97F4A7C15ull >> 32) % nv;
    if (U.deg[v]) s = v;
  }
  const uint32_t samples = (uint32_t)__syncthreads_count(s != kInvalid);
  if (s != kInvalid) {
    const uint32_t r = wcc_root(P, s);
    uint32_t h = uf_order(r) & (2 * kWccSamples - 1);
    while (true) {
      const uint32_t old = atomicCAS(&key[h], kInvalid, r);
      if (old == kInvalid || old == r) break;
      h = (h + 1) & (2 * kWccSamples - 1);
    }
    const uint32_t n = atomicAdd(&cnt[h], 1u) + 1u;  // the last adder sees the whole count
    // larger count first, then the smaller root
    atomicMax(&best, ((unsigned long long)n << 32) | (0xFFFFFFFFu - r));
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    *big = samples ? 0xFFFFFFFFu - (uint32_t)best : 0u;
    *enough = (uint32_t)(best >> 32) * 2 >= samples;
  }
}

// Every parent made a root (a plain walk, as in k_wcc_compress), and the vertices with arcs
// outside the largest component listed; those of more than kHeavyBuckets buckets a second time.
__global__ void __launch_bounds__(kBlock) k_wcc_rest(DView U, uint32_t* P, uint32_t nv, const uint32_t* big,
                                                     uint32_t* rest, uint32_t* nrest, uint32_t* heavy,
                                                     uint32_t* nheavy) {
  __shared__ Stage S[2];
  stage_open(S[0], rest, nrest);
  stage_open(S[1], heavy, nheavy);
  __syncthreads();
  const uint32_t skip = *big;
  for (uint32_t base = blockIdx.x * kBlock; base < nv; base += gridDim.x * kBlock) {
    const uint32_t v = base + threadIdx.x;
    bool out = false, hv = false;
    if (v < nv) {
      const uint32_t r = wcc_root(P, v);
      __hip_atomic_store(P + v, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (r != skip) {
        out = U.deg[v] != 0;
        hv = out && U.nbk[v] > kHeavyBuckets;
      }
    }
    stage_push(S[0], out, v);
    stage_push(S[1], hv, v);
  }
  stage_close(S);
}

// Unite every listed vertex with all its neighbours: a lane to a vertex of one
// bucket, a 16-lane group to one of up to kHeavyBuckets, a block to the others.
__global__ void __launch_bounds__(kBlock) k_wcc_walk(DView V, uint32_t* P, const uint32_t* rest, const uint32_t* nrest,
                                                     const uint32_t* heavy, const uint32_t* nheavy) {
  const uint32_t n = *nrest, nh = *nheavy;
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  auto unite = [&](uint32_t u, uint32_t ru, uint64_t x, bool data) {
    const uint32_t v = (uint32_t)x;
    if (data && valid_key(v) && ld_u32(P + v) != ru) uf_union_any(P, u, v);
  };
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const uint32_t u = rest[i];
    if (V.nbk[u] != 1 || V.deg[u] == 0) continue;
    const uint32_t ru = uf_find(P, u);
    Slab sl;
    uint32_t t = u;
    while (true) {
      load_slab(V, t, sl);
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j) unite(u, ru, sl.w[j], true);
      t = (uint32_t)sl.w[15];
      if (t == kInvalid) break;
    }
  }
  for (uint32_t i = g0; i < n; i += ng) {
    const uint32_t u = rest[i], nb = V.nbk[u];
    if (nb == 1 || nb > kHeavyBuckets) continue;
    const uint32_t ru = uf_find(P, u);
    for_each_slab(V, u, [&](uint64_t x, bool data) { unite(u, ru, x, data); });
  }
  const uint32_t gib = threadIdx.x / kGroup;
  for (uint32_t j = blockIdx.x; j < nh; j += gridDim.x) {
    const uint32_t u = heavy[j];
    const uint32_t ru = uf_find(P, u);
    for_each_slab_strided(V, u, gib, kGroupsPerBlock, [&](uint64_t x, bool data) { unite(u, ru, x, data); });
  }
}

// The smallest id of each component at its root's entry of M.  No union runs any more, so the
// roots are final.  The members of the largest sampled component make one atomic per block
// (one per wave took 1.4 ms, all on one word); those of the others go straight to their entry,
// unless a smaller id is there already.
__global__ void __launch_bounds__(kBlock) k_wcc_min(uint32_t* P, uint32_t* M, uint32_t nv, const uint32_t* big) {
  __shared__ uint32_t lowest;
  if (threadIdx.x == 0) lowest = kInvalid;
  __syncthreads();
  const uint32_t rb = wcc_root(P, *big);
  uint32_t mine = kInvalid;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t r = wcc_root(P, v);
    __hip_atomic_store(P + v, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (r == rb) mine = min(mine, v);
    else if (v < ld_u32(M + r)) atomicMin(M + r, v);
  }
  for (int o = 32; o > 0; o >>= 1) mine = min(mine, (uint32_t)__shfl_xor((int)mine, o));
  if ((threadIdx.x & 63) == 0) atomicMin(&lowest, mine);
  __syncthreads();
  if (threadIdx.x == 0 && lowest < ld_u32(M + rb)) atomicMin(M + rb, lowest);
}

__global__ void k_wcc_label(uint32_t* P, const uint32_t* M, uint32_t nv, uint32_t* label) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t l = M[P[v]];
    P[v] = l;
    label[v] = l;
  }
}

// IterationScheme2 (section 3.4): one 16-lane group per bucket chain <v, i>, in a
// grid-stride loop over the pair list.  Bucket i > 0 of v is the extra head slab
// N + off[v] - v + i - 1 = N + k - v - 1 (the extra head slabs were laid out by the same
// scan); bucket 0 is v's primary slab, with 14 data words when v has several buckets.
template <class F>
__device__ inline void walk_pair(const DView& V, const uint32_t* pv, const uint32_t* pi, uint32_t nv,
                                 uint32_t k, uint32_t& v, F&& f) {
  v = pv[k];
  const uint32_t i = pi[k];
  const uint32_t h = i == 0 ? v : nv + k - v - 1;
  const uint64_t x = ld_word(slab_ptr(V, h) + glane());
  int nd = kKeysPerSlab;
  if (i == 0 && (uint32_t)(gbcast64(x, 15) >> 32) > 1) nd = kKeysPerSlab - 1;
  walk_chain(V, h, x, nd, f);
}

// Static WCC under IterationScheme2: union over the arcs of every bucket chain.
__global__ void __launch_bounds__(kBlock) k_wcc_pairs(DView F, uint32_t* P, const uint32_t* pv,
                                                      const uint32_t* pi, uint32_t np, uint32_t nv) {
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  for (uint32_t k = g0; k < np; k += ng) {
    const uint32_t u = pv[k];
    const uint32_t ru = uf_find(P, u);
    uint32_t vv;
    walk_pair(F, pv, pi, nv, k, vv, [&](uint64_t x, bool data) {
      const uint32_t v = (uint32_t)x;
      if (data && valid_key(v) && ld_u32(P + v) != ru) uf_union(P, u, v);
    });
  }
}

__global__ void k_wcc_batch(uint32_t* P, Log lg, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    if (lg.st[i] == 1) uf_union(P, lg.s[i], lg.d[i]);
}

// ----------------------------------------------------------------- incremental WCC schemes
// The vertices that gained out-arcs in a pending insert batch, each listed once (the
// to_union flags of section 4.4): vertices with more than kHeavyBuckets buckets go to a
// second list that is walked a block per vertex.
__global__ void k_wcc_flag(Log lg, uint64_t n, const uint32_t* nbk, uint32_t* flag, uint32_t* light,
                           uint32_t* nlight, uint32_t* heavy, uint32_t* nheavy) {
  __shared__ Stage S[2];
  stage_open(S[0], light, nlight);
  stage_open(S[1], heavy, nheavy);
  __syncthreads();
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x; base < n; base += stride) {
    const uint64_t i = base + threadIdx.x;
    bool p = false, hv = false;
    uint32_t u = 0;
    if (i < n && lg.st[i] == 1) {
      u = lg.s[i];
      p = ld_u32(flag + u) == 0u && atomicExch(flag + u, 1u) == 0u;
      hv = p && nbk[u] > kHeavyBuckets;
    }
    stage_push(S[0], p && !hv, u);
    stage_push(S[1], hv, u);
  }
  stage_close(S);
}

__global__ void k_wcc_unflag(uint32_t* flag, const uint32_t* light, const uint32_t* nlight,
                             const uint32_t* heavy, const uint32_t* nheavy) {
  const uint32_t nl = *nlight, nh = *nheavy;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nl + nh; i += gridDim.x * blockDim.x)
    flag[i < nl ? light[i] : heavy[i - nl]] = 0u;
}

// UpdateIterator over one bucket chain (section 3.4).  The chain's mark is <slab + 1, lane>
// of the first word the last pass did not unite (0: the head slab, lane 0).  As a chain's
// filled words always form a prefix, everything inserted since then lies at or past the
// mark, and the first EMPTY word met is the chain's new end: the mark moves there (the
// paper's UpdateSlabPointers, done by the pass itself).  A chain with no new word costs one
// slab read: the paper's per-chain is_updated flag is derived, not stored.
__device__ inline void wcc_update_chain(const DView& F, uint64_t* marks, uint32_t* P, uint32_t h,
                                        int nd0, uint32_t u, uint32_t ru) {
  const int gl = glane();
  const uint64_t m = ld_u64(marks + h);
  uint32_t s = (uint32_t)m ? (uint32_t)m - 1u : h;
  int l = (uint32_t)m ? (int)(m >> 32) : 0;
  int nd = s == h ? nd0 : kKeysPerSlab;
  while (true) {
    const uint64_t x = ld_word(slab_ptr(F, s) + gl);
    const uint32_t v = (uint32_t)x;
    const bool data = gl >= l && gl < nd;
    if (data && valid_key(v) && ld_u32(P + v) != ru) uf_union(P, u, v);
    const uint32_t e = gballot(data && v == kEmptyKey);
    if (e) {
      l = __ffs(e) - 1;
      break;
    }
    const uint32_t nx = gbcast(v, 15);
    if (nx == kInvalid) {
      l = nd;
      break;
    }
    s = nx;
    l = 0;
    nd = kKeysPerSlab;
  }
  const uint64_t nm = ((uint64_t)(uint32_t)l << 32) | (s + 1u);
  if (gl == 0 && nm != m) marks[h] = nm;
}

// Incremental WCC over the listed vertices: every slab of each (SlabIterator scheme, marks
// null) or only the words past each chain's mark (UpdateIterator scheme).  Light vertices
// take a 16-lane group each, heavy ones a block with its groups striding over the buckets.
__global__ void __launch_bounds__(kBlock) k_wcc_listed(DView F, uint32_t* P, uint64_t* marks,
                                                       const uint32_t* light, const uint32_t* nlight,
                                                       const uint32_t* heavy, const uint32_t* nheavy) {
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  const uint32_t gib = threadIdx.x / kGroup;
  auto walk = [&](uint32_t u, uint32_t b0, uint32_t stride) {
    const uint32_t ru = uf_find(P, u);
    if (!marks) {
      for_each_slab_strided(F, u, b0, stride, [&](uint64_t x, bool data) {
        const uint32_t v = (uint32_t)x;
        if (data && valid_key(v) && ld_u32(P + v) != ru) uf_union(P, u, v);
      });
      return;
    }
    const Table t = group_table(F, u);
    for (uint32_t b = b0; b < t.nb; b += stride)
      wcc_update_chain(F, marks, P, b ? t.xb + b - 1 : u,
                       (b == 0 && t.nb > 1) ? kKeysPerSlab - 1 : kKeysPerSlab, u, ru);
  };
  const uint32_t nl = *nlight;
  for (uint32_t i = g0; i < nl; i += ng) walk(light[i], 0, 1);
  const uint32_t nh = *nheavy;
  for (uint32_t j = blockIdx.x; j < nh; j += gridDim.x) walk(heavy[j], gib, kGroupsPerBlock);
}

// UpdateSlabPointers over every chain: each mark moves to its chain's end (the first EMPTY
// word, or past the last slab's data words when the chain is full).  One group per chain.
__global__ void __launch_bounds__(kBlock) k_mark_all(DView F, uint64_t* marks, uint64_t n_head,
                                                     uint32_t nv) {
  const uint64_t g0 = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint64_t ng = (uint64_t)gridDim.x * kGroupsPerBlock;
  const int gl = glane();
  for (uint64_t h = g0; h < n_head; h += ng) {
    uint32_t s = (uint32_t)h;
    uint64_t y = ld_word(slab_ptr(F, s) + gl);
    int nd = (h < nv && (uint32_t)(gbcast64(y, 15) >> 32) > 1) ? kKeysPerSlab - 1 : kKeysPerSlab;
    int l;
    while (true) {
      const uint32_t e = gballot(gl < nd && (uint32_t)y == kEmptyKey);
      if (e) {
        l = __ffs(e) - 1;
        break;
      }
      const uint32_t nx = gbcast((uint32_t)y, 15);
      if (nx == kInvalid) {
        l = nd;
        break;
      }
      s = nx;
      nd = kKeysPerSlab;
      y = ld_word(slab_ptr(F, s) + gl);
    }
    if (gl == 0) marks[h] = ((uint64_t)(uint32_t)l << 32) | (s + 1u);
  }
}

// Full path compression and the labels.  No union runs here, so every root is final and
// any parent a thread reads (the value the union kernels left, or the root another thread
// has just stored) leads to it.  The walk must not halve paths: a halving store computed
// from an earlier read could land after another thread's final store to the same vertex
// and leave it pointing at a non-root.
__global__ void k_wcc_compress(uint32_t* P, uint32_t nv, uint32_t* label) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    uint32_t r = v;
    for (uint32_t p = ld_u32(P + r); p != r; p = ld_u32(P + r)) r = p;
    __hip_atomic_store(P + v, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    label[v] = r;
  }
}

__global__ void k_copy_u32(const uint32_t* a, uint32_t* b, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) b[i] = a[i];
}

// ================================================================= PageRank
__device__ inline double block_sum(double v, double* lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[w] = v;
  __syncthreads();
  double s = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += lds[i];
  return s;  // valid in thread 0
}

__global__ void k_copy_f32(const float* a, float* b, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) b[i] = a[i];
}
__global__ void k_pr_fill(float* x, uint32_t nv, float v) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) x[i] = v;
}

// Contribution per vertex C[u] = PR[u] / out[u] (the FindContributionPerVertex kernel),
// plus the FP64 sum of the ranks of zero-out-degree vertices (FindTeleportProb).
__global__ void __launch_bounds__(kBlock) k_pr_contrib(const float* __restrict__ x,
                                                       const uint32_t* __restrict__ outdeg,
                                                       float* __restrict__ c, uint32_t nv,
                                                       double* dpart, const uint32_t* state) {
  __shared__ double lds[kBlock / 64];
  if (state[0]) return;
  double local = 0;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t o = outdeg[v];
    const float xv = x[v];
    c[v] = o ? xv / (float)o : 0.f;
    if (!o) local += xv;
  }
  const double s = block_sum(local, lds);
  if (threadIdx.x == 0) dpart[blockIdx.x] = s;
}

// Sum of per-block partial sums in a fixed order (one block): the dangling mass and the L1
// change of an iteration are deterministic and take no same-address atomics.  (The in-arc
// sums of vertices split into bucket work items are the exception: their FP64 partials are
// added by atomics, so the order, and the last bits of those ranks, can vary between runs.)
__device__ inline double sum_parts(const double* part, uint32_t n, double* lds) {
  double v = 0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) v += part[i];
  return block_sum(v, lds);
}

__global__ void __launch_bounds__(kBlock) k_pr_sum(const double* part, uint32_t n, double* out,
                                                   const uint32_t* state) {
  __shared__ double lds[kBlock / 64];
  if (state[0]) return;
  const double s = sum_parts(part, n, lds);
  if (threadIdx.x == 0) *out = s;
}

// Pull over in-arcs (reverse view): PR'[v] = (1-d)/N + d * (sum C[u] + dangling/N),
// and the FP64 L1 change sum |PR'[v] - PR[v]|.
__global__ void __launch_bounds__(kBlock) k_pr_gather(DView R, const float* __restrict__ c,
                                                      const float* __restrict__ x,
                                                      float* __restrict__ y, uint32_t nv, float damping,
                                                      const double* dang, double* delta,
                                                      const uint32_t* heavy, const uint32_t* nheavy,
                                                      const uint32_t* hcnt, const uint32_t* hoff,
                                                      double* hacc, const uint32_t* state) {
  __shared__ double lds[kBlock / 64];
  if (state[0]) return;
  const double base = (1.0 - (double)damping) / nv + (double)damping * (*dang) / nv;
  double local = 0;
  // single-bucket vertices (most of a power-law graph): one lane per vertex, so a wave keeps
  // 64 slab reads and their gathers in flight
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    if (R.nbk[v] != 1) continue;
    double s = 0;
    if (R.deg[v] != 0) {  // vertices without in-arcs need no slab read
      Slab sl;
      uint32_t t = v;
      while (true) {
        load_slab(R, t, sl);
#pragma unroll
        for (int j = 0; j < kKeysPerSlab; ++j) {
          const uint32_t u = (uint32_t)sl.w[j];
          if (valid_key(u)) s += (double)c[u];
        }
        t = (uint32_t)sl.w[15];
        if (t == kInvalid) break;
      }
    }
    const float nvl = (float)(base + (double)damping * s);
    y[v] = nvl;
    local += fabs((double)nvl - (double)x[v]);
  }
  // vertices with 2 .. kHeavyBuckets buckets: one 16-lane group per vertex.  The group
  // issues the loads of all its head slabs at once, then all their contribution gathers,
  // and only then follows the (rare) chains, rather than one dependent slab at a time.
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  const int gl = glane();
  for (uint32_t v = g0; v < nv; v += ng) {
    const uint32_t nb = R.nbk[v];
    if (nb == 1 || nb > kHeavyBuckets) continue;
    const uint64_t x0 = ld_word(slab_ptr(R, v) + gl);
    const uint32_t xb = gbcast((uint32_t)x0, 14);
    double s = 0;
    for (uint32_t b0 = 0; b0 < nb; b0 += kPrBatch) {
      uint64_t hw[kPrBatch];
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {
        const uint32_t b = b0 + j;
        hw[j] = b == 0 ? x0 : (b < nb ? ld_word(slab_ptr(R, xb + b - 1) + gl) : kEmptyWord);
      }
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {
        const uint32_t u = (uint32_t)hw[j];
        const bool data = gl < (b0 + j == 0 ? kKeysPerSlab - 1 : kKeysPerSlab);
        if (data && valid_key(u)) s += (double)c[u];
      }
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {  // chained slabs after a full head slab
        if (b0 + j >= nb) break;
        const uint32_t next = gbcast((uint32_t)hw[j], 15);
        if (next == kInvalid) continue;
        walk_chain(R, next, ld_word(slab_ptr(R, next) + gl), kKeysPerSlab, [&](uint64_t w, bool data) {
          const uint32_t u = (uint32_t)w;
          if (data && valid_key(u)) s += (double)c[u];
        });
      }
    }
    s = gsum(s);
    if (glane() == 0) {
      const float nvl = (float)(base + (double)damping * s);
      y[v] = nvl;
      local += fabs((double)nvl - (double)x[v]);
    }
  }
  // heavy vertices: work items of kPrChunk buckets spread over every group; partial sums
  // go to hacc[j] and k_pr_heavy_final turns them into ranks
  const uint32_t nh = *nheavy;
  if (nh) {
    const uint32_t items = hoff[nh - 1] + hcnt[nh - 1];
    for (uint32_t it = g0; it < items; it += ng) {
      uint32_t lo = 0, hi = nh;  // last j with hoff[j] <= it
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (hoff[mid] <= it) lo = mid;
        else hi = mid;
      }
      const uint32_t v = heavy[lo];
      const uint32_t b0 = (it - hoff[lo]) * kPrChunk;
      double s = 0;
      for_each_bucket_range(R, v, b0, b0 + kPrChunk, [&](uint64_t w, bool data) {
        const uint32_t u = (uint32_t)w;
        if (data && valid_key(u)) s += (double)c[u];
      });
      s = gsum(s);
      if (glane() == 0 && s != 0.0) atomicAdd(hacc + lo, s);
    }
  }
  const double s = block_sum(local, lds);
  if (threadIdx.x == 0) delta[blockIdx.x] = s;
}

// ---------------------------------------------------------------- packed iterations
// MK_ITER_PACKED.  A call first packs the graph for its iterations:
//   * the vertices are ordered by out-degree class, largest first (a stable 6-bit radix sort), so
//     that the sources of most in-arcs come first; everything below is indexed by a vertex's
//     rank in that order, so that an iteration reads and writes its vectors in place;
//   * k_pr_pack copies each vertex's in-arc sources, as ranks, out of the slabs into one list,
//     segment after segment (off = the exclusive scan of the in-degrees);
//   * the list and the vertices' segment ends are cut into tiles of kPrTile list entries and
//     segment ends together (merge path), so that every tile is the same work whatever the
//     degrees: fv[t] is the first vertex whose end lies in tile t or later, and tile t's entries
//     start at t * kPrTile - fv[t].
// An iteration (k_pr_flat) gives each wave a tile at a time: 8 consecutive list entries per
// lane, their contributions gathered at once, an FP64 prefix sum over the tile, and a vertex's
// sum as the difference of two prefixes.  A segment that runs over tile borders leaves the
// sum of its last part in heads[t] and of the earlier ones in tails[], which k_pr_fix adds.
//
// What bounds an iteration: the random contribution gathers and the lines they bring into the
// L2s.  So each block keeps the first kPrHot contributions in LDS: half of R-MAT scale 22's arcs
// start there, two thirds of scale 20's.  Scale 22 as built, per iteration: 240 us, 0.94 GB fetched
// (3.9 TB/s; list and vectors are 0.33 GB), and 16 us in the two small kernels (a lane or a group per
// vertex with all gathers through L2: 411 us and 48 us in four small ones).  Of the 240 us, 94
// remain without the cold gathers; 324 us are taken with every gather through L2, 271 with 8,000
// contributions in LDS.  After millions of uniform arcs, whose sources are cold, 277 to 302 us and
// 1.25 GB, near the rate of a copy.  The packing takes 1.0 ms a call, half of it the rank reads,
// which have no hot-first order to help them.
constexpr uint32_t kPrTile = 512;            // list entries and segment ends per tile
constexpr uint32_t kPrFlatThreads = 1024;    // one block per CU: 16 waves share its hot contributions
constexpr uint32_t kPrFlatBlocks = 256;
constexpr uint32_t kPrHot = 24000;           // contributions in LDS (96,000 of 163,840 bytes)
constexpr uint32_t kPrFixBlocks = 512;
constexpr uint32_t kPrFixOne = 8192;         // up to this many tiles one block fixes and checks
static_assert(kPrTile == 64 * 8, "a lane takes 8 entries");

__global__ void k_pr_class(const uint32_t* __restrict__ outdeg, uint32_t nv, uint32_t* key, uint32_t* idx) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    key[v] = (uint32_t)__clz(outdeg[v] + 1u);  // 31 - floor(log2(out + 1)), in [0, 31]
    idx[v] = v;
  }
}

// In rank order: out- and in-degrees, a zero packing cursor; every vertex's rank; no packing item.
__global__ void k_pr_order(const uint32_t* __restrict__ perm, const uint32_t* __restrict__ outdeg,
                           const uint32_t* __restrict__ indeg, uint32_t nv, uint32_t* __restrict__ od,
                           uint32_t* __restrict__ id, uint32_t* __restrict__ rank, uint32_t* __restrict__ cur,
                           uint32_t* nitems) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *nitems = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    const uint32_t v = perm[i];
    od[i] = outdeg[v];
    id[i] = indeg[v];
    rank[v] = i;
    cur[i] = 0;
  }
}

// The identity order, for graphs whose contributions all fit the LDS copy anyway.
__global__ void k_pr_identity(const uint32_t* __restrict__ outdeg, const uint32_t* __restrict__ indeg, uint32_t nv,
                              uint32_t* __restrict__ perm, uint32_t* __restrict__ od, uint32_t* __restrict__ id,
                              uint32_t* __restrict__ rank, uint32_t* __restrict__ cur, uint32_t* nitems) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *nitems = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    perm[i] = rank[i] = i;
    od[i] = outdeg[i];
    id[i] = indeg[i];
    cur[i] = 0;
  }
}

// The merge-path tiles: vertex i's segment end sits at off[i + 1] + i among entries and ends.
// Also off[nv], and the packing items of vertices with more than kHeavyBuckets buckets.
constexpr uint32_t kPackChunk = 64;  // buckets per packing item (a 16-lane group)
__global__ void k_pr_tiles(uint32_t* __restrict__ off, const uint32_t* __restrict__ id, uint32_t nv,
                           uint32_t* __restrict__ fv, const uint32_t* __restrict__ perm,
                           const uint32_t* __restrict__ nbk, uint32_t* item_i, uint32_t* item_c, uint32_t* nitems) {
  const uint32_t ln = threadIdx.x & 63;
  for (uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x - ln; i0 < nv; i0 += gridDim.x * blockDim.x) {
    const uint32_t i = i0 + ln;
    uint32_t k = 0;  // packing items of vertex i
    if (i < nv) {
      const uint64_t o = off[i], q = o + id[i] + i;  // this end; the tile borders after the previous
      for (uint64_t t = i ? (o + i - 1) / kPrTile + 1 : 0; t <= q / kPrTile; ++t) fv[t] = i;
      if (i == nv - 1) {
        off[nv] = (uint32_t)(o + id[i]);
        fv[q / kPrTile + 1] = nv;
      }
      const uint32_t nb = nbk[perm[i]];
      if (nb > kHeavyBuckets) k = (nb + kPackChunk - 1) / kPackChunk;
    }
    if (!__ballot(k != 0)) continue;
    uint32_t incl = k;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if ((int)ln >= o) incl += y;
    }
    uint32_t at = 0;
    if (ln == 63) at = atomicAdd(nitems, incl);
    at = __shfl(at, 63) + incl - k;
    for (uint32_t j = 0; j < k; ++j) {
      item_i[at + j] = i;
      item_c[at + j] = j;
    }
  }
}

// Copy the in-arc sources, as ranks, out of the reverse view's slabs: vertex i (rank order) to
// list[off[i] .. off[i + 1]).  A vertex of more than kHeavyBuckets buckets is several items, whose
// keys take their places through cur[i] (so their order can vary between runs).
__global__ void __launch_bounds__(kBlock) k_pr_pack(DView R, const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ rank, const uint32_t* __restrict__ off,
                                                    uint32_t nv, uint32_t* __restrict__ list, uint32_t* cur,
                                                    const uint32_t* item_i, const uint32_t* item_c,
                                                    const uint32_t* nitems) {
  const uint32_t below = (1u << glane()) - 1u;
  // Head slabs b0 .. b1 - 1 of v (several buckets) and their chains into v's segment [o, o + n), by
  // the calling group: kPrBatch slabs are read at once, then their ranks.  take(k) is the place
  // of the next k keys in the segment.
  auto pack = [&](uint32_t v, uint32_t b0, uint32_t b1, uint32_t o, uint32_t n, auto&& take) {
    const uint32_t xb = (uint32_t)ld_word(slab_ptr(R, v) + 14);
    for (; b0 < b1; b0 += kPrBatch) {
      uint64_t hw[kPrBatch];
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {
        const uint32_t b = b0 + j;
        hw[j] = b < b1 ? ld_word(slab_ptr(R, b ? xb + b - 1 : v) + glane()) : kNextNone;
      }
      uint32_t r[kPrBatch], m[kPrBatch], total = 0;
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {
        const uint32_t u = (uint32_t)hw[j];
        const bool ok = glane() < (b0 + j ? kKeysPerSlab : kKeysPerSlab - 1) && valid_key(u);
        r[j] = rank[ok ? u : 0u];  // unconditional: the compiler would wait for each otherwise
        m[j] = gballot(ok);
        total += __popc(m[j]);
      }
      uint32_t at = take(total);
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {
        const uint32_t p = at + __popc(m[j] & below);
        if ((m[j] >> glane() & 1) && p < n) list[o + p] = r[j];
        at += __popc(m[j]);
      }
#pragma unroll
      for (uint32_t j = 0; j < kPrBatch; ++j) {  // chained slabs after a full head slab
        const uint32_t next = gbcast((uint32_t)hw[j], 15);
        if (b0 + j >= b1 || next == kInvalid) continue;
        walk_chain(R, next, ld_word(slab_ptr(R, next) + glane()), kKeysPerSlab, [&](uint64_t w, bool data) {
          const bool ok = data && valid_key((uint32_t)w);
          const uint32_t k = gballot(ok), p = take(__popc(k)) + __popc(k & below);
          if (ok && p < n) list[o + p] = rank[(uint32_t)w];
        });
      }
    }
  };
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  const uint32_t items = *nitems;
  for (uint32_t it = g0; it < items; it += ng) {
    const uint32_t i = item_i[it], v = perm[i], b0 = item_c[it] * kPackChunk;
    const uint32_t o = off[i], n = off[i + 1] - o;
    pack(v, b0, min(R.nbk[v], b0 + kPackChunk), o, n, [&](uint32_t k) {
      uint32_t at = 0;
      if (glane() == 0 && k) at = atomicAdd(cur + i, k);
      return gbcast(at, 0);
    });
  }
  // single-bucket vertices: a lane each
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < nv; i += gridDim.x * kBlock) {
    const uint32_t o = off[i], n = off[i + 1] - o;
    if (n == 0) continue;
    const uint32_t v = perm[i];
    if (R.nbk[v] != 1) continue;
    Slab sl;
    uint32_t s = v, at = 0;
    while (true) {
      load_slab(R, s, sl);
      uint32_t r[kKeysPerSlab];
      const uint32_t live = live_words(sl, kKeysPerSlab);
      load_of_keys<uint32_t>(rank, sl, live, 0u, r);
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j)
        if (live >> j & 1) {
          if (at < n) list[o + at] = r[j];
          ++at;
        }
      s = (uint32_t)sl.w[15];
      if (s == kInvalid) break;
    }
  }
  // 2 .. kHeavyBuckets buckets: a 16-lane group each
  for (uint32_t i = g0; i < nv; i += ng) {
    const uint32_t o = off[i], n = off[i + 1] - o;
    if (n == 0) continue;
    const uint32_t v = perm[i], nb = R.nbk[v];
    if (nb == 1 || nb > kHeavyBuckets) continue;
    uint32_t at = 0;  // the same in every lane of the group
    pack(v, 0, nb, o, n, [&](uint32_t k) {
      at += k;
      return at - k;
    });
  }
}

// The ranks in rank order, the contributions, and the FP64 mass of the vertices without out-arcs.
__global__ void __launch_bounds__(kBlock) k_pr_load(const float* __restrict__ keep, const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ od, uint32_t nv, float* __restrict__ x,
                                                    float* __restrict__ c, double* dpart) {
  __shared__ double lds[kBlock / 64];
  double local = 0;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    const float xv = keep[perm[i]];
    const uint32_t o = od[i];
    x[i] = xv;
    c[i] = o ? xv / (float)o : 0.f;
    if (!o) local += xv;
  }
  const double s = block_sum(local, lds);
  if (threadIdx.x == 0) dpart[blockIdx.x] = s;
}

__device__ inline bool pr_check_step(Counters* C, int slot, double tol, uint32_t max_iter, double d, uint32_t* pin);

// What an iteration reads and writes (all in rank order).
struct PrIter {
  const uint32_t *off, *list, *fv, *od;
  const float *c, *x;   // contributions and ranks of this iteration
  float *cn, *y;        // and of the next
  double *heads, *tails;  // per tile: the parts of segments that run over tile borders
  double *ddang, *ddelta;  // per block: dangling mass of y, L1 change
  const uint32_t* state;
  const double* dang;   // dangling mass of x
  uint32_t nv;
  float damping;
};

__device__ inline double pr_base(const PrIter& a) {
  return (1.0 - (double)a.damping) / a.nv + (double)a.damping * (*a.dang) / a.nv;
}
// The new rank of vertex i from its in-arc sum, its contribution, and its shares of the L1
// change and the dangling mass.
__device__ inline void pr_finish(const PrIter& a, double base, uint32_t i, double s, float x, uint32_t od,
                                 double& delta, double& dang) {
  const float r = (float)(base + (double)a.damping * s);
  a.y[i] = r;
  a.cn[i] = od ? r / (float)od : 0.f;
  if (!od) dang += r;
  delta += fabs((double)r - (double)x);
}

// Inclusive sum over the lanes of a wave (every lane active): DPP moves within the rows of 16
// lanes, then row totals broadcast to the rows behind them; a lane without a source adds zero.
template <int kCtrl, int kRows>
__device__ inline double dpp_or_zero(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, kRows, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, kRows, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ inline double wave_scan(double v) {
  v += dpp_or_zero<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);  // lane 15 of a row to the next row, rows 1 and 3
  v += dpp_or_zero<0x143, 0xC>(v);  // lane 31 to rows 2 and 3
  return v;
}

struct __attribute__((packed, aligned(4))) U4 {  // four list entries at any entry's address
  uint32_t v[4];
};

__global__ void __launch_bounds__(kPrFlatThreads) k_pr_flat(PrIter a) {
  constexpr uint32_t kWaves = kPrFlatThreads / 64;
  __shared__ __align__(16) float hot[kPrHot];
  __shared__ double pre[kWaves][kPrTile + 1];
  __shared__ double lds[2][kWaves];
  if (a.state[0]) return;
  const uint32_t nv = a.nv, nh = min(nv, kPrHot);
  for (uint32_t i = threadIdx.x; i < nh; i += kPrFlatThreads) hot[i] = a.c[i];
  __syncthreads();
  const double base = pr_base(a);
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t M = a.off[nv];
  const uint32_t T = (uint32_t)(((uint64_t)M + nv + kPrTile - 1) / kPrTile);  // pr_tiles
  double* P = pre[w];
  // the prefix before entry k of the tile; entry 8 l + j sits at 64 j + l, so that the lanes'
  // stores do not meet in a bank
  auto at = [&](uint32_t k) { return P[k == kPrTile ? kPrTile : (k & 7) * 64 + (k >> 3)]; };
  double delta = 0, dang = 0;
  constexpr uint32_t kStep = kPrFlatBlocks * kWaves;
  // While a tile is worked on, the next one's list entries are on their way, and the borders of
  // the one after it (four waves to a SIMD do not hide a tile's chain of loads by themselves).
  // The list has a tile of slack behind its last entry, fv two entries.
  struct Border {
    uint32_t f0, f1;
  };
  auto border = [&](uint32_t t) { return t < T ? Border{a.fv[t], a.fv[t + 1]} : Border{nv, nv}; };
  auto first_entry = [&](uint32_t t, uint32_t f0) { return t < T ? (uint32_t)((uint64_t)t * kPrTile - f0) : M; };
  uint32_t t = blockIdx.x * kWaves + w;
  Border cur = border(t), nxt = border(t + kStep);
  const U4* p = reinterpret_cast<const U4*>(a.list + first_entry(t, cur.f0) + 8 * lane);
  U4 q0 = p[0], q1 = p[1];
  for (; t < T; t += kStep) {
    const uint32_t f0 = cur.f0, f1 = cur.f1;
    const uint32_t e0 = first_entry(t, f0);
    const uint32_t e1 = t + 1 == T ? M : (uint32_t)((uint64_t)(t + 1) * kPrTile - f1);
    const uint32_t ne = e1 - e0;
    uint32_t u[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) u[k] = min(k < 4 ? q0.v[k] : q1.v[k - 4], nv - 1);
    // a hot entry's global load goes to one shared line, a cold one's LDS read to the last slot
    float g[8], l[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) g[k] = a.c[max(u[k], nh - 1)];
    const Border after = border(t + 2 * kStep);
    p = reinterpret_cast<const U4*>(a.list + first_entry(t + kStep, nxt.f0) + 8 * lane);
    q0 = p[0];
    q1 = p[1];
    // the segment borders, old ranks and out-degrees of the tile's first 64 vertices
    uint32_t v = min(f0 + lane, nv - 1);
    uint32_t o0 = a.off[v], o1 = a.off[v + 1], od = a.od[v];
    float xv = a.x[v];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) l[k] = hot[min(u[k], nh - 1)];
    double sum = 0, ex[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      ex[k] = sum;
      const float cv = u[k] < nh ? l[k] : g[k];
      sum += 8 * lane + k < ne ? (double)cv : 0.0;
    }
    const double incl = wave_scan(sum);
    const double before = incl - sum;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) P[k * 64 + lane] = before + ex[k];
    if (lane == 63) P[kPrTile] = incl;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t v0 = f0; v0 < f1; v0 += 64) {
      v = v0 + lane;
      if (v0 != f0) {
        const uint32_t vc = min(v, nv - 1);
        o0 = a.off[vc];
        o1 = a.off[vc + 1];
        od = a.od[vc];
        xv = a.x[vc];
      }
      if (v < f1) {
        const double s = at(o1 - e0) - at(max(o0, e0) - e0);
        if (o0 < e0) a.heads[t] = s;  // only v == f0: its segment began in an earlier tile
        else pr_finish(a, base, v, s, xv, od, delta, dang);
      }
    }
    if (lane == 0 && f1 < nv) a.tails[t] = at(ne) - at(min(max(a.off[f1], e0), e1) - e0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    cur = nxt;
    nxt = after;
  }
  for (int o = 32; o > 0; o >>= 1) {
    delta += __shfl_xor(delta, o);
    dang += __shfl_xor(dang, o);
  }
  if (lane == 0) {
    lds[0][w] = delta;
    lds[1][w] = dang;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0;
    for (uint32_t i = 0; i < kWaves; ++i) s += lds[threadIdx.x][i];
    (threadIdx.x == 0 ? a.ddelta : a.ddang)[blockIdx.x] = s;
  }
}

// The vertices whose segment runs over a tile border, tiles [t0, T) by steps of `stride` (a wave
// takes 64 consecutive tiles): a lane per tile adds the parts of the vertex that ends there, the
// whole wave where there are many.  finish(v, sum) is called by one lane per such vertex.
template <class Finish>
__device__ inline void pr_fix_tiles(const PrIter& a, uint32_t t0, uint32_t T, uint32_t stride, Finish&& finish) {
  const uint32_t lane = threadIdx.x & 63;
  for (; t0 < T; t0 += stride) {
    const uint32_t t = t0 + lane;
    uint32_t v = 0, first = t;
    bool mine = false;
    if (t > 0 && t < T) {
      v = a.fv[t];
      if (v < a.fv[t + 1]) {
        const uint64_t e0 = (uint64_t)t * kPrTile - v;
        const uint32_t o0 = a.off[v];
        if (o0 < e0) {
          mine = true;
          first = (uint32_t)(((uint64_t)o0 + v) / kPrTile);  // the tile the segment begins in
        }
      }
    }
    const uint32_t span = t - first;
    if (mine && span <= 8) {
      double s = 0;
      for (uint32_t k = first; k < t; ++k) s += a.tails[k];
      finish(v, s + a.heads[t]);
    }
    for (uint64_t m = __ballot(mine && span > 8); m; m &= m - 1) {
      const int from = __builtin_ctzll(m);
      const uint32_t b = __shfl(first, from), e = __shfl(t, from);
      double s = 0;
      for (uint32_t k = b + lane; k < e; k += 64) s += a.tails[k];
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      if ((int)lane == from) finish(v, s + a.heads[t]);
    }
  }
}

__device__ inline uint32_t pr_tiles(const PrIter& a) {
  return (uint32_t)(((uint64_t)a.off[a.nv] + a.nv + kPrTile - 1) / kPrTile);
}

__global__ void __launch_bounds__(kBlock) k_pr_fix(PrIter a) {
  __shared__ double lds[kBlock / 64];
  if (a.state[0]) return;
  const double base = pr_base(a);
  double delta = 0, dang = 0;
  pr_fix_tiles(a, (blockIdx.x * kBlock + threadIdx.x) & ~63u, pr_tiles(a), kPrFixBlocks * kBlock,
               [&](uint32_t v, double s) { pr_finish(a, base, v, s, a.x[v], a.od[v], delta, dang); });
  const double s0 = block_sum(delta, lds), s1 = block_sum(dang, lds);
  if (threadIdx.x == 0) {
    a.ddelta[kPrFlatBlocks + blockIdx.x] = s0;
    a.ddang[kPrFlatBlocks + blockIdx.x] = s1;
  }
}

// The same and the convergence check in one block, for graphs of few tiles (kPrFixOne).
__global__ void __launch_bounds__(1024) k_pr_fix_check(PrIter a, Counters* C, int slot, double tol, uint32_t max_iter,
                                                       uint32_t* pin) {
  __shared__ double lds[1024 / 64];
  if (a.state[0]) return;
  const double base = pr_base(a);
  double delta = 0, dang = 0;
  pr_fix_tiles(a, threadIdx.x & ~63u, pr_tiles(a), 1024,
               [&](uint32_t v, double s) { pr_finish(a, base, v, s, a.x[v], a.od[v], delta, dang); });
  if (threadIdx.x < kPrFlatBlocks) {
    delta += a.ddelta[threadIdx.x];
    dang += a.ddang[threadIdx.x];
  }
  const double d = block_sum(delta, lds), next = block_sum(dang, lds);
  if (threadIdx.x != 0) return;
  C->pr_acc[2 * ((slot + 1) & 3)] = next;
  pr_check_step(C, slot, tol, max_iter, d, pin);
}

// Every iteration of a small graph in one launch of one block (at most kPrSmallN vertices, and
// kPrSmallTiles tiles before one block takes longer than the launches): the contributions
// of this and the next iteration are in LDS, the waves meet at barriers, and the check decides
// whether to go on.  An iteration of the 4,096-vertex random graph takes 10 us; as three launches,
// with a read-back every fourth time, 20 us.  A call, one launch / launches, us: 2,000 vertices at 35
// tiles 172 / 344, at 121 210 / 257, at 160 234 / 208, at 238 296 / 208; 8,000 at 78 396 / 466, at 140
// 342 / 339; R-MAT of 4,096 at 112 273 / 277, of 8,192 at 130 371 / 355.
constexpr uint32_t kPrSmallN = 11800, kPrSmallTiles = 128;
__global__ void __launch_bounds__(kPrFlatThreads) k_pr_small(PrIter a, float* x1, Counters* C, double tol,
                                                             uint32_t max_iter, uint32_t* pin) {
  constexpr uint32_t kWaves = kPrFlatThreads / 64;
  __shared__ float cl[2][kPrSmallN];
  __shared__ double pre[kWaves][kPrTile + 1], lds[kWaves];
  __shared__ double dang_s;
  __shared__ uint32_t go;
  const uint32_t nv = a.nv, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t M = a.off[nv], T = pr_tiles(a);
  float* x[2] = {const_cast<float*>(a.x), x1};
  double* P = pre[w];
  auto at = [&](uint32_t k) { return P[k == kPrTile ? kPrTile : (k & 7) * 64 + (k >> 3)]; };
  double d0 = 0;
  for (uint32_t i = threadIdx.x; i < nv; i += kPrFlatThreads) {
    const uint32_t o = a.od[i];
    const float xv = x[0][i];
    cl[0][i] = o ? xv / (float)o : 0.f;
    if (!o) d0 += xv;
  }
  d0 = block_sum(d0, lds);
  if (threadIdx.x == 0) dang_s = d0;
  a.dang = &dang_s;
  for (uint32_t it = 0;; ++it) {
    __syncthreads();
    const float* c = cl[it & 1];
    a.x = x[it & 1];
    a.y = x[(it + 1) & 1];
    a.cn = cl[(it + 1) & 1];
    const double base = pr_base(a);
    double delta = 0, dang = 0;
    for (uint32_t t = w; t < T; t += kWaves) {
      const uint32_t f0 = a.fv[t], f1 = a.fv[t + 1];
      const uint32_t e0 = t * kPrTile - f0, e1 = t + 1 == T ? M : (t + 1) * kPrTile - f1, ne = e1 - e0;
      const U4* p = reinterpret_cast<const U4*>(a.list + e0 + 8 * lane);
      const U4 q0 = p[0], q1 = p[1];
      double sum = 0, ex[8];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) {
        const float cv = c[min(k < 4 ? q0.v[k] : q1.v[k - 4], nv - 1)];
        ex[k] = sum;
        sum += 8 * lane + k < ne ? (double)cv : 0.0;
      }
      const double incl = wave_scan(sum), before = incl - sum;
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) P[k * 64 + lane] = before + ex[k];
      if (lane == 63) P[kPrTile] = incl;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (uint32_t v = f0 + lane; v < f1; v += 64) {
        const uint32_t o0 = a.off[v], o1 = a.off[v + 1];
        const double s = at(o1 - e0) - at(max(o0, e0) - e0);
        if (o0 < e0) a.heads[t] = s;
        else pr_finish(a, base, v, s, a.x[v], a.od[v], delta, dang);
      }
      if (lane == 0 && f1 < nv) a.tails[t] = at(ne) - at(min(max(a.off[f1], e0), e1) - e0);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    pr_fix_tiles(a, threadIdx.x & ~63u, T, kPrFlatThreads,
                 [&](uint32_t v, double s) { pr_finish(a, base, v, s, a.x[v], a.od[v], delta, dang); });
    const double d = block_sum(delta, lds), next = block_sum(dang, lds);
    if (threadIdx.x == 0) {
      dang_s = next;
      go = !pr_check_step(C, (int)(it & 3), tol, max_iter, d, pin);
    }
    __syncthreads();
    if (!go) return;  // the same in every thread
  }
}

// PageRank pull under IterationScheme2: the FP64 in-arc sum of every reverse-view bucket
// chain into pp[k]; k_pr_final_s2 adds a vertex's buckets in bucket order.
__global__ void __launch_bounds__(kBlock) k_pr_gather_s2(DView R, const float* __restrict__ c,
                                                         const uint32_t* pv, const uint32_t* pi, uint32_t np,
                                                         uint32_t nv, double* __restrict__ pp,
                                                         const uint32_t* state) {
  if (state[0]) return;
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  for (uint32_t k = g0; k < np; k += ng) {
    double s = 0;
    uint32_t v;
    walk_pair(R, pv, pi, nv, k, v, [&](uint64_t w, bool data) {
      const uint32_t u = (uint32_t)w;
      if (data && valid_key(u)) s += (double)c[u];
    });
    s = gsum(s);
    if (glane() == 0) pp[k] = s;
  }
}

__global__ void __launch_bounds__(kBlock) k_pr_final_s2(const uint32_t* __restrict__ nbk,
                                                        const uint32_t* __restrict__ off,
                                                        const double* __restrict__ pp, const float* __restrict__ x,
                                                        float* __restrict__ y, uint32_t nv, float damping,
                                                        const double* dang, double* delta, const uint32_t* state) {
  __shared__ double lds[kBlock / 64];
  if (state[0]) return;
  const double base = (1.0 - (double)damping) / nv + (double)damping * (*dang) / nv;
  double local = 0;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t o = off[v], nb = nbk[v];
    double s = 0;
    for (uint32_t i = 0; i < nb; ++i) s += pp[o + i];
    const float nvl = (float)(base + (double)damping * s);
    y[v] = nvl;
    local += fabs((double)nvl - (double)x[v]);
  }
  const double s = block_sum(local, lds);
  if (threadIdx.x == 0) delta[blockIdx.x] = s;
}

// Work items per heavy vertex: ceil(buckets / kPrChunk).
__global__ void k_heavy_items(const uint32_t* nbk, const uint32_t* heavy, const uint32_t* nheavy,
                              uint32_t* cnt, double* acc) {
  const uint32_t nh = *nheavy;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < nh; j += gridDim.x * blockDim.x) {
    cnt[j] = (nbk[heavy[j]] + kPrChunk - 1) / kPrChunk;
    acc[j] = 0.0;
  }
}

// Ranks of the heavy vertices from their partial sums (and their share of the L1 change).
__global__ void __launch_bounds__(kBlock) k_pr_heavy_final(const uint32_t* heavy, const uint32_t* nheavy,
                                                           double* acc, const float* x, float* y,
                                                           uint32_t nv, float damping, const double* dang,
                                                           double* delta, const uint32_t* state) {
  __shared__ double lds[kBlock / 64];
  if (state[0]) return;
  const double base = (1.0 - (double)damping) / nv + (double)damping * (*dang) / nv;
  const uint32_t nh = *nheavy;
  double local = 0;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < nh; j += gridDim.x * blockDim.x) {
    const uint32_t v = heavy[j];
    const float nvl = (float)(base + (double)damping * acc[j]);
    y[v] = nvl;
    acc[j] = 0.0;
    local += fabs((double)nvl - (double)x[v]);
  }
  const double s = block_sum(local, lds);
  if (threadIdx.x == 0) delta[blockIdx.x] = s;
}

// Convergence bookkeeping for one iteration (one thread): d is its L1 change.  Stop at d <= tol,
// when the change has not improved for three iterations (the FP32 noise floor), or at max_iter.
// The done flag and the iteration count also go to `pin`, two words of pinned host memory, so
// that the host needs a synchronization and no copy to read them (null where it does not read them).
__device__ inline bool pr_check_step(Counters* C, int slot, double tol, uint32_t max_iter, double d, uint32_t* pin) {
  uint32_t* st = C->pr_state;
  C->pr_acc[2 * slot + 1] = d;
  st[1] += 1;
  C->pr_last = d;
  if (d < C->pr_best * 0.999) {
    C->pr_best = d;
    st[2] = 0;
  } else {
    st[2] += 1;
  }
  const bool done = d <= tol || st[2] >= 3 || st[1] >= max_iter;
  if (done) st[0] = 1;
  if (pin) {
    pin[0] = done ? 1u : 0u;
    pin[1] = st[1];
  }
  return done;
}

// The check over per-block partial sums.  With `gpart` (the packed iterations), it also sums the
// next iteration's dangling mass.
__global__ void __launch_bounds__(kBlock) k_pr_check(Counters* C, int slot, double tol, uint32_t max_iter,
                                                     const double* dpart, uint32_t nparts, const double* gpart,
                                                     uint32_t* pin) {
  __shared__ double lds[kBlock / 64];
  if (C->pr_state[0]) return;
  const double d = sum_parts(dpart, nparts, lds);
  const double next = gpart ? sum_parts(gpart, nparts, lds) : 0.0;
  if (threadIdx.x != 0) return;
  if (gpart) C->pr_acc[2 * ((slot + 1) & 3)] = next;
  pr_check_step(C, slot, tol, max_iter, d, pin);
}

__global__ void k_pr_start(Counters* C) {
  if (threadIdx.x != 0) return;
  for (int i = 0; i < 8; ++i) C->pr_acc[i] = 0.0;
  C->pr_state[0] = 0;
  C->pr_state[1] = 0;
  C->pr_state[2] = 0;
  C->pr_last = 0;
  C->pr_best = 1e300;
}

// Copy the final vector (buffer iters % 2) to the persistent state and the output.
__global__ void k_pr_final(const Counters* C, const float* a, const float* b, float* keep, float* out,
                           uint32_t nv, uint32_t* iters_out) {
  const uint32_t it = C->pr_state[1];
  const float* src = (it & 1) ? b : a;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += gridDim.x * blockDim.x) {
    const float v = src[i];
    if (keep != src) keep[i] = v;
    out[i] = v;
  }
  if (iters_out && blockIdx.x == 0 && threadIdx.x == 0) *iters_out = it;
}

// The same from the rank order of the packed iterations.
__global__ void k_pr_store(const Counters* C, const float* a, const float* b, const uint32_t* __restrict__ rank,
                           float* __restrict__ keep, float* __restrict__ out, uint32_t nv, uint32_t* iters_out) {
  const uint32_t it = C->pr_state[1];
  const float* src = (it & 1) ? b : a;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const float r = src[rank[v]];
    keep[v] = r;
    out[v] = r;
  }
  if (iters_out && blockIdx.x == 0 && threadIdx.x == 0) *iters_out = it;
}

// ================================================================= triangle counting
// |N(a) intersect N(b)| counted by the calling group: walk N(a), each lane probes its
// neighbour in b's table.  Returns the group total in every lane.
__device__ inline uint64_t group_intersect(const DView& U, uint32_t a, uint32_t b) {
  const Table tb = group_table(U, b);
  uint64_t c = 0;
  for_each_slab(U, a, [&](uint64_t x, bool data) {
    const uint32_t k = (uint32_t)x;
    if (data && valid_key(k) && k != b) c += lane_has(U, tb, k);
  });
  return gsum_u64(c);
}

// Keys of the batch graph: both directions of each effective undirected change, or a
// sentinel (vertex N) that sorts last.
__global__ void k_tc_keys(Log lg, uint64_t n, uint32_t nv, uint64_t* keys) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    uint64_t k0 = (uint64_t)nv << 32, k1 = k0;
    if (lg.uf[i]) {
      const uint32_t a = min(lg.s[i], lg.d[i]), b = max(lg.s[i], lg.d[i]);
      k0 = ((uint64_t)a << 32) | b;
      k1 = ((uint64_t)b << 32) | a;
    }
    keys[2 * i] = k0;
    keys[2 * i + 1] = k1;
  }
}

__device__ inline uint64_t lower_bound_u64(const uint64_t* a, uint64_t n, uint64_t key) {
  uint64_t lo = 0, hi = n;
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if (a[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Where each source's arcs start and end in the sorted batch keys (every vertex of a batch
// arc is the source of the reverse arc too, so both ends of an arc have a segment).
__global__ void k_tc_segs(const uint64_t* keys, uint64_t nk, uint32_t nv, uint32_t* seg_lo, uint32_t* seg_hi) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nk;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t src = (uint32_t)(keys[i] >> 32);
    if (src >= nv) continue;  // sentinels sort last
    if (i == 0 || (uint32_t)(keys[i - 1] >> 32) != src) seg_lo[src] = (uint32_t)i;
    if (i + 1 == nk || (uint32_t)(keys[i + 1] >> 32) != src) seg_hi[src] = (uint32_t)(i + 1);
  }
}

// Which end of a canonical batch edge {u, v} (u < v) is walked for S1: the end of smaller
// live degree (ties: u).  The other end, b, is the one whose neighbourhood is looked up.
__device__ inline bool tc_walk_u(const DView& U, uint32_t u, uint32_t v) { return U.deg[u] <= U.deg[v]; }
// The walked end of the batch edge {x, y}, in either order.
__device__ inline uint32_t tc_walked(const DView& U, uint32_t x, uint32_t y) {
  const uint32_t u = min(x, y), v = max(x, y);
  return tc_walk_u(U, u, v) ? u : v;
}

// A vertex b with more than kTcHubDeg neighbours and at least kTcHubEdges batch edges is a
// hub; so is one with more than kTcHubBig neighbours and fewer batch edges when one of its
// batch partners has more than kTcHubDeg neighbours (that edge's walk would otherwise take
// hundreds of slabs on one 16-lane group, the tail of a small batch; a large vertex whose few
// partners are small costs less by probing, the common case after uniform inserts).  Every
// caller sees b's segment [lo, hi) of the sorted batch keys.
// The S1 terms of the batch edges whose looked-up end is a hub, the S2 terms of every batch
// arc leaving a hub and of every arc into a hub from its walked end, are counted by k_tc_hub,
// which loads the hub's neighbourhood into an LDS hash set once for all of them (a smaller
// vertex with few batch edges costs less by probing).  Every other term is counted by
// k_tc_batch, one group per batch arc.
constexpr uint32_t kTcHubDeg = 512;
constexpr uint32_t kTcHubEdges = 4;
constexpr uint32_t kTcHubBig = 2048;
__device__ inline bool tc_is_hub(const DView& U, uint32_t b, const uint64_t* keys, uint32_t lo, uint32_t hi) {
  const uint32_t d = U.deg[b];
  if (d <= kTcHubDeg) return false;
  if (hi - lo >= kTcHubEdges) return true;
  if (d <= kTcHubBig) return false;
  for (uint32_t i = lo; i < hi; ++i)  // fewer than kTcHubEdges entries
    if (U.deg[(uint32_t)keys[i]] > kTcHubDeg) return true;
  return false;
}

// S1, S2 and S3 of the batch identity, one group per batch arc (u, v):
//   S1 += |N_G(u) & N_G(v)|, S2 += |N_G(u) & N_B(v)|, S3 += |N_B(u) & N_B(v)|
// with G the graph after the batch and B the graph of the batch alone (S1 and S3 on the
// canonical direction u < v, counted twice).  The terms k_tc_hub counts are skipped, and with
// kList S1 of an arc whose walked end has more than kTcLong buckets is listed for k_tc_long, a block
// per arc: walked by one group, a vertex of 2,000 neighbours took 200 us, the whole kernel's time
// after a batch of 1,000 arcs.  That pays where the batch leaves the chip idle; where it fills it, a
// block per arc only idles lanes.  k_tc_batch + k_tc_long, us: scale 16, 997 arcs: 46 with more than
// 8 buckets listed, 43 with 16, 67 with 32 or 64 (209 without); scale 20, 100K arcs: 405 at 8, 435
// at 16 or 32, 340 at 64 (349 without); scale 22, 1M deleted arcs: 1,739 at 64
// (1,400 without).
constexpr uint64_t kTcFewKeys = 65536;
constexpr uint32_t kTcLong = 16;
template <bool kList>
__global__ void __launch_bounds__(kBlock) k_tc_batch(DView U, const uint64_t* keys, uint64_t nk,
                                                     const uint32_t* seg_lo, const uint32_t* seg_hi,
                                                     uint32_t nv, bool s2in, unsigned long long* S,
                                                     uint32_t* longs, uint32_t* nlongs) {
  __shared__ Stage L[1];
  if (kList) {
    stage_open(L[0], longs, nlongs);
    __syncthreads();
  }
  const uint64_t g0 = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint64_t ng = (uint64_t)gridDim.x * kGroupsPerBlock;
  uint64_t s1 = 0, s2 = 0, s3 = 0;
  const int gl = glane();
  for (uint64_t i = g0; i < nk; i += ng) {
    const uint64_t key = keys[i];
    const uint32_t u = (uint32_t)(key >> 32), v = (uint32_t)key;
    if (u >= nv) break;  // sentinels sort last
    const bool canon = u < v;
    const uint32_t a = tc_walked(U, u, v), b = a == u ? v : u;
    const bool hub = tc_is_hub(U, b, keys, seg_lo[b], seg_hi[b]);
    uint64_t c1 = 0;
    const bool is_long = kList && canon && !hub && U.nbk[a] > kTcLong;
    if (kList) stage_push(L[0], is_long && gl == 0, (uint32_t)i);
    if (canon && !hub && !is_long) c1 = 2 * group_intersect(U, a, b);  // walk the smaller side, probe the other
    // batch neighbourhoods: the segments of v and u in the sorted key list
    const uint64_t vlo = seg_lo[v], vhi = seg_hi[v];
    const uint64_t ulo = seg_lo[u], uhi = seg_hi[u];
    auto in_seg = [&](uint64_t lo, uint64_t hi, uint32_t src, uint32_t x) {
      const uint64_t want = ((uint64_t)src << 32) | x;
      const uint64_t q = lower_bound_u64(keys + lo, hi - lo, want);
      return q < hi - lo && keys[lo + q] == want;
    };
    uint64_t c2 = 0, c3 = 0;
    if (tc_is_hub(U, u, keys, (uint32_t)ulo, (uint32_t)uhi)) {
      // S2 of a hub's directions is counted by k_tc_hub against its LDS sets
    } else if (s2in && tc_is_hub(U, v, keys, (uint32_t)vlo, (uint32_t)vhi) && a == u) {
      // so is S2 of an arc into a hub from the end walked against the hub's set
    } else if (2ull * U.deg[u] < vhi - vlo) {
      // S2 from the smaller side: walk N_G(u), look each key up in v's sorted segment
      for_each_slab(U, u, [&](uint64_t w, bool data) {
        const uint32_t x = (uint32_t)w;
        if (data && valid_key(x)) c2 += in_seg(vlo, vhi, v, x);
      });
    } else {
      // S2 by probing: every x of N_B(v) in u's table
      const Table tu = group_table(U, u);
      for (uint64_t j = vlo + gl; j < vhi; j += kGroup) {
        const uint32_t x = (uint32_t)keys[j];
        if (x != u) c2 += lane_has(U, tu, x);
      }
    }
    if (canon) {
      // S3: the smaller segment's entries looked up in the other segment
      const bool u_short = uhi - ulo <= vhi - vlo;
      const uint64_t lo = u_short ? ulo : vlo, hi = u_short ? uhi : vhi;
      const uint64_t olo = u_short ? vlo : ulo, ohi = u_short ? vhi : uhi;
      const uint32_t other = u_short ? v : u;
      for (uint64_t j = lo + gl; j < hi; j += kGroup) {
        const uint32_t x = (uint32_t)keys[j];
        if (x != other) c3 += 2 * in_seg(olo, ohi, other, x);
      }
    }
    c2 = gsum_u64(c2);
    c3 = gsum_u64(c3);
    if (gl == 0) {
      s1 += c1;
      s2 += c2;
      s3 += c3;
    }
  }
  if (gl == 0) {
    if (s1) atomicAdd(S + 0, (unsigned long long)s1);
    if (s2) atomicAdd(S + 1, (unsigned long long)s2);
    if (s3) atomicAdd(S + 2, (unsigned long long)s3);
  }
  if (kList) stage_close(L);
}

// S1 of the listed arcs: a block walks the smaller side, its groups striding over the buckets, and
// probes the other side's table.
__global__ void __launch_bounds__(kBlock) k_tc_long(DView U, const uint64_t* keys, const uint32_t* longs,
                                                    const uint32_t* nlongs, unsigned long long* S) {
  const uint32_t n = *nlongs;
  uint64_t c = 0;
  for (uint32_t j = blockIdx.x; j < n; j += gridDim.x) {
    const uint64_t key = keys[longs[j]];
    const uint32_t u = (uint32_t)(key >> 32), v = (uint32_t)key;
    const uint32_t a = tc_walked(U, u, v), b = a == u ? v : u;
    const Table tb = group_table(U, b);
    for_each_slab_strided(U, a, threadIdx.x / kGroup, kGroupsPerBlock, [&](uint64_t x, bool data) {
      const uint32_t k = (uint32_t)x;
      if (data && valid_key(k) && k != b) c += lane_has(U, tb, k);
    });
  }
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if (lane64() == 0 && c) atomicAdd(S, 2ull * c);
}


// ---------------------------------------------------------------- hub edges through LDS sets
// A hub b (tc_is_hub, with its segment in the sorted batch keys) owns the batch edges {a, b}
// whose walked end is a.  Its work is split into items <b, pass p, chunk c>: pass p keeps the
// keys of N(b) whose partition hash is p (P_b passes, so that one pass fits the LDS set),
// chunk c is a run of entries of b's segment.  An item loads its part of N(b) into an LDS
// hash set, then reads the packed list of every partner a in its chunk (spread over the
// whole block) and looks each key of the pass up (S1); it also looks up, for the arcs
// (b, a), every entry of a's batch segment that falls in the pass (S2), and, with b's own
// batch segment in the set as tagged keys, counts S2 of the arcs (a, b) on the same lookups.
//
// The set is bucketized: 4 slots (16 bytes, one LDS read) per bucket, linear probing over
// buckets.  At the set's load factor a lookup mostly reads one bucket, so the lanes of a wave
// rarely wait for each other's probe chains (one slot per probe step cost about twice as
// much in the measurements).
//
// Two classes of hubs, one launch each: a small hub (at most HubClass<true>::kKeys
// neighbours) takes a 256-thread block with a 32 KiB set, four blocks to a CU, so that the
// latency of one item's dependent steps overlaps the others'; a large one takes a
// 1024-thread block with a 128 KiB set, one to a CU, in as many passes as it needs.
template <bool Small>
struct HubClass {
  static constexpr uint32_t kThreads = Small ? 256 : 1024;
  static constexpr uint32_t kSlots = Small ? 8192 : 32768;  // u32 keys of the LDS set
  static constexpr uint32_t kKeys = kSlots * 5 / 16;        // keys per pass (load <= 0.3125)
  static constexpr uint32_t kChunk = Small ? 128 : 512;     // segment entries per item
  static constexpr uint32_t kBlocks = Small ? 1024 : 512;   // persistent blocks
  static_assert(kChunk % 64 == 0 && kChunk <= kThreads && kThreads >= 128, "a wave scans a chunk");
};
constexpr uint32_t kTcHubRun = 8;  // list tasks a wave loads at once
__device__ inline bool tc_small_hub(const DView& U, uint32_t b) { return U.deg[b] <= HubClass<true>::kKeys; }

__device__ inline uint32_t tc_part(uint32_t k, uint32_t P) {
  return (uint32_t)(((uint64_t)(k * 0x85EBCA6Bu) * P) >> 32);
}
// Keys of b's batch segment share b's set, tagged with the top bit (vertex ids stay below
// 2^31 when the tag is in use); the bucket hash ignores that bit, so a key and its tagged
// copy share a home bucket and one probe sees both.
constexpr uint32_t kTcTag = 0x80000000u;
__device__ inline uint32_t tc_bucket(uint32_t k, uint32_t bmask) {
  return ((k & ~kTcTag) * 0x9E3779B1u) >> 9 & bmask;
}
template <bool Small>
__device__ inline uint32_t tc_hub_passes(uint32_t deg) {
  return max(1u, (deg + HubClass<Small>::kKeys - 1) / HubClass<Small>::kKeys);
}

// Insert `key` into the bucketized LDS set of bmask + 1 buckets; false when the set is full.
__device__ inline bool lds_insert(uint32_t* tab, uint32_t bmask, uint32_t key) {
  uint32_t h = tc_bucket(key, bmask);
  for (uint32_t n = 0; n <= bmask; ++n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t old = atomicCAS(&tab[4 * h + i], kInvalid, key);
      if (old == kInvalid || old == key) return true;
    }
    h = (h + 1) & bmask;
  }
  return false;
}
// Whether `key` is in the set, probing from bucket h on (its hash bucket, or a later one
// when the earlier ones are known full and without it).
__device__ inline bool lds_has_from(const uint32_t* tab, uint32_t bmask, uint32_t key, uint32_t h) {
  for (uint32_t n = 0; n <= bmask; ++n) {
    const uint4 q = reinterpret_cast<const uint4*>(tab)[h];
    if (q.x == key || q.y == key || q.z == key || q.w == key) return true;
    if (q.x == kInvalid || q.y == kInvalid || q.z == kInvalid || q.w == kInvalid) return false;
    h = (h + 1) & bmask;
  }
  return false;
}
__device__ inline bool lds_has(const uint32_t* tab, uint32_t bmask, uint32_t key) {
  return lds_has_from(tab, bmask, key, tc_bucket(key, bmask));
}
// Whether `key` (bit 0) and `tkey` (bit 1) are in the set, probing from bucket h on: both
// lie before the first bucket with an empty slot.
__device__ inline uint32_t lds_has2_from(const uint32_t* tab, uint32_t bmask, uint32_t key, uint32_t tkey,
                                         uint32_t h) {
  uint32_t f = 0;
  for (uint32_t n = 0; n <= bmask; ++n) {
    const uint4 q = reinterpret_cast<const uint4*>(tab)[h];
    if (q.x == key || q.y == key || q.z == key || q.w == key) f |= 1u;
    if (q.x == tkey || q.y == tkey || q.z == tkey || q.w == tkey) f |= 2u;
    if (q.x == kInvalid || q.y == kInvalid || q.z == kInvalid || q.w == kInvalid) break;
    h = (h + 1) & bmask;
  }
  return f;
}

// The last position i < n with off[i] <= t, for a non-decreasing off with off[0] <= t,
// searched by a whole wave at once: each round the 64 lanes test 64 evenly spaced
// positions, so a range of n entries takes ceil(log64 n) rounds of dependent loads instead
// of log2 n.  Every lane of the wave must call it; every lane gets the result.
__device__ inline uint64_t wave_last_le(const uint32_t* off, uint64_t n, uint32_t t) {
  const uint64_t lane = __lane_id();
  uint64_t lo = 0, end = n;
  while (end - lo > 1) {
    const uint64_t step = (end - lo + 63) / 64;
    const uint64_t i = lo + lane * step;
    const unsigned long long m = __ballot(i < end && off[i] <= t);  // a prefix of the lanes
    lo += (uint64_t)(63 - __clzll(m)) * step;
    end = min(end, lo + step);
  }
  return lo;
}

// Packed neighbour lists.  A partner's neighbourhood is read once per hub edge and pass, so
// the partners' keys are first copied out of their slabs into contiguous u32 lists: each
// later read is a coalesced 256-byte run instead of a chain of scattered 128-byte slabs
// that are 15/16 filled with 8-byte words.
//
// k_tc_need marks every vertex walked against a hub's set (the walked end of a batch edge
// whose other end is a hub), exactly the partners k_tc_hub reads.
__global__ void k_tc_need(DView U, const uint64_t* keys, uint64_t nk, const uint32_t* seg_lo,
                          const uint32_t* seg_hi, uint32_t nv, uint32_t* need) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nk;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t key = keys[i];
    const uint32_t b = (uint32_t)(key >> 32), a = (uint32_t)key;
    if (b >= nv) continue;  // sentinels
    if (tc_is_hub(U, b, keys, seg_lo[b], seg_hi[b]) && tc_walked(U, a, b) == a) need[a] = 1;
  }
}

constexpr uint32_t kPackBuckets = 256;  // buckets per packing item (one wave, 4 rounds of 64)

// Per vertex: its list length (the live degree when marked, else 0) and its packing items;
// the mark becomes the vertex's write cursor (0).
__global__ void k_tc_pack_count(DView U, uint32_t nv, uint32_t* need, uint32_t* dcnt, uint32_t* icnt) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const bool on = need[v] != 0 && U.deg[v] > 0;
    need[v] = 0;
    dcnt[v] = on ? U.deg[v] : 0u;
    icnt[v] = on ? (U.nbk[v] + kPackBuckets - 1) / kPackBuckets : 0u;
  }
}

// One wave per item <vertex a, buckets [q * kPackBuckets, ...)>: a lane walks one bucket
// chain, reading whole slabs; per round the wave reserves room for its valid keys (with one
// atomic on a's cursor when a has several items) and each lane writes its keys at its
// prefix (key order in a list is arbitrary).  Writes stay inside a's range
// [doff[a], doff[a] + deg(a)).
__global__ void __launch_bounds__(kBlock) k_tc_pack(DView U, uint32_t nv, const uint64_t* doff,
                                                    const uint32_t* icnt, const uint32_t* ioff,
                                                    uint32_t* cur, uint32_t* list) {
  if (nv == 0) return;
  const uint32_t total = ioff[nv - 1] + icnt[nv - 1];
  const uint32_t ln = threadIdx.x & 63;
  const uint32_t nw = gridDim.x * (blockDim.x / 64);
  for (uint32_t t = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; t < total; t += nw) {
    const uint32_t a = (uint32_t)wave_last_le(ioff, nv, t);  // ioff[a] <= t < ioff[a] + icnt[a]
    const uint32_t q = t - ioff[a], dv = U.deg[a];
    const uint64_t* hs = slab_ptr(U, a);
    const uint32_t nb = (uint32_t)(ld_word(hs + 15) >> 32);
    const uint32_t xb = nb > 1 ? (uint32_t)ld_word(hs + 14) : 0u;
    const uint32_t bend = min(nb, (q + 1) * kPackBuckets);
    uint32_t* out = list + doff[a];
    const bool single = icnt[a] == 1;  // one item: no other wave writes a's list
    uint32_t own = 0;
    for (uint32_t b0 = q * kPackBuckets; b0 < bend; b0 += 64) {
      const uint32_t bk = b0 + ln;
      uint32_t s = kInvalid;
      int nd = kKeysPerSlab;
      if (bk < bend) {
        s = bk == 0 ? a : xb + bk - 1;
        nd = (bk == 0 && nb > 1) ? kKeysPerSlab - 1 : kKeysPerSlab;
      }
      while (__ballot(s != kInvalid) != 0) {  // wave-uniform: every lane takes every round
        Slab sl;
        uint32_t n = 0;
        const bool act = s != kInvalid;
        if (act) {
          load_slab(U, s, sl);
#pragma unroll
          for (int i = 0; i < kKeysPerSlab; ++i) n += (i < nd && valid_key((uint32_t)sl.w[i])) ? 1u : 0u;
        }
        uint32_t incl = n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t y = __shfl_up(incl, o);
          if ((int)ln >= o) incl += y;
        }
        uint32_t base = 0;
        if (single) {  // the wave owns a's whole list
          base = own;
          own += __shfl(incl, 63);
        } else {
          if (ln == 63 && incl) base = atomicAdd(cur + a, incl);
          base = __shfl(base, 63);
        }
        base += incl - n;
        if (act) {
#pragma unroll
          for (int i = 0; i < kKeysPerSlab; ++i) {
            const uint32_t key = (uint32_t)sl.w[i];
            if (i < nd && valid_key(key)) {
              if (base < dv) out[base] = key;
              ++base;
            }
          }
          s = (uint32_t)sl.w[15];
          nd = kKeysPerSlab;
        }
      }
    }
  }
}

// Work items per segment start: P_b * ceil(|segment| / chunk) at the first key of a hub's
// segment when the hub is of the class, 0 elsewhere (an exclusive scan numbers the items).
template <bool Small>
__global__ void k_tc_hub_count(DView U, const uint64_t* keys, uint64_t nk, const uint32_t* seg_hi,
                               uint32_t nv, uint32_t* cnt) {
  using H = HubClass<Small>;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nk;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t b = (uint32_t)(keys[i] >> 32);
    uint32_t c = 0;
    if (b < nv && (i == 0 || (uint32_t)(keys[i - 1] >> 32) != b) && tc_is_hub(U, b, keys, (uint32_t)i, seg_hi[b]) &&
        tc_small_hub(U, b) == Small) {
      const uint64_t len = seg_hi[b] - i;
      c = tc_hub_passes<Small>(U.deg[b]) * (uint32_t)((len + H::kChunk - 1) / H::kChunk);
    }
    cnt[i] = c;
  }
}

// Persistent blocks take items from a counter until none is left.
template <bool Small>
__global__ void __launch_bounds__(HubClass<Small>::kThreads) k_tc_hub(DView U, const uint64_t* keys, uint64_t nk,
                                                         const uint32_t* seg_lo, const uint32_t* seg_hi,
                                                         const uint32_t* cnt,
                                                         const uint32_t* off, uint32_t* next,
                                                         const uint32_t* list, const uint64_t* loff,
                                                         bool s2in, unsigned long long* S) {
  using H = HubClass<Small>;
  __shared__ uint4 tab4[H::kSlots / 4];
  uint32_t* tab = reinterpret_cast<uint32_t*>(tab4);
  // per partner: its packed list (start, length) and its 64-key tasks, scanned into pre
  __shared__ uint64_t pbase[H::kChunk], qb[H::kChunk];
  __shared__ uint32_t plen[H::kChunk], ql[H::kChunk], qpre[H::kChunk + 1], nq_s;
  __shared__ uint32_t pslo[H::kChunk], pre2[H::kChunk + 1];  // partners' batch segments
  __shared__ uint32_t item_s[8];
  __shared__ uint32_t full;  // a key found no free slot: this item looks keys up in b's slabs
  __shared__ unsigned long long part[2][H::kThreads / 64];
  const uint32_t total = nk ? off[nk - 1] + cnt[nk - 1] : 0u;
  uint64_t hits = 0, h2 = 0;  // S1 and S2 matches
  while (true) {
    if (threadIdx.x < 64) {  // wave 0 fetches the next item
      uint32_t t = 0;
      if (threadIdx.x == 0) t = atomicAdd(next, 1u);
      t = __shfl(t, 0);
      // the segment start of item t: the last key position with off <= t
      const uint64_t lo = t < total ? wave_last_le(off, nk, t) : 0;
      if (threadIdx.x == 0) item_s[0] = t;
      if (threadIdx.x == 0 && t < total) {
        const uint32_t b = (uint32_t)(keys[lo] >> 32);
        const uint32_t P = tc_hub_passes<Small>(U.deg[b]);
        const uint32_t C = cnt[lo] / P;
        const uint32_t local = t - off[lo];
        const uint64_t c0 = lo + (uint64_t)(local % C) * H::kChunk;
        item_s[1] = b;
        item_s[2] = P;
        item_s[3] = local / C;
        item_s[4] = (uint32_t)c0;
        item_s[5] = (uint32_t)min<uint64_t>(c0 + H::kChunk, seg_hi[b]) - (uint32_t)c0;
      }
    }
    __syncthreads();
    if (item_s[0] >= total) break;  // every thread reads the same value
    // the item, wave-uniform: in scalar registers
    const uint32_t b = __builtin_amdgcn_readfirstlane(item_s[1]), P = __builtin_amdgcn_readfirstlane(item_s[2]);
    const uint32_t p = __builtin_amdgcn_readfirstlane(item_s[3]), c0 = __builtin_amdgcn_readfirstlane(item_s[4]);
    const uint32_t np = __builtin_amdgcn_readfirstlane(item_s[5]);
    // buckets: a power of two, at least 3.2 slots per key of the pass, within the LDS array (a
    // key's first bucket is then rarely full, and a probe rarely reads a second one)
    const uint32_t blo = seg_lo[b], bhi = seg_hi[b];  // b's batch segment: N_B(b)
    const uint32_t want = (U.deg[b] + P - 1) / P + (s2in ? (bhi - blo + P - 1) / P : 0u);
    uint32_t slots = 64;
    while (slots < H::kSlots && slots * 5 < want * 16) slots <<= 1;
    const uint32_t bmask = __builtin_amdgcn_readfirstlane(slots / 4 - 1);
    for (uint32_t i = threadIdx.x; i < slots; i += H::kThreads) tab[i] = kInvalid;
    if (threadIdx.x == 0) full = 0;
    // partners of this chunk: a is walked when tc_walked picks it over b
    for (uint32_t j = threadIdx.x; j < np; j += H::kThreads) {
      const uint32_t a = (uint32_t)keys[c0 + j];
      const uint32_t len = tc_walked(U, a, b) == a ? U.deg[a] : 0u;
      pbase[j] = len ? loff[a] : 0;
      plen[j] = len;
      pslo[j] = seg_lo[a];
      // S2 of the arc (b, a), over a's segment (its length, scanned below); not when a is a
      // hub that walks b against its own set: a's items count that arc with b's tagged keys
      const bool by_a = s2in && tc_walked(U, a, b) == b && tc_is_hub(U, a, keys, seg_lo[a], seg_hi[a]);
      pre2[j] = by_a ? 0u : seg_hi[a] - seg_lo[a];
    }
    if (threadIdx.x == 64) {  // b's bucket count and first extra head slab
      const uint64_t* ps = slab_ptr(U, b);
      const uint32_t nbb0 = (uint32_t)(ld_word(ps + 15) >> 32);
      item_s[6] = nbb0;
      item_s[7] = nbb0 > 1 ? (uint32_t)ld_word(ps + 14) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < 128) {
      // two scans, one wave each, a lane owning H::kChunk / 64 consecutive partners.
      // Wave 0 compacts the partners with a non-empty list, in order, into qb / ql with the
      // exclusive prefix of their 64-key tasks in qpre (qpre[nq] = all tasks); wave 1 turns
      // the partners' batch-segment lengths in pre2 into their exclusive prefix.
      constexpr uint32_t kPer = H::kChunk / 64;
      const uint32_t ln = threadIdx.x & 63;
      const bool w0 = threadIdx.x < 64;
      uint32_t v[kPer], sum = 0, nz = 0;
#pragma unroll
      for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t j = ln * kPer + k;
        v[k] = j >= np ? 0u : w0 ? (plen[j] + 63) / 64 : pre2[j];
        sum += v[k];
        nz += v[k] != 0;
      }
      uint32_t incl = sum, zincl = nz;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o), z = __shfl_up(zincl, o);
        if ((int)ln >= o) {
          incl += t;
          zincl += z;
        }
      }
      uint32_t acc = incl - sum, q = zincl - nz;
#pragma unroll
      for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t j = ln * kPer + k;
        if (w0) {
          if (v[k]) {
            qpre[q] = acc;
            qb[q] = pbase[j];
            ql[q] = plen[j];
            ++q;
          }
        } else if (j < np) {
          pre2[j] = acc;
        }
        acc += v[k];
      }
      if (ln == 63) {
        if (w0) {
          qpre[zincl] = incl;
          nq_s = zincl;
        } else {
          pre2[np] = incl;
        }
      }
    }
    // this pass's keys of N(b), one bucket chain per lane (each lane reads whole slabs, so a
    // wave keeps 64 slab reads in flight)
    const uint32_t nbb = item_s[6], xbb = item_s[7];
    for (uint32_t k = threadIdx.x; k < nbb; k += H::kThreads) {
      uint32_t s = k == 0 ? b : xbb + k - 1;
      int nd = (k == 0 && nbb > 1) ? kKeysPerSlab - 1 : kKeysPerSlab;
      while (true) {
        Slab sl;
        load_slab(U, s, sl);
#pragma unroll
        for (int i = 0; i < kKeysPerSlab; ++i) {
          const uint32_t key = (uint32_t)sl.w[i];
          if (i >= nd || !valid_key(key) || tc_part(key, P) != p) continue;
          if (!lds_insert(tab, bmask, key)) full = 1;
        }
        s = (uint32_t)sl.w[15];
        if (s == kInvalid) break;
        nd = kKeysPerSlab;
      }
    }
    if (s2in) {  // and this pass's keys of N_B(b), tagged
      for (uint32_t j = blo + threadIdx.x; j < bhi; j += H::kThreads) {
        const uint32_t x = (uint32_t)keys[j];
        if (tc_part(x, P) == p && !lds_insert(tab, bmask, x | kTcTag)) full = 1;
      }
    }
    __syncthreads();
    const bool in_lds = full == 0;
    const Table tb{b, nbb, xbb};
    // S2 of the arcs (b, a): N_B(a) of every partner a against this pass's keys of N(b), one
    // segment entry per lane
    const uint32_t tasks2 = pre2[np];
    for (uint32_t t = threadIdx.x; t < tasks2; t += H::kThreads) {
      uint32_t lo = 0, hi = np;  // the partner j with pre2[j] <= t < pre2[j + 1]
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pre2[mid] <= t) lo = mid;
        else hi = mid;
      }
      const uint32_t x = (uint32_t)keys[pslo[lo] + (t - pre2[lo])];
      if (x == b || tc_part(x, P) != p) continue;
      h2 += in_lds ? lds_has(tab, bmask, x) : lane_has(U, tb, x);
    }
    // the partners' packed lists against this pass's keys of N(b).  Wave w takes a run of
    // consecutive 64-key tasks, kTcHubRun at a time: the tasks' partners come from kTcHubRun
    // lookahead prefixes (a partner has at least one task), the keys from one coalesced load
    // per task, and each key's first bucket from one LDS read, all issued before any is used.
    // Everything that selects a task's partner is wave-uniform and kept in scalar registers
    // (readfirstlane), so the vector units only form addresses, hash and compare keys.
    const uint32_t nq = __builtin_amdgcn_readfirstlane(nq_s);
    const uint32_t tasks = __builtin_amdgcn_readfirstlane(qpre[nq]);
    const uint32_t per = (tasks + H::kThreads / 64 - 1) / (H::kThreads / 64);
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t tb0 = min(tasks, wv * per), te = min(tasks, tb0 + per);
    const uint32_t lane = threadIdx.x & 63;
    uint32_t j = 0;  // the partner of task tb0: the last j with qpre[j] <= tb0
    if (tb0 < te) {
      uint32_t hi = nq;
      while (hi - j > 1) {
        const uint32_t mid = (j + hi) >> 1;
        if (__builtin_amdgcn_readfirstlane(qpre[mid]) <= tb0) j = mid;
        else hi = mid;
      }
    }
    // a run's partners are j .. j + kTcHubRun - 1: their prefixes, lengths and list starts are
    // read at once, and each task selects its own by the count of prefixes at or below it
    auto runs = [&](auto&& probe) {
      for (uint32_t t0 = tb0; t0 < te; t0 += kTcHubRun) {
        uint32_t nx[kTcHubRun], ln_[kTcHubRun], blo[kTcHubRun], bhi[kTcHubRun];
#pragma unroll
        for (uint32_t k = 0; k < kTcHubRun; ++k) {
          nx[k] = __builtin_amdgcn_readfirstlane(qpre[min(j + 1 + k, nq)]);
          ln_[k] = __builtin_amdgcn_readfirstlane(ql[min(j + k, nq - 1)]);
          const uint64_t bq = qb[min(j + k, nq - 1)];
          blo[k] = __builtin_amdgcn_readfirstlane((uint32_t)bq);
          bhi[k] = __builtin_amdgcn_readfirstlane((uint32_t)(bq >> 32));
        }
        const uint32_t pj = __builtin_amdgcn_readfirstlane(qpre[j]);
        uint32_t key[kTcHubRun];
#pragma unroll
        for (uint32_t r = 0; r < kTcHubRun; ++r) {
          const uint32_t t = t0 + r;  // its partner is j + c, c <= r (a partner has >= 1 task)
          uint32_t start = pj, len = ln_[0], lo = blo[0], hi = bhi[0];
#pragma unroll
          for (uint32_t k = 0; k + 1 < kTcHubRun; ++k)
            if (nx[k] <= t) {
              start = nx[k];
              len = ln_[k + 1];
              lo = blo[k + 1];
              hi = bhi[k + 1];
            }
          const uint32_t pos = (t - start) * 64 + lane;
          const uint32_t* src = list + (((uint64_t)hi << 32) | lo);
          key[r] = t < te && pos < len ? src[pos] : kInvalid;
        }
        uint32_t cn = 0;  // the partner of the next run's first task, t0 + kTcHubRun: j + cn
#pragma unroll
        for (uint32_t k = 0; k < kTcHubRun; ++k) cn += nx[k] <= t0 + kTcHubRun;
        j = min(j + cn, nq - 1);
        const uint64_t f = probe(key);  // S1 matches, and S2 matches << 32
        hits += (uint32_t)f;
        h2 += f >> 32;
      }
    };
    // keys of this pass: all of them when b takes one pass
    auto wanted = [&](uint32_t x) { return x != kInvalid && x != b && (P == 1 || tc_part(x, P) == p); };
    // With s2in, a key x of N(a) found tagged counts S2 of the arc (a, b): x in N_B(b).
    if (in_lds) {
      runs([&](const uint32_t (&key)[kTcHubRun]) -> uint64_t {
        uint32_t h[kTcHubRun];
        uint4 q4[kTcHubRun];
#pragma unroll
        for (uint32_t r = 0; r < kTcHubRun; ++r) {  // every first bucket, before any is tested
          h[r] = tc_bucket(key[r], bmask);
          q4[r] = tab4[h[r]];
        }
        uint32_t n = 0, n2 = 0, pend = 0, got = 0;
#pragma unroll
        for (uint32_t r = 0; r < kTcHubRun; ++r) {
          const uint32_t x = key[r], tx = s2in ? x | kTcTag : kInvalid;
          if (!wanted(x)) continue;
          const bool f1 = q4[r].x == x || q4[r].y == x || q4[r].z == x || q4[r].w == x;
          const bool f2 = s2in && (q4[r].x == tx || q4[r].y == tx || q4[r].z == tx || q4[r].w == tx);
          n += f1;
          n2 += f2;
          got |= (f1 ? 1u : 0u) << (2 * r) | (f2 ? 2u : 0u) << (2 * r);
          const bool fullb = q4[r].x != kInvalid && q4[r].y != kInvalid && q4[r].z != kInvalid && q4[r].w != kInvalid;
          if (fullb && (!f1 || (s2in && !f2))) pend |= 1u << r;  // a full first bucket
        }
        while (pend) {  // keys whose first bucket was full, all runs of the wave at once
          const uint32_t r = __builtin_ctz(pend);
          pend &= pend - 1;
          uint32_t x = key[0], hh = h[0];
#pragma unroll
          for (uint32_t k = 1; k < kTcHubRun; ++k)
            if (k == r) {
              x = key[k];
              hh = h[k];
            }
          const uint32_t f = lds_has2_from(tab, bmask, x, s2in ? x | kTcTag : kInvalid, (hh + 1) & bmask) &
                             ~(got >> (2 * r));
          n += f & 1u;
          n2 += s2in ? (f >> 1) & 1u : 0u;
        }
        return ((uint64_t)n2 << 32) | n;
      });
    } else {  // the pass overflowed its set: look the keys up in b's slabs and b's segment
      runs([&](const uint32_t (&key)[kTcHubRun]) -> uint64_t {
        uint32_t n = 0, n2 = 0;
#pragma unroll 1
        for (uint32_t r = 0; r < kTcHubRun; ++r) {
          if (!wanted(key[r])) continue;
          n += lane_has(U, tb, key[r]);
          if (s2in) {
            const uint64_t want_k = ((uint64_t)b << 32) | key[r];
            const uint64_t q = lower_bound_u64(keys + blo, bhi - blo, want_k);
            n2 += q < bhi - blo && keys[blo + q] == want_k;
          }
        }
        return ((uint64_t)n2 << 32) | n;
      });
    }
    __syncthreads();  // the set and partner arrays are rebuilt by the next item
  }
  // an S1 match counts twice (S1 adds both directions of an edge)
  uint64_t hs[2] = {2 * hits, h2};
  for (int k = 0; k < 2; ++k) {
    for (int o = 32; o > 0; o >>= 1) hs[k] += __shfl_xor(hs[k], o);
    if ((threadIdx.x & 63) == 0) part[k][threadIdx.x >> 6] = hs[k];
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long t = 0;
    for (uint32_t i = 0; i < H::kThreads / 64; ++i) t += part[threadIdx.x][i];
    if (t) atomicAdd(S + threadIdx.x, t);
  }
}

// ---------------------------------------------------------------- static count
// Every undirected edge is directed from its lower (degree, id) end to its higher one; A(u) are
// the out-neighbours of u in that orientation (at most sqrt(2 m) of them, however large the
// degree).  A triangle is counted once, at its lowest vertex u: for every v in A(u), the keys
// of A(v) that lie in A(u).  k_tc_orient copies the A(u) out of the slabs into packed lists;
// the counting kernels hold A(u) in an LDS hash set and stream the lists of its members, 64
// keys to a wave, one bucket read per key.
//
// What bounds it: the streamed keys, sum over directed edges of |A(v)| (660M at R-MAT scale 18),
// which the LDS reads (16 bytes per key) and the vector compares handle at about the rate the
// caches deliver them.  Walking slabs and probing the other end's slab table, a 128-byte read
// per key, took 39.5 ms at scale 18 and 1.35 to 1.56 s at scale 22; this takes 1.7 and 59 ms.
//
// A count of a small graph is its launches (the random graph of 4,096 vertices of degree 8: 84 us with
// ten of them, 65 with five), so the first kernel makes room for the lists and collects the large
// vertices, and the second puts the vertices into their classes.

// A list segment of its degree for every vertex (in no order), and the vertices of more than kHeavyBuckets
// buckets.  The next kernels' counters are zeroed here; tc_alloc and n_heavy_tc, which this kernel
// counts in, by k_tc_finish.
constexpr uint32_t kTcRoom = 4;  // vertices a thread
__global__ void __launch_bounds__(kBlock) k_tc_room(DView U, uint32_t nv, uint64_t* off, uint32_t* heavy, Counters* C) {
  __shared__ Stage S[1];
  __shared__ uint64_t first[kBlock / 64 + 1];
  stage_open(S[0], heavy, &C->n_heavy_tc);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    C->u64tmp[0] = 0;
    C->tc_class[0] = C->tc_class[1] = C->tc_class[2] = 0;
  }
  const uint32_t w = threadIdx.x >> 6, ln = threadIdx.x & 63;
  for (uint32_t base = blockIdx.x * kBlock * kTcRoom; base < nv; base += gridDim.x * kBlock * kTcRoom) {
    uint32_t d[kTcRoom];
    uint64_t sum = 0;
    __syncthreads();  // the stage is open; first[] has been read
#pragma unroll
    for (uint32_t k = 0; k < kTcRoom; ++k) {
      const uint32_t v = base + k * kBlock + threadIdx.x;
      d[k] = v < nv ? U.deg[v] : 0u;
      sum += d[k];
      stage_push(S[0], v < nv && U.nbk[v] > kHeavyBuckets, v);
    }
    uint64_t incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t below = ((uint64_t)__shfl_up((uint32_t)(incl >> 32), o) << 32) | __shfl_up((uint32_t)incl, o);
      if ((int)ln >= o) incl += below;
    }
    if (ln == 63) first[w] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint64_t total = 0;
      for (uint32_t i = 0; i < kBlock / 64; ++i) {
        const uint64_t x = first[i];
        first[i] = total;
        total += x;
      }
      const uint64_t at = total ? atomicAdd(&C->tc_alloc, (unsigned long long)total) : 0u;
      for (uint32_t i = 0; i < kBlock / 64; ++i) first[i] += at;
    }
    __syncthreads();
    uint64_t o = first[w] + incl - sum;
#pragma unroll
    for (uint32_t k = 0; k < kTcRoom; ++k) {
      const uint32_t v = base + k * kBlock + threadIdx.x;
      if (v < nv) off[v] = o;
      o += d[k];
    }
  }
  stage_close(S);
}

// Classes of vertices by |A(u)| (a vertex with fewer than two out-neighbours closes no
// triangle): a wave, a 256-thread block or a 1024-thread block to a vertex, with LDS sets that
// keep the classes at full occupancy; only the last needs several passes for the largest sets.
// A set has at least 3.2 slots per key, so that a key's first bucket is rarely full.
constexpr uint32_t kTcWaveKeys = 64, kTcWaveSlots = 256;
template <bool Mid>
struct CountClass {
  static constexpr uint32_t kThreads = Mid ? 256 : 1024;
  static constexpr uint32_t kSlots = Mid ? 2048 : 16384;
  static constexpr uint32_t kKeys = kSlots * 5 / 16;
  static constexpr uint32_t kBlocks = Mid ? 2048 : 512;
};

// The vertices of each class (q[0] wave, q[1] small block, q[2] large block) and their numbers.
struct TcClasses {
  uint32_t *q[3], *n;
};

__global__ void __launch_bounds__(kBlock) k_tc_orient(DView U, uint32_t nv, const uint32_t* heavy, const uint32_t* nheavy,
                                                      const uint64_t* off, uint32_t* list, uint32_t* dplus, TcClasses cls) {
  __shared__ Stage S[3];
  __shared__ uint32_t cur;
  const uint32_t ln = threadIdx.x & 63;
  for (int k = 0; k < 3; ++k) stage_open(S[k], cls.q[k], cls.n + k);
  __syncthreads();
  // |A(u)| = d, by one lane of those that found it
  auto store = [&](bool mine, uint32_t u, uint32_t d) {
    if (mine) dplus[u] = d;
    stage_push(S[0], mine && d >= 2 && d <= kTcWaveKeys, u);
    stage_push(S[1], mine && d > kTcWaveKeys && d <= CountClass<true>::kKeys, u);
    stage_push(S[2], mine && d > CountClass<true>::kKeys, u);
  };
  // u's out-neighbours among the words of one slab: bit j for word j
  auto higher = [&](uint32_t u, uint32_t du, const Slab& sl, int nd) -> uint32_t {
    const uint32_t live = live_words(sl, nd);
    uint32_t dv[kKeysPerSlab], keep = 0;
    load_of_keys<uint32_t>(U.deg, sl, live, 0u, dv);
#pragma unroll
    for (int j = 0; j < kKeysPerSlab; ++j)
      if (dv[j] > du || (dv[j] == du && (uint32_t)sl.w[j] > u)) keep |= 1u << j;
    return keep & live;  // a word without a key passes the test when u has lost all its arcs (du == 0)
  };
  // vertices of more than kHeavyBuckets buckets first (the longest): a block each, a lane per chain
  const uint32_t nh = *nheavy;
  for (uint32_t i = blockIdx.x; i < nh; i += gridDim.x) {
    const uint32_t u = heavy[i], du = U.deg[u];
    __syncthreads();
    if (threadIdx.x == 0) cur = 0;
    __syncthreads();
    const uint32_t nb = (uint32_t)(ld_word(slab_ptr(U, u) + 15) >> 32), xb = (uint32_t)ld_word(slab_ptr(U, u) + 14);
    uint32_t* out = list + off[u];
    for (uint32_t b0 = 0; b0 < nb; b0 += kBlock) {
      const uint32_t b = b0 + threadIdx.x;
      uint32_t s = b >= nb ? kInvalid : b ? xb + b - 1 : u;
      int nd = b ? kKeysPerSlab : kKeysPerSlab - 1;
      while (__ballot(s != kInvalid) != 0) {  // wave-uniform
        Slab sl;
        uint32_t keep = 0;
        if (s != kInvalid) {
          load_slab(U, s, sl);
          keep = higher(u, du, sl, nd);
          s = (uint32_t)sl.w[15];
          nd = kKeysPerSlab;
        }
        const uint32_t n = (uint32_t)__popc(keep);
        uint32_t excl = 0, total = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint64_t m = __ballot((n >> k) & 1u);
          excl += lanes_below(m) << k;
          total += (uint32_t)__popcll(m) << k;
        }
        uint32_t base = 0;
        if (ln == 0 && total) base = atomicAdd(&cur, total);
        base = __shfl(base, 0) + excl;
#pragma unroll
        for (int j = 0; j < kKeysPerSlab; ++j)
          if (keep >> j & 1) out[base++] = (uint32_t)sl.w[j];
      }
    }
    __syncthreads();
    store(threadIdx.x == 0, u, cur);
  }
  // single-bucket vertices: a lane each
  for (uint32_t u = blockIdx.x * kBlock + threadIdx.x; u < nv; u += gridDim.x * kBlock) {
    if (U.nbk[u] != 1) continue;
    const uint32_t du = U.deg[u];
    uint32_t n = 0;
    if (du) {
      uint32_t* out = list + off[u];
      Slab sl;
      uint32_t s = u;
      while (true) {
        load_slab(U, s, sl);
        const uint32_t keep = higher(u, du, sl, kKeysPerSlab);
#pragma unroll
        for (int j = 0; j < kKeysPerSlab; ++j)
          if (keep >> j & 1) out[n++] = (uint32_t)sl.w[j];
        s = (uint32_t)sl.w[15];
        if (s == kInvalid) break;
      }
    }
    store(true, u, n);
  }
  // 2 .. kHeavyBuckets buckets: a 16-lane group each
  const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  for (uint32_t u = g0; u < nv; u += ng) {
    const uint32_t nb = U.nbk[u];
    if (nb == 1 || nb > kHeavyBuckets) continue;
    const uint32_t du = U.deg[u];
    uint32_t* out = list + off[u];
    uint32_t n = 0;  // the same in every lane of the group
    for_each_slab(U, u, [&](uint64_t x, bool data) {
      const uint32_t v = (uint32_t)x;
      bool keep = false;
      if (data && valid_key(v)) {
        const uint32_t dv = U.deg[v];
        keep = dv > du || (dv == du && v > u);
      }
      const uint32_t m = gballot(keep);
      if (keep) out[n + __popc(m & ((1u << glane()) - 1u))] = v;
      n += __popc(m);
    });
    store(glane() == 0, u, n);
  }
  stage_close(S);
}

// The keys of up to 64 packed lists (lane i of the wave holds the start and the length of list i)
// that lie in the LDS set.  kTcLists lists are read side by side, with loads whose indexes are
// clamped into the list instead of masked, so that a wave has that many loads and then bucket
// reads in flight; keys whose first bucket is full are probed further afterwards, together.
// (8 in the block classes, 4 in the wave class, whose short sets make a longer round waste slots.)
template <uint32_t kTcLists>
__device__ inline uint32_t tc_stream(const uint32_t* __restrict__ list, uint64_t poff, uint32_t plen, uint32_t np,
                                     const uint4* tab4, uint32_t bmask) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t* tab = reinterpret_cast<const uint32_t*>(tab4);
  uint32_t hits = 0;
  for (uint32_t j = 0; j < np; j += kTcLists) {
    const uint32_t* src[kTcLists];
    uint32_t len[kTcLists], most = 0;
#pragma unroll
    for (uint32_t k = 0; k < kTcLists; ++k) {
      const int from = (int)min(j + k, np - 1);
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)poff, from);
      const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(poff >> 32), from);
      src[k] = list + (((uint64_t)hi << 32) | lo);
      len[k] = j + k < np ? __builtin_amdgcn_readlane(plen, from) : 0u;
      most = max(most, len[k]);
    }
    for (uint32_t c = 0; c < most; c += 64) {
      uint32_t x[kTcLists], h[kTcLists];
      // an empty list's vertex still has a degree, so its segment has a first entry to read
#pragma unroll
      for (uint32_t k = 0; k < kTcLists; ++k) x[k] = src[k][min(c + lane, max(len[k], 1u) - 1u)];
      uint32_t pend = 0;
#pragma unroll
      for (uint32_t k0 = 0; k0 < kTcLists; k0 += 4) {  // four bucket reads at a time (registers)
        uint4 q[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
          h[k0 + i] = tc_bucket(x[k0 + i], bmask);
          q[i] = tab4[h[k0 + i]];
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
          const uint32_t k = k0 + i, y = x[k];
          const bool in = c + lane < len[k];
          const bool hit = (q[i].x == y) | (q[i].y == y) | (q[i].z == y) | (q[i].w == y);
          // slots of a bucket fill in order, so a bucket is full when its last slot is taken
          hits += in & hit;
          pend |= (uint32_t)(in & !hit & (q[i].w != kInvalid)) << k;
        }
      }
      while (pend) {
        const uint32_t k = __builtin_ctz(pend);
        pend &= pend - 1;
        uint32_t y = x[0], hh = h[0];
#pragma unroll
        for (uint32_t i = 1; i < kTcLists; ++i)
          if (i == k) {
            y = x[i];
            hh = h[i];
          }
        hits += lds_has_from(tab, bmask, y, (hh + 1) & bmask);
      }
    }
  }
  return hits;
}

__device__ inline void tc_total(uint64_t local, unsigned long long* acc) {
  for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
  if ((threadIdx.x & 63) == 0 && local) atomicAdd(acc, (unsigned long long)local);
}

// Where every vertex has a few neighbours in one or two buckets, lists and sets do not pay: a group
// per vertex walks its table and, for every edge to a higher vertex, probes that vertex's table with
// its neighbours (each triangle is met at its three edges).  Three launches, by lists in six / so, us:
// grids of side 64: 69 / 26, 256: 75 / 41, 1,024: 387 / 317, 2,048: 1,905 / 1,377; the random graph of 500
// vertices of degree 8, whose vertices have up to three buckets: 58 / 64.
__global__ void __launch_bounds__(kBlock) k_tc_few(DView U, uint32_t nv, unsigned long long* acc) {
  uint64_t local = 0;
  const uint32_t ng = gridDim.x * kGroupsPerBlock;
  for (uint32_t u = (blockIdx.x * kBlock + threadIdx.x) / kGroup; u < nv; u += ng) {
    const uint32_t du = U.deg[u];
    if (du < 2) continue;
    for_each_slab(U, u, [&](uint64_t x, bool data) {
      const uint32_t v = (uint32_t)x;
      bool higher = false;
      if (data && valid_key(v)) {
        const uint32_t dv = U.deg[v];
        higher = dv > du || (dv == du && v > u);
      }
      for (uint32_t todo = gballot(higher); todo; todo &= todo - 1) {
        const uint64_t c = group_intersect(U, u, gbcast(v, __builtin_ctz(todo)));
        if (glane() == 0) local += c;
      }
    });
  }
  tc_total(local, acc);
}

__global__ void __launch_bounds__(kBlock) k_tc_count_wave(const uint32_t* __restrict__ list, const uint64_t* __restrict__ off,
                                                          const uint32_t* __restrict__ dplus, const uint32_t* q,
                                                          const uint32_t* nq, unsigned long long* acc) {
  __shared__ uint4 tabs[kBlock / 64][kTcWaveSlots / 4];
  static_assert(kTcWaveSlots / 4 == 64 && kTcWaveKeys == 64, "a lane clears a bucket and holds a key");
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63, n = *nq;
  uint4* tab4 = tabs[w];
  constexpr uint32_t bmask = kTcWaveSlots / 4 - 1;
  uint64_t local = 0;
  for (uint32_t i = blockIdx.x * (kBlock / 64) + w; i < n; i += gridDim.x * (kBlock / 64)) {
    const uint32_t u = q[i], d = __builtin_amdgcn_readfirstlane(dplus[u]);
    tab4[lane] = make_uint4(kInvalid, kInvalid, kInvalid, kInvalid);
    const uint32_t key = lane < d ? list[off[u] + lane] : kInvalid;
    const uint32_t plen = lane < d ? dplus[key] : 0u;
    const uint64_t poff = lane < d ? off[key] : 0u;
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    if (lane < d) lds_insert(reinterpret_cast<uint32_t*>(tab4), bmask, key);  // at most 64 keys in 256 slots
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    local += tc_stream<4>(list, poff, plen, d, tab4, bmask);
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
  }
  tc_total(local, acc);
}

template <bool Mid>
__global__ void __launch_bounds__(CountClass<Mid>::kThreads) k_tc_count_block(DView U, const uint32_t* __restrict__ list,
                                                                              const uint64_t* __restrict__ off,
                                                                              const uint32_t* __restrict__ dplus,
                                                                              const uint32_t* q, const uint32_t* nq,
                                                                              unsigned long long* acc) {
  using H = CountClass<Mid>;
  constexpr uint32_t kWaves = H::kThreads / 64;
  __shared__ uint4 tab4[H::kSlots / 4];
  __shared__ uint32_t full;  // a key found no free slot: this pass looks keys up in u's slabs
  uint32_t* tab = reinterpret_cast<uint32_t*>(tab4);
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = *nq;
  uint64_t local = 0;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t u = q[i], d = __builtin_amdgcn_readfirstlane(dplus[u]);
    const uint32_t* mine = list + off[u];
    // passes: pass p holds the keys whose partition hash is p, at most kKeys of them on average
    // (kSlots / kKeys = 3.2 leaves room for an uneven split)
    const uint32_t P = (d + H::kKeys - 1) / H::kKeys;
    uint32_t slots = 256;
    while (slots < H::kSlots && slots * 5 < (d + P - 1) / P * 16) slots <<= 1;
    const uint32_t bmask = slots / 4 - 1;
    for (uint32_t p = 0; p < P; ++p) {
      __syncthreads();  // the last set is no longer read
      for (uint32_t k = threadIdx.x; k < slots / 4; k += H::kThreads)
        tab4[k] = make_uint4(kInvalid, kInvalid, kInvalid, kInvalid);
      if (threadIdx.x == 0) full = 0;
      __syncthreads();
      for (uint32_t k = threadIdx.x; k < d; k += H::kThreads) {
        const uint32_t key = mine[k];
        if ((P == 1 || tc_part(key, P) == p) && !lds_insert(tab, bmask, key)) full = 1;
      }
      __syncthreads();
      if (full) {  // only an adversarial choice of ids splits this unevenly
        // a key of A(v) ranks above v and so above u: it lies in A(u) when it is u's neighbour
        const Table tu = group_table(U, u);
        for (uint32_t j = 0; j < d; ++j) {
          const uint32_t v = mine[j], len = dplus[v];
          for (uint32_t c = threadIdx.x; c < len; c += H::kThreads) {
            const uint32_t x = list[off[v] + c];
            if (tc_part(x, P) == p) local += lane_has(U, tu, x);
          }
        }
        continue;
      }
      // the lists of A(u)'s members, dealt to the waves in turn: wave w takes members w, w + kWaves ...
      for (uint32_t j0 = 0; j0 < d; j0 += H::kThreads) {
        const uint32_t j = j0 + lane * kWaves + w;
        uint32_t plen = 0;
        uint64_t poff = 0;
        if (j < d) {
          const uint32_t key = mine[j];
          plen = dplus[key];
          poff = off[key];
        }
        const uint32_t np = d - j0 > w ? min(64u, (d - j0 - w + kWaves - 1) / kWaves) : 0u;
        local += tc_stream<8>(list, poff, plen, np, tab4, bmask);
      }
    }
  }
  tc_total(local, acc);
}

__global__ void k_tc_begin(Counters* C) {
  if (threadIdx.x != 0) return;
  C->tc_s[0] = C->tc_s[1] = C->tc_s[2] = 0;
  C->tc_work = 0;
}

// insert: T += (S1 - S2 + S3/3) / 2;  delete: T -= (S1 + S2 + S3/3) / 2;  static: T = the sum
// (kind 4: a third of it), and k_tc_room's counters go back to zero for the next count
__global__ void k_tc_finish(Counters* C, int kind, unsigned long long* out) {
  if (threadIdx.x != 0) return;
  const unsigned long long s1 = C->tc_s[0], s2 = C->tc_s[1], s3 = C->tc_s[2];
  if (kind == 0) C->tc_total += (s1 - s2 + s3 / 3) / 2;
  else if (kind == 1) C->tc_total -= (s1 + s2 + s3 / 3) / 2;
  else if (kind == 2 || kind == 4) {
    C->tc_total = kind == 4 ? C->u64tmp[0] / 3 : C->u64tmp[0];
    C->tc_alloc = 0;
    C->n_heavy_tc = 0;
  }
  if (out) *out = C->tc_total;
}

Log log_at(const mk_graph* g, uint64_t off) {
  Log l = g->log;
  l.s += off;
  l.d += off;
  l.w += off;
  l.st += off;
  l.uf += off;
  return l;
}

// PageRank iterations under IterationScheme2 from the ranks in g->pr_x (the caller has
// initialized or kept them): contributions, one group per reverse-view bucket chain, then
// the per-vertex sums in bucket order.
mk_status pagerank_scheme2(mk_graph* g, float damping, double tol_l1, uint32_t max_iter, float* d_rank,
                           uint32_t* d_iters, hipStream_t stream) {
  const uint32_t N = g->n;
  if (mk_status st = ensure_pairs(g, VR, stream); st != MK_OK) return st;
  const ViewHost& vh = g->view[VR];
  hipLaunchKernelGGL(k_pr_start, dim3(1), dim3(64), 0, stream, g->ctr);
  float* buf[2] = {g->pr_x, g->pr_y};
  const uint32_t cb = blocks_for(N, kPrContribBlocks);
  double* dpart = g->pr_part + kPrContribBlocks;
  uint32_t it = 0;
  while (true) {
    for (int k = 0; k < kPrSyncEvery; ++k, ++it) {
      const int slot = it & 3;
      const float* x = buf[it & 1];
      float* y = buf[(it + 1) & 1];
      double* dang = &g->ctr->pr_acc[2 * slot];
      hipLaunchKernelGGL(k_pr_contrib, dim3(cb), dim3(kBlock), 0, stream, x, g->view[VF].d.deg, g->pr_c,
                         N, g->pr_part, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_sum, dim3(1), dim3(kBlock), 0, stream, g->pr_part, cb, dang, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_gather_s2, dim3(kWalkBlocks), dim3(kBlock), 0, stream, vh.d, g->pr_c,
                         vh.pair_v, vh.pair_i, (uint32_t)vh.n_head, N, g->pr_pair, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_final_s2, dim3(kWalkBlocks), dim3(kBlock), 0, stream, vh.nbk, vh.pair_off,
                         g->pr_pair, x, y, N, damping, dang, dpart, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_check, dim3(1), dim3(kBlock), 0, stream, g->ctr, slot, tol_l1, max_iter, dpart,
                         kWalkBlocks, nullptr, reinterpret_cast<uint32_t*>(g->h_pin));
      MK_LAUNCH(g, "pagerank iteration (scheme 2)");
    }
    MK_HIP(g, hipStreamSynchronize(stream));
    if (*(volatile uint32_t*)g->h_pin) break;
  }
  hipLaunchKernelGGL(k_pr_final, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->ctr, g->pr_x,
                     g->pr_y, g->pr_x, d_rank, N, d_iters);
  MK_LAUNCH(g, "pagerank final");
  g->pr.valid = true;
  mark_seen(g, g->pr);
  return MK_OK;
}

// PageRank by packed iterations from the ranks in g->pr_x.
mk_status pagerank_packed(mk_graph* g, float damping, double tol_l1, uint32_t max_iter, float* d_rank,
                          uint32_t* d_iters, hipStream_t stream) {
  const uint32_t N = g->n;
  const DView& R = g->view[VR].d;
  const uint32_t* outdeg = g->view[VF].d.deg;
  uint32_t *od = g->pr_skey[0], *id = g->pr_skey[1];  // the sort's keys are free after it
  float* x[2] = {reinterpret_cast<float*>(g->pr_cr), reinterpret_cast<float*>(g->pr_cr) + N};
  float* c[2] = {g->pr_c, g->pr_cp};
  uint32_t *cur = g->fq[0], *item_i = g->lv_multi[0], *item_c = g->lv_multi[1];  // traversal scratch
  uint32_t* nitems = &g->ctr->n_heavy_pr;
  if (N <= kPrHot) {
    hipLaunchKernelGGL(k_pr_identity, dim3(blocks_for(N)), dim3(kBlock), 0, stream, outdeg, R.deg, N, g->pr_perm, od,
                       id, g->pr_rank, cur, nitems);
  } else {
    hipLaunchKernelGGL(k_pr_class, dim3(blocks_for(N)), dim3(kBlock), 0, stream, outdeg, N, g->pr_skey[0], g->pr_sidx);
    size_t sb = g->pr_sort_bytes;
    if (rocprim::radix_sort_pairs(g->pr_sort_tmp, sb, g->pr_skey[0], g->pr_skey[1], g->pr_sidx, g->pr_perm,
                                  (size_t)N, 0, 6, stream) != hipSuccess)
      return MK_ERR_HIP;
    hipLaunchKernelGGL(k_pr_order, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->pr_perm, outdeg, R.deg, N, od, id,
                       g->pr_rank, cur, nitems);
  }
  size_t tb = g->scan_tmp_bytes;
  if (rocprim::exclusive_scan(g->scan_tmp, tb, id, g->pr_off, 0u, (size_t)N, rocprim::plus<uint32_t>(), stream) !=
      hipSuccess)
    return MK_ERR_HIP;
  hipLaunchKernelGGL(k_pr_start, dim3(1), dim3(64), 0, stream, g->ctr);
  hipLaunchKernelGGL(k_pr_tiles, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->pr_off, id, N, g->pr_fv, g->pr_perm,
                     R.nbk, item_i, item_c, nitems);
  hipLaunchKernelGGL(k_pr_pack, dim3(kWalkBlocks), dim3(kBlock), 0, stream, R, g->pr_perm, g->pr_rank, g->pr_off, N,
                     g->pr_list, cur, item_i, item_c, nitems);
  uint32_t* pin = reinterpret_cast<uint32_t*>(g->h_pin);
  PrIter a;
  a.off = g->pr_off;
  a.list = g->pr_list;
  a.fv = g->pr_fv;
  a.od = od;
  a.heads = g->pr_tile[0];
  a.tails = g->pr_tile[1];
  a.ddelta = g->pr_part;
  a.ddang = g->pr_part + kPrParts / 2;
  a.state = g->ctr->pr_state;
  a.nv = N;
  a.damping = damping;
  // The host does not know the in-arcs.  The arcs ever passed in bound them, and so do the words of all
  // slabs in use, with the chained ones: a graph created empty and filled by inserts has nearly all
  // its words there.  Both drift upwards over a stream of batches (the pool's figure counts a slab
  // per inserted arc until it is read back), so a graph of few vertices that they would send
  // to the launches below has its list's length read back first.
  const ViewHost& rv = g->view[VR];
  uint64_t tiles =
      (std::min((rv.n_head + rv.pool_used_est) * kKeysPerSlab, g->m0 + rv.added) + N) / kPrTile + 1;
  if (N <= kPrSmallN && tiles > kPrSmallTiles) {
    read_back(g->pr_off + N, pin, 1, stream);
    MK_LAUNCH(g, "pagerank tiles");
    MK_HIP(g, hipStreamSynchronize(stream));
    tiles = ((uint64_t)*(volatile uint32_t*)pin + N + kPrTile - 1) / kPrTile;
  }
  if (N <= kPrSmallN && tiles <= kPrSmallTiles) {
    hipLaunchKernelGGL(k_copy_f32, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->pr_x, x[0], N);
    a.x = x[0];
    // nothing is read back: the ranks are in stream order like any other call's (a wait here took 40 us
    // of the launches that follow out of its shadow)
    hipLaunchKernelGGL(k_pr_small, dim3(1), dim3(kPrFlatThreads), 0, stream, a, x[1], g->ctr, tol_l1, max_iter,
                       (uint32_t*)nullptr);
  } else {
    const uint32_t cb = blocks_for(N, kPrContribBlocks);
    hipLaunchKernelGGL(k_pr_load, dim3(cb), dim3(kBlock), 0, stream, g->pr_x, g->pr_perm, od, N, x[0], c[0], g->pr_part);
    hipLaunchKernelGGL(k_pr_sum, dim3(1), dim3(kBlock), 0, stream, g->pr_part, cb, &g->ctr->pr_acc[0], g->ctr->pr_state);
    MK_LAUNCH(g, "pagerank packing");
    uint32_t it = 0;
    while (true) {
      for (int k = 0; k < kPrSyncEvery; ++k, ++it) {
        const int slot = it & 3;
        a.c = c[it & 1];
        a.x = x[it & 1];
        a.cn = c[(it + 1) & 1];
        a.y = x[(it + 1) & 1];
        a.dang = &g->ctr->pr_acc[2 * slot];
        hipLaunchKernelGGL(k_pr_flat, dim3(kPrFlatBlocks), dim3(kPrFlatThreads), 0, stream, a);
        if (tiles <= kPrFixOne) {
          hipLaunchKernelGGL(k_pr_fix_check, dim3(1), dim3(1024), 0, stream, a, g->ctr, slot, tol_l1, max_iter, pin);
        } else {
          hipLaunchKernelGGL(k_pr_fix, dim3(kPrFixBlocks), dim3(kBlock), 0, stream, a);
          hipLaunchKernelGGL(k_pr_check, dim3(1), dim3(kBlock), 0, stream, g->ctr, slot, tol_l1, max_iter, a.ddelta,
                             kPrFlatBlocks + kPrFixBlocks, a.ddang, pin);
        }
        MK_LAUNCH(g, "pagerank iteration (packed)");
      }
      MK_HIP(g, hipStreamSynchronize(stream));
      if (*(volatile uint32_t*)pin) break;
    }
  }
  hipLaunchKernelGGL(k_pr_store, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->ctr, x[0], x[1], g->pr_rank, g->pr_x,
                     d_rank, N, d_iters);
  MK_LAUNCH(g, "pagerank final");
  g->pr.valid = true;
  mark_seen(g, g->pr);
  return MK_OK;
}

}  // namespace

extern "C" {

mk_status mk_incr_wcc(mk_graph* g, uint32_t* d_label, mk_mode mode, hipStream_t stream) {
  return mk_incr_wcc_scheme(g, d_label, mode, MK_WCC_LOG, stream);
}

mk_status mk_incr_wcc_scheme(mk_graph* g, uint32_t* d_label, mk_mode mode, mk_wcc_scheme scheme,
                             hipStream_t stream) {
  if (!g || !d_label || (uint32_t)scheme > (uint32_t)MK_WCC_UPDATE) return MK_ERR_INVALID_ARG;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  const uint32_t N = g->n;
  Pending p = pending_for(g, g->wcc);
  bool full = mode == MK_RECOMPUTE || !g->wcc.valid || p.lost || (p.kinds & 2);
  if (!full && mode == MK_AUTO)
    if (mk_status s = auto_prefers_recompute(g, MK_ALGO_WCC, p, stream, &full); s != MK_OK) return s;
  uint32_t* P = g->wcc_parent;
  const DView F = g->view[VF].d;
  auto all_arcs = [&]() -> mk_status {  // union over every arc
    if (g->iter_scheme == MK_ITER_SCHEME2) {  // one group per bucket chain
      if (mk_status st = ensure_pairs(g, VF, stream); st != MK_OK) return st;
      const ViewHost& vh = g->view[VF];
      hipLaunchKernelGGL(k_wcc_pairs, dim3(kWalkBlocks), dim3(kBlock), 0, stream, F, P, vh.pair_v, vh.pair_i,
                         (uint32_t)vh.n_head, N);
      return MK_OK;
    }
    // IterationScheme1, collecting the heavy vertices first
    uint32_t* nh = &g->ctr->n_heavy_wcc;
    const bool single = g->view[VF].n_head == N;
    if (!single) {
      hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, nh, 1u);
      hipLaunchKernelGGL(k_collect_heavy, dim3(blocks_for(N)), dim3(kBlock), 0, stream,
                         g->view[VF].nbk, N, g->fq[2], nh);
    }
    // A lane per vertex; where some have several buckets, at least 256 blocks for the groups and blocks
    // that take those (R-MAT scale 10, edge factor 4: 98 us with 4 blocks, 64 with 256).
    // In a recompute the unions of more lanes meet on few words, and the best number of blocks grows with
    // the root of the vertices, up to sizes that want all the chip holds.  A lane per vertex / so, us: grids,
    // no vertex of several buckets: side 256: 86 / 77, 512: 197 / 129, after inserts 300 / 137, 724: 315 /
    // 197, 1,024: 370 / 250, 2,048: 713 / 713 (side 512 with 64, 128, 256, 512 blocks: 250, 162, 129, 143;
    // 1,024 with 256, 512, 1,024: 318, 250, 290).  Others, medians: uniform, degree 4, 300,000 vertices: 830 /
    // 369, 2^20: 1,069 / 415; degree 10: 667 / 565, 2,289 / 951; R-MAT edge factor 4, scale 18: 608 / 397, 19:
    // 948 / 571, 20: 656 / 647; edge factor 16, scale 18: 720 / 582, 20: 1,908 / 1,772; scale 22 with 1,024
    // blocks takes 1,784 and 3,161, with a lane each 1,389 and 2,739.
    // An incremental pass finds nearly every arc united and only reads: all the blocks the chip holds
    // (scale 18, edge factor 8: 87 us, 108 with the lanes' 1,024).
    uint32_t blocks = blocks_for(N, 16384);
    if (full && N < (single ? kRootMost : kRootMostMixed))
      blocks = std::min(blocks, std::max(1u, (uint32_t)(std::sqrt((double)N) / 2)));
    if (!single) blocks = std::max(blocks, full ? 256u : kWalkBlocks);
    hipLaunchKernelGGL(k_wcc_all, dim3(blocks), dim3(kBlock), 0, stream, F, P, N, g->fq[2], nh, single);
    return MK_OK;
  };
  // the sampled static WCC: needs the undirected view (scratch: traversal queues)
  bool labelled = false;  // k_wcc_label has written the labels
  const dim3 all(blocks_for(N)), block(kBlock);
  auto sampled = [&]() {
    const DView U = g->view[VU].d;
    uint32_t *M = g->fq[0], *rest = g->fq[1], *heavy = g->fq[2];
    Counters* c = g->ctr;
    hipLaunchKernelGGL(k_wcc_hook, all, block, 0, stream, U, P, M, N);
    hipLaunchKernelGGL(k_wcc_link, all, block, 0, stream, U, P, N, false, &c->wcc_enough);
    for (int again = 0; again < 2; ++again) {
      if (again) hipLaunchKernelGGL(k_wcc_link, all, block, 0, stream, U, P, N, true, &c->wcc_enough);
      hipLaunchKernelGGL(k_wcc_big, dim3(1), dim3(kWccSamples), 0, stream, U, P, N, &c->wcc_big, &c->wcc_enough,
                         again != 0);
    }
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, &c->n_listed_light, 2u);
    hipLaunchKernelGGL(k_wcc_rest, all, block, 0, stream, U, P, N, &c->wcc_big, rest, &c->n_listed_light, heavy,
                       &c->n_listed_heavy);
    hipLaunchKernelGGL(k_wcc_walk, dim3(blocks_for(N, 2048)), block, 0, stream, U, P, rest, &c->n_listed_light, heavy,
                       &c->n_listed_heavy);
    hipLaunchKernelGGL(k_wcc_min, all, block, 0, stream, P, M, N, &c->wcc_big);
    hipLaunchKernelGGL(k_wcc_label, all, block, 0, stream, P, M, N, d_label);
    labelled = true;
  };
  // Where next to no vertex has many neighbours (at creation they fitted the primary slabs, and most arcs
  // are from creation: arcs that came and went again do not count), there is no largest component to find
  // early, and the unions meet on few words: hooks by id, jumps and the walk over the forward view do
  // better.  Sampled / so, us: grids of side 64: 81 / 36, 256: 92 / 76, 512: 150 / 127, 1,024: 515 / 260,
  // 2,048: 800 / 712, 4,096: 7,040 / 2,125.  A few chained slabs are let pass, not the chain of a hub, which
  // one lane would walk.
  const ViewHost& und = g->view[VU];
  const bool few = und.on && g->view[VF].n_head == N && und.n_head - N <= N / 512 && und.pool_built <= 64 &&
                   g->m0 >= N && g->net_added <= g->m0;
  if (full) {
    if (g->view[VU].on && !few && g->iter_scheme != MK_ITER_SCHEME2) {
      sampled();
    } else {
      const bool hook = g->view[VF].n_head == N || (N >= kHookLeast && N <= kHookMost);
      if (g->iter_scheme == MK_ITER_SCHEME2 || !hook) {
        hipLaunchKernelGGL(k_wcc_init, all, block, 0, stream, P, N);
      } else {
        hipLaunchKernelGGL(k_wcc_hook_min, all, block, 0, stream, F, P, N);
        for (int k = 0; k < kWccJumps; ++k) hipLaunchKernelGGL(k_wcc_jump, all, block, 0, stream, P, N);
      }
      if (mk_status st = all_arcs(); st != MK_OK) return st;
    }
    if (scheme == MK_WCC_UPDATE)
      hipLaunchKernelGGL(k_mark_all, dim3(grid_for_groups(std::min<uint64_t>(g->view[VF].n_head, 1u << 20))),
                         dim3(kBlock), 0, stream, F, g->upd_mark, g->view[VF].n_head, N);
  } else if (!p.list.empty()) {
    if (scheme == MK_WCC_LOG) {
      for (const BatchRec* b : p.list)
        hipLaunchKernelGGL(k_wcc_batch, dim3(blocks_for(b->n)), dim3(kBlock), 0, stream, P,
                           log_at(g, b->off), b->n);
    } else if (scheme == MK_WCC_NAIVE) {
      if (mk_status st = all_arcs(); st != MK_OK) return st;
    } else {
      uint32_t* nl = &g->ctr->n_listed_light;
      uint32_t* nh = &g->ctr->n_listed_heavy;
      hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, nl, 2u);
      uint64_t ops = 0;
      for (const BatchRec* b : p.list) {
        hipLaunchKernelGGL(k_wcc_flag, dim3(blocks_for(b->n)), dim3(kBlock), 0, stream,
                           log_at(g, b->off), b->n, g->view[VF].nbk, g->wcc_flag, g->fq[0], nl,
                           g->fq[1], nh);
        ops += b->n;
      }
      hipLaunchKernelGGL(k_wcc_listed, dim3(blocks_for(ops * kGroup)), dim3(kBlock), 0, stream, F, P,
                         scheme == MK_WCC_UPDATE ? g->upd_mark : nullptr, g->fq[0], nl, g->fq[1], nh);
      hipLaunchKernelGGL(k_wcc_unflag, dim3(blocks_for(ops)), dim3(kBlock), 0, stream, g->wcc_flag,
                         g->fq[0], nl, g->fq[1], nh);
    }
  }
  if (labelled) {
  } else if (full || !p.list.empty())
    hipLaunchKernelGGL(k_wcc_compress, dim3(blocks_for(N)), dim3(kBlock), 0, stream, P, N, d_label);
  else  // nothing changed: the parents are the compressed labels of the last call
    hipLaunchKernelGGL(k_copy_u32, dim3(blocks_for(N)), dim3(kBlock), 0, stream, P, d_label, N);
  MK_LAUNCH(g, "wcc");
  g->wcc.valid = true;
  mark_seen(g, g->wcc);
  return MK_OK;
}

mk_status mk_incr_pagerank(mk_graph* g, float damping, double tol_l1, uint32_t max_iter,
                           float* d_rank, uint32_t* d_iters, mk_mode mode, hipStream_t stream) {
  if (!g || !d_rank || !(damping >= 0.f && damping < 1.f) || max_iter == 0) return MK_ERR_INVALID_ARG;
  if (!g->view[VR].on) return MK_ERR_STATE;
  const uint32_t N = g->n;
  Pending p = pending_for(g, g->pr);
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  bool warm = mode != MK_RECOMPUTE && g->pr.valid && !p.lost;
  if (warm && mode == MK_AUTO) {
    bool rec = false;
    if (mk_status s = auto_prefers_recompute(g, MK_ALGO_PAGERANK, p, stream, &rec); s != MK_OK) return s;
    warm = !rec;
  }
  if (warm && p.list.empty()) {
    hipLaunchKernelGGL(k_pr_start, dim3(1), dim3(64), 0, stream, g->ctr);
    hipLaunchKernelGGL(k_pr_final, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->ctr, g->pr_x,
                       g->pr_y, g->pr_x, d_rank, N, d_iters);
    MK_LAUNCH(g, "pagerank copy");
    return MK_OK;
  }
  // The iterations' number is not known beforehand: the loops wait for convergence, which a capturing
  // stream cannot, and the sizes that choose between them are read now, not at a replay.
  if (stream_capturing(stream)) return hip_fail(g, hipErrorStreamCaptureUnsupported, "mk_incr_pagerank");
  if (!warm)
    hipLaunchKernelGGL(k_pr_fill, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->pr_x, N, 1.f / N);
  if (g->iter_scheme == MK_ITER_SCHEME2) return pagerank_scheme2(g, damping, tol_l1, max_iter, d_rank, d_iters, stream);
  if (g->iter_scheme == MK_ITER_PACKED) return pagerank_packed(g, damping, tol_l1, max_iter, d_rank, d_iters, stream);
  uint32_t* nh = &g->ctr->n_heavy_pr;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, nh, 1u);
  hipLaunchKernelGGL(k_collect_heavy, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->view[VR].nbk,
                     N, g->heavy_rev, nh);
  // heavy-vertex work items: counts, exclusive offsets, FP64 partial sums (scratch: the
  // traversal queues, which PageRank does not use)
  uint32_t* hcnt = g->fq[0];
  uint32_t* hoff = g->fq[1];
  double* hacc = g->pr_hacc;
  hipLaunchKernelGGL(k_heavy_items, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->view[VR].nbk,
                     g->heavy_rev, nh, hcnt, hacc);
  {
    size_t tb = g->scan_tmp_bytes;
    if (rocprim::exclusive_scan(g->scan_tmp, tb, hcnt, hoff, 0u, (size_t)N, rocprim::plus<uint32_t>(),
                                stream) != hipSuccess)
      return MK_ERR_HIP;
  }
  const DView& Rd = g->view[VR].d;
  hipLaunchKernelGGL(k_pr_start, dim3(1), dim3(64), 0, stream, g->ctr);
  MK_LAUNCH(g, "pagerank setup");
  float* buf[2] = {g->pr_x, g->pr_y};
  // per-block partial sums: the dangling mass (contribution blocks), then the L1 change
  // (gather blocks, heavy-final blocks)
  const uint32_t cb = blocks_for(N, kPrContribBlocks), hb = blocks_for(N, kPrFinalBlocks);
  double* dpart = g->pr_part + kPrContribBlocks;
  uint32_t it = 0;
  while (true) {
    for (int k = 0; k < kPrSyncEvery; ++k, ++it) {
      const int slot = it & 3;
      const float* x = buf[it & 1];
      float* y = buf[(it + 1) & 1];
      double* dang = &g->ctr->pr_acc[2 * slot];
      hipLaunchKernelGGL(k_pr_contrib, dim3(cb), dim3(kBlock), 0, stream, x, g->view[VF].d.deg, g->pr_c, N,
                         g->pr_part, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_sum, dim3(1), dim3(kBlock), 0, stream, g->pr_part, cb, dang, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_gather, dim3(kWalkBlocks), dim3(kBlock), 0, stream, Rd, g->pr_c, x, y, N, damping, dang,
                         dpart, g->heavy_rev, nh, hcnt, hoff, hacc, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_heavy_final, dim3(hb), dim3(kBlock), 0, stream, g->heavy_rev, nh, hacc, x, y,
                         N, damping, dang, dpart + kWalkBlocks, g->ctr->pr_state);
      hipLaunchKernelGGL(k_pr_check, dim3(1), dim3(kBlock), 0, stream, g->ctr, slot, tol_l1, max_iter, dpart,
                         kWalkBlocks + hb, nullptr, reinterpret_cast<uint32_t*>(g->h_pin));
      MK_LAUNCH(g, "pagerank iteration");
    }
    MK_HIP(g, hipStreamSynchronize(stream));
    if (*(volatile uint32_t*)g->h_pin) break;
  }
  hipLaunchKernelGGL(k_pr_final, dim3(blocks_for(N)), dim3(kBlock), 0, stream, g->ctr, g->pr_x,
                     g->pr_y, g->pr_x, d_rank, N, d_iters);
  MK_LAUNCH(g, "pagerank final");
  g->pr.valid = true;
  mark_seen(g, g->pr);
  return MK_OK;
}

mk_status mk_count_triangles(mk_graph* g, uint64_t* d_count, mk_mode mode, hipStream_t stream) {
  if (!g || !d_count) return MK_ERR_INVALID_ARG;
  if (!g->view[VU].on) return MK_ERR_STATE;
  const uint32_t N = g->n;
  const DView U = g->view[VU].d;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  Pending p = pending_for(g, g->tc);
  bool full = mode == MK_RECOMPUTE || !g->tc.valid || p.lost || p.kinds == 3;
  if (!full && mode == MK_AUTO)
    if (mk_status s = auto_prefers_recompute(g, MK_ALGO_TC, p, stream, &full); s != MK_OK) return s;
  unsigned long long* out = reinterpret_cast<unsigned long long*>(d_count);
  if (full) {
    Counters* C = g->ctr;
    uint32_t *dplus = g->fq[0], *heavy = g->fq[4];  // scratch: the traversal queues
    const TcClasses cls = {{g->fq[1], g->fq[2], g->fq[3]}, C->tc_class};
    unsigned long long* sum = &C->u64tmp[0];
    // |A(u)| = k takes k neighbours of degree k or more, so k^2 <= 2 m, and u's own degree is at most
    // what its buckets were sized for, or the words of its slabs, and the arcs inserted since: a class
    // that cannot have a vertex is not launched, and one that can gets no more blocks than vertices.  (The
    // host does not know what replays of a captured insert added, nor the graph that replays of this count
    // meet.)
    const ViewHost& und = g->view[VU];
    const bool unknown = g->captured_update || stream_capturing(stream);
    const uint64_t added = unknown ? UINT64_MAX / 4 : g->view[VF].added;
    const uint64_t m = g->m0 + added;
    uint64_t built = kKeysPerSlab * (und.nb_max + und.pool_built);  // the largest degree at creation
    if (g->cfg.load_factor > 0.f)
      built = std::min(built, (uint64_t)((double)g->cfg.load_factor * kKeysPerSlab * und.nb_max) + 1);
    const uint64_t degree = built + added;
    const auto blocks = [&](uint64_t keys, uint32_t most) -> uint32_t {
      return degree <= keys || 2 * m < (keys + 1) * (keys + 1) ? 0u : (uint32_t)std::min<uint64_t>(most, m / keys + 1);
    };
    const uint32_t mid = blocks(kTcWaveKeys, CountClass<true>::kBlocks);
    const uint32_t large = blocks(CountClass<true>::kKeys, CountClass<false>::kBlocks);
    // (a few arcs more leave the degrees as they were; should they all meet at one vertex, the count takes
    // longer and is the same)
    if (und.nb_max <= 2 && built <= kTcWaveKeys && !unknown && g->net_added <= 64 + N / 64) {
      hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(sum), 2u);
      hipLaunchKernelGGL(k_tc_few, dim3(blocks_for((uint64_t)N * kGroup)), dim3(kBlock), 0, stream, U, N, sum);
      hipLaunchKernelGGL(k_tc_finish, dim3(1), dim3(64), 0, stream, g->ctr, 4, out);
    } else {
      hipLaunchKernelGGL(k_tc_room, dim3(blocks_for((N + kTcRoom - 1) / kTcRoom)), dim3(kBlock), 0, stream, U, N, g->tc_off,
                         heavy, C);
      hipLaunchKernelGGL(k_tc_orient, dim3(blocks_for(N)), dim3(kBlock), 0, stream, U, N, heavy, &C->n_heavy_tc,
                         g->tc_off, g->tc_list, dplus, cls);
      if (large)
        hipLaunchKernelGGL(k_tc_count_block<false>, dim3(large), dim3(CountClass<false>::kThreads), 0, stream, U,
                           g->tc_list, g->tc_off, dplus, cls.q[2], cls.n + 2, sum);
      if (mid)
        hipLaunchKernelGGL(k_tc_count_block<true>, dim3(mid), dim3(CountClass<true>::kThreads), 0, stream, U, g->tc_list,
                           g->tc_off, dplus, cls.q[1], cls.n + 1, sum);
      hipLaunchKernelGGL(k_tc_count_wave, dim3(blocks_for((uint64_t)N * 64)), dim3(kBlock), 0, stream, g->tc_list,
                         g->tc_off, dplus, cls.q[0], cls.n, sum);
      hipLaunchKernelGGL(k_tc_finish, dim3(1), dim3(64), 0, stream, g->ctr, 2, out);
    }
  } else if (p.list.empty()) {
    hipLaunchKernelGGL(k_tc_finish, dim3(1), dim3(64), 0, stream, g->ctr, 3, out);
  } else {
    // all pending batches are of one kind: their union is one effective batch
    uint64_t nk = 0;
    for (const BatchRec* b : p.list) {
      hipLaunchKernelGGL(k_tc_keys, dim3(blocks_for(b->n)), dim3(kBlock), 0, stream,
                         log_at(g, b->off), b->n, N, g->tc_keys[0] + nk);
      nk += 2 * b->n;
    }
    if (nk > 2 * g->log_cap) return MK_ERR_CAPACITY;
    unsigned end_bit = 32;
    while (end_bit < 64 && ((uint64_t)N >> (end_bit - 32)) != 0) ++end_bit;
    size_t tb = g->sort_tmp_bytes;
    if (rocprim::radix_sort_keys(g->sort_tmp, tb, g->tc_keys[0], g->tc_keys[1], (size_t)nk, 0,
                                 end_bit, stream) != hipSuccess)
      return MK_ERR_HIP;
    hipLaunchKernelGGL(k_tc_begin, dim3(1), dim3(64), 0, stream, g->ctr);
    // segment bounds per source vertex (scratch: two traversal queues, unused here)
    hipLaunchKernelGGL(k_tc_segs, dim3(blocks_for(nk)), dim3(kBlock), 0, stream, g->tc_keys[1], nk, N,
                       g->fq[4], g->fq[5]);
    // S2 of arcs into hubs goes through the hubs' sets when ids leave the tag bit free
    const bool s2in = N <= 0x7FFFFFFFu;
    uint32_t* longs = reinterpret_cast<uint32_t*>(g->tc_keys[0]);  // free after the sort
    const dim3 groups(grid_for_groups(std::min<uint64_t>(nk, 1u << 20)));
    if (nk < kTcFewKeys && g->view[VU].nb_max > kTcLong) {
      hipLaunchKernelGGL(k_tc_batch<true>, groups, dim3(kBlock), 0, stream, U, g->tc_keys[1], nk, g->fq[4], g->fq[5],
                         N, s2in, g->ctr->tc_s, longs, &g->ctr->tc_work);
      hipLaunchKernelGGL(k_tc_long, dim3((uint32_t)std::min<uint64_t>(nk, 4096)), dim3(kBlock), 0, stream, U,
                         g->tc_keys[1], longs, &g->ctr->tc_work, g->ctr->tc_s);
    } else {
      hipLaunchKernelGGL(k_tc_batch<false>, groups, dim3(kBlock), 0, stream, U, g->tc_keys[1], nk, g->fq[4],
                         g->fq[5], N, s2in, g->ctr->tc_s, longs, &g->ctr->tc_work);
    }
    // hub edges: work items numbered by an exclusive scan over the key
    // positions, in the sort's input buffer (free after the sort; 2 * nk u32 fit in it)
    uint32_t* hcnt = reinterpret_cast<uint32_t*>(g->tc_keys[0]);
    uint32_t* hoff = hcnt + nk;
    // packed lists of the hub partners (scratch: the other traversal queues)
    uint32_t *dcnt = g->fq[0], *icnt = g->fq[1], *ioff = g->fq[2], *need = g->fq[3];
    hipLaunchKernelGGL(k_zero_u32, dim3(blocks_for(N)), dim3(kBlock), 0, stream, need, N);
    hipLaunchKernelGGL(k_tc_need, dim3(blocks_for(nk)), dim3(kBlock), 0, stream, U, g->tc_keys[1], nk,
                       g->fq[4], g->fq[5], N, need);
    hipLaunchKernelGGL(k_tc_pack_count, dim3(blocks_for(N)), dim3(kBlock), 0, stream, U, N, need, dcnt, icnt);
    {
      size_t tb2 = g->scan_tmp_bytes;
      if (rocprim::exclusive_scan(g->scan_tmp, tb2, dcnt, g->tc_off, (uint64_t)0, (size_t)N,
                                  rocprim::plus<uint64_t>(), stream) != hipSuccess)
        return MK_ERR_HIP;
      tb2 = g->scan_tmp_bytes;
      if (rocprim::exclusive_scan(g->scan_tmp, tb2, icnt, ioff, 0u, (size_t)N, rocprim::plus<uint32_t>(),
                                  stream) != hipSuccess)
        return MK_ERR_HIP;
    }
    hipLaunchKernelGGL(k_tc_pack, dim3(kWalkBlocks), dim3(kBlock), 0, stream, U, N, g->tc_off, icnt, ioff, need,
                       g->tc_list);
    // the small hubs' items, then the large ones' (the item numbering is redone per class)
    auto hub_launch = [&](auto cls) -> bool {
      constexpr bool kSmall = decltype(cls)::value;
      using H = HubClass<kSmall>;
      hipLaunchKernelGGL(k_tc_hub_count<kSmall>, dim3(blocks_for(nk)), dim3(kBlock), 0, stream, U,
                         g->tc_keys[1], nk, g->fq[5], N, hcnt);
      size_t tb2 = g->scan_tmp_bytes;
      if (rocprim::exclusive_scan(g->scan_tmp, tb2, hcnt, hoff, 0u, (size_t)nk, rocprim::plus<uint32_t>(),
                                  stream) != hipSuccess)
        return false;
      hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, &g->ctr->tc_work, 1u);
      hipLaunchKernelGGL(k_tc_hub<kSmall>, dim3(H::kBlocks), dim3(H::kThreads), 0, stream, U, g->tc_keys[1], nk,
                         g->fq[4], g->fq[5], hcnt, hoff, &g->ctr->tc_work, g->tc_list, g->tc_off, s2in,
                         g->ctr->tc_s);
      return true;
    };
    if (!hub_launch(std::true_type{}) || !hub_launch(std::false_type{})) return MK_ERR_HIP;
    hipLaunchKernelGGL(k_tc_finish, dim3(1), dim3(64), 0, stream, g->ctr,
                       p.kinds == 1 ? 0 : 1, out);
  }
  MK_LAUNCH(g, "triangles");
  g->tc.valid = true;
  mark_seen(g, g->tc);
  return MK_OK;
}

}  // extern "C"
