// Dynamic BFS and SSSP (section 4.2, the batch-dynamic SSSP algorithm; BFS uses the same
// kernels with unit weights).
//
// Each vertex keeps a 64-bit tree node <distance, parent> (the footnote on the packed
// pair) updated by a 64-bit atomic minimum, so among equal distances the smallest parent
// id wins and the fixed point is unique.  A batch is applied by a prologue followed by
// the common frontier epilogue:
//   insert prologue : relax every effective inserted arc (u, v, w) with a finite u;
//   delete prologue : invalidate v for each deleted tree arc (parent(v) == u), invalidate
//                     the whole dependence subtree below it, then pull each invalidated
//                     vertex's best candidate from its valid in-neighbours (reverse view);
//                     this is the decremental frontier of valid -> invalid arcs;
//   epilogue        : expand the frontier until it is empty.
//
// Differences from the paper's kernels (same fixed point): the frontier holds vertices,
// not edges (a per-iteration stamp keeps each vertex once); subtree invalidation walks
// the tree top-down through the forward view instead of walking every vertex's parent
// chain to the source; vertices with many buckets are expanded by a whole block.
//
// Weighted epilogue in distance bands (near-far): an improved vertex joins the frontier
// only if its new distance is below the current band's threshold T, else it waits on a
// far pile.  When the frontier empties, the pile's smallest pending distance f gives the
// next threshold f + delta, the pile entries below it form the next frontier and the
// rest stay.  Any order of relaxations reaches the same unique fixed point; expanding
// nearer vertices first only avoids re-expanding vertices whose distance drops again.
#include <algorithm>

#include "mk_internal.h"

using namespace mk;

namespace {

constexpr uint32_t kExpandBlocks = 2048;  // 256 CUs x 8 resident blocks
constexpr int kSyncFirst = 4, kSyncMax = 16;  // frontier launches between size read-backs: 4,
                                              // then doubling while the frontier lasts
constexpr uint32_t kSmallGraph = 1u << 17;    // vertices of a graph whose loops start with 2

__device__ inline uint64_t tree_node(uint64_t dist, uint32_t parent) {
  if (dist >= 0xFFFFFFFFull) dist = 0xFFFFFFFEull;  // saturate below INF
  return (dist << 32) | parent;
}

constexpr uint32_t kGiantBuckets = 512;  // vertices with more buckets are split over 256 groups
constexpr uint32_t kGiantSplit = 256;

// Where pushed vertices go: light (<= kHeavyBuckets buckets), heavy (<= kGiantBuckets)
// and giant queues with their size counters.
struct PushQ {
  uint32_t* q[3];
  uint32_t* c[3];
};

// Near-far routing of the weighted epilogue.  T == nullptr: every push is near.
struct Route {
  const uint32_t* T;   // threshold of the current band
  uint32_t* far;       // far pile of the current band and its size
  uint32_t* far_cnt;
  uint32_t* far_mark;  // band id of the last far push of each vertex
  uint32_t band;
};

__device__ inline uint32_t band_limit(const Route& r) { return r.T ? *r.T : 0xFFFFFFFFu; }


// Routed pushes through block stages: a vertex improved to distance `dist` goes to the near
// queues ([0..2] light, heavy, giant of Q) when dist < T, else onto the far pile of r ([3],
// once per band); open_routed opens the four stages.
__device__ inline void open_routed(Stage (&S)[4], const PushQ& Q, const Route& r) {
  for (int k = 0; k < 3; ++k) stage_open(S[k], Q.q[k], Q.c[k]);
  stage_open(S[3], r.far, r.far_cnt);
  __syncthreads();
}

__device__ inline void push_staged(Stage (&S)[4], const uint32_t* nbk, const Route& r, uint32_t T,
                                   uint32_t* mark, uint32_t stamp, bool p, uint32_t v, uint32_t dist) {
  const bool near = p && dist < T;
  bool take = false, take_far = false;
  if (near) take = atomicExch(mark + v, stamp) != stamp;
  else if (p) take_far = atomicExch(r.far_mark + v, r.band) != r.band;
  const uint32_t nb = take ? nbk[v] : 0u;
  stage_push(S[3], take_far, v);
  stage_push(S[0], take && nb <= kHeavyBuckets, v);
  stage_push(S[1], take && nb > kHeavyBuckets && nb <= kGiantBuckets, v);
  stage_push(S[2], take && nb > kGiantBuckets, v);
}

struct Queues {
  const uint32_t* cur[3];  // light, heavy, giant
  PushQ next;
  uint32_t* cnt;  // [3k .. 3k+2]: rotating sizes of queue k
  int icur, iclear;
};

// Stage the keys of the slab words selected by `mask` (bit j: word j) of every active lane.
__device__ inline void stage_words(Stage& S, uint32_t mask, const Slab& sl) {
  bool any;
  const StageSlots t = stage_reserve(S, (uint32_t)__popc(mask), any);
  if (!any) return;
  uint32_t pos = t.pos;
#pragma unroll
  for (int j = 0; j < kKeysPerSlab; ++j)
    if (mask >> j & 1) stage_put(S, t, pos++, (uint32_t)sl.w[j]);
}

// Relax the 15 out-arcs of a whole slab held by one lane: the distance loads, then the atomic
// minima together with the frontier marks and the bucket counts, each as one independent
// batch, and the pushes of the wave with one counter atomic per queue.
//
// A neighbour is marked, and pushed by whoever marks it first, as soon as the candidate beats
// the distance read, without waiting for the minimum to return: if another lane's candidate was
// smaller still, that lane's improvement needs the push as well.  (A vertex whose candidate is far
// may then wait on the pile in vain; the band step drops it.)  `single`: no vertex of the graph
// has several buckets, so no bucket count is read.  *more counts the further buckets of the light
// vertices pushed (inner steps).
template <bool kUnit>
__device__ inline void relax_slab_lane(const DView& F, uint64_t* D, uint32_t u, uint64_t du, const Slab& sl,
                                       int nd, Stage (&S)[4], const Route& r, uint32_t T, uint32_t* mark,
                                       uint32_t stamp, bool single, uint32_t* more) {
  uint64_t cand[kKeysPerSlab], cur[kKeysPerSlab];
  load_of_keys<uint64_t>(D, sl, live_words(sl, nd), 0ull, cur);
#pragma unroll
  for (int j = 0; j < kKeysPerSlab; ++j) cand[j] = tree_node(du + (kUnit ? 1ull : (sl.w[j] >> 32)), u);
  uint32_t near = 0, far = 0;
#pragma unroll
  for (int j = 0; j < kKeysPerSlab; ++j) {
    if (cand[j] >= cur[j]) continue;
    if (kUnit || (uint32_t)(cand[j] >> 32) < T) near |= 1u << j;
    else far |= 1u << j;
  }
  uint32_t tk[kKeysPerSlab], nb[kKeysPerSlab];
#pragma unroll
  for (int j = 0; j < kKeysPerSlab; ++j) {
    const uint32_t v = (uint32_t)sl.w[j];
    tk[j] = 0;
    nb[j] = 1;
    if (near >> j & 1) {
      tk[j] = atomicExch(mark + v, stamp);
      if (!single) nb[j] = F.nbk[v];
    } else if (far >> j & 1) {
      tk[j] = atomicExch(r.far_mark + v, r.band);
    }
    if ((near | far) >> j & 1) (void)amin64(D + v, cand[j]);
  }
  uint32_t tn = 0, tf = 0, heavy = 0, giant = 0, further = 0;
#pragma unroll
  for (int j = 0; j < kKeysPerSlab; ++j) {
    if ((near >> j & 1) && tk[j] != stamp) {
      if (nb[j] > kGiantBuckets) giant |= 1u << j;
      else if (nb[j] > kHeavyBuckets) heavy |= 1u << j;
      else {
        tn |= 1u << j;
        further += nb[j] - 1;
      }
    }
    if ((far >> j & 1) && tk[j] != r.band) tf |= 1u << j;
  }
  stage_words(S[0], tn, sl);
  if (!single) {
    if (further) atomicAdd(more, further);
    stage_words(S[1], heavy, sl);
    stage_words(S[2], giant, sl);
  }
  if (!kUnit) stage_words(S[3], tf, sl);
}

constexpr uint32_t kGiantLanes = kGiantSplit * kGroup;  // lanes sharing one giant vertex
// A light frontier of at most kInnerMost vertices is expanded by one block, which goes on with
// the frontiers that follow, up to kInnerSteps of them, while they fit its LDS stage and hold no
// heavy vertex: a step then costs its own chain of dependent loads (about 10 us) instead of a
// launch and the reads that find the frontier as well (about 16 us).  Where vertices have several
// buckets, the buckets count: at most kInnerMixed to begin with and kInnerOn to go on, kInnerMany where
// they have many (kManyBuckets).  512 vertices of 15 buckets are 30 rounds of a block, and took 100 us
// where the whole chip takes 20.  Bounds of 256, of 384 and 512, and of 512 and 1,024, us: 4,096 vertices of
// degree 8, 1,000 arcs deleted 196, 190, 190, inserted back 114, 106, 106, one-off BFS 135, 131, 164;
// degree 16 one-off SSSP 392, 385, 445.
constexpr uint32_t kInnerMost = 512, kInnerMixed = 384, kInnerOn = 512, kInnerMany = 256;
constexpr uint32_t kInnerSteps = 64;

// After a step of an inner loop: the frontier staged in S[0] becomes the block's list in LDS, or
// the loop ends (empty, too large, heavy vertices, or out of steps) and the stages hold the
// launch's output.  Every thread of the block gets the same answer.
__device__ inline bool inner_next(Stage (&S)[4], uint32_t* list, uint32_t* more, bool single, bool many,
                                  uint32_t& n, uint32_t& step) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this step's atomics have been performed
  __syncthreads();
  // and the next step reads what they left, not a cache line from before them (a stale distance
  // of a vertex improved a step ago would push it again)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const uint32_t k = S[0].n;
  const bool go = k > 0 && k + *more <= (single ? kStage : many ? kInnerMany : kInnerOn) && S[1].n == 0 &&
                  S[2].n == 0 && step + 1 < kInnerSteps;
  if (!go) return false;
  for (uint32_t i = threadIdx.x; i < k; i += kBlock) list[i] = S[0].buf[i];
  __syncthreads();
  if (threadIdx.x == 0) S[0].n = *more = 0;
  __syncthreads();
  n = k;
  ++step;
  return true;
}

// How a launch's blocks share the light vertices.  Where no vertex has several buckets: a lane each.
// Else 16 lanes each, a lane to a bucket, when there are lanes enough (kWideMost vertices) or the
// vertices have many buckets (kManyBuckets on average).  Else a lane each again, with kShareBlocks
// blocks to spread them over, whose other lanes take the further buckets.  One-off traversals, us, BFS
// and SSSP, with 256 vertices to a block always / with 32 to 256 / so: 20,000 vertices of degree 150
// 560, 2,113 / 235, 747 / 243, 714; 4,096 of degree 16 175, 596 / 139, 480 / 125, 386; 100,000 of degree
// 30 419, 1,436 / 218, 884 / 201, 796; R-MAT scale 16 336, 922 / 206, 594 / 198, 535, scale 18 414, 983 /
// 276, 726 / 264, 704.  With 16 lanes each whatever the number, R-MAT scale 20 takes 752, 1,684 instead
// of 657, 1,463.
struct Share {
  uint32_t n;  // light vertices to a block and round
  bool wide;   // 16 lanes each
};
constexpr uint32_t kWideMost = 16384, kShareBlocks = 512, kManyBuckets = 4;
__device__ inline Share light_share(uint32_t nl, bool single, bool many) {
  if (single) return Share{kBlock, false};
  if (many || nl <= kWideMost) return Share{kGroupsPerBlock, true};
  return Share{min((uint32_t)kBlock, (nl + kShareBlocks - 1) / kShareBlocks), false};
}

// Whether a block of a frontier kernel has nothing to do (the same in all its threads).
__device__ inline bool no_work(uint32_t nl, uint32_t nh, uint32_t ngi, uint32_t share) {
  return (uint64_t)blockIdx.x * share >= nl && blockIdx.x >= nh && blockIdx.x >= ngi * (kGiantLanes / kBlock);
}

// Whether one block takes this frontier (and those that follow): every block with work finds the
// same answer.  *more is zero before the call and after it, when the block has synchronized.
__device__ inline bool inner_first(const DView& F, const uint32_t* light, uint32_t nl, uint32_t nh, uint32_t ngi,
                                   bool single, bool many, uint32_t* more) {
  if (nl > kInnerMost || nh || ngi) return false;
  if (single) return true;
  const uint32_t lim = many ? kInnerMany : kInnerMixed;
  if (nl > lim) return false;
  if (nl * kHeavyBuckets <= lim) return true;
  uint32_t b = 0;
  for (uint32_t i = threadIdx.x; i < nl; i += kBlock) b += F.nbk[light[i]];
  for (int o = 32; o > 0; o >>= 1) b += __shfl_xor(b, o);
  if (threadIdx.x == 0) *more = 0;
  __syncthreads();
  if (lane64() == 0) atomicAdd(more, b);
  __syncthreads();
  const uint32_t total = *more;
  __syncthreads();
  return total <= lim;
}

// Slabs of light vertices' further buckets, collected while the block visits the primary slabs.
// Each round of 256 vertices counts in its turn's word of n, which is zero when the round begins.
// One word would not do: after a round that collected nothing, a wave that is ahead adds for the next
// round while another has yet to read this round's count.  The word of the next turn is cleared
// before this round's barrier; it was read last two rounds ago, before the barrier of the round
// between, so no wave can still want it.
constexpr uint32_t kExtras = 1024;
struct Extras {
  uint32_t n[3];
  uint32_t u[kExtras], s[kExtras];
};
__device__ inline void open_extras(Extras& E) {  // the caller then synchronizes the block
  if (threadIdx.x < 3) E.n[threadIdx.x] = 0;
}

// Visit every slab of the frontier's vertices, a lane to a bucket chain: the primary slabs of `share`
// light vertices at a time, then those vertices' further buckets (collected in E, so that the
// lanes share them evenly; a lane walks its own where E is full), a block to a heavy vertex,
// kGiantLanes lanes to a giant one.  begin(u) is called before a slab of u is read, so that what
// it loads is on its way together with the slab; body(u, begin's result, slab, data words) once
// per slab.  There is one call site of body, as its code is long.  Every thread of the block
// calls this; `list` replaces the light queue (inner steps), `stride` blocks share the work, `turn`
// (0 before the first call) goes from one call to the next.
template <class Begin, class Body>
__device__ inline void walk_frontier(const DView& F, const Queues& q, const uint32_t* list, uint32_t nl, uint32_t nh,
                                     uint32_t ngi, uint32_t stride, const Share& share, bool single, Extras& E,
                                     uint32_t& turn,
                                     Begin&& begin, Body&& body) {
  int mode = 0;  // block-uniform: 0 light vertices, 1 their further buckets, 2 heavy, 3 giant
  const bool wide = share.wide;
  uint32_t base = blockIdx.x * share.n, eb = 0, ne = 0, hb = 0;
  const uint32_t tid = threadIdx.x;
  while (true) {
    uint32_t u = 0, s = kInvalid, own = 0, own_end = 0;  // own: further buckets this lane walks itself
    int nd = kKeysPerSlab;
    if (mode == 0) {
      if (base >= nl) {
        mode = 2;
        base = blockIdx.x;
        continue;
      }
      if (wide) {
        const uint32_t i = base + tid / kGroup, b = tid % kGroup;
        if (i < nl) {
          u = list[i];
          const uint4 w = reinterpret_cast<const uint4*>(slab_ptr(F, u))[7];
          if (b < w.w) s = b ? w.x + b - 1 : u;
          if (b == 0 && w.w > 1) nd = kKeysPerSlab - 1;
        }
      } else if (tid < share.n && base + tid < nl) {
        u = s = list[base + tid];
      }
    } else if (mode == 1) {
      if (eb + tid < ne) {
        u = E.u[eb + tid];
        s = E.s[eb + tid];
      }
    } else {
      const uint32_t per = mode == 2 ? kBlock : kGiantLanes;  // lanes that share the vertex
      const uint32_t split = per / kBlock;
      if (base >= (mode == 2 ? nh : ngi * split)) {
        if (mode == 3) return;
        mode = 3;
        base = blockIdx.x;
        continue;
      }
      u = q.cur[mode - 1][base / split];
      const uint4 w = reinterpret_cast<const uint4*>(slab_ptr(F, u))[7];  // extra head slabs, bucket count
      const uint32_t b = hb + (base % split) * kBlock + tid;
      if (b < w.w) {
        s = b ? w.x + b - 1 : u;
        nd = b ? kKeysPerSlab : kKeysPerSlab - 1;
      }
      hb += per;
      if (hb + (base % split) * kBlock >= w.w) {  // the vertex's buckets are dealt out
        hb = 0;
        base += stride;
      }
    }
    if (s != kInvalid) {
      const auto ctx = begin(u);
      Slab sl;
      load_slab(F, s, sl);
      if (mode == 0 && !wide) {
        const uint32_t nb = (uint32_t)(sl.w[15] >> 32);
        if (nb > 1) {
          nd = kKeysPerSlab - 1;
          const uint32_t xb = (uint32_t)sl.w[14];
          const uint32_t at = atomicAdd(&E.n[turn], nb - 1);
          for (uint32_t k = 0; k < nb - 1; ++k) {
            if (at + k < kExtras) {
              E.u[at + k] = u;
              E.s[at + k] = xb + k;
            } else {
              own = xb + k;
              own_end = xb + nb - 1;
              break;
            }
          }
        }
      }
      while (true) {
        body(u, ctx, sl, nd);
        s = (uint32_t)sl.w[15];
        if (s == kInvalid) {
          if (own == own_end) break;
          s = own++;
        }
        nd = kKeysPerSlab;
        load_slab(F, s, sl);
      }
    }
    if (mode == 0) {
      if (!single && !wide) {
        const uint32_t after = turn == 2 ? 0u : turn + 1;
        if (tid == 0) E.n[after] = 0;
        __syncthreads();
        ne = min(E.n[turn], kExtras);
        turn = after;
        eb = 0;
        if (ne) mode = 1;
      }
      if (mode == 0) base += stride * share.n;
    } else if (mode == 1) {
      eb += kBlock;
      if (eb >= ne) {
        __syncthreads();  // the next round writes E.u and E.s
        mode = 0;
        base += stride * share.n;
      }
    }
  }
}

// Frontier expansion: relax every arc that leaves a frontier vertex.
//
// What bounds it where frontiers are small (a road network, a small graph): the chain of
// dependent memory accesses of one vertex: queue, slab and distance, neighbours' distances,
// marks, queue counter.  A launch over 50,000 light vertices of the 4096 x 4096 grid takes 13 us
// (slab 2.2, distances and marks 5.5, staging 1.8, queue counter and copy 1.5; 18-20 us with the
// bucket counts, the distance and the slab read one after the other and every block opening and
// closing its stages); an inner step takes 10 us and no launch.
template <bool kUnit>
__global__ void __launch_bounds__(kBlock) k_expand(DView F, uint64_t* D, Queues q, Route r, uint32_t* mark,
                                                   uint32_t stamp, bool single, bool many) {
  uint32_t nl = q.cnt[q.icur];
  const uint32_t nh = q.cnt[3 + q.icur], ngi = q.cnt[6 + q.icur];
  if (blockIdx.x == 0 && threadIdx.x < 3) q.cnt[3 * threadIdx.x + q.iclear] = 0;
  Share share = light_share(nl, single, many);
  if (no_work(nl, nh, ngi, share.n)) return;  // also an empty frontier
  __shared__ uint32_t more;
  const bool inner = inner_first(F, q.cur[0], nl, nh, ngi, single, many, &more);
  if (inner && blockIdx.x != 0) return;
  if (inner) share = Share{kBlock, false};
  __shared__ Stage S[4];
  __shared__ uint32_t list[kStage];
  __shared__ Extras E;
  open_extras(E);
  if (threadIdx.x == 0) more = 0;
  open_routed(S, q.next, r);
  const uint32_t T = kUnit ? 0xFFFFFFFFu : band_limit(r);
  uint32_t step = 0, turn = 0;
  do {
    walk_frontier(F, q, step ? list : q.cur[0], nl, nh, ngi, inner ? 1u : gridDim.x, share, single, E, turn,
                  [&](uint32_t u) { return ld_u64(D + u) >> 32; },
                  [&](uint32_t u, uint64_t du, const Slab& sl, int nd) {
                    relax_slab_lane<kUnit>(F, D, u, du, sl, nd, S, r, T, mark, stamp + step, single, &more);
                  });
  } while (inner && inner_next(S, list, &more, single, many, nl, step));
  stage_close(S);
}

// Band step, part 1: the smallest distance on the far pile at or above the old threshold
// (an entry below it was expanded, at its current distance, in an earlier band).  The size of
// the pile about to be filled is reset here, the minimum by the step before (or the reset).
__global__ void k_band_min(const uint64_t* D, const uint32_t* far, const uint32_t* far_cnt, const uint32_t* T,
                           uint32_t* fmin, uint32_t* next_cnt) {
  const uint32_t n = *far_cnt, told = *T;
  if (blockIdx.x == 0 && threadIdx.x == 0) *next_cnt = 0;
  uint32_t m = 0xFFFFFFFFu;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t d = (uint32_t)(ld_u64(D + far[i]) >> 32);
    if (d >= told && d < m) m = d;
  }
  for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, o));
  if (lane64() == 0 && m != 0xFFFFFFFFu) atomicMin(fmin, m);
}

// Band step, part 2: the new threshold is fmin + delta; pile entries in [old T, new T) form
// the frontier of the next band, later ones move to the other pile under the new band id.
// Appends are staged per block (with an atomic per wave and output, 700,000 entries took 130 us).
__global__ void __launch_bounds__(kBlock) k_band_split(const uint32_t* nbk, const uint64_t* D, const uint32_t* far,
                                                       const uint32_t* far_cnt, const uint32_t* T, const uint32_t* fmin,
                                                       uint32_t* fmin_next, uint32_t delta, uint32_t* T_next, PushQ Q,
                                                       uint32_t* far_next, uint32_t* next_cnt, uint32_t* far_mark,
                                                       uint32_t band_next, bool single) {
  const uint32_t n = *far_cnt, told = *T, fm = *fmin;
  const uint32_t tnew = fm == 0xFFFFFFFFu ? told : (fm >= 0xFFFFFFFFu - delta ? 0xFFFFFFFFu : fm + delta);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *T_next = tnew;
    *fmin_next = 0xFFFFFFFFu;
  }
  if (blockIdx.x * kBlock >= n) return;
  __shared__ Stage S[4];
  for (int k = 0; k < 3; ++k) stage_open(S[k], Q.q[k], Q.c[k]);
  stage_open(S[3], far_next, next_cnt);
  __syncthreads();
  for (uint32_t base = blockIdx.x * kBlock; base < n; base += gridDim.x * kBlock) {
    const uint32_t i = base + threadIdx.x;
    bool near = false, keep = false;
    uint32_t v = 0, nb = 1;
    if (i < n) {
      v = far[i];
      const uint32_t d = (uint32_t)(ld_u64(D + v) >> 32);
      near = d >= told && d < tnew;
      keep = d >= tnew;
    }
    if (keep) far_mark[v] = band_next;
    if (near && !single) nb = nbk[v];
    stage_push(S[3], keep, v);
    stage_push(S[0], near && nb <= kHeavyBuckets, v);
    if (!single) {
      stage_push(S[1], near && nb > kHeavyBuckets && nb <= kGiantBuckets, v);
      stage_push(S[2], near && nb > kGiantBuckets, v);
    }
  }
  stage_close(S);
}

__global__ void k_trav_init(uint64_t* D, uint32_t nv, uint32_t src) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x)
    D[v] = v == src ? (uint64_t)src : kTreeNone;
}

// Reset the rotating counters so that slot 0 is the current frontier, empty both far
// piles, reset their minima and set the first threshold to 0 (every prologue push of a weighted traversal
// waits on the pile until the first band step).
__global__ void k_queue_reset(uint32_t* cnt, uint32_t* inval_cnt) {
  if (threadIdx.x < 13) cnt[threadIdx.x] = 0;
  if (threadIdx.x == 13 || threadIdx.x == 14) cnt[threadIdx.x] = 0xFFFFFFFFu;  // pile minima
  if (threadIdx.x == 0 && inval_cnt) *inval_cnt = 0;
}

__global__ void k_seed_source(DView F, uint32_t src, PushQ Q, Route r, uint32_t* mark, uint32_t stamp) {
  if (threadIdx.x != 0) return;
  if (r.T) {  // weighted: the source waits on the far pile for the first band step
    r.far_mark[src] = r.band;
    r.far[0] = src;
    *r.far_cnt = 1;
    return;
  }
  mark[src] = stamp;
  const uint32_t nb = F.nbk[src];
  const int k = nb <= kHeavyBuckets ? 0 : (nb <= kGiantBuckets ? 1 : 2);
  Q.q[k][0] = src;
  *Q.c[k] = 1;
}

// Insert prologue: relax each effective inserted arc.
template <bool kUnit>
__global__ void k_relax_batch(DView F, uint64_t* D, Log lg, uint64_t n, PushQ Q, Route r, uint32_t* mark,
                              uint32_t stamp) {
  __shared__ Stage S[4];
  open_routed(S, Q, r);
  const uint32_t T = band_limit(r);
  // whole waves step together so that the wave-wide push sees every lane
  const uint64_t lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; base < n;
       base += stride) {
    const uint64_t i = base + lane;
    bool improve = false;
    uint32_t v = 0;
    uint64_t cand = kTreeNone;
    if (i < n && lg.st[i] == 1) {
      const uint32_t u = lg.s[i];
      v = lg.d[i];
      const uint64_t du = ld_u64(D + u);
      if (du != kTreeNone) {
        cand = tree_node((du >> 32) + (kUnit ? 1u : lg.w[i]), u);
        if (cand < D[v]) improve = amin64(D + v, cand) > cand;
      }
    }
    push_staged(S, F.nbk, r, T, mark, stamp, improve, v, (uint32_t)(cand >> 32));
  }
  stage_close(S);
}

// A vertex cut from the tree (by exactly one successful CAS, so it needs no frontier
// mark) is staged to [3] the invalidated list and [0..2] the light, heavy or giant queue.
__device__ inline void stage_cut(Stage (&S)[4], const uint32_t* nbk, bool hit, uint32_t y) {
  const uint32_t nb = hit ? nbk[y] : 0u;
  stage_push(S[3], hit, y);
  stage_push(S[0], hit && nb <= kHeavyBuckets, y);
  stage_push(S[1], hit && nb > kHeavyBuckets && nb <= kGiantBuckets, y);
  stage_push(S[2], hit && nb > kGiantBuckets, y);
}

// Delete prologue, step 1: a deleted arc (u, v) of the dependence tree invalidates v.
__global__ void k_invalidate(DView F, uint64_t* D, Log lg, uint64_t n, PushQ Q, uint32_t* inval,
                             uint32_t* inval_cnt) {
  // a vertex is cut by exactly one successful CAS, so it needs no frontier mark
  __shared__ Stage S[4];
  for (int k = 0; k < 3; ++k) stage_open(S[k], Q.q[k], Q.c[k]);
  stage_open(S[3], inval, inval_cnt);
  __syncthreads();
  const uint64_t lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; base < n;
       base += stride) {
    const uint64_t i = base + lane;
    bool hit = false;
    uint32_t v = 0;
    if (i < n && lg.st[i] == 1) {
      const uint32_t u = lg.s[i];
      v = lg.d[i];
      const uint64_t dv = ld_u64(D + v);
      if (dv != kTreeNone && (uint32_t)dv == u) hit = cas64(D + v, dv, kTreeNone) == dv;
    }
    stage_cut(S, F.nbk, hit, v);
  }
  stage_close(S);
}

// Delete prologue, step 2: invalidate the subtree below each invalidated vertex x (its
// tree children are the out-neighbours y whose parent is x).  The child tests of a slab are
// issued together.
__global__ void __launch_bounds__(kBlock) k_propagate(DView F, uint64_t* D, Queues q, uint32_t* inval,
                                                      uint32_t* inval_cnt, bool single, bool many) {
  uint32_t nl = q.cnt[q.icur];
  const uint32_t nh = q.cnt[3 + q.icur], ngi = q.cnt[6 + q.icur];
  if (blockIdx.x == 0 && threadIdx.x < 3) q.cnt[3 * threadIdx.x + q.iclear] = 0;
  Share share = light_share(nl, single, many);
  if (no_work(nl, nh, ngi, share.n)) return;  // also an empty frontier
  __shared__ uint32_t more;
  const bool inner = inner_first(F, q.cur[0], nl, nh, ngi, single, many, &more);
  if (inner && blockIdx.x != 0) return;
  if (inner) share = Share{kBlock, false};
  __shared__ Stage S[4];
  __shared__ uint32_t list[kStage];
  __shared__ Extras E;
  open_extras(E);
  if (threadIdx.x == 0) more = 0;
  for (int k = 0; k < 3; ++k) stage_open(S[k], q.next.q[k], q.next.c[k]);
  stage_open(S[3], inval, inval_cnt);
  __syncthreads();
  uint32_t step = 0, turn = 0;
  do {
    walk_frontier(F, q, step ? list : q.cur[0], nl, nh, ngi, inner ? 1u : gridDim.x, share, single, E, turn,
                  [](uint32_t) { return 0; },
                  [&](uint32_t x, int, const Slab& sl, int nd) {
                    uint64_t dy[kKeysPerSlab];
                    load_of_keys<uint64_t>(D, sl, live_words(sl, nd), kTreeNone, dy);
                    uint32_t nb[kKeysPerSlab];
#pragma unroll
                    for (int j = 0; j < kKeysPerSlab; ++j) {
                      const uint32_t y = (uint32_t)sl.w[j];
                      const bool child = dy[j] != kTreeNone && (uint32_t)dy[j] == x;
                      nb[j] = child && !single ? F.nbk[y] : 1u;
                      dy[j] = child ? cas64(D + y, dy[j], kTreeNone) ^ dy[j] : 1ull;  // 0: this lane cut y
                    }
                    uint32_t cut = 0, heavy = 0, giant = 0, further = 0;
#pragma unroll
                    for (int j = 0; j < kKeysPerSlab; ++j) {
                      if (dy[j] != 0) continue;
                      cut |= 1u << j;
                      if (nb[j] > kGiantBuckets) giant |= 1u << j;
                      else if (nb[j] > kHeavyBuckets) heavy |= 1u << j;
                      else further += nb[j] - 1;
                    }
                    stage_words(S[3], cut, sl);
                    stage_words(S[0], cut & ~(heavy | giant), sl);
                    if (!single) {
                      if (further) atomicAdd(&more, further);
                      stage_words(S[1], heavy, sl);
                      stage_words(S[2], giant, sl);
                    }
                  });
  } while (inner && inner_next(S, list, &more, single, many, nl, step));
  stage_close(S);
}

// Delete prologue, step 3: each invalidated vertex takes the best candidate offered by
// its still-valid in-neighbours (reverse view) and, if reached, joins the frontier.
// Single-bucket vertices are pulled by one lane, up to kHeavyBuckets buckets by a 16-lane
// group, larger ones by a whole block (each group offers its own best; the atomic
// minimum keeps the smallest).
//
// A vertex is listed once, so the lane or group that pulls it is the only writer of its node and
// its mark: plain stores, no exchange.  Its neighbours' loads stay under their own conditions
// here: the kernel is bound by the random accesses of millions of vertices, and the registers of
// 15 loads in flight would halve the waves that hide them (1.46 -> 3.26 ms on the grid).
template <bool kUnit>
__device__ inline uint64_t pull_word(const uint64_t* D, uint64_t x, bool data) {
  const uint32_t u = (uint32_t)x;
  if (!data || !valid_key(u)) return kTreeNone;
  const uint64_t du = ld_u64(D + u);
  if (du == kTreeNone) return kTreeNone;
  return tree_node((du >> 32) + (kUnit ? 1ull : (x >> 32)), u);
}

// A vertex pulled by its only lane or group joins the frontier (distance below T) or the pile.
__device__ inline void push_pulled(Stage (&S)[4], const uint32_t* nbk, const Route& r, uint32_t T, uint32_t* mark,
                                   uint32_t stamp, bool single, uint32_t y, uint64_t best) {
  const bool p = best != kTreeNone, near = p && (uint32_t)(best >> 32) < T;
  if (near) mark[y] = stamp;
  else if (p) r.far_mark[y] = r.band;
  const uint32_t nb = near && !single ? nbk[y] : 1u;
  stage_push(S[3], p && !near, y);
  stage_push(S[0], near && nb <= kHeavyBuckets, y);
  if (!single) {
    stage_push(S[1], near && nb > kHeavyBuckets && nb <= kGiantBuckets, y);
    stage_push(S[2], near && nb > kGiantBuckets, y);
  }
}

template <bool kUnit>
__global__ void __launch_bounds__(kBlock) k_dec_pull(DView F, DView R, uint64_t* D,
                                                     const uint32_t* inval, const uint32_t* inval_cnt,
                                                     PushQ Q, Route r, uint32_t* mark, uint32_t stamp, bool single,
                                                     bool r_single) {
  const uint32_t n = *inval_cnt;
  if ((uint64_t)blockIdx.x * (r_single ? kBlock : 1) >= n) return;
  __shared__ Stage S[4];
  open_routed(S, Q, r);
  const uint32_t T = kUnit ? 0xFFFFFFFFu : band_limit(r);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t y = inval[i];
    uint64_t best = kTreeNone;
    Slab sl;
    load_slab(R, y, sl);
    if ((uint32_t)(sl.w[15] >> 32) != 1) continue;
    while (true) {
      uint64_t c[kKeysPerSlab];
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j) c[j] = pull_word<kUnit>(D, sl.w[j], true);
#pragma unroll
      for (int j = 0; j < kKeysPerSlab; ++j) best = c[j] < best ? c[j] : best;
      const uint32_t t = (uint32_t)sl.w[15];
      if (t == kInvalid) break;
      load_slab(R, t, sl);
    }
    if (best != kTreeNone) __hip_atomic_store(D + y, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    push_pulled(S, F.nbk, r, T, mark, stamp, single, y, best);
  }
  if (!r_single) {
    const uint32_t g0 = (blockIdx.x * kBlock + threadIdx.x) / kGroup;
    const uint32_t ng = gridDim.x * kGroupsPerBlock;
    for (uint32_t i = g0; i < n; i += ng) {
      const uint32_t y = inval[i];
      const uint32_t nb = R.nbk[y];
      if (nb == 1 || nb > kHeavyBuckets) continue;
      uint64_t best = kTreeNone;
      for_each_slab(R, y, [&](uint64_t x, bool data) {
        const uint64_t c = pull_word<kUnit>(D, x, data);
        best = c < best ? c : best;
      });
      best = gmin_u64(best);
      if (glane() != 0) best = kTreeNone;  // lane 0 writes and pushes
      if (best != kTreeNone) __hip_atomic_store(D + y, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      push_pulled(S, F.nbk, r, T, mark, stamp, single, y, best);
    }
    const uint32_t gib = threadIdx.x / kGroup;
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
      const uint32_t y = inval[i];
      if (R.nbk[y] <= kHeavyBuckets) continue;
      uint64_t best = kTreeNone;
      for_each_slab_strided(R, y, gib, kGroupsPerBlock, [&](uint64_t x, bool data) {
        const uint64_t c = pull_word<kUnit>(D, x, data);
        best = c < best ? c : best;
      });
      best = gmin_u64(best);
      bool improve = false;
      if (glane() == 0 && best != kTreeNone) improve = amin64(D + y, best) > best;
      push_staged(S, F.nbk, r, T, mark, stamp, improve, y, (uint32_t)(best >> 32));
    }
  }
  stage_close(S);
}

__global__ void k_fill_mark(uint32_t* mark, uint32_t nv) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) mark[v] = 0;
}

__global__ void k_split(const uint64_t* D, uint32_t nv, uint32_t* dist, uint32_t* parent) {
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint64_t x = D[v];
    dist[v] = (uint32_t)(x >> 32);
    if (parent) parent[v] = (uint32_t)x;
  }
}

inline uint32_t blocks_for(uint64_t n, uint32_t cap = 4096) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + kBlock - 1) / kBlock, cap));
}

// Where a traversal keeps its state: the graph's own arrays for the maintained BFS/SSSP,
// or a caller workspace for a one-off traversal that other reads may overlap.
struct TravCtx {
  uint64_t* D;
  uint32_t* fq[6];  // light, heavy and giant queues, two of each
  uint32_t* mark;
  uint32_t* inval;
  uint32_t* far[2];     // far piles of the weighted epilogue
  uint32_t* far_mark;
  uint32_t* cnt;        // [0..8] rotating frontier sizes, [9..10] pile sizes,
                        // [11..12] band thresholds, [13..14] smallest pile distance, by band
  uint32_t* inval_cnt;  // invalidated-list size
  uint32_t* stamp;      // host-side counter of frontier stamps
  uint32_t* bands;      // host-side counter that numbers the bands
  uint32_t n;           // vertices
  bool single;          // every vertex has one bucket
  bool many;            // the vertices have kManyBuckets or more on average
  uint64_t* h_pin;      // pinned host words for size read-backs
  uint32_t delta;       // band width
};

TravCtx graph_ctx(mk_graph* g, uint64_t* D) {
  TravCtx c;
  c.D = D;
  for (int i = 0; i < 6; ++i) c.fq[i] = g->fq[i];
  c.mark = g->mark;
  c.inval = g->inval;
  c.far[0] = g->far[0];
  c.far[1] = g->far[1];
  c.far_mark = g->far_mark;
  c.cnt = g->ctr->frontier;
  c.inval_cnt = &g->ctr->inval;
  c.stamp = &g->stamp;
  c.bands = &g->bands;
  c.n = g->n;
  c.single = g->view[VF].n_head == g->n;
  c.many = g->view[VF].n_head >= (uint64_t)kManyBuckets * g->n;
  c.h_pin = g->h_pin;
  c.delta = g->sssp_delta;
  return c;
}

// Host-side band state of one weighted traversal: which pile and threshold word are current.
struct Bands {
  int fb = 0, tb = 0;
  uint32_t band = 0;
};

Route route_of(const TravCtx& c, const Bands& b) {
  return Route{c.cnt + 11 + b.tb, c.far[b.fb], c.cnt + 9 + b.fb, c.far_mark, b.band};
}

// Band 0 of a weighted traversal (kUnit == false): threshold 0, so every prologue push
// lands on pile 0.  Unweighted traversals route nothing.
template <bool kUnit>
Route first_route(const TravCtx& c, Bands& b) {
  if (kUnit) return Route{nullptr, nullptr, nullptr, nullptr, 0};
  b = Bands{};
  b.band = ++*c.bands;
  return route_of(c, b);
}

// The queues of iteration 0 (and of every prologue): fq[0], fq[2], fq[4] with slot 0.
PushQ first_push(const TravCtx& c) {
  PushQ Q;
  for (int k = 0; k < 3; ++k) {
    Q.q[k] = c.fq[2 * k];
    Q.c[k] = c.cnt + 3 * k;
  }
  return Q;
}

Queues queues(const TravCtx& c, uint64_t it) {
  Queues q;
  const int a = (int)(it & 1);
  const int inext = (int)((it + 1) % 3);
  for (int k = 0; k < 3; ++k) {
    q.cur[k] = c.fq[2 * k + a];
    q.next.q[k] = c.fq[2 * k + (a ^ 1)];
    q.next.c[k] = c.cnt + 3 * k + inext;
  }
  q.cnt = c.cnt;
  q.icur = (int)(it % 3);
  q.iclear = (int)((it + 2) % 3);
  return q;
}

// The first of `steps` fresh stamps.  Marks only matter within one step, so when the stamps run
// out the marks are cleared and the count starts again.
uint32_t next_stamps(const TravCtx& c, uint32_t steps, hipStream_t stream) {
  if (*c.stamp > 0xFFFFFFFFu - 2 * kInnerSteps) {
    hipLaunchKernelGGL(k_fill_mark, dim3(blocks_for(c.n)), dim3(kBlock), 0, stream, c.mark, c.n);
    *c.stamp = 0;
  }
  const uint32_t first = *c.stamp + 1;
  *c.stamp += steps;
  return first;
}

// Run frontier iterations (expand or propagate) from iteration *it until the frontier is
// empty.  Iteration `it` reads slot it%3; the frontier of iteration 0 sits in fq[0] /
// fq[2] / fq[4] and slot 0.  On return *it is the first iteration with an empty frontier
// and c.h_pin holds the counters read back last.
template <class Launch>
mk_status run_frontier(mk_graph* g, const TravCtx& c, hipStream_t stream, Launch&& launch,
                       uint64_t* it_io = nullptr) {
  uint64_t it = it_io ? *it_io : 0;
  // a small graph's frontiers mostly end inside one launch (kInnerSteps), unless they hold many buckets
  int every = c.n <= kSmallGraph && !c.many ? kSyncFirst / 2 : kSyncFirst;
  for (;; every = every < kSyncMax ? 2 * every : kSyncMax) {
    for (int k = 0; k < every; ++k, ++it) {
      launch(queues(c, it), next_stamps(c, kInnerSteps, stream));
      MK_LAUNCH(g, "frontier kernel");
    }
    const int slot = (int)(it % 3);
    read_back(c.cnt, c.h_pin, 14, stream);
    MK_HIP(g, hipStreamSynchronize(stream));
    const volatile uint32_t* h = reinterpret_cast<const volatile uint32_t*>(c.h_pin);
    if (h[slot] == 0 && h[3 + slot] == 0 && h[6 + slot] == 0) break;
  }
  if (it_io) *it_io = it;
  return MK_OK;
}

constexpr uint32_t kBandBlocks = 1024;

// Frontier epilogue.  Unweighted: expand until the frontier is empty.  Weighted: band by
// band; each band step moves the next band of the far pile into the (empty) frontier of
// the current iteration, then the band is expanded until its frontier is empty.
template <bool kUnit>
mk_status run_expand(mk_graph* g, const TravCtx& c, hipStream_t stream, Bands& b) {
  const DView F = g->view[VF].d;
  if (kUnit) {
    const Route r{nullptr, nullptr, nullptr, nullptr, 0};
    return run_frontier(g, c, stream, [&](Queues q, uint32_t stamp) {
      hipLaunchKernelGGL(k_expand<kUnit>, dim3(kExpandBlocks), dim3(kBlock), 0, stream, F, c.D, q, r,
                         c.mark, stamp, c.single, c.many);
    });
  }
  uint64_t it = 0;
  for (uint32_t k = 0;; ++k) {
    const int nf = b.fb ^ 1, nt = b.tb ^ 1;
    const uint32_t band_next = ++*c.bands;
    uint32_t *fmin = c.cnt + 13 + (k & 1), *fmin_next = c.cnt + 13 + (~k & 1);
    hipLaunchKernelGGL(k_band_min, dim3(kBandBlocks), dim3(kBlock), 0, stream, c.D, c.far[b.fb],
                       c.cnt + 9 + b.fb, c.cnt + 11 + b.tb, fmin, c.cnt + 9 + nf);
    PushQ cur;
    for (int k = 0; k < 3; ++k) {
      cur.q[k] = c.fq[2 * k + (int)(it & 1)];
      cur.c[k] = c.cnt + 3 * k + (int)(it % 3);
    }
    hipLaunchKernelGGL(k_band_split, dim3(kBandBlocks), dim3(kBlock), 0, stream, F.nbk, c.D, c.far[b.fb],
                       c.cnt + 9 + b.fb, c.cnt + 11 + b.tb, fmin, fmin_next, c.delta, c.cnt + 11 + nt, cur, c.far[nf],
                       c.cnt + 9 + nf, c.far_mark, band_next, c.single);
    MK_LAUNCH(g, "band step");
    b.fb = nf;
    b.tb = nt;
    b.band = band_next;
    const Route r = route_of(c, b);
    mk_status s = run_frontier(g, c, stream, [&](Queues q, uint32_t stamp) {
      hipLaunchKernelGGL(k_expand<kUnit>, dim3(kExpandBlocks), dim3(kBlock), 0, stream, F, c.D, q, r,
                         c.mark, stamp, c.single, c.many);
    }, &it);
    if (s != MK_OK) return s;
    const volatile uint32_t* h = reinterpret_cast<const volatile uint32_t*>(c.h_pin);
    if (h[9 + b.fb] == 0) break;  // the frontier and the pile are both empty
  }
  return MK_OK;
}

template <bool kUnit>
mk_status static_from(mk_graph* g, const TravCtx& c, uint32_t source, hipStream_t stream) {
  const DView F = g->view[VF].d;
  const uint32_t stamp0 = next_stamps(c, 1, stream);
  hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, stream, c.cnt, c.inval_cnt);
  hipLaunchKernelGGL(k_trav_init, dim3(blocks_for(g->n)), dim3(kBlock), 0, stream, c.D, g->n, source);
  Bands b;
  const Route r0 = first_route<kUnit>(c, b);
  hipLaunchKernelGGL(k_seed_source, dim3(1), dim3(64), 0, stream, F, source, first_push(c), r0, c.mark,
                     stamp0);
  MK_LAUNCH(g, "traversal init");
  return run_expand<kUnit>(g, c, stream, b);
}

template <bool kUnit>
mk_status traverse(mk_graph* g, AlgoState& st, uint64_t* D, uint32_t source, uint32_t* d_out,
                   uint32_t* d_parent, mk_mode mode, hipStream_t stream) {
  if (source >= g->n || !d_out) return MK_ERR_INVALID_ARG;
  const DView F = g->view[VF].d;
  const uint32_t N = g->n;
  const TravCtx c = graph_ctx(g, D);
  Pending p = pending_for(g, st);
  const bool can_dec = g->view[VR].on;
  bool full = mode == MK_RECOMPUTE || !st.valid || st.source != source || p.lost ||
              p.kinds == 3 || (p.kinds == 2 && !can_dec);
  if (!full && mode == MK_AUTO) {  // the cost model, when one is set, may prefer a recompute
    mk_status s = auto_prefers_recompute(g, kUnit ? MK_ALGO_BFS : MK_ALGO_SSSP, p, stream, &full);
    if (s != MK_OK) return s;
  }
  if (full) {
    // A graph with the reverse view and a mean out-degree of at least 8: distances first
    // (direction-optimizing BFS levels, or the distance-only SSSP), then every vertex's
    // parent from its in-arcs.  On sparser graphs (a road network) the tree traversal in
    // one pass beats distances plus parents.
    const bool by_dist = can_dec && g->m0 >= 8ull * N;
    mk_status s = !by_dist ? static_from<kUnit>(g, c, source, stream)
                  : kUnit  ? bfs_tree_by_levels(g, source, d_out, D, stream)
                           : sssp_tree_by_distances(g, source, d_out, D, stream);
    if (s != MK_OK) return s;
  } else if (!p.list.empty()) {
    const uint32_t stamp0 = next_stamps(c, 1, stream);
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, stream, c.cnt, c.inval_cnt);
    Bands bands;
    if (p.kinds == 1) {
      const Route r0 = first_route<kUnit>(c, bands);
      for (const BatchRec* b : p.list) {
        Log lg = g->log;
        lg.s += b->off; lg.d += b->off; lg.w += b->off; lg.st += b->off; lg.uf += b->off;
        hipLaunchKernelGGL(k_relax_batch<kUnit>, dim3(blocks_for(b->n)), dim3(kBlock), 0, stream, F, D,
                           lg, b->n, first_push(c), r0, c.mark, stamp0);
      }
    } else {  // deletions only
      for (const BatchRec* b : p.list) {
        Log lg = g->log;
        lg.s += b->off; lg.d += b->off; lg.w += b->off; lg.st += b->off; lg.uf += b->off;
        hipLaunchKernelGGL(k_invalidate, dim3(blocks_for(b->n)), dim3(kBlock), 0, stream, F, D, lg, b->n,
                           first_push(c), c.inval, c.inval_cnt);
      }
      MK_LAUNCH(g, "k_invalidate");
      mk_status s = run_frontier(g, c, stream, [&](Queues q, uint32_t stamp) {
        hipLaunchKernelGGL(k_propagate, dim3(kExpandBlocks), dim3(kBlock), 0, stream, F, D, q, c.inval,
                           c.inval_cnt, c.single, c.many);
      });
      if (s != MK_OK) return s;
      hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, stream, c.cnt, nullptr);
      const uint32_t stamp1 = next_stamps(c, 1, stream);
      const Route r0 = first_route<kUnit>(c, bands);
      hipLaunchKernelGGL(k_dec_pull<kUnit>, dim3(kExpandBlocks), dim3(kBlock), 0, stream, F,
                         g->view[VR].d, D, c.inval, c.inval_cnt, first_push(c), r0, c.mark, stamp1, c.single,
                         g->view[VR].n_head == N);
    }
    MK_LAUNCH(g, "traversal prologue");
    mk_status s = run_expand<kUnit>(g, c, stream, bands);
    if (s != MK_OK) return s;
  }
  hipLaunchKernelGGL(k_split, dim3(blocks_for(N)), dim3(kBlock), 0, stream, D, N, d_out, d_parent);
  MK_LAUNCH(g, "k_split");
  st.valid = true;
  st.source = source;
  mark_seen(g, st);
  return MK_OK;
}

size_t ws_bytes_for(uint32_t n) {
  // D (8 B); six queues, stamps, the invalidated list, two far piles and the band marks
  // (4 B each); counters; 256-byte alignment of each of the 13 regions
  return (size_t)n * (8 + 11 * 4) + 128 + 14 * 256;
}

}  // namespace

extern "C" {

mk_status mk_incr_bfs(mk_graph* g, uint32_t source, uint32_t* d_level, uint32_t* d_parent,
                      mk_mode mode, hipStream_t stream) {
  if (!g) return MK_ERR_INVALID_ARG;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  return traverse<true>(g, g->bfs, g->bfs_D, source, d_level, d_parent, mode, stream);
}

mk_status mk_incr_sssp(mk_graph* g, uint32_t source, uint32_t* d_dist, uint32_t* d_parent,
                       mk_mode mode, hipStream_t stream) {
  if (!g) return MK_ERR_INVALID_ARG;
  if (mk_status gs = graph_guard(g); gs != MK_OK) return gs;
  return traverse<false>(g, g->sssp, g->sssp_D, source, d_dist, d_parent, mode, stream);
}

size_t mk_traversal_workspace_bytes(const mk_graph* g) { return g ? ws_bytes_for(g->n) : 0; }

mk_status mk_traverse_from(mk_graph* g, uint32_t source, int weighted, void* d_ws, size_t ws_bytes,
                           uint32_t slot, uint32_t* d_dist, uint32_t* d_parent, hipStream_t stream) {
  if (!g || !d_ws || !d_dist || source >= g->n || slot >= kSlots) return MK_ERR_INVALID_ARG;
  if (ws_bytes < ws_bytes_for(g->n)) return MK_ERR_CAPACITY;
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
  TravCtx c;
  c.D = reinterpret_cast<uint64_t*>(take((size_t)N * 8));
  for (int i = 0; i < 6; ++i) c.fq[i] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.mark = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.inval = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.far[0] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.far[1] = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.far_mark = reinterpret_cast<uint32_t*>(take((size_t)N * 4));
  c.cnt = reinterpret_cast<uint32_t*>(take(128));
  c.inval_cnt = c.cnt + 16;
  uint32_t stamp = 0, bands = 0;
  c.stamp = &stamp;
  c.bands = &bands;
  c.n = N;
  c.single = g->view[VF].n_head == N;
  c.many = g->view[VF].n_head >= (uint64_t)kManyBuckets * N;
  c.h_pin = g->slot_pin[slot];
  c.delta = g->sssp_delta;
  hipLaunchKernelGGL(k_fill_mark, dim3(blocks_for(N)), dim3(kBlock), 0, stream, c.mark, N);
  hipLaunchKernelGGL(k_fill_mark, dim3(blocks_for(N)), dim3(kBlock), 0, stream, c.far_mark, N);
  mk_status s = weighted ? static_from<false>(g, c, source, stream) : static_from<true>(g, c, source, stream);
  if (s != MK_OK) return s;
  hipLaunchKernelGGL(k_split, dim3(blocks_for(N)), dim3(kBlock), 0, stream, c.D, N, d_dist, d_parent);
  MK_LAUNCH(g, "k_split");
  return MK_OK;
}

}  // extern "C"
