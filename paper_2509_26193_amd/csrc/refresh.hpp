// Vacancy refresh (Sec. III-B, "Division of work"): the leaves and the inner nodes bottom-up,
// by chunks of the tree (see chunks_k).
// A leaf takes its neuron's count (its position stays in its record); an inner node the
// sum of its children's counts and the count-weighted mean of their centroids, accumulated
// in float64 left to right in octant order with one rounding per operation (the
// library is compiled without FP contraction, so no product is fused into a sum).
#pragma once

#include "build.hpp"

namespace msp {

constexpr int kRefreshBlock = 256;

struct Acc3 {
  int64_t v = 0;
  double x = 0.0, y = 0.0, z = 0.0;
  __device__ __forceinline__ void add(int64_t vk, double cx, double cy, double cz) {
    v += vk;
    if (vk > 0) {
      const double w = (double)vk;
      x = x + w * cx;
      y = y + w * cy;
      z = z + w * cz;
    }
  }
  __device__ __forceinline__ void store(NodeRec& r, int32_t* err) const {
    if (v > 0x7FFFFFFF) atomicOr(err, kErrOverflow);
    r.v = (int32_t)v;
    if (v > 0) {
      const double d = (double)v;
      r.x = x / d;
      r.y = y / d;
      r.z = z / d;
    } else {
      r.x = r.y = r.z = 0.0;
    }
  }
};

// The inner node x with meta word `meta` from its children (ascending, -1: none), after every
// deeper node below it. The children's records are loaded four at a time, not one after
// the other as their subtree ends lead from one to the next.
__device__ __forceinline__ void refresh_node(int32_t x, uint32_t meta, const int32_t (&kids)[8],
                                             NodeRec* r0, NodeRec* r1, int32_t* err) {
  Acc3 A, B;
#pragma unroll
  for (int k = 0; k < 8; k += 4) {
    if (kids[k] < 0) break;
    NodeRec a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t c = kids[k + q] < 0 ? kids[k] : kids[k + q];
      a[q] = r0[c];
      b[q] = r1[c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (kids[k + q] < 0) break;
      A.add(a[q].v, a[q].x, a[q].y, a[q].z);
      B.add(b[q].v, b[q].x, b[q].y, b[q].z);
    }
  }
  NodeRec e, f;
  e.meta = f.meta = meta;
  A.store(e, err);
  B.store(f, err);
  r0[x] = e;
  r1[x] = f;
}

// The subtree ends of a chunk's nodes in LDS (those past `room` stay in global memory), and the
// children of its inner nodes found through them.
constexpr int kSkipRoomOne = kNodesOne;    // trees of one chunk
constexpr int kSkipRoom = 2048;            // (with 32 KB of LDS a block of 512 threads leaves
                                           // a CU's wavefronts short)

struct ChunkSkips {
  const int32_t* lds;
  const int32_t* skip;
  int32_t x0, room;
  __device__ __forceinline__ int32_t operator()(int32_t x) const {
    return x - x0 < room ? lds[x - x0] : skip[x];
  }
  __device__ __forceinline__ void kids(int32_t x, int32_t end, int32_t (&k)[8]) const {
    int32_t c = x + 1;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool in = c < end;
      k[q] = in ? c : -1;
      if (in) c = (*this)(c);
    }
  }
};

// The octree's chunks, as the kernels read them.
struct Chunks {
  int32_t log, nch, nsup;
  const int32_t* x;
  const int32_t* off;
  const int32_t* nodes;
  const int32_t* cross;
  const int32_t* cross2;
  const int32_t* cross_kids;
  const int32_t* cross2_kids;
  const int32_t* skip;
};

inline Chunks chunks_of(const msp_octree_s* t) {
  return Chunks{t->chunk_log, t->nch, t->nsup, t->chunk_x, t->chunk_off, t->chunk_nodes,
                t->cross, t->cross2, t->cross_kids, t->cross2_kids, t->skip};
}

// The node of depth d that crosses the end of chunk (or run) c, with its children.
struct CrossNode {
  int32_t x, kids[8];
  __device__ __forceinline__ CrossNode(const int32_t* cross, const int32_t* kids_of, int count,
                                       int c, int d) {
    const int64_t at = (int64_t)d * count + (c < count ? c : 0);
    x = c < count ? cross[at] : -1;
#pragma unroll
    for (int k = 0; k < 8; ++k) kids[k] = kids_of[8 * at + k];
  }
};

// Both types' counts by id side by side, for the refresh of a tree of more than kPairMin neurons:
// its gathers by id then fetch one line per neuron instead of two (8M neurons: 0.84 ms for the
// chunks without, 0.81 with). Smaller trees' counts stay in the L2 caches.
constexpr int64_t kPairMin = (int64_t)1 << 18;

__global__ void pair_counts_k(const int32_t* __restrict__ vexc, const int32_t* __restrict__ vinh,
                              int64_t n, int2* __restrict__ both) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) both[i] = make_int2(vexc[i], vinh[i]);
}

// A bucket's members are consecutive: every lane forms its neuron's terms, and the wave that has
// the first member adds them up in order, from lane to lane (8M neurons in cells of 64: 2.90 ->
// 0.86 ms, where one thread loaded one member after the other; in cells of 2: 5.88
// -> 5.71).
__device__ __forceinline__ void bucket_terms(int2 w, const double* __restrict__ pos, int32_t i,
                                             double (&d)[6]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double c = pos[3 * (int64_t)i + a];
    d[a] = w.x > 0 ? (double)w.x * c : -0.0;       // (-0.0 leaves any sum as it is)
    d[3 + a] = w.y > 0 ? (double)w.y * c : -0.0;
  }
}

// Lane k's value, in every lane.
__device__ __forceinline__ double lane_f64(double v, int k) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, k);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), k);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ void bucket_add(Acc3& A, Acc3& B, int2 w, const double (&d)[6], int from,
                                           int to) {
  for (int k = from; k < to; ++k) {
    A.v += __builtin_amdgcn_readlane(w.x, k);
    B.v += __builtin_amdgcn_readlane(w.y, k);
    A.x = A.x + lane_f64(d[0], k);
    A.y = A.y + lane_f64(d[1], k);
    A.z = A.z + lane_f64(d[2], k);
    B.x = B.x + lane_f64(d[3], k);
    B.y = B.y + lane_f64(d[4], k);
    B.z = B.z + lane_f64(d[5], k);
  }
}

// One block per chunk: its leaves (the caller's vacancy arrays are gathered by id; a bucket
// leaf is done by its first member's wave, its members in sorted order, which is id order
// within the finest cell), then its inner nodes by depth, deepest first. Bound by the
// gathers (a 128-byte line for 8 bytes per neuron) and the records read and written; small
// trees by the chain over the depths. The whole refresh, against a kernel for the leaves and
// one per depth: 8M neurons 0.88 ms (1.39), 2M 0.30 (0.37), 4 096 47 us in one launch (41 us
// in nine, and 22 us for the lists of the depths). A thread's neurons, and its first node of
// the next depth, are loaded together and ahead: 8M 0.81 -> 0.75 ms for the chunks.
template <bool PAIRS, bool ONE>
__global__ void __launch_bounds__(ONE ? 1024 : 512) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : 6)))
refresh_chunk_k(
    int64_t n, Chunks C, NodeRec* r0, NodeRec* r1, const int32_t* __restrict__ leaf_at,
    const int32_t* __restrict__ order, const double* __restrict__ pos,
    const int32_t* __restrict__ vexc, const int32_t* __restrict__ vinh,
    const int2* __restrict__ both, int32_t* __restrict__ vs0, int32_t* __restrict__ vs1,
    int32_t* err) {
  constexpr int kRoom = ONE ? kSkipRoomOne : kSkipRoom;
  constexpr int kAtOnce = ONE ? 4 : 2;             // a thread's neurons, loaded together
  __shared__ int32_t skips[kRoom];
  __shared__ int32_t off[kDepths + 1];
  const int c = (int)blockIdx.x, t = (int)threadIdx.x, threads = (int)blockDim.x;
  const int32_t x0 = C.x[c], x1 = C.x[c + 1];
  if (t <= kDepths) off[t] = C.off[(int64_t)c * (kDepths + 1) + t];
  for (int32_t x = x0 + t; x < x1 && x - x0 < kRoom; x += threads) skips[x - x0] = C.skip[x];
  const ChunkSkips S{skips, C.skip, x0, kRoom};
  auto load = [&](int32_t id) -> int2 {
    return PAIRS ? both[id] : make_int2(vexc[id], vinh[id]);
  };
  auto checked = [&](int2 v) -> int2 {
    if (v.x < 0 || v.y < 0) atomicOr(err, kErrNegative);
    return make_int2(v.x < 0 ? 0 : v.x, v.y < 0 ? 0 : v.y);
  };
  const int lane = t & (kWave - 1);
  const int64_t p0 = (int64_t)c << C.log;
  const int64_t p1 = p0 + ((int64_t)1 << C.log) < n ? p0 + ((int64_t)1 << C.log) : n;
  // (every wave takes its whole turns: its lanes add up buckets together)
  for (int64_t b = p0 + t; b - lane < p1; b += kAtOnce * threads) {
    int32_t at[kAtOnce], before[kAtOnce], after[kAtOnce], id[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int64_t p = b + u * threads < p1 ? b + u * threads : p1 - 1;
      at[u] = leaf_at[p];
      before[u] = p > 0 ? leaf_at[p - 1] : -1;
      after[u] = p + 1 < n ? leaf_at[p + 1] : -1;
      id[u] = order[p];
    }
    int2 v[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) v[u] = load(id[u]);
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) asm volatile("" : "+v"(v[u].x), "+v"(v[u].y));
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int64_t p = b + u * threads;
      const int32_t x = at[u];
      const bool mine = p < p1;
      const bool member = mine && (before[u] == x || after[u] == x);       // of a bucket
      if (mine && !member) {
        const int2 w = checked(v[u]);
        r0[x].v = w.x;
        r1[x].v = w.y;
      }
      if (!__any(member)) continue;
      int2 w = make_int2(0, 0);
      double d[6];
      if (member) {
        w = checked(v[u]);
        vs0[p] = w.x;
        vs1[p] = w.y;
        bucket_terms(w, pos, id[u], d);
      }
      const bool head = member && before[u] != x;
      const int last = __popcll(__ballot(mine)) - 1;
      int64_t sum0 = 0, sum1 = 0;                  // a head's counts (its sums: in d)
      for (uint64_t left = __ballot(head); left; left &= left - 1) {       // (uniform)
        const int from = __ffsll((unsigned long long)left) - 1;
        const int32_t xb = __builtin_amdgcn_readlane(x, from);
        Acc3 A, B;
        int to = from + __popcll(__ballot(mine && x == xb));
        bucket_add(A, B, w, d, from, to);
        // those past the wave's neurons
        for (int64_t q0 = p - lane + last + 1; to == last + 1 || to == kWave; q0 += kWave) {
          const int64_t q = q0 + lane;
          const bool more = q < n && leaf_at[q < n ? q : p0] == xb;
          int2 w2 = make_int2(0, 0);
          double d2[6];
          if (more) {
            const int32_t i = order[q];
            w2 = load(i);
            w2 = make_int2(w2.x < 0 ? 0 : w2.x, w2.y < 0 ? 0 : w2.y);
            bucket_terms(w2, pos, i, d2);
          }
          to = __popcll(__ballot(more));
          if (to == 0) break;
          bucket_add(A, B, w2, d2, 0, to);
          if (to < kWave) break;
        }
        if (lane == from) {
          sum0 = A.v;
          sum1 = B.v;
          d[0] = A.x;
          d[1] = A.y;
          d[2] = A.z;
          d[3] = B.x;
          d[4] = B.y;
          d[5] = B.z;
        }
      }
      if (head) {
        Acc3 A, B;
        A.v = sum0;
        A.x = d[0];
        A.y = d[1];
        A.z = d[2];
        B.v = sum1;
        B.x = d[3];
        B.y = d[4];
        B.z = d[5];
        NodeRec e, f;
        e.meta = f.meta = kLeafBit | kBucketBit | (uint32_t)x;
        A.store(e, err);
        B.store(f, err);
        r0[x] = e;
        r1[x] = f;
      }
    }
  }
  // the lists of the depths follow one another: a thread's first node of the next depth is
  // loaded ahead of the barrier
  const int32_t* nodes = C.nodes + x0;
  __syncthreads();
  const int32_t all = off[kDepths];
  int32_t lo = 0, next = t < all ? nodes[t] : 0;
  for (int k = 1; k <= kDepths; ++k) {             // depth kMaxDepth + 1 - k
    const int32_t hi = off[k];
    if (hi == lo) continue;                        // (uniform over the block)
    int32_t x = next;
    next = hi + t < all ? nodes[hi + t] : 0;
    for (int32_t q = lo + t; q < hi; q += threads) {
      if (q != lo + t) x = nodes[q];
      const int32_t end = S(x);
      int32_t kids[8];
      S.kids(x, end, kids);
      refresh_node(x, (uint32_t)end | ((uint32_t)(kMaxDepth + 1 - k) << kSkipBits), kids, r0, r1,
                   err);
    }
    lo = hi;
    __syncthreads();
  }
}

// The depths (bit d: depth d) at which a thread of the block has a crossing node.
__device__ __forceinline__ uint32_t cross_depths(const int32_t* cross, int count, int c,
                                                 uint32_t* lds) {
  if (threadIdx.x == 0) *lds = 0;
  uint32_t mine = 0;
#pragma unroll
  for (int d = 0; d < kDepths; ++d)
    if (c < count && cross[(int64_t)d * count + c] >= 0) mine |= 1u << d;
  __syncthreads();
  if (mine) atomicOr(lds, mine);
  __syncthreads();
  return *lds;
}

// One block per run of kSuper chunks, a chunk per thread: the nodes that cross chunk ends
// inside the run, by depth; with cross2 (one block, a run per thread) those that cross the
// ends of runs. Bound by the chain over the depths (a barrier and the children's records
// each), so only depths with such nodes are visited, and the next one's nodes and children
// are loaded ahead of the barrier (20 011 neurons: 28 -> 25 us).
constexpr int kCross2Block = 512;          // runs of a tree of kMaxNodes neurons

__global__ void __launch_bounds__(kCross2Block) refresh_cross_k(
    const int32_t* __restrict__ cross, const int32_t* __restrict__ kids_of,
    const int32_t* __restrict__ skip, int count, NodeRec* r0, NodeRec* r1, int32_t* err) {
  __shared__ uint32_t depths;
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  uint32_t left = cross_depths(cross, count, c, &depths);
  if (left == 0) return;
  int d = 31 - __clz(left);
  CrossNode next(cross, kids_of, count, c, d);
  while (left) {
    const CrossNode at = next;
    const int here = d;
    left &= ~(1u << d);
    if (left) {
      d = 31 - __clz(left);
      next = CrossNode(cross, kids_of, count, c, d);
    }
    if (at.x >= 0)
      refresh_node(at.x, (uint32_t)skip[at.x] | ((uint32_t)here << kSkipBits), at.kids, r0, r1,
                   err);
    __syncthreads();
  }
}

}  // namespace msp
