// Octree construction (Sec. III-B, "Spatial octree"): Morton keys, sort, and the
// node topology in depth-first pre-order, derived from adjacent common prefixes.
#pragma once

#include "common.hpp"
#include "scan.hpp"

namespace msp {

constexpr int kBuildBlock = 256;

// Quantise each axis to 21 bits and interleave: digit k (1..21, most significant
// first) = 4*x_bit + 2*y_bit + z_bit of bit (21-k). Non-finite positions raise a flag.
__device__ __forceinline__ uint64_t spread3(uint64_t v) {   // 21 bits -> every third bit
  v &= 0x1FFFFFull;
  v = (v | (v << 32)) & 0x1F00000000FFFFull;
  v = (v | (v << 16)) & 0x1F0000FF0000FFull;
  v = (v | (v << 8)) & 0x100F00F00F00F00Full;
  v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

__device__ __forceinline__ uint64_t quantise(double x, double lo, double edge) {
  double f = floor(((x - lo) / edge) * 2097152.0);
  f = (f >= 0.0) ? f : 0.0;
  f = (f > 2097151.0) ? 2097151.0 : f;
  return (uint64_t)f;
}

__global__ void __launch_bounds__(kBuildBlock) keys_k(const double* __restrict__ pos_in, int64_t n,
                                                     double x0, double y0, double z0, double edge,
                                                     double* __restrict__ pos, uint64_t* keys,
                                                     int32_t* ids, int32_t* err,
                                                     int32_t* outside) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = pos_in[3 * i + 0], y = pos_in[3 * i + 1], z = pos_in[3 * i + 2];
  if (!isfinite(x) || !isfinite(y) || !isfinite(z)) atomicOr(err, kErrNonFinite);
  // a position outside the closed cube (it is clamped into an edge cell); one atomic
  // per wave at most
  const bool out = !(x >= x0 && x <= x0 + edge && y >= y0 && y <= y0 + edge && z >= z0 &&
                     z <= z0 + edge);
  const uint64_t outs = __ballot(out);
  if (outs && (threadIdx.x & 63) == (unsigned)(__ffsll((unsigned long long)outs) - 1))
    atomicOr(outside, 1);
  pos[3 * i + 0] = x;
  pos[3 * i + 1] = y;
  pos[3 * i + 2] = z;
  const uint64_t qx = quantise(x, x0, edge), qy = quantise(y, y0, edge), qz = quantise(z, z0, edge);
  keys[i] = (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
  ids[i] = (int32_t)i;
}

// Number of equal leading octant digits of two 63-bit keys (21 if equal).
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  if (x == 0) return kMaxDepth;
  return (__clzll((long long)x) - 1) / 3;
}

// The keys are sorted by their leading kLeadBits bits; neurons that share them (few, unless
// they lie within a 2^-10 of the cube's edge of one another in many) are then put in order
// by the whole key, run by run of equal leading bits: half the passes of the sort (0.8 -> 0.4
// ms at 8M neurons). A run of more than kRunMax neurons is left as it is; where that is out of
// order, node_count_k reports it, and the keys are sorted once more by all the bits that
// differ. (The build of 8M neurons with one sort of whole keys -> here: uniform 1.95 -> 1.52 ms;
// in groups of twenty within 10^-4 of the edge 2.28 -> 1.92; all within 2^-11 of it 1.97 -> 1.97,
// eight passes either way; half of them within 2^-12, the rest anywhere 1.94 -> 2.30, twelve.)
constexpr int kLeadBits = 32;
constexpr int kLeadShift = 63 - kLeadBits;
constexpr int kRunMax = 128;
static_assert(kRunMax <= kBuildBlock, "a thread takes at most two neurons of a window");

// A window of consecutive keys in LDS: a block's, the one before them and the kRunMax after; and
// the bits of those whose leading bits differ from the one before.
constexpr int kRunWindow = kBuildBlock + kRunMax + 1;

struct RunWindow {
  static constexpr int kWords = (kRunWindow + kWave - 1) / kWave;
  static constexpr int kEach = (kWords * kWave + kBuildBlock - 1) / kBuildBlock;
  uint64_t key[kRunWindow];
  uint64_t first[kEach * kBuildBlock / kWave];

  // Keys b0, b0 + 1, ... of n (past either end: leading bits that no key has); synchronises.
  __device__ __forceinline__ void load(const uint64_t* keys, int64_t b0, int64_t n) {
    for (int q = (int)threadIdx.x; q < kRunWindow; q += kBuildBlock) {
      const int64_t p = b0 + q;
      key[q] = p >= 0 && p < n ? keys[p] : ~0ull;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int q = (int)threadIdx.x + u * kBuildBlock;
      const uint64_t b = __ballot(q == 0 || q >= kRunWindow ||
                                  key[q] >> kLeadShift != key[q - 1] >> kLeadShift);
      if ((threadIdx.x & (kWave - 1)) == 0) first[q / kWave] = b;
    }
    __syncthreads();
  }
  // The run around entry `at`: [a, e) as far as the window goes.
  __device__ __forceinline__ void run(int at, int& a, int& e) const {
    int w = at / kWave;
    uint64_t b = first[w] & (~0ull >> (kWave - 1 - at % kWave));
    while (b == 0) b = first[--w];                 // (entry 0's bit is set)
    a = w * kWave + kWave - 1 - __clzll((long long)b);
    w = (at + 1) / kWave;
    b = w < kWords ? first[w] & (~0ull << ((at + 1) % kWave)) : 0;
    while (b == 0 && ++w < kWords) b = first[w];
    e = b == 0 ? kRunWindow : w * kWave + __ffsll((unsigned long long)b) - 1;
    e = e < kRunWindow ? e : kRunWindow;
  }
};

// Every neuron of a run of up to kRunMax to its place in it. A block takes the runs that begin
// among its kBuildBlock neurons, from a window of their keys and the next kRunMax (other
// blocks' stores change no leading bits, and no key of these runs). Bound by reading the keys
// (8M neurons in runs of 20: 2.6 ms with a thread per run that inserted in global memory).
__global__ void __launch_bounds__(kBuildBlock) order_runs_k(uint64_t* __restrict__ keys,
                                                           int32_t* __restrict__ ids, int64_t n) {
  __shared__ RunWindow win;
  const int64_t b0 = (int64_t)blockIdx.x * kBuildBlock - 1;
  win.load(keys, b0, n);
  int64_t to[2] = {-1, -1};
  uint64_t key[2];
  int32_t id[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int at = 1 + (int)threadIdx.x + u * kBuildBlock;
    if (at >= kRunWindow || b0 + at >= n) continue;
    int a, e;
    win.run(at, a, e);
    // (a == 0: begins before the block)
    if (e - a < 2 || e - a > kRunMax || a < 1 || a > kBuildBlock) continue;
    key[u] = win.key[at];
    int place = a;                                      // stable: in the order of the ids
    for (int q = a; q < e; ++q)
      place += win.key[q] < key[u] || (win.key[q] == key[u] && q < at) ? 1 : 0;
    if (place == at) continue;
    to[u] = b0 + place;
    id[u] = ids[b0 + at];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    if (to[u] < 0) continue;
    keys[to[u]] = key[u];
    ids[to[u]] = id[u];
  }
}

// Node (start m, depth k) exists for k in [k_lo(m), k_hi(m)] with
// k_lo = cl + 1 and k_hi = min(21, max(cl, cr) + 1), where cl / cr are the common digit
// counts with the left / right neighbour in sorted order (-1 at the ends). Pre-order
// numbering: node index = (nodes starting before m) + (k - k_lo).
__global__ void __launch_bounds__(kBuildBlock) node_count_k(const uint64_t* __restrict__ keys,
                                                           int64_t n, int32_t* cnt,
                                                           int32_t* unsorted) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n) return;
  if (m > 0 && keys[m - 1] > keys[m]) *unsorted = 1;     // (every writer writes the same)
  const int cl = m == 0 ? -1 : common_digits(keys[m - 1], keys[m]);
  const int cr = m == n - 1 ? -1 : common_digits(keys[m], keys[m + 1]);
  const int klo = cl + 1;
  const int khi = min(kMaxDepth, max(cl, cr) + 1);
  cnt[m] = khi >= klo ? khi - klo + 1 : 0;
}

__device__ __forceinline__ uint64_t prefix_of(uint64_t key, int k) {
  return k == 0 ? 0ull : key >> (3 * (kMaxDepth - k));
}

// The nodes that start at sorted neuron m, one thread per m: topology, search records
// (an inner node's meta word holds its subtree end and depth, a leaf's its neuron, a
// bucket leaf's its own index; counts start at 0; a leaf's position stays as it is) and the
// record after the last. The block's keys and the next ones lie in LDS, where most
// cells end (a cell's end is galloped for, then bisected). Bound by its gathers and scatters
// by id and by the records written (64 B per node): 8M neurons 0.80 ms, where one kernel for
// the topology (every probe a dependent load) and one for the records took 0.70 ms and left
// the positions' gather to every refresh.
constexpr int kKeyWindow = 4 * kBuildBlock;

__global__ void __launch_bounds__(kBuildBlock) nodes_k(
    const uint64_t* __restrict__ keys, const int32_t* __restrict__ order,
    const double* __restrict__ pos, int64_t n, const int32_t* __restrict__ base, int32_t* skip,
    uint8_t* depth, int32_t* nbeg, int32_t* nend, int32_t* leaf_of, int32_t* leaf_at, NodeRec* r0,
    NodeRec* r1) {
  __shared__ uint64_t win[kKeyWindow];
  const int64_t m0 = (int64_t)blockIdx.x * kBuildBlock;
#pragma unroll
  for (int q = 0; q < kKeyWindow / kBuildBlock; ++q) {
    const int64_t i = m0 + q * kBuildBlock + threadIdx.x;
    win[q * kBuildBlock + threadIdx.x] = i < n ? keys[i] : 0ull;
  }
  __syncthreads();
  const int64_t m = m0 + threadIdx.x;
  if (m >= n) return;
  auto key = [&](int64_t i) -> uint64_t { return i < m0 + kKeyWindow ? win[i - m0] : keys[i]; };
  const uint64_t km = win[threadIdx.x];
  const int cl = m == 0 ? -1 : common_digits(threadIdx.x ? win[threadIdx.x - 1] : keys[m - 1], km);
  const int cr = m == n - 1 ? -1 : common_digits(km, key(m + 1));
  const int klo = cl + 1;
  const int khi = min(kMaxDepth, max(cl, cr) + 1);
  NodeRec r;
  r.v = 0;
  if (m == n - 1) {                      // the record after the last node
    r.x = r.y = r.z = 0.0;
    r.meta = 0;
    r0[base[n]] = r;
    r1[base[n]] = r;
  }
  if (khi < klo) return;
  int64_t end = m + 1;              // ranges grow as the depth decreases
  for (int k = khi; k >= klo; --k) {
    int64_t e;
    if (k == 0) {
      e = n;
    } else {
      const uint64_t P = prefix_of(km, k);
      if (end >= n || prefix_of(key(end), k) != P) {
        e = end;
      } else {                     // gallop then bisect for the first key outside the cell
        int64_t lo = end, step = 1;
        while (lo + step < n && prefix_of(key(lo + step), k) == P) {
          lo += step;
          step <<= 1;
        }
        int64_t hi = lo + step < n ? lo + step : n;
        while (hi - lo > 1) {
          const int64_t mid = lo + (hi - lo) / 2;
          if (prefix_of(key(mid), k) == P) lo = mid; else hi = mid;
        }
        e = hi;
      }
    }
    end = e;
    const int32_t idx = base[m] + (k - klo);
    const int32_t sk = base[e];
    skip[idx] = sk;
    depth[idx] = (uint8_t)k;
    nbeg[idx] = (int32_t)m;
    nend[idx] = (int32_t)e;
    r.x = r.y = r.z = 0.0;
    if (e - m == 1) {
      const int32_t id = order[m];
      leaf_of[id] = idx;
      leaf_at[m] = idx;
      r.x = pos[3 * (int64_t)id];
      r.y = pos[3 * (int64_t)id + 1];
      r.z = pos[3 * (int64_t)id + 2];
      r.meta = kLeafBit | (uint32_t)id;
    } else if (k == kMaxDepth) {
      for (int64_t p = m; p < e; ++p) {
        leaf_of[order[p]] = idx;
        leaf_at[p] = idx;
      }
      r.meta = kLeafBit | kBucketBit | (uint32_t)idx;
    } else {
      r.meta = ((uint32_t)sk & kSkipMask) | ((uint32_t)k << kSkipBits);
    }
    r0[idx] = r;
    r1[idx] = r;
  }
}

// The passes over the tree go by chunks of 2^log sorted neurons. The inner nodes whose
// neurons all lie in a chunk are listed by depth, deepest first: one block takes them
// bottom-up (or top-down) with barriers between the depths. A node that starts in the chunk
// and ends beyond it contains the neuron at the chunk's end, so there is at most one per
// depth (cross); those that end within the same run of kSuper chunks are taken by a block
// per run, a chunk per thread and depth by depth, the others by one block for all runs
// (cross2). A pass over the tree is thus one launch for up to 4 096 neurons, two up to
// 131 072 and three beyond, instead of one per depth; small trees are bound by that.
constexpr int kChunkLog = 10;
constexpr int kChunkLogOne = 12;           // trees of up to 2^12 neurons are one chunk, if they
                                           // have up to kNodesOne nodes
constexpr int kSuper = 128;
constexpr int kDepths = kMaxDepth + 1;
constexpr int kChunksOne = 1024;           // threads of chunks_k for a tree of one chunk (4 096
                                           // neurons: 19 us with 256, 8.5 with these)

// Trees of few neurons and nodes are one chunk (4 000 neurons in 2 000 cells at the finest depth,
// 36 000 nodes: the refresh takes 115 us by four chunks, 203 by one).
constexpr int64_t kNodesOne = 8192;

inline int chunk_log(int64_t n, int64_t N) {
  return n <= ((int64_t)1 << kChunkLogOne) && N <= kNodesOne ? kChunkLogOne : kChunkLog;
}

__global__ void __launch_bounds__(kChunksOne) chunks_k(
    const uint8_t* __restrict__ depth, const int32_t* __restrict__ skip,
    const int32_t* __restrict__ base, int64_t n, int log, int nch, int nsup, int32_t* chunk_x,
    int32_t* chunk_off, int32_t* chunk_nodes, int32_t* cross, int32_t* cross2, int32_t* cross_kids,
    int32_t* cross2_kids) {
  __shared__ int32_t cnt[kDepths], at[kDepths], cr[kDepths], cr2[kDepths];
  const int c = (int)blockIdx.x, t = (int)threadIdx.x;
  const int64_t p0 = (int64_t)c << log, p1 = p0 + ((int64_t)1 << log);
  const int32_t x0 = base[p0], x1 = base[p1 < n ? p1 : n];
  const int64_t p2 = (int64_t)(c / kSuper + 1) * kSuper << log;
  const int32_t x2 = base[p2 < n ? p2 : n];        // the end of the chunk's run of chunks
  if (t < kDepths) {
    cnt[t] = 0;
    cr[t] = cr2[t] = -1;
  }
  __syncthreads();
  for (int32_t x = x0 + t; x < x1; x += (int32_t)blockDim.x) {
    const int32_t sk = skip[x];
    if (sk == x + 1) continue;                     // a leaf
    const int d = depth[x];
    if (sk <= x1) atomicAdd(&cnt[d], 1);
    else if (sk <= x2) cr[d] = x;
    else cr2[d] = x;
  }
  __syncthreads();
  if (t < kDepths) {
    int32_t before = 0;                            // deepest first
    for (int d = kMaxDepth; d > t; --d) before += cnt[d];
    at[t] = before;
    chunk_off[(int64_t)c * (kDepths + 1) + (kMaxDepth - t)] = before;
    if (t == 0) chunk_off[(int64_t)c * (kDepths + 1) + kDepths] = before + cnt[0];
    cross[(int64_t)t * nch + c] = cr[t];
    const int32_t two = cr2[t];
    if (two >= 0) cross2[(int64_t)t * nsup + c / kSuper] = two;
    // the children of either
    const int32_t x = two >= 0 ? two : cr[t];
    if (x >= 0) {
      int32_t* kids = two >= 0 ? cross2_kids + 8 * ((int64_t)t * nsup + c / kSuper)
                               : cross_kids + 8 * ((int64_t)t * nch + c);
      const int32_t end = skip[x];
      int32_t y = x + 1;
      for (int k = 0; k < 8; ++k) {
        kids[k] = y < end ? y : -1;
        y = y < end ? skip[y] : y;
      }
    }
  }
  if (t == 0) {
    chunk_x[c] = x0;
    if (c == nch - 1) chunk_x[nch] = x1;
  }
  __syncthreads();
  for (int32_t x = x0 + t; x < x1; x += (int32_t)blockDim.x) {
    const int32_t sk = skip[x];
    if (sk == x + 1 || sk > x1) continue;
    chunk_nodes[x0 + atomicAdd(&at[(int)depth[x]], 1)] = x;
  }
}

// Boxes of runs of consecutive sorted neurons, in grid cells: runs of 2^run_log(n)
// neurons and runs of 64 such runs. They tell how the steps of a tile's walk spread over
// the pre-order (see part_cuts_k). Each is 6 arrays (x, y, z minima, then maxima) over
// the runs, so that the lanes of a wave read neighbouring runs coalesced.
constexpr int kRunLogMin = 3;
constexpr int64_t kMaxRuns1 = 1024;        // runs of 64 runs: at most this many

inline int64_t runs_of(int64_t n, int log) { return (n + ((int64_t)1 << log) - 1) >> log; }

inline int run_log(int64_t n) {
  int b = kRunLogMin;
  while (runs_of(n, 6 + b) > kMaxRuns1) ++b;
  return b;
}

__device__ __forceinline__ uint32_t gather3(uint64_t v) {   // every third bit -> 21 bits
  v &= 0x1249249249249249ull;
  v = (v | (v >> 2)) & 0x10C30C30C30C30C3ull;
  v = (v | (v >> 4)) & 0x100F00F00F00F00Full;
  v = (v | (v >> 8)) & 0x1F0000FF0000FFull;
  v = (v | (v >> 16)) & 0x1F00000000FFFFull;
  v = (v | (v >> 32)) & 0x1FFFFFull;
  return (uint32_t)v;
}

// One block per run of 64 runs. Bound by reading the keys once (8 B per neuron); the
// minima and maxima go across the lanes of a run, then across the runs through LDS.
__global__ void __launch_bounds__(kBuildBlock) boxes_k(const uint64_t* __restrict__ keys,
                                                      int64_t n, int log, int64_t r0, int64_t r1,
                                                      float* __restrict__ box0,
                                                      float* __restrict__ box1) {
  __shared__ uint32_t b[6][64];
  const int lane = (int)(threadIdx.x & (kWave - 1));
  const int wave = (int)(threadIdx.x / kWave);
  const int64_t first = ((int64_t)blockIdx.x * 64) << log;      // the block's neurons
  const int per = log < 6 ? 6 - log : 0;                         // log2 of runs per pass
  const int passes = log < 6 ? 1 : 1 << (log - 6);               // passes per run
  for (int r = wave << per; r < 64; r += (kBuildBlock / kWave) << per) {
    uint32_t lo[3] = {~0u, ~0u, ~0u}, hi[3] = {0, 0, 0};
    for (int q = 0; q < passes; ++q) {
      const int64_t p = first + ((int64_t)r << log) + (int64_t)q * kWave + lane;
      if (p < n) {
        const uint64_t k = keys[p];
        const uint32_t c[3] = {gather3(k >> 2), gather3(k >> 1), gather3(k)};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          lo[a] = c[a] < lo[a] ? c[a] : lo[a];
          hi[a] = c[a] > hi[a] ? c[a] : hi[a];
        }
      }
    }
    const int span = log < 6 ? 1 << log : kWave;
    for (int o = 1; o < span; o <<= 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const uint32_t l = (uint32_t)__shfl_xor((int)lo[a], o, kWave);
        const uint32_t h = (uint32_t)__shfl_xor((int)hi[a], o, kWave);
        lo[a] = l < lo[a] ? l : lo[a];
        hi[a] = h > hi[a] ? h : hi[a];
      }
    }
    if ((lane & (span - 1)) == 0) {
      const int k = r + (log < 6 ? lane >> log : 0);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        b[a][k] = lo[a];
        b[3 + a][k] = hi[a];
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  const int64_t run = (int64_t)blockIdx.x * 64 + lane;
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    uint32_t v = b[a][lane];
    if (run < r0) box0[(int64_t)a * r0 + run] = (float)v;       // 21 bits: exact
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t w = (uint32_t)__shfl_xor((int)v, o, kWave);
      v = a < 3 ? (w < v ? w : v) : (w > v ? w : v);
    }
    if (lane == 0) box1[(int64_t)a * r1 + blockIdx.x] = (float)v;
  }
}

}  // namespace msp
