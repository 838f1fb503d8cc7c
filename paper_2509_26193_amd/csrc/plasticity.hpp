// The change of the network between two connectivity updates (Sec. III-A, "Update of
// synaptic elements" and the first sub-phase of "Update of synapses"), on the device:
//   * growth: per neuron j and element kind k (0 axon, 1 excitatory dendrite,
//     2 inhibitory dendrite) a calcium value Ca ~ N(mean, sd) (Box-Muller on Philox
//     words 0 and 1, key (seed, 2), counter (j, k, step, 0)) moves the continuous
//     element count by dz = steps * nu * (2 exp(-((Ca - xi) / zeta)^2) - 1), with
//     xi = (eta + eps) / 2 and zeta = (eps - eta) / (2 sqrt(ln 2)); z = max(z + dz, 0);
//   * deletion: the round(frac * m) synapses of smallest (Philox word 0, key (seed, 3),
//     counter (s, step, 0, 0); then s) go, s being the place in the list at the start
//     of the step;
//   * retraction, for k = 0, 1, 2 in turn: a neuron whose floor(z) fell below its
//     bound elements of kind k loses that many of its synapses of that kind, those of
//     smallest (top 32 bits of Philox word 0, key (seed, 4), counter (s, step, k, 0);
//     then s);
//   * a synapse (i, g, type) binds one axonal element of i and one dendritic element
//     of kind 1 + type of g; breaking it frees both; the list keeps its order;
//   * vacant elements: floor(z) - bound.
// Selections are by 64-bit keys (priority; or priority and synapse index) with the
// synapse index as the tie-break, so every choice is exact and reproducible.
#pragma once

#include "scan.hpp"

namespace msp {

constexpr int kPlastBlock = 256;

struct SynList {
  int32_t* src;
  int32_t* tgt;
  uint8_t* type;
};

struct Growth {
  double ca_mean, ca_sd, xi, zeta, scale;
};

// Element count g (kind g / n of neuron g % n) after the growth.
__device__ __forceinline__ void grow(double* __restrict__ z, int64_t g, int64_t n, uint64_t seed,
                                     uint64_t step, const Growth& c) {
  const int64_t k = g / n, j = g - k * n;
  uint64_t c0 = (uint64_t)j, c1 = (uint64_t)k, c2 = step, c3 = 0;
  philox4x64_10(c0, c1, c2, c3, seed, 2);
  const double u1 = (double)((c0 >> 11) + 1) * 0x1p-53;     // (0, 1]
  const double u2 = (double)(c1 >> 11) * 0x1p-53;           // [0, 1)
  const double two_pi = 6.283185307179586476925286766559;
  const double gauss = sqrt(-2.0 * log(u1)) * cos(two_pi * u2);
  const double ca = c.ca_mean + c.ca_sd * gauss;
  const double r = (ca - c.xi) / c.zeta;
  const double e = exp(-(r * r));
  const double zz = z[g] + c.scale * (2.0 * e - 1.0);
  z[g] = zz > 0.0 ? zz : 0.0;
}

// Whether synapse s binds elements: one recorded with an endpoint outside [0, n) or a type
// above 1 does not (see bind_k).
__device__ __forceinline__ bool binds(const SynList& L, int64_t s, int64_t n) {
  const int32_t i = L.src[s], g = L.tgt[s];
  return i >= 0 && i < n && g >= 0 && g < n && L.type[s] <= 1;
}

// Frees the two elements a synapse binds.
__device__ __forceinline__ void unbind(const SynList& L, int64_t s, int64_t n, int32_t* bound) {
  if (!binds(L, s, n)) return;
  atomicSub(&bound[L.src[s]], 1);
  atomicSub(&bound[(1 + (int64_t)L.type[s]) * n + L.tgt[s]], 1);
}

// Synapses a deletion removes from a list of m: round(frac m), halves up, at most m
// (the product and the sum rounded separately, as on the host).
__host__ __device__ inline int64_t delete_count(double frac, int64_t m) {
#pragma clang fp contract(off)
  const double w = floor(frac * (double)m + 0.5);
  const int64_t c = (int64_t)w;
  return c < m ? c : m;
}

// Deletion as a selection: the `want` synapses of smallest (priority, index) go. The
// priorities are uniform 64-bit numbers, so the want-th smallest lies within a few standard
// deviations of want / m: one pass draws all priorities, counts those below that range
// and keeps those in it (their number grows as sqrt(m)), one block finds the want-th
// smallest among the kept ones, and one pass marks. (Eight passes of digit histograms over
// all priorities, a pick after each and a scan of the ties took 22 launches, 0.3 ms at 2M
// neurons.) Whatever the priorities, the choice is exact: where the range misses the
// want-th smallest or a block's room overflows, the one block searches all priorities.
constexpr int kDelRoom = 256;              // kept priorities per block
constexpr int kDelAll = 4096;              // up to this many synapses, all are kept
constexpr int kDelSigma = 7;               // half width of the range, standard deviations

struct DelSelect {
  uint64_t key;                 // synapses below (key, index) go, that one included
  int64_t index;                // -1: none goes
};

struct DelWs {
  DelSelect* st;
  int64_t* below;               // [blocks] priorities below the range
  int32_t* kept;                // [blocks] priorities in the range (more than kDelRoom: overflow)
  uint64_t* ckey;               // [blocks][kDelRoom]
  int32_t* cidx;
};

// The range [lo, hi] of priorities that are kept (hi included).
__device__ __forceinline__ void del_range(int64_t want, int64_t m, uint64_t& lo, uint64_t& hi) {
  lo = 0;
  hi = ~0ull;
  if (m <= kDelAll) return;
  const double p = (double)want / (double)m;
  const double w = kDelSigma * sqrt(p * (1.0 - p) / (double)m) + 64.0 / (double)m;
  if (p - w > 0.0) lo = (uint64_t)((p - w) * 0x1p64);
  if (p + w < 1.0) hi = (uint64_t)((p + w) * 0x1p64);
}

// Growth of all element counts, then (frac > 0) the priorities of all m synapses, each
// block's kept ones and counts. Bound by the random numbers' 64-bit products.
__global__ void __launch_bounds__(kPlastBlock) grow_draw_k(double* __restrict__ z, int64_t n,
                                                          Growth c, double frac, DevCount mc,
                                                          uint64_t seed, DevStep step,
                                                          uint64_t* __restrict__ key, DelWs W) {
  __shared__ int32_t nkept;
  __shared__ int32_t nbelow[kPlastBlock / kWave];
  if (threadIdx.x == 0) nkept = 0;
  __syncthreads();
  const uint64_t st = step.get();
  for (int64_t g = gtid(); g < 3 * n; g += gstride()) grow(z, g, n, seed, st, c);
  const int64_t m = mc.get();
  if (!(frac > 0.0) || !W.st) return;
  uint64_t lo, hi;
  del_range(delete_count(frac, m), m, lo, hi);
  int32_t mine = 0;
  for (int64_t s = gtid(); s < m; s += gstride()) {
    const uint64_t k = philox_word0(seed, 3, (uint64_t)s, st, 0, 0);
    key[s] = k;
    mine += k < lo ? 1 : 0;
    if (k >= lo && k <= hi) {
      const int at = atomicAdd(&nkept, 1);
      if (at < kDelRoom) {
        W.ckey[(int64_t)blockIdx.x * kDelRoom + at] = k;
        W.cidx[(int64_t)blockIdx.x * kDelRoom + at] = (int32_t)s;
      }
    }
  }
  for (int o = 1; o < kWave; o <<= 1) mine += __shfl_xor(mine, o, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) nbelow[threadIdx.x / kWave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t b = 0;
    for (int w = 0; w < kPlastBlock / kWave; ++w) b += nbelow[w];
    W.below[blockIdx.x] = b;
    W.kept[blockIdx.x] = nkept;
  }
}

// Selection of the r-th smallest of many 64-bit keys by one block: a histogram of twelve bits,
// most significant first, then of the next twelve among the keys in the bin that holds it,
// until few enough are left to be ranked. LDS of a block of THREADS threads:
constexpr int kPickBlock = 1024;
constexpr int kPickBits = 12;
constexpr int kPickBins = 1 << kPickBits;
constexpr int kPickList = 256;             // keys that are ranked

template <int THREADS>
struct PickRoom {
  union {
    uint32_t hist[kPickBins];
    struct {
      uint64_t lk[kPickList];
      int32_t li[kPickList];
    };
  };
  int64_t lds[THREADS / kWave];
  int64_t before;
  DelSelect found;
  int32_t bin, nlist;
};

// The value of each thread summed over the block; synchronises.
template <int THREADS>
__device__ __forceinline__ int64_t pick_sum(int64_t v, int64_t* lds) {
  for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o, kWave);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = v;
  __syncthreads();
  int64_t s = 0;
  for (int w = 0; w < THREADS / kWave; ++w) s += lds[w];
  return s;
}

// The bin that holds the r-th item (r from 1) of the room's histogram, the items before it
// and those in it; synchronises at the end.
template <int THREADS>
__device__ __forceinline__ void pick_bin(PickRoom<THREADS>& L, int64_t r, int& bin, int64_t& before,
                                         int64_t& count) {
  constexpr int kPer = kPickBins / THREADS;
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  int64_t s = 0;
  for (int q = 0; q < kPer; ++q) s += L.hist[t * kPer + q];
  int64_t x = s;
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == kWave - 1) L.lds[w] = x;
  __syncthreads();
  int64_t at = x - s;
  for (int k = 0; k < w; ++k) at += L.lds[k];
  for (int q = 0; q < kPer; ++q) {
    const int64_t h = L.hist[t * kPer + q];
    if (at < r && r <= at + h) {
      L.bin = t * kPer + q;
      L.before = at;
    }
    at += h;
  }
  __syncthreads();
  bin = L.bin;
  before = L.before;
  count = L.hist[bin];
  __syncthreads();
}

// The r-th of the room's list (nlist keys), by (key, index); synchronises.
template <int THREADS>
__device__ __forceinline__ DelSelect pick_listed(PickRoom<THREADS>& L, int64_t r) {
  const int nlist = L.nlist;
  for (int l = (int)threadIdx.x; l < nlist; l += THREADS) {
    const uint64_t k = L.lk[l];
    const int32_t i = L.li[l];
    int64_t rank = 0;
    for (int q = 0; q < nlist; ++q)
      rank += (L.lk[q] < k || (L.lk[q] == k && L.li[q] < i)) ? 1 : 0;
    if (rank == r - 1) L.found = DelSelect{k, i};
  }
  __syncthreads();
  return L.found;
}

// f(key, index) for each of c keys, a thread's next four loaded together: a block alone is
// bound by the latency of its loads.
template <int THREADS, class F>
__device__ __forceinline__ void pick_scan(const uint64_t* __restrict__ key, int64_t c, F f) {
  constexpr int kAtOnce = 4;
  for (int64_t b = (int64_t)threadIdx.x; b < c; b += kAtOnce * THREADS) {
    uint64_t k[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int64_t i = b + u * THREADS;
      k[u] = key[i < c ? i : b];
    }
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      if (b + u * THREADS < c) f(k[u], b + u * THREADS);
  }
}

// The r-th smallest (r from 1 to c) of c keys and its index, equal keys in the order of their
// indices. Every thread of the block gets it.
template <int THREADS>
__device__ __forceinline__ DelSelect kth_key(const uint64_t* __restrict__ key, int64_t c, int64_t r,
                             PickRoom<THREADS>& L) {
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  uint64_t prefix = 0, mask = 0;
  int64_t count = c;
  for (int shift = 64 - kPickBits; shift > -kPickBits && count > kPickList; shift -= kPickBits) {
    const int s0 = shift < 0 ? 0 : shift;
    const uint64_t digit = shift < 0 ? (1u << (kPickBits + shift)) - 1 : kPickBins - 1;
    __syncthreads();
    for (int q = t; q < kPickBins; q += THREADS) L.hist[q] = 0;
    __syncthreads();
    pick_scan<THREADS>(key, c, [&](uint64_t k, int64_t) {
      if ((k & mask) == prefix) atomicAdd(&L.hist[(k >> s0) & digit], 1u);
    });
    __syncthreads();
    int bin;
    int64_t before;
    pick_bin(L, r, bin, before, count);
    prefix |= (uint64_t)bin << s0;
    mask |= digit << s0;
    r -= before;
  }
  __syncthreads();
  if (count <= kPickList) {
    if (t == 0) L.nlist = 0;
    __syncthreads();
    pick_scan<THREADS>(key, c, [&](uint64_t k, int64_t i) {
      if ((k & mask) != prefix) return;
      const int l = atomicAdd(&L.nlist, 1);
      L.lk[l] = k;
      L.li[l] = (int32_t)i;
    });
    __syncthreads();
    return pick_listed(L, r);
  }
  // all the bits are spent: the r-th of the equal keys
  for (int64_t s0 = 0; s0 < c; s0 += THREADS) {
    const int64_t s = s0 + t;
    const bool eq = s < c && key[s] == prefix;
    const int64_t n = pick_sum<THREADS>(eq ? 1 : 0, L.lds);
    if (n < r) {
      r -= n;
      continue;
    }
    const uint64_t b = __ballot(eq);
    __syncthreads();
    if (lane == 0) L.lds[w] = __popcll(b);
    __syncthreads();
    int64_t rank = __popcll(b & ((1ull << lane) - 1ull));
    for (int k = 0; k < w; ++k) rank += L.lds[k];
    if (eq && rank == r - 1) L.found = DelSelect{prefix, s};
    break;
  }
  __syncthreads();
  return L.found;
}

// One block: the want-th smallest (priority, index).
__global__ void __launch_bounds__(kPickBlock) del_pick_k(double frac, DevCount mc, int blocks,
                                                        const uint64_t* __restrict__ key,
                                                        DelWs W) {
  __shared__ PickRoom<kPickBlock> L;
  __shared__ int32_t first[kStrideGrid + 1];     // kept priorities of the blocks before
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  const int64_t m = mc.get();
  const int64_t want = delete_count(frac, m);
  if (want <= 0) {
    if (t == 0) *W.st = DelSelect{0, -1};
    return;
  }
  uint64_t lo, hi;
  del_range(want, m, lo, hi);
  constexpr int kPer = (int)kStrideGrid / kPickBlock;           // consecutive blocks of a thread
  int64_t nb = 0, nk = 0, over = 0;
  int32_t kept[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int b = t * kPer + q;
    kept[q] = b < blocks ? W.kept[b] : 0;
    nb += b < blocks ? W.below[b] : 0;
    over += kept[q] > kDelRoom ? 1 : 0;
    nk += kept[q];
  }
  int64_t x = nk;
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) L.lds[w] = x;
  __syncthreads();
  int64_t at = x - nk;
  for (int k = 0; k < w; ++k) at += L.lds[k];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    first[t * kPer + q] = (int32_t)at;
    at += kept[q];
  }
  if (t == kPickBlock - 1) first[kStrideGrid] = (int32_t)at;
  nb = pick_sum<kPickBlock>(nb, L.lds);
  over = pick_sum<kPickBlock>(over, L.lds);
  nk = first[kStrideGrid];
  const int64_t r = want - nb;
  // the i-th kept priority of all: its place in the blocks' rooms
  auto place = [&](int i) -> int64_t {
    int lo_ = 0, hi_ = (int)kStrideGrid - 1;
    while (lo_ < hi_) {
      const int mid = (lo_ + hi_ + 1) >> 1;
      if (first[mid] <= i) lo_ = mid; else hi_ = mid - 1;
    }
    return (int64_t)lo_ * kDelRoom + (i - first[lo_]);
  };
  if (over == 0 && r >= 1 && r <= nk) {
    // bins of equal width over the range, then the few in the one that holds the r-th
    const uint64_t width = hi - lo;
    int sh = 0;
    while ((width >> sh) >= kPickBins) ++sh;
    for (int q = t; q < kPickBins; q += kPickBlock) L.hist[q] = 0;
    __syncthreads();
    for (int i = t; i < (int)nk; i += kPickBlock)
      atomicAdd(&L.hist[(W.ckey[place(i)] - lo) >> sh], 1u);
    __syncthreads();
    int bin;
    int64_t before, count;
    pick_bin(L, r, bin, before, count);
    if (count <= kPickList) {
      if (t == 0) L.nlist = 0;
      __syncthreads();
      for (int i = t; i < (int)nk; i += kPickBlock) {
        const int64_t p = place(i);
        const uint64_t k = W.ckey[p];
        if ((int)((k - lo) >> sh) != bin) continue;
        const int l = atomicAdd(&L.nlist, 1);
        L.lk[l] = k;
        L.li[l] = W.cidx[p];
      }
      __syncthreads();
      const DelSelect d = pick_listed(L, r - before);
      if (t == 0) *W.st = d;
      return;
    }
  }
  const DelSelect d = kth_key(key, m, want, L);
  if (t == 0) *W.st = d;
}

// Marks the deleted synapses (st null: none, all marks cleared) and frees their elements.
__global__ void __launch_bounds__(kPlastBlock) del_mark_k(const uint64_t* __restrict__ key,
                                                         DevCount mc, const DelSelect* st,
                                                         SynList L, int64_t n,
                                                         uint8_t* __restrict__ dead,
                                                         int32_t* bound) {
  const int64_t m = mc.get();
  const DelSelect d = st ? *st : DelSelect{0, -1};
  for (int64_t s = gtid(); s < m; s += gstride()) {
    bool go = false;
    if (d.index >= 0) {
      const uint64_t k = key[s];
      go = k < d.key || (k == d.key && s <= d.index);
    }
    dead[s] = go ? 1 : 0;
    if (go) unbind(L, s, n, bound);
  }
}

// Retraction. Kind 0 (axons) goes first: it frees dendritic elements too. Kinds 1 and 2 go
// together, their owners being different arrays: a synapse has one dendritic element, of
// the kind its type says. Of an owner's live synapses of the kind, the `excess` of smallest
// (priority, index) go. The candidates (the synapses of owners with an excess) are counted
// per owner, laid out by owner (a scan and a scatter), and ranked within their owner, in
// place of a sort of them all by (owner, priority) for each kind: 6 launches twice instead
// of 18 to 45 three times.
struct RetractWs {
  uint32_t* exc;                // [owners] elements to retract, times two, plus one where the
                                // owner has more than kSegLarge elements; 0: none
  int32_t* cnt;                 // [owners] candidates
  int32_t* off;                 // [owners] candidates of the owners before
  uint8_t* flag;                // [m] candidate
  int32_t* within;              // [m] place among the owner's candidates
  uint64_t* seg;                // [candidates] (priority << 32 | synapse), by owner
  int32_t* nlarge;              // [2] owners with more than kSegSmall candidates, with more
                                // than kSegLarge,
  int32_t* large;               // [m / kSegSmall + 1] and which
  int32_t* huge;                // [m / kSegLarge + 1]
};
constexpr int kSegSmall = 64;   // candidates of an owner ranked by one thread each
constexpr int kSegLarge = 16384;           // candidates of an owner that one block takes
constexpr int kSegBlocks = 32;  // blocks of an owner with more: each selects, and marks its share

// Owner of synapse s: kind 0: its source; kinds 1 and 2 (k = 1): its target in its type's
// array (-1: no such neuron or array).
__device__ __forceinline__ int64_t owner_of(const SynList& L, int64_t s, int64_t n, int k) {
  const int32_t j = k == 0 ? L.src[s] : L.tgt[s];
  const int t = k == 0 ? 0 : (int)L.type[s];
  return j < 0 || j >= n || t > 1 ? -1 : t * n + j;
}

__global__ void __launch_bounds__(kPlastBlock) excess_k(const int32_t* __restrict__ bound_k,
                                                       const double* __restrict__ z_k,
                                                       int64_t owners, RetractWs R) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < 2) R.nlarge[j] = 0;
  if (j >= owners) return;
  const int32_t b = bound_k[j], e = b - (int32_t)floor(z_k[j]);
  R.exc[j] = e > 0 ? (uint32_t)e << 1 | (b > kSegLarge ? 1u : 0u) : 0u;
  R.cnt[j] = 0;
}

// Owners with many elements take one atomic per wave and owner: additions to one address
// follow one another. (A step over 2 M synapses, a third of them one neuron's, takes 1.3 ms with
// this and the blocks of kSegBlocks, 19 ms without, 0.3 ms over the same list without that
// neuron.)
__global__ void __launch_bounds__(kPlastBlock) retract_count_k(SynList L, int64_t n, int k,
                                                              const uint8_t* __restrict__ dead,
                                                              DevCount mc, RetractWs R) {
  const int64_t m = mc.get();
  const int lane = (int)(threadIdx.x & (kWave - 1));
  for (int64_t s = gtid(); s < m; s += gstride()) {
    bool f = false, many = false;
    int64_t o = -1;
    if (!dead[s]) {
      o = owner_of(L, s, n, k);
      const uint32_t e = o >= 0 ? R.exc[o] : 0u;
      f = e > 0 && binds(L, s, n);
      many = f && (e & 1u);
    }
    if (f && !many) R.within[s] = atomicAdd(&R.cnt[o], 1);
    for (uint64_t left = __ballot(many); left;) {            // (uniform over the wave)
      const int first = __ffsll((unsigned long long)left) - 1;
      const uint64_t same = __ballot(many && o == __shfl(o, first, kWave));
      int32_t at = 0;
      if (lane == first) at = atomicAdd(&R.cnt[o], __popcll(same));
      at = __shfl(at, first, kWave);
      if (same >> lane & 1) R.within[s] = at + __popcll(same & ((1ull << lane) - 1ull));
      left &= ~same;
    }
    R.flag[s] = f ? 1 : 0;
  }
}

__global__ void __launch_bounds__(kPlastBlock) retract_lay_k(SynList L, int64_t n, int k,
                                                            DevCount mc, uint64_t seed,
                                                            DevStep step, RetractWs R) {
  const int64_t m = mc.get();
  const uint64_t st = step.get();
  for (int64_t s = gtid(); s < m; s += gstride()) {
    if (!R.flag[s]) continue;
    const int64_t o = owner_of(L, s, n, k);
    const uint64_t kind = k == 0 ? 0 : 1 + (uint64_t)L.type[s];
    const uint64_t q = philox_word0(seed, 4, (uint64_t)s, st, kind, 0) >> 32;
    const int32_t at = R.within[s];
    R.seg[(int64_t)R.off[o] + at] = (q << 32) | (uint64_t)s;
    if (at == 0) {
      const int32_t c = R.cnt[o];
      if (c > kSegLarge) R.huge[atomicAdd(&R.nlarge[1], 1)] = (int32_t)o;
      else if (c > kSegSmall) R.large[atomicAdd(&R.nlarge[0], 1)] = (int32_t)o;
    }
  }
}

// Each candidate's rank among its owner's, one thread each; the owners with many candidates a
// block each, those with very many kSegBlocks blocks that mark a share each (every one of them
// selects the excess-th smallest by itself: no launch or wait between).
__global__ void __launch_bounds__(kPlastBlock) __attribute__((amdgpu_waves_per_eu(8))) retract_k(
    SynList L, int64_t n, int k, DevCount mc, uint8_t* __restrict__ dead, int32_t* bound,
    RetractWs R) {
  __shared__ PickRoom<kPlastBlock> room;
  const int64_t m = mc.get();
  for (int64_t s = gtid(); s < m; s += gstride()) {
    if (!R.flag[s]) continue;
    const int64_t o = owner_of(L, s, n, k);
    const int32_t c = R.cnt[o], e = (int32_t)(R.exc[o] >> 1);
    if (c > kSegSmall) continue;
    const uint64_t* seg = R.seg + R.off[o];
    int32_t rank = 0;
    if (c > e) {
      const uint64_t me = seg[R.within[s]];
      for (int32_t q = 0; q < c; ++q) rank += seg[q] < me ? 1 : 0;
    }
    if (rank < e) {
      dead[s] = 1;
      unbind(L, s, n, bound);
    }
  }
  const int64_t huge = (int64_t)R.nlarge[1] * kSegBlocks, all = huge + R.nlarge[0];
  const int t = (int)threadIdx.x;
  for (int64_t q = blockIdx.x; q < all; q += gridDim.x) {       // uniform over the block
    const int64_t o = q < huge ? R.huge[q / kSegBlocks] : R.large[q - huge];
    const int64_t c = R.cnt[o], e = R.exc[o] >> 1;
    const int share = q < huge ? (int)(q % kSegBlocks) : 0, shares = q < huge ? kSegBlocks : 1;
    const uint64_t* seg = R.seg + R.off[o];
    const uint64_t last = e < c ? kth_key(seg, c, e, room).key : ~0ull;
    int32_t gone = 0;
    for (int64_t i = c * share / shares + t; i < c * (share + 1) / shares; i += kPlastBlock) {
      if (seg[i] > last) continue;
      const int64_t s = (int64_t)(uint32_t)seg[i];
      dead[s] = 1;
      ++gone;
      atomicSub(&bound[k == 0 ? (1 + (int64_t)L.type[s]) * n + L.tgt[s] : L.src[s]], 1);
    }
    for (int w = 1; w < kWave; w <<= 1) gone += __shfl_xor(gone, w, kWave);
    if ((t & (kWave - 1)) == 0 && gone) atomicSub(&bound[k * n + o], gone);     // the owner's
    __syncthreads();
  }
}

struct LiveFlag {
  const uint8_t* dead;
  __device__ int32_t operator()(int32_t, int64_t s) const { return dead[s] ? 0 : 1; }
};

__global__ void __launch_bounds__(kPlastBlock) compact_k(SynList in, const uint8_t* __restrict__ dead,
                                                        const int32_t* __restrict__ pos, DevCount m,
                                                        SynList out, int64_t* survivors) {
  const int64_t m_ = m.get();
  if (gtid() == 0) *survivors = pos[m_];
  for (int64_t s = gtid(); s < m_; s += gstride()) {
    if (dead[s]) continue;
    const int64_t p = pos[s];
    out.src[p] = in.src[s];
    out.tgt[p] = in.tgt[s];
    out.type[p] = in.type[s];
  }
}

// The first `cnt` synapses of one list into another.
__global__ void __launch_bounds__(kPlastBlock) copy_list_k(SynList from, DevCount cnt, SynList to) {
  const int64_t c = cnt.get();
  for (int64_t s = gtid(); s < c; s += gstride()) {
    to.src[s] = from.src[s];
    to.tgt[s] = from.tgt[s];
    to.type[s] = from.type[s];
  }
}

__global__ void __launch_bounds__(kPlastBlock) vacancy_k(const double* __restrict__ z,
                                                        const int32_t* __restrict__ bound,
                                                        int64_t n, int32_t* va, int32_t* ve,
                                                        int32_t* vi, const int64_t* m,
                                                        int64_t* m_out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g == 0) *m_out = m ? *m : 0;       // the list's length, once nothing reads the old one
  if (g >= 3 * n) return;
  const int64_t k = g / n, j = g - k * n;
  int32_t* out = k == 0 ? va : k == 1 ? ve : vi;
  out[j] = (int32_t)floor(z[g]) - bound[g];
}

// New synapses appended at `to`; they bind their elements.
__global__ void __launch_bounds__(kPlastBlock) bind_k(const int32_t* src, const int32_t* tgt,
                                                     const uint8_t* type, int64_t c, SynList to,
                                                     int64_t n, int32_t* bound, int32_t* err) {
  for (int64_t q = gtid(); q < c; q += gstride()) {
    const int32_t i = src[q], g = tgt[q];
    const uint8_t ty = type[q];
    to.src[q] = i;
    to.tgt[q] = g;
    to.type[q] = ty;
    if (i < 0 || i >= n || g < 0 || g >= n || ty > 1) {
      atomicOr(err, 1);
      continue;
    }
    atomicAdd(&bound[i], 1);
    atomicAdd(&bound[(1 + (int64_t)ty) * n + g], 1);
  }
}

// Appends the *cnt synapses of `from` to the list L after its *m entries and binds
// their elements, if the list (capacity cap) holds them all; else appends nothing and
// sets kRecordCapacity in *flags. record_end_k then advances *m.
constexpr int32_t kRecordCapacity = 1;

__global__ void __launch_bounds__(kPlastBlock) record_k(SynList from, DevCount cnt, SynList L,
                                                       const int64_t* __restrict__ m, int64_t cap,
                                                       int64_t n, int32_t* bound, int32_t* flags) {
  const int64_t c = cnt.get();
  const int64_t base = *m;
  if (c == 0) return;
  if (base + c > cap) {
    if (gtid() == 0) atomicOr(flags, kRecordCapacity);
    return;
  }
  for (int64_t q = gtid(); q < c; q += gstride()) {
    const int32_t i = from.src[q], g = from.tgt[q];
    const uint8_t ty = from.type[q];
    L.src[base + q] = i;
    L.tgt[base + q] = g;
    L.type[base + q] = ty;
    atomicAdd(&bound[i], 1);
    atomicAdd(&bound[(1 + (int64_t)ty) * n + g], 1);
  }
}

__global__ void record_end_k(DevCount cnt, int64_t* m, int64_t cap) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int64_t c = cnt.get();
  if (*m + c <= cap) *m += c;
}

}  // namespace msp
