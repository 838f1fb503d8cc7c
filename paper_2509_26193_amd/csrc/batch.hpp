// Search over a batch of independent simulations: one set of launches for all of
// them. A single simulation (the plain msp_find_targets) is the batch of one, so a
// simulation's results do not depend on the batch it runs in.
//
// Every simulation s has its own octree, sources, parameters and outputs, described
// by a SimDesc in a device table. Flat index spaces concatenate the simulations'
// neurons (neuron g of the batch = neuron g - nbase[s] of simulation s) and their
// 64-source tiles (tile t belongs to simulation s for tile_base[s] <= t <
// tile_base[s + 1]). Preparation (CSR offsets, Morton worklists) runs as flat
// kernels over the batch; the sweep's persistent waves pull tiles of any simulation.
// Nothing here allocates or synchronises: the scratch comes from the caller, so the
// whole sequence can be captured in a HIP graph and replayed.
#pragma once

#include <algorithm>

#include "build.hpp"
#include "scan.hpp"
#include "search_wave.hpp"

namespace msp {

// LDS bytes per thread of the kernels that run restart levels: a level's kept weights
// and ids (see restart_search).
constexpr size_t kRestartLds = kRestartKeep * (sizeof(double) + sizeof(uint32_t));

// Persistent waves take units (runs of parts of 64-source tiles, in tile order) from the
// range of their own die (neighbouring sources share upper-tree nodes in that die's L2):
// the first one by the wave's own index, the following ones from the die's counter, then
// from the other dies' counters. A unit's simulation is found from the unit bases. An
// atomic on a counter takes about 25 ns of the one memory channel that holds it, and what
// else that channel serves waits: with all the counters in one cache line and every wave
// asking all of them, a launch of 2 800 short units took 650 us, most of it that. The
// counters lie 128 bytes apart, and none is asked that has nothing left.
// Scalar registers: on this chip a wave that needs more than 80 (the count the compiler
// reports, with VCC) leaves room for only 7 waves per SIMD, although the compiler and the
// occupancy query both count 8 (measured: 78 give 8 resident waves per SIMD, 82 give 7).
// The sweep hides record latency with resident waves, so it is held to 80; what does not
// fit is kept in vector-register lanes on the rare paths (bucket leaves, thinning).
template <bool DIAG, bool CKPT, bool OWN>
__global__ void __launch_bounds__(kWaveBlock) __attribute__((amdgpu_num_sgpr(80)))
search_sweep_k(BatchDev, SweepOut) {
  const auto K = (cptr<SweepKernargs>)__builtin_amdgcn_kernarg_segment_ptr();
  const int lane = threadIdx.x & (kWave - 1);
  int q = park(0);
  int prev = park(0);
  int mine = park((int)(blockIdx.x / kXcd * (kWaveBlock / kWave) + threadIdx.x / kWave));
  while (unpark(q) < kXcd) {
    const cptr<SweepKernargs> Kq = again(K);
    const int nunits = *Kq->W.unit_count;
    const int qq = (int)((blockIdx.x + unpark(q)) % kXcd);
    const int lo = (int)((int64_t)nunits * qq / kXcd);
    const int count = (int)((int64_t)nunits * (qq + 1) / kXcd) - lo;
    // the die's waves take its first units by their own index
    const int fixed = ((int)gridDim.x - qq + kXcd - 1) / kXcd * (kWaveBlock / kWave);
    int got = unpark(mine);
    if (got < 0) {
      got = count;
      if (count > fixed) {
        int at = 0;
        if (lane == 0) {
          int32_t* next = &Kq->W.queue[qq * kQueueStride];
          at = __hip_atomic_load(next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (at + fixed < count) at = atomicAdd(next, 1);
        }
        got = __builtin_amdgcn_readfirstlane(at) + fixed;
      }
    }
    mine = park(-1);
    if (got >= count) {
      q = park(unpark(q) + 1);
      continue;
    }
    prev = park(sweep_unit<DIAG, CKPT, OWN>(again(K), lo + got, lane, unpark(prev)));
  }
}

// One thread per worklist slot (source) and share of its elements: their draws and
// restarts. The 64 slots of a wavefront form one tile, so the simulation is uniform across
// the wave. In launches of up to kDrawSplitTiles tiles a source's elements go to kDrawSplit
// threads (element j to share j % kDrawSplit, one share's blocks after the other's): such a
// launch takes as long as its longest chains of record loads (4 096 neurons with up to 2
// elements: 88 -> 49 us, 60 001: 144 -> 86, 1 M clustered with up to 4: 1.11 -> 1.02 ms). Larger
// ones are bound by the lines that miss the L2 (8M neurons: 20 GB fetched, 5.8 TB/s), and the
// tile's data would be read twice (3.55 -> 3.93 ms, 64 simulations 1.52 -> 1.65).
// In both, groups of kDrawGroup neighbouring blocks share a die's L2 (8M neurons: 3.55 -> 3.49
// ms, 64 simulations 1.52 -> 1.44; 128 blocks: the same, but 1 M clustered neurons 1.09 -> 1.21).
constexpr int kDrawSplit = 2;
constexpr int kDrawSplitTiles = 16384;
constexpr int kDrawGroup = 32;

// Six waves per SIMD, the most that the LDS of the restart levels leaves; counting launches
// keep five, whose registers hold the counts without spilling most of them.
template <bool DIAG, bool DEFER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DIAG ? 5 : 6)))
search_draw_k(BatchDev B, SweepOut W) {
  const int tiles = *as_const(W.tile_count);
  if (tiles <= 0) return;
  const int split = tiles <= kDrawSplitTiles ? kDrawSplit : 1;
  const int per = (int)blockDim.x / kWave, blocks = (tiles + per - 1) / per;
  const int group = blocks < kXcd * kDrawGroup ? 1 : kDrawGroup;
  const int padded = (blocks + kXcd * group - 1) / (kXcd * group) * (kXcd * group);
  const int share = (int)blockIdx.x / padded, c = (int)blockIdx.x % padded, b = c / kXcd;
  if (share >= split) return;
  const int64_t at = (int64_t)(b / group * kXcd + c % kXcd) * group + b % group;
  const int64_t slot = at * blockDim.x + threadIdx.x;
  const int64_t tile = slot / kWave;
  if (tile >= tiles) return;
  const int sim = __builtin_amdgcn_readfirstlane(find_sim(as_const(B.tile_base), B.nsims, tile));
  const SearchArgs A = args_of(B.sims, sim, B.work);
  const int plog = __builtin_amdgcn_readfirstlane((int)as_const(B.plog)[sim]);
  const int nslog = __builtin_amdgcn_readfirstlane((int)as_const(B.nslog)[sim]);
  const int64_t p0 = (tile - (int64_t)as_const(B.tile_base)[sim]) << plog;
  const int64_t u0 = as_const(B.part_base)[sim] + p0;
  const int64_t s0 = as_const(B.slot_base)[sim] + (p0 << nslog);
  DiagOut D{};
  if (DIAG) {
    const cptr<SimDesc> d = as_const(B.sims) + sim;
    D.z0 = d->diag.z0;
    D.levels = d->diag.levels;
    D.visits = d->diag.visits;
    D.opens = d->diag.opens;
    D.visits0 = d->diag.visits0;
    D.opens0 = d->diag.opens0;
    D.entries0 = d->diag.entries0;
  }
  // the restart levels' entries: kRestartKeep weights, then as many ids, per thread,
  // in LDS sized by the launch (kRestartLds bytes per thread)
  extern __shared__ double keep_lds[];
  const KeptEntries keep{keep_lds + threadIdx.x,
                         reinterpret_cast<uint32_t*>(keep_lds + kRestartKeep * blockDim.x) +
                             threadIdx.x,
                         (int)blockDim.x};
  draw_slot<DIAG, DEFER>(A, D, W, slot, share, split, u0, plog, s0, nslog, &keep);
}

// Second phase of a two-phase search (one simulation): one thread per request in
// cell order (keys sorted); each continues its search from the deferred cell with the
// same draws as the one-phase search, so the target is the same.
template <bool DIAG>
__global__ void __launch_bounds__(256) search_phase2_k(BatchDev B, SweepOut W, int64_t nreq) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nreq) return;
  const uint64_t key = W.defer.key[q];
  if (key == W.defer.none) return;              // sorted last: no request from here on
  const int64_t e = W.defer.val[q];
  const SearchArgs A = args_of(B.sims, 0, B.work);
  const int32_t i = W.defer.src[e];
  const int32_t j = W.defer.elem[e];
  const int t = A.type[i] ? 1 : 0;
  const NodeRec* __restrict__ R = A.rec[t];
  const int32_t li = A.leaf_of[i];
  const double xi = A.pos[3 * (int64_t)i], yi = A.pos[3 * (int64_t)i + 1],
               zi = A.pos[3 * (int64_t)i + 2];
  int lev = W.defer.level[e];
  Count c;
  DiagOut D{};
  if (DIAG) {
    const cptr<SimDesc> d = as_const(B.sims);
    D.levels = d->diag.levels;
    D.visits = d->diag.visits;
    D.opens = d->diag.opens;
    if (D.visits) c.visits = D.visits[e];
    if (D.opens) c.opens = D.opens[e];
  }
  int32_t none = -1;
  extern __shared__ double keep_lds[];      // kRestartLds bytes per thread (see search_draw_k)
  const KeptEntries keep{keep_lds + threadIdx.x,
                         reinterpret_cast<uint32_t*>(keep_lds + kRestartKeep * blockDim.x) +
                             threadIdx.x,
                         (int)blockDim.x};
  const int32_t tgt = restart_search<DIAG, false>(A, R, A.vs[t], W.defer.cell[e], lev, kNoDefer,
                                                  i, j, li, xi, yi, zi, &lev, c, &none, &keep);
  A.target[e] = tgt;
  if (DIAG) {
    if (D.levels) D.levels[e] = lev;
    if (D.visits) D.visits[e] = c.visits;
    if (D.opens) D.opens[e] = c.opens;
  }
}

// Number of requests: the first position whose sorted key is `none`.
__global__ void phase2_count_k(SweepOut W, int64_t nreq, int64_t* out) {
  int64_t lo = 0, hi = nreq;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (W.defer.key[mid] == W.defer.none) hi = mid; else lo = mid + 1;
  }
  *out = lo;
}

// Statuses and counters at 0, the worklist empty (-1).
__global__ void b_clear_k(BatchDev B, int32_t* counters) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < B.max_slots) B.work[q] = -1;
  if (q < B.nsims) B.status[q] = 0;
  if (q < kCounters) counters[q] = 0;
}

// Validity of vac_axon and types; per-simulation status starts at 0 (b_clear_k).
__global__ void b_check_k(BatchDev B, int64_t total) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int s = find_sim(B.nbase, B.nsims, g);
  const int64_t i = g - B.nbase[s];
  const SimDesc& d = B.sims[s];
  const int32_t a = d.vac_axon[i];
  int32_t f = (a < 0 || d.type[i] > 1) ? kSimInvalid : 0;
  if (a > 0 && d.target == nullptr) f |= kSimCapacity;
  // one atomic per wave and flag where the wave's lanes share a simulation (the
  // usual case); a wave that straddles two simulations reports lane by lane
  const int s0 = __builtin_amdgcn_readfirstlane(s);
  if (__all(s == s0)) {
    const bool inv = __ballot((f & kSimInvalid) != 0) != 0;
    const bool cap = __ballot((f & kSimCapacity) != 0) != 0;
    const int first = __ffsll((unsigned long long)__ballot(1)) - 1;
    const int32_t want = (inv ? kSimInvalid : 0) | (cap ? kSimCapacity : 0);
    // most waves of a failing simulation find the flags already set: no atomic then
    if (want && (int)(threadIdx.x & (kWave - 1)) == first &&
        (__hip_atomic_load(&B.status[s0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & want) !=
            want)
      atomicOr(&B.status[s0], want);
  } else if (f) {
    atomicOr(&B.status[s], f);
  }
}

struct FlatAxon {               // vac_axon of flat neuron g (by id), clamped at 0
  BatchDev B;
  __device__ int64_t operator()(int32_t, int64_t g) const {
    const int s = find_sim(B.nbase, B.nsims, g);
    const int32_t a = B.sims[s].vac_axon[g - B.nbase[s]];
    return a > 0 ? (int64_t)a : 0;
  }
};

// Per-simulation CSR offsets and the capacity check.
__global__ void b_offsets_k(BatchDev B, int64_t total) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int s = find_sim(B.nbase, B.nsims, g);
  const int64_t b = B.nbase[s], e = B.nbase[s + 1];
  const SimDesc& d = B.sims[s];
  d.elem_off[g - b] = B.ea[g] - B.ea[b];
  if (g == e - 1) {
    const int64_t S = B.ea[e] - B.ea[b];
    d.elem_off[e - b] = S;
    if (S > d.capacity) atomicOr(&B.status[s], kSimCapacity);
  }
}

// src_type[g]: the type (0, 1) of the neuron at flat Morton position g if it is a
// source of a simulation without errors, else 2. One gather per neuron; the scans and
// the worklist then read it in order.
__global__ void b_src_type_k(BatchDev B, int64_t total) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int s = find_sim(B.nbase, B.nsims, g);
  uint8_t st = 2;
  if (B.status[s] == 0) {
    const SimDesc& d = B.sims[s];
    const int32_t id = d.order[g - B.nbase[s]];
    if (d.vac_axon[id] > 0) st = d.type[id] ? 1 : 0;
  }
  B.src_type[g] = st;
}

struct FlatSource {             // flat Morton position g: a source of type 0 (low word) or 1
  const uint8_t* src_type;
  __device__ int64_t operator()(int32_t, int64_t g) const {
    const uint8_t t = src_type[g];
    return t == 0 ? 1 : t == 1 ? 1ll << 32 : 0;
  }
};

__device__ __forceinline__ int32_t sources0(int64_t p) { return (int32_t)(uint32_t)p; }
__device__ __forceinline__ int32_t sources1(int64_t p) { return (int32_t)(p >> 32); }
__device__ __forceinline__ int64_t sources(int64_t p) {
  return (int64_t)sources0(p) + sources1(p);
}

// log2 of the parts of each of a simulation's `ts` tiles (force >= 0: that). A launch with
// few tiles takes as long as the longest chain of dependent record loads in it: the more
// parts, the shorter that is (4 096 neurons, 45 tiles: the sweep takes 25 us with 64 parts
// per tile, 356 us with 2; 20 011 neurons, 12 % searching: 100 and 898 us). Every part
// costs its wave a start (the ancestors of its first node, about 4 us) and the draw a
// sum to pass over, so parts are no longer added once every wave has one: with 16 or more
// per tile up to 16 384 parts, 60 001 neurons at theta = 0.2 take 1.78 instead of 1.87 ms,
// but a batch of 64 simulations 13.2 instead of 11.9 ms; 8 parts of 2 000 to 16 000 tiles
// balance the waves' loads (1.5 M neurons, 12 % searching: search 3.05 ms, with 2 parts
// 4.0 ms; 1 M clustered neurons: 6.6 ms with 8, 7.1 ms with 2). The number depends on the
// simulation alone, so that its results do not depend on the batch it runs in.
__host__ __device__ inline int parts_log(int64_t ts, int force) {
  if (force >= 0) return force;
  int p = 0;
  while (p < kPartLogMax && (ts << (p + 1)) <= (p + 1 > 3   ? (int64_t)kPartsFine
                                                : p + 1 > 1 ? (int64_t)kPartsMax
                                                            : 2 * (int64_t)kPartsMax))
    ++p;
  return p;
}

// log2 of the checkpoint slots of each part of a tile with 2^p parts, after `cut` halvings:
// twice a part's share of the tile's `ck_slots`, at least kMinSlots of them, never under two.
__host__ __device__ inline int slots_log(int p, int ck_slots, int cut) {
  if (ck_slots == 0) return 0;
  int want = (2 * ck_slots) >> p;
  want = want > ck_slots ? ck_slots : want < kMinSlots ? kMinSlots : want;
  int l = 0;
  while (want >> (l + 1)) ++l;
  return l - cut < 1 ? 1 : l - cut;
}

// Halvings after which every part has its two slots: 0 without checkpoints, where nothing has
// to fit (eight rounds of block scans took 6 us of each of a gradient's two preparations).
__host__ __device__ inline int slot_cuts(int ck_slots) {
  int cut = 0;
  while (slots_log(0, ck_slots, cut) > 1) ++cut;
  return cut;
}

// Tiles per simulation: excitatory sources padded to a multiple of 64, then
// inhibitory ones, so no tile mixes simulations or types; their parts, the parts' units
// (a launch with more than kUnitsMax parts groups 2^g consecutive parts of a tile into a
// unit, or as many as its tile has) and the parts' checkpoint slots (slots_log), halved until
// all fit into `ck_cap` slots; two for every part always do (see search_size_in). One block; a
// thread takes every kTilesBlock-th simulation. Also writes the tile and unit counts and the
// number of sources (the length of the Hilbert sort).
constexpr int kTilesBlock = kScanBlock;

__global__ void __launch_bounds__(kTilesBlock) b_tiles_k(BatchDev B, int32_t* tile_count,
                                                        int32_t* unit_count, int32_t* nsources,
                                                        int64_t total, int force, int ck_slots,
                                                        int64_t ck_cap) {
  __shared__ int64_t lds[kTilesBlock / kWave];
  const int t = (int)threadIdx.x;
  auto tiles = [&](int s) -> int64_t {
    if (s >= B.nsims) return 0;
    const int64_t b = B.nbase[s], e = B.nbase[s + 1];
    const int64_t c = B.sources[e] - B.sources[b];
    const int32_t c0 = sources0(c), c1 = sources1(c);
    return (c0 + kWave - 1) / kWave + (c1 + kWave - 1) / kWave;
  };
  // the launch's parts, and its slots at ever fewer per part
  int64_t parts = 0;
  for (int s0 = 0; s0 < B.nsims; s0 += kTilesBlock) {
    const int64_t ts = tiles(s0 + t);
    int64_t tot;
    (void)block_exclusive_scan<int64_t>(ts << parts_log(ts, force), lds, &tot);
    parts += tot;
  }
  int g = 0;
  while (g < kPartLogMax && (parts >> g) > kUnitsMax) ++g;
  if (force >= 0 || B.nsims == 1) g = 0;
  int cut = 0;
  for (const int cuts = slot_cuts(ck_slots); cut < cuts; ++cut) {
    int64_t sum = 0;
    for (int s0 = 0; s0 < B.nsims; s0 += kTilesBlock) {
      const int64_t ts = tiles(s0 + t);
      const int p = parts_log(ts, force);
      int64_t tot;
      (void)block_exclusive_scan<int64_t>((ts << p) << slots_log(p, ck_slots, cut), lds, &tot);
      sum += tot;
    }
    if (sum <= ck_cap) break;
  }
  int64_t at_t = 0, at_p = 0, at_u = 0, at_s = 0;
  for (int s0 = 0; s0 < B.nsims; s0 += kTilesBlock) {
    const int s = s0 + t;
    const int64_t ts = tiles(s);
    const int p = parts_log(ts, force);
    const int u = p > g ? p - g : 0;
    const int l = slots_log(p, ck_slots, cut);
    int64_t tt, tp, tu, tl;
    const int64_t et = block_exclusive_scan<int64_t>(ts, lds, &tt);
    const int64_t ep = block_exclusive_scan<int64_t>(ts << p, lds, &tp);
    const int64_t eu = block_exclusive_scan<int64_t>(ts << u, lds, &tu);
    const int64_t el = block_exclusive_scan<int64_t>((ts << p) << l, lds, &tl);
    if (s < B.nsims) {
      B.tile_base[s] = (int32_t)(at_t + et);
      B.part_base[s] = (int32_t)(at_p + ep);
      B.unit_base[s] = (int32_t)(at_u + eu);
      B.slot_base[s] = at_s + el;
      B.plog[s] = (uint8_t)p;
      B.ulog[s] = (uint8_t)u;
      B.nslog[s] = (uint8_t)l;
    }
    at_t += tt;
    at_p += tp;
    at_u += tu;
    at_s += tl;
  }
  if (t == 0) {
    B.tile_base[B.nsims] = (int32_t)at_t;
    B.part_base[B.nsims] = (int32_t)at_p;
    B.unit_base[B.nsims] = (int32_t)at_u;
    B.slot_base[B.nsims] = at_s;
    *tile_count = (int32_t)at_t;
    *unit_count = (int32_t)at_u;
    *nsources = (int32_t)sources(B.sources[total]);
  }
}

// The cuts of a tile with 4 parts or more, one block per tile. A model of the walk says
// how many of its steps fall on a run of sorted neurons (a run's nodes are a range of the
// pre-order): all of the run's nodes, about 1.45 per neuron, where the run's box meets
// the box of the tile's sources; else the cells that the walk accepts at the distance d
// between the two boxes, whose edge is about theta d, so V / (theta d)^3 of them in the
// run's volume V, if that is less. The model is evaluated on every run of 64 runs and,
// where such a one holds more than a few steps, on its 64 runs; the cuts then lie on run
// boundaries at equal shares of the steps. (A host count of the walks' steps gives the
// longest of 64 parts 1.6-1.9 times the mean one and the longest of 8 parts 1.2 times,
// uniform or clustered, dense or sparse sources; cuts at m +- s, 8 s and 64 s around the
// sources' median m gave the longest of 8 parts 2.5-3.4 times, and two parts cut at m
// 1.2-1.3 times.) Any ascending cuts give the same lists: the model only
// balances the parts. Bound by latency where tiles are few (13 us at 45 tiles, 18 us at
// 640), by the model's vector instructions where they are many.
constexpr int kCutBlock = 256;
constexpr int kFineRuns = 64;              // runs of 64 runs that are looked into, per tile
constexpr int kCutThr = 8;                 // thresholds tried, each twice the one before

__device__ __forceinline__ float run_steps(const float* __restrict__ box, int64_t stride,
                                           int64_t r, float m, const float* lo, const float* hi,
                                           float inv_t3) {
  float e[3], gap[3], ext = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float bl = box[a * stride + r], bh = box[(3 + a) * stride + r];
    e[a] = bh - bl;
    ext = fmaxf(ext, e[a]);
    gap[a] = fmaxf(0.0f, fmaxf(bl - hi[a], lo[a] - bh));
  }
  float V = 1.0f, d2 = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float w = fmaxf(e[a], 0.25f * ext);
    V *= w;
    const float q = gap[a] > 0.0f ? gap[a] + 0.25f * w : 0.0f;
    d2 += q * q;
  }
  const float all = 1.45f * m;
  return d2 > 0.0f ? fminf(all, V * inv_t3 / (d2 * sqrtf(d2))) : all;
}

// One value per thread summed over the block (every thread gets the sum).
__device__ __forceinline__ float cut_block_sum(float v, float* lds, int lane, int wave) {
  for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o, kWave);
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < kCutBlock / kWave; ++w) s += lds[w];
  return s;
}

__global__ void __launch_bounds__(kCutBlock) part_cuts_k(BatchDev B, const int32_t* tile_count) {
  __shared__ float c1[kMaxRuns1 + 1];          // steps of each run of 64 runs, then before it
  __shared__ float c0[kFineRuns][kWave + 1];   // steps before each run of those looked into
  __shared__ uint8_t fine[kMaxRuns1];          // 1 + its row of c0; 0: none
  __shared__ int32_t rows[kFineRuns];
  __shared__ float tot[2][kCutBlock / kWave];
  __shared__ float tbox[6];
  __shared__ int32_t above[kCutThr], nfine;
  const int tile = (int)blockIdx.x;
  if (tile >= *tile_count) return;
  const int sim = __builtin_amdgcn_readfirstlane(find_sim(as_const(B.tile_base), B.nsims, tile));
  const int plog = __builtin_amdgcn_readfirstlane((int)as_const(B.plog)[sim]);
  if (plog < 2) return;
  const cptr<SimDesc> d = as_const(B.sims) + sim;
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int64_t n = d->n;
  const int log = d->run_log;
  const int64_t r0 = (n + ((int64_t)1 << log) - 1) >> log;
  const int nr = (int)((n + ((int64_t)64 << log) - 1) >> (log + 6));   // <= kMaxRuns1
  if (wave == 0) {
    // the box of the tile's sources, in grid cells
    const int32_t i = B.work[(int64_t)tile * kWave + lane];
    float lo[3] = {3e38f, 3e38f, 3e38f}, hi[3] = {-3e38f, -3e38f, -3e38f};
    if (i >= 0) {
      const double* p = d->pos + 3 * (int64_t)i;
      const double o[3] = {d->x0, d->y0, d->z0};
      const double s = 2097152.0 / d->edge;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double f = (p[a] - o[a]) * s;
        lo[a] = hi[a] = (float)(f < 0.0 ? 0.0 : f > 2097151.0 ? 2097151.0 : f);
      }
    }
    for (int k = 1; k < kWave; k <<= 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = fminf(lo[a], __shfl_xor(lo[a], k, kWave));
        hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], k, kWave));
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        tbox[a] = lo[a];
        tbox[3 + a] = hi[a];
      }
    }
  }
  if (t < kCutThr) above[t] = 0;
  if (t == 0) nfine = 0;
  __syncthreads();
  float lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = tbox[a];
    hi[a] = tbox[3 + a];
  }
  const double theta = sqrt(d->theta2);
  const float inv_t3 = (float)(1.0 / fmax(theta * d->theta2, 1e-30));
  float sum = 0.0f;
  for (int r = t; r < nr; r += kCutBlock) {
    const int64_t left = n - ((int64_t)r << (log + 6));
    const int64_t m = left < ((int64_t)64 << log) ? left : ((int64_t)64 << log);
    const float c = run_steps(d->box[1], nr, r, (float)m, lo, hi, inv_t3);
    c1[r] = c;
    fine[r] = 0;
    sum += c;
  }
  sum = cut_block_sum(sum, tot[0], lane, wave);
  // look into the runs of 64 runs with more than 1/32 of a part's steps (at least 16),
  // or the first doubling of it that at most kFineRuns of them exceed
  const float thr0 = fmaxf(16.0f, sum * (0.03125f / (float)(1 << plog)));
  for (int r = t; r < nr; r += kCutBlock) {
    const float c = c1[r];
    float thr = thr0;
    for (int k = 0; k < kCutThr && c > thr; ++k) {
      atomicAdd(&above[k], 1);
      thr *= 2.0f;
    }
  }
  __syncthreads();
  float thr = thr0;
  int pick = 0;
  while (pick < kCutThr && above[pick] > kFineRuns) {
    ++pick;
    thr *= 2.0f;
  }
  for (int r = t; r < nr; r += kCutBlock) {
    if (c1[r] > thr) {
      const int at = atomicAdd(&nfine, 1);
      if (at < kFineRuns) {
        rows[at] = r;
        fine[r] = (uint8_t)(at + 1);
      }
    }
  }
  __syncthreads();
  const int nf = nfine < kFineRuns ? nfine : kFineRuns;
  constexpr int kRows = 4;                 // rows a wave reads at once
  for (int f0 = wave * kRows; f0 < nf; f0 += kRows * kCutBlock / kWave) {
    float c[kRows], x[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const int f = f0 + u < nf ? f0 + u : nf - 1;
      const int64_t run = (int64_t)rows[f] * 64 + lane;
      const int64_t left = n - (run << log);
      const float m = (float)(left < ((int64_t)1 << log) ? left : (int64_t)1 << log);
      c[u] = run_steps(d->box[0], r0, run < r0 ? run : r0 - 1, m, lo, hi, inv_t3);
      c[u] = run < r0 ? c[u] : 0.0f;
      x[u] = c[u];
    }
    for (int o = 1; o < kWave; o <<= 1) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const float y = __shfl_up(x[u], o, kWave);
        if (lane >= o) x[u] += y;
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (f0 + u >= nf) break;
      c0[f0 + u][lane + 1] = x[u];
      if (lane == 0) c0[f0 + u][0] = 0.0f;
      if (lane == kWave - 1) c1[rows[f0 + u]] = x[u];
    }
  }
  __syncthreads();
  // the steps before each run of 64 runs, each thread kPer consecutive ones
  constexpr int kPer = kMaxRuns1 / kCutBlock;
  float v[kPer], s = 0.0f;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int r = t * kPer + q;
    v[q] = r < nr ? c1[r] : 0.0f;
    s += v[q];
  }
  float x = s;
  for (int o = 1; o < kWave; o <<= 1) {
    const float y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) tot[1][wave] = x;
  __syncthreads();
  float before = x - s, total = 0.0f;
#pragma unroll
  for (int w = 0; w < kCutBlock / kWave; ++w) {
    before += w < wave ? tot[1][w] : 0.0f;
    total += tot[1][w];
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    c1[t * kPer + q] = before;
    before += v[q];
  }
  if (t == kCutBlock - 1) c1[kMaxRuns1] = before;
  __syncthreads();
  if (t >= 1 << plog) return;
  const uint32_t root = d->rec[0][0].meta;
  const int32_t end = (root & kLeafBit) ? 1 : (int32_t)(root & kSkipMask);
  int32_t cut = 1;
  if (t > 0) {
    const float want = total * ((float)t / (float)(1 << plog));
    int a = 0, b = nr - 1;               // the run of 64 runs that holds it
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (c1[mid] <= want) a = mid; else b = mid - 1;
    }
    const float have = want - c1[a];
    int64_t m;
    if (fine[a]) {
      const float* row = c0[fine[a] - 1];
      int k = 0;
      for (int o = kWave / 2; o > 0; o >>= 1) k += row[k + o] <= have ? o : 0;
      m = ((int64_t)a * 64 + k + (have - row[k] > 0.5f * (row[k + 1] - row[k]) ? 1 : 0)) << log;
    } else {
      m = (int64_t)(a + (have > 0.5f * (c1[a + 1] - c1[a]) ? 1 : 0)) << (log + 6);
    }
    if (m >= n) {
      cut = end;
    } else if (m > 0) {
      // the first node that starts at sorted neuron m
      const int32_t leaf = d->leaf_at[m];
      cut = leaf - ((int32_t)d->depth[leaf] - common_digits(d->keys[m - 1], d->keys[m]) - 1);
      cut = cut < 1 ? 1 : cut > end ? end : cut;
    }
  }
  const int64_t p = (int64_t)(tile - B.tile_base[sim]) << plog;
  B.cuts[B.part_base[sim] + p + t] = cut;
}

// Hilbert index of a cell of the 2^21 grid (J. Skilling, "Programming the Hilbert
// curve", AIP Conf. Proc. 707, 2004: axes to transposed index, then bit interleave).
// Only the order it induces matters here: sources consecutive along the curve are
// close in space, with none of the long jumps the Morton order makes between octants.
__device__ __forceinline__ uint64_t hilbert3(uint32_t x0, uint32_t x1, uint32_t x2) {
  uint32_t X[3] = {x0, x1, x2};
  for (uint32_t Q = 1u << 20; Q > 1; Q >>= 1) {
    const uint32_t P = Q - 1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (X[i] & Q) {
        X[0] ^= P;                                  // invert
      } else {
        const uint32_t t = (X[0] ^ X[i]) & P;       // exchange
        X[0] ^= t;
        X[i] ^= t;
      }
    }
  }
  X[1] ^= X[0];
  X[2] ^= X[1];
  uint32_t t = 0;
  for (uint32_t Q = 1u << 20; Q > 1; Q >>= 1)
    if (X[2] & Q) t ^= Q - 1;
  X[0] ^= t;
  X[1] ^= t;
  X[2] ^= t;
  uint64_t h = 0;
  for (int b = 20; b >= 0; --b)
    h = (h << 3) | ((uint64_t)((X[0] >> b) & 1u) << 2) | ((uint64_t)((X[1] >> b) & 1u) << 1) |
        (uint64_t)((X[2] >> b) & 1u);
  return h;
}

// The three 21-bit cell coordinates of a Morton key (digit 4x + 2y + z per level).
__device__ __forceinline__ void morton_decode(uint64_t k, uint32_t& x, uint32_t& y, uint32_t& z) {
  x = y = z = 0;
  for (int b = 20; b >= 0; --b) {
    const uint32_t d = (uint32_t)(k >> (3 * b)) & 7u;
    x = (x << 1) | (d >> 2);
    y = (y << 1) | ((d >> 1) & 1u);
    z = (z << 1) | (d & 1u);
  }
}

// Leading bits of the Hilbert index that order the sources of a simulation of n neurons: by
// n alone, so that its tiles, the cuts of their walks and the last bits of its sums are
// the same in every batch. Six bits more than it takes to number the neurons leave about a
// neuron per cell where they lie 64 times denser than on average; 20 or more make cells of
// a hundredth of the box edge. (1 M clustered neurons by 26 bits or by 31: the sweep takes 3.48
// and 3.49 ms.)
__host__ __device__ inline int hilbert_bits(int64_t n) {
  int b = 20;
  while (b < 31 && ((int64_t)1 << (b - 6)) < n) ++b;
  return b;
}

// Sort key of a source: its (simulation, type) group, then its simulation's `own` bits of
// the Hilbert index in a field of `bits`, those of the launch's largest simulation.
__host__ __device__ inline uint64_t source_key(uint64_t group, uint64_t h, int own, int bits) {
  return (group << bits) | ((h >> (63 - own)) << (bits - own));
}

// Sort keys of the sources; value = flat Morton position. Sources are packed in Morton order
// (position p0 + p1), so only that prefix is sorted.
__global__ void b_hkeys_k(BatchDev B, int64_t total, int bits, uint64_t* key, int32_t* val) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int t = B.src_type[g];
  if (t > 1) return;
  const int s = find_sim(B.nbase, B.nsims, g);
  const SimDesc& d = B.sims[s];
  uint32_t x, y, z;
  morton_decode(d.keys[g - B.nbase[s]], x, y, z);
  const int64_t idx = sources(B.sources[g]);
  key[idx] = source_key((uint64_t)(2 * s + t), hilbert3(x, y, z),
                        hilbert_bits(B.nbase[s + 1] - B.nbase[s]), bits);
  val[idx] = (int32_t)g;
}

// Worklist from the sorted sources: the rank within a (simulation, type) group is the
// sorted position minus the group's start.
__global__ void b_work_sorted_k(BatchDev B, int64_t total, const int32_t* __restrict__ val) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= sources(B.sources[total])) return;
  const int64_t g = val[p];
  const int s = find_sim(B.nbase, B.nsims, g);
  const int64_t b = B.nbase[s], e = B.nbase[s + 1];
  const SimDesc& d = B.sims[s];
  const int32_t id = d.order[g - b];
  const int t = B.src_type[g];
  const int32_t c0 = sources0(B.sources[e] - B.sources[b]);
  const int64_t start = sources(B.sources[b]) + (t ? c0 : 0);
  const int64_t base = (int64_t)B.tile_base[s] * kWave +
                       (t ? (int64_t)((c0 + kWave - 1) / kWave) * kWave : 0);
  B.work[base + (p - start)] = id;
}

// ---------------------------------------------------------------------------
// Scratch layout (device), carved from one buffer.
// ---------------------------------------------------------------------------
// What the working memory of a search is sized by: `slots` checkpoints aimed at per tile
// (0: no checkpoints, for launches without draws) and ck_cap checkpoint slots in all; force
// >= 0: every tile has 2^force parts; counts: a launch that counts visits and opens.
struct SearchSize {
  int64_t total_n;
  int nsims;
  int slots;
  int64_t ck_cap;
  int force;
  bool counts;
};

// Checkpoint bytes per slot: the wave position and, per lane, the running sum and the
// mask end.
constexpr size_t kCkptSlotBytes = sizeof(int32_t) + kWave * (sizeof(double) + sizeof(int32_t));

struct SearchScratch {
  SearchSize q;
  int64_t max_n;                // neurons of the largest simulation
  BatchDev B;
  SweepOut W;
  int32_t* counters;            // [0] tile count, [1] sources, [2] units, then the dies'
                                // queues, kQueueStride apart
  void* scan_tmp;
  uint64_t* hkey[2];            // [total_n] sort keys of the Hilbert-ordered worklist
  int32_t* hval[2];             // [total_n] their flat positions
  void* hsort;                  // radix sort workspace
  bool own_cell;                // the sweep tests for the source's own cell (see sweep_unit)
};

inline int64_t max_tiles_for(int64_t total_n, int nsims) { return total_n / kWave + 2 * nsims + 1; }

// Parts of all tiles (see parts_log), of at most mt tiles; with the parts forced to
// 2^force (force >= 0), exactly that many per tile.
inline int64_t max_parts_for(int64_t total_n, int nsims, int force = -1) {
  const int64_t mt = max_tiles_for(total_n, nsims);
  if (force >= 0) return mt << force;
  // per simulation of ts tiles: ts, or 2 ts <= 2 kPartsMax, or 8 ts <= kPartsMax, or
  // 64 ts <= kPartsFine
  const int64_t two = std::max(mt, std::min(mt << 1, (int64_t)nsims * 2 * kPartsMax)),
                eight = std::min(mt << 3, (int64_t)nsims * kPartsMax),
                fine = std::min(mt << kPartLogMax, (int64_t)nsims * kPartsFine);
  return nsims == 1 ? std::max(two, std::max(eight, fine))
                    : std::min(mt << kPartLogMax, two + eight + fine);
}

// The checkpoints of a search on a device of `mem` bytes: kCkptMax aimed at per tile if that
// many slots per tile fit in an eighth of it, else kCkptMin. More slots mean shorter re-walks
// in the draw kernel; the targets do not depend on the choice. Slots in all: as many per tile,
// and as many more as that eighth holds up to twice that (the forced parts' share, where
// parts are forced) or kMinSlots for each part of a launch with few tiles; and in any case
// two for every part there can be, which b_tiles_k counts on. (An ensemble of 9 000
// simulations of 4 096 neurons needs more for that than the eighth of 288 GB holds.)
inline SearchSize search_size_in(size_t mem, int64_t total_n, int nsims, int force, bool counts) {
  const int64_t mt = max_tiles_for(total_n, nsims);
  const double budget = (double)(mem / 8);
  const int slots = (double)mt * kCkptMax * (double)kCkptSlotBytes <= budget ? kCkptMax : kCkptMin;
  const int64_t fine = std::min(mt << kPartLogMax, (int64_t)nsims * kPartsFine) * kMinSlots;
  const int64_t want = force >= 0 ? (mt << force) * slots : std::max(2 * mt * slots, fine);
  const int64_t fit = (int64_t)(budget / (double)kCkptSlotBytes);
  const int64_t least = std::max(mt * slots, 2 * max_parts_for(total_n, nsims, force));
  return SearchSize{total_n, nsims, slots, std::max(least, std::min(want, fit)), force, counts};
}

// Sweep units of all tiles: the parts, in a batch grouped to about kUnitsMax.
inline int64_t max_units_for(int64_t total_n, int nsims, int force = -1) {
  const int64_t mp = max_parts_for(total_n, nsims, force);
  if (force >= 0 || nsims == 1) return mp;
  return std::min(mp, std::max<int64_t>(kUnitsMax, max_tiles_for(total_n, nsims)));
}

struct ScratchSizes {
  size_t ea, p, base, slot_base, log, status, work, Z, v, nck, cuts, ckx, ckP, ckme, counters,
      scan, srct, hkey, hval, hsort, total;
};

inline ScratchSizes scratch_sizes(const SearchSize& q) {
  ScratchSizes z;
  const int64_t mt = max_tiles_for(q.total_n, q.nsims);
  const int64_t ms = mt * kWave;
  const int64_t mp = max_parts_for(q.total_n, q.nsims, q.force);
  const bool ck = q.slots > 0;
  z.ea = align_up(sizeof(int64_t) * (q.total_n + 1));
  z.p = align_up(sizeof(int64_t) * (q.total_n + 1));
  z.base = align_up(sizeof(int32_t) * (q.nsims + 1));
  z.slot_base = align_up(sizeof(int64_t) * (q.nsims + 1));
  z.log = align_up(sizeof(uint8_t) * q.nsims);
  z.status = align_up(sizeof(int32_t) * q.nsims);
  z.work = align_up(sizeof(int32_t) * ms);
  z.Z = align_up(sizeof(double) * mp * kWave);
  z.v = q.counts ? align_up(sizeof(int32_t) * mp * kWave) : 0;
  z.nck = ck ? align_up(sizeof(int32_t) * mp) : 0;
  z.cuts = align_up(sizeof(int32_t) * mp);
  z.ckx = ck ? align_up(sizeof(int32_t) * q.ck_cap) : 0;
  z.ckP = ck ? align_up(sizeof(double) * q.ck_cap * kWave) : 0;
  z.ckme = ck ? align_up(sizeof(int32_t) * q.ck_cap * kWave) : 0;
  z.counters = align_up(sizeof(int32_t) * kCounters);
  z.scan = align_up(std::max(scan_tmp_bytes<int64_t>(q.total_n),
                             scan_tmp_bytes<int32_t>(q.total_n)));
  z.srct = align_up(sizeof(uint8_t) * q.total_n);
  z.hkey = align_up(sizeof(uint64_t) * q.total_n);
  z.hval = align_up(sizeof(int32_t) * q.total_n);
  z.hsort = align_up(radix_sort_ws_bytes(q.total_n));
  z.total = z.ea + z.p + 3 * z.base + z.slot_base + 3 * z.log + z.status + z.work + z.Z +
            3 * z.v + z.nck + z.cuts + z.ckx + z.ckP + z.ckme + z.counters + z.scan + z.srct +
            2 * z.hkey + 2 * z.hval + z.hsort;
  return z;
}

inline SearchScratch carve(void* base, const SearchSize& q, const SimDesc* d_sims,
                           const int64_t* d_nbase) {
  const ScratchSizes z = scratch_sizes(q);
  char* p = static_cast<char*>(base);
  auto take = [&](size_t bytes) {
    char* r = bytes ? p : nullptr;
    p += bytes;
    return r;
  };
  SearchScratch S{};
  S.q = q;
  S.max_n = q.total_n;
  S.B.sims = d_sims;
  S.B.nsims = q.nsims;
  S.B.nbase = d_nbase;
  S.B.ea = reinterpret_cast<int64_t*>(take(z.ea));
  S.B.sources = reinterpret_cast<int64_t*>(take(z.p));
  S.B.tile_base = reinterpret_cast<int32_t*>(take(z.base));
  S.B.part_base = reinterpret_cast<int32_t*>(take(z.base));
  S.B.unit_base = reinterpret_cast<int32_t*>(take(z.base));
  S.B.slot_base = reinterpret_cast<int64_t*>(take(z.slot_base));
  S.B.plog = reinterpret_cast<uint8_t*>(take(z.log));
  S.B.ulog = reinterpret_cast<uint8_t*>(take(z.log));
  S.B.nslog = reinterpret_cast<uint8_t*>(take(z.log));
  S.B.status = reinterpret_cast<int32_t*>(take(z.status));
  S.B.work = reinterpret_cast<int32_t*>(take(z.work));
  S.B.max_slots = max_tiles_for(q.total_n, q.nsims) * kWave;
  S.W.Z = reinterpret_cast<double*>(take(z.Z));
  S.W.v0 = reinterpret_cast<int32_t*>(take(z.v));
  S.W.o0 = reinterpret_cast<int32_t*>(take(z.v));
  S.W.e0 = reinterpret_cast<int32_t*>(take(z.v));
  S.W.nck = reinterpret_cast<int32_t*>(take(z.nck));
  S.B.cuts = reinterpret_cast<int32_t*>(take(z.cuts));
  S.W.ck_x = reinterpret_cast<int32_t*>(take(z.ckx));
  S.W.ck_P = reinterpret_cast<double*>(take(z.ckP));
  S.W.ck_me = reinterpret_cast<int32_t*>(take(z.ckme));
  S.W.ck_slots = q.slots;
  S.W.ck_cap = q.ck_cap;
  S.counters = reinterpret_cast<int32_t*>(take(z.counters));
  S.W.tile_count = S.counters;
  S.W.unit_count = S.counters + 2;
  S.W.queue = S.counters + kQueueStride;
  S.W.wave_steps = nullptr;
  S.own_cell = true;
  S.scan_tmp = take(z.scan);
  S.B.src_type = reinterpret_cast<uint8_t*>(take(z.srct));
  S.hkey[0] = reinterpret_cast<uint64_t*>(take(z.hkey));
  S.hkey[1] = reinterpret_cast<uint64_t*>(take(z.hkey));
  S.hval[0] = reinterpret_cast<int32_t*>(take(z.hval));
  S.hval[1] = reinterpret_cast<int32_t*>(take(z.hval));
  S.hsort = take(z.hsort);
  return S;
}

// Preparation: status, CSR offsets, worklists, tile, part and unit bases, the parts' cuts.
// Kernels only.
inline hipError_t enqueue_prep(SearchScratch& S, hipStream_t s) {
  BatchDev& B = S.B;
  const int64_t total_n = S.q.total_n;
  const unsigned g = grid_for(total_n, 256);
  b_clear_k<<<grid_for(std::max<int64_t>(B.max_slots, std::max<int64_t>(B.nsims, kCounters)), 256),
              256, 0, s>>>(B, S.counters);
  b_check_k<<<g, 256, 0, s>>>(B, total_n);
  hipError_t e = exclusive_scan<int64_t, int32_t, FlatAxon>(nullptr, B.ea, total_n, FlatAxon{B},
                                                             true, s, S.scan_tmp);
  if (e != hipSuccess) return e;
  b_offsets_k<<<g, 256, 0, s>>>(B, total_n);
  b_src_type_k<<<g, 256, 0, s>>>(B, total_n);
  e = exclusive_scan<int64_t, int32_t, FlatSource>(nullptr, B.sources, total_n,
                                                   FlatSource{B.src_type}, true, s, S.scan_tmp);
  if (e != hipSuccess) return e;
  b_tiles_k<<<1, kTilesBlock, 0, s>>>(B, S.counters, S.counters + 2, S.counters + 1, total_n,
                                      S.q.force, S.W.ck_slots, S.W.ck_cap);
  // 64-source tiles in Hilbert order within each (simulation, type) group
  // (24 bits for one simulation of up to 2^17 neurons or a few small ones, 32 for one of any
  // size, 64 of up to 2^18 or 2 048 of up to 2^14)
  int gb = 1;
  while ((1ll << gb) < 2ll * B.nsims) ++gb;
  const int bits = hilbert_bits(S.max_n), kb = (gb + bits + 7) / 8 * 8;
  b_hkeys_k<<<g, 256, 0, s>>>(B, total_n, bits, S.hkey[0], S.hval[0]);
  int at = 0;
  e = radix_sort_pairs_ws(S.hkey[0], S.hval[0], S.hkey[1], S.hval[1], total_n, 0, kb, s, S.hsort,
                          S.counters + 1, &at);
  if (e != hipSuccess) return e;
  b_work_sorted_k<<<g, 256, 0, s>>>(B, total_n, S.hval[at]);
  // a simulation with 4 parts per tile or more has at most kPartsMax / 4 tiles, unless forced
  int64_t tiles = max_tiles_for(total_n, B.nsims);
  if (S.q.force < 0) tiles = B.nsims == 1 ? std::min<int64_t>(tiles, kPartsMax / 4) : tiles;
  if (S.q.force < 0 || S.q.force >= 2)
    part_cuts_k<<<(unsigned)tiles, kCutBlock, 0, s>>>(B, S.counters);
  return hipGetLastError();
}

// The sweep and draw launches. `sweep_blocks` persistent blocks; the draw covers
// every possible slot (threads past the tile count return at once).
template <bool DIAG, bool CKPT>
inline void launch_sweep(const SearchScratch& S, unsigned blocks, hipStream_t s) {
  if (S.own_cell)
    search_sweep_k<DIAG, CKPT, true><<<blocks, kWaveBlock, 0, s>>>(S.B, S.W);
  else
    search_sweep_k<DIAG, CKPT, false><<<blocks, kWaveBlock, 0, s>>>(S.B, S.W);
}

template <bool DIAG>
inline void launch_draw(const SearchScratch& S, unsigned grid, int block, hipStream_t s) {
  if (S.W.defer.depth < kNoDefer)
    search_draw_k<DIAG, true><<<grid, block, kRestartLds * block, s>>>(S.B, S.W);
  else
    search_draw_k<DIAG, false><<<grid, block, kRestartLds * block, s>>>(S.B, S.W);
}

inline hipError_t enqueue_search(SearchScratch& S, bool diag, unsigned sweep_blocks,
                                 int draw_block, hipStream_t s, hipEvent_t mid = nullptr) {
  // (whole groups of blocks on every die, once for each share of the elements)
  const unsigned turn =
      S.B.max_slots < (int64_t)kXcd * kDrawGroup * draw_block ? kXcd : kXcd * kDrawGroup;
  const unsigned draw_grid =
      (grid_for(S.B.max_slots, draw_block) + turn - 1) / turn * turn * kDrawSplit;
  if (diag)
    launch_sweep<true, true>(S, sweep_blocks, s);
  else
    launch_sweep<false, true>(S, sweep_blocks, s);
  if (mid) {
    hipError_t e = hipEventRecord(mid, s);
    if (e != hipSuccess) return e;
  }
  if (diag)
    launch_draw<true>(S, draw_grid, draw_block, s);
  else
    launch_draw<false>(S, draw_grid, draw_block, s);
  return hipGetLastError();
}

}  // namespace msp
