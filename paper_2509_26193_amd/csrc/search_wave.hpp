// Wave-coherent Barnes-Hut search, in two kernels.
//
// search_sweep_k: the 64 lanes of a wavefront hold 64 sources adjacent in Morton
// order (and of one type) and walk the union of their level-0 expansions together.
// The node at the wave's position is read once (uniform address: scalar loads) and
// every lane applies its own rules to it:
//   - a lane is active at node x unless x lies inside a subtree it has already
//     accepted or skipped (x < mask_end), so each lane sees exactly the nodes of its
//     own depth-first walk, in the same order;
//   - the wave descends into x if any active lane opens it, otherwise jumps over
//     the subtree.
// It produces each source's level-0 normaliser Z and, every `interval` wave steps,
// a checkpoint per lane (running sum, mask_end) with the wave position.
//
// Parts: where a simulation has few tiles, each tile's pre-order range is cut into
// 2^p consecutive parts. A work unit is one part, or in a large batch a run of parts
// of a tile, walked by one wave. A unit's walk starts from the lane states at its first
// node, found from that node's ancestors, so every lane sees the same nodes as in one
// walk; every part has its own sum and checkpoints (running sums from the part's
// start), and the part sums add up to Z in part order. The cuts and their number
// depend on the simulation alone, so neither does Z on how parts are grouped into units.
//
// search_draw_k: one thread per source and element j: T = u Z, then the source's
// own walk restarts from the last checkpoint whose running sum does not exceed T
// (not from the root), then restart levels (a drawn cell) run per thread.
#pragma once

#include "build.hpp"
#include "search.hpp"

namespace msp {

constexpr int kCkptMax = 256;      // checkpoint slots per tile: this many where memory
constexpr int kCkptMin = 32;       // allows, else this many (both powers of two)
constexpr int kCkptStepMin = 16;   // smallest checkpoint interval, wave steps
constexpr int kPartLogMax = 6;     // at most 2^6 parts per tile
constexpr int kPartsFine = 4096;   // 16 or more parts per tile while a simulation has at
                                   // most this many
constexpr int kPartsMax = 131072;  // 4 or 8 parts per tile up to this many, 2 up to twice
constexpr int kUnitsMax = 131072;  // a launch with more parts groups them into units
constexpr int kMinSlots = 16;      // checkpoint slots of a part, where memory allows
constexpr int kWaveBlock = 256;    // 4 independent waves per block
constexpr int kXcd = 8;            // accelerator dies; workgroup b runs on die b % 8
constexpr int kQueueStride = 32;   // the dies' unit counters lie in cache lines of their own
constexpr int kCounters = (1 + kXcd) * kQueueStride;
constexpr uint32_t kAheadBytes = 256;   // the sweep requests the records this far ahead
                                        // of its position into the L2
constexpr int64_t kAheadRecords = kAheadBytes / sizeof(NodeRec);   // room kept after the
                                        // sentinel record for those requests
constexpr int kRawBufferWord3 = 0x00020000;   // buffer descriptor word 3: raw dwords

// Requests of the second phase of a two-phase search (one simulation): one entry per
// element e; key[e] is the deferred cell's pre-order index >> shift, or `none` if the
// element was finished in the first phase. Sorting by key groups the requests by
// pre-order range, and the pre-order makes every subtree (a branch cell's in
// particular) one contiguous range.
struct DeferOut {
  int depth = kNoDefer;            // cells at this depth or deeper are deferred
  int shift = 0;
  uint64_t none = ~0ull;
  uint64_t* key = nullptr;         // [S]
  int32_t* val = nullptr;          // [S] e
  int32_t* cell = nullptr;         // [S] the deferred cell
  int32_t* src = nullptr;          // [S] source neuron
  int32_t* elem = nullptr;         // [S] element j of the source
  uint8_t* level = nullptr;        // [S] level of the deferred expansion
};

struct SweepOut {
  double* Z;                       // [parts][64] level-0 sum of the part
  int32_t* v0;                     // [parts][64] level-0 visits (counting launches only)
  int32_t* o0;                     // [parts][64] level-0 opens
  int32_t* e0;                     // [parts][64] level-0 accepted entries
  int32_t* nck;                    // [parts] checkpoints written
  int32_t* ck_x;                   // [slots] wave position (a part's slots are consecutive)
  double* ck_P;                    // [slots][64] running sum
  int32_t* ck_me;                  // [slots][64] mask_end
  int ck_slots;                    // checkpoints aimed at per tile: kCkptMax or kCkptMin
  int64_t ck_cap;                  // slots in all
  const int32_t* tile_count;       // device scalar
  const int32_t* unit_count;       // device scalar: the launch's units
  int32_t* queue;                  // the dies' unit counters, kQueueStride apart, zero at
                                   // launch
  unsigned long long* wave_steps;  // counting launches: total wave steps (nullable)
  DeferOut defer;                  // two-phase search (depth kNoDefer: one phase)
};

// Read-only data seen through the constant address space: wave-uniform loads from
// it become scalar loads into SGPRs (the data is not written during the search).
template <class T>
using cptr = const __attribute__((address_space(4))) T*;

template <class T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  return (cptr<T>)(p);
}

// Record x as one 32-byte scalar load with a 32-bit byte offset in a register (no
// per-node 64-bit address arithmetic; the empty asm keeps the compiler from widening
// the offset computation to 64 bits).
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ NodeRec load_rec_u(cptr<NodeRec> R, uint32_t x) {
  uint32_t off = x * (uint32_t)sizeof(NodeRec);
  asm("" : "+s"(off));
  const u32x8 w =
      *(cptr<u32x8>)((const __attribute__((address_space(4))) char*)R + off);
  NodeRec r;
  r.x = __builtin_bit_cast(double, ((uint64_t)w[1] << 32) | w[0]);
  r.y = __builtin_bit_cast(double, ((uint64_t)w[3] << 32) | w[2]);
  r.z = __builtin_bit_cast(double, ((uint64_t)w[5] << 32) | w[4]);
  r.v = (int32_t)w[6];
  r.meta = w[7];
  return r;
}

// Record at byte offset `off` (a multiple of the record size).
__device__ __forceinline__ NodeRec load_rec_b(cptr<NodeRec> R, uint32_t off) {
  const u32x8 w =
      *(cptr<u32x8>)((const __attribute__((address_space(4))) char*)R + off);
  NodeRec r;
  r.x = __builtin_bit_cast(double, ((uint64_t)w[1] << 32) | w[0]);
  r.y = __builtin_bit_cast(double, ((uint64_t)w[3] << 32) | w[2]);
  r.z = __builtin_bit_cast(double, ((uint64_t)w[5] << 32) | w[4]);
  r.v = (int32_t)w[6];
  r.meta = w[7];
  return r;
}

__device__ __forceinline__ NodeRec load_rec(cptr<NodeRec> R, int64_t x) {
  NodeRec r;
  r.x = R[x].x;
  r.y = R[x].y;
  r.z = R[x].z;
  r.v = R[x].v;
  r.meta = R[x].meta;
  return r;
}

struct SimDesc {
  const NodeRec* rec[2];
  const int32_t* vs[2];
  const double* pos;
  const int32_t* order;
  const uint64_t* keys;         // [n] sorted Morton keys (position g: neuron order[g])
  const int32_t* nbeg;
  const int32_t* nend;
  const int32_t* leaf_of;
  const int32_t* leaf_at;
  const uint8_t* depth;
  const float* box[2];          // boxes of the runs of sorted neurons (see boxes_k)
  int32_t run_log;
  double x0, y0, z0, edge;      // the octree's cube
  int32_t own;                  // per-thread walks test for the source's own cell
  int32_t inside;               // the octree's positions lie inside its cube
  int32_t* err;                 // the octree's sticky device flag
  const uint8_t* type;          // [n]
  const int32_t* vac_axon;      // [n]
  int64_t* elem_off;            // [n + 1] output
  int32_t* target;              // [capacity] output
  int64_t capacity;
  int64_t n;
  double L2, theta2, acc_d2, k2;  // acc_d2: accept_bound(L2, theta2)
  uint64_t seed, step;
  DiagOut diag;                 // nullable outputs of counting launches
};

// per-simulation status bits (device), 0 = ok
constexpr int32_t kSimInvalid = 1;     // negative vac_axon or a type > 1
constexpr int32_t kSimCapacity = 2;    // more searches than target capacity

struct BatchDev {
  const SimDesc* sims;          // [nsims]
  int32_t nsims;
  const int64_t* nbase;         // [nsims + 1] flat neuron offsets
  int64_t* ea;                  // [total + 1] flat exclusive scan of vac_axon
  int64_t* sources;             // [total + 1] flat scan, Morton order: excitatory sources in
                                // the low word, inhibitory ones in the high word
  uint8_t* src_type;            // [total] type of the source at flat position g, 2: none
  int32_t* tile_base;           // [nsims + 1]
  int32_t* part_base;           // [nsims + 1] parts of tiles before each
  int32_t* unit_base;           // [nsims + 1] sweep units (runs of a tile's parts) before each
  int64_t* slot_base;           // [nsims + 1] checkpoint slots before each
  uint8_t* plog;                // [nsims] log2 of the parts per tile
  uint8_t* ulog;                // [nsims] log2 of the units per tile
  uint8_t* nslog;               // [nsims] log2 of the checkpoint slots per part
  int32_t* cuts;                // [parts] first node of each part, tiles with 4 parts or more
  int32_t* status;              // [nsims]
  int32_t* work;                // [max_slots] source id per slot, -1 = padding
  int64_t max_slots;
};

// Largest s with base[s] <= g (base ascending, base[0] = 0).
template <class T>
__device__ __forceinline__ int find_sim(const T* base, int nsims, int64_t g) {
  int lo = 0, hi = nsims - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int64_t)base[mid] <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ SearchArgs args_of(const SimDesc* sims, int s, const int32_t* work) {
  const cptr<SimDesc> d = as_const(sims) + s;
  SearchArgs A;
  A.rec[0] = d->rec[0];
  A.rec[1] = d->rec[1];
  A.vs[0] = d->vs[0];
  A.vs[1] = d->vs[1];
  A.pos = d->pos;
  A.order = d->order;
  A.keys = d->keys;
  A.nbeg = d->nbeg;
  A.nend = d->nend;
  A.leaf_of = d->leaf_of;
  A.own = d->own != 0;
  A.type = d->type;
  A.vac_axon = d->vac_axon;
  A.elem_off = d->elem_off;
  A.work = work;
  A.target = d->target;
  A.err = d->err;
  A.L2 = d->L2;
  A.theta2 = d->theta2;
  A.acc_d2 = d->acc_d2;
  A.k2 = d->k2;
  A.seed = d->seed;
  A.step = d->step;
  return A;
}

// The median of the sources' leaf positions (wave-uniform), in [1, end]: the cut of a
// tile with two parts.
__device__ __forceinline__ int32_t median_cut(int32_t li, bool valid, int lane, int32_t end) {
  const int32_t key = valid ? li : INT32_MAX;
  int32_t rank = 0;
  for (int m = 0; m < kWave; ++m) {
    const int32_t km = __builtin_amdgcn_readlane(key, m);
    rank += (km < key || (km == key && m < lane)) ? 1 : 0;
  }
  const int nv = __popcll(__ballot(valid));
  const uint64_t at = __ballot(valid && rank == nv / 2);
  const int32_t med = __builtin_amdgcn_readlane(key, __ffsll((unsigned long long)at) - 1);
  return __builtin_amdgcn_readfirstlane(med < 1 ? 1 : med > end ? end : med);
}

// A run of a tile's parts, walked by one wave.
struct UnitParts {
  int plog;                        // the tile has 2^plog parts
  int part;                        // the first part of the unit in the tile
  int count;                       // parts in the unit
  int64_t index;                   // the first part among all parts of the launch
  const int32_t* cuts;             // [parts] first node of each part (plog >= 2)
  int64_t slot;                    // the first part's first checkpoint slot
  int nslog;                       // log2 of the slots per part
};

// The end of the unit's part q: its tile's next cut (med: the cut of two parts).
__device__ __forceinline__ int32_t part_end(const UnitParts& U, int q, int32_t med, int32_t end) {
  const int p = U.part + q + 1;
  if (p == 1 << U.plog) return end;
  return U.plog == 1 ? med : as_const(U.cuts)[U.index + q + 1];
}

// The first node of the unit.
__device__ __forceinline__ int32_t unit_begin(const UnitParts& U, int32_t med) {
  if (U.part == 0) return 1;
  return U.plog == 1 ? med : as_const(U.cuts)[U.index];
}

// Unit `unit` of the launch (wave-uniform): its simulation, tile and parts.
template <class BATCH>                       // BatchDev, in any address space
__device__ __forceinline__ UnitParts unit_parts(const BATCH& B, int unit, int& sim, int& tile) {
  sim = __builtin_amdgcn_readfirstlane(find_sim(as_const(B.unit_base), B.nsims, (int64_t)unit));
  const int local = __builtin_amdgcn_readfirstlane(unit - as_const(B.unit_base)[sim]);
  const int ulog = __builtin_amdgcn_readfirstlane((int)as_const(B.ulog)[sim]);
  UnitParts U;
  U.plog = __builtin_amdgcn_readfirstlane((int)as_const(B.plog)[sim]);
  U.count = 1 << (U.plog - ulog);
  U.part = (local & ((1 << ulog) - 1)) << (U.plog - ulog);
  U.cuts = B.cuts;
  U.nslog = __builtin_amdgcn_readfirstlane((int)as_const(B.nslog)[sim]);
  const int64_t p = ((int64_t)(local >> ulog) << U.plog) + U.part;
  U.index = as_const(B.part_base)[sim] + p;
  U.slot = as_const(B.slot_base)[sim] + (p << U.nslog);
  tile = as_const(B.tile_base)[sim] + (local >> ulog);
  return U;
}

// The sweep's arguments in the kernel's argument segment. The walk's scalar registers are
// scarce (see search_sweep_k): what is needed only around it is read where it is needed,
// through a pointer that the compiler takes for a new one each time (`again`), instead
// of staying in registers, or being spilled from them, across the walk.
struct SweepKernargs {
  BatchDev B;
  SweepOut W;
};

template <class T>
__device__ __forceinline__ cptr<T> again(cptr<T> p) {
  asm volatile("" : "+s"(p));
  return p;
}

// A wave-uniform value kept in a vector register until it is read (unpark).
__device__ __forceinline__ int park(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ int unpark(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A lane's mask end at node x0 > 1 of a walk that starts there: the end of the
// subtree of the first ancestor of x0 that the lane's own walk does not enter
// (accepted, or holding no vacancy), else `me` unchanged (the lane is active at x0). The
// ancestors are found by following the pre-order from the root's first child:
// over a subtree that ends at or before x0, into one that holds it.
template <bool OWN>
__device__ __forceinline__ int32_t mask_at(double L2, double theta2, double acc_d2,
                                           cptr<NodeRec> R, int32_t x0, int32_t me, int32_t li,
                                           double xi, double yi, double zi) {
  int32_t y = 1;
  while (y < x0) {
    const NodeRec r = load_rec_u(R, (uint32_t)y);
    int32_t sk = y + 1;
    if ((int32_t)r.meta >= 0) {
      const int32_t e = (int32_t)(r.meta & kSkipMask);
      sk = e > y ? e : y + 1;
    }
    if (sk > x0) {                       // an ancestor of x0 (inner node)
      bool out = true;                   // v == 0: the walk jumps over the subtree
      if (r.v != 0) {
        const double d2 = dist2(xi, yi, zi, r.x, r.y, r.z);
        const bool contains = OWN && (uint32_t)(li - y) < (uint32_t)(sk - y);
        out = !contains && (OWN ? bh_accept_u(L2, theta2, d2, r.meta)
                                : bh_accept_d(acc_d2, d2, r.meta));
      }
      if (me <= y && out) me = sk;
      y = y + 1;
    } else {
      y = sk;
    }
  }
  return me;
}

// Walks the parts of unit `unit` of the launch. `prev`: wave steps per part of the wave's
// previous unit (0: none), from which the initial checkpoint interval is chosen so that the
// slots rarely have to be thinned out. Returns the wave steps per part of this unit.
// OWN: test whether an inner node holds the source's own leaf (such a node is always
// opened). Launches drop the test only where it can never fire: with theta <= 1/2 and
// every position inside the cube, the source and the node's centroid lie in (or,
// through rounding, within a tiny fraction of an edge of) the node's cell of edge l,
// so d^2 <= 3 l^2 (1 + 2^-4) and theta^2 d^2 < l^2: the acceptance test fails anyway.
template <bool DIAG, bool CKPT, bool OWN>
__device__ __forceinline__ int sweep_unit(cptr<SweepKernargs> K, int unit, int lane, int prev) {
  int sim, tile;
  const UnitParts U = unit_parts(K->B, unit, sim, tile);
  cptr<SimDesc> d = as_const(K->B.sims) + sim;
  const int32_t i = K->B.work[(int64_t)tile * kWave + lane];     // -1: padding lane
  const bool valid = i >= 0;
  const int32_t i0 = __builtin_amdgcn_readfirstlane(i);         // lane 0 is never padding
  const int t = d->type[i0] ? 1 : 0;
  const cptr<NodeRec> R = as_const(d->rec[t]);
  int32_t li = -1;
  double xi = 0.0, yi = 0.0, zi = 0.0;
  if (valid) {
    li = d->leaf_of[i];
    const double* p = d->pos + 3 * (int64_t)i;
    xi = p[0];
    yi = p[1];
    zi = p[2];
  }
  // complete the source loads before the walk: inside it, checkpoint stores share
  // the vector-memory counter and would otherwise make every use of the source
  // coordinates wait for them
  __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
  const double L2 = d->L2, theta2 = d->theta2, acc_d2 = d->acc_d2, k2 = d->k2;
  double Z = 0.0;
  Count c0;
  int steps = park(0);
  const NodeRec root = load_rec(R, 0);
  // a one-neuron tree has no list (the only neuron is the source itself): no part of it
  // has a node to walk
  const bool inner = !(root.meta & kLeafBit);
  if (DIAG && valid && U.part == 0) {
    c0.visits = 1;
    c0.opens = inner ? 1 : 0;
  }
  // checkpoint interval: about as many checkpoints as the part has slots over a walk as
  // long as the previous one; as many checkpoints per tile as without parts, where that
  // leaves a few per part: the rest of its slots is headroom (no thinning in long parts)
  int step0 = U.plog > 3 ? kCkptStepMin : 2 * kCkptStepMin;
  if (CKPT && prev > 0) {
    const int aim = max(K->W.ck_slots >> U.plog, kMinSlots / 2);
    step0 = kCkptStepMin;
    while (step0 * aim < prev) step0 <<= 1;
  }
  {
    const int32_t root_end = inner ? (int32_t)(root.meta & kSkipMask) : 1;
    const int32_t med = U.plog == 1 ? median_cut(li, valid, lane, root_end) : 0;
    const int32_t x = unit_begin(U, med);
    int32_t me = valid ? 0 : 0x7FFFFFFF;     // padding lanes are never active
    if (x > 1 && x < part_end(U, U.count - 1, med, root_end))
      me = mask_at<OWN>(L2, theta2, acc_d2, R, x, me, li, xi, yi, zi);
    const int nslog = park(U.nslog), plog = park(U.plog), first = park(U.part),
              index = park((int)U.index), count = park(U.count), med_ = park(med),
              root_ = park(root_end), sim_ = park(sim);
    // (the slots of a launch are below 2^37: the first one of the unit in two words)
    const int slot_lo = park((int)(uint32_t)U.slot), slot_hi = park((int)(U.slot >> 32));
    // the unit's parts once more, from the values kept aside
    auto parts = [&]() {
      UnitParts V;
      V.plog = unpark(plog);
      V.part = unpark(first);
      V.count = unpark(count);
      V.index = unpark(index);
      V.cuts = again(K)->B.cuts;
      V.slot = ((int64_t)unpark(slot_hi) << 32) | (uint32_t)unpark(slot_lo);
      V.nslog = unpark(nslog);
      return V;
    };
    // Steps are counted in `ph`: the step index modulo the checkpoint interval (a power
    // of two, 2^32 / inc), kept in the top bits, so that it is 0 exactly at the
    // multiples of the interval and the step needs no separate test; s1 is the next
    // multiple to be reached (the current one while ph is 0).
    uint32_t inc = 1u << (32 - __builtin_ctz((uint32_t)__builtin_amdgcn_readfirstlane(step0)));
    uint32_t ph = 0;
    int s1 = 0;
    // the walk counts positions in bytes of the record array (position x at 32 x):
    // the next record's address is then the position itself
    constexpr int kRecShift = 5;
    static_assert(sizeof(NodeRec) == (1 << kRecShift), "32-byte records");
    // (unsigned: up to kMaxNodes positions, the sentinel's offset is 2^31)
    uint32_t xb = (uint32_t)x << kRecShift;
    uint32_t meb = valid ? (uint32_t)me << kRecShift : ~0u;  // padding lanes: never active
    const uint32_t lib = (uint32_t)li << kRecShift;
    NodeRec cur = load_rec_b(R, xb);
    // Most wave steps go to a record a little ahead of the current one (the next one,
    // or the end of a small subtree), and a record that misses the L2 costs the step a
    // trip to the Infinity Cache or HBM. Every step therefore also requests the line
    // kAheadBytes past the new position into the L2: a buffer load whose data goes to
    // local memory (one scratch word per lane, never read), so that it holds no register
    // and nothing ever waits for it. The record array keeps kAheadRecords of room after
    // the sentinel (the position is at most the sentinel's), and the buffer covers them.
    // The distance is the instruction's immediate offset, which the hardware may also add
    // to the local-memory address: the sink keeps that much room after the last wave's
    // words, so every write stays inside the block's own local memory either way.
    __shared__ uint32_t ahead_sink[kWaveBlock + kAheadBytes / sizeof(uint32_t)];
    const __amdgpu_buffer_rsrc_t ahead_buf = __builtin_amdgcn_make_buffer_rsrc(
        (void*)R, (short)0, (int)((uint32_t)(root_end + 1 + kAheadRecords) << kRecShift),
        kRawBufferWord3);
    auto* ahead_lds = (__attribute__((address_space(3))) void*)(
        ahead_sink + __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~(kWave - 1))));
    for (int part = park(0); unpark(part) < unpark(count); part = park(unpark(part) + 1)) {
      const UnitParts V = parts();
      const uint32_t endb = (uint32_t)part_end(V, unpark(part), unpark(med_), unpark(root_))
                            << kRecShift;
      // the part's checkpoints (lane 0 keeps the wave positions)
      const int64_t ck0 = V.slot + ((int64_t)unpark(part) << V.nslog);
      const cptr<SweepKernargs> Kc = again(K);
      int32_t* ckx = Kc->W.ck_x + ck0 + lane;      // (per lane: a vector register)
      double* ckP = Kc->W.ck_P + ck0 * kWave + lane;
      int32_t* ckme = Kc->W.ck_me + ck0 * kWave + lane;
      int nck = 0;
      int done = 0;                          // the part's steps
      ph = 0;
      s1 = 0;
      Z = 0.0;
      // a checkpoint at step index s1, a multiple of the interval; a full buffer keeps every
      // other one and doubles the interval
      auto checkpoint = [&]() {
        if (__builtin_expect(nck == 1 << unpark(nslog), 0)) {
          const int ns = 1 << unpark(nslog);
#pragma unroll 1
          for (int k = 1; k < ns / 2; ++k) {
            ckP[k * kWave] = ckP[2 * k * kWave];
            ckme[k * kWave] = ckme[2 * k * kWave];
            if (lane == 0) ckx[k] = ckx[2 * k];
          }
          nck = ns / 2;
          inc >>= 1;
          const int half = (int)(1u << (31 - __builtin_ctz(inc)));   // the old interval
          if (s1 & half) {                // half way between multiples of the new one
            ph = 0x80000000u;
            s1 += half;
            return;
          }
        }
        ckP[nck * kWave] = Z;
        ckme[nck * kWave] = (int32_t)(meb >> kRecShift);
        if (lane == 0) ckx[nck] = (int32_t)(xb >> kRecShift);
        nck = __builtin_amdgcn_readfirstlane(nck + 1);
        s1 += (int)(1u << (32 - __builtin_ctz(inc)));   // the interval
      };
      if (CKPT && xb < endb) {           // the first step's
        ckP[0] = 0.0;
        ckme[0] = (int32_t)(meb >> kRecShift);
        if (lane == 0) ckx[0] = (int32_t)(xb >> kRecShift);
        nck = 1;
        s1 = (int)(1u << (32 - __builtin_ctz(inc)));
      }
      uint32_t bound;
      if (xb < endb) for (;;) {
        do {
          // one node: uniform branches on its kind, per-lane decisions as lane masks, the
          // weight evaluated on every lane and added where the lane takes the entry. The
          // next record's load is issued as soon as the next node is known (a leaf's at
          // once, an inner node's after the ballot), so it is in flight while this node's
          // weights are computed.
          // Lane decisions are lane masks: a ballot of each compare (its mask itself),
          // combined on the scalar unit, and turned back into a lane condition where a
          // select needs one (inverse ballot: the same mask).
          const uint32_t meta = cur.meta;
          const uint64_t m_act = __builtin_amdgcn_ballot_w64(xb >= meb);
          const bool active = __builtin_amdgcn_inverse_ballot_w64(m_act);
          if (DIAG && active) c0.visits += 1;
          uint32_t next;                                         // bytes
          NodeRec nxt;
          if (__builtin_expect((int32_t)meta < 0, 0)) {          // leaf
            next = xb + (1 << kRecShift);                        // index N: the sentinel
            if (cur.v == 0) {
              nxt = load_rec_b(R, next);
            } else if (!(meta & kBucketBit)) {
              const int32_t id = (int32_t)(meta & kIdMask);
              const bool keep = active && id != i;
              if (DIAG && keep) c0.entries += 1;
              const double d2 = dist2(xi, yi, zi, cur.x, cur.y, cur.z);
              const double vd = (double)cur.v;
              // the record is no longer needed: its registers take the next one; the
              // weight is computed while the load is in flight (no instruction of it may
              // be scheduled above the load)
              nxt = load_rec_b(R, next);
              __builtin_amdgcn_sched_barrier(0);
              Z = kernel_add(Z, keep, vd, d2, k2);
            } else {                              // several neurons at one finest cell
              nxt = load_rec_b(R, next);
              const int32_t x = (int32_t)(xb >> kRecShift);
              const cptr<SimDesc> db = again(as_const(again(K)->B.sims) + unpark(sim_));
              const cptr<int32_t> vs = as_const(R == as_const(db->rec[0]) ? db->vs[0] : db->vs[1]);
              const cptr<int32_t> order = as_const(db->order);
              const cptr<double> pos = as_const(db->pos);
              const int32_t pe = as_const(db->nend)[x];
              for (int32_t p = as_const(db->nbeg)[x]; p < pe; ++p) {
                const int32_t id = order[p];
                const int32_t v = vs[p];
                if (v == 0) continue;
                if (DIAG && active && id != i) c0.entries += 1;
                Z = kernel_add(Z, active && id != i, (double)v,
                               dist2(xi, yi, zi, pos[3 * (int64_t)id], pos[3 * (int64_t)id + 1],
                                     pos[3 * (int64_t)id + 2]),
                               k2);
              }
            }
          } else if (__builtin_expect(cur.v == 0, 0)) {   // no vacancy below: over the subtree
            next = (meta & kSkipMask) << kRecShift;
            nxt = load_rec_b(R, next);
          } else {                                               // inner node
            const uint32_t sk = (meta & kSkipMask) << kRecShift;   // > xb
            const double d2 = dist2(xi, yi, zi, cur.x, cur.y, cur.z);
            uint64_t m_far = __builtin_amdgcn_ballot_w64(
                OWN ? bh_accept_u(L2, theta2, d2, meta) : bh_accept_d(acc_d2, d2, meta));
            // li in [x, sk), as offsets (padding lanes have li = -1: far above, unsigned)
            if (OWN) m_far &= ~__builtin_amdgcn_ballot_w64(lib - xb < sk - xb);
            const uint64_t m_take = m_act & m_far;
            const double vd = (double)cur.v;
            // the wave descends iff a lane opens x; the record is no longer needed: its
            // registers take the next one. (The and-not sets the scalar condition code to
            // "some lane opens", which the select uses directly.)
            uint64_t m_open;
            asm("s_andn2_b64 %0, %2, %3\n\ts_cselect_b32 %1, %4, %5"
                : "=&s"(m_open), "=s"(next)
                : "s"(m_act), "s"(m_far), "s"(xb + (1 << kRecShift)), "s"(sk)
                : "scc");
            nxt = load_rec_b(R, next);
            __builtin_amdgcn_sched_barrier(0);
            // the lanes that take the node: its weight added, their mask end after it, under
            // the execution mask (every lane of the wave is active here: whole blocks, and
            // uniform branches only): two vector instructions for two scalar ones, of which
            // a step then has as many as its unit takes in the same time (kernel_add's
            // comment has the times; the sum alone under the mask gains nothing)
            const double w = kernel_term(true, d2, k2);
            asm("s_mov_b64 exec, %2\n\tv_mov_b32_e32 %1, %3\n\tv_fma_f64 %0, %4, %5, %0\n\t"
                "s_mov_b64 exec, -1"
                : "+v"(Z), "+v"(meb)
                : "s"(m_take), "s"(sk), "v"(w), "v"(vd));
            if (DIAG && __builtin_amdgcn_inverse_ballot_w64(m_open)) c0.opens += 1;
            if (DIAG && __builtin_amdgcn_inverse_ballot_w64(m_take)) c0.entries += 1;
          }
          xb = next;
          cur = nxt;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(ahead_buf, ahead_lds, 4, 0, (int)xb,
                                                   (int)kAheadBytes, 0);
          // one branch for both events: go on while the part has not ended and no
          // checkpoint is due (the step count's carry: a bound of 0 that nothing is below)
          if (CKPT) {
            asm("s_add_u32 %0, %0, %2\n\ts_cselect_b32 %1, 0, %3"
                : "+s"(ph), "=s"(bound) : "s"(inc), "s"(endb) : "scc");
          } else {
            if (DIAG) ++done;
            bound = endb;
          }
        } while (xb < bound);
        if (!CKPT || !(xb < endb)) break;
        checkpoint();
      }
      if (CKPT) done = s1 - (int)((0u - ph) >> __builtin_ctz(inc));
      steps = park(unpark(steps) + done);
      const cptr<SweepKernargs> Ke = again(K);
      const int64_t at = (int64_t)unpark(index) + unpark(part);
      const int64_t us = at * kWave + lane;
      if (CKPT && lane == 0) Ke->W.nck[at] = nck;
      Ke->W.Z[us] = Z;
      if (DIAG) {
        Ke->W.v0[us] = c0.visits;
        Ke->W.o0[us] = c0.opens;
        Ke->W.e0[us] = c0.entries;
        c0 = Count{};
      }
    }
    if (DIAG) {
      unsigned long long* ws = again(K)->W.wave_steps;
      if (ws && lane == 0) atomicAdd(ws, (unsigned long long)unpark(steps));
    }
    const int c = unpark(count);
    return c == 1 ? unpark(steps) : unpark(steps) / c;
  }
}

// The source's walk over its level-0 list [1, end) for a sum so small that its entries lie
// close to where the weights end (kMaxY) or beyond. Where the tree's cells bound the positions
// and centroids in them (no own-cell test, see own_cell_needed), a cell that would be opened
// is passed over if all of it lies beyond that distance: its entries weigh exactly 0. The
// distance is that of the grid cells between the source's and the cell's, so no rounding of
// the positions matters (the factor covers that of the centroids and products).
template <class F>
__device__ void expand_near(const SearchArgs& A, const NodeRec* __restrict__ R, const int32_t* vs,
                            int32_t end, int32_t i, int32_t li, double xi, double yi, double zi,
                            F& f) {
  const double reach2 =
      kMaxY / A.k2 / edge2_at(A.L2, (uint32_t)kMaxDepth << kSkipBits) * (1.0 + 0x1p-9);
  const uint64_t mine = A.keys[A.nbeg[li]];
  const int32_t q[3] = {(int32_t)gather3(mine >> 2), (int32_t)gather3(mine >> 1),
                        (int32_t)gather3(mine)};
  int32_t x = 1;
  while (x < end) {
    const NodeRec r = R[x];
    if (r.meta & kLeafBit) {
      if (r.v != 0 && leaf_entries(A, vs, x, r, i, xi, yi, zi, f)) return;
      ++x;
      continue;
    }
    int32_t sk = (int32_t)(r.meta & kSkipMask);
    sk = sk > x ? sk : x + 1;
    if (r.v == 0) {
      x = sk;
      continue;
    }
    if (A.own) {
      if (li >= x && li < sk) {
        ++x;
        continue;
      }
    }
    const double d2 = dist2(xi, yi, zi, r.x, r.y, r.z);
    if (bh_accept(A.L2, A.theta2, d2, r.meta)) {
      if (f(x, false, r.v, d2)) return;
      x = sk;
      continue;
    }
    ++x;
    if (A.own) continue;
    const uint64_t key = A.keys[A.nbeg[x - 1]];
    const int up = kMaxDepth - cell_depth(r.meta);
    double gap2 = 0.0;                        // squared, in grid cells
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int32_t lo = (int32_t)(gather3(key >> (2 - a)) >> up << up), hi = lo + (1 << up);
      const int32_t g = lo > q[a] ? lo - q[a] - 1 : q[a] - hi;       // (hi: the first after)
      const double gd = (double)(g > 0 ? g : 0);
      gap2 += gd * gd;
    }
    if (gap2 > reach2) x = sk;
  }
}

// A level-0 sum below kTinyZ once more, from the rounded products (see kernel_add), with the
// entries of weight above 0 kept where there is room.
__device__ __forceinline__ double tiny_sum(const SearchArgs& A, const NodeRec* __restrict__ R,
                                           const int32_t* vs, int32_t end, int32_t i, int32_t li,
                                           double xi, double yi, double zi,
                                           const KeptEntries& keep, int& n) {
  SumKeepPass<true> s{A.k2, keep};
  expand_near(A, R, vs, end, i, li, xi, yi, zi, s);
  n = s.n;
  return s.Z;
}

// The draws and restarts of elements first, first + split, ... of the source in worklist
// slot `slot` (DEFER: restarts from cells at depth >= W.defer.depth become second-phase
// requests). The slot's tile has 2^plog parts, the launch's parts u0, u0 + 1, ... with
// checkpoint slots from s0 on, 2^nslog each. keep: the thread's memory for a restart level's entries (see restart_search).
template <bool DIAG, bool DEFER>
__device__ __forceinline__ void draw_slot(const SearchArgs& A, const DiagOut& D, const SweepOut& W,
                                          int64_t slot, int first, int split, int64_t u0, int plog,
                                          int64_t s0, int nslog, const KeptEntries* keep) {
  const int32_t i = A.work[slot];
  if (i < 0) return;
  const int lane = (int)(slot % kWave);
  const int t = A.type[i] ? 1 : 0;
  const NodeRec* __restrict__ R = A.rec[t];
  const int32_t* vs = A.vs[t];
  const int32_t li = A.leaf_of[i];
  const double xi = A.pos[3 * (int64_t)i], yi = A.pos[3 * (int64_t)i + 1],
               zi = A.pos[3 * (int64_t)i + 2];
  const int np = 1 << plog;
  const double* Zp = W.Z + u0 * kWave + lane;        // the part sums, in part order
  double Z = 0.0;
  int q0 = 0;
  for (; q0 + 8 <= np; q0 += 8) {                    // eight loads in flight
    double z[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) z[q] = Zp[(q0 + q) * kWave];
#pragma unroll
    for (int q = 0; q < 8; ++q) Z = Z + z[q];
  }
  for (; q0 < np; ++q0) Z = Z + Zp[q0 * kWave];
  const NodeRec root = R[0];             // Z > 0 implies an inner root
  const int32_t end = (int32_t)(root.meta & kSkipMask);
  const bool tiny = Z < kTinyZ && root.v > 0 && !(root.meta & kLeafBit);
  const int32_t a = A.vac_axon[i];
  const int64_t off = A.elem_off[i];
  Count c0;
  if (DIAG) {
    for (int q = 0; q < np; ++q) {
      c0.visits += W.v0[(u0 + q) * kWave + lane];
      c0.opens += W.o0[(u0 + q) * kWave + lane];
      c0.entries += W.e0[(u0 + q) * kWave + lane];
    }
  }
  // element j with its level-0 choice: restarts and outputs
  auto finish = [&](int32_t j, int32_t id, bool neuron) {
    int lev = 1;
    Count c = c0;
    int32_t tgt = -1;
    int32_t deferred = -1;
    if (id >= 0)
      tgt = neuron ? id
                   : restart_search<DIAG, DEFER>(A, R, vs, id, 1, W.defer.depth, i, j, li, xi,
                                                 yi, zi, &lev, c, &deferred, keep);
    if (DEFER) {
      const int64_t e = off + j;
      if (tgt == kDeferred) {
        W.defer.key[e] = (uint64_t)((uint32_t)deferred >> W.defer.shift);
        W.defer.cell[e] = deferred;
        W.defer.src[e] = i;
        W.defer.elem[e] = j;
        W.defer.level[e] = (uint8_t)lev;
        tgt = -1;                               // the second phase overwrites it
      } else {
        W.defer.key[e] = W.defer.none;
      }
      W.defer.val[e] = (int32_t)e;
    }
    A.target[off + j] = tgt;
    if (DIAG) {
      if (D.z0) D.z0[off + j] = Z;
      if (D.levels) D.levels[off + j] = lev;
      if (D.visits) D.visits[off + j] = c.visits;
      if (D.opens) D.opens[off + j] = c.opens;
      if (D.visits0) D.visits0[off + j] = c0.visits;
      if (D.opens0) D.opens0[off + j] = c0.opens;
      if (D.entries0) D.entries0[off + j] = c0.entries;
    }
  };
  // (a loop of its own: inside the other one it has every thread spill three more values)
  if (__builtin_expect(tiny, 0)) {
    for (int32_t j = first; j < a; j += split) {
      int32_t id = -1;
      bool neuron = false;
      int n = 0;
      Z = tiny_sum(A, R, vs, end, i, li, xi, yi, zi, *keep, n);
      if (Z > 0.0) {
        const double T = draw_u(A.seed, i, j, A.step, 0) * Z;
        if (n <= kRestartKeep) {
          choose_kept(*keep, n, T, id, neuron);
        } else {
          SelectPass<false> s{A.k2, T};
          expand_near(A, R, vs, end, i, li, xi, yi, zi, s);
          id = s.chosen >= 0 ? s.chosen : s.last;
          neuron = s.chosen >= 0 ? s.chosen_neuron : s.last_neuron;
        }
      }
      finish(j, id, neuron);
    }
    return;
  }
  for (int32_t j = first; j < a; j += split) {
    int32_t id = -1;
    bool neuron = false;
    if (Z > 0.0) {
      const double T = draw_u(A.seed, i, j, A.step, 0) * Z;
      SelectPass<true> p{A.k2, T};
      Count none;
      // the part where the running sum crosses T (the sums added as for Z), and T
      // from that part's start
      int k = -1;
      double Tk = T, pre = 0.0;
      for (int q = 0; q < np && k < 0; q += 2) {
        const double za = Zp[q * kWave], zb = q + 1 < np ? Zp[(q + 1) * kWave] : 0.0;
        const double na = pre + za, nb = na + zb;
        if (za > 0.0 && na > T) {
          k = q;
          Tk = T - pre;
        } else if (zb > 0.0 && nb > T) {
          k = q + 1;
          Tk = T - na;
        }
        pre = nb;
      }
      if (k >= 0) {
        const int nck = W.nck[u0 + k];
        const int64_t ck0 = s0 + ((int64_t)k << nslog);
        const int32_t* ckx = W.ck_x + ck0;
        const double* ckP = W.ck_P + ck0 * kWave + lane;
        const int32_t* ckme = W.ck_me + ck0 * kWave + lane;
        // last checkpoint whose running sum does not exceed Tk (checkpoint 0 holds 0)
        int lo = 0, hi = nck - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (ckP[mid * kWave] <= Tk) lo = mid; else hi = mid - 1;
        }
        p.P = ckP[lo * kWave];
        p.T = Tk;
        const int32_t cx = ckx[lo], cm = ckme[lo * kWave];
        expand_range<false>(A, R, vs, cx > cm ? cx : cm, end, i, li, xi, yi, zi, p, none);
      }
      if (p.chosen < 0) {                       // not crossed (rounding): full walk
        p = SelectPass<true>{A.k2, T};
        expand_range<false>(A, R, vs, 1, end, i, li, xi, yi, zi, p, none);
      }
      id = p.chosen >= 0 ? p.chosen : p.last;
      neuron = p.chosen >= 0 ? p.chosen_neuron : p.last_neuron;
    }
    finish(j, id, neuron);
  }
}

}  // namespace msp
