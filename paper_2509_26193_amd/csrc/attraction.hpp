// Expected attraction and its adjoint (the differentiated form of the search).
//
// For a source i with vacant axonal elements, Z_i is the normaliser of its level-0
// list: the sum over the accepted entries e (cells and neurons, type of i) of
// w_e = v_e exp(-|x_i - c_e|^2 / sigma^2). Given upstream gradients g_i = dLoss/dZ_i,
// with every acceptance decision held at the current geometry:
//   dZ_i/dx_i     = sum_e w_e * (-2 (x_i - c_e) / sigma^2)
//   dZ_i/dc_e     = w_e * 2 (x_i - c_e) / sigma^2        (a neuron entry: c_e = x_j)
//   dZ_i/dsigma   = sum_e w_e * 2 |x_i - c_e|^2 / sigma^3
//   dc_C/dx_j     = (v_j / v_C) I for every neuron j of cell C (a centroid is the
//                   vacancy-weighted mean of its neurons).
// The forward pass is the search's level-0 sweep without checkpoints (Z per source).
// The backward sweep walks the sources' lists coherently (as the search does); per
// node, the contributions of all lanes of the wave are summed across the wave first
// and added to the node's gradient G with one float64 atomic per component. A
// neuron's leaf is a node like any other (its centroid is the neuron's position), so
// leaves need no separate path. The waves of each die add into that die's own copy
// of G, so the atomics of concurrent waves on the nodes they all share (the upper
// tree) are spread over eight addresses instead of queueing on one; a reduction
// sums the copies. A top-down pass then carries sum_{C containing j} G_C / v_C to
// each neuron.
#pragma once

#include "batch.hpp"
#include "refresh.hpp"

namespace msp {

constexpr int kGradCopies = 8;  // one per die (XCC)

struct AttractArgs {
  const float* gZ;              // [n] upstream gradient, by neuron id
  double* G;                    // [kGradCopies][2][N][3] per-node centroid gradients
  double* dpos;                 // [n][3] float64 accumulator
  double* dsigma;               // scalar accumulator
  double two_over_s2;           // 2 / sigma^2
  double one_over_s;            // 1 / sigma
  int64_t N;
};

// The die (XCC) this wave runs on: bits 3:0 of hardware register XCC_ID (20). It only
// selects a copy of G; any value in 0..7 gives the same sums.
__device__ __forceinline__ int xcc_id() {
  return (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)) & (kGradCopies - 1));
}



// v moved across lanes by a DPP pattern (both 32-bit halves); lanes of rows outside
// row_mask get 0.0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Sum over the 64 lanes of the wave (every lane active), returned to every lane. DPP
// steps: pairs, quads (quad_perm), halves of a row (row_half_mirror), rows of 16
// (row_mirror); then rows 0+1 and 2+3 (row_bcast:15), all four (row_bcast:31), which
// leaves the total in lane 63.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1, 0xF>(v);        // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E, 0xF>(v);        // quad_perm [2,3,0,1]
  v += dpp_f64<0x141, 0xF>(v);       // row_half_mirror
  v += dpp_f64<0x140, 0xF>(v);       // row_mirror
  v += dpp_f64<0x142, 0xA>(v);       // row_bcast:15 into rows 1 and 3
  v += dpp_f64<0x143, 0xC>(v);       // row_bcast:31 into rows 2 and 3
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The wave's contributions to nodes, summed over its lanes kSumNodes nodes at a time: every
// lane puts the three components of its entry into LDS, and when the rows are full four lanes
// per sum add up 16 values each and one atomic instruction sends all sums. The walk is bound by
// vector instructions, and this takes about 9 per entry, where exchanges between the lanes
// down to one sum per entry took 30 and waited for each other (262 144 neurons: 2.64 -> 1.88 ms).
// The rows' stride and the lanes' share of the columns keep the reads (16 bytes a lane, 16
// lanes at a time) on different banks.
constexpr int kBwdBlock = 128;
constexpr int kSumNodes = 4;
constexpr int kSumStride = 72;
constexpr int kSumRoom = 3 * kSumNodes * kSumStride;

typedef double f64x2 __attribute__((ext_vector_type(2)));

struct NodeSums {
  double* buf;                     // [kSumNodes][3][kSumStride], the wave's own
  double* G;                       // node gradients of the wave's die and type
  double* dpos;
  int lane;
  int filled = 0;
  int32_t to = 0;                  // the lane's sum's node, or ~(neuron of a bucket)

  __device__ __forceinline__ int node() const { return (lane >> 2) / 3; }

  __device__ __forceinline__ void add(double fx, double fy, double fz, int32_t dst) {
    double* p = buf + filled * (3 * kSumStride) + lane;
    p[0] = fx;
    p[kSumStride] = fy;
    p[2 * kSumStride] = fz;
    to = node() == filled ? dst : to;
    if (++filled == kSumNodes) flush();
  }

  __device__ __forceinline__ void flush() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int row = lane >> 2, comp = row - 3 * node();
    if (row < 3 * filled) {
      const f64x2* p = reinterpret_cast<const f64x2*>(buf + row * kSumStride) + (lane & 3);
      f64x2 v = p[0];
#pragma unroll
      for (int k = 1; k < 8; ++k) v += p[4 * k];
      double s = v.x + v.y;
      s += dpp_f64<0xB1, 0xF>(s);        // quad_perm [1,0,3,2]
      s += dpp_f64<0x4E, 0xF>(s);        // quad_perm [2,3,0,1]
      if ((lane & 3) == 0 && s != 0.0)
        atomicAdd((to < 0 ? dpos + 3 * (int64_t)~to : G + 3 * (int64_t)to) + comp, s);
    }
    filled = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
};

// The parts of unit U of the tile (the search's level-0 sweep cut into parts: the lane
// states at the unit's first node come from its ancestors). OWN: as in the search's sweep.
template <bool OWN>
__device__ void attract_unit(const SearchArgs& A, const AttractArgs& O, int tile,
                             const UnitParts& U, int lane, double* sums) {
  const int64_t slot = (int64_t)tile * kWave + lane;
  const int32_t i = A.work[slot];
  const bool valid = i >= 0;
  const int32_t i0 = __builtin_amdgcn_readfirstlane(i);
  const int t = A.type[i0] ? 1 : 0;
  const cptr<NodeRec> R = as_const(A.rec[t]);
  int32_t li = -1;
  double xi = 0.0, yi = 0.0, zi = 0.0, g = 0.0;
  if (valid) {
    li = A.leaf_of[i];
    xi = A.pos[3 * (int64_t)i];
    yi = A.pos[3 * (int64_t)i + 1];
    zi = A.pos[3 * (int64_t)i + 2];
    g = (double)O.gZ[i];
  }
  double dxi = 0.0, dyi = 0.0, dzi = 0.0, ds = 0.0;   // ds: the sum of f d2
  NodeSums S{sums, O.G + ((int64_t)xcc_id() * 2 + t) * O.N * 3, O.dpos, lane};
  // an entry that the lanes of mask m accept: the gradient factor f = g * w * 2 / sigma^2
  // applied to the offset (x_i - c). Evaluated on every lane, with weight 0 where the lane
  // does not take the entry; a source whose gradient is not finite gets an explicit 0.
  const double g2 = g * O.two_over_s2;
  const bool odd = __any(!(fabs(g2) <= DBL_MAX));
  auto take = [&](uint64_t m, int32_t v, double cx, double cy, double cz, double d2, int32_t dst) {
    const bool on = __builtin_amdgcn_inverse_ballot_w64(m);
    double f = g2 * kernel_weight_if(on, v, d2, A.k2);
    double ex = xi - cx, ey = yi - cy, ez = zi - cz, e2 = d2;
    if (OWN || __builtin_expect(odd, 0)) {   // (outside the cube offsets may overflow)
      f = on ? f : 0.0;
      ex = on ? ex : 0.0;
      ey = on ? ey : 0.0;
      ez = on ? ez : 0.0;
      e2 = on ? e2 : 0.0;
    }
    const double fx = f * ex, fy = f * ey, fz = f * ez;
    dxi -= fx;
    dyi -= fy;
    dzi -= fz;
    ds = __builtin_fma(f, e2, ds);
    S.add(fx, fy, fz, dst);
  };
  const NodeRec root = load_rec(R, 0);
  if (!(root.meta & kLeafBit)) {
    const int32_t root_end = (int32_t)(root.meta & kSkipMask);
    const int32_t med = U.plog == 1 ? median_cut(li, valid, lane, root_end) : 0;
    int32_t x = unit_begin(U, med);
    const int32_t end = part_end(U, U.count - 1, med, root_end);
    int32_t me = valid ? 0 : 0x7FFFFFFF;
    if (x > 1 && x < end) me = mask_at<OWN>(A.L2, A.theta2, A.acc_d2, R, x, me, li, xi, yi, zi);
    NodeRec nxt = load_rec_u(R, (uint32_t)x);
    while (x < end) {
      // the next record is requested as soon as the next node is known, ahead of this one's
      // weights (position N: the record after the last)
      const NodeRec cur = nxt;
      const uint64_t m_act = __builtin_amdgcn_ballot_w64(x >= me);
      const uint32_t meta = cur.meta;
      const int32_t here = x;
      if (meta & kLeafBit) {
        x = x + 1;
        nxt = load_rec_u(R, (uint32_t)x);
        if (cur.v == 0) continue;
        if (!(meta & kBucketBit)) {
          // a neuron's leaf: its gradient reaches the neuron through the push-down
          const int32_t id = (int32_t)(meta & kIdMask);
          const uint64_t m = m_act & __builtin_amdgcn_ballot_w64(id != i);
          if (m)
            take(m, cur.v, cur.x, cur.y, cur.z, dist2(xi, yi, zi, cur.x, cur.y, cur.z), here);
        } else {
          // members of a bucket are entries at their own positions
          const cptr<int32_t> vs = as_const(A.vs[t]);
          const cptr<int32_t> order = as_const(A.order);
          const cptr<double> pos = as_const(A.pos);
          const int32_t pe = as_const(A.nend)[here];
          for (int32_t p = as_const(A.nbeg)[here]; p < pe; ++p) {
            const int32_t id = order[p];
            const int32_t v = vs[p];
            const uint64_t m = m_act & __builtin_amdgcn_ballot_w64(id != i);
            if (v == 0 || !m) continue;
            const double cx = pos[3 * (int64_t)id], cy = pos[3 * (int64_t)id + 1],
                         cz = pos[3 * (int64_t)id + 2];
            take(m, v, cx, cy, cz, dist2(xi, yi, zi, cx, cy, cz), ~id);
          }
        }
        continue;
      }
      int32_t sk = (int32_t)(meta & kSkipMask);
      sk = sk > x ? sk : x + 1;
      if (cur.v == 0) {
        x = sk;
        nxt = load_rec_u(R, (uint32_t)x);
        continue;
      }
      const double d2 = dist2(xi, yi, zi, cur.x, cur.y, cur.z);
      uint64_t m_far = __builtin_amdgcn_ballot_w64(
          OWN ? bh_accept_u(A.L2, A.theta2, d2, meta) : bh_accept_d(A.acc_d2, d2, meta));
      if (OWN) m_far &= ~__builtin_amdgcn_ballot_w64(li >= x && li < sk);
      const uint64_t m = m_act & m_far;
      x = m_act & ~m_far ? x + 1 : sk;
      nxt = load_rec_u(R, (uint32_t)x);
      if (m) {
        __builtin_amdgcn_sched_barrier(0);
        take(m, cur.v, cur.x, cur.y, cur.z, d2, here);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) me = sk;
      }
    }
  }
  S.flush();
  if (valid) {
    atomicAdd(O.dpos + 3 * (int64_t)i + 0, dxi);
    atomicAdd(O.dpos + 3 * (int64_t)i + 1, dyi);
    atomicAdd(O.dpos + 3 * (int64_t)i + 2, dzi);
  }
  ds = wave_sum(ds);
  if (lane == 0 && ds != 0.0) atomicAdd(O.dsigma, ds * O.one_over_s);
}

// Persistent waves take the units as the search's sweep does (see search_sweep_k): each die has
// a range of neighbouring units, so that the nodes near them, whose gradients make up
// most of the additions, are read by one die (262 144 neurons: 1.88 -> 1.81 ms; 17 M steps of
// about 37 vector instructions, the vector units busy three quarters of the time).
template <bool OWN>
__global__ void __launch_bounds__(kBwdBlock) attract_bwd_k(BatchDev B, SweepOut W, AttractArgs O) {
  __shared__ __attribute__((aligned(16))) double sums[kBwdBlock / kWave][kSumRoom];
  const int lane = threadIdx.x & (kWave - 1);
  const int nunits = *as_const(W.unit_count);
  const SearchArgs A = args_of(B.sims, 0, B.work);
  int got = (int)(blockIdx.x / kXcd * (kBwdBlock / kWave) + threadIdx.x / kWave);
  for (int q = 0; q < kXcd;) {
    const int qq = (int)((blockIdx.x + q) % kXcd);
    const int lo = (int)((int64_t)nunits * qq / kXcd);
    const int count = (int)((int64_t)nunits * (qq + 1) / kXcd) - lo;
    const int fixed = ((int)gridDim.x - qq + kXcd - 1) / kXcd * (kBwdBlock / kWave);
    if (got < 0) {
      int at = 0;
      if (lane == 0 && count > fixed) {
        int32_t* next = &W.queue[qq * kQueueStride];
        at = __hip_atomic_load(next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (at + fixed < count) at = atomicAdd(next, 1);
      }
      got = __builtin_amdgcn_readfirstlane(at) + fixed;
    }
    got = __builtin_amdgcn_readfirstlane(got);
    if (got < count) {
      int sim, tile;
      const UnitParts U = unit_parts(B, lo + got, sim, tile);
      attract_unit<OWN>(A, O, tile, U, lane, sums[threadIdx.x / kWave]);
    } else {
      ++q;
    }
    got = -1;
  }
}

// Z of every source from the sweep's part sums (added in part order, then rounded to
// float32); other neurons keep 0.
__global__ void z_scatter_k(BatchDev B, SweepOut W, float* __restrict__ Z) {
  const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tile = slot / kWave;
  if (tile >= *W.tile_count) return;
  const int32_t i = B.work[slot];
  if (i < 0) return;
  const int sim = find_sim(B.tile_base, B.nsims, tile);
  const int plog = B.plog[sim];
  const int64_t u0 = (int64_t)B.part_base[sim] + ((tile - (int64_t)B.tile_base[sim]) << plog);
  const int64_t lane = slot % kWave;
  double z = 0.0;
  for (int q = 0; q < (1 << plog); ++q) z = z + W.Z[(u0 + q) * kWave + lane];
  Z[i] = (float)z;
}

// G = sum of the per-die copies, in die order.
__global__ void grad_sum_k(double* __restrict__ G, int64_t count) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  double s = G[k];
  for (int c = 1; c < kGradCopies; ++c) s += G[(int64_t)c * count + k];
  G[k] = s;
}

__global__ void fill_f64_k(double* p, int64_t n, double v) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = v;
}

// Top-down: H(child) = H(node) + G(child) / v(child), per type; the root's H is
// G(root) / v(root) (zero: the root is never accepted).
__device__ __forceinline__ void push_node(int32_t x, const int32_t (&kids)[8],
                                          const NodeRec* __restrict__ r0,
                                          const NodeRec* __restrict__ r1,
                                          const double* __restrict__ G, double* H, int64_t N) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const NodeRec* r = t ? r1 : r0;
    const double* Gt = G + (int64_t)t * N * 3;
    double* Ht = H + (int64_t)t * N * 3;
    const double hx = Ht[3 * (int64_t)x], hy = Ht[3 * (int64_t)x + 1], hz = Ht[3 * (int64_t)x + 2];
    int32_t v[8];
    double g[8][3];
#pragma unroll
    for (int k = 0; k < 8; ++k) {          // all children's loads in flight at once
      const int64_t c = kids[k] < 0 ? kids[0] : kids[k];
      v[k] = r[c].v;
#pragma unroll
      for (int a = 0; a < 3; ++a) g[k][a] = Gt[3 * c + a];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (kids[k] < 0) break;
      const int64_t c = kids[k];
      double ax = hx, ay = hy, az = hz;
      if (v[k] > 0) {
        const double iv = 1.0 / (double)v[k];
        ax += g[k][0] * iv;
        ay += g[k][1] * iv;
        az += g[k][2] * iv;
      }
      Ht[3 * c] = ax;
      Ht[3 * c + 1] = ay;
      Ht[3 * c + 2] = az;
    }
  }
}

// The chunks' passes top-down: the nodes that cross runs of chunks, then chunk ends, then
// those inside (the refresh's kernels in the other order).
__global__ void __launch_bounds__(kCross2Block) push_cross_k(
    const int32_t* __restrict__ cross, const int32_t* __restrict__ kids_of, int count,
    const NodeRec* __restrict__ r0, const NodeRec* __restrict__ r1, const double* __restrict__ G,
    double* H, int64_t N) {
  __shared__ uint32_t depths;
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  uint32_t left = cross_depths(cross, count, c, &depths);
  if (left == 0) return;
  CrossNode next(cross, kids_of, count, c, __ffs((int)left) - 1);
  while (left) {
    const CrossNode at = next;
    left &= left - 1;
    if (left) next = CrossNode(cross, kids_of, count, c, __ffs((int)left) - 1);
    if (at.x >= 0) push_node(at.x, at.kids, r0, r1, G, H, N);
    __syncthreads();
  }
}

template <bool ONE>
__global__ void __launch_bounds__(512) push_chunk_k(Chunks C, const NodeRec* __restrict__ r0,
                                                   const NodeRec* __restrict__ r1,
                                                   const double* __restrict__ G, double* H,
                                                   int64_t N) {
  constexpr int kRoom = ONE ? kSkipRoomOne : kSkipRoom;
  __shared__ int32_t skips[kRoom];
  const int32_t x0 = C.x[blockIdx.x], x1 = C.x[blockIdx.x + 1];
  for (int32_t x = x0 + (int)threadIdx.x; x < x1 && x - x0 < kRoom; x += blockDim.x)
    skips[x - x0] = C.skip[x];
  __syncthreads();
  const ChunkSkips S{skips, C.skip, x0, kRoom};
  const int32_t* off = C.off + (int64_t)blockIdx.x * (kDepths + 1);
  const int32_t* nodes = C.nodes + x0;
  for (int k = kDepths; k >= 1; --k) {
    const int32_t lo = off[k - 1], hi = off[k];
    if (hi == lo) continue;                        // (uniform over the block)
    for (int32_t q = lo + (int)threadIdx.x; q < hi; q += blockDim.x) {
      int32_t kids[8];
      S.kids(nodes[q], S(nodes[q]), kids);
      push_node(nodes[q], kids, r0, r1, G, H, N);
    }
    __syncthreads();
  }
}

// Neurons: dpos_j += sum_t v_j^t H^t(leaf of j); then convert to float32.
__global__ void push_leaves_k(const int32_t* __restrict__ leaf_of, const int32_t* __restrict__ nbeg,
                              const int32_t* __restrict__ nend, const int32_t* __restrict__ order,
                              const NodeRec* __restrict__ r0, const NodeRec* __restrict__ r1,
                              const int32_t* __restrict__ vs0, const int32_t* __restrict__ vs1,
                              const double* __restrict__ H, int64_t N, int64_t n,
                              const double* __restrict__ dpos64, float* __restrict__ dpos) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int32_t x = leaf_of[j];
  // in a bucket, the neuron's position in sorted order, to read its per-type counts
  const bool bucket = (r0[x].meta & kBucketBit) != 0;
  int32_t p = 0;
  if (bucket) {
    p = nbeg[x];
    while (p < nend[x] && order[p] != (int32_t)j) ++p;
  }
  double a[3] = {dpos64[3 * j], dpos64[3 * j + 1], dpos64[3 * j + 2]};
  for (int t = 0; t < 2; ++t) {
    const int32_t v = bucket ? (t ? vs1[p] : vs0[p]) : (t ? r1[x].v : r0[x].v);
    if (v <= 0) continue;
    const double* Ht = H + (int64_t)t * N * 3 + 3 * (int64_t)x;
    for (int k = 0; k < 3; ++k) a[k] += (double)v * Ht[k];
  }
  for (int k = 0; k < 3; ++k) dpos[3 * j + k] = (float)a[k];
}

}  // namespace msp
