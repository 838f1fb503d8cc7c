// Electrical activity between connectivity updates (Sec. II, "Update of electrical
// activity"), with the firing-rate approximation of Sec. IV-B. One step is 1 ms:
//   * exchange: the spike a source recorded in the previous step reaches the target.
//     Exact synapses are grouped by source once per run (act_setup_k, act_group_k),
//     and a neuron that spikes delivers along its own group into the next step's
//     arrival counts (act_neuron_k; act_deliver_k for the spikes recorded before the
//     run), so a step touches only the synapses of the neurons that fired.
//     Approximated synapses (approx 1: those whose two neurons carry different ranks;
//     approx 2: all) carry a spike at step t iff u < f_i, f_i being the source's
//     frequency over the previous epoch (spikes per step) and u = (Philox word 0 >> 11)
//     2^-53, key (seed, 5), counter (s, t, 0, 0) (one thread per synapse and step: with the
//     step before, or in act_approx_k). Targets count excitatory and inhibitory arrivals
//     (exact integer atomics, so the order of the deliveries does not matter);
//   * neuron model (act_neuron_k, one thread per neuron): Izhikevich 2003, regular
//     spiking (excitatory) or fast spiking (inhibitory):
//       I = w_e e - w_i h + mu + width (u' - 1/2), u' from key (seed, 6), counter (g, t, 0, 0);
//       v += (0.04 v^2 + 5 v + 140 - u + I) / 2, twice (two half-millisecond steps);
//       u += a (b v - u); v >= 30: spike, v = c, u += d;
//   * calcium, a running average of the spikes: Ca -= Ca / tau, then += beta on a spike;
//   * a step t with (t + 1) % delta == 0 closes an epoch: f = spikes in it / delta.
// Only +, -, * and comparisons on fp64 (1/tau and 1/delta come from the host), with
// no contraction, so every value is exactly the IEEE evaluation of these formulas.
#pragma once

#include "common.hpp"

namespace msp {

constexpr int kActBlock = 256;
constexpr unsigned kApproxBlocks = 2048; // blocks of the approximated synapses, at most
constexpr unsigned kSpikeSlots = 1024;   // spike counters of the blocks

struct ActParams {
  double a[2], b[2], c[2], d[2];   // per neuron type (0 excitatory, 1 inhibitory)
  double w_e, w_i, mu, width, beta, inv_tau, inv_delta;
  int32_t delta;
};

// Start of the activity (one thread per neuron): the membrane potential at the reset
// value c of the neuron's type, the recovery variable at its resting relation u = b c,
// no calcium, no spike, an empty epoch and no frequency yet.
__global__ void __launch_bounds__(kActBlock) act_init_k(
    int64_t n, const uint8_t* __restrict__ type, ActParams P, double* __restrict__ v,
    double* __restrict__ u, double* __restrict__ calcium, uint8_t* __restrict__ spiked,
    int32_t* __restrict__ count, double* __restrict__ freq, int32_t* err) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const uint8_t t8 = type[g];
  if (t8 > 1) atomicOr(err, 1);
  const int t = t8 ? 1 : 0;
  v[g] = P.c[t];
  u[g] = P.b[t] * P.c[t];
  calcium[g] = 0.0;
  spiked[g] = 0;
  count[g] = 0;
  freq[g] = 0.0;
}

// Run setup, one thread per synapse: a synapse with an endpoint outside [0, n) or a
// type > 1 sets *err and takes no part in the run; with approx 1, remote[s] = 1 marks the
// approximated ones (neurons of different ranks: the two rank gathers are paid once per run,
// not every step). The exact ones are grouped by source: each is counted at its source (cnt)
// and keeps its place there (within; -1: not exact), and act_group_k puts its target there.
// Bound by the atomics, which memory carries out one by one (7.5 M synapses of 8M neurons: 290
// us and the grouping 222, 357 with a second atomic per synapse; sorting them by source takes
// 340 instead of 510 us, but its buffers cost the call more than that).
__global__ void __launch_bounds__(kActBlock) act_setup_k(
    int64_t n, int64_t m, const int32_t* __restrict__ src, const int32_t* __restrict__ tgt,
    const uint8_t* __restrict__ stype, const int32_t* __restrict__ rank, int32_t approx,
    int32_t* cnt, int32_t* __restrict__ within, uint8_t* __restrict__ remote, int32_t* err) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const int32_t i = src[s], g = tgt[s];
  const bool ok = i >= 0 && i < n && g >= 0 && g < n && stype[s] <= 1;
  if (!ok) atomicOr(err, 1);
  const bool approxd = approx == 2 || (approx == 1 && ok && rank[i] != rank[g]);
  if (remote) remote[s] = ok && approxd ? 1 : 0;
  if (within) within[s] = ok && !approxd ? atomicAdd(&cnt[i], 1) : -1;
}

__global__ void __launch_bounds__(kActBlock) act_group_k(
    int64_t m, const int32_t* __restrict__ src, const int32_t* __restrict__ tgt,
    const uint8_t* __restrict__ stype, const int32_t* __restrict__ soff,
    const int32_t* __restrict__ within, uint32_t* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const int32_t q = within[s];
  if (q >= 0) out[soff[src[s]] + q] = (uint32_t)tgt[s] | ((uint32_t)stype[s] << 31);
}

// The arrival counts of one step: excitatory e[n], inhibitory h[n].
struct Arrivals {
  int32_t* e;
  int32_t* h;

  __device__ __forceinline__ void add(int32_t g, bool inh) const {
    atomicAdd(inh ? &h[g] : &e[g], 1);
  }
};

// The exact synapses by source: out[off[i] .. off[i + 1]) are the targets of neuron i, with
// the synapse's type in the top bit, so that a spike is two gathers away from its targets
// (off null: none).
struct Exact {
  const int32_t* off;
  const uint32_t* out;
};

// A spike along the exact synapses [q, q1) of its neuron, four targets read at a time.
__device__ __forceinline__ void act_send(int32_t q, int32_t q1, const uint32_t* __restrict__ out,
                                         const Arrivals& A) {
  for (; q < q1; q += 4) {
    uint32_t to[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) to[k] = out[q + k < q1 ? q + k : q];
    // (all four before the first is used: the compiler would wait for each in turn)
    asm volatile("" : "+v"(to[0]), "+v"(to[1]), "+v"(to[2]), "+v"(to[3]));
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (q + k < q1) A.add((int32_t)(to[k] & 0x7FFFFFFFu), to[k] >> 31);
  }
}

// The spikes recorded before the run (spk), delivered for its first step.
__global__ void __launch_bounds__(kActBlock) act_deliver_k(int64_t n,
                                                          const uint8_t* __restrict__ spk,
                                                          Exact X, Arrivals A) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n || !spk[g]) return;
  act_send(X.off[g], X.off[g + 1], X.out, A);
}

// The approximated synapses of approx 1, packed in synapse order (pos: exclusive scan
// of remote): their index (the draw's counter), endpoints and type.
__global__ void __launch_bounds__(kActBlock) act_pack_k(
    int64_t m, const int32_t* __restrict__ src, const int32_t* __restrict__ tgt,
    const uint8_t* __restrict__ stype, const uint8_t* __restrict__ remote,
    const int32_t* __restrict__ pos, int32_t* __restrict__ aidx, int32_t* __restrict__ asrc,
    int32_t* __restrict__ atgt, uint8_t* __restrict__ atype) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m || !remote[s]) return;
  const int32_t q = pos[s];
  aidx[q] = (int32_t)s;
  asrc[q] = src[s];
  atgt[q] = tgt[s];
  atype[q] = stype[s];
}

// The approximated synapses: the packed list of approx 1 (idx non-null, count *count), or
// every synapse with valid endpoints (approx 2).
struct Approximated {
  const int32_t* src;
  const int32_t* tgt;
  const uint8_t* type;
  const int32_t* idx;
  const int32_t* count;
  int64_t m;
};

// Approximated synapse q at step t.
__device__ __forceinline__ void act_approx(int64_t q, int64_t n, const Approximated& S,
                                           uint64_t seed, uint64_t t,
                                           const double* __restrict__ freq, const Arrivals& A) {
  int32_t i = S.src[q], g = S.tgt[q], ty = S.type[q], x = S.idx ? S.idx[q] : 0;
  asm volatile("" : "+v"(i), "+v"(g), "+v"(ty), "+v"(x));       // (loaded together)
  if (i < 0 || i >= n || g < 0 || g >= n || ty > 1) return;     // reported at setup
  const uint64_t s = S.idx ? (uint64_t)x : (uint64_t)q;
  const double u = (double)(philox_word0(seed, 5, s, t, 0, 0) >> 11) * 0x1p-53;
  if (u < freq[i]) A.add(g, ty);
}

__global__ void __launch_bounds__(kActBlock) act_approx_k(int64_t n, Approximated S, uint64_t seed,
                                                         uint64_t t,
                                                         const double* __restrict__ freq,
                                                         Arrivals A) {
  const int64_t count = S.idx ? (int64_t)*S.count : S.m;
  for (int64_t q = (int64_t)blockIdx.x * kActBlock + threadIdx.x; q < count;
       q += (int64_t)gridDim.x * kActBlock)
    act_approx(q, n, S, seed, t, freq, A);
}

// One step: the arrivals A are consumed (and cleared for the step after next) here; a
// neuron that fires sends along its exact synapses into the next step's B. The blocks from `neurons` on, if there are any, take the next step's
// approximated synapses, which need nothing of this step unless it closes an epoch: a launch
// less per step.
// Bound by memory in large networks: per neuron 8 bytes read and written for each of v, u
// and calcium, 4 for each arrival count, 1 + 1 for its type and spike; the epoch's count only
// where it changes (8M neurons at 15 Hz: 151 -> 125 us, 0.5 GB; marks of neurons with
// arrivals, to skip the others' counts, and two or four neurons per thread gain nothing). In
// small ones by the chain of loads behind a spike (131 101 neurons, 2 synapses each: 8.7 +
// 3.0 us in two launches -> 6.6 us in one).
__global__ void __launch_bounds__(kActBlock) act_neuron_k(
    int64_t n, unsigned neurons, const uint8_t* __restrict__ ntype, ActParams P, uint64_t seed,
    uint64_t t, bool closes, double* __restrict__ v, double* __restrict__ u,
    double* __restrict__ ca, uint8_t* __restrict__ spk, int32_t* __restrict__ count,
    double* __restrict__ freq, Arrivals A, int32_t* __restrict__ last_input,
    unsigned long long* part, Exact X, Arrivals B, Approximated S) {
  if (blockIdx.x >= neurons) {
    const int64_t total = S.idx ? (int64_t)*S.count : S.m;
    for (int64_t q = (int64_t)(blockIdx.x - neurons) * kActBlock + threadIdx.x; q < total;
         q += (int64_t)(gridDim.x - neurons) * kActBlock)
      act_approx(q, n, S, seed, t + 1, freq, B);
    return;
  }
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool f = false;
  if (g < n) {
    const int k = ntype[g] ? 1 : 0;
    double vv = v[g], w = u[g], c = ca[g];
    const int32_t ne = A.e[g], nh = A.h[g];
    A.e[g] = 0;
    A.h[g] = 0;
    if (last_input) {
      last_input[g] = ne;
      last_input[n + g] = nh;
    }
    const double uu = (double)(philox_word0(seed, 6, (uint64_t)g, t, 0, 0) >> 11) * 0x1p-53;
    const double I = P.w_e * (double)ne - P.w_i * (double)nh + (P.mu + P.width * (uu - 0.5));
    vv = vv + 0.5 * (0.04 * vv * vv + 5.0 * vv + 140.0 - w + I);
    vv = vv + 0.5 * (0.04 * vv * vv + 5.0 * vv + 140.0 - w + I);
    w = w + P.a[k] * (P.b[k] * vv - w);
    f = vv >= 30.0;
    if (f) {
      vv = P.c[k];
      w = w + P.d[k];
    }
    if (f && X.off) act_send(X.off[g], X.off[g + 1], X.out, B);
    v[g] = vv;
    u[g] = w;
    c = c - c * P.inv_tau;
    if (f) c = c + P.beta;
    ca[g] = c;
    spk[g] = f ? 1 : 0;
    if (f || closes) {
      const int32_t cnt = count[g] + (f ? 1 : 0);
      if (closes) freq[g] = (double)cnt * P.inv_delta;
      count[g] = closes ? 0 : cnt;
    }
  }
  if (part) {                       // this block's spikes, added to its slot
    __shared__ int32_t wave_spikes[kActBlock / 64];
    const uint64_t b = __ballot(f);
    if ((threadIdx.x & 63) == 0) wave_spikes[threadIdx.x >> 6] = __popcll(b);
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t sum = 0;
      for (int w = 0; w < kActBlock / 64; ++w) sum += wave_spikes[w];
      if (sum) atomicAdd(&part[blockIdx.x % kSpikeSlots], (unsigned long long)sum);
    }
  }
}

// Sum of the blocks' spike counts, added to *spikes (one block).
__global__ void __launch_bounds__(kActBlock) act_spikes_k(const int64_t* __restrict__ part,
                                                         int64_t slots, int64_t* spikes) {
  __shared__ int64_t acc[kActBlock];
  int64_t sum = 0;
  for (int64_t q = threadIdx.x; q < slots; q += kActBlock) sum += part[q];
  acc[threadIdx.x] = sum;
  __syncthreads();
  for (int w = kActBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) acc[threadIdx.x] += acc[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *spikes += acc[0];
}

}  // namespace msp
