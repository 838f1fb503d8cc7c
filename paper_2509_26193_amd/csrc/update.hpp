// One connectivity update after the search (Sec. III-A, "Update of synapses" and
// "Update of synaptic elements"), enqueued as kernels only: the request acceptance
// (commit), the recording of the new synapses, and the plasticity step (growth,
// deletion, retraction, vacancies). Every count the sequence needs (requests,
// synapses, retraction candidates, survivors) may be known on the host or only on the
// device (DevCount); nothing is read back and nothing is allocated, so the same
// sequence serves the host entry points (which then read their status once) and the
// update cycle (msp_cycle), which captures it in a graph.
#pragma once

#include "commit.hpp"
#include "plasticity.hpp"
#include "scan.hpp"

namespace msp {

// ---------------------------------------------------------------------------- commit
// Working memory of the acceptance of up to `cap_S` requests among n neurons.
struct CommitWs {
  int32_t* src_of;
  int64_t* key;
  uint64_t* prio;
  int32_t* cnt;                 // [2n] requests per group, then the accepted ones; the flags
  int32_t* within;              // [cap_S] each request's place in its group
  GroupThr* thr;                // [2n] each group's decision
  int32_t* seg_off;             // [2n + 1]
  int32_t* seg;
  uint8_t* acc;
  int64_t* dst;                 // [cap_S + 1]
  int32_t* flags;               // [1] kErrArgs, kCommitCapacity
  void* scan_ws;
};

inline CommitWs commit_ws(void* base, int64_t n, int64_t cap_S, size_t* bytes) {
  Carver c{static_cast<char*>(base)};
  CommitWs w;
  w.src_of = c.take<int32_t>(cap_S);
  w.key = c.take<int64_t>(cap_S);
  w.prio = c.take<uint64_t>(cap_S);
  w.cnt = c.take<int32_t>(2 * n + 1);
  w.flags = w.cnt ? w.cnt + 2 * n : nullptr;
  w.within = c.take<int32_t>(cap_S);
  w.thr = c.take<GroupThr>(2 * n);
  w.seg_off = c.take<int32_t>(2 * n + 1);
  w.seg = c.take<int32_t>(cap_S);
  w.acc = c.take<uint8_t>(cap_S);
  w.dst = c.take<int64_t>(cap_S + 1);
  w.scan_ws = c.take_bytes(std::max(scan_tmp_bytes<int32_t>(2 * n),
                                    scan_tmp_bytes<int64_t>(cap_S + 1)));
  *bytes = c.off;
  return w;
}

// The S requests (slots of `target` in (source, element) order; elem_offset [n + 1])
// compete per (target, type) group for its vacancies; the accepted ones become
// synapses at syn_* [0, *n_formed) and take one vacancy of each side. If the accepted
// requests exceed syn_capacity, or a target is >= n, nothing is written and
// *n_formed = 0 (w.flags says which).
inline hipError_t enqueue_commit(const CommitWs& w, const int32_t* target,
                                 const int64_t* elem_offset, const uint8_t* neuron_type,
                                 int64_t n, DevCount S, int32_t* vac_axon, int32_t* vac_exc,
                                 int32_t* vac_inh, uint64_t seed, DevStep step, int32_t* syn_src,
                                 int32_t* syn_tgt, uint8_t* syn_type, int64_t syn_capacity,
                                 int64_t* n_formed, uint8_t* accepted_out, hipStream_t s) {
  const unsigned gs = grid_cap(S.v, kCommitBlock);
  commit_start_k<<<grid_for(n + 1, kCommitBlock), kCommitBlock, 0, s>>>(elem_offset, n, S,
                                                                       w.src_of, w.cnt);
  req_key_k<<<gs, kCommitBlock, 0, s>>>(target, elem_offset, w.src_of, neuron_type, S, n, seed,
                                        step, w.key, w.prio, w.cnt, w.within, w.flags);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = exclusive_scan<int32_t, int32_t, Ident<int32_t>>(w.cnt, w.seg_off, 2 * n, Ident<int32_t>(),
                                                       true, s, w.scan_ws);
  if (e != hipSuccess) return e;
  req_scatter_k<<<gs, kCommitBlock, 0, s>>>(w.key, S, w.seg_off, w.within, w.seg);
  // decisions per group (w.cnt now takes each group's accepted count), then per request
  const unsigned gg = grid_cap(2 * n, kCommitBlock);
  group_thr_k<<<gg, kCommitBlock, 0, s>>>(w.prio, w.seg_off, w.seg, 2 * n, vac_exc, vac_inh,
                                          w.thr, w.cnt);
  req_decide_k<<<gs, kCommitBlock, 0, s>>>(w.key, w.prio, w.thr, w.seg_off, w.seg, S, vac_exc,
                                           vac_inh, w.acc);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = exclusive_scan<int64_t, uint8_t, AccFlag>(w.acc, w.dst, S.v, AccFlag(), true, s, w.scan_ws,
                                                S.p);
  if (e != hipSuccess) return e;
  commit_end_k<<<std::max(gs, gg), kCommitBlock, 0, s>>>(
      w.acc, w.dst, w.key, w.src_of, w.cnt, elem_offset, n, S, syn_capacity, syn_src, syn_tgt,
      syn_type, accepted_out, vac_exc, vac_inh, vac_axon, n_formed, w.flags);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------- plasticity
struct PlastConst {
  Growth growth;                            // growth rule (see grow)
  double delete_fraction;
};

// Working memory of a plasticity step over a list of up to cap_m synapses.
struct PlastWs {
  uint8_t* dead;
  uint64_t* key;                // [cap_m] deletion priorities, then the retraction candidates
  int32_t* pos;                 // [cap_m + 1] places among the candidates, then the survivors
  DelWs del;
  RetractWs ret;                // (2n owners)
  void* scan_ws;
  SynList O;                    // the survivors, compacted
  int64_t* cnt;                 // [1] survivors
};

inline PlastWs plast_ws(void* base, int64_t n, int64_t cap_m, size_t* bytes) {
  Carver c{static_cast<char*>(base)};
  const int64_t blocks = kStrideGrid;
  PlastWs w;
  w.dead = c.take<uint8_t>(cap_m);
  w.key = c.take<uint64_t>(cap_m);
  w.pos = c.take<int32_t>(cap_m + 1);
  w.del.st = c.take<DelSelect>(1);
  w.del.below = c.take<int64_t>(blocks);
  w.del.kept = c.take<int32_t>(blocks);
  w.del.ckey = c.take<uint64_t>(blocks * kDelRoom);
  w.del.cidx = c.take<int32_t>(blocks * kDelRoom);
  w.ret.exc = c.take<uint32_t>(2 * n);
  w.ret.cnt = c.take<int32_t>(2 * n);
  w.ret.off = c.take<int32_t>(2 * n);
  w.ret.flag = c.take<uint8_t>(cap_m);
  w.ret.within = w.pos;
  w.ret.seg = w.key;
  w.ret.nlarge = c.take<int32_t>(2);
  w.ret.large = c.take<int32_t>(cap_m / kSegSmall + 1);
  w.ret.huge = c.take<int32_t>(cap_m / kSegLarge + 1);
  w.scan_ws = c.take_bytes(std::max(scan_tmp_bytes<int32_t>(cap_m + 1),
                                    scan_tmp_bytes<int32_t>(2 * n)));
  w.O.src = c.take<int32_t>(cap_m);
  w.O.tgt = c.take<int32_t>(cap_m);
  w.O.type = c.take<uint8_t>(cap_m);
  w.cnt = c.take<int64_t>(1);
  *bytes = c.off;
  return w;
}

// Growth, deletion and retraction over the m synapses of L, then the vacancies
// (plasticity.hpp states the rules). The survivors keep their order; their count goes
// to *m_out (which may be m's own device count: it is written last).
inline hipError_t enqueue_plasticity(const PlastWs& w, int64_t n, const PlastConst& c,
                                     uint64_t seed, DevStep step, double* z, int32_t* bound,
                                     SynList L, DevCount m, int64_t* m_out, int32_t* vac_axon,
                                     int32_t* vac_exc, int32_t* vac_inh, hipStream_t s) {
  const unsigned gm = grid_cap(m.v, kPlastBlock);
  const bool del = m.v > 0 && c.delete_fraction > 0.0;
  // (the blocks that draw priorities are those of a launch over the list, bounded alike)
  const unsigned gg = std::max(gm, grid_cap(3 * n, kPlastBlock));
  DelWs dw = w.del;
  if (!del) dw.st = nullptr;
  grow_draw_k<<<gg, kPlastBlock, 0, s>>>(z, n, c.growth, c.delete_fraction, m, seed, step, w.key,
                                         dw);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t* survivors = nullptr;
  if (m.v > 0) {
    if (del) del_pick_k<<<1, kPickBlock, 0, s>>>(c.delete_fraction, m, (int)gg, w.key, w.del);
    del_mark_k<<<gm, kPlastBlock, 0, s>>>(w.key, m, dw.st, L, n, w.dead, bound);
    for (int k = 0; k < 2; ++k) {
      const int64_t owners = k == 0 ? n : 2 * n;
      excess_k<<<grid_for(owners, kPlastBlock), kPlastBlock, 0, s>>>(bound + k * n, z + k * n,
                                                                    owners, w.ret);
      retract_count_k<<<gm, kPlastBlock, 0, s>>>(L, n, k, w.dead, m, w.ret);
      e = exclusive_scan<int32_t, int32_t, Ident<int32_t>>(w.ret.cnt, w.ret.off, owners,
                                                           Ident<int32_t>(), false, s, w.scan_ws);
      if (e != hipSuccess) return e;
      retract_lay_k<<<gm, kPlastBlock, 0, s>>>(L, n, k, m, seed, step, w.ret);
      retract_k<<<gm, kPlastBlock, 0, s>>>(L, n, k, m, w.dead, bound, w.ret);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    e = exclusive_scan<int32_t, int32_t, LiveFlag>(nullptr, w.pos, m.v, LiveFlag{w.dead}, true, s,
                                                   w.scan_ws, m.p);
    if (e != hipSuccess) return e;
    compact_k<<<gm, kPlastBlock, 0, s>>>(L, w.dead, w.pos, m, w.O, w.cnt);
    copy_list_k<<<gm, kPlastBlock, 0, s>>>(w.O, DevCount{m.v, w.cnt}, L);
    survivors = w.cnt;
  }
  vacancy_k<<<grid_for(3 * n, kPlastBlock), kPlastBlock, 0, s>>>(z, bound, n, vac_axon, vac_exc,
                                                                vac_inh, survivors, m_out);
  return hipGetLastError();
}

}  // namespace msp
