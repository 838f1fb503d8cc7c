// Launches the library's selection of a key by its rank (csrc/plasticity.hpp) on given arrays,
// for tests of forms that uniform priorities do not reach.
#include <algorithm>

#include "plasticity.hpp"

using namespace msp;

template <int THREADS>
__global__ void __launch_bounds__(THREADS) kth_k(const uint64_t* key, int64_t c, const int64_t* r,
                                                 uint64_t* out_key, int64_t* out_index) {
  __shared__ PickRoom<THREADS> room;
  const DelSelect d = kth_key(key, c, r[blockIdx.x], room);
  if (threadIdx.x == 0) {
    out_key[blockIdx.x] = d.key;
    out_index[blockIdx.x] = d.index;
  }
}

extern "C" {

// The r[q]-th smallest (1 <= r[q] <= c) of c device keys, for q < count, by blocks of 256
// threads or of 1 024. Every pointer is a device pointer.
int probe_kth(const uint64_t* key, int64_t c, const int64_t* r, int count, int threads,
              uint64_t* out_key, int64_t* out_index) {
  if (c < 1 || count < 1 || (threads != kPlastBlock && threads != kPickBlock)) return 1;
  if (threads == kPlastBlock)
    kth_k<kPlastBlock><<<count, kPlastBlock>>>(key, c, r, out_key, out_index);
  else
    kth_k<kPickBlock><<<count, kPickBlock>>>(key, c, r, out_key, out_index);
  return hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess;
}

// del_pick_k over m keys, with what `blocks` blocks of the draw would have counted and kept
// (below, kept [blocks]; ckey, cidx [blocks][kDelRoom]). st: the selection, 16 bytes.
int probe_del_pick(double frac, int64_t m, int blocks, const uint64_t* key, int64_t* below,
                   int32_t* kept, uint64_t* ckey, int32_t* cidx, void* st) {
  if (m < 1 || blocks < 1 || blocks > (int)kStrideGrid) return 1;
  const DelWs W{static_cast<DelSelect*>(st), below, kept, ckey, cidx};
  del_pick_k<<<1, kPickBlock>>>(frac, host_count(m), blocks, key, W);
  return hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess;
}

int probe_del_room() { return kDelRoom; }

}  // extern "C"
