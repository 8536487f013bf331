// Class lists of the attention kernels from the neighbour counts: centre i goes
// to the first launched class (bit set active, the top class among them) that
// holds its neighbours.  count [8] (zeroed beforehand, in LDS or in memory):
// centres listed per class [0..3], centres per neighbour-count class [4..7];
// clist [4][nloc].  Called by whole wavefronts; i at or past nloc counts nowhere.
#ifndef DPA1_ATTN_CLASSES_H
#define DPA1_ATTN_CLASSES_H

#include <hip/hip_runtime.h>

namespace dpa1 {

__device__ __forceinline__ void attn_class_lists(int i, const int *nnei, int nloc, int active,
                                                 int *count, int *clist) {
  const int lane = threadIdx.x & 63;
  const int n = i < nloc ? nnei[i] : 0;
  const int nat = n > 0 ? (n - 1) >> 5 : -1;
  int cls = nat;
  if (cls >= 0)
    while (cls < 3 && !((active >> cls) & 1)) ++cls;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const unsigned long long bn = __ballot(nat == c);
    if (bn != 0ull && lane == __ffsll((long long)bn) - 1) atomicAdd(&count[4 + c], __popcll(bn));
    const unsigned long long b = __ballot(cls == c);
    if (b == 0ull) continue;
    const int leader = __ffsll((long long)b) - 1;
    int pos0 = 0;
    if (lane == leader) pos0 = atomicAdd(&count[c], __popcll(b));
    pos0 = __shfl(pos0, leader);
    if (cls == c) clist[(size_t)c * nloc + pos0 + __popcll(b & ((1ull << lane) - 1ull))] = i;
  }
}

}  // namespace dpa1

#endif  // DPA1_ATTN_CLASSES_H
