// What the decode kernel that leaves a call's candidate records and the kernels that read them share.
#pragma once
#include <hip/hip_runtime.h>

namespace lazyev {
namespace {

// x / y for 0 <= x < 2^24, y > 0, the same in all lanes of a wave: the compiler's own sequence for a divisor that it does
// not know is some thirty instructions, in a chain.  The rounded quotient is off by one at most.
__host__ __device__ inline int wave_div(int x, int y) {
#ifdef __HIP_DEVICE_COMPILE__
  if (!__builtin_constant_p(y)) {
    int q = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<float>(x) * __builtin_amdgcn_rcpf(static_cast<float>(y))));
    const int r = x - q * y;
    q += r >= y ? 1 : 0;
    return q - (r < 0 ? 1 : 0);
  }
#endif
  return x / y;
}

constexpr int kWaves = 4;               // stream waves of a block
constexpr int kHeadPad = 8;             // logits and statistics are stored for 8 heads per unit
// Most sub-tiles one wave takes.
__host__ __device__ inline int fused_wave_run(int n_sub, int n_split) {
  return wave_div(n_sub + kWaves * n_split - 1, kWaves * n_split);
}
// How a unit's n_sub sub-tiles of 16 entries are dealt to the kWaves * n_split waves of its
// n_split blocks: wave wv (= kWaves * (n_split - 1 - split) + wave) takes wv, wv + kWaves * n_split,
// ..., so the waves of a unit read one moving window of the cache together (measured against a
// region of consecutive sub-tiles per block: 28.6 against 29.2 us per call on the 2048-entry
// workload).  The unit's LAST block comes first in that order: when the sub-tiles do not divide
// evenly its waves take the longer runs, and it is the block that finishes the unit,
// so the other blocks' partials are on their way while it still streams.
struct WaveMap { int first, step, cnt; };
__host__ __device__ inline WaveMap fused_wave_map(int n_sub, int n_split, int split, int wave) {
  WaveMap m;
  m.first = (n_split - 1 - split) * kWaves + wave;
  m.step = kWaves * n_split;
  const int run = fused_wave_run(n_sub, n_split);
  m.cnt = m.first + (run - 1) * m.step < n_sub ? run : run - 1;
  return m;
}

// Slots of a block's region of candidate records in a call with n_parts blocks per unit: one
// for the count and one for each entry the block can own.
__host__ __device__ inline int fused_part_cap(int n_old, int n_parts) {
  const int n_sub = (n_old + 1 + 15) >> 4;
  return fused_wave_run(n_sub, n_parts) * (kWaves * 16) + 1;
}

// Records in a block's region, and the entry that one of them names.  A captured call may be replayed when
// calls of other lengths, whose regions begin elsewhere, have used the buffer since, or may leave its own regions under a
// call that is still to be tracked: a count or an index is then any word, and must not lead out of the buffers.
__device__ __forceinline__ int region_count(const float *region, int cap) {
  // (below zero: none; cap instead of cap - 1, which would be another scalar register to keep, 0.1 - 0.2 us a call: the slot
  // behind a unit's last region still lies in the workspace)
  return min(*reinterpret_cast<const int32_t *>(region), cap);
}
__device__ __forceinline__ int record_entry(int word, int n_old) {   // (any other word: the appended entry, which starts in any case)
  return static_cast<int>(min(static_cast<unsigned>(word), static_cast<unsigned>(n_old)));
}

template <bool kPrecise>
__device__ __forceinline__ float exp_of(float x) {
  if constexpr (kPrecise) return expf(x);
  else return __expf(x);
}
// The weight the activation test of Alg. 1 compares with alpha.
template <bool kPrecise>
__device__ __forceinline__ float weight_of(float s, float m, float invl) { return exp_of<kPrecise>(s - m) * invl; }

}  // namespace
}  // namespace lazyev
