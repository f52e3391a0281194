// Bits of activation sets: transposition across lanes, and the longest gap in a set.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace lazyev {

// Transposes the N x N bits of N lanes (16 or 32; lane c of each group of N): bit x of lane c -> bit c of
// lane x.  Of N = 16 the bits are kept twice in the register, so that a rotation by s serves the lower and (by 32 - s)
// the upper half.  lane ^ 1, 2, 4 (= 7 ^ 3) and 8 are data-parallel moves within the vector ALU.
template <int N>
__device__ __forceinline__ unsigned transpose_bits(unsigned bits, int c) {
  static_assert(N == 16 || N == 32, "");
  unsigned m = N == 16 ? bits | (bits << 16) : bits;
  auto step = [&](unsigned other, int s, unsigned keep) {
    const bool up = c & s;
    const unsigned turned = __builtin_amdgcn_alignbit(other, other, up ? s : 32 - s);   // rotated right
    const unsigned k = up ? ~keep : keep;
    m = (m & k) | (turned & ~k);
  };
  auto move = [](unsigned x, auto ctrl) { return static_cast<unsigned>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), decltype(ctrl)::value, 0xF, 0xF, true)); };
  if (N == 32) step(static_cast<unsigned>(__builtin_amdgcn_ds_swizzle(static_cast<int>(m), 0x401F)), 16, 0x0000FFFFu);   // lane ^ 16
  step(move(m, std::integral_constant<int, 0x128>{}), 8, 0x00FF00FFu);       // row_ror:8
  step(move(move(m, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{}), 4, 0x0F0F0F0Fu);   // row_half_mirror, quad_perm 3 2 1 0
  step(move(m, std::integral_constant<int, 0x4E>{}), 2, 0x33333333u);        // quad_perm 2 3 0 1
  step(move(m, std::integral_constant<int, 0xB1>{}), 1, 0x55555555u);        // quad_perm 1 0 3 2
  return N == 16 ? m & 0xFFFFu : m;
}

// Length of the longest run of ones among the lowest N bits of z (fewer than N): x2, x4, ... mark where 2, 4, ...
// ones in a row start.
template <int N>
__device__ __forceinline__ int longest_run(unsigned z) {
  const unsigned x2 = z & (z >> 1), x4 = x2 & (x2 >> 2), x8 = x4 & (x4 >> 4), x16 = N > 16 ? x8 & (x8 >> 8) : 0u;
  int r = 0;
  unsigned at = ~0u, t;                            // starts of runs of at least r ones
  if (N > 16 && x16) { r = 16; at = x16; }
  t = at & (x8 >> r);
  if (t) { r += 8; at = t; }
  t = at & (x4 >> r);
  if (t) { r += 4; at = t; }
  t = at & (x2 >> r);
  if (t) { r += 2; at = t; }
  return (at & (z >> r)) ? r + 1 : r;
}

// The largest distance between neighbouring ones of `set` whose lowest and highest ones are lo < hi.
template <int N>
__device__ __forceinline__ int longest_gap(unsigned set, int lo, int hi) {
  return 1 + longest_run<N>(~set & ((1u << hi) - (1u << lo)));
}

// Alg. 1 (first loop) and Eq. 1 for one entry and up to 32 calls of consecutive steps: bit s of `calls` says that it
// was active at step t + s.
__device__ __forceinline__ void apply_calls(unsigned calls, int32_t t, int32_t &ts, int32_t &mri) {
  if (calls == 0) return;
  const int lo = __builtin_ctz(calls), hi = 31 - __builtin_clz(calls);
  mri = max(mri, t + lo - ts);
  if (hi > lo) mri = max(mri, longest_gap<32>(calls, lo, hi));
  ts = t + hi;
}

}  // namespace lazyev
