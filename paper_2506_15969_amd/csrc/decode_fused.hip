// Decode step of one layer in ONE launch: append, attention (Eq. 4 of the
// paper) and, one call behind, the recurrence tracking of Alg. 1 / Eq. 1.
//
// A unit's cache is cut into 16-entry sub-tiles, dealt to the 4 * n_split stream waves of the
// unit's n_split blocks in turn (fused_wave_map: the waves of a unit read one moving window of the
// cache together, which keeps DRAM pages open).  Per sub-tile a wave
//   loads      K and V as whole 256-byte rows (16 lanes per row), non-temporal; the next
//              sub-tile is requested while the current one is multiplied, the first one from the
//              arguments a wave is handed in registers, before the argument block is read
//   K layout   K rows go through a wave-private LDS area to reach the MFMA operand layout
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, the G query rows padded to 16 columns
//   logits     scaled logits are kept in LDS as [entry][8 heads]; what the tracking needs of
//              them goes to the workspace when the wave's run ends (a store among the loads
//              would hold up the in-order load counter)
//   softmax    per wave: reference maximum m, sum l, output accumulator O.  The reference is
//              raised only when a logit exceeds it by more than 8, so rescaling O is rare;
//              exp(s - m) <= e^8 stays far from overflow
//   O += P V   v_mfma_f32_16x16x16_bf16 after an in-lane 4x8 transpose of the V rows
// The four stream waves of a block merge their (m, l, O) in LDS into one partial per block.
// What follows the stream is serial code of single waves, where instructions, not bytes, set
// the time: no branches where a select does, addresses worked out beforehand.
//
// Partials of a unit.  One block: its partial is the result.  More (decode_fused_split): they are handed over as records of
// stamped 64-bit words (see "hand-over" below): no acknowledgement is waited for, nothing is signalled, one memory
// round trip.  Up to eight blocks: the unit's last one merges the others' records with its own partial.  More: blocks
// of their own behind the stream blocks do (merge_columns), so that few units can have the whole chip, or the unit's last
// block again where the chip is full (merging_blocks).
// The partials are merged in an order that depends on the split and on who merges alone, and the finishing block
// leaves the unit's softmax statistics (max, 1 / sum per head) for the tracking.
//
// Tracking.  The activation test of Alg. 1 needs p = exp(s - m) / l with the statistics of the
// WHOLE unit, which exist only when the unit's last block is done.  Doing it there puts a
// chain of dependent memory round trips at the end of every launch, so it is deferred: the
// NEXT launch carries, behind its stream blocks, as many tracking blocks (spread over the
// compute units the same way) that apply the previous call's tracking from the stored logits
// and statistics (>= alpha test over the query group, TS / MRI update, start of the appended
// entry) while the new call streams; lazyev_stats applies what is pending
// through track_kernel, an eviction in its selection.  Logits and statistics are double-buffered.
// In a uniform batch the tracking blocks do not touch TS / MRI themselves (a 128-byte line read
// and written for every 4-byte word of an active entry, beside the stream): they leave one bit
// per cache entry in the layer's activation log, and track_flush_kernel applies the logged calls
// in step order before anything reads TS / MRI (TrackArgs::bitlog), or the selection of an eviction does.
//
// Candidate lists (kernel instances with kCompact; every call whose
// logits nobody reads as such).  A block knows, once its four stream waves are done, its own
// share of every head's softmax denominator, which bounds the
// true denominator from below: an entry whose weight relative to the BLOCK's denominator
// stays under alpha in every head cannot reach alpha.  The block then writes only the other
// entries ("candidates", about a tenth on the benchmark workloads; the appended entry always)
// as records (7 logits, entry index) into its own region of the logits buffer, and the
// tracking applies the exact test to the records: the same state bit for bit.  A wave whose run
// is longer than the sub-tiles it keeps in LDS (kLong) writes the candidates
// of every full segment while it streams, with the cut that the block's waves' running sums give
// at that moment, and only the last segment after the stream.  Where all blocks of the launch
// fit the chip at once with eight waves each (kListWaves), four more waves per
// block ("list waves") sleep through the stream and build the lists beside the merge.
//
// The above is for bf16 rows of 128 elements.  The other row types (Rows) differ in the loads and the
// two products: bf16 rows of 64 have two sub-tiles on their way and their weights split into three bf16
// terms, fp32 rows need no LDS on the way to v_mfma_f32_16x16x4_f32.  us per call, these against the split +
// merge kernels that served them before: bf16 64, 64 units x 1595 entries 37.5 -> 10.8; fp32 128, 32 x
// 1032 28.3 -> 13.8; fp32 64, 4 x 145 11.5 -> 6.0; 128 units x 6200 entries 203 -> 48.8 (bf16 64), 251 ->
// 147 (fp32 128, 5.5 TB/s), 160 -> 82 (fp32 64).  Out and weights are as far from 64 bits as before.
//
// MFMA operand layouts (lane l, c = l % 16, g = l / 16):
//   16x16x32: A[row c][k = 8g..8g+7]  B[k = 8g..8g+7][col c]  C[row 4g+i][col c]
//   16x16x16: A[row c][k = 4g..4g+3]  B[k = 4g..4g+3][col c]  C[row 4g+i][col c]
//   16x16x4:  A[row c][k = g]  B[k = g][col c]  C[row 4g+i][col c]   (fp32)
// so a lane that owns head c and entries 4g..4g+3 of a sub-tile after the first product already
// holds the A operand of the second.
#include "bits.h"
#include "kernels.h"
#include "track.h"

#include <cfloat>
#include <cstddef>
#include <type_traits>

namespace lazyev {
namespace {

constexpr int kBlock = 256;
static_assert(kWaves == kBlock / 64, "");
constexpr int kFusedSplitMax = 64;      // blocks per unit
constexpr float kRaise = 8.0f;          // the reference maximum moves when exceeded by this much
constexpr int kTrackRows = 3;           // entries per thread per tracking batch
constexpr int kRunMax = 20;             // sub-tiles whose logits a wave keeps in LDS (10 KB) before it writes them out
// Unit and place in the unit of stream block b: the first blocks of all units, the second ones, and so
// on.  A block then waits for blocks of lower indices only, and, as blocks go to the eight XCDs round
// robin, the blocks of a unit share an XCD where the units are a multiple of eight (or two XCDs where they are one of four),
// which makes the hand-over shorter, while the finishing blocks are dealt to all XCDs.  us per call, with
// the blocks of a unit side by side but its finishing block / like this: 32 units x 1040 entries 7.6
// / 6.9, 48 x 1040 9.5 / 8.7, 8 x 2080 9.0 / 8.6, 4 x 9000 12.2 / 11.1; with the finishing block beside the others, 8
// blocks a unit, every finishing block sat on one XCD (2 us more).
// kSplit > 0: the units have kSplit blocks, and no division is needed.
struct BlockPlace { int unit, split; };
template <int kSplit>
__device__ __forceinline__ BlockPlace block_place(int b, int n_split, int units) {
  if constexpr (kSplit > 0) {
    int split = 0, first = 0;
#pragma unroll
    for (int s = 1; s < kSplit; ++s) {
      if (b >= s * units) { split = s; first = s * units; }
    }
    return {b - first, split};
  }
  if (n_split == 1) return {b, 0};
  const int split = wave_div(b, units);
  return {b - split * units, split};
}

#ifdef LAZYEV_TIMELINE
// Measuring build only (liblazyev_timeline.so, see build.py): every block of the LAST launch
// leaves time stamps of the constant 100 MHz counter: 0 block start, 1 first sub-tile multiplied,
// 2 end of wave 0's stream, 3 all four waves done, 4 all partials there, 5 block end (a merging block: 2 half of the unit's
// records there, 3 all there; a tracking block: 0 and 5 only); word 6: the XCD the block ran on (hardware register XCC_ID);
// word 7: 1 a stream block, 2 one that finished its unit, 3 a merging block, 4 a tracking block, and the launch's number times
// 256 (rows of another number are an earlier launch's).  Read with lazyev_timeline_read.
__device__ unsigned long long lz_stamp[2048 * 8];
#define STAMP(i) do { if (threadIdx.x == 0 && blockIdx.x < 2048) lz_stamp[blockIdx.x * 8 + (i)] = wall_clock64(); } while (0)
#define STAMPV(i, v) do { if (threadIdx.x == 0 && blockIdx.x < 2048) lz_stamp[blockIdx.x * 8 + (i)] = (v); } while (0)
__device__ inline unsigned long long xcc_id() {
  unsigned x;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
  return x & 15u;
}
#else
#define STAMP(i) do {} while (0)
#define STAMPV(i, v) do {} while (0)
#endif

typedef unsigned short bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

// two floats as bf16, rounded to nearest even (one instruction), the first in the lower half
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ unsigned pair_to_bf16(float lo, float hi) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// x + (x of lane ^ 16) + (the same of lane ^ 32), and the maximum likewise: the sum / maximum over
// the four lanes c, c + 16, c + 32, c + 48.  v_permlane16_swap / v_permlane32_swap exchange 16-
// and 32-lane halves between two registers in the vector ALU; applied to two copies of x they
// leave the two summands of every lane side by side (same pairs, same roundings as the
// shuffles through the LDS crossbar they replace, which cost a wave a round trip each).
__device__ __forceinline__ float sum_over_lane_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_over_lane_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The same over the eight lanes c, c + 8, ..., c + 56 (a rotation of 8 within the rows of 16 lanes comes first).
__device__ __forceinline__ float lane_8_on(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false));
}
__device__ __forceinline__ float sum_over_eight(float x) { return sum_over_lane_groups(x + lane_8_on(x)); }
__device__ __forceinline__ float max_over_eight(float x) { return max_over_lane_groups(fmaxf(x, lane_8_on(x))); }

// What the kernel needs to know of a row type: bf16 or fp32, 64 or 128 elements.
template <typename T, int D>
struct Rows {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int kBytes = D * static_cast<int>(sizeof(T));
  static constexpr int kLanes = kBytes / 16;       // lanes of 16 bytes that cover a row
  static constexpr int kAcc = D / 16;              // accumulators (16 heads x 16 columns) of the output
  // 16-byte loads per lane and sub-tile: K; V comes in 16-byte pieces, of 64-element bf16 rows in 8-byte ones
  static constexpr int kK = kBytes / 64;
  static constexpr int kV = kBytes >= 256 ? kBytes / 64 : 2;
  // sub-tiles on their way per wave: rows of 128 bytes need two of them for the bytes in flight that
  // one sub-tile of longer rows has
  static constexpr int kDepth = kBytes == 128 ? 2 : 1;
  // fp32 rows of 128 elements take 128 registers for a sub-tile, the accumulators and the queries
  // alone: two waves per SIMD instead of four, so no list waves
  static constexpr bool kWide = kBytes == 512;
  // weights keep their fp32 value in the second product, and exponentials are expf; only the
  // 128-element bf16 rows round the weights to bf16
  static constexpr bool kPrecise = !(sizeof(T) == 2 && D == 128);
  struct SubTile {
    u32x4_t k[kK];
    u32x4_t v[kV];
  };
};
// Two bf16 numbers with infinities and NaNs replaced by zero.
__device__ __forceinline__ unsigned finite_bf16(unsigned w) {
  const unsigned top = ((w & 0x7FFF7FFFu) + 0x00800080u) & 0x80008000u;   // of the halves whose exponent is all ones
  return w & ~((top >> 15) * 0xFFFFu);
}
// ----------------------------------------------------------------------------- tracking
// Alg. 1 (first loop) and Eq. 1 for a share of one unit of a finished decode call:
// probabilities from the stored logits and statistics, >= alpha over the query group, TS / MRI
// update, start of the appended entry.  Part `part` of `n_parts` takes the entries
// track_entry(part, n_parts, r), r = 0, 1, ...
struct TrackBatch {
  float4 sa[kTrackRows], sb[kTrackRows];
};

// Entry that thread `tid` of part `part` (of n_parts) handles in round r: the parts own the
// 16-entry sub-tiles exactly as the stream blocks of a launch with n_parts blocks per unit do
// (fused_wave_map), so a tracking block that runs on the XCD of the stream block with the same
// index (see places_of) finds the logits that block wrote in its L2.  Beyond the part's share: a number no
// cache reaches.
__device__ __forceinline__ int track_entry(int n_sub, int part, int n_parts, int r) {
  const int j = r * (kBlock / 16) + (static_cast<int>(threadIdx.x) >> 4);   // wave j % kWaves, its sub-tile j / kWaves
  const WaveMap m = fused_wave_map(n_sub, n_parts, part, j % kWaves);
  const int it = j / kWaves;
  return it < m.cnt ? (m.first + it * m.step) * 16 + (static_cast<int>(threadIdx.x) & 15) : 0x7FFFFFF0;
}
// Rounds of kBlock entries that cover the largest part.
__device__ __forceinline__ int track_rounds(int n_sub, int n_parts) {
  return (kWaves * fused_wave_run(n_sub, n_parts) + kBlock / 16 - 1) / (kBlock / 16);
}

__device__ __forceinline__ void track_load(const TrackArgs &k, int unit, int part, int n_parts, int r0,
                                           TrackBatch &b) {
  const float *lg = k.logits + static_cast<size_t>(unit) * k.p_stride * kHeadPad;
  const int n1 = k.n_old + 1;
  const int n_sub = (n1 + 15) >> 4;
#pragma unroll
  for (int r = 0; r < kTrackRows; ++r) {
    const int i = track_entry(n_sub, part, n_parts, r0 + r);
    b.sa[r] = b.sb[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < n1) {
      b.sa[r] = *reinterpret_cast<const float4 *>(lg + static_cast<size_t>(i) * kHeadPad);
      b.sb[r] = *reinterpret_cast<const float4 *>(lg + static_cast<size_t>(i) * kHeadPad + 4);
    }
  }
}

// The activation test and the TS / MRI update of entry i (Alg. 1, Eq. 1); true if active.
// log_mask (LDS, or null): the call is logged; an active entry then only sets its bit there.
// kWeights: the caller may have asked for the weights or brought some (never with candidate records).
template <bool kPrecise, bool kWeights>
__device__ __forceinline__ bool track_one(const TrackArgs &k, int unit, int i, const float (&s)[kHeadPad],
                                          const float (&m)[kHeadPad], const float (&invl)[kHeadPad],
                                          unsigned *log_mask) {
  const int seq = unit / k.n_kv_heads, kvh = unit % k.n_kv_heads;
  const int G = k.group;
  const size_t head0 = static_cast<size_t>(seq) * k.n_q_heads + static_cast<size_t>(kvh) * G;
  int32_t *ts = k.ts + static_cast<size_t>(unit) * k.capacity;
  int32_t *mri = k.mri + static_cast<size_t>(unit) * k.capacity;
  bool act = false;
#pragma unroll
  for (int h = 0; h < kHeadPad; ++h) {
    if (h < G) {
      float p = weight_of<kPrecise>(s[h], m[h], invl[h]);
      const size_t at = (head0 + h) * k.capacity + i;
      if (kWeights && k.p_out) k.p_out[at] = p;
      if (kWeights && k.p_override) p = k.p_override[at];
      act = act || (p >= k.alpha);
    }
  }
  if (i == k.n_old) {                              // the appended entry starts here (Sec. 4)
    if (!log_mask) {                               // (of a logged call: when the log is applied)
      ts[i] = k.t;
      mri[i] = 0;
      k.pos[static_cast<size_t>(unit) * k.capacity + i] = k.prompt_len + k.t - 1;
    }
  } else if (act) {                                // few entries are active: TS / MRI are read only here
    if (log_mask) {
      atomicOr(log_mask + (i >> 5), 1u << (i & 31));
    } else {
      const int32_t gap = k.t - ts[i];
      if (gap > mri[i]) mri[i] = gap;              // Eq. 1
      ts[i] = k.t;                                 // Alg. 1
    }
  }
  return act;
}

template <bool kPrecise>
__device__ __forceinline__ unsigned track_apply(const TrackArgs &k, int unit, int part, int n_parts,
                                                int r0, const TrackBatch &b, const float (&m)[kHeadPad],
                                                const float (&invl)[kHeadPad], unsigned *log_mask) {
  const int n1 = k.n_old + 1, n_sub = (n1 + 15) >> 4;
  unsigned n_act = 0;
#pragma unroll
  for (int r = 0; r < kTrackRows; ++r) {
    const int i = track_entry(n_sub, part, n_parts, r0 + r);
    if (i >= n1) continue;
    const float s[kHeadPad] = {b.sa[r].x, b.sa[r].y, b.sa[r].z, b.sa[r].w,
                               b.sb[r].x, b.sb[r].y, b.sb[r].z, b.sb[r].w};
    n_act += track_one<kPrecise, true>(k, unit, i, s, m, invl, log_mask) ? 1u : 0u;
  }
  return n_act;
}

// Tracking from the candidate records of the call's blocks b = part, part + step, ...
template <bool kPrecise>
__device__ __forceinline__ unsigned track_records(const TrackArgs &k, int unit, int part, int step,
                                                  const float (&m)[kHeadPad], const float (&invl)[kHeadPad],
                                                  unsigned *log_mask) {
  const int cap = fused_part_cap(k.n_old, k.n_parts);
  unsigned n_act = 0;
  for (int b = part; b < k.n_parts; b += step) {
    const size_t at = static_cast<size_t>(unit) * k.p_stride + static_cast<size_t>(b) * cap;
    const float *region = k.logits + at * kHeadPad;
    const int n = region_count(region, cap);
    auto track = [&](int r, auto eight) {          // (groups of eight have the index beside the records)
      const float4 sa = *reinterpret_cast<const float4 *>(region + static_cast<size_t>(1 + r) * kHeadPad);
      const float4 sb = *reinterpret_cast<const float4 *>(region + static_cast<size_t>(1 + r) * kHeadPad + 4);
      const int i = record_entry(decltype(eight)::value ? k.cand_index[at + 1 + r] : __float_as_int(sb.w), k.n_old);
      const float s[kHeadPad] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, decltype(eight)::value ? sb.w : 0.f};
      n_act += track_one<kPrecise, false>(k, unit, i, s, m, invl, log_mask) ? 1u : 0u;
    };
    if (k.group == kHeadPad)
      for (int r = threadIdx.x; r < n; r += kBlock) track(r, std::true_type{});
    else
      for (int r = threadIdx.x; r < n; r += kBlock) track(r, std::false_type{});
  }
  return n_act;
}

// With per-sequence timing: the call's arguments as they hold for one unit (its own cache length,
// local step and prompt length).  False: the unit's sequence takes no part in that call.
__device__ __forceinline__ bool track_for_unit(const TrackArgs &k, int unit, TrackArgs &ku) {
  ku = k;
  if (!k.slots.prompt_len) return true;
  const int seq = unit / k.n_kv_heads;
  const int32_t P = k.slots.prompt_len[seq], tau = k.t - k.slots.t0[seq];
  if (P < 0 || tau < 1) return false;
  ku.n_old = slot_n_old(P, tau, k.slots.budget, k.slots.window);
  ku.t = tau;
  ku.prompt_len = P;
  return true;
}

__device__ __forceinline__ void track_stats(const TrackArgs &k, int unit, float (&m)[kHeadPad],
                                            float (&invl)[kHeadPad]) {
  const float *st = k.stat + static_cast<size_t>(unit) * (2 * kHeadPad);
#pragma unroll
  for (int h = 0; h < kHeadPad; ++h) { m[h] = st[2 * h]; invl[h] = st[2 * h + 1]; }
}

// Adds up the block's activation count; every (unit, part) owns one counter slot.
__device__ void track_count(const TrackArgs &k, int unit, int part, unsigned n_act, unsigned *cnt_lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) n_act += __shfl_xor(n_act, o);
  if (lane == 0) cnt_lds[wave] = n_act;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned total = 0;
    for (int w = 0; w < kWaves; ++w) total += cnt_lds[w];
    if (total) k.activation_counter[unit * 64 + part] += total;
  }
}

// Tracking alone (lazyev_stats, evictions with per-sequence timing or of more entries than the selection holds, or a caller
// that wants the weights at once).
template <bool kPrecise>
__global__ __launch_bounds__(kBlock) void track_kernel(const TrackArgs k_all, int n_parts) {
  __shared__ unsigned cnt_lds[kWaves];
  const int unit = blockIdx.x / n_parts, part = blockIdx.x % n_parts;
  TrackArgs k;
  if (!track_for_unit(k_all, unit, k)) return;
  float m[kHeadPad], invl[kHeadPad];
  track_stats(k, unit, m, invl);
  unsigned n_act = 0;
  if (k.compact) {
    n_act = track_records<kPrecise>(k, unit, part, n_parts, m, invl, nullptr);
  } else {
    const int rounds = track_rounds((k.n_old + 1 + 15) >> 4, n_parts);
    for (int r0 = 0; r0 < rounds; r0 += kTrackRows) {
      TrackBatch b;
      track_load(k, unit, part, n_parts, r0, b);
      n_act += track_apply<kPrecise>(k, unit, part, n_parts, r0, b, m, invl, nullptr);
    }
  }
  track_count(k, unit, part, n_act, cnt_lds);
}

// The logged calls of a layer applied to TS / MRI.  An entry's bit in the words of a call says that it
// was active there (TrackArgs::bitlog).  Block b works on the kFlushSpan entries from kFlushSpan * (b % spans)
// on of unit (b / spans) % units of layer b / spans / units, spans = blocks per unit; a wave on 128
// of them: lane (half, j) brings the words 2 half and 2 half + 1 of call s + j, and after a transposition across the 32
// lanes holds the 32 calls of entries 64 half + j and 64 half + 32 + j.  A logged
// call's step is the one before it plus one, so the largest gap between activations is a run of zeros and no call is
// looked at by itself.  (Walking the set bits, the steps from LDS, took as long as the wave's most active
// entry: 256 units of 1152 entries x 127 calls, in two launches as the layers differed by a call, 72 us, now 8.)
constexpr int kFlushWords = 2;                     // per lane and call
constexpr int kFlushSpan = kWaves * 64 * kFlushWords;
__global__ __launch_bounds__(kBlock) void track_flush_kernel(const FlushArgs f) {
  const int spans = (f.capacity + kFlushSpan - 1) / kFlushSpan;
  const int span = blockIdx.x % spans, lu = blockIdx.x / spans;
  const int layer = lu / f.units, unit = lu % f.units;
  const FlushArgs::Layer of = f.layer[layer];
  if (of.n_calls == 0) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, j = lane & 31;
  const size_t slab = (static_cast<size_t>(layer) * f.units + unit) * f.capacity;
  const uint32_t *log = f.bitlog + (static_cast<size_t>(layer) * f.units + unit) * f.log_slots * f.log_words;   // (a unit's slots lie together)
  const int word = span * (kFlushSpan / 32) + (wave * 2 + half) * kFlushWords;
  constexpr int kBatch = 4;                        // sets of 32 calls requested together
  unsigned w[kBatch][kFlushWords];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const uint32_t *row = log + static_cast<size_t>(min(s0 + 32 * b + j, of.n_calls - 1)) * f.log_words;
#pragma unroll
      for (int x = 0; x < kFlushWords; ++x) w[b][x] = row[min(word + x, f.log_words - 1)];
    }
  };
  fetch(0);
  int32_t ts[kFlushWords], mri[kFlushWords];
  bool touched[kFlushWords];
#pragma unroll
  for (int x = 0; x < kFlushWords; ++x) {          // (requested while the words travel)
    const int i = (word + x) * 32 + j;
    ts[x] = mri[x] = 0;
    if (i < f.capacity) { ts[x] = f.ts[slab + i]; mri[x] = f.mri[slab + i]; }
  }
#pragma unroll
  for (int x = 0; x < kFlushWords; ++x) {
    // An entry that one of the calls appended starts there (Sec. 4): no earlier call has a bit for it
    const int i = (word + x) * 32 + j, s_new = i - of.n_old;
    touched[x] = i < f.capacity && s_new >= 0 && s_new < of.n_calls;
    if (touched[x]) {
      ts[x] = of.t + s_new;
      mri[x] = 0;
      f.pos[slab + i] = f.prompt_len + ts[x] - 1;
    }
  }
  for (int s0 = 0; s0 < of.n_calls; s0 += 32 * kBatch) {
    if (s0 > 0) fetch(s0);
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int s = s0 + 32 * b;
      if (s >= of.n_calls) break;                  // (uniform)
#pragma unroll
      for (int x = 0; x < kFlushWords; ++x) {
        const unsigned calls = transpose_bits<32>(s + j < of.n_calls ? w[b][x] : 0u, j);
        apply_calls(calls, of.t + s, ts[x], mri[x]);
        touched[x] = touched[x] || calls != 0;
      }
    }
  }
#pragma unroll
  for (int x = 0; x < kFlushWords; ++x) {
    const int i = (word + x) * 32 + j;
    if (touched[x] && i < f.capacity) { f.ts[slab + i] = ts[x]; f.mri[slab + i] = mri[x]; }
  }
}

// ------------------------------------------------------------- merging the partials of a unit
// A merged partial: maximum, sum and this thread's four output values of n partials, in block order, each scaled to the
// largest of the maxima: that is found first, so that the exponentials do not wait for one another and every
// partial takes one.  Every product and sum is written out with its rounding (no contraction left to the
// compiler), so that all kernel instances produce the same bits from the same partials.
template <bool kPrecise>
struct Merge {
  float m, l;
  float o[4];
  // (a block without entries has the lowest maximum, sum = 0, values = 0)
  __device__ __forceinline__ void start(float m_all, float mj, float lj, const f32x4_t &oj) {
#pragma clang fp contract(off)
    m = m_all;
    const float f = exp_of<kPrecise>(mj - m);
    l = lj * f;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = oj[i] * f;
  }
  __device__ __forceinline__ void add(float mj, float lj, const f32x4_t &oj) {
#pragma clang fp contract(off)
    const float f = exp_of<kPrecise>(mj - m);
    l = fmaf(lj, f, l);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = fmaf(oj[i], f, o[i]);
  }
};

// The merged row of a unit: thread t writes output elements 4t .. 4t+3 (all of head h) and, as
// the owner of a head's first elements, the head's softmax statistics for the tracking.
template <typename T, int D, typename Args>
__device__ __forceinline__ void write_unit_row(const Args &a, int unit, int G, const Merge<Rows<T, D>::kPrecise> &mg, int e0, int h) {
  if (e0 >= G * D) return;
  const float invl = 1.0f / mg.l;
  T *out = a.out + static_cast<size_t>(unit) * G * D + e0;   // (a unit's query heads follow one another, unit after unit)
  if constexpr (Rows<T, D>::kF32) {
    *reinterpret_cast<f32x4_t *>(out) = f32x4_t{mg.o[0] * invl, mg.o[1] * invl, mg.o[2] * invl, mg.o[3] * invl};
  } else {
  u32x2_t w;
  w[0] = pair_to_bf16(mg.o[0] * invl, mg.o[1] * invl);
  w[1] = pair_to_bf16(mg.o[2] * invl, mg.o[3] * invl);
  *reinterpret_cast<u32x2_t *>(out) = w;
  }
  if (e0 % D == 0) {
    float *st = a.stat_out + static_cast<size_t>(unit) * (2 * kHeadPad) + 2 * h;
    st[0] = mg.m;
    st[1] = invl;
  }
}

// ------------------------------------------------------------------- hand-over of partials
// A block hands its partial over to a block of a higher index as a record of 64-bit words, each = 16 bits of the
// launch's number, 16 bits of the maximum or the sum, 32 bits of an output value, written and read with 64-bit
// device-scope atomics.  A word that shows this launch's number holds this launch's values, whatever else is still on
// its way, so the writer neither waits for its stores nor signals, and the reader needs no second round trip after a
// flag: it reads the words it needs until all of them carry the number.  Blocks are started in index order and a
// block waits for blocks of lower indices only, so every wait ends; it is bounded all the same (spin_ticks of the 100
// MHz counter), after which the block raises the workspace's fault word and goes on.
// The number is an argument, so a captured call has the same one in every replay and would find the records of the
// replay before complete: a call that is being captured has its records cleared by a launch before it, and all
// captured calls have kSeqCaptured for their number, which no eager call has: an eager one would find what a replay
// left complete as soon as the numbers had started over (see lazyev_decode_step).
// One hop for any number of blocks: up to kPairMax, the unit's last block merges what the others hand over; of more, all
// hand over and blocks behind the stream blocks merge (merge_columns), or the last block merges nine at a time
// (merging_blocks).  (Before, the last of every eight blocks merged
// those and handed over in turn: the second hop took 1.5 us, and seven records are 28 loads for every thread of the one
// block that merges.  us per call, 8 units x 2080 entries 6.65 (8 blocks) -> 5.4 (32), 4 x 3000 7.8 (8) -> 5.5 (32), 16 x
// 4000 10.8 (8) -> 8.7 (16), 2 units of 128 x bf16 x 12000 9.7 (64) -> 8.3 (64), 8 x 2080 of 128 x fp32 15.0 (8) -> 8.8
// (32), with 7 query heads 14.9 -> 9.1; 220 random shapes of 1 .. 60 units x 130 .. 24000 entries 0.93 of the time.)
// Record of a block: for each of the four waves four rows of 64 words; row i holds the output element 4 t + i of
// thread t (one store instruction of a wave writes 512 contiguous bytes), and the 16 bits beside it are a half of the
// maximum (rows 0 and 1) or the sum of thread t's head (each thread its own copy: what the reader needs of a head
// then never waits for another wave's store).  What a merge costs is the instructions of single waves: with a word of
// its own, half of it the number, for each of the six values, a merge of seven records was 42 loads and 42
// comparisons, now 28 loads, 14 exclusive ors and 7 comparisons, and with one exponential per record instead of two
// that wait for those before (see Merge) 8 units x 2081 entries take 2074 us for 256 calls instead of 2218, 32 x 1040
// 241 for 32 instead of 256.
constexpr int kRecWords = 4 * kBlock;
// thread t's first word, as a byte offset
__device__ __forceinline__ unsigned rec_at(int t) { return (static_cast<unsigned>(t >> 6) * (4 * 64) + (t & 63)) * 8u; }
constexpr int kPairMax = 8;             // blocks of a unit whose last one finishes it
constexpr uint32_t kSeqMax = 0xFFFE, kSeqCaptured = 0xFFFF;

__device__ __forceinline__ void rec_word_store(unsigned long long *p, float v, unsigned top) {
  __hip_atomic_store(p, (static_cast<unsigned long long>(top) << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void rec_store(unsigned long long *rec, int t_own, const f32x4_t &o, float m, float l, unsigned seq) {
  const unsigned mu = __float_as_uint(m), lu = __float_as_uint(l), number = seq << 16;
  const unsigned top[4] = {number | (mu >> 16), number | (mu & 0xFFFFu), number | (lu >> 16), number | (lu & 0xFFFFu)};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    rec_word_store(reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(rec) + rec_at(t_own)) + i * 64, o[i], top[i]);
}
// What one thread reads of another block's record: its four output elements, its head's max and sum.
struct RecPart { unsigned long long w[4]; };
// (rec, the same for the whole wave, is kept a scalar: with the four addresses of every record in vector registers
// seven records spill)
__device__ __forceinline__ void rec_load(RecPart &r, const unsigned long long *rec, unsigned at) {
  auto base = (const __attribute__((address_space(1))) char *)rec;
  __asm__ volatile("" : "+s"(base));
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r.w[i] = __hip_atomic_load((const __attribute__((address_space(1))) unsigned long long *)(base + at) + i * 64, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned rec_top(const RecPart &r, int i) { return static_cast<unsigned>(r.w[i] >> 32); }
// the upper halves of words i and i + 1 (upper) or the lower ones
__device__ __forceinline__ unsigned rec_halves(const RecPart &r, int i, bool upper) {
  return __builtin_amdgcn_perm(rec_top(r, i), rec_top(r, i + 1), upper ? 0x07060302u : 0x05040100u);
}
__device__ __forceinline__ bool rec_valid(const RecPart &r, unsigned seq) {
  const unsigned twice = seq | (seq << 16);
  return ((rec_halves(r, 0, true) ^ twice) | (rec_halves(r, 2, true) ^ twice)) == 0;
}
__device__ __forceinline__ float rec_max(const RecPart &r) { return __uint_as_float(rec_halves(r, 0, false)); }
__device__ __forceinline__ float rec_sum(const RecPart &r) { return __uint_as_float(rec_halves(r, 2, false)); }
__device__ __forceinline__ f32x4_t rec_values(const RecPart &r) {
  auto value = [&](int i) { return __uint_as_float(static_cast<unsigned>(r.w[i])); };
  return f32x4_t{value(0), value(1), value(2), value(3)};
}

// What one thread needs of n <= N records, one behind the other, all requested together, again
// until every word carries the launch's number; then the records and (m, l, o) merged in this order.
template <int N, bool kPrecise, typename Args>
__device__ __forceinline__ Merge<kPrecise> merge_records(const Args &a, const unsigned long long *rec, int n,
                                               int t_own, float m, float l, const f32x4_t &o) {
  Merge<kPrecise> mg;
  if (n == 0) {                                    // uniform
    mg.m = m; mg.l = l;
#pragma unroll
    for (int i = 0; i < 4; ++i) mg.o[i] = o[i];
    return mg;
  }
  RecPart r[N];
  const unsigned at = rec_at(t_own);
  unsigned long long t_first = 0;
  for (;;) {
#pragma unroll
    for (int j = 0; j < N; ++j)                    // (beyond n: the last record once more, no branches among the loads)
      rec_load(r[j], rec + min(j, n - 1) * kRecWords, at);
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) ok = ok & rec_valid(r[j], a.seq);
    if (__builtin_amdgcn_ballot_w64(!ok) == 0) break;   // (the wave goes on together)
    const unsigned long long now = wall_clock64();
    if (t_first == 0) t_first = now;
    if (now - t_first >= a.spin_ticks) {           // (a limit of 0: no second look)
      atomicOr(a.fault, 1);                        // (cannot happen otherwise, see above; the row is then wrong)
      break;
    }
  }
  float m_all = m;
#pragma unroll
  for (int j = 0; j < N; ++j) m_all = fmaxf(m_all, rec_max(r[j]));
  mg.start(m_all, rec_max(r[0]), rec_sum(r[0]), rec_values(r[0]));
#pragma unroll
  for (int j = 1; j < N; ++j)
    if (j < n) mg.add(rec_max(r[j]), rec_sum(r[j]), rec_values(r[j]));
  mg.add(m, l, o);
  return mg;
}

// The first n_records records of every unit (block b: unit b) as before any launch.
__global__ __launch_bounds__(kBlock) void clear_records_kernel(unsigned long long *rec, int rec_per_unit, int n_records) {
  unsigned long long *mine = rec + static_cast<size_t>(blockIdx.x) * rec_per_unit * kRecWords;
  for (int i = threadIdx.x; i < n_records * kRecWords; i += kBlock) mine[i] = 0;
}

// ------------------------------------------------------------------------------- the kernel
// The kernel's arguments as they lie in memory.  The argument block `a` is read through args_from_here only: left to
// itself the compiler fetches words of it at the top of the kernel for whichever path needs them, and a stream wave,
// whose first loads need none of them, waited there for such a fetch (its registers were used again), 0.5 us in every
// call; the queries took another round trip behind it.  us per pass, before and now (queries from the leading
// arguments, the block read behind the first loads): 64 units x 1563 entries of 64 x bf16 1283 -> 1188, 8 units x
// 2081 2385 -> 2218, 128 x 2081 3128 -> 3066.
template <typename T>
struct Kernarg {
  const T *k_cache, *v_cache, *k_new, *v_new, *q;
  int n_old, capacity;
  unsigned shape;
  DecodeArgs a;
};
typedef const __attribute__((address_space(4))) DecodeArgs *const_args_t;
template <typename T>
__device__ __forceinline__ const DecodeArgs &args_from_here() {
  // (that the compiler lays the kernel's own arguments out like this struct: tests/test_kernel_resources.py)
  static_assert(offsetof(Kernarg<T>, a) == 56, "five pointers, two lengths and the shape, then the block, aligned to 8 bytes");
  uintptr_t p = reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()) + offsetof(Kernarg<T>, a);
  __asm__ volatile("" : "+s"(p));                  // (nothing of it is read before this place)
  return *(const DecodeArgs *)reinterpret_cast<const_args_t>(p);
}
// What a wave needs of the argument block: read in one go while its first loads travel and kept (a word that
// is read where it is used, behind the stream, is a round trip on the way of the whole launch).
template <typename T>
struct CallArgs {
  float scale, alpha;
  int p_stride, rec_per_unit;
  uint32_t seq, spin_ticks;
  float *logits_out, *stat_out;
  int32_t *cand_index_out, *fault;
  T *out;
  unsigned long long *part_rec;
  __device__ __forceinline__ void read() {
    const DecodeArgs &a = args_from_here<T>();
    scale = a.scale; alpha = a.alpha;
    p_stride = a.p_stride; rec_per_unit = a.rec_per_unit;
    seq = a.seq; spin_ticks = a.spin_ticks;
    logits_out = a.logits_out; stat_out = a.stat_out;
    cand_index_out = a.cand_index_out; fault = a.ws.fault;
    out = static_cast<T *>(a.out);
    part_rec = a.ws.part_rec;
    __asm__ volatile("" : "+s"(scale), "+s"(alpha), "+s"(p_stride), "+s"(rec_per_unit), "+s"(seq), "+s"(spin_ticks));
    keep(logits_out); keep(stat_out); keep(cand_index_out); keep(fault); keep(out); keep(part_rec);
  }
  template <typename P>
  static __device__ __forceinline__ void keep(P *&p) {   // (known as an address of global memory: flat stores would have every load wait for all)
    auto g = (__attribute__((address_space(1))) P *)p;
    __asm__ volatile("" : "+s"(g));
    p = (P *)g;
  }
};
// Units, blocks per unit, query heads per unit, whether sequences have their own timing, whether there are merging blocks and whether
// they come last, in one scalar argument
// (what a wave is handed in registers at its start is limited to a few words).
static_assert(kFusedSplitMax < 128, "seven bits");
inline unsigned pack_shape(int units, int n_split, int group, bool slots, bool merged, bool merge_last) {
  return static_cast<unsigned>(units) | (static_cast<unsigned>(n_split) << 16) | (static_cast<unsigned>(group - 1) << 23) |
         (slots ? 1u << 26 : 0u) | (merged ? 1u << 27 : 0u) | (merge_last ? 1u << 28 : 0u);
}
__device__ __forceinline__ int shape_units(unsigned s) { return static_cast<int>(s & 0xFFFFu); }
__device__ __forceinline__ int shape_split(unsigned s) { return static_cast<int>((s >> 16) & 127u); }
__device__ __forceinline__ int shape_group(unsigned s) { return static_cast<int>((s >> 23) & 7u) + 1; }
__device__ __forceinline__ bool shape_slots(unsigned s) { return (s >> 26) & 1u; }
__device__ __forceinline__ bool shape_merged(unsigned s) { return (s >> 27) & 1u; }
__device__ __forceinline__ bool shape_merge_last(unsigned s) { return (s >> 28) & 1u; }
// Does the sequence of a unit take this step?  (per-sequence timing)
__device__ __forceinline__ bool takes_part(const DecodeArgs &a, int unit) {
  const int seq = unit / a.n_kv_heads;
  return a.slots.prompt_len[seq] >= 0 && a.t - a.slots.t0[seq] >= 1;
}
// Waves of a block that merge, each 32 output elements, and blocks of them per unit.  What a wave reads, 256 bytes of every
// record, passes through its compute unit's L1 at 64 bytes a cycle: with eight waves a block 32 records a unit took 0.2 us
// more (8 units x 2080: 5.67 / 5.50), 16 records 0.3.
__host__ __device__ constexpr int merge_waves(int n_split) { return n_split <= 16 ? 4 : 2; }
__host__ __device__ constexpr int merge_blocks(int head_dim, int group, int waves) { return (group * (head_dim / 32) + waves - 1) / waves; }
// Where a launch's blocks that do not stream begin: the merging blocks, if there are any, and the tracking blocks.  Blocks go to
// the eight XCDs round robin, and a tracking block reads the logits that the stream block of its number has just written
// (see track_entry): the tracking blocks of a launch with merging blocks begin at a multiple of eight, up to seven blocks
// before them do nothing.  us per call, right behind the merging blocks / like this: 5 units x 19000 entries of 128 x
// bf16 14.4 / 12.6, 25 x 4000 14.6 / 12.9, 19 x 8200 18.5 / 16.3; 9 x 24000 of 64 x bf16 18.0 / 14.8; 10 x 13000 of 64 x fp32 18.5 / 15.8;
// 15 x 13000 of 128 x fp32 41.9 / 37.3.
// merge_last (see merges_last): the tracking blocks, as many as stream blocks, come before the merging blocks.
struct Places { int merge, track; };
__host__ __device__ inline Places places_of(int n_stream, int n_merge, bool merge_last) {
  if (n_merge == 0) return {n_stream, n_stream};
  const int track = (n_stream + (merge_last ? 0 : n_merge) + 7) & ~7;
  return {merge_last ? track + n_stream : n_stream, track};
}
// The output elements 32 columns .. + 31 of a unit of n blocks (kPairMax < n <= 8 N), merged by one wave: lane (c, g)
// reads the elements 4 c .. 4 c + 3 of the records g, g + 8, ..., and the eight lanes of a column merge across the wave,
// with no LDS and no barrier.  What bounds it is the chain partial stored - seen - loaded - stored, 1.4 us from the last
// block's end to the launch's.  First one word of every record is looked at, until half of them are there: blocks of
// equal work end close together, and a look at all words of 32 records is 16 loads that hold up the ones that will find them
// (from the first record on: 8 units x 2080 5.96 / 5.92, 4 x 3000 6.46 / 6.03; only when all are there 6.5 / 6.7).
// Before that the wave sleeps for what a run of sub-tiles takes at least, 0.5 us each (128-byte rows 0.25) from the third on, and
// looks at one word of one record where the run is long: the looks go to memory, where they are in the stream's way (16 units x
// 24000 39.6 -> 38.8 with the sleep; 15 x 24000 of 128 x fp32 72.6 -> 71.8, 20 x 24000 of 128 x bf16 49.4 -> 49.1 with the single word; shorter runs
// lose by it, 9 x 13000 of 64 x bf16 10.1 / 10.4).
// It waits for blocks of lower indices only, like any reader of records, but for as long as a whole run takes: the limit of
// the single word and that of the looks until half of the records are there are 64 times the one for the others.
template <typename T, int D, int N, typename Args>
__device__ __forceinline__ void merge_columns(const Args &a, int unit, int G, int n, int run, int columns) {
  constexpr bool kPrecise = Rows<T, D>::kPrecise;
  const int lane = static_cast<int>(threadIdx.x) & 63, c = lane & 7, g = lane >> 3;
  const int t_own = columns * 8 + c;
  const unsigned long long *recs = a.part_rec + static_cast<size_t>(unit) * a.rec_per_unit * kRecWords;
  const unsigned long long t_start = wall_clock64();
  const unsigned quiet = run > 2 ? static_cast<unsigned>(run - 2) * (Rows<T, D>::kBytes >= 256 ? 50 : 25) : 0u;
  while (wall_clock64() - t_start < quiet) __builtin_amdgcn_s_sleep(4);
  unsigned long long t_first = 0;
  {
    auto base = (const __attribute__((address_space(1))) char *)recs;
    __asm__ volatile("" : "+s"(base));
    // (long runs: a single word until the record of the unit's first block is there)
    while (run > kRunMax) {
      unsigned long long w = 0;
      if (lane == 0)
        w = __hip_atomic_load((const __attribute__((address_space(1))) unsigned long long *)(base + rec_at(columns * 8)), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_ballot_w64(static_cast<unsigned>(w >> 48) == a.seq) != 0) break;
      const unsigned long long now = wall_clock64();
      if (t_first == 0) t_first = now;
      if (now - t_first >= 64ull * a.spin_ticks) break;
      __builtin_amdgcn_s_sleep(16);
    }
    t_first = 0;
    const unsigned at = static_cast<unsigned>(min(lane, n - 1)) * (kRecWords * 8) + rec_at(columns * 8);
    for (;;) {
      const unsigned long long w = __hip_atomic_load((const __attribute__((address_space(1))) unsigned long long *)(base + at),
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__popcll(__builtin_amdgcn_ballot_w64(lane < n && static_cast<unsigned>(w >> 48) == a.seq)) >= n - n / 2) break;
      const unsigned long long now = wall_clock64();
      if (t_first == 0) t_first = now;
      if (now - t_first >= 64ull * a.spin_ticks) break;
      __builtin_amdgcn_s_sleep(1);
    }
  }
  STAMP(2);
  t_first = 0;
  RecPart r[N];
  for (;;) {
#pragma unroll
    for (int j = 0; j < N; ++j)
      rec_load(r[j], recs, rec_at(t_own) + static_cast<unsigned>(min(8 * j + g, n - 1)) * (kRecWords * 8));
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) ok = ok & rec_valid(r[j], a.seq);
    if (__builtin_amdgcn_ballot_w64(!ok) == 0) break;
    const unsigned long long now = wall_clock64();
    if (t_first == 0) t_first = now;
    if (now - t_first >= a.spin_ticks) {
      atomicOr(a.fault, 1);
      break;
    }
  }
  STAMP(3);
  Merge<kPrecise> mg;
  float m = rec_max(r[0]);
#pragma unroll
  for (int j = 1; j < N; ++j) m = fmaxf(m, rec_max(r[j]));
  mg.m = max_over_eight(m);
  float l = 0.f;
  f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < N; ++j) {
#pragma clang fp contract(off)
    const bool mine = 8 * j + g < n;
    const float f = exp_of<kPrecise>(rec_max(r[j]) - mg.m);
    const f32x4_t x = rec_values(r[j]);
    l = fmaf(mine ? rec_sum(r[j]) : 0.f, f, l);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = fmaf(mine ? x[i] : 0.f, f, o[i]);
  }
  mg.l = sum_over_eight(l);
#pragma unroll
  for (int i = 0; i < 4; ++i) mg.o[i] = sum_over_eight(o[i]);
  if (g == 0) write_unit_row<T, D>(a, unit, G, mg, 4 * t_own, 4 * t_own / D);
}
// kCompact: this call leaves candidate lists instead of every logit.
// The leading scalar arguments repeat what a stream wave needs to request its queries and first sub-tile
// (the same values are in `a`): scalar kernel arguments are handed to a wave in registers at its
// start (kernel-argument preload, see build.py), a struct has to be fetched from memory first.
// kLong (with kCompact): a wave's run is longer than the kRunMax sub-tiles whose logits it keeps
// in LDS; every kRunMax sub-tiles it then writes the candidates among them, found with the cut
// that the block's four waves' running statistics give at that moment (a lower bound of the
// final denominator at any time, so the cut only errs towards more candidates).
// kListWaves (with kCompact): blocks of 2 * kWaves waves.  The second four ("list waves") sleep at
// the block barrier while the first four stream, and then build the candidate lists from the
// logits in LDS while the first four merge, exchange and finish the unit; that phase is serial
// code of one wave per SIMD, so a second wave per SIMD takes the lists off its path.  Used when
// all blocks of the launch are resident at once with eight waves each (a stream block and a
// tracking block per compute unit: these instances keep to 128 registers per lane); a launch of
// more blocks, and fp32 rows of 128 elements (up to 230 registers), run four-wave blocks whose
// stream waves build their own lists.
// Launches with merging blocks have none either: their lists are built while the records travel (with list waves 20 units
// x 10500 of 64 x bf16 18.6 us, 13.7 without).
// kSplit > 0: the instance is for units of exactly kSplit blocks (1 .. 8, with list waves).  What
// precedes and follows the stream is serial code of single waves, and a split known at compile time takes the
// loads of a variable number of records and the divisions by the split out of it
// (us per call with an instance of its own / with the one for any split: 32 units x 600 entries, 3 blocks 6.4
// / 7.7, 4 6.3 / 7.2, 6 6.5 / 7.0).
template <typename T, int D, bool kCompact, bool kLong = false, bool kListWaves = false, int kSplit = 0>
__global__ __launch_bounds__(kListWaves ? 2 * kBlock : kBlock, (Rows<T, D>::kWide ? 2 : 4)) void decode_fused_kernel(
    const T *k_cache, const T *v_cache, const T *k_new_all, const T *v_new_all, const T *q_all, const int n_old_call, const int capacity,
    const unsigned shape, const DecodeArgs) {
  using R = Rows<T, D>;
  using SubTile = typename R::SubTile;
  constexpr bool kPrecise = R::kPrecise;
  const int units_call = shape_units(shape), G = shape_group(shape);
  const bool slots_on = shape_slots(shape);
  const int n_split = kSplit > 0 ? kSplit : shape_split(shape);   // (a constant where the instance fixes it)
  __shared__ float m_lds[kWaves][16], lsum_lds[kWaves][16];
  // one 16-row K sub-tile per wave while streaming; afterwards the wave's output accumulator
  __shared__ u32x4_t stage_lds[kWaves][16 * 16];
  __shared__ u32x4_t new_lds[kWaves][2 * Rows<T, D>::kLanes];   // the appended rows of K and V, a copy per wave
  extern __shared__ float logit_lds[];             // [kWaves][min(run, kRunMax)][16 entries][8 heads]
  __shared__ unsigned cnt_lds[kWaves];
  __shared__ unsigned cand_total;                  // candidate records of this block so far
  __shared__ float run_lse[kWaves][kHeadPad];      // kLong: each wave's latest log-sum-exp per head (one word: no torn reads)

  STAMP(0);
#ifdef LAZYEV_TIMELINE
  STAMPV(6, xcc_id());
#endif
  const int n_stream = n_split * units_call;
  const bool merged = kSplit == 0 && shape_merged(shape);   // a unit's partials are merged by blocks of their own
  const int per_merge = merge_waves(n_split);
  const Places places = places_of(n_stream, merged ? merge_blocks(D, G, per_merge) * units_call : 0, shape_merge_last(shape));
  if (static_cast<int>(blockIdx.x) >= places.track && static_cast<int>(blockIdx.x) < places.track + n_stream) {
    // tracking of the previous call: n_split blocks per unit, spread over the compute units
    // like the stream blocks
    if (kListWaves && threadIdx.x >= kBlock) return;  // (the tracking has no use for list waves)
    const DecodeArgs &a = args_from_here<T>();
    const int tb = blockIdx.x - places.track;
    const int n_track = a.n_track;
    const BlockPlace at = block_place<kSplit>(tb, n_track, units_call);
    const int unit = at.unit, part = at.split;
    TrackArgs k;
    if (!track_for_unit(a.track, unit, k)) return;
    float m[kHeadPad], invl[kHeadPad];
    track_stats(k, unit, m, invl);
    unsigned n_act = 0;
    // a logged call: the active entries' bits are collected in LDS (the K staging area, which
    // a tracking block has no other use for) ...
    unsigned *log_mask = nullptr;
    if (k.bitlog) {
      log_mask = reinterpret_cast<unsigned *>(&stage_lds[0][0]);
      for (int j = threadIdx.x; j < k.log_words; j += kBlock) log_mask[j] = 0;
      __syncthreads();
    }
    if (k.compact) {
      n_act = track_records<kPrecise>(k, unit, part, n_track, m, invl, log_mask);
    } else {
      const int rounds = track_rounds((k.n_old + 1 + 15) >> 4, n_track);
      for (int r0 = 0; r0 < rounds; r0 += kTrackRows) {
        TrackBatch b;
        track_load(k, unit, part, n_track, r0, b);
        n_act += track_apply<kPrecise>(k, unit, part, n_track, r0, b, m, invl, log_mask);
      }
    }
    if (k.bitlog) {
      // ... and every word of the unit is written by the one block whose entries it covers: word
      // j holds sub-tiles 2j and 2j + 1, which the wave map gives to one block (an even wave and
      // the next one); with candidate records that is a block of the logged call's own split,
      // whose records this tracking block reads if the block's index is its own modulo n_track
      __syncthreads();
      const int parts = k.compact ? k.n_parts : n_track;
      uint32_t *dst = k.bitlog + static_cast<size_t>(unit) * k.log_unit_stride;
      for (int j = threadIdx.x; j < k.log_words; j += kBlock) {
        const int wv = (2 * j) % (kWaves * parts);
        const int owner = (parts - 1 - wv / kWaves) % n_track;
        if (owner == part) dst[j] = log_mask[j];
      }
    }
    track_count(k, unit, part, n_act, cnt_lds);
    STAMPV(7, 4 | (static_cast<unsigned long long>(a.seq) << 8));
    STAMP(5);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform: scalar branches below
  if (merged && static_cast<int>(blockIdx.x) >= n_stream) {
    if (static_cast<int>(blockIdx.x) < places.merge) return;
    const BlockPlace at = block_place<0>(blockIdx.x - places.merge, 2, units_call);
    const int columns = at.split * per_merge + wave;
    if (wave >= per_merge || columns >= G * (D / 32)) return;   // (a block between the merging and the tracking blocks among them)
    if (slots_on && !takes_part(args_from_here<T>(), at.unit)) return;
    CallArgs<T> a;
    a.read();
    const int run = fused_wave_run((n_old_call + 16) >> 4, n_split);
    if (n_split <= 16) merge_columns<T, D, 2>(a, at.unit, G, n_split, run, columns);
    else if (n_split <= 32) merge_columns<T, D, 4>(a, at.unit, G, n_split, run, columns);
    else merge_columns<T, D, 8>(a, at.unit, G, n_split, run, columns);
    STAMPV(7, 3 | (static_cast<unsigned long long>(a.seq) << 8));
    STAMP(5);
    return;
  }
  if (kCompact && tid == 0) cand_total = 0;        // (the block barrier after the stream orders it)
  if constexpr (kLong) {                           // (here the waves add to it while they stream)
    if (tid < kWaves * kHeadPad) run_lse[tid / kHeadPad][tid % kHeadPad] = -INFINITY;   // nothing seen yet
    __syncthreads();
  }
  const int c = lane & 15, g = lane >> 4;
  const BlockPlace place = block_place<kSplit>(blockIdx.x, n_split, units_call);
  const int unit = place.unit, split = place.split;
  int n_old = n_old_call, n1 = n_old + 1, n_sub = (n1 + 15) >> 4;
  // Per-sequence timing: this unit's own length, at the end of two round trips.  False: the whole unit sits this call out.
  auto own_length = [&]() -> bool {
    typedef const __attribute__((address_space(4))) int32_t *scalar_t;   // (written by earlier launches only)
    const DecodeArgs &a = args_from_here<T>();
    const int seq_s = unit / a.n_kv_heads;
    const int32_t P = ((scalar_t)a.slots.prompt_len)[seq_s], tau = a.t - ((scalar_t)a.slots.t0)[seq_s];
    n_old = slot_n_old(P, tau, a.slots.budget, a.slots.window);
    n1 = n_old + 1;
    n_sub = (n1 + 15) >> 4;
    return P >= 0 && tau >= 1;
  };

  // Two ways to a sub-tile's rows.  kFlat: they lie one after the other in the cache, so a scalar address and one
  // 32-bit offset per lane and load reach them, rows beyond the cache taken as its last one; the row to be appended
  // is not there yet, and is put in place (K in the staging area, V by patch_v) when the unit's last sub-tile, which
  // alone has it, is worked on.  Otherwise every load chooses the source of its row, 64 of the 230 vector
  // instructions of a sub-tile.  Where the bytes set the time those cost nothing, and the replacement at the end of
  // the run does: us per pass, chosen / flat, 128 units x 2081 3009 / 3029, x 4129 of 80 (2 blocks a unit) 5766 /
  // 5816; with three blocks a unit or more, and for rows of 128 bytes, the latency of a sub-tile does: 8 units x 2081
  // 1999 / 1950, 48 units x 1000 1273 / 1254, 64 units x 1563 of 64 x bf16 1160 / 1090.  (fp32 rows: the products are
  // longer than either, 840 / 842.  The instances for any split with long runs or all logits have no registers left for it.)
  constexpr bool kFlat = !R::kF32 && ((kSplit == 0 && kCompact && !kLong) || kSplit >= 3 || R::kBytes == 128);
  // ... Such a wave's first sub-tile does not depend on the unit's length but for the clamp of its rows, so with
  // per-sequence timing the length is worked out while that travels (its rows clamped to the unit's capacity): 48
  // units x 1000, a pass of continuous_batch's shapes, 1240 -> 1225 us.
  if (slots_on && !(kFlat && wave < kWaves))
    if (!own_length()) return;

  CallArgs<T> a;                                   // (read where a wave has nothing better to do)
  // the appended row goes to slot N (the stream waves read it from k_new / v_new, nobody from the slot)
  auto append_row = [&]() {
    const T *kn = k_new_all + static_cast<size_t>(unit) * D, *vn = v_new_all + static_cast<size_t>(unit) * D;
    T *ku = const_cast<T *>(k_cache) + static_cast<size_t>(unit) * capacity * D;
    T *vu = const_cast<T *>(v_cache) + static_cast<size_t>(unit) * capacity * D;
    if (lane < R::kLanes)
      reinterpret_cast<uint4 *>(ku + static_cast<size_t>(n_old) * D)[lane] = reinterpret_cast<const uint4 *>(kn)[lane];
    else if (lane < 2 * R::kLanes)
      reinterpret_cast<uint4 *>(vu + static_cast<size_t>(n_old) * D)[lane - R::kLanes] = reinterpret_cast<const uint4 *>(vn)[lane - R::kLanes];
  };

  // ---- candidate list of the sub-tiles that stream wave w leaves in LDS (for a long run: the last
  // segment; the earlier ones went out while the wave streamed), i.e. the entries that can reach
  // alpha in some head.  p_h = exp(s_h - m_h) / l_h <= exp(s_h - mb_h) / lb_h with the block's
  // own (mb, lb), so p_h >= alpha needs s_h >= mb_h + log(alpha lb_h); 2 % slack covers the
  // rounding of the two sides.  In two steps: what does not depend on the logits (plan), and
  // the rest, after the block barrier that ends the stream (run).  Four sub-tiles per round, one
  // entry per lane.
  constexpr int kRounds = (kRunMax + 3) / 4;
  struct ScanPlan {
    const float *src[kRounds];
    int entry[kRounds];
    bool always[kRounds], may[kRounds];
    char *region;
    int32_t *index;                                // of the region's slots (groups of eight)
    int group;
    float alpha98;
  };
  auto plan_scan = [&](ScanPlan &sp, int w) {
    const WaveMap wmap = fused_wave_map(n_sub, n_split, split, w);
    const int cnt_w = wmap.cnt;
    const int s0 = (kLong && cnt_w > 0) ? (cnt_w - 1) / kRunMax * kRunMax : 0;
    const int run_w = min(fused_wave_run(n_sub, n_split), kRunMax);
    const float *logits = logit_lds + static_cast<size_t>(w) * run_w * (16 * kHeadPad);
    sp.group = G;
    sp.alpha98 = 0.98f * a.alpha;
    sp.region = reinterpret_cast<char *>(a.logits_out + (static_cast<size_t>(unit) * a.p_stride +
                                                         static_cast<size_t>(split) * fused_part_cap(n_old, n_split)) * kHeadPad);
    sp.index = a.cand_index_out + static_cast<size_t>(unit) * a.p_stride + static_cast<size_t>(split) * fused_part_cap(n_old, n_split);
    const int e_in = lane & 15;
#pragma unroll
    for (int rd = 0; rd < kRounds; ++rd) {
      // (reads of a round beyond the run are clamped to its last sub-tile and not used)
      const int it = s0 + 4 * rd + (lane >> 4);
      const int itc = max(min(it, cnt_w - 1), s0);
      sp.src[rd] = logits + (itc - s0) * (16 * kHeadPad) + e_in * kHeadPad;
      sp.entry[rd] = (wmap.first + it * wmap.step) * 16 + e_in;
      sp.may[rd] = it < cnt_w && sp.entry[rd] < n1;
      sp.always[rd] = it < cnt_w && sp.entry[rd] == n_old;   // the appended entry starts its tracking there
    }
  };
  auto run_scan = [&](ScanPlan &sp) {
    // lane h < 8 works out the cut of head h, everybody reads the eight cuts
    const int hh = lane & 7;
    float mbh = m_lds[0][hh];
#pragma unroll
    for (int w2 = 1; w2 < kWaves; ++w2) mbh = fmaxf(mbh, m_lds[w2][hh]);
    float lbh = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < kWaves; ++w2) {
      lbh = fmaf(__expf(m_lds[w2][hh] - mbh), lsum_lds[w2][hh], lbh);
    }
    // the logits of all rounds are read first ...
    f32x4_t sa[kRounds], sb[kRounds];
#pragma unroll
    for (int rd = 0; rd < kRounds; ++rd) {
      sa[rd] = *reinterpret_cast<const f32x4_t *>(sp.src[rd]);
      sb[rd] = *reinterpret_cast<const f32x4_t *>(sp.src[rd] + 4);
    }
    const float cut_h = (hh < sp.group && lbh > 0.f) ? mbh + __logf(sp.alpha98 * lbh) : INFINITY;
    float cut[kHeadPad];
#pragma unroll
    for (int h = 0; h < kHeadPad; ++h)
      cut[h] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cut_h), h));
    unsigned long long mask[kRounds];
    unsigned n_rec = 0;
#pragma unroll
    for (int rd = 0; rd < kRounds; ++rd) {
      // s_h >= cut_h in some head  <=>  the largest s_h - cut_h is not negative
      const float d = fmaxf(fmaxf(fmaxf(sa[rd][0] - cut[0], sa[rd][1] - cut[1]), fmaxf(sa[rd][2] - cut[2], sa[rd][3] - cut[3])),
                            fmaxf(fmaxf(sb[rd][0] - cut[4], sb[rd][1] - cut[5]), fmaxf(sb[rd][2] - cut[6], sb[rd][3] - cut[7])));
      const bool cand = ((d >= 0.f) & sp.may[rd]) | sp.always[rd];
      if (sp.group < kHeadPad) sb[rd][3] = __int_as_float(sp.entry[rd]);   // (the 8th place is free)
      mask[rd] = __builtin_amdgcn_ballot_w64(cand);
      n_rec += static_cast<unsigned>(__popcll(mask[rd]));
    }
    // ... then ONE addition to the block's record count reserves the places of all of the wave's records
    if (n_rec != 0) {                              // wave-uniform
      unsigned base = 0;
      if (lane == 0) base = atomicAdd(&cand_total, n_rec);
      base = __builtin_amdgcn_readfirstlane(base) + 1;
#pragma unroll
      for (int rd = 0; rd < kRounds; ++rd) {
        if ((mask[rd] >> lane) & 1ull) {
          const unsigned at = base + __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask[rd] >> 32),
                                                              __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask[rd]), 0u));
          char *dst = sp.region + at * static_cast<unsigned>(kHeadPad * sizeof(float));   // (a 32-bit offset: under 4 GB)
          *reinterpret_cast<f32x4_t *>(dst) = sa[rd];
          *reinterpret_cast<f32x4_t *>(dst + 16) = sb[rd];
          if (sp.group == kHeadPad) sp.index[at] = sp.entry[rd];
        }
        base += static_cast<unsigned>(__popcll(mask[rd]));
      }
    }
  };

  if (kListWaves && wave >= kWaves) {
    // ---- list wave kWaves + w: appends the new row (one of them), plans, sleeps at the barrier
    // that ends the stream, builds stream wave w's list
    const int w = wave - kWaves;
    a.read();
    if (split == 0 && w == 1) append_row();
    ScanPlan sp;
    plan_scan(sp, w);
    __syncthreads();                               // the stream has ended, the waves' statistics are in LDS
    run_scan(sp);
    __syncthreads();                               // cand_total is complete
    return;
  }

  // this wave's sub-tiles (fused_wave_map)
  WaveMap wm = fused_wave_map(n_sub, n_split, split, wave);
  int cnt = wm.cnt;                                // (0 for a wave beyond a short cache)
  int row_last = kFlat && slots_on ? capacity - 1 : n_old;   // kFlat: rows beyond are read as this one
  auto sub_of = [&](int it) { return wm.first + it * wm.step; };

  const T *kc = k_cache + static_cast<size_t>(unit) * capacity * D;
  const T *vc = v_cache + static_cast<size_t>(unit) * capacity * D;
  const T *k_new = k_new_all + static_cast<size_t>(unit) * D;
  const T *v_new = v_new_all + static_cast<size_t>(unit) * D;

  auto load_k = [&](SubTile &t, int it) {
    if constexpr (!kFlat) {
      const int sub = sub_of(it);
      if constexpr (R::kF32) {
        // fp32: straight into the MFMA operand layout, lane (c, g): row c, columns 16 j + 4 g .. + 3
        const int row = min(sub * 16 + c, n_old);
        const T *src = ((row == n_old) ? k_new : kc + static_cast<size_t>(row) * D) + 4 * g;
#pragma unroll
        for (int j = 0; j < R::kK; ++j) t.k[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + 16 * j));
      } else {
        // bf16: whole rows, kLanes lanes per row; re-laid out through LDS
#pragma unroll
        for (int j = 0; j < R::kK; ++j) {
          const int row = min(sub * 16 + j * (64 / R::kLanes) + lane / R::kLanes, n_old);
          const T *src = (row == n_old) ? k_new : kc + static_cast<size_t>(row) * D;
          t.k[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + (lane % R::kLanes) * 8));
        }
      }
      return;
    }
    const int sub = min(sub_of(it), row_last >> 4), left = row_last - sub * 16;
    const char *rows = reinterpret_cast<const char *>(kc) + static_cast<size_t>(sub) * (16 * R::kBytes);
    const unsigned last = static_cast<unsigned>(min(left, 16) * R::kBytes + (lane % R::kLanes) * 16);
#pragma unroll
    for (int j = 0; j < R::kK; ++j)
      t.k[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(rows + min(static_cast<unsigned>(lane * 16 + j * 1024), last)));
  };
  auto load_v = [&](SubTile &t, int it) {
    if constexpr (!kFlat) {
      const int sub = sub_of(it);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = min(sub * 16 + 4 * g + i, n_old);
        const T *src = (row == n_old) ? v_new : vc + static_cast<size_t>(row) * D;
        if constexpr (R::kF32) {                     // columns 64 h + 4 c .. + 3
#pragma unroll
          for (int h = 0; h < D / 64; ++h)
            t.v[i * (D / 64) + h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + 64 * h + c * 4));
        } else if constexpr (D == 128) {             // columns 8 c .. + 7
          t.v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + c * 8));
        } else {                                     // columns 4 c .. + 3
          const u32x2_t x = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t *>(src + c * 4));
          t.v[i / 2][2 * (i % 2)] = x[0];
          t.v[i / 2][2 * (i % 2) + 1] = x[1];
        }
      }
      return;
    }
    const int sub = min(sub_of(it), row_last >> 4), left = row_last - sub * 16;
    const char *rows = reinterpret_cast<const char *>(vc) + static_cast<size_t>(sub) * (16 * R::kBytes);
    const unsigned last = static_cast<unsigned>(min(left, 16) * R::kBytes + c * (D / 8));
#pragma unroll
    for (int i = 0; i < 4; ++i) {                  // rows 4 g .. 4 g + 3; columns 8 c .. + 7 or 4 c .. + 3
      const unsigned at = min(static_cast<unsigned>((4 * g + i) * R::kBytes + c * (D / 8)), last);
      if constexpr (D == 128) {
        t.v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(rows + at));
      } else {
        const u32x2_t x = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t *>(rows + at));
        t.v[i / 2][2 * (i % 2)] = x[0];
        t.v[i / 2][2 * (i % 2) + 1] = x[1];
      }
    }
  };
  // kFlat, the unit's last sub-tile: the lanes whose row is the appended one, or beyond it, get V from where the wave
  // has kept it in LDS since its start (K: see compute).  kPrecise: rows beyond count as zero: zero times an infinite
  // element is NaN.
  auto patch_v = [&](SubTile &t, int left) {
    const char *row = reinterpret_cast<const char *>(new_lds[wave]) + R::kBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool here = 4 * g + i >= left, beyond = kPrecise && 4 * g + i > left;
      if constexpr (D == 128) {
        const u32x4_t x = *reinterpret_cast<const u32x4_t *>(row + c * 16);
        t.v[i] = here ? x : t.v[i];
      } else {
        u32x2_t x = *reinterpret_cast<const u32x2_t *>(row + c * 8);
        x = beyond ? u32x2_t{0, 0} : x;
        t.v[i / 2][2 * (i % 2)] = here ? x[0] : t.v[i / 2][2 * (i % 2)];
        t.v[i / 2][2 * (i % 2) + 1] = here ? x[1] : t.v[i / 2][2 * (i % 2) + 1];
      }
    }
  };
  // ---- the stream starts here: the queries and the first sub-tile are requested with what the wave was handed
  // in registers, before anything is read from the argument block in memory
  // B operand of the logits: Q^T, head c (zero rows beyond the group); piece kk goes with K's piece kk
  const int hc = min(c, G - 1);
  const T *q_row = q_all + (static_cast<size_t>(unit) * G + hc) * D + g * (16 / sizeof(T));
  u32x4_t qb[R::kK];
#pragma unroll
  for (int kk = 0; kk < R::kK; ++kk) qb[kk] = *reinterpret_cast<const u32x4_t *>(q_row + kk * (64 / sizeof(T)));
  u32x4_t new_piece = {0, 0, 0, 0};
  if (kFlat) new_piece = reinterpret_cast<const u32x4_t *>(lane & R::kLanes ? v_new : k_new)[lane % R::kLanes];
  SubTile buf[R::kDepth];
#pragma unroll
  for (int x = 0; x < R::kDepth; ++x) {            // (unconditionally, for exact load counts: beyond a short cache, copies of its end)
    load_k(buf[x], x);
    load_v(buf[x], x);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (kFlat && slots_on) {
    if (!own_length()) return;
    wm = fused_wave_map(n_sub, n_split, split, wave);
    cnt = wm.cnt;
    row_last = n_old;
  }
  a.read();
  if constexpr (kFlat) {
    new_lds[wave][lane % (2 * R::kLanes)] = new_piece;   // (where fewer lanes cover it, several write the same)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  const int run = min(fused_wave_run(n_sub, n_split), kRunMax);
  float *my_logits = logit_lds + static_cast<size_t>(wave) * run * (16 * kHeadPad);
  int seg0 = 0;                                    // first of this wave's sub-tiles whose logits are still in LDS
  float *logits_out = a.logits_out + static_cast<size_t>(unit) * a.p_stride * kHeadPad;

  // (no reference yet: the lowest number, below which no logit but -inf lies and from which that has the weight 0)
  float m_ref = -FLT_MAX, lsum = 0.f;
  f32x4_t o[R::kAcc];
#pragma unroll
  for (int e = 0; e < R::kAcc; ++e) o[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int kk = 0; kk < R::kK; ++kk) qb[kk] = c < G ? qb[kk] : u32x4_t{0, 0, 0, 0};

  // kMore (a std::bool_constant): the wave has a sub-tile kDepth after this one and requests it here.
  // kAgain: the wave goes over its run once more because an accumulator became NaN (see below)
  auto compute = [&](SubTile &t, int it, auto more_tag, auto again_tag) {
    constexpr bool kMore = decltype(more_tag)::value, kAgain = decltype(again_tag)::value;
    const int sub = sub_of(it);
    const bool last_sub = !kMore && sub == n_sub - 1;   // (wave-uniform)
    const int left = n_old - sub * 16;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (R::kF32) {
      // Four terms per instruction; which four of the row's columns go together does not matter as
      // long as K and Q agree.  Sums of four, then a tree: one chain over the row has the
      // logit of a strongly matching key (about 45 at 128 columns) off by enough to move its weight by 1e-5.
      f32x4_t sum[R::kK / 2];
#pragma unroll
      for (int y = 0; y < R::kK / 2; ++y) {
        f32x4_t x[8];
#pragma unroll
        for (int z = 0; z < 8; ++z)
          x[z] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(t.k[2 * y + z / 4][z % 4]), __uint_as_float(qb[2 * y + z / 4][z % 4]),
                                                      f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        sum[y] = ((x[0] + x[4]) + (x[1] + x[5])) + ((x[2] + x[6]) + (x[3] + x[7]));
      }
      acc = sum[0] + sum[1];
      if constexpr (R::kK == 8) acc += sum[2] + sum[3];
      if constexpr (kMore) load_k(t, it + R::kDepth);
    } else {
    // K rows -> MFMA A layout (lane (c, g): row c, chunks 4kk+g).  Chunk x of row r sits at
    // slot x ^ r of the row, so both the row-wise writes and the column-wise reads touch
    // every LDS bank once (rows of 8 chunks: at most twice).  The staging area is private to the wave: LDS operations of one
    // wave execute in order, the fences only stop the compiler from reordering them.
    u32x4_t ka[R::kK];
    {
      u32x4_t *stage = stage_lds[wave];
      int here = lane;
      if constexpr (kLong && !kMore) __asm__ volatile("" : "+v"(here));   // (addresses of its own: see segment_candidates)
      const int ch = here % R::kLanes, r0 = here / R::kLanes, c = here & 15, g = here >> 4;
#pragma unroll
      for (int j = 0; j < R::kK; ++j) {
        const int r = j * (64 / R::kLanes) + r0;
        stage[r * R::kLanes + (ch ^ (r % R::kLanes))] = t.k[j];
      }
      if (kFlat && last_sub && lane < R::kLanes) stage[left * R::kLanes + (lane ^ (left % R::kLanes))] = new_lds[wave][lane];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // the K registers are free again: the next sub-tile's K rows travel during the arithmetic
      if constexpr (kMore) {
        load_k(t, it + R::kDepth);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kk = 0; kk < R::kK; ++kk) ka[kk] = stage[c * R::kLanes + ((4 * kk + g) ^ (c % R::kLanes))];
    }
    if constexpr (kPrecise) {                      // (two sums of 32 terms, then their sum)
      const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[0]), __builtin_bit_cast(bf16x8_t, qb[0]), zero, 0, 0, 0) +
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[1]), __builtin_bit_cast(bf16x8_t, qb[1]), zero, 0, 0, 0);
    } else {
#pragma unroll
      for (int kk = 0; kk < R::kK; ++kk)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[kk]),
                                                      __builtin_bit_cast(bf16x8_t, qb[kk]), acc, 0, 0, 0);
    }
    }
    float s[4];
    const int e0 = sub * 16 + 4 * g;
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = kMore || e0 + i < n1 ? acc[i] * a.scale : -INFINITY;   // (a wave's earlier sub-tiles are full)
    // logits of the sub-tile -> [entry][head] in LDS; written out when the wave's run ends (a
    // store among the loads would hold up the in-order load counter)
    if (!kAgain && c < kHeadPad) {
      float *dst = my_logits + (it - seg0) * (16 * kHeadPad);
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[(4 * g + i) * kHeadPad + c] = s[i];
    }
    float tmax = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    tmax = max_over_lane_groups(tmax);
    if (__builtin_amdgcn_ballot_w64(tmax > m_ref + kRaise) != 0) {   // wave-uniform, rare
      const float m_new = fmaxf(m_ref, tmax);
      const float f = exp_of<kPrecise>(m_ref - m_new);   // 0 on the first sub-tile
      lsum *= f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float fh = __shfl(f, 4 * g + i);     // factor of head 4g+i (lane 4g+i owns it)
#pragma unroll
        for (int e = 0; e < R::kAcc; ++e) o[e][i] *= fh;
      }
      m_ref = m_new;
    }
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = exp_of<kPrecise>(s[i] - m_ref);
    lsum += (p[0] + p[1]) + (p[2] + p[3]);
    if (kFlat && last_sub) patch_v(t, left);
    if constexpr (kPrecise && !kFlat && !kMore) {
      // The unit's last sub-tile: rows beyond the cache are copies of the appended one with a weight of zero, and
      // zero times an infinite element is NaN
      if (sub == n_sub - 1) {                      // wave-uniform
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (e0 + i < n1) continue;
          if constexpr (R::kF32) {
#pragma unroll
            for (int h = 0; h < D / 64; ++h) t.v[i * (D / 64) + h] = u32x4_t{0, 0, 0, 0};
          } else {
            t.v[i / 2][2 * (i % 2)] = t.v[i / 2][2 * (i % 2) + 1] = 0;
          }
        }
      }
    }
    if constexpr (R::kF32) {
      // lane (c, g) holds the weights of head c for the entries 4g .. 4g+3: the A operand of the
      // product over entries 4g' + i, g' = 0..3, is p[i].  The sub-tile's 16 terms are summed on their
      // own and then added: the running sum takes one rounding per sub-tile instead of 16.
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f32x4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            x = __builtin_amdgcn_mfma_f32_16x16x4f32(p[i], __uint_as_float(t.v[i * (D / 64) + h][e]), x, 0, 0, 0);
          o[4 * h + e] += x;
        }
    } else {
    // weights as bf16 operands: rounded once, or (kPrecise) as three bf16 terms that add up to the fp32
    // value exactly (8 bits of the significand each)
    constexpr int kTerms = kPrecise ? 3 : 1;
    s16x4_t pa[kTerms];
#pragma unroll
    for (int x = 0; x < kTerms; ++x) {
      u32x2_t pw;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        pw[i] = pair_to_bf16(p[2 * i], p[2 * i + 1]);
        if (kPrecise) {
          p[2 * i] -= __uint_as_float(pw[i] << 16);
          p[2 * i + 1] -= __uint_as_float(pw[i] & 0xFFFF0000u);
        }
      }
      pa[x] = __builtin_bit_cast(s16x4_t, pw);
    }
#pragma unroll
    for (int e = 0; e < R::kAcc; ++e) {
      const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
      auto v_word = [&](int i) {                   // columns (8 c or 4 c) + 2 (e / 2), + 1 of row 4 g + i
        if constexpr (D == 128) return t.v[i][e >> 1];
        else return t.v[i / 2][2 * (i % 2) + (e >> 1)];
      };
      u32x2_t vb;
      vb[0] = __builtin_amdgcn_perm(v_word(1), v_word(0), sel);
      vb[1] = __builtin_amdgcn_perm(v_word(3), v_word(2), sel);
#pragma unroll
      for (int x = 0; x < kTerms; ++x) {
        o[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa[x], __builtin_bit_cast(s16x4_t, vb), o[e], 0, 0, 0);
        if (kAgain && x == 0) { vb[0] = finite_bf16(vb[0]); vb[1] = finite_bf16(vb[1]); }
      }
    }
    }
    if constexpr (kMore) load_v(t, it + R::kDepth);
  };

  // this wave's logits -> workspace, 512 bytes per sub-tile: when the run ends, and for a
  // long run every kRunMax sub-tiles
  auto flush = [&](int it0, int it1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int it = it0 + (lane >> 5); it < it1; it += 2)
      *reinterpret_cast<float4 *>(logits_out + static_cast<size_t>(sub_of(it)) * (16 * kHeadPad) + (lane & 31) * 4) =
          *reinterpret_cast<const float4 *>(my_logits + (it - it0) * (16 * kHeadPad) + (lane & 31) * 4);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // candidates among this wave's sub-tiles it_a .. it_b - 1 (their logits are in LDS from slot 0
  // on) under the cuts of the eight heads -> records in the block's region
  auto emit_candidates = [&](int it_a, int it_b, int lane, const float (&cut)[kHeadPad]) {
    float *region = a.logits_out + (static_cast<size_t>(unit) * a.p_stride +
                                    static_cast<size_t>(split) * fused_part_cap(n_old, n_split)) * kHeadPad;
    const int e_in = lane & 15;
    for (int it0 = it_a; it0 < it_b; it0 += 4) {   // four sub-tiles per round, one entry per lane
      const int it = it0 + (lane >> 4);
      bool cand = false;
      int entry = 0;
      f32x4_t sa = {0.f, 0.f, 0.f, 0.f}, sb = sa;
      if (it < it_b) {
        const float *src = my_logits + (it - it_a) * (16 * kHeadPad) + e_in * kHeadPad;
        sa = *reinterpret_cast<const f32x4_t *>(src);
        sb = *reinterpret_cast<const f32x4_t *>(src + 4);
        entry = sub_of(it) * 16 + e_in;
        cand = sa[0] >= cut[0] || sa[1] >= cut[1] || sa[2] >= cut[2] || sa[3] >= cut[3] ||
               sb[0] >= cut[4] || sb[1] >= cut[5] || sb[2] >= cut[6] || sb[3] >= cut[7];
        cand = (cand && entry < n1) || entry == n_old;
      }
      const unsigned long long mask = __builtin_amdgcn_ballot_w64(cand);
      if (mask != 0) {                             // wave-uniform
        unsigned base = 0;
        if (lane == 0) base = atomicAdd(&cand_total, static_cast<unsigned>(__popcll(mask)));
        base = __builtin_amdgcn_readfirstlane(base);
        if (cand) {
          const unsigned at = 1 + base + __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u));
          if (G < kHeadPad) sb[3] = __int_as_float(entry);
          else a.cand_index_out[static_cast<size_t>(unit) * a.p_stride + static_cast<size_t>(split) * fused_part_cap(n_old, n_split) + at] = entry;
          *reinterpret_cast<f32x4_t *>(region + static_cast<size_t>(at) * kHeadPad) = sa;
          *reinterpret_cast<f32x4_t *>(region + static_cast<size_t>(at) * kHeadPad + 4) = sb;
        }
      }
    }
  };
  // kLong: the segment it_a .. it_b - 1 is complete.  The wave publishes the log-sum-exp of
  // every head over what it has seen and takes the cut from what the four waves have published
  // so far: the sums only grow, so p <= exp(s - lse) holds with the log-sum-exp of any subset of
  // the entries at any earlier time.
  auto segment_candidates = [&](int it_a, int it_b) {
    // (the lane's number is worked out again, hidden from the compiler, which would otherwise keep addresses that
    // depend on it in registers through the stream and spill one: 64 units x 6200 entries 41.3 us a call, 40.7 without
    // scratch; 24 units x 16400 44.2 / 43.6)
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    __asm__ volatile("" : "+v"(lane));
    const int c = lane & 15, g = lane >> 4;
    float ls = lsum;
    ls = sum_over_lane_groups(ls);
    if (g == 0 && c < kHeadPad) run_lse[wave][c] = ls > 0.f ? m_ref + __logf(ls) : -INFINITY;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int hh = lane & 7;
    float lw[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) lw[w] = run_lse[w][hh];
    float lmax = lw[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) lmax = fmaxf(lmax, lw[w]);
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
      if (lw[w] != -INFINITY) sum += __expf(lw[w] - lmax);
    const float cut_h = (hh < G && sum > 0.f) ? lmax + __logf(0.98f * a.alpha * sum) : INFINITY;
    float cut[kHeadPad];
#pragma unroll
    for (int h = 0; h < kHeadPad; ++h)
      cut[h] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cut_h), h));
    emit_candidates(it_a, it_b, lane, cut);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the LDS slots are written again next
    __builtin_amdgcn_wave_barrier();
  };
  // logits of a long run leave LDS every kRunMax sub-tiles
  auto segment_end = [&](int it) {
    if constexpr (kCompact && !kLong) return;      // (its runs are no longer than that)
    if (it + 1 - seg0 == kRunMax && it + 1 < cnt) {
      if constexpr (kLong) segment_candidates(seg0, it + 1);
      else flush(seg0, it + 1);
      seg0 = it + 1;
    }
  };
  // (the wave's last sub-tiles stand outside the loop, so that the loop requests the ones to come
  // unconditionally: no branch between the loads, exact load counts for the waits)
  if constexpr (R::kDepth == 1) {
    for (int it = 0; it + 1 < cnt; ++it) {
      compute(buf[0], it, std::true_type{}, std::false_type{});
#ifdef LAZYEV_TIMELINE
      if (it == 0) STAMP(1);
#endif
      segment_end(it);
    }
    if (cnt > 0) compute(buf[0], cnt - 1, std::false_type{}, std::false_type{});
  } else {
    int it = 0;
    for (; it + 3 < cnt; it += 2) {
      compute(buf[0], it, std::true_type{}, std::false_type{});
      segment_end(it);
      compute(buf[1], it + 1, std::true_type{}, std::false_type{});
      segment_end(it + 1);
    }
    if (it + 2 < cnt) {
      compute(buf[0], it, std::true_type{}, std::false_type{});
      segment_end(it);
      compute(buf[1], it + 1, std::false_type{}, std::false_type{});
      segment_end(it + 1);
      compute(buf[0], it + 2, std::false_type{}, std::false_type{});
    } else {
      if (it < cnt) { compute(buf[0], it, std::false_type{}, std::false_type{}); segment_end(it); }
      if (it + 1 < cnt) compute(buf[1], it + 1, std::false_type{}, std::false_type{});
    }
  }
  if constexpr (kPrecise && !R::kF32) {
    // The second and third bf16 terms of a weight may be negative or zero, so an infinite element of V, which
    // the weight itself would leave infinite, becomes NaN.  Such a wave goes over its run once more, these products
    // left out of it (one look at the accumulators per run; a look at the V words would be on the way of every sub-tile).
    float any = 0.f;
#pragma unroll
    for (int e = 0; e < R::kAcc; ++e) any += (o[e][0] + o[e][1]) + (o[e][2] + o[e][3]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(any != any) != 0, 0)) {   // wave-uniform
      m_ref = -FLT_MAX;
      lsum = 0.f;
#pragma unroll
      for (int e = 0; e < R::kAcc; ++e) o[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      for (int it = 0; it < cnt; ++it) {
        load_k(buf[0], it);
        load_v(buf[0], it);
        compute(buf[0], it, std::false_type{}, std::true_type{});
      }
    }
  }
  STAMP(2);
  if (!kCompact) flush(seg0, cnt);
  // ---- the four waves of the block -> one partial
  lsum = sum_over_lane_groups(lsum);
  if (g == 0) { m_lds[wave][c] = m_ref; lsum_lds[wave][c] = lsum; }
  constexpr int kAccStride = 16 * 16 * 4;         // (floats of stage_lds[wave])
  static_assert(8 * D <= kAccStride, "a wave's accumulators fit its staging area");
  float *acc_lds = reinterpret_cast<float *>(&stage_lds[0][0]);   // a wave's own 4 KB: others may still be streaming
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int head = 4 * g + i;
    if (head < G) {
      // accumulators 4 x .. 4 x + 3 hold the columns 8 c + 4 x .. (128-element bf16 rows) or 64 x + 4 c ..
      float *row = acc_lds + wave * kAccStride + head * D;
#pragma unroll
      for (int x = 0; x < R::kAcc / 4; ++x)
        *reinterpret_cast<float4 *>(row + (!R::kF32 && D == 128 ? 8 * c + 4 * x : 64 * x + 4 * c)) =
            make_float4(o[4 * x][i], o[4 * x + 1][i], o[4 * x + 2][i], o[4 * x + 3][i]);
    }
  }
  __syncthreads();
  STAMP(3);
  // ---- this block's partial: thread owns output elements 4 tid .. 4 tid + 3, all of one head
  // (threads beyond the group's rows work on a valid place and store nothing)
  const int e0 = 4 * tid;
  const int ec = min(e0, G * D - 4);
  const int h_own = ec / D;
  float mb_own = m_lds[0][h_own];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mb_own = fmaxf(mb_own, m_lds[w][h_own]);
  float l_own = 0.f;
  f32x4_t v_own = {0.f, 0.f, 0.f, 0.f};
  // (no branches from here on where a select does: this phase is a single wave per SIMD running
  // serial code, every instruction counts)
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float f = exp_of<kPrecise>(m_lds[w][h_own] - mb_own);   // (a wave without entries: sum and values 0)
    const f32x4_t x = *reinterpret_cast<const f32x4_t *>(acc_lds + w * kAccStride + ec);
#pragma unroll
    for (int i = 0; i < 4; ++i) v_own[i] = fmaf(f, x[i], v_own[i]);
    l_own = fmaf(f, lsum_lds[w][h_own], l_own);
  }
  const bool finisher = !merged && split == n_split - 1;      // the unit's last block
  const int t_own = ec >> 2;                       // (threads beyond the group's rows read a valid place)
  unsigned long long *recs = a.part_rec + static_cast<size_t>(unit) * a.rec_per_unit * kRecWords;
  if (!finisher && e0 < G * D) rec_store(recs + static_cast<size_t>(split) * kRecWords, tid, v_own, mb_own, l_own, a.seq);
  // what only the NEXT launch needs, while the partial travels: the appended row and this wave's
  // candidate list (list waves, where the block has them, do both meanwhile)
  if constexpr (!kListWaves) {
    if (split == 0 && wave == 1) append_row();
    if constexpr (kCompact) {
      ScanPlan sp;
      plan_scan(sp, wave);
      run_scan(sp);
    }
  }
  if (finisher) {
    constexpr int kIn = kSplit > 1 ? kSplit - 1 : kSplit == 1 ? 1 : R::kWide ? 18 : 9;
    const int n_in = kSplit > 0 ? kSplit - 1 : n_split - 1;
    Merge<kPrecise> mg = merge_records<kIn, kPrecise>(a, recs, min(n_in, kIn), t_own, mb_own, l_own, v_own);
    if constexpr (kSplit == 0) {                   // (at most 18 records where the split is the library's own)
      for (int j = kIn; j < n_in; j += kIn)
        mg = merge_records<kIn, kPrecise>(a, recs + static_cast<size_t>(j) * kRecWords, min(n_in - j, kIn), t_own, mg.m, mg.l,
                                          f32x4_t{mg.o[0], mg.o[1], mg.o[2], mg.o[3]});
    }
    STAMP(4);
    write_unit_row<T, D>(a, unit, G, mg, e0, h_own);
  }
  if (kCompact) {
    __syncthreads();                               // cand_total is complete
    if (tid == 0)
      *reinterpret_cast<int32_t *>(a.logits_out + (static_cast<size_t>(unit) * a.p_stride +
                                                   static_cast<size_t>(split) * fused_part_cap(n_old, n_split)) * kHeadPad) =
          static_cast<int32_t>(cand_total);
  }
  STAMPV(7, (finisher ? 2 : 1) | (static_cast<unsigned long long>(a.seq) << 8));
  STAMP(5);
}

// ------------------------------------------------------------------------------- host side
// Compute units of the current device (asked once; 256, the whole chip's, without one).
int compute_units() {
  static const int n = [] {
    int dev = 0, v = 0;
    return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0 ? v : 256;
  }();
  return n;
}

// Four-wave blocks that the chip holds at once in a launch whose waves run over `run` sub-tiles: by their LDS, which is
// handed out in pieces of 1280 bytes of 160 KB, and by their registers.
int fused_slots(int run, bool f32, int head_dim) {
  const int stationary = 17056 + (f32 ? 0 : head_dim == 64 ? 1024 : 2048);   // (what is not logit_lds)
  const int lds = kWaves * (run < kRunMax ? run : kRunMax) * 16 * kHeadPad * static_cast<int>(sizeof(float)) + stationary;
  const int by_lds = 160 * 1024 / ((lds + 1279) / 1280 * 1280), by_registers = f32 && head_dim == 128 ? 2 : 4;
  return compute_units() * (by_lds < by_registers ? by_lds : by_registers);
}

// Merging blocks of a launch: for units of more than kPairMax blocks, where they fit the chip beside the stream blocks or all but
// a few do.  With two stream blocks on every compute unit (long caches) they would start only when stream blocks end, before the tracking blocks,
// and hold their places until the unit's last block is there: that one merges then.  us per call, merging blocks / its last
// block: 53 units x 13000 / 20000 entries, 9 blocks, 128 x bf16 70.6 / 69.2, 109.9 / 105.9 (7 or 8 query heads to a KV head 52 x
// 20000 115.9 / 106.9), 128 x fp32 (7) 139.3 / 135.6, 64 x fp32 (7) 117.8 / 114.3; 28 x 24000, 18 blocks, 128 x bf16 (5) 70.4 / 66.4, 128 x fp32
// 127.2 / 125.5; but with three blocks to a compute unit 53 x 8200 of 128 x bf16 44.5 / 46.2, of 64 x fp32 45.4 / 47.0, 28 x 17000
// of 64 x fp32 52.7 / 55.5; and with a tenth of a block per compute unit too many 52 x 8200 of 128 x fp32, one query head to a KV head,
// 76.0 / 80.2, 53 x 16000 of 128 x bf16 79.0 / 80.6 (54 x 24000, more than that, 130 / 126).
int merging_blocks(int units, int n_sub, int n_split, int group, bool f32, int head_dim) {
  if (n_split <= kPairMax) return 0;
  const long long n = static_cast<long long>(merge_blocks(head_dim, group, merge_waves(n_split))) * units;
  const int slots = fused_slots(fused_wave_run(n_sub, n_split), f32, head_dim);
  return static_cast<long long>(n_split) * units + n <= slots + compute_units() / 10 ? static_cast<int>(n) : 0;
}

// Do they come behind the tracking blocks?  They have nothing to do until the stream ends, but where not all blocks fit the chip
// at once they hold places that tracking blocks then wait for until others of their kind end, and the blocks of a unit get
// out of step.  us per call, merging blocks first / last: 25 units x 19000 entries of 128 x fp32 (600 blocks for 512 places)
// 99.2 / 93.0, 17 x 19000 (7 heads, 629) 66.5 / 61.2, 20 x 13000 of 128 x bf16 (8 heads, 640) 29.8 / 27.1.  First where all fit, or all but
// a tenth of the places: they start later otherwise (8 x 8200 of 128 x bf16 8.8 / 9.0, 20 x 10500 of 64 x bf16 13.5 / 13.9, 14 x
// 19000 of 128 x fp32, 560 blocks, 55.3 / 56.4), and where two stream blocks on a compute unit leave the tracking blocks no places
// in any order (56 x 8200 of 128 x bf16 45.9 / 48.0).  Only with tracking blocks in the launch: their number is taken as that of the stream
// blocks.
// First with sequences of their own lengths: places become free where short ones end, and the tracking blocks, which update TS and
// MRI themselves there, then start in those instead of beside the streams from the start on (that this is why is not shown); last /
// first, 7 query heads, 16 units x 20000 32.9 / 28.7, 20 x 16000 32.7 / 29.0, 24 x 12000 30.2 / 27.6, 28 x 12000 34.1 / 29.8 (4
// heads 30.5 / 28.7).
bool merges_last(int n_stream, int n_tracking, int n_merge, int run, bool f32, int head_dim, bool own_lengths) {
  if (own_lengths) return false;
  const long long slots = fused_slots(run, f32, head_dim), others = static_cast<long long>(n_stream) + n_tracking;
  return n_merge > 0 && n_tracking > 0 && others <= slots && 10 * (others + n_merge) > 11 * slots;
}

template <typename T, int D>
hipError_t launch_rows(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev) {
  if (ev) (void)hipEventRecord(ev[0], stream);
  const int n_sub = (a.n_old + 1 + 15) / 16;
  int run = fused_wave_run(n_sub, a.n_split);
  if (run > kRunMax) run = kRunMax;
  const size_t lds_all = static_cast<size_t>(kWaves) * run * 16 * kHeadPad * sizeof(float);
  const int units = a.batch * a.n_kv_heads;
  const int sb = a.n_split * units;
  const T *kc = static_cast<const T *>(a.k_cache), *vc = static_cast<const T *>(a.v_cache);
  const T *kn = static_cast<const T *>(a.k_new), *vn = static_cast<const T *>(a.v_new);
  const T *q = static_cast<const T *>(a.q);
  const int n_merge = merging_blocks(units, n_sub, a.n_split, a.group, Rows<T, D>::kF32, D);
  const bool long_run = fused_wave_run(n_sub, a.n_split) > kRunMax;
  // list waves (blocks of eight waves) where every block of the launch is resident at once: two
  // such blocks fit a compute unit
  constexpr bool kList = !Rows<T, D>::kWide;
  const int tracking = a.track.valid ? sb : 0;     // (n_track is n_split)
  const bool merge_last = merges_last(sb, tracking, n_merge, run, Rows<T, D>::kF32, D, a.slots.prompt_len != nullptr);
  const Places places = places_of(sb, n_merge, merge_last);
  const unsigned shape = pack_shape(units, a.n_split, a.group, a.slots.prompt_len != nullptr, n_merge > 0, merge_last);
  const bool resident = a.n_split <= kPairMax && sb + tracking <= 2 * compute_units();
  const dim3 grid((merge_last ? places.merge + n_merge : places.track + tracking)), block(kBlock), block_l(kList ? 2 * kBlock : kBlock);
#define LAZYEV_LAUNCH(block, ...) \
  hipLaunchKernelGGL((decode_fused_kernel<T, D, __VA_ARGS__>), grid, block, lds_all, stream, kc, vc, kn, vn, q, a.n_old, a.capacity, shape, a)
#define LAZYEV_SPLIT(n) \
  case n: \
    if (long_run) LAZYEV_LAUNCH(block_l, true, true, kList, n); \
    else LAZYEV_LAUNCH(block_l, true, false, kList, n); \
    break;
  if (a.variant == 6 && resident) {   // (n_split <= kPairMax)
    switch (a.n_split) {
      LAZYEV_SPLIT(1)
      LAZYEV_SPLIT(2)
      LAZYEV_SPLIT(3)
      LAZYEV_SPLIT(4)
      LAZYEV_SPLIT(5)
      LAZYEV_SPLIT(6)
      LAZYEV_SPLIT(7)
      LAZYEV_SPLIT(8)
    }
  } else if (a.variant == 6 && a.n_split == 1) {
    // (more than 256 units: no blocks to wait for, no divisions; with the instance for any split 320 units x 64 entries
    // 6.97 us, 6.36 with this one, x 1040 34.2 / 33.5, x 2200 73.4 / 71.1)
    if (long_run) LAZYEV_LAUNCH(block, true, true, false, 1);
    else LAZYEV_LAUNCH(block, true, false, false, 1);
  } else if (a.variant == 6 && long_run) LAZYEV_LAUNCH(block, true, true, false, 0);
  else if (a.variant == 6) LAZYEV_LAUNCH(block, true, false, false, 0);
  else LAZYEV_LAUNCH(block, false, false, false, 0);
#undef LAZYEV_SPLIT
#undef LAZYEV_LAUNCH
  const hipError_t e = hipGetLastError();
  if (ev) { (void)hipEventRecord(ev[1], stream); (void)hipEventRecord(ev[2], stream); }
  return e;
}

}  // namespace

// This file is compiled once per row type (see build.py): the instances for 128-element bf16 rows with
// everything that does not depend on the row type, and the other three row types on their own.
#ifndef LAZYEV_ROWS
#define LAZYEV_ROWS 0
#endif
hipError_t launch_fused_bf16_64(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev);
hipError_t launch_fused_f32_64(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev);
hipError_t launch_fused_f32_128(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev);
#if LAZYEV_ROWS == 0

#ifdef LAZYEV_TIMELINE
// (host) copies the first n_words words of the stamps of the last launch; waits for the device
extern "C" int lazyev_timeline_read(unsigned long long *out, int n_words) {
  if (!out || n_words < 0 || n_words > 2048 * 8) return -1;
  return static_cast<int>(hipMemcpyFromSymbol(out, HIP_SYMBOL(lz_stamp), sizeof(unsigned long long) * n_words));
}
#endif
int decode_fused_split_max() { return kFusedSplitMax; }
uint32_t decode_fused_seq_max() { return kSeqMax; }
uint32_t decode_fused_seq_captured() { return kSeqCaptured; }
size_t decode_fused_record_bytes() { return static_cast<size_t>(kRecWords) * sizeof(unsigned long long); }

// Blocks per unit where there is room for more than kPairMax of them (`most`) and the cache has more than 43 sub-tiles;
// 0: kPairMax or fewer (decode_fused_split).  us per call, 4 query heads to a KV head, one count / another:
//   * all that there is room for up to 15: 20 units x 2000 / 8200 / 20000 entries 8 / 12 8.1 / 7.0, 18.0 / 16.7, 44.0 /
//     41.6 (64 x bf16 8.1 / 6.8, 14.5 / 12.1, 30.7 / 27.9; 128 x fp32 14.5 / 12.5, x 4000 22.5 / 18.8).  22 units x 2000 / 8200 /
//     13000 / 19500 8 / 11 7.7 / 6.7, 18.6 / 17.8, 30.6 / 27.8, 46.4 / 43.0 (64 x bf16 x 2000 / 13000 7.9 / 6.8, 22.1 / 19.1; two blocks to a
//     compute unit, 23, x 24000 53.3 / 52.7 with 11, 64 x bf16 34.0 / 35.5, but with 7 heads 34.8 / 34.3).  28 units x 1000 / 2000 /
//     8200 / 16000 8 / 9 6.2 / 5.8, 7.8 / 7.1, 21.6 / 21.7, 46.4 / 45.4 (7 heads); fp32 (64) 7.7 / 6.9, 9.8 / 8.9, 24.1 / 23.1, 51.9 /
//     50.1; sequences of their own lengths 6.6 / 6.0, 7.6 / 7.0, 18.4 / 18.2, 37.2 / 37.8.
//   * of 128 x bf16 nine and ten from 46 sub-tiles on: 24 units x 690 / 722 6 / 10 5.8 / 6.0, 6.2 / 6.2.  Nine until two blocks to a
//     compute unit take over: 26 units x 16300 / 24000 9 / 19 42.6 / 44.0, 63.7 / 61.5 (64 x bf16 28.0 / 29.0, 40.6 / 39.7, fp32 (64) 47.1 /
//     46.4, 71.3 / 63.5, (128) 84.0 / 82.8, 127 / 119), 28 x 18500 of their own lengths 9 / 18 43.8 / 41.6.
//   * all up to 28 where a wave would have two sub-tiles or more to do with 16, and these otherwise (8 units x 1500 16 / 24 5.5 /
//     5.5, 10 units x 2000 24 / 25 5.7 / 5.6; fp32 rows, whose sub-tiles take longer, before: 6 units x 1500 16 / 24 (64) 6.6 / 6.0, (128) 9.0 /
//     7.7): 11 units x 4000 / 8200 / 24000 16 / 23 7.1 / 6.7, 10.7 / 9.9, 29.1 / 26.0 (64 x bf16 7.1 / 6.8, 9.3 / 8.4, 21.2 / 16.9, fp32 (64) 8.9
//     / 8.1, 13.6 / 11.4, 34.6 / 28.2, (128) 13.6 / 11.9, 23.0 / 19.4, 61.0 / 50.0); 15 units x 8200 / 24000 fp32 16 / 17 (64) 14.7 / 14.3, 38.9 /
//     38.1, (128) 25.7 / 24.7, 72.3 / 68.2; 9 units x 4000 / 8200 / 24000 24 / 28 6.5 / 6.4, 9.0 / 8.6, 21.1 / 21.5 (fp32 (128) 11.3 / 11.3, 18.2 /
//     16.9, 42.4 / 40.9).  But a merging wave reads a record per lane and eight blocks: of bf16 rows 16 instead of 17 and 18 (15 units x
//     4000 / 13000 7.6 / 7.7, 19.4 / 19.8), up to 500 sub-tiles instead of 19 (13 units x 4000 / 8200 7.2 / 7.4, 11.7 / 11.5), up to 240
//     instead of 21 and 23 (12 units x 2000 16 / 21 5.7 / 5.6, with 7 heads 5.8 / 5.8).
//   * beyond, 32 for 6 and 7 units (6 units x 8200 32 / 42 7.1 / 7.6, 7 units 32 / 36 7.7 / 8.0; fp32 rows of 6 units 42 from 500 sub-tiles on: x
//     8200 / 19000 (64) 9.4 / 9.0, 15.4 / 14.7, (128) 14.6 / 13.7, 26.3 / 24.4); 48 and 64, of fp32 rows 51 and 64, for fewer units once a
//     wave has three to do: 4 units x 4000 / 6000 / 12000 32 / 64 6.0 / 6.3, 6.5 / 6.4, 9.0 / 8.4; 5 units x 8200 / 13000 32 / 48 6.9 / 7.1,
//     9.0 / 8.5 (64 x bf16 7.3 / 7.5, 8.4 / 8.4), fp32 rows 32 / 51 (64) 9.4 / 8.5, 11.7 / 10.3, (128) 14.4 / 12.0, 18.8 / 16.3; 4 units of
//     128 x fp32 x 3000 32 / 48 9.2 / 8.6, x 4000 32 / 64 9.5 / 8.9.
static int two_per_compute_unit_from(bool f32, bool own_lengths) { return f32 || own_lengths ? 1024 : 1200; }
static int merged_split(int n_sub, bool f32, int head_dim, bool own_lengths, int most) {
  const int by_length = (n_sub + kWaves - 1) / kWaves;
  if (most <= kPairMax || n_sub < (most <= kPairMax + 2 && !f32 && head_dim == 128 ? 46 : 44)) return 0;
  if (most == kPairMax + 1 && n_sub >= two_per_compute_unit_from(f32, own_lengths)) return 0;
  int n = most;
  if (most >= 16) {
    if (n_sub < (f32 ? 80 : 112)) n = 16;
    else if (most < 24) n = f32 || (most > 18 && n_sub >= (most > 20 ? 240 : 500)) ? most : 16;
    else if (most < 32) n = most;
    else if (most < 48) n = f32 && most >= 40 && n_sub >= 500 ? most : 32;
    else if (n_sub < (f32 && head_dim == 128 && most == kFusedSplitMax ? 180 : !f32 && most < kFusedSplitMax ? 700 : 376)) n = 32;
    else n = f32 ? most : most / 16 * 16;
  }
  return n < by_length ? n : by_length;
}

// Blocks per unit.  us per call, 7 query heads to a KV head, 128 x bf16 unless it says otherwise (one layer again and
// again):
//   * no more blocks than compute units: a second stream block on some of them holds up the whole launch (80 units x
//     2200 entries: 3 blocks per unit 15.6, 4 20.6; 48 units: 5 10.5, 6 14.2), and with two on all of them the bytes
//     in flight only widen the spread of the blocks' ends (128 units x 4144: 49.8 with one, 50.9 with two).
//   * more than eight where there is room: merged_split.
//   * seven or eight blocks where they leave some compute units to the tracking (28 units x 1040 / 2060 / 4200: 6
//     blocks 6.3 / 8.3 / 13.1, 8 6.4 / 8.1 / 12.6); where they fill the chip to the last one, six up to some thousand
//     entries (32 units x 1040 / 4100 / 6200: 6 blocks 6.0 / 13.7 / 18.9, 8 6.2 / 13.5 / 19.5; x 8200 / 12000 26.4 /
//     40.2, 8 25.1 / 37.6; 36 units x 6200 / 12000: 6 21.8 / 43.9, 7 23.2 / 42.5).  The other row types have more to
//     do per byte, or fewer bytes per entry: eight from about 1800 entries on (32 units x 2060 / 4100, 6 / 8: 64 x
//     bf16 8.1 / 8.1, 11.2 / 10.7; 64 x fp32 11.0 / 10.5, 17.2 / 15.5; 128 x fp32 18.3 / 17.1, 29.0 / 26.8; the line
//     is from 128 x fp32 x 1016), and before that where they take a round of sub-tiles less (128 x fp32 x 860 / 960 / 1100 /
//     1300, 6 / 8 12.3 / 10.9, 12.3 / 11.0, 12.9 / 13.3, 14.6 / 13.5; 64 x fp32 x 960 / 1300 7.9 / 8.0, 9.0 / 8.4).
//   * two sub-tiles or more per wave up to 48 (8 units x 500: 4 blocks 5.1, 8 5.4; x 350: 2 5.0, 3 4.9, 4 4.8), but two
//     blocks from a unit's fifth sub-tile on (x 70: 1 4.1, 2 3.8; x 136: 1 4.7, 2 4.3, 3 4.3).  Beyond 48 as many as there is room
//     for, up to eight: six take a third round (30 units x 690 / 760 / 790 6 / 8 6.3 / 6.6, 6.7 / 6.7, 6.8 / 6.7, 64 x bf16 6.1 / 6.4, 6.6 / 6.4, 6.7
//     / 6.5, fp32 (64) 7.1 / 7.4, 7.5 / 7.4, 7.9 / 7.4, (128) 10.5 / 10.8, 10.5 / 10.7, 12.1 / 10.9).  A sub-tile of fp32 rows takes longer
//     than a record more: 4 units x 130 2 / 3 blocks (64) 5.2 / 4.8, (128) 8.4 / 6.9; x 200 2 / 4 5.6 / 5.2, 8.7 / 7.3; x 400
//     (64) 4 / 7 5.9 / 6.0, (128) 4 / 7 8.9 / 8.1; x 500 4 / 5 6.4 / 6.0, 10.3 / 9.1.
//   * where one block per compute unit leaves a good part of the chip idle and the cache is long, up to two per
//     compute unit (96 units x 6200: 2 blocks per unit 60.6, 5 57.0; 144 units: 1 96.9, 3 90.2; x 2200 18.5 against
//     22.3 and 32.6 against 30.1: from 32 sub-tiles per wave on).  From 171 units on that would be two blocks, and
//     one is the better (1 / 2 blocks, 172 units x 600 11.1 / 12.7, x 2200 35.8 / 36.7, x 6200 110 / 117; 192 units
//     11.2 / 12.9, 36.6 / 38.2, 118 / 125; 240 units 12.5 / 15.2, 44.8 / 44.5, 139 / 143), as it is for fp32 rows
//     (192 units x 2200, 64 43.8 / 44.4, 128 79.3 / 84.9); bf16 rows of 64 would gain from two (176 units x 2200 24.3
//     / 22.5).
int decode_fused_split(int units, int n_sub, bool f32, int head_dim, bool own_lengths) {
  const int chip = compute_units();                // (the figures above are from 256)
  int n = chip / units;
  if (n < 1) n = 1;
  const int merged = merged_split(n_sub, f32, head_dim, own_lengths, n < kFusedSplitMax ? n : kFusedSplitMax);
  if (merged > kPairMax) return merged;
  if (n > kPairMax) n = kPairMax;
  const bool fewer = f32 && n == kPairMax && (head_dim == 128 || n_sub > 72) && fused_wave_run(n_sub, n) < fused_wave_run(n_sub, 6);
  if (n > 6 && 16 * n * units > 15 * chip && n_sub < (n < kPairMax ? 512 : !f32 && head_dim == 128 ? 480 : 112) && !fewer) n = 6;
  int by_work = n_sub <= kWaves ? 1 : n_sub < 4 * kWaves ? 2 : n_sub <= 48 ? (n_sub + kWaves) / (2 * kWaves) : kPairMax;
  if (f32 && n_sub <= (head_dim == 128 ? 32 : 16)) by_work = (n_sub + kWaves - 1) / kWaves;
  else if (f32 && n_sub < 44) by_work = head_dim == 128 ? (n_sub + 7) / 8 : (n_sub + 6) / 7;
  if (n > by_work) n = by_work;
  const int n2 = 2 * chip / units;
  // (28 units x 17000 of 128 x bf16: 8 blocks 48.0, 18 50.8; x 20000 56.1, 55.3; 128 x fp32 x 17000 96.8, 93.7)
  const int two_from = n == kPairMax ? two_per_compute_unit_from(f32, own_lengths) : 32 * kWaves * n;
  if (units < chip && n_sub >= two_from && 10 * n2 * units >= 10 * 2 * n * units + 2 * chip) n = n2;
  return n;
}

void decode_fused_places(int units, int n_sub, int n_split, int group, bool tracking, bool f32, int head_dim, bool own_lengths,
                         int32_t *merge, int32_t *n_merge, int32_t *track) {
  const int sb = units * n_split, run = fused_wave_run(n_sub, n_split);
  *n_merge = merging_blocks(units, n_sub, n_split, group, f32, head_dim);
  const Places p = places_of(sb, *n_merge, merges_last(sb, tracking ? sb : 0, *n_merge, run, f32, head_dim, own_lengths));
  *merge = p.merge;
  *track = p.track;
}

// A unit of up to kPairMax blocks hands over a record less than it has blocks, one of more a record each (also where its last
// block merges and hands over none: which it is differs from call to call).  With decode_fused_split's two blocks per
// compute unit that is an area of 4.5 MB at most; lazyev_set_target_blocks may ask for more, as far as the area that is there
// anyway holds them.
int decode_fused_records_of(int n_split) { return n_split > kPairMax ? n_split : n_split - 1; }
int decode_fused_records_needed(int units, int capacity) {
  const int by_length = ((capacity + 15) / 16 + 3) / 4, by_units = (2 * 256 + units - 1) / units;   // (of the whole chip: without a device too)
  const int n = by_length < by_units ? by_length : by_units;
  return decode_fused_records_of(n < kFusedSplitMax ? n : kFusedSplitMax);
}
int decode_fused_records_held(int units, int capacity, size_t bytes) {
  const int by_length = ((capacity + 15) / 16 + 3) / 4;
  const int most = decode_fused_records_of(by_length < kFusedSplitMax ? by_length : kFusedSplitMax);
  const size_t n = bytes / (decode_fused_record_bytes() * units);
  return n < static_cast<size_t>(most) ? static_cast<int>(n) : most;
}

hipError_t launch_clear_records(unsigned long long *rec, int units, int rec_per_unit, int n_records, hipStream_t stream) {
  if (!rec || units < 1 || n_records < 0 || n_records > rec_per_unit) return hipErrorInvalidValue;
  if (n_records == 0) return hipSuccess;
  hipLaunchKernelGGL(clear_records_kernel, dim3(units), dim3(kBlock), 0, stream, rec, rec_per_unit, n_records);
  return hipGetLastError();
}

bool decode_fused_compact_fits(int n_old, int n_split, int p_stride, int group) {
  if (n_split < 1 || n_split > kFusedSplitMax || group > kHeadPad) return false;
  const int cap = fused_part_cap(n_old, n_split);
  return static_cast<long long>(cap) * n_split <= p_stride;
}

hipError_t launch_track(const TrackArgs &k, hipStream_t stream) {
  if (!k.valid || k.units < 1 || k.group > kHeadPad || !k.logits || !k.stat ||
      k.p_stride < (k.n_old + 16) / 16 * 16)
    return hipErrorInvalidValue;
  if (k.compact && k.group == kHeadPad && !k.cand_index) return hipErrorInvalidValue;
  if (k.compact && (k.p_out || k.p_override || !decode_fused_compact_fits(k.n_old, k.n_parts, k.p_stride, k.group)))
    return hipErrorInvalidValue;
  int n_parts = (k.n_old + 1 + 2 * kBlock - 1) / (2 * kBlock);   // about two entries per thread
  if (n_parts > 64) n_parts = 64;
  if (k.compact) n_parts = k.n_parts;              // one block per block of the call
  if (k.precise) hipLaunchKernelGGL(track_kernel<true>, dim3(k.units * n_parts), dim3(kBlock), 0, stream, k, n_parts);
  else hipLaunchKernelGGL(track_kernel<false>, dim3(k.units * n_parts), dim3(kBlock), 0, stream, k, n_parts);
  return hipGetLastError();
}

int decode_fused_log_words_max() { return static_cast<int>(sizeof(u32x4_t) * kWaves * 256 / sizeof(unsigned)); }

hipError_t launch_track_flush(const FlushArgs &f, int n_layers, hipStream_t stream) {
  if (!f.ts || !f.mri || !f.pos || !f.bitlog || f.units < 1 || n_layers < 1 || n_layers > kFlushLayers ||
      f.capacity < 1 || f.log_words < (f.capacity + 31) / 32 || f.log_slots > kLogSlotsMax)
    return hipErrorInvalidValue;
  bool any = false;
  for (int l = 0; l < n_layers; ++l) {
    if (f.layer[l].n_calls < 0 || f.layer[l].n_calls > f.log_slots) return hipErrorInvalidValue;
    any = any || f.layer[l].n_calls > 0;
  }
  if (!any) return hipSuccess;
  const unsigned spans = static_cast<unsigned>((f.capacity + kFlushSpan - 1) / kFlushSpan);
  hipLaunchKernelGGL(track_flush_kernel, dim3(static_cast<unsigned>(n_layers) * f.units * spans), dim3(kBlock), 0, stream, f);
  return hipGetLastError();
}

hipError_t launch_decode_fused(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev) {
  const int units = a.batch * a.n_kv_heads;
  if (a.group > kHeadPad || a.n_split < 1 ||
      a.n_split > kFusedSplitMax || decode_fused_records_of(a.n_split) > a.rec_per_unit || a.n_track != a.n_split || !a.logits_out ||
      !a.ws.part_rec || !a.ws.fault || a.seq == 0 || a.seq > kSeqCaptured ||
      !a.stat_out || a.p_stride < (a.n_old + 16) / 16 * 16 ||
      (a.track.valid && (a.track.units != units || !a.track.logits || !a.track.stat ||
                         a.track.logits == a.logits_out || a.track.stat == a.stat_out)) ||
      (a.track.valid && a.track.compact &&
       (a.track.p_out || a.track.p_override ||
        !decode_fused_compact_fits(a.track.n_old, a.track.n_parts, a.track.p_stride, a.track.group))) ||
      (a.track.valid && a.track.bitlog &&
       (a.track.log_words < (a.track.capacity + 31) / 32 || a.track.log_words > decode_fused_log_words_max() ||
        a.track.log_unit_stride < a.track.log_words ||
        a.track.slots.prompt_len)) ||
      (a.track.valid && a.track.compact && a.track.group == kHeadPad && !a.track.cand_index) ||
      (a.variant == 6 && a.group == kHeadPad && !a.cand_index_out) ||
      (a.variant == 6 && (a.p_out || a.p_override || !decode_fused_compact_fits(a.n_old, a.n_split, a.p_stride, a.group))))
    return hipErrorInvalidValue;
  if (a.dtype == 1 && a.head_dim == 128) return launch_rows<bf16_t, 128>(a, stream, ev);
  if (a.dtype == 1 && a.head_dim == 64) return launch_fused_bf16_64(a, stream, ev);
  if (a.dtype == 0 && a.head_dim == 64) return launch_fused_f32_64(a, stream, ev);
  if (a.dtype == 0 && a.head_dim == 128) return launch_fused_f32_128(a, stream, ev);
  return hipErrorInvalidValue;
}

#elif LAZYEV_ROWS == 1
hipError_t launch_fused_bf16_64(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev) { return launch_rows<bf16_t, 64>(a, stream, ev); }
#elif LAZYEV_ROWS == 2
hipError_t launch_fused_f32_64(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev) { return launch_rows<float, 64>(a, stream, ev); }
#elif LAZYEV_ROWS == 3
hipError_t launch_fused_f32_128(const DecodeArgs &a, hipStream_t stream, hipEvent_t *ev) { return launch_rows<float, 128>(a, stream, ev); }
#endif

}  // namespace lazyev
