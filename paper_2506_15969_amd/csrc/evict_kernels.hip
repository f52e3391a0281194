// Lagged eviction of one layer (Sec. 4 "MRI-Centric Eviction", Eq. 3, Eq. 6, Alg. 1 of the
// paper), as two kernels:
//   select  one block per unit: applies the tracking that is outstanding (see evict_applies_tracking),
//           scores every candidate entry (all but the last W) in binary64,
//           finds the (B-W)-th largest score with an 8-bit radix select over the score bit
//           patterns held in registers (beyond 8192 entries in LDS, beyond 8192 candidates in the
//           workspace), breaks ties in favour of the more recent entry, prefix-scans
//           the keep flags into destination slots, compacts TS / MRI / pos in place and leaves
//           the gather list (source entry of every survivor) in the workspace.
//   move    blocks per (unit, K|V, 128-byte column part): walk the gather list in order and
//           move the rows whose slot changes; loads of a tile complete before its stores.
//
// This file is compiled with floating-point contraction off: the score is a fixed sequence of
// individually rounded binary64 operations so that it can be reproduced bit for bit elsewhere.
#include "bits.h"
#include "kernels.h"
#include "track.h"

#include <type_traits>

namespace lazyev {
namespace {

constexpr int kSelBlock = 1024;
constexpr int kSelWaves = kSelBlock / 64;
constexpr int kMoveBlock = 1024;
constexpr int kLdsCandidates = 8192;               // keys of 8 bytes in the 64 KB of dynamic LDS a launch gets
constexpr int kSmallSet = 256;                     // radix select: at most this many keys left -> ranked directly

// 2*sigmoid(-x) = 2/(1+e^x) for x >= 0.  e^x = 2^k * e^r with k = round(x/ln 2) and
// r = x - k ln 2 taken in two pieces (the high piece of ln 2 has 32 significant bits, so
// k * kLn2Hi is exact); e^r by the degree-13 Taylor polynomial in Horner form.  Every
// multiply, add and divide below is a separate round-to-nearest operation.
__device__ double two_sigmoid_neg(double x) {
#pragma clang fp contract(off)
  constexpr double kLog2e = 0x1.71547652b82fep+0;
  constexpr double kLn2Hi = 0x1.62e42fee00000p-1;
  constexpr double kLn2Lo = 0x1.a39ef35793c76p-33;
  constexpr double kCoef[14] = {1.0 / 1.0, 1.0 / 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0,
                                1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0, 1.0 / 40320.0,
                                1.0 / 362880.0, 1.0 / 3628800.0, 1.0 / 39916800.0,
                                1.0 / 479001600.0, 1.0 / 6227020800.0};
  if (!(x < 700.0)) return 0.0;
  const double k = floor(x * kLog2e + 0.5);
  const double r = (x - k * kLn2Hi) - k * kLn2Lo;
  double p = kCoef[13];
#pragma unroll
  for (int n = 12; n >= 0; --n) {
    p = p * r;
    p = p + kCoef[n];
  }
  const double e = ldexp(p, static_cast<int>(k));
  return 2.0 / (1.0 + e);
}

// Eq. 3.  delta_t = t - TS >= 0, mri >= 0.
__device__ double mri_centric_score(int32_t delta_t, int32_t mri, int32_t flags) {
#pragma clang fp contract(off)
  double h1 = 0.0, h2 = 0.0;
  if (flags & 1) {
    if (mri > 0) h1 = two_sigmoid_neg(static_cast<double>(delta_t) / static_cast<double>(mri));
    else h1 = (delta_t == 0) ? 1.0 : 0.0;
  }
  if ((flags & 2) && mri > 1) h2 = two_sigmoid_neg(1.0 / (static_cast<double>(mri) - 1.0));
  // reflected second term (falls with MRI, as the prose of Sec. 4 item 2 and App. D ask)
  if ((flags & 2) && (flags & 16)) h2 = (mri >= 1) ? 1.0 - h2 : 0.0;
  return h1 + h2;
}

__global__ void score_pairs_kernel(const int32_t *dt, const int32_t *mri, double *score,
                                   int64_t n, int32_t flags) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) score[i] = mri_centric_score(dt[i], mri[i], flags);
}

// Counts the first n entries (seq_len[sequence], when not null) of every unit by MRI value; values >=
// n_bins - 1 share the last bin.  A block counts kHistSpan entries of one unit in LDS and adds its
// bins to the result once: with an addition to global memory per entry the few values that most
// entries have were a queue of some hundred thousand (32 units of 16400 entries in all, 460 -> 5.6 us).  Most entries
// have MRI = 0: those are counted per wave, not per lane.
constexpr int kHistBlock = 256;
constexpr int kHistSpan = 8 * kHistBlock;
__global__ __launch_bounds__(kHistBlock) void mri_histogram_kernel(const int32_t *mri, int32_t capacity, int32_t n_kv_heads,
                                                                   const int32_t *seq_len, int32_t n, int32_t spans,
                                                                   int32_t n_bins, unsigned long long *hist) {
  extern __shared__ unsigned bins[];
  const int unit = blockIdx.x / spans, first = blockIdx.x % spans * kHistSpan;
  const int len = seq_len ? min(seq_len[unit / n_kv_heads], n) : n;
  if (first >= len) return;
  const int32_t *m_unit = mri + static_cast<size_t>(unit) * capacity;
  int32_t m[kHistSpan / kHistBlock];
#pragma unroll
  for (int r = 0; r < kHistSpan / kHistBlock; ++r) {
    const int i = first + r * kHistBlock + static_cast<int>(threadIdx.x);
    m[r] = i < len ? m_unit[i] : -1;
  }
  for (int b = threadIdx.x; b < n_bins; b += kHistBlock) bins[b] = 0;
  __syncthreads();
  unsigned zeros = 0;
#pragma unroll
  for (int r = 0; r < kHistSpan / kHistBlock; ++r) {
    zeros += static_cast<unsigned>(__popcll(__builtin_amdgcn_ballot_w64(m[r] == 0)));
    if (m[r] > 0) atomicAdd(&bins[min(m[r], n_bins - 1)], 1u);
  }
  if ((threadIdx.x & 63) == 0 && zeros != 0) atomicAdd(&bins[0], zeros);
  __syncthreads();
  for (int b = threadIdx.x; b < n_bins; b += kHistBlock)
    if (bins[b] != 0) atomicAdd(&hist[b], static_cast<unsigned long long>(bins[b]));
}

// A sequence starts over in its slot: the state of lazyev_init for its units in every layer,
// and its timing record.
__global__ void init_slot_kernel(int32_t *ts, int32_t *mri, int32_t *pos, int32_t n_layers,
                                 int32_t batch, int32_t n_kv_heads, int32_t capacity, int32_t seq,
                                 int32_t prompt_len, int32_t *dev_prompt_len, int32_t *dev_t0,
                                 int32_t t0) {
  const int64_t per_layer = static_cast<int64_t>(n_kv_heads) * capacity;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i == 0) { dev_prompt_len[seq] = prompt_len; dev_t0[seq] = t0; }
  if (i >= n_layers * per_layer) return;
  const int64_t layer = i / per_layer, r = i % per_layer;
  const int64_t at = ((layer * batch + seq) * n_kv_heads) * capacity + r;
  const int32_t slot = static_cast<int32_t>(r % capacity);
  ts[at] = 0;
  mri[at] = 0;
  pos[at] = slot < prompt_len ? slot : -1;
}

// The state of every entry, and the first rec_words of the rec_stride words that each of rec_units units has for its
// records of partials (here, because a launch of their own added 4 us to lazyev_init).
__global__ void init_state_kernel(int32_t *ts, int32_t *mri, int32_t *pos, int64_t total,
                                  int32_t capacity, int32_t prompt_len, unsigned long long *rec, int32_t rec_units,
                                  int32_t rec_stride, int32_t rec_words) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t words = static_cast<int64_t>(rec_units) * rec_words;
  for (int64_t j = i; j < words; j += static_cast<int64_t>(gridDim.x) * blockDim.x)
    rec[j / rec_words * rec_stride + j % rec_words] = 0;
  if (i >= total) return;
  const int32_t slot = static_cast<int32_t>(i % capacity);
  ts[i] = 0;
  mri[i] = 0;
  pos[i] = slot < prompt_len ? slot : -1;
}

// Exclusive prefix sum of one value per thread over the whole block; `total` is the block sum.
__device__ unsigned block_exclusive_scan(unsigned v, unsigned *wave_tot, unsigned &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  unsigned base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const unsigned x = wave_tot[w];
    all += x;
    if (w < wave) base += x;
  }
  __syncthreads();
  total = all;
  return base + incl - v;
}

// Entries of the unit and its step, if its eviction is due (with per-sequence timing a launch also holds units that
// have none).
__device__ __forceinline__ bool unit_due(const EvictArgs &a, int unit, int &n, int &t) {
  n = a.n;
  t = a.t;
  if (!a.slots.prompt_len) return true;
  const int seq = (unit % a.units_per_layer) / a.n_kv_heads;
  const int32_t P = a.slots.prompt_len[seq], tau = a.t - a.slots.t0[seq];
  if (P < 0 || tau < 1 || tau % a.window != 0) return false;
  n = slot_n_old(P, tau, a.budget, a.window) + 1;
  t = tau;
  return n > a.budget;
}

// Score = the weight each candidate received at this step, largest over the query group: the same
// fp32 expression the tracking uses, widened exactly.
__device__ __forceinline__ void weight_keys(const EvictArgs &a, int unit, int n_cand, unsigned long long *keys) {
  const float *lg = a.logits + static_cast<size_t>(unit) * a.p_stride * 8;
  const float *st = a.stat + static_cast<size_t>(unit) * 16;
  for (int i = threadIdx.x; i < n_cand; i += kSelBlock) {
    const float4 sa = *reinterpret_cast<const float4 *>(lg + static_cast<size_t>(i) * 8);
    const float4 sb = *reinterpret_cast<const float4 *>(lg + static_cast<size_t>(i) * 8 + 4);
    const float sv[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
    float best = 0.f;
#pragma unroll
    for (int h = 0; h < 8; ++h)
      if (h < a.group) best = fmaxf(best, __expf(sv[h] - st[2 * h]) * st[2 * h + 1]);
    keys[i] = static_cast<unsigned long long>(__double_as_longlong(static_cast<double>(best)));
  }
}

// Inclusive sums over the lanes of a wave, by moves within the vector ALU: inside the rows of 16, then the last
// lane of a row (of the lower half) into the next row (the upper half).
__device__ __forceinline__ unsigned wave_scan(unsigned v) {
  auto add = [&](auto ctrl, auto rows) {
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
  };
  constexpr std::integral_constant<int, 0xF> all{};
  add(std::integral_constant<int, 0x111>{}, all);  // row_shr:1
  add(std::integral_constant<int, 0x112>{}, all);
  add(std::integral_constant<int, 0x114>{}, all);
  add(std::integral_constant<int, 0x118>{}, all);  // row_shr:8
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});   // row_bcast:15 into rows 1 and 3
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});   // row_bcast:31 into rows 2 and 3
  return v;
}

// The records of the last call before the eviction (Alg. 1, first loop): bits of the active entries.  Wave w takes
// the regions w, w + 16, ... of the unit.
template <bool kPrecise>
__device__ __forceinline__ unsigned last_call_bits(const TrackArgs &k, int unit, unsigned *active) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cap = fused_part_cap(k.n_old, k.n_parts);
  float m[kHeadPad], invl[kHeadPad];
#pragma unroll
  for (int h = 0; h < kHeadPad; ++h) {
    m[h] = k.stat[static_cast<size_t>(unit) * (2 * kHeadPad) + 2 * h];
    invl[h] = k.stat[static_cast<size_t>(unit) * (2 * kHeadPad) + 2 * h + 1];
  }
  unsigned n_act = 0;
  for (int b = wave; b < k.n_parts; b += kSelWaves) {
    const size_t at = static_cast<size_t>(unit) * k.p_stride + static_cast<size_t>(b) * cap;
    const float *region = k.logits + at * kHeadPad;
    const int n = region_count(region, cap);
    for (int r = lane; r < n; r += 64) {
      const float4 sa = *reinterpret_cast<const float4 *>(region + static_cast<size_t>(1 + r) * kHeadPad);
      const float4 sb = *reinterpret_cast<const float4 *>(region + static_cast<size_t>(1 + r) * kHeadPad + 4);
      const bool eight = k.group == kHeadPad;      // (groups of eight have the index beside the records)
      const int i = record_entry(eight ? k.cand_index[at + 1 + r] : __float_as_int(sb.w), k.n_old);
      const float s[kHeadPad] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
      bool act = false;
#pragma unroll
      for (int h = 0; h < kHeadPad; ++h)
        if (h < k.group) act = act || weight_of<kPrecise>(s[h], m[h], invl[h]) >= k.alpha;
      if (act) {
        n_act += 1;
        if (i != k.n_old) atomicOr(&active[i >> 5], 1u << (i & 31));   // (the appended entry starts at its own step)
      }
    }
  }
  return n_act;
}

// Applies what is outstanding to the entries in registers, entry r * kSelBlock + tid in place r: the updates of
// track_flush_kernel and track_kernel.  A wave has 64 entries in a row, two words of a call: lane (half, j) brings
// word `half` of call s + j, and after a transposition across the 32 lanes holds the 32 calls of entry 32 half + j.
template <int R>
__device__ __forceinline__ void apply_outstanding(const EvictArgs &a, int unit, int32_t (&v_ts)[R], int32_t (&v_mri)[R], int32_t (&v_pos)[R],
                                                  unsigned *active, unsigned *n_active) {
  const OutstandingArgs &o = a.todo;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int layer = unit / a.units_per_layer, unit_l = unit % a.units_per_layer;
  const FlushArgs::Layer of = o.layer[layer];
  const bool last = layer == o.last_layer;
  if (last) {
    for (int i = tid; i < R * kSelBlock / 32; i += kSelBlock) active[i] = 0;
    if (tid == 0) *n_active = 0;
    __syncthreads();
    unsigned n = o.last.precise ? last_call_bits<true>(o.last, unit_l, active) : last_call_bits<false>(o.last, unit_l, active);
    for (int x = 32; x > 0; x >>= 1) n += __shfl_xor(n, x);
    if (lane == 0 && n) atomicAdd(n_active, n);
  }
  const int half = lane >> 5, j = lane & 31;
  const uint32_t *log = o.bitlog + static_cast<size_t>(unit) * o.log_slots * o.log_words;   // (a unit's slots lie together)
#pragma unroll
  for (int r = 0; r < R; ++r) {                    // entries that the logged calls appended start there
    const int s_new = r * kSelBlock + tid - of.n_old;
    if (s_new >= 0 && s_new < of.n_calls) {
      v_ts[r] = of.t + s_new;
      v_mri[r] = 0;
      v_pos[r] = o.prompt_len + v_ts[r] - 1;
    }
  }
  constexpr int kBatch = R <= 3 ? 4 : 2;           // sets of 32 calls requested together
  for (int s0 = 0; s0 < of.n_calls; s0 += 32 * kBatch) {
    unsigned w[kBatch][R];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const uint32_t *row = log + static_cast<size_t>(min(s0 + 32 * b + j, of.n_calls - 1)) * o.log_words;
#pragma unroll
      for (int r = 0; r < R; ++r) w[b][r] = row[min((r * kSelBlock + wave * 64) / 32 + half, o.log_words - 1)];
    }
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int s = s0 + 32 * b;
      if (s >= of.n_calls) break;                  // (uniform)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        apply_calls(transpose_bits<32>(s + j < of.n_calls ? w[b][r] : 0u, j), of.t + s, v_ts[r], v_mri[r]);
      }
    }
  }
  if (last) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = r * kSelBlock + tid;
      if (i == o.last.n_old) {
        v_ts[r] = o.last.t;
        v_mri[r] = 0;
        v_pos[r] = o.last.prompt_len + o.last.t - 1;
      } else if ((active[i >> 5] >> (i & 31)) & 1u) {
        v_mri[r] = max(v_mri[r], o.last.t - v_ts[r]);
        v_ts[r] = o.last.t;
      }
    }
    if (tid == 0) o.last.activation_counter[unit_l * 64] += *n_active;
  }
}

// The selection for units of at most R * kSelBlock entries.  One block per unit, so what bounds it is the chain of
// its steps (and the scores, at 4096 entries): memory is read once, at the start (TS, MRI and pos stay in registers,
// R entries per thread), the keys lie in registers, every wave finds the threshold's digit for itself, and the
// destinations of all entries come from one exchange of counts.  us, before (keys in LDS, shuffles of 16 waves
// queueing up at it for ANDs, ORs and scans, a pass over TS / MRI / pos per 1024 entries at the end, as
// evict_select_kernel still has it) and now: 144 entries 9.2 -> 5.3, 1056 15.6 -> 7.2, 2112 17.5 -> 10.0, 256 units
// of 4160 29.6 -> 17.1.
// The first digit is 0 for the score 0 (the usual threshold: the entries that were never re-activated) and the score
// in steps of 1 / 126 from 1 on (scores lie in 0 .. 2, weights in 0 .. 1), which tells keys apart better than their
// leading byte: mostly one pass ends at the zeros or leaves at most kSmallSet keys.  The following digits are the
// bytes, the highest first, of the keys still in play.
// kTodo: tracking is outstanding (a.todo).  Evictions without, those of many units among them, have an instance of
// their own, as the registers of the other leave room for fewer blocks on a compute unit (3 entries per thread: 68
// instead of 56): us, tracking and row move included, one instance for both / this one, 2048 units of 432 entries
// 178 / 166, 3584 302 / 283.
template <int R, bool kTodo>
__global__ __launch_bounds__(kSelBlock) void evict_select_held_kernel(const EvictArgs a) {
  extern __shared__ unsigned long long keys_lds[];      // score bit pattern of each candidate
  __shared__ unsigned active[kTodo ? R * kSelBlock / 32 : 1];   // the last call's activations, a bit per entry
  __shared__ unsigned n_active;
  __shared__ unsigned hist[3][256];                // of passes p, p + 1, p + 2: a barrier lies between the last reading
  __shared__ unsigned long long wave_key[2][kSelWaves];   // of one, its clearing and its next use
  __shared__ unsigned wave_kind[2][kSelWaves];     // keys of the wave in play: 0 none, 1 all wave_key, 2 several values
  __shared__ unsigned long long small_keys[kSmallSet];
  __shared__ unsigned small_n, moved, sel_rem, sel_cnt;
  __shared__ unsigned long long small_thr;
  __shared__ unsigned count[128];                  // [R][waves] ties << 16 | certain survivors
  static_assert(R * kSelWaves <= 128 && R * kSelBlock < 65536, "counts of a unit");

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = evict_unit_of(a, blockIdx.x);
  int n, t;
  if (!unit_due(a, unit, n, t)) return;
  const int n_cand = n - a.window, k_keep = a.budget - a.window;
  int32_t *ts = a.ts + static_cast<size_t>(unit) * a.capacity;
  int32_t *mri = a.mri + static_cast<size_t>(unit) * a.capacity;
  int32_t *pos = a.pos + static_cast<size_t>(unit) * a.capacity;
  int32_t *src_index = a.ws.src_index + static_cast<size_t>(unit) * a.capacity;
  int32_t v_ts[R], v_mri[R], v_pos[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int slot = r * kSelBlock + tid;
    v_ts[r] = v_mri[r] = v_pos[r] = 0;
    if (slot < n) { v_ts[r] = ts[slot]; v_mri[r] = mri[slot]; v_pos[r] = pos[slot]; }
  }
  if constexpr (kTodo) apply_outstanding<R>(a, unit, v_ts, v_mri, v_pos, active, &n_active);
  if (tid < 256) hist[0][tid] = hist[1][tid] = hist[2][tid] = 0;
  if (tid == 0) { small_n = 0; moved = 0; }

  // scores (non-negative doubles order like their bit patterns); the slots of a thread are its own, and its
  // loop over them stays a loop: the code of R scores in a row would have to be fetched by every launch
  if (a.score_flags & 32) {
    weight_keys(a, unit, n_cand, keys_lds);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int slot = r * kSelBlock + tid;
      if (slot < n_cand)
        keys_lds[slot] = (static_cast<unsigned long long>(static_cast<unsigned>(t - v_ts[r])) << 32) | static_cast<unsigned>(v_mri[r]);
    }
#pragma unroll 1
    for (int i = tid; i < n_cand; i += kSelBlock) {
      const unsigned long long x = keys_lds[i];
      keys_lds[i] = static_cast<unsigned long long>(__double_as_longlong(
          mri_centric_score(static_cast<int32_t>(x >> 32), static_cast<int32_t>(x), a.score_flags)));
    }
  }
  unsigned long long key[R];
  unsigned alive = 0;                              // bit r: key[r] is still in play
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int slot = r * kSelBlock + tid;
    key[r] = slot < n_cand ? keys_lds[slot] : 0ull;
    alive |= (slot < n_cand ? 1u : 0u) << r;
  }
  __syncthreads();                                 // the counters are cleared

  unsigned long long thr = 0;
  unsigned k_rem = static_cast<unsigned>(k_keep);  // kept among the keys still in play ...
  unsigned ties_total = static_cast<unsigned>(n_cand);   // ... of which there are this many
  for (int pass = 0, pb = 0;; ++pass, pb = pb == 2 ? 0 : pb + 1) {
    auto digit_of = [&](unsigned long long k) -> unsigned {
      if (pass == 0) return k == 0ull ? 0u : 1u + min(static_cast<unsigned>(__longlong_as_double(static_cast<long long>(k)) * 126.0), 254u);
      return static_cast<unsigned>(k >> (64 - 8 * min(pass, 8))) & 255u;
    };
    // this wave's keys in play: are they one value?  (No shuffles: those of 16 waves queue up at the LDS.)
    unsigned long long some = 0;
#pragma unroll
    for (int r = R - 1; r >= 0; --r) some = (alive >> r) & 1u ? key[r] : some;
    const unsigned long long any = __builtin_amdgcn_ballot_w64(alive != 0);
    const int first = any ? __ffsll(static_cast<long long>(any)) - 1 : 0;
    const unsigned long long ref =
        (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(some >> 32), first))) << 32) |
        static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(some), first));
    bool other = false;
    unsigned zeros = 0;                            // (a third of the keys or so are 0: counted per wave)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool in = (alive >> r) & 1u;
      zeros += static_cast<unsigned>(__popcll(__builtin_amdgcn_ballot_w64(in && key[r] == 0ull)));
      other = other || (in && key[r] != ref);
      if (in && key[r] != 0ull) atomicAdd(&hist[pb][digit_of(key[r])], 1u);
    }
    const bool mixed = __builtin_amdgcn_ballot_w64(other) != 0;
    if (lane == 0) {
      if (zeros) atomicAdd(&hist[pb][0], zeros);
      wave_key[pass & 1][wave] = ref;
      wave_kind[pass & 1][wave] = any == 0 ? 0u : mixed ? 2u : 1u;
    }
    __syncthreads();
    {
      const unsigned kind = lane < kSelWaves ? wave_kind[pass & 1][lane] : 0u;
      const unsigned long long k = lane < kSelWaves ? wave_key[pass & 1][lane] : 0ull;
      const unsigned long long single = __builtin_amdgcn_ballot_w64(kind == 1u);
      const int at = single ? __ffsll(static_cast<long long>(single)) - 1 : 0;
      thr = (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(k >> 32), at))) << 32) |
            static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(k), at));
      // all keys in play are one value (at the latest after the last byte)
      if (__builtin_amdgcn_ballot_w64(kind == 2u || (kind == 1u && k != thr)) == 0 || pass == 9) break;
    }
    // lane l of every wave takes the digits 255 - 4 l .. 252 - 4 l, the largest first
    const uint4 h = *reinterpret_cast<const uint4 *>(&hist[pb][252 - 4 * lane]);
    const unsigned sum = h.x + h.y + h.z + h.w;
    unsigned above = wave_scan(sum) - sum;
    const unsigned in_lane[4] = {h.w, h.z, h.y, h.x};
    unsigned found = 0, rem = 0, cnt = 0;          // found: digit + 1
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (above < k_rem && k_rem <= above + in_lane[x]) { found = 256u - 4 * lane - x; rem = k_rem - above; cnt = in_lane[x]; }
      above += in_lane[x];
    }
    const int at = __ffsll(static_cast<long long>(__builtin_amdgcn_ballot_w64(found != 0))) - 1;   // (one lane has it)
    const unsigned digit = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(found), at)) - 1u;
    k_rem = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(rem), at));
    ties_total = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(cnt), at));
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (digit_of(key[r]) != digit) alive &= ~(1u << r);
    if (pass == 0 && digit == 0u) {                // the threshold falls among the zeros
      thr = 0;
      break;
    }
    const int clear = pb == 0 ? 2 : pb - 1;        // (of the pass before: nobody reads it any more)
    if (tid < 256) hist[clear][tid] = 0;
    if (ties_total <= static_cast<unsigned>(kSmallSet)) {
      // few keys left: listed, and each (four threads) counts the listed keys above it and equal to it
#pragma unroll
      for (int r = 0; r < R; ++r)
        if ((alive >> r) & 1u) small_keys[atomicAdd(&small_n, 1u)] = key[r];
      __syncthreads();
      const unsigned mine = static_cast<unsigned>(tid) >> 2;
      const unsigned long long k = small_keys[mine < ties_total ? mine : 0];
      unsigned gt = 0, eq = 0;
      for (unsigned j = tid & 3; j < ties_total; j += 4) {
        const unsigned long long other = small_keys[j];
        gt += other > k ? 1u : 0u;
        eq += other == k ? 1u : 0u;
      }
      gt += __shfl_xor(gt, 1); eq += __shfl_xor(eq, 1);
      gt += __shfl_xor(gt, 2); eq += __shfl_xor(eq, 2);
      if (mine < ties_total && gt < k_rem && k_rem <= gt + eq) {   // (every holder of that value writes the same)
        small_thr = k;
        sel_rem = k_rem - gt;
        sel_cnt = eq;
      }
      __syncthreads();
      thr = small_thr;
      k_rem = sel_rem;
      ties_total = sel_cnt;
      break;
    }
  }
  // thr is the threshold key; k_rem of the ties_total entries equal to it are kept, the most
  // recent ones (largest slots) first.
  const unsigned drop_ties = ties_total - k_rem;
  unsigned long long definite[R], tie[R];          // of the wave's lanes
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int slot = r * kSelBlock + tid;
    definite[r] = __builtin_amdgcn_ballot_w64(slot < n && (slot >= n_cand || key[r] > thr));
    tie[r] = __builtin_amdgcn_ballot_w64(slot < n_cand && key[r] == thr);
    if (lane == 0)
      count[r * kSelWaves + wave] = (static_cast<unsigned>(__popcll(tie[r])) << 16) | static_cast<unsigned>(__popcll(definite[r]));
    // every read precedes the writes: the loads have returned (touching the values makes the compiler wait for
    // them; the barrier alone only drains the LDS counter), in every thread
    __asm__ volatile("" : "+v"(v_ts[r]), "+v"(v_mri[r]), "+v"(v_pos[r]));
  }
  __syncthreads();
  const unsigned c0 = 2 * lane < R * kSelWaves ? count[2 * lane] : 0u, c1 = 2 * lane < R * kSelWaves ? count[2 * lane + 1] : 0u;
  const unsigned before = wave_scan(c0 + c1) - (c0 + c1);
  unsigned n_moved = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int slot = r * kSelBlock + tid, e = r * kSelWaves + wave;
    unsigned ex = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(before), e >> 1));
    if (e & 1) ex += static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(c0), e >> 1));
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned def_before = (ex & 0xFFFFu) + static_cast<unsigned>(__popcll(definite[r] & below));
    const unsigned tie_rank = (ex >> 16) + static_cast<unsigned>(__popcll(tie[r] & below));
    const bool keep = ((definite[r] >> lane) & 1ull) || (((tie[r] >> lane) & 1ull) && tie_rank >= drop_ties);
    const unsigned dst = def_before + (tie_rank > drop_ties ? tie_rank - drop_ties : 0u);
    if (keep) {
      ts[dst] = v_ts[r]; mri[dst] = v_mri[r]; pos[dst] = v_pos[r];
      src_index[dst] = slot;
    }
    if (kTodo && slot >= a.budget && slot < n) {   // (places that no survivor takes: as the tracking leaves them)
      ts[slot] = v_ts[r]; mri[slot] = v_mri[r]; pos[slot] = v_pos[r];
    }
    n_moved += static_cast<unsigned>(__popcll(__builtin_amdgcn_ballot_w64(keep && dst != static_cast<unsigned>(slot))));
  }
  // how many survivors change slot (what the row move has to copy); one writer per unit
  if (lane == 0 && n_moved) atomicAdd(&moved, n_moved);
  __syncthreads();
  if (tid == 0) a.rows_moved[unit] += moved;
}

// The selection for more entries than a block holds in registers.
// kKeysInLds: the candidates' keys fit the dynamic LDS of the launch (the usual case); otherwise
// they go through the unit's part of the workspace (same passes over global memory, slower).
template <bool kKeysInLds>
__global__ __launch_bounds__(kSelBlock) void evict_select_kernel(const EvictArgs a) {
  extern __shared__ unsigned long long keys_lds[];      // score bit pattern of each candidate
  __shared__ unsigned hist[256];
  __shared__ unsigned wave_tot[kSelWaves];
  __shared__ unsigned sel_bin, sel_rem, sel_cnt;
  __shared__ unsigned long long and_k[2], or_k[2];
  __shared__ unsigned long long small_keys[kSmallSet];   // the keys still in play, once they are few
  __shared__ unsigned small_n;
  __shared__ unsigned long long small_thr;

  const int tid = threadIdx.x;
  const int unit = evict_unit_of(a, blockIdx.x);
  int n, t;
  if (!unit_due(a, unit, n, t)) return;
  const int n_cand = n - a.window, k_keep = a.budget - a.window;
  int32_t *ts = a.ts + static_cast<size_t>(unit) * a.capacity;
  int32_t *mri = a.mri + static_cast<size_t>(unit) * a.capacity;
  int32_t *pos = a.pos + static_cast<size_t>(unit) * a.capacity;
  int32_t *src_index = a.ws.src_index + static_cast<size_t>(unit) * a.capacity;
  unsigned long long *keys = keys_lds;
  if (!kKeysInLds) keys = a.ws.sel_keys + static_cast<size_t>(unit) * a.capacity;

  // scores (non-negative doubles order like their bit patterns)
  if (a.score_flags & 32) {
    weight_keys(a, unit, n_cand, keys);
  } else {
    for (int i = tid; i < n_cand; i += kSelBlock)
      keys[i] = static_cast<unsigned long long>(
          __double_as_longlong(mri_centric_score(t - ts[i], mri[i], a.score_flags)));
  }
  __syncthreads();

  // Radix select of the k_keep-th largest key, most significant byte first, until at most
  // kSmallSet keys are left in play, which are then ranked directly.  Every pass also
  // forms the AND and the OR of the keys still in play: when they agree, all those keys are
  // the same value (the usual case: the threshold falls among the entries that were never
  // re-activated, which all score exactly 0) and the remaining passes are skipped.
  if (tid < 256) hist[tid] = 0;
  if (tid < 2) { and_k[tid] = ~0ull; or_k[tid] = 0ull; }
  __syncthreads();                                    // also: every key is in LDS
  unsigned long long prefix = 0, mask = 0, thr = 0;
  unsigned k_rem = static_cast<unsigned>(k_keep);     // kept among the keys still in play ...
  unsigned ties_total = static_cast<unsigned>(n_cand);   // ... of which there are this many
  bool all_equal = false;
  for (int shift = 56, pass = 0; shift >= 0; shift -= 8, ++pass) {
    const int pb = pass & 1;
    unsigned long long and_acc = ~0ull, or_acc = 0ull;
    for (int i = tid; i < n_cand; i += kSelBlock) {
      const unsigned long long key = keys[i];
      if ((key & mask) == prefix) {
        atomicAdd(&hist[static_cast<unsigned>(key >> shift) & 255u], 1u);
        and_acc &= key;
        or_acc |= key;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      and_acc &= __shfl_xor(and_acc, o);
      or_acc |= __shfl_xor(or_acc, o);
    }
    if ((tid & 63) == 0) { atomicAnd(&and_k[pb], and_acc); atomicOr(&or_k[pb], or_acc); }
    __syncthreads();
    if (and_k[pb] == or_k[pb]) {                      // the same for every thread of the block
      thr = and_k[pb];
      all_equal = true;
      break;
    }
    const unsigned bin = 255u - static_cast<unsigned>(tid);      // descending digit order
    const unsigned v = tid < 256 ? hist[bin] : 0u;
    unsigned total;
    const unsigned above = block_exclusive_scan(v, wave_tot, total);   // keys in larger digits
    if (tid < 256 && above < k_rem && k_rem <= above + v) {
      sel_bin = bin;
      sel_rem = k_rem - above;
      sel_cnt = v;
    }
    if (tid < 256) hist[tid] = 0;                     // for the next pass (the scan's barriers lie
    if (tid == 0) { and_k[pb ^ 1] = ~0ull; or_k[pb ^ 1] = 0ull; }   // between the reads and this)
    __syncthreads();
    prefix |= static_cast<unsigned long long>(sel_bin) << shift;
    mask |= 255ull << shift;
    k_rem = sel_rem;
    ties_total = sel_cnt;
    if (shift > 0 && ties_total <= static_cast<unsigned>(kSmallSet)) {
      // Few keys left in play: instead of one pass per remaining byte, list them and let each
      // count the listed keys above it and equal to it; the k_rem-th largest is the threshold.
      if (tid == 0) small_n = 0;
      __syncthreads();
      for (int i = tid; i < n_cand; i += kSelBlock) {
        const unsigned long long key = keys[i];
        if ((key & mask) == prefix) small_keys[atomicAdd(&small_n, 1u)] = key;
      }
      __syncthreads();
      if (static_cast<unsigned>(tid) < small_n) {
        const unsigned long long key = small_keys[tid];
        unsigned gt = 0, eq = 0;
        for (unsigned j = 0; j < small_n; ++j) {
          const unsigned long long other = small_keys[j];
          gt += other > key ? 1u : 0u;
          eq += other == key ? 1u : 0u;
        }
        if (gt < k_rem && k_rem <= gt + eq) {         // (every holder of that value writes the same)
          small_thr = key;
          sel_rem = k_rem - gt;
          sel_cnt = eq;
        }
      }
      __syncthreads();
      thr = small_thr;
      k_rem = sel_rem;
      ties_total = sel_cnt;
      all_equal = true;
      break;
    }
  }
  if (!all_equal) thr = prefix;
  // thr is the threshold key; k_rem of the ties_total entries equal to it are kept, the most
  // recent ones (largest slots) first.
  const unsigned drop_ties = ties_total - k_rem;

  unsigned run_def = 0, run_tie = 0, n_moved = 0;
  for (int base = 0; base < n; base += kSelBlock) {
    const int slot = base + tid;
    const bool valid = slot < n;
    const bool cand = slot < n_cand;
    const unsigned long long key = cand ? keys[slot] : 0ull;
    const bool definite = valid && (!cand || key > thr);
    const bool tie = cand && key == thr;
    unsigned total;
    const unsigned ex = block_exclusive_scan((tie ? 65536u : 0u) | (definite ? 1u : 0u),
                                             wave_tot, total);
    const unsigned tie_rank = run_tie + (ex >> 16);
    const unsigned def_before = run_def + (ex & 0xFFFFu);
    const bool keep = definite || (tie && tie_rank >= drop_ties);
    const unsigned kept_ties_before = tie_rank > drop_ties ? tie_rank - drop_ties : 0u;
    const unsigned dst = def_before + kept_ties_before;
    int32_t v_ts = 0, v_mri = 0, v_pos = 0;
    if (keep) { v_ts = ts[slot]; v_mri = mri[slot]; v_pos = pos[slot]; }
    // every read of this pass precedes its writes: the loads have returned (the barrier alone
    // only drains the LDS counter), in every thread
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0)
    __syncthreads();
    if (keep) {
      ts[dst] = v_ts; mri[dst] = v_mri; pos[dst] = v_pos;
      src_index[dst] = slot;
      if (dst != static_cast<unsigned>(slot)) n_moved += 1;
    }
    run_def += total & 0xFFFFu;
    run_tie += total >> 16;
  }
  // how many survivors change slot (what the row move has to copy); one writer per unit
  for (int o = 32; o > 0; o >>= 1) n_moved += __shfl_xor(n_moved, o);
  __syncthreads();
  if ((tid & 63) == 0) wave_tot[tid >> 6] = n_moved;
  __syncthreads();
  if (tid == 0) {
    unsigned all = 0;
    for (int w = 0; w < kSelWaves; ++w) all += wave_tot[w];
    a.rows_moved[unit] += all;
  }
}

// Moves rows of K (blockIdx.y = 0) or V (1): row j <- row src_index[j], j < budget.
// Row parts are 256 bytes (16 lanes of 16 bytes; a whole row for bf16 with d = 128) or, for
// shorter rows and few units, 128 bytes.  A block of 1024 threads owns one part of every row of one unit and
// walks the rows in tiles of (1024 / LPP) * U; loads and stores are marked non-temporal (every
// byte is touched once: measured 14 % faster than plain ones); inside a tile every load
// completes before the first store (a destination row may be another thread's source row),
// and because sources never lie below their destinations and both grow with j, a tile's
// stores cannot touch what a later tile still has to read.  The loads of the next tile are requested before this tile
// is stored, so the block always has reads in flight.
template <int U, int LPP>                      // LPP lanes of 16 bytes per row part
__global__ __launch_bounds__(kMoveBlock) void evict_move_kernel(const EvictArgs a, int row_bytes) {
  constexpr int ROWS = kMoveBlock / LPP;       // rows per block load
  const int tid = threadIdx.x;
  const int part = blockIdx.x, unit = evict_unit_of(a, blockIdx.z);
  if (a.slots.prompt_len) {                        // only units whose eviction was due have a gather list
    const int seq = (unit % a.units_per_layer) / a.n_kv_heads;
    const int32_t P = a.slots.prompt_len[seq], tau = a.t - a.slots.t0[seq];
    if (P < 0 || tau < 1 || tau % a.window != 0 ||
        slot_n_old(P, tau, a.budget, a.window) + 1 <= a.budget)
      return;
  }
  char *slab = static_cast<char *>(blockIdx.y == 0 ? a.k_cache : a.v_cache) +
               static_cast<size_t>(unit) * a.capacity * row_bytes + part * (LPP * 16) + (tid % LPP) * 16;
  const int32_t *src_index = a.ws.src_index + static_cast<size_t>(unit) * a.capacity;

  // rows below the first evicted slot stay where they are: start at the tile that holds it
  int first = 0;
  while (first + ROWS * U < a.budget && src_index[first + ROWS * U - 1] == first + ROWS * U - 1)
    first += ROWS * U;

  typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
  struct Tile { u32x4_t v[U]; int src[U]; };
  auto load = [&](Tile &t, int tile) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tile + u * ROWS + tid / LPP;
      t.src[u] = j < a.budget ? src_index[j] : -1;
      t.v[u] = u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tile + u * ROWS + tid / LPP;
      if (t.src[u] >= 0 && t.src[u] != j)
        t.v[u] = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4_t *>(slab + static_cast<size_t>(t.src[u]) * row_bytes));
    }
  };
  // the tile's loads have landed in every thread (touching the values makes the compiler wait
  // for exactly those loads), then the barrier, then its stores
  auto store = [&](Tile &t, int tile) {
#pragma unroll
    for (int u = 0; u < U; ++u) __asm__ volatile("" : "+v"(t.v[u]));
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tile + u * ROWS + tid / LPP;
      if (t.src[u] >= 0 && t.src[u] != j)
        __builtin_nontemporal_store(t.v[u], reinterpret_cast<u32x4_t *>(slab + static_cast<size_t>(j) * row_bytes));
    }
  };

  Tile t0, t1;
  load(t0, first);
  for (int tile = first; tile < a.budget; tile += 2 * ROWS * U) {
    const bool more1 = tile + ROWS * U < a.budget;
    if (more1) load(t1, tile + ROWS * U);
    store(t0, tile);
    if (!more1) break;
    const bool more2 = tile + 2 * ROWS * U < a.budget;
    if (more2) load(t0, tile + 2 * ROWS * U);
    store(t1, tile + ROWS * U);
    if (!more2) break;
  }
}

}  // namespace

int evict_lds_candidates() { return kLdsCandidates; }
// Up to 3 entries per thread, and up to 5 from 32 units on.  One block applies all that is outstanding for its unit,
// a launch of its own spreads a unit over several: with more entries the chain of the one block takes longer than the
// launches it saves.  us for an eviction of 64 calls' tracking, launches of their own / in the selection: 4 units x
// 1064 22 / 19, x 2564 30 / 28, x 4264 36.7 / 39.6, x 5264 46 / 52, x 8064 65 / 75; 32 units x 2564 40.2 / 36.6, x
// 4264 57.0 / 55.2, x 5264 69.5 / 71.5, x 8064 89.5 / 94.3; 128 units x 4264 136 / 133, x 5264 164 / 166, x 8064 232
// / 236; 256 units x 8064 418 / 415.
// Of more units than the chip holds selection blocks at once (two per compute unit) the chain is what the launch waits
// for again and again: 512 units of 432 / 1152 / 2112 entries 55 / 52, 118 / 113, 221 / 214; 768 73.3 / 72.4, 167 /
// 162, 323 / 314; 1024 91.9 / 93.3, 216 / 211, 423 / 411; 2048 165 / 178, 402 / 410, 818 / 813; 3584 of 432 281 / 301.
bool evict_applies_tracking(int n, int units) {
  return (n <= 3 * kSelBlock || (n <= 5 * kSelBlock && units >= 32)) && units <= 512;
}

hipError_t launch_evict(const EvictArgs &a, hipStream_t stream, hipEvent_t *ev) {
  const int n_cand = a.n - a.window;
  if (n_cand <= a.budget - a.window || a.n > a.capacity) return hipErrorInvalidValue;
  if (a.units_per_layer < 1 || a.units % a.units_per_layer != 0 || a.units > 65535) return hipErrorInvalidValue;
  if (a.slots.prompt_len && (!a.slots.t0 || a.n_kv_heads < 1 || a.units_per_layer % a.n_kv_heads != 0))
    return hipErrorInvalidValue;
  if ((a.score_flags & 32) && a.units != a.units_per_layer) return hipErrorInvalidValue;
  if ((a.score_flags & 32) && (!a.logits || !a.stat || a.group < 1 || a.group > 8 || a.p_stride < a.n))
    return hipErrorInvalidValue;
  const size_t lds = static_cast<size_t>(n_cand) * sizeof(unsigned long long);
  if (n_cand > kLdsCandidates && !a.ws.sel_keys) return hipErrorInvalidValue;
  if (a.todo.on && (!evict_applies_tracking(a.n, a.units) || a.slots.prompt_len || !a.todo.bitlog || a.units / a.units_per_layer > kFlushLayers ||
                    a.todo.log_words < (a.n + 31) / 32 || a.todo.log_slots < 1 || a.todo.last_layer >= a.units / a.units_per_layer))
    return hipErrorInvalidValue;
  if (a.todo.on && a.todo.last_layer >= 0) {
    const TrackArgs &k = a.todo.last;
    if (!k.compact || k.units != a.units_per_layer || !k.logits || !k.stat || k.group > kHeadPad || (k.group == kHeadPad && !k.cand_index) ||
        k.n_old + 1 != a.n || !k.activation_counter ||
        static_cast<long long>(fused_part_cap(k.n_old, k.n_parts)) * k.n_parts > k.p_stride)
      return hipErrorInvalidValue;
  }
  int n_blocks = a.units;                          // one per unit, or only the due sequences' units
  if (a.n_due > 0) {
    if (!a.slots.prompt_len || a.n_due > 8) return hipErrorInvalidValue;
    for (int i = 0; i < a.n_due; ++i)
      if (a.due_seq[i] < 0 || a.due_seq[i] * a.n_kv_heads >= a.units_per_layer) return hipErrorInvalidValue;
    n_blocks = a.units / a.units_per_layer * a.n_due * a.n_kv_heads;
  }
  if (ev) (void)hipEventRecord(ev[0], stream);
  // as few entries per thread as hold the unit (an instance of 8 for all: 1056 entries 12.4 instead of 7.2 us, 2112
  // 13.0 instead of 10.0); beyond 8 and its 64 KB of keys the passes go over memory
#define LAZYEV_SELECT(R) \
  do { \
    if (a.todo.on) hipLaunchKernelGGL((evict_select_held_kernel<R, true>), dim3(n_blocks), dim3(kSelBlock), lds, stream, a); \
    else hipLaunchKernelGGL((evict_select_held_kernel<R, false>), dim3(n_blocks), dim3(kSelBlock), lds, stream, a); \
  } while (0)
  if (a.n <= 2 * kSelBlock) LAZYEV_SELECT(2);
  else if (a.n <= 3 * kSelBlock) LAZYEV_SELECT(3);
  else if (a.n <= 5 * kSelBlock) LAZYEV_SELECT(5);
  else if (a.n <= kLdsCandidates)                  // (nothing outstanding: evict_applies_tracking)
    hipLaunchKernelGGL((evict_select_held_kernel<8, false>), dim3(n_blocks), dim3(kSelBlock), lds, stream, a);
#undef LAZYEV_SELECT
  else if (n_cand <= kLdsCandidates)
    hipLaunchKernelGGL(evict_select_kernel<true>, dim3(n_blocks), dim3(kSelBlock), lds, stream, a);
  else
    hipLaunchKernelGGL(evict_select_kernel<false>, dim3(n_blocks), dim3(kSelBlock), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev) (void)hipEventRecord(ev[1], stream);
  const int row_bytes = a.head_dim * (a.dtype == 0 ? 4 : 2);
  // Parts of 256 bytes where their blocks come to three quarters of the chip's compute units, else parts of 128 bytes
  // and twice the blocks.  us, 256 / 128: 8 units x 4096 rows of 256 bytes 33.9 / 21.0, 48 x 1024 16.5 / 12.3, 64 x
  // 2048 28.7 / 24.9, 96 x 2048 (192 blocks) 43.0 / 41.8; 48 x 1024 rows of 512 bytes (192 blocks) 18.8 / 21.0.
  // (Parts of 64 bytes: 4 units x 144 2.4, as with 128; 32 x 1024 11.2 / 10.3.)
  if (row_bytes % 256 == 0 && 2 * n_blocks * (row_bytes / 256) >= 192) {
    hipLaunchKernelGGL((evict_move_kernel<8, 16>), dim3(row_bytes / 256, 2, n_blocks), dim3(kMoveBlock),
                       0, stream, a, row_bytes);
  } else {
    hipLaunchKernelGGL((evict_move_kernel<8, 8>), dim3(row_bytes / 128, 2, n_blocks), dim3(kMoveBlock),
                       0, stream, a, row_bytes);
  }
  e = hipGetLastError();
  if (ev) (void)hipEventRecord(ev[2], stream);
  return e;
}

hipError_t launch_init_state(int32_t *ts, int32_t *mri, int32_t *pos, int64_t n_units,
                             int32_t capacity, int32_t prompt_len, unsigned long long *rec, int32_t rec_units,
                             int32_t rec_stride, int32_t rec_words, hipStream_t stream) {
  if (rec_words > rec_stride || (rec_words > 0 && !rec)) return hipErrorInvalidValue;
  const int64_t total = n_units * capacity, words = static_cast<int64_t>(rec_units) * rec_words;
  const unsigned blocks = static_cast<unsigned>(((total > words ? total : words) + 255) / 256);
  hipLaunchKernelGGL(init_state_kernel, dim3(blocks), dim3(256), 0, stream, ts, mri, pos, total,
                     capacity, prompt_len, rec, rec_units, rec_stride, rec_words);
  return hipGetLastError();
}

hipError_t launch_mri_histogram(const int32_t *mri, int64_t n_units, int32_t capacity, int32_t n_kv_heads,
                                const int32_t *seq_len, int32_t n, int32_t n_bins, unsigned long long *hist,
                                hipStream_t stream) {
  if (n_units <= 0 || n <= 0) return hipSuccess;
  const int32_t spans = (n + kHistSpan - 1) / kHistSpan;
  if (n > capacity || n_bins < 2 || n_kv_heads < 1 || n_units * spans > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mri_histogram_kernel, dim3(static_cast<unsigned>(n_units * spans)), dim3(kHistBlock),
                     n_bins * sizeof(unsigned), stream, mri, capacity, n_kv_heads, seq_len, n, spans, n_bins, hist);
  return hipGetLastError();
}

hipError_t launch_init_slot(int32_t *ts, int32_t *mri, int32_t *pos, int32_t n_layers, int32_t batch,
                            int32_t n_kv_heads, int32_t capacity, int32_t seq, int32_t prompt_len,
                            int32_t *dev_prompt_len, int32_t *dev_t0, int32_t t0, hipStream_t stream) {
  if (seq < 0 || seq >= batch || prompt_len > capacity || !dev_prompt_len || !dev_t0)
    return hipErrorInvalidValue;
  // prompt_len < 0 empties the slot: only the timing record changes
  const int64_t total = prompt_len < 0 ? 1 : static_cast<int64_t>(n_layers) * n_kv_heads * capacity;
  const unsigned blocks = static_cast<unsigned>((total + 255) / 256);
  hipLaunchKernelGGL(init_slot_kernel, dim3(blocks), dim3(256), 0, stream, ts, mri, pos,
                     prompt_len < 0 ? 0 : n_layers, batch, n_kv_heads, capacity, seq, prompt_len,
                     dev_prompt_len, dev_t0, t0);
  return hipGetLastError();
}

hipError_t launch_score_pairs(const int32_t *dt, const int32_t *mri, double *score, int64_t n,
                              int32_t flags, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const unsigned blocks = static_cast<unsigned>((n + 255) / 256);
  hipLaunchKernelGGL(score_pairs_kernel, dim3(blocks), dim3(256), 0, stream, dt, mri, score, n,
                     flags);
  return hipGetLastError();
}

}  // namespace lazyev
