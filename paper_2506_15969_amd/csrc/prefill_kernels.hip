// Recurrence tracking over the prompt: the first loop of Alg. 1 and Eq. 1 of the
// paper applied to the prompt's own causal attention, so that prompt entries enter the
// decode phase with a TS / MRI history instead of TS = 0, MRI = 0.  Prompt position i (0-based,
// P positions) acts as the query of step tau_i = i + 1 - P over the keys 0..i; entry i is born
// with TS = tau_i, MRI = 0; decoding continues at step 1.
//
// Two kernels, both built on S^T = K Q^T tiles of 16 keys x 16 queries of ONE head
// (v_mfma_f32_16x16x32_bf16, or v_mfma_f32_16x16x4_f32 for fp32 rows); MFMA layouts (lane l, c = l % 16, g = l / 16)
//   16x16x32: A[row c][k = 8g..8g+7]  B[k = 8g..8g+7][col c]  C[row 4g+i][col c]
//   16x16x4:  A[row c][k = g]         B[k = g][col c]         C[row 4g+i][col c]
//   stats  the four waves of a block keep NB tiles of 16 queries each of one head in registers and walk the
//          key tiles 0..their own together, keeping every query's softmax sum relative to a
//          reference that is raised only when a weight would leave the range of fp32; leaves the
//          log-sum-exp of every (unit, head, position) in the workspace
//   track  the four waves of a block keep NB tiles of 16 keys each in registers and walk
//          the (query tile, head) pairs from the block's own position upwards together.  The
//          largest logarithm of the key's weight over the heads of the group decides (exp is monotone): one
//          maximum per logit and head, one compare with the logarithm of alpha per weight
//          after the group's last head.  The activations of each key are then applied in order
//          of the query position (one key per lane).
// The streamed tiles (keys in the first kernel, queries in the second) are fetched once per block,
// a stage of 4 KB (8 KB for fp32 rows of 128) at a time, and shared through LDS, one barrier per stage: fetched
// per wave, the second kernel read 7 GB per call past the L2 for 128 units x 2048 positions.  Four
// products per streamed tile and wave where that fills the chip (two: 1312 instead of 1190 us there, the operand
// reads from LDS are twice as many); short prompts and few units take one
// tile per wave.  The second kernel also cuts the queries into segments whose
// results (first and last activation, largest gap between) a third kernel joins, where its blocks are few.
// Blocks start in index order, so the heaviest tiles get the lowest indices.  No wave waits for another block.
//
// What bounds it: the vector work beside the products (a multiply-add, an exponential and an addition per weight
// in the first kernel, a maximum in the second; the matrix cores are busy 45 % of the time).  Measured, us for both
// kernels, before (a running maximum with two exponentials per weight, an exponential and a comparison per
// weight in the second kernel, rows of 64 and fp32 rows on a kernel without matrix instructions) and now, calls back to
// back (3 % from box to box; the other figures in this file are against 1190 - 1223 us for 2048 positions in their own runs):
//   32 sequences, 28 / 4 heads of 128, bf16   600 positions 292 -> 154, 2048 positions 1370 -> 1050
//   16 sequences, 40 / 8 heads of 128, bf16  4096 positions 3520 -> 2760
//    8 sequences, 28 / 4 heads of 128, bf16  1024 positions 350 -> 100
//    1 sequence,  28 / 4 heads of 128, bf16    33 positions 22.9 -> 10.4,  400 positions 141 -> 19.7
//    4 sequences, 32 / 8 heads of  64, bf16   499 positions 5470 -> 26
//    2 sequences, 28 / 4 heads of 128, fp32   300 positions 10880 -> 39
// (Of the first two 1158 -> 1050 and 2960 -> 2760 by loops without a way out of their middle, whose stages therefore waited for their own
// request, by masks and maxima in place instead of copies of 16 registers a stage, and by four waves per SIMD in the first kernel.
// The clock falls as the matrix cores get busier, 1.98 -> 1.87 GHz under the profiler: 16 % fewer cycles were 12 % of the time.)
#include "bits.h"
#include "kernels.h"

#include <cfloat>
#include <climits>
#include <type_traits>

namespace lazyev {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kHeadMax = 8;
// stages on their way from memory (one: 1250 instead of 1190 us for 128 units x 2048 positions; four: 1190)
constexpr int kAhead = 2;
typedef unsigned short bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;

template <typename T, int D>
struct Rows {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int kChunks = D * static_cast<int>(sizeof(T)) / 16;   // 16-byte chunks of a row
  static constexpr int kK = kChunks / 4;           // operand registers of 16 bytes per lane and tile
  static constexpr int kStage = kChunks == 8 ? 2 : 1;   // tiles per stage (4 KB; 8 KB for fp32 rows of 128)
  static constexpr int kSlots = kStage * 16 * kChunks;                   // 16-byte chunks of a stage
  static constexpr int kFetch = kSlots / kBlock;   // of them per thread
  // The weight of a key: exp2((q.k - r) c2 - ll) with a reference product r next to the log-sum-exp and what the
  // sum of the weights relative to it leaves, ll, kept apart, so that nothing is rounded at the magnitude of the
  // log-sum-exp; 128-element bf16 rows fold both into one number that the product starts
  // from, b = -(m + log2 l) / c2 (c2 = scale log2 e, m = r c2).
  static constexpr bool kApart = !(sizeof(T) == 2 && D == 128);
  static constexpr int kTiles = kK == 8 ? 2 : 4;   // tiles a wave keeps in registers where there is work for all
  // waves per SIMD the registers are held to: in the second kernel, and in the first (128 x bf16: 128 registers just
  // suffice for four; three 1086, four 1070 us for both kernels, 128 units x 2048 positions)
  static constexpr int waves(int nb) { return nb == 1 ? 4 : kF32 ? 2 : 3; }
  static constexpr int stats_waves(int nb) { return nb == 1 || !kF32 ? 4 : 2; }
};

// 16 rows at `rows` (row stride `stride` elements), rows clamped to `last`, as an MFMA A or B
// operand: lane (c, g) takes the 16-byte chunks 4 kk + g of row c.
template <typename T, int D>
__device__ __forceinline__ void load_operand(const T *rows, int first, int last, size_t stride, int c, int g,
                                             u32x4_t (&x)[Rows<T, D>::kK]) {
  const int r = min(first + c, last);
  const T *p = rows + static_cast<size_t>(r) * stride + g * (16 / sizeof(T));
#pragma unroll
  for (int kk = 0; kk < Rows<T, D>::kK; ++kk) x[kk] = *reinterpret_cast<const u32x4_t *>(p + kk * (64 / sizeof(T)));
}

// acc[n] += a tile x tile n for N tiles of which either the keys (kKeys) or the queries are the N and the
// other operand is one tile.  The N chains of dependent products go side by side.  (fp32 rows: four
// products per operand register; which columns of the row go together does not matter as long as both
// operands agree; two chains each, added at the end.)
template <typename T, int D, int N, bool kKeys>
__device__ __forceinline__ void logits_tiles(const u32x4_t (&many)[N][Rows<T, D>::kK], const u32x4_t (&one)[Rows<T, D>::kK],
                                             f32x4_t (&acc)[N]) {
  if constexpr (Rows<T, D>::kF32) {
    f32x4_t odd[N];
#pragma unroll
    for (int n = 0; n < N; ++n) odd[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < Rows<T, D>::kK; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < N; ++n) {
          const float x = __uint_as_float(kKeys ? many[n][kk][e] : one[kk][e]), y = __uint_as_float(kKeys ? one[kk][e] : many[n][kk][e]);
          f32x4_t &to = e % 2 ? odd[n] : acc[n];
          to = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, to, 0, 0, 0);
        }
#pragma unroll
    for (int n = 0; n < N; ++n) acc[n] += odd[n];
  } else {
#pragma unroll
    for (int kk = 0; kk < Rows<T, D>::kK; ++kk)
#pragma unroll
      for (int n = 0; n < N; ++n)
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kKeys ? many[n][kk] : one[kk]),
                                                         __builtin_bit_cast(bf16x8_t, kKeys ? one[kk] : many[n][kk]), acc[n], 0, 0, 0);
  }
}

// The streamed rows of a stage: thread t brings the 16-byte chunks t, t + 256, ... in row order (whole
// rows), the block keeps them in LDS, and every wave reads its MFMA operands from there.  Chunk x
// of row r sits at slot x ^ r of the row, so that the row-wise writes and the column-wise operand
// reads both spread over the banks.
template <typename T, int D>
struct SharedTile {
  u32x4_t slot[2][Rows<T, D>::kSlots];             // double-buffered
};
template <typename T, int D>
__device__ __forceinline__ void stage_put(SharedTile<T, D> &t, int buf, const u32x4_t (&v)[Rows<T, D>::kFetch]) {
  constexpr int C = Rows<T, D>::kChunks;
#pragma unroll
  for (int u = 0; u < Rows<T, D>::kFetch; ++u) {
    const int at = static_cast<int>(threadIdx.x) + u * kBlock, r = at / C, x = at % C;
    t.slot[buf][r * C + (x ^ (r % C))] = v[u];
  }
}
template <typename T, int D>
__device__ __forceinline__ void tile_operand(const SharedTile<T, D> &t, int buf, int j, u32x4_t (&x)[Rows<T, D>::kK], int c, int g) {
  constexpr int C = Rows<T, D>::kChunks;
#pragma unroll
  for (int kk = 0; kk < Rows<T, D>::kK; ++kk) x[kk] = t.slot[buf][(16 * j + c) * C + ((4 * kk + g) ^ ((16 * j + c) % C))];
}

// The operands a wave keeps have arrived before the loop starts.  The waits in the loop are then for its own
// stages alone, in the order of their requests: a load from before the loop, a path through it that
// leaves stages out, or a way out of its middle (from where the compiler sees a way to its top) would have the waits in it
// count to (nearly) zero, i.e. a stage wait for its own request.
template <int N, int K>
__device__ __forceinline__ void settle(u32x4_t (&x)[N][K]) {
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int k = 0; k < K; ++k) __asm__ volatile("" : "+v"(x[n][k]));
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kFar = 0x1p64f;                    // a sum of four weights beyond this raises the reference
// A reference is a rounded product, so up to a magnitude of 2^24 the exact product (a fused multiply-add) is within 1
// of it, and within the rounding of the logits at any.  Beyond, the difference could leave the range of exp2: then
// the product is rounded first, as the reference was.
constexpr float kHuge = 0x1p24f;
__device__ __forceinline__ float rounded_product(float x, float c2) {
  float s = x * c2;
  __asm__("" : "+v"(s));                           // (not fused with what follows)
  return s;
}

// (this file is compiled with -fno-honor-nans, so that a maximum is one instruction and not three that
// first make signalling NaNs quiet)
__device__ __forceinline__ float max_f32(float a, float b) { return __builtin_fmaxf(a, b); }

// One key tile against the wave's NB query tiles in the statistics kernel.  Logits are kept in units of log 2 (scaled
// by c2 = scale * log2(e)), so a weight is one multiply-add and one v_exp_f32.  Every lane sums ITS four key rows of
// every tile (the four lanes of a query column are merged once, at the end): no cross-lane traffic inside the loop.
// The reference m of a query need not be its maximum: a floating-point sum is as exact relative to any reference
// within the range of the exponent, so there is no running maximum, only a look whether the weights leave the range
// (first: there is no reference yet; where all logits of the first tile are -inf it is the lowest finite number, and
// the first other logit raises it).  limit: kFar, or, once some reference of the wave is beyond kHuge, a number that
// every sum exceeds.  mask: the tile may hold keys newer than a query or positions beyond the prompt.
template <typename T, int D, int NB, bool kFirst>
__device__ __forceinline__ void stats_tiles(bool mask, const u32x4_t (&ka)[Rows<T, D>::kK], const u32x4_t (&qb)[NB][Rows<T, D>::kK],
                                            float c2, int key0, int query0, int P, float (&r)[NB], float (&m)[NB], float (&l)[NB], float &limit) {
  f32x4_t acc[NB];
  float ps[NB], far = 0.f;
#pragma unroll
  for (int n = 0; n < NB; ++n) acc[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  logits_tiles<T, D, NB, false>(qb, ka, acc);
  if (mask) {                                      // (wave-uniform)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[n][i] = (key0 + i <= query0 + 16 * n && key0 + i < P) ? acc[n][i] : -INFINITY;
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    if (kFirst) {                                  // (key 0 is visible to every query, but to one of the column's four lanes only)
      float top = max_f32(max_f32(acc[n][0], acc[n][1]), max_f32(acc[n][2], acc[n][3]));
      top = max_f32(top, __shfl_xor(top, 16));
      top = max_f32(max_f32(top, __shfl_xor(top, 32)), -FLT_MAX);
      if (Rows<T, D>::kApart) r[n] = top;
      m[n] = max_f32(top * c2, -FLT_MAX);
    }
    auto weight = [&](int i) { return __builtin_amdgcn_exp2f(fmaf(acc[n][i], c2, -m[n])); };
    ps[n] = (weight(0) + weight(1)) + (weight(2) + weight(3));
    far = n == 0 ? ps[n] : max_f32(far, ps[n]);
  }
  if (kFirst || __builtin_expect(__builtin_amdgcn_ballot_w64(far > limit) != 0, 0)) {   // (wave-uniform)
    __asm__ volatile("");                          // (stays a branch: not worked out beforehand)
    float largest = 0.f;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (!kFirst) {
        const float top = max_f32(max_f32(acc[n][0], acc[n][1]), max_f32(acc[n][2], acc[n][3]));
        if (Rows<T, D>::kApart) r[n] = max_f32(r[n], top);
        const float up = max_f32(m[n], top * c2);
        l[n] *= __builtin_amdgcn_exp2f(m[n] - up);
        m[n] = up;
      }
      largest = max_f32(largest, fabsf(m[n]));
    }
    const bool huge = __builtin_amdgcn_ballot_w64(largest > kHuge) != 0;
    limit = huge ? -1.f : kFar;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (kFirst && !huge) continue;               // (as worked out above)
      auto weight = [&](int i) {
        return __builtin_amdgcn_exp2f(huge ? rounded_product(acc[n][i], c2) - m[n] : fmaf(acc[n][i], c2, -m[n]));
      };
      ps[n] = (weight(0) + weight(1)) + (weight(2) + weight(3));
    }
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) l[n] += ps[n];
}

// Softmax statistics of every (head, prompt position) of a unit:
// blocks = units * G * ceil(P / (64 NB)); the four waves of a block hold consecutive query
// spans of one head and walk the key tiles together.
template <typename T, int D, int NB>
__global__ __launch_bounds__(kBlock, (Rows<T, D>::stats_waves(NB))) void prefill_stats_kernel(const PrefillArgs a) {
  using R = Rows<T, D>;
  constexpr int kSpan = 16 * NB;
  __shared__ SharedTile<T, D> tile;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int P = a.prompt_len, G = a.group;
  const int n_qt = (P + kWaves * kSpan - 1) / (kWaves * kSpan);
  // Blocks start in index order and late query tiles carry more work than early ones: the
  // heaviest tiles get the lowest block indices (they start first, the light ones fill the
  // end), and consecutive blocks, which go to different XCDs, hold the same tile position of
  // different (unit, head) pairs, so every XCD gets every tile position equally often.  (All blocks of a unit on
  // one XCD, for its L2: 580 instead of 566 us for 128 units x 2048 positions.)
  const int n_uh = a.batch * a.n_kv_heads * G;
  const int qt = n_qt - 1 - static_cast<int>(blockIdx.x) / n_uh;
  const int uh = static_cast<int>(blockIdx.x) % n_uh;
  const int unit = uh / G, h = uh % G;
  const int i0 = (qt * kWaves + wave) * kSpan;     // this wave's queries: i0 .. i0 + kSpan - 1
  const bool have = i0 < P;                        // (a wave without queries still fetches and waits with the block)
  const int seq = unit / a.n_kv_heads, kvh = unit % a.n_kv_heads;
  const T *q = static_cast<const T *>(a.q_prompt) + (static_cast<size_t>(seq) * P * a.n_q_heads + kvh * G + h) * D;
  const T *kc = static_cast<const T *>(a.k_cache) + static_cast<size_t>(unit) * a.capacity * D;
  const float c2 = a.scale * kLog2e;
  u32x4_t qb[NB][R::kK];
#pragma unroll
  for (int n = 0; n < NB; ++n)
    load_operand<T, D>(q, i0 + 16 * n, P - 1, static_cast<size_t>(a.n_q_heads) * D, c, g, qb[n]);

  float r[NB], m[NB], l[NB];                       // of query i0 + 16 n + c, over this lane's key rows; m = r c2
#pragma unroll
  for (int n = 0; n < NB; ++n) { r[n] = 0.f; m[n] = 0.f; l[n] = 0.f; }
  float limit = kFar;
  const int my_last = have ? min(i0 + kSpan - 1, P - 1) >> 4 : -1;
  const int block_last = min(qt * kWaves * kSpan + kWaves * kSpan - 1, P - 1) >> 4;
  const int n_stages = block_last / R::kStage + 1;
  // the rows of a stage follow one another in the cache: thread t's chunks lie 16 t (+ 4096 u) bytes in
  auto fetch = [&](int st, u32x4_t (&v)[R::kFetch]) {
    const int left = P - 1 - st * (16 * R::kStage);  // last row of the stage that exists
    const T *base = kc + static_cast<size_t>(st) * (16 * R::kStage) * D;
#pragma unroll
    for (int u = 0; u < R::kFetch; ++u) {
      const int at = static_cast<int>(threadIdx.x) + u * kBlock;
      const unsigned off = static_cast<unsigned>(min(at / R::kChunks, left)) * R::kChunks + at % R::kChunks;
      v[u] = reinterpret_cast<const u32x4_t *>(base)[off];
    }
  };
  u32x4_t next[kAhead][R::kFetch];                 // stage s in next[s % kAhead]
  fetch(0, next[0]);
  stage_put<T, D>(tile, 0, next[0]);
#pragma unroll
  for (int x = 1; x <= kAhead; ++x) {
    fetch(min(x, n_stages - 1), next[x % kAhead]);
    __builtin_amdgcn_sched_barrier(0);             // (in this order: the waits in the loop count on it)
  }
  __syncthreads();
  // kFirst: stage 0.  The stage's number modulo kAhead is known to the code.
  auto stage = [&](int st, auto tag, auto first) {
    constexpr int buf = decltype(tag)::value % 2, reg = (decltype(tag)::value + 1) % kAhead;
#pragma unroll
    for (int j = 0; j < R::kStage; ++j) {
      const int jt = st * R::kStage + j;
      if (jt <= my_last) {                         // (wave-uniform)
        u32x4_t ka[R::kK];
        tile_operand<T, D>(tile, buf, j, ka, c, g);
        // only the wave's last NB key tiles can hold keys newer than a query (or positions beyond the prompt)
        const bool mask = jt * 16 + 15 > i0 || jt * 16 + 15 >= P;
        if (decltype(first)::value && j == 0)
          stats_tiles<T, D, NB, true>(true, ka, qb, c2, 4 * g, i0 + c, P, r, m, l, limit);
        else
          stats_tiles<T, D, NB, false>(mask, ka, qb, c2, jt * 16 + 4 * g, i0 + c, P, r, m, l, limit);
      }
    }
    stage_put<T, D>(tile, buf ^ 1, next[reg]);
    fetch(min(st + 1 + kAhead, n_stages - 1), next[reg]);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();                               // stage st + 1 is complete, stage st no longer read
  };
  settle(qb);
  stage(0, std::integral_constant<int, 0>{}, std::true_type{});
  int st = 1;
  for (; st + 1 < n_stages; st += kAhead) {        // (whole rounds: see settle)
    stage(st, std::integral_constant<int, 1>{}, std::false_type{});
    stage(st + 1, std::integral_constant<int, 0>{}, std::false_type{});
  }
  if (st < n_stages) stage(st, std::integral_constant<int, 1>{}, std::false_type{});
  if (!have) return;
  // the four lanes of a query column (g = 0..3) -> the column's reference and sum
#pragma unroll
  for (int n = 0; n < NB; ++n) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ro = __shfl_xor(r[n], o), mo = __shfl_xor(m[n], o), lo = __shfl_xor(l[n], o);
      const float mx = fmaxf(m[n], mo);
      l[n] = l[n] * __builtin_amdgcn_exp2f(m[n] - mx) + lo * __builtin_amdgcn_exp2f(mo - mx);
      r[n] = max_f32(r[n], ro);
      m[n] = mx;
    }
  }
  if (g == 0) {
    float *st = a.stat + (static_cast<size_t>(unit) * G + h) * a.p16;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int i = i0 + 16 * n + c;
      if (i >= P) continue;
      if constexpr (R::kApart) {
        // The reference moved next to the log-sum-exp, by the whole part of log2 l: near = r + step - lost, exactly
        // (the error of a sum, Knuth).  What m and step lost when they were rounded goes into ll (huge references: m was
        // that of rounded products).
        const float whole = floorf(__builtin_amdgcn_logf(l[n]));
        const float step = c2 > 1e-30f ? whole / c2 : 0.f, near = r[n] + step, part = near - r[n];   // (a finite step)
        const float lost = (r[n] - (near - part)) + (step - part);
        const float off = (limit < 0.f ? 0.f : fmaf(r[n], c2, -m[n])) + fmaf(step, c2, -whole) - lost * c2;
        st[i] = near;
        a.stat2[(static_cast<size_t>(unit) * G + h) * a.p16 + i] =
            __builtin_amdgcn_logf(l[n] * __builtin_amdgcn_exp2f(-whole)) - off;
      } else {                                     // b: see Rows
        st[i] = -(m[n] + __builtin_amdgcn_logf(l[n])) / c2;
      }
    }
  }
}

// Tracking: blocks = units * ceil(P / (64 NB)) * segments; a wave owns the keys j0 .. j0 + 16 NB - 1.
// kIO: the weights are exported and / or replaced (a checker's route).  kSeg: the block walks its segment of
// the queries only and leaves, of every key, its first (INT_MAX: none) and last activation there, the largest gap
// between two of them and their number, instead of TS / MRI.
template <typename T, int D, int NB, bool kIO, bool kSeg>
__global__ __launch_bounds__(kBlock, (Rows<T, D>::waves(NB))) void prefill_track_kernel(const PrefillArgs a) {
  using R = Rows<T, D>;
  constexpr int kSpan = 16 * NB;
  __shared__ SharedTile<T, D> tile;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int P = a.prompt_len, G = a.group;
  const int n_kt = (P + kWaves * kSpan - 1) / (kWaves * kSpan);
  // early keys carry more work: heaviest first, as in the first kernel
  const int units = a.batch * a.n_kv_heads;
  const int unit = static_cast<int>(blockIdx.x) % units, kz = static_cast<int>(blockIdx.x) / units;
  const int kt = kSeg ? kz / a.segments : kz, z = kSeg ? kz % a.segments : 0;
  const int j0 = (kt * kWaves + wave) * kSpan;
  const bool have = j0 < P;                        // (a wave without keys still fetches and waits with the block)
  const int seq = unit / a.n_kv_heads, kvh = unit % a.n_kv_heads;
  const T *q = static_cast<const T *>(a.q_prompt) + (static_cast<size_t>(seq) * P * a.n_q_heads + kvh * G) * D;
  const T *kc = static_cast<const T *>(a.k_cache) + static_cast<size_t>(unit) * a.capacity * D;
  const float *stat = a.stat + static_cast<size_t>(unit) * G * a.p16;
  const float *stat2 = R::kApart ? a.stat2 + static_cast<size_t>(unit) * G * a.p16 : nullptr;
  const float c2 = a.scale * kLog2e;
  u32x4_t ka[NB][R::kK];
#pragma unroll
  for (int n = 0; n < NB; ++n) load_operand<T, D>(kc, j0 + 16 * n, P - 1, D, c, g, ka[n]);

  // lane (c, g), c < 4 NB, carries the state of key row 4 g + (c & 3) of key tile c >> 2
  const int my_key = j0 + 16 * (c >> 2) + 4 * g + (c & 3);
  int32_t ts = kSeg ? INT_MIN : my_key + 1 - P, mri = 0, first = INT_MAX;
  unsigned n_act = 0;
  // this block's query tiles, and in them the (query tile, head) pairs in order, the same for the four waves of the
  // block (a wave skips the query tiles before its own keys); the query tiles of a stage are fetched
  // once per block, the next stage's travel during the arithmetic of the current one
  const int n_it = (P + 15) >> 4, it_first = (kt * kWaves * kSpan) >> 4;      // (the block's oldest key tile)
  const int it_begin = kSeg ? max(it_first, z * a.seg_tiles) : it_first;
  const int it_end = kSeg ? min(n_it, (z + 1) * a.seg_tiles) : n_it;
  if (kSeg && it_begin >= it_end) return;          // (no query of the segment sees these keys; nobody reads a record of it)
  const int my_first = j0 >> 4;
  const int plain_first = (j0 + kSpan - 1 + 15) >> 4, plain_end = j0 + kSpan - 1 < P ? P >> 4 : 0;
  const size_t q_stride = static_cast<size_t>(a.n_q_heads) * D;
  // A place in the sequence of pairs: 16 queries from it * 16 on of head h, the first of their rows, where
  // their statistics lie, and the pairs behind it.  It stays on the block's last pair.
  struct Place { int it, h; const T *rows; int stat_at, left; };
  const int stat_wrap = 16 - (G - 1) * a.p16;
  const ptrdiff_t rows_wrap = static_cast<ptrdiff_t>(16 * q_stride) - (G - 1) * D;
  auto next_pair = [&](Place &x) {
    if (x.left == 0) return;                       // (uniform)
    const bool wrap = x.h + 1 == G;
    x.left -= 1;
    x.rows += wrap ? rows_wrap : D;
    x.stat_at += wrap ? stat_wrap : a.p16;
    x.it += wrap ? 1 : 0;
    x.h = wrap ? 0 : x.h + 1;
  };
  // this thread's chunks of a tile's rows as byte offsets (16 rows of all heads are under 4 GB): rows beyond the
  // prompt, in its last tile, are replaced by the last one
  const int t_row = static_cast<int>(threadIdx.x) & (R::kStage == 2 ? kBlock / 2 - 1 : kBlock - 1);
  unsigned row_off[R::kFetch], row_off_end[R::kFetch];
#pragma unroll
  for (int u = 0; u < R::kFetch; ++u) {
    const int at = t_row + u * kBlock, r = at / R::kChunks;
    row_off[u] = static_cast<unsigned>(r * q_stride * sizeof(T)) + at % R::kChunks * 16;
    row_off_end[u] = static_cast<unsigned>(min(r, (P - 1) & 15) * q_stride * sizeof(T)) + at % R::kChunks * 16;
  }
  // rows of the stage whose first pair is at x
  auto fetch_rows = [&](Place x, u32x4_t (&v)[R::kFetch]) {
    if (R::kStage == 2) {                          // (two tiles per load: waves 2 and 3 bring the second)
      Place y = x;
      next_pair(y);
      x.it = wave >= kWaves / 2 ? y.it : x.it;
      x.rows = wave >= kWaves / 2 ? y.rows : x.rows;
    }
    const bool end = x.it == n_it - 1;
#pragma unroll
    for (int u = 0; u < R::kFetch; ++u)
      v[u] = *reinterpret_cast<const u32x4_t *>(reinterpret_cast<const char *>(x.rows) + (end ? row_off_end[u] : row_off[u]));
  };
  // ... and the statistics of this lane's queries in it (p16 covers the last tile)
  struct Stats { float b[R::kStage], ll[R::kStage]; };
  auto fetch_stats = [&](Place x, Stats &s) {
#pragma unroll
    for (int j = 0; j < R::kStage; ++j) {
      auto of_lane = [&](const float *p) { return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p + x.stat_at) + 4u * c); };
      s.b[j] = of_lane(stat);
      s.ll[j] = R::kApart ? of_lane(stat2) : 0.f;
      next_pair(x);
    }
  };
  auto advance = [&](int &it, int &h) {
    if (++h == G) { h = 0; ++it; }
  };
  auto weight = [&](float lw) { return __builtin_amdgcn_exp2f(R::kApart ? lw : lw * c2); };
  // The logarithm from which on the weight is >= alpha, so that the test is one comparison and no exponential:
  // the first float x with weight(x) >= alpha (alphas below the normal range count as the smallest normal number, like
  // the weights there).  It lies within a few floats of the logarithm of alpha, but for alphas close to 1: there
  // hundreds of floats x have one weight, at 1 some hundred million.  64 floats around the logarithm are tried
  // at once; if it is not among them, all floats are searched in their order, u = 0 .. 2^32 - 1, 64 places at a time
  // (weight never falls from a float to the next: v_exp_f32 tried on all of them).
  // alpha = 0: every key that is no newer (amax is -inf where none was seen).
  float reach = -FLT_MAX;
  if (a.alpha > 0.f) {
    const float alpha = max_f32(a.alpha, 0x1p-126f);
    auto float_at = [](unsigned u) {             // (from -FLT_MAX to +inf, the ends repeated)
      u = min(max(u, 0x00800000u), 0xFF800000u);
      return __uint_as_float((u >> 31) ? u ^ 0x80000000u : ~u);
    };
    auto under = [&](unsigned u, int shift) {    // the lanes whose place has a weight < alpha
      return __builtin_amdgcn_ballot_w64(weight(float_at(u + (static_cast<unsigned>(lane) << shift))) < alpha);
    };
    const unsigned guess = __float_as_uint(__builtin_amdgcn_logf(alpha) / (R::kApart ? 1.f : c2));
    unsigned below = ((guess >> 31) ? ~guess : guess ^ 0x80000000u) - 32u;
    unsigned long long m = under(below, 0);
    if ((m & 1) == 0 || (m >> 63) != 0) {        // (wave-uniform)
      below = 0;
      m = 1;
#pragma unroll 1
      for (int s = 26; s >= -4; s -= 6) {
        const int shift = max(s, 0);
        m = under(below, shift);
        below += static_cast<unsigned>(__popcll(m) - 1) << shift;
      }
      m = 1;
    }
    reach = float_at(below + static_cast<unsigned>(__popcll(m)));
  }
  // amax[4 n + i]: largest logarithm of a weight over the heads seen so far of the current query tile, for key
  // row 4 g + i of key tile n and query column c (-inf: the key is newer than the query)
  float amax[4 * NB];
#pragma unroll
  for (int x = 0; x < 4 * NB; ++x) amax[x] = -INFINITY;
  unsigned over = 0;                               // kIO with injected weights: bit 4 n + i = some head's weight >= alpha
  {
    int it = it_begin, h = 0;                      // the pair worked on
    // the block's stage s: rows in next[s % kAhead] until they are in LDS, statistics in bs[s % kAhead] until used
    u32x4_t next[kAhead][R::kFetch];
    Stats bs[kAhead];
    Place to_come = {it_begin, 0, q + static_cast<size_t>(it_begin) * 16 * q_stride, it_begin * 16, (it_end - it_begin) * G - 1};   // first pair of the next stage to request
    Place before = to_come;                        // ... and of the one before it, whose statistics are requested now
    auto more_rows = [&](u32x4_t (&to)[R::kFetch]) {
      fetch_rows(to_come, to);
      before = to_come;
#pragma unroll
      for (int j = 0; j < R::kStage; ++j) next_pair(to_come);
    };
    auto more_stats = [&](Stats &to) { fetch_stats(before, to); };
    more_rows(next[0]);
    stage_put<T, D>(tile, 0, next[0]);
#pragma unroll
    for (int x = 0; x < kAhead; ++x) {             // (in this order: the waits in the loop count on it)
      more_stats(bs[x]);
      more_rows(next[(x + 1) % kAhead]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    auto stage = [&](auto tag) {                   // (its number modulo kAhead is known to the code)
      constexpr int buf = decltype(tag)::value % 2, reg = (decltype(tag)::value + 1) % kAhead;
#pragma unroll
      for (int j = 0; j < R::kStage; ++j) {
        if (it < it_end && have && it >= my_first) {
          const int qi = it * 16 + c;              // this lane's query column
          const float b = bs[decltype(tag)::value].b[j], ll = bs[decltype(tag)::value].ll[j];
          u32x4_t qb[R::kK];
          tile_operand<T, D>(tile, buf, j, qb, c, g);
          const float start = R::kApart ? 0.f : b;
          f32x4_t acc[NB];
#pragma unroll
          for (int n = 0; n < NB; ++n) acc[n] = f32x4_t{start, start, start, start};
          logits_tiles<T, D, NB, true>(ka, qb, acc);
          // the logarithm of the weight, in units of log 2 (over c2 where b is folded in)
          auto log_weight = [&](float x) { return R::kApart ? fmaf(x - b, c2, -ll) : x; };
          // every key of the wave exists and is no newer than any query of the tile, and every
          // query of the tile exists: nothing to mask (all but the wave's first NB query tiles,
          // the prompt's last tile and its last wave)
          const bool plain = !kIO && it >= plain_first && it < plain_end;
          if constexpr (R::kApart) {
            if (plain) {
#pragma unroll
              for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) amax[4 * n + i] = max_f32(amax[4 * n + i], log_weight(acc[n][i]));
            } else {
#pragma unroll
              for (int n = 0; n < NB; ++n) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const int key = j0 + 16 * n + 4 * g + i;
                  const bool seen = key <= qi && qi < P;   // (key <= qi < P implies key < P)
                  const float lw = log_weight(acc[n][i]);
                  if (seen) amax[4 * n + i] = max_f32(amax[4 * n + i], lw);
                  if (kIO) {
                    if (seen) {
                      const size_t at = ((static_cast<size_t>(seq) * a.n_q_heads + kvh * G + h) * P + qi) * P + key;
                      if (a.p_out) a.p_out[at] = weight(lw);
                      if (a.p_override && a.p_override[at] >= a.alpha) over |= 1u << (4 * n + i);
                    }
                  }
                }
              }
            }
          } else {
            // (masked in place and then one maximum for both: with a maximum on either way the 16 of them are copied
            // around every stage, 1105 instead of 1040 us for 128 units x 2048 positions; with the products'
            // differences above it is the other way, 31.8 / 30.6)
            float lw[4 * NB];
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
              for (int i = 0; i < 4; ++i) lw[4 * n + i] = log_weight(acc[n][i]);
            if (!plain) {
#pragma unroll
              for (int n = 0; n < NB; ++n) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const int key = j0 + 16 * n + 4 * g + i;
                  const bool seen = key <= qi && qi < P;   // (key <= qi < P implies key < P)
                  if (kIO) {
                    if (seen) {
                      const size_t at = ((static_cast<size_t>(seq) * a.n_q_heads + kvh * G + h) * P + qi) * P + key;
                      if (a.p_out) a.p_out[at] = weight(lw[4 * n + i]);
                      if (a.p_override && a.p_override[at] >= a.alpha) over |= 1u << (4 * n + i);
                    }
                  }
                  lw[4 * n + i] = seen ? lw[4 * n + i] : -INFINITY;
                }
              }
            }
#pragma unroll
            for (int x = 0; x < 4 * NB; ++x) amax[x] = max_f32(amax[x], lw[x]);
          }
          if (h == G - 1) {                        // the tile's last head: apply its activations
            // bit 4 n + i of this lane: key row 4 g + i of key tile n and query column c; after the transposition
            // bit q of lane (c, g): the key row and tile with 4 n + i = c, query q
            unsigned bits = 0;
#pragma unroll
            for (int x = 4 * NB - 1; x >= 0; --x) {
              const bool on = (kIO && a.p_override) ? (over >> x) & 1u : amax[x] >= reach;   // weight(amax[x]) >= alpha
              bits = bits + bits + (on ? 1u : 0u);
              amax[x] = -INFINITY;
            }
            over = 0;
            if (__builtin_amdgcn_ballot_w64(bits != 0) != 0) {   // (wave-uniform)
              const unsigned mask = transpose_bits<16>(bits, c);
              n_act += __popc(mask);
              if (mask != 0) {                     // in order of the query position (Alg. 1, Eq. 1)
                const int lo = __builtin_ctz(mask), hi = 31 - __builtin_clz(mask);
                const int32_t tau = it * 16 + 1 - P;
                if (kSeg && ts == INT_MIN) first = tau + lo;
                else mri = max(mri, tau + lo - ts);
                if (hi > lo) mri = max(mri, longest_gap<16>(mask, lo, hi));
                ts = tau + hi;
              }
            }
          }
        }
        advance(it, h);
      }
      stage_put<T, D>(tile, buf ^ 1, next[reg]);
      more_stats(bs[decltype(tag)::value]);
      more_rows(next[reg]);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();                             // the next stage is complete, this one no longer read
    };
    settle(ka);
    // Whole rounds (see settle); a stage too many works on nothing.  Narrow blocks of 128-byte rows end in the middle
    // of one: their stages are two tiles each and few (us, whole rounds / this, 64 x bf16, 28 / 4 heads x 20 / 33 /
    // 100 positions 11.0 / 10.8, 13.5 / 13.2, 17.6 / 17.4; 16 sequences x 20 / 33 11.5 / 11.3, 14.0 / 13.7; the same
    // from 180 positions on).
    do {
      stage(std::integral_constant<int, 0>{});
      if (NB == 1 && R::kStage == 2 && it >= it_end) break;
      stage(std::integral_constant<int, 1>{});
    } while (it < it_end);
  }
  if (!have) return;
  const bool owner = c < 4 * NB && my_key < P;
  if constexpr (kSeg) {
    if (owner)
      a.seg[(static_cast<size_t>(z) * units + unit) * P + my_key] = make_int4(first, ts, mri, static_cast<int32_t>(n_act));
    return;
  }
  if (owner) {
    a.ts[static_cast<size_t>(unit) * a.capacity + my_key] = ts;
    a.mri[static_cast<size_t>(unit) * a.capacity + my_key] = mri;
  }
  if (a.activation_counter) {
    for (int o = 32; o > 0; o >>= 1) n_act += __shfl_xor(n_act, o);
    if (lane == 0 && n_act) atomicAdd(a.activation_counter + unit * a.counter_stride, static_cast<unsigned long long>(n_act));
  }
}

// The segments of every key joined in order (Eq. 1): between two segments lies the gap from the last activation
// before to the first one in it.  What bounds it is the chain of its loads: the records of kJoin segments are
// requested together (4 sequences, 32 / 8 heads of 64 x 499 positions, all three kernels: one after the other 29.5 us, 27.1 now).
constexpr int kJoin = 8;
__global__ __launch_bounds__(kBlock) void prefill_join_kernel(const PrefillArgs a) {
  const int units = a.batch * a.n_kv_heads, P = a.prompt_len;
  const int spans = (P + kBlock - 1) / kBlock;
  const int unit = static_cast<int>(blockIdx.x) / spans, key = static_cast<int>(blockIdx.x) % spans * kBlock + threadIdx.x;
  unsigned n_act = 0;
  if (key < P) {
    int32_t ts = key + 1 - P, mri = 0;             // born at its own step
    // (the first segment that a block of its wave's keys worked on)
    for (int z0 = key / a.seg_block * (a.seg_block / 16) / a.seg_tiles; z0 < a.segments; z0 += kJoin) {
      int4 s[kJoin];
#pragma unroll
      for (int j = 0; j < kJoin; ++j)              // (beyond the last segment: that one once more)
        s[j] = a.seg[(static_cast<size_t>(min(z0 + j, a.segments - 1)) * units + unit) * P + key];
#pragma unroll
      for (int j = 0; j < kJoin; ++j) {
        if (z0 + j >= a.segments || s[j].x == INT_MAX) continue;
        mri = max(mri, max(s[j].x - ts, s[j].z));
        ts = s[j].y;
        n_act += static_cast<unsigned>(s[j].w);
      }
    }
    a.ts[static_cast<size_t>(unit) * a.capacity + key] = ts;
    a.mri[static_cast<size_t>(unit) * a.capacity + key] = mri;
  }
  if (a.activation_counter) {
    for (int o = 32; o > 0; o >>= 1) n_act += __shfl_xor(n_act, o);
    if ((threadIdx.x & 63) == 0 && n_act) atomicAdd(a.activation_counter + unit * a.counter_stride, static_cast<unsigned long long>(n_act));
  }
}

template <typename T, int D>
hipError_t launch_rows(PrefillArgs a, hipStream_t stream) {
  constexpr int NB = Rows<T, D>::kTiles;
  const long long units = static_cast<long long>(a.batch) * a.n_kv_heads;
  const long long wide = (a.prompt_len + kWaves * 16 * NB - 1) / (kWaves * 16 * NB), narrow = (a.prompt_len + kWaves * 16 - 1) / (kWaves * 16);
  if (units * a.group * narrow > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  // Wide blocks where there are eight per compute unit; with fewer the last of them leave more of the chip idle than their
  // products save (us for the three kernels, narrow from 512 / 2048 wide blocks down: 28 / 4 heads of 128 x bf16, 8
  // sequences x 600 positions 55.6 / 48.4, 2 x 2600 185 / 169, 32 x 60 19.0 / 16.1; 8 of 32 / 8 heads of 64 x 300 29.2 / 23.2;
  // from 4096 down: 32 x 600 154 / 203).  128 x bf16 already where the narrow ones are sixteen per compute unit: wide / narrow, 4
  // heads to a KV head, 64 units x 1500 193 / 237 (6144 narrow blocks), 128 x 600 95.8 / 108 (5120), 32 x 2000 174 / 181 (4096); 42 x
  // 1300 of 7 heads 128 / 121 (3528); the other types gain from narrow ones up to there (64 x bf16 x 1500 181 / 182, 600 84 / 75).
  constexpr bool kProductsLong = D == 128 && sizeof(T) == 2;
  if (units * a.group * wide >= 2048 || (kProductsLong && units * a.group * narrow >= 4096))
    hipLaunchKernelGGL((prefill_stats_kernel<T, D, NB>), dim3(static_cast<unsigned>(units * a.group * wide)), dim3(kBlock), 0, stream, a);
  else
    hipLaunchKernelGGL((prefill_stats_kernel<T, D, 1>), dim3(static_cast<unsigned>(units * a.group * narrow)), dim3(kBlock), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.p_out || a.p_override) {
    hipLaunchKernelGGL((prefill_track_kernel<T, D, 1, true, false>), dim3(static_cast<unsigned>(units * narrow)), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
  }
  // Blocks of four waves with NB key tiles each, or with one each where that does not fill the chip.  The
  // queries are cut into segments where the blocks are fewer than eight per compute unit:
  // early keys have all queries to walk, one after the other, and with one block for that the chip ends
  // on the few blocks of the earliest keys.  One segment / cut, us for both kernels: 32 units x 1024 positions
  // 267 / 112, 8 units x 8192 2129 / 1146, 128 units x 600 230 / 169; from 2048 blocks on nothing is gained
  // (128 units x 4096, 4096 blocks asked for instead: 2966 / 2900).  A segment is a query tile at
  // least (wide: two): what a block walks one after the other costs more than the records of more segments.  us for the
  // three kernels, 512 narrow blocks of two query tiles and wide ones of four / like this: 28 / 4 heads of 128 x bf16 x 33
  // positions 12.7 / 10.4, x 164 16.4 / 13.0, 2 sequences x 1500 102 / 74, x 2600 258 / 184, 16 x 250 37.9 / 30.1, 8 x 600 59.7 /
  // 55.4; 4 sequences of 32 / 8 heads of 64 x bf16 x 499 27.7 / 26.0; fp32 rows of 128, 2 x 300 46.0 / 39.5.
  // Where narrow blocks have fewer than 32 tiles of queries to walk, over all heads (fp32 rows: 16), 1024 of them (1024 / 2048, one head to a KV
  // head: 128 x bf16, 32 units x 250 14.5 / 16.0, 192 x 164 15.6 / 17.0; 64 x bf16, 64 x 164 13.1 / 14.5; but 8 units x 2600 71.3 / 66.6, three heads
  // 111 / 95.9; 48 of fp32 (128) x 250, three heads 47.0 / 43.8, 96 x 100, four heads 33.6 / 31.7).  Likewise segments of four tiles at least for wide
  // blocks below 40 tiles (four / two, one head: 128 x bf16, 96 units x 400 24.4 / 28.2, 64 x bf16 21.1 / 25.2, 64 x fp32, 48 x 400 34.4 /
  // 36.5; but four heads, 48 x 400 32.7 / 29.4; fp32 rows of 128, one head, 48 x 300 38.7 / 35.6).
  // Up to three query tiles are cut only where what is walked costs more than the third launch, which one segment does
  // without: 32 units, one segment / cut, 128 x bf16 x 33 1 / 2 / 4 / 7 heads 7.8 / 9.4, 8.6 / 9.4, 10.2 / 9.8, 13.5 / 11.6; x 20 7 heads equal;
  // fp32 (64) x 33 1 / 2 / 4 heads 9.2 / 10.2, equal, 12.7 / 10.9; with 256 blocks of one segment 12.0 / 13.0 (128 x bf16 x 33, 4 heads).
  // Wide blocks where 512 of them would have four query tiles each (a.segments: what the workspace holds records for): from
  // 512 of two tiles on, narrow / wide instead, 24 units of 128 x bf16 x 400 21.3 / 25.7, 12 of 128 x fp32 x 400 45.2 / 57.6, 24 of 64 x
  // fp32 x 400 39.9 / 54.8 (96 of 64 x bf16 x 250 25.6 / 22.7).
  const long long n_it = (a.prompt_len + 15) / 16;
  const long long most = n_it / 4 < a.segments ? n_it / 4 : a.segments;
  const bool use_wide = units * wide * (most < 1 ? 1 : most) >= 512;
  const long long per_unit = use_wide ? wide : narrow, want = use_wide || a.group * n_it >= (sizeof(T) == 4 ? 16 : 32) ? 2048 : 1024;
  long long z = (want + units * per_unit - 1) / (units * per_unit);
  const long long least = !use_wide ? 1 : a.group * n_it < 40 && !(sizeof(T) == 4 && D == 128) ? 4 : 2;    // query tiles of a segment
  if (z > n_it / least) z = n_it / least;
  if (n_it <= 3 && a.group * (n_it - 1) < (sizeof(T) == 4 ? 4 : 8) * (units * per_unit > 128 ? 2 : 1)) z = 1;
  if (z > a.segments) z = a.segments;
  if (z <= 1) {
    const dim3 grid(static_cast<unsigned>(units * per_unit));
    if (use_wide) hipLaunchKernelGGL((prefill_track_kernel<T, D, NB, false, false>), grid, dim3(kBlock), 0, stream, a);
    else hipLaunchKernelGGL((prefill_track_kernel<T, D, 1, false, false>), grid, dim3(kBlock), 0, stream, a);
    return hipGetLastError();
  }
  a.seg_tiles = static_cast<int32_t>((n_it + z - 1) / z);
  z = (n_it + a.seg_tiles - 1) / a.seg_tiles;
  a.seg_block = kWaves * 16 * (use_wide ? NB : 1);
  a.segments = static_cast<int32_t>(z);
  if (units * per_unit * z > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(units * per_unit * z));
  if (use_wide) hipLaunchKernelGGL((prefill_track_kernel<T, D, NB, false, true>), grid, dim3(kBlock), 0, stream, a);
  else hipLaunchKernelGGL((prefill_track_kernel<T, D, 1, false, true>), grid, dim3(kBlock), 0, stream, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long spans = (a.prompt_len + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(prefill_join_kernel, dim3(static_cast<unsigned>(units * spans)), dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_track(const PrefillArgs &a, hipStream_t stream) {
  if (a.prompt_len < 1 || a.prompt_len > a.capacity || a.group < 1 || a.group > kHeadMax ||
      a.n_q_heads != a.n_kv_heads * a.group || a.batch < 1 || a.p16 < (a.prompt_len + 15) / 16 * 16 ||
      !a.q_prompt || !a.k_cache || !a.ts || !a.mri || !a.stat || (!a.stat2 && !(a.dtype == 1 && a.head_dim == 128)) ||
      a.counter_stride < 1 ||
      (a.segments > 1 && !a.seg))
    return hipErrorInvalidValue;
  if (a.dtype == 0 && a.head_dim == 64) return launch_rows<float, 64>(a, stream);
  if (a.dtype == 0 && a.head_dim == 128) return launch_rows<float, 128>(a, stream);
  if (a.dtype == 1 && a.head_dim == 64) return launch_rows<bf16_t, 64>(a, stream);
  if (a.dtype == 1 && a.head_dim == 128) return launch_rows<bf16_t, 128>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace lazyev
