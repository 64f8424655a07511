// Indexer stage: page scores (Sec. 3.1 Eq. 2; Sec. 3.2 Quest) and the selection of sink,
// local and top-scoring pages (Sec. 3.1 Eq. 3; Sec. 6.4 setup).
//
// score_kernel   HBM-bound stream over the summaries, on a persistent grid: balanced
//                contiguous ranges of the batch's page references per workgroup (Appendix C
//                template).  A row of 16 lanes owns one (page, KV head) item.  Each lane
//                holds D/16 channels of the summary and of the query view.  Products
//                accumulate in fp64 and reduce across the row with DPP, then round once to
//                fp32.  Output goes to a scratch table scores[h][i][j] (rows padded to 4).
// topk_bucket_kernel  One workgroup per (request, KV head): the exact selection from scores or from
//                bounds with re-scoring of the pages they leave undecided, by one histogram of
//                equal-width bins; topk_wave_kernel does it in one wave for short requests.
// topk_radix_kernel  The options' radix selection on the same page slots.
// topk_long_kernel  (request bounds past the slots of both) One workgroup per (request, KV head).
//                Rows that fit page slots take the radix selection above; longer ones run the same
//                exact radix select over
//                an order-preserving uint32 key of the fp32 score.  Passes start at the
//                highest bit where the candidates' smallest and largest keys differ and take
//                up to 8 bits each.  Each pass builds a double-buffered LDS histogram, and
//                one wave scans its bins.  Each pass re-reads the scores from memory.  That finds
//                the K_free-th best candidate.
//                Ties at the threshold go to the lowest page index.  Each thread owns a
//                contiguous page range: one block scan ranks the tied pages and a second
//                compacts the forced and chosen pages in ascending order.
#include "summary_task.h"
#include "vx_device.h"
#include "vx_internal.h"

#include <algorithm>

namespace vx {
namespace {

constexpr int kThreads = 256;
constexpr int kRows = kThreads / 16;     // 16-lane rows per workgroup

// Score kinds.  The first three are the ABI's 0..2; kMeanBound is the first pass of the exact
// two-pass block-mean selection (bf16 means give an approximate score and a rigorous bound);
// the envelope flows of the agent-proposed algorithms (Appendix G) are the ABI's 3..5:
//   kQuestConsensus  min over heads of sum_c max(q Max, q Min)   (head-consensus Quest)
//   kEnvLower        max over heads of sum_c min(q Max, q Min)   (pessimistic envelope)
//   kQuestRectified  max over heads of sum_c ReLU(q Max)         (rectified Quest)
// kHeadDot is the first step of the NSA flow, one logit q_r . Mean per query head (its own kernel,
// head_score_kernel).
// kQuestBound .. kRectifiedBound are the first passes of the exact two-pass selection for the
// four envelope kinds: fp32 sums of the exact products with a rigorous bound, an interval that
// holds the one-pass score.
enum { kMeanDot = 0, kQuest = 1, kMaxDot = 2, kMeanBound = 3, kQuestConsensus = 4, kEnvLower = 5,
       kQuestRectified = 6, kHeadDot = 7, kQuestBound = 8, kConsensusBound = 9, kEnvLowerBound = 10,
       kRectifiedBound = 11 };
constexpr int kNoRescore = -1;           // two-pass re-scoring kind of a one-pass selection
// ABI kinds beyond the first six: the block mean over the content channels (scored by kMeanDot
// with the other query channels zero), NSA (kHeadDot, then the flow kernel) and positional
// smoothing (kMeanDot, then the flow kernel).
constexpr int kAbiContent = 6, kAbiNsa = 7, kAbiSmooth = 8;
// Envelope kinds (a per-head Max/Min envelope), those that read Min too, and those that read q
// per head (staged as fp32 in row order) instead of the group mean.
constexpr bool is_env(int k) { return k == kQuest || k == kQuestConsensus || k == kEnvLower || k == kQuestRectified; }
constexpr bool is_env_bound(int k) { return k >= kQuestBound && k <= kRectifiedBound; }
// envelope kind of a bound kind, and the bound kind of an envelope kind
constexpr int env_of_bound(int k) {
  return k == kQuestBound ? kQuest : k == kConsensusBound ? kQuestConsensus : k == kEnvLowerBound ? kEnvLower
                                                                                                 : kQuestRectified;
}
constexpr int bound_of_env(int k) {
  return k == kQuest ? kQuestBound : k == kQuestConsensus ? kConsensusBound : k == kEnvLower ? kEnvLowerBound
                                                                                             : kRectifiedBound;
}
constexpr bool needs_min(int k) {
  return k == kQuest || k == kQuestConsensus || k == kEnvLower || k == kQuestBound || k == kConsensusBound ||
         k == kEnvLowerBound;
}
constexpr bool per_head(int k) { return is_env(k) || is_env_bound(k); }
// Kinds whose scores table holds a lower and an upper plane.
constexpr bool has_bounds(int k) { return k == kMeanBound || is_env_bound(k); }
// Kinds that read fp32 Mean rows.
constexpr bool reads_mean(int k) { return k == kMeanDot; }
// Internal kind of an ABI score kind.
constexpr int internal_kind(int abi) {
  return abi <= 2 ? abi : abi <= 5 ? abi + 1 : abi == kAbiNsa ? kHeadDot : kMeanDot;
}

// Channel mapping of a 16-lane row: lane u owns the chunks u, u+16, u+32, ... of a summary
// row, so every load instruction of a row reads 16 contiguous chunks.  The query
// view uses the same mapping (a dot product does not care about channel order).
template <int D, bool BF16>
struct RowMap {
  // 16-byte chunks, or 8-byte bf16 ones when D is not a multiple of 128 (D = 64, 576)
  static constexpr int kElemsPerChunk = BF16 ? (D % 128 == 0 ? 8 : 4) : 4;
  static constexpr int kChunks = D / kElemsPerChunk / 16;     // chunks per lane
  static constexpr int E = kChunks * kElemsPerChunk;          // channels per lane
  static_assert(E * 16 == D, "a row of 16 lanes must cover every channel");
  __device__ static int channel(int u, int c, int e) { return (u + 16 * c) * kElemsPerChunk + e; }
};

// Raw words of one summary row held by one lane: W 32-bit words (fp32 values, or bf16 pairs).
template <int D, bool BF16>
struct RowWords {
  using M = RowMap<D, BF16>;
  static constexpr int W = BF16 ? M::E / 2 : M::E;
  static constexpr int kWordsPerChunk = W / M::kChunks;
};

template <int D, bool BF16>
__device__ __forceinline__ void load_row_words(const void* base, int u, uint32_t (&w)[RowWords<D, BF16>::W]) {
  using M = RowMap<D, BF16>;
  using R = RowWords<D, BF16>;
  const char* b = reinterpret_cast<const char*>(base);
  constexpr int kBytesPerElem = BF16 ? 2 : 4;
#pragma unroll
  for (int c = 0; c < M::kChunks; c++) {
    const char* src = b + (size_t)M::channel(u, c, 0) * kBytesPerElem;
    if constexpr (R::kWordsPerChunk == 4) {
      const uint4 v = load_stream_u4(src);
      w[4 * c] = v.x;
      w[4 * c + 1] = v.y;
      w[4 * c + 2] = v.z;
      w[4 * c + 3] = v.w;
    } else {
      const uint2 v = load_stream_u2(src);
      w[2 * c] = v.x;
      w[2 * c + 1] = v.y;
    }
  }
}

// Channel value e of a lane's row from its raw words.
template <int D, bool BF16>
__device__ __forceinline__ float row_value(const uint32_t (&w)[RowWords<D, BF16>::W], int e) {
  if constexpr (BF16) return (e & 1) ? bf16hi(w[e >> 1]) : bf16lo(w[e >> 1]);
  else return __uint_as_float(w[e]);
}

// Items (page, KV head) per row in one pipeline stage: about 128 bytes of loads per lane
// (64 for the envelope kinds, one-pass and bound pass), in two stages, one loading while the
// other computes.  Measured on the bench workload: 128 bytes per lane beat 64 and 256 (fewer
// waves fit per SIMD at 256), also for the per-head logits.  The envelope bound passes keep four
// waves per SIMD at 64 bytes (115 VGPRs, 149 at 128): Quest on the long-generation workload
// takes 53.4 us at 64 bytes, 54.2 at 128.
template <int D, int KIND>
constexpr int items_per_stage() {
  constexpr int bytes_per_item = (reads_mean(KIND) || needs_min(KIND) ? 4 : 2) * D / 16;
  constexpr int u = (is_env(KIND) || is_env_bound(KIND) ? 64 : 128) / bytes_per_item;
  return u < 1 ? 1 : (u > 8 ? 8 : u);
}

// Row stride of the scores table: a multiple of 4 floats, so that rows can be read as float4.
constexpr int score_stride(int max_pages) { return (max_pages + 3) & ~3; }

constexpr int kChunk = 256;           // page ids staged per chunk (one per thread)
constexpr int kMaxLdsBatch = 4096;    // page_indptr staged in LDS up to this batch
constexpr size_t kLdsPerCu = 160 * 1024;
// Balanced ranges per resident workgroup slot.  Above 1, workgroups queue for slots and the
// dispatcher hands them out as slots free up.
constexpr int kScoreGridFactor = 1;

// The block-mean (or Max) score of one (page, head) row: fp64 products of the lane's
// channels in RowMap order, then the fp64 DPP sum over the 16-lane row, rounded to fp32.
// The one-pass kernel and the two-pass re-scoring both call this, so the two selections
// see bit-identical scores.
template <int D, bool BF16>
__device__ __forceinline__ float exact_row_score(const double (&qb)[D / 16],
                                                 const uint32_t (&w)[RowWords<D, BF16>::W]) {
  double acc = 0.0;
#pragma unroll
  for (int e = 0; e < D / 16; e++) acc = fma(qb[e], (double)row_value<D, BF16>(w, e), acc);
  return (float)row16_sum_f64(acc);
}

// Group-mean query view in RowMap order: fp64 sums of the group's bf16 query values (exact),
// then one division (a multiplication by 1/g when g is a power of two, also exact).
__device__ __forceinline__ double finish_qbar_one(double sum, int g) {
  return (g & (g - 1)) == 0 ? sum * (1.0 / (double)g) : sum / (double)g;
}

// First four 16-byte chunks of each thread (chunks tid + kThreads*t) of request i's Hq x D
// bf16 query block, loaded early so that they travel with other loads.
struct QueryPrefetch {
  uint4 v[4];
  int req = -1;
};
__device__ __forceinline__ void query_prefetch(const uint16_t* __restrict__ q, int i, int n8, QueryPrefetch& p) {
  const uint4* src = reinterpret_cast<const uint4*>(q + (int64_t)i * n8 * 8);
#pragma unroll
  for (int t = 0; t < 4; t++) p.v[t] = src[min((int)threadIdx.x + kThreads * t, n8 - 1)];
  p.req = i;
}

// Request i's query block (n8 chunks) into LDS through put(chunk, index): the prefetched
// chunks when they are request i's, the rest loaded four per thread per round trip.  Indices
// past the end are clamped (a duplicate rewrites the same value), so no load waits behind a
// branch.
template <class Put>
__device__ __forceinline__ void stage_query_block(const uint16_t* __restrict__ q, int i, int n8,
                                                  const QueryPrefetch& pre, Put put) {
  const uint4* src = reinterpret_cast<const uint4*>(q + (int64_t)i * n8 * 8);
  int x0 = threadIdx.x;
  if (pre.req == i) {
#pragma unroll
    for (int t = 0; t < 4; t++) put(pre.v[t], min(x0 + kThreads * t, n8 - 1));
    x0 += 4 * kThreads;
  }
  for (; x0 < n8; x0 += 4 * kThreads) {
    uint4 v[4];
#pragma unroll
    for (int t = 0; t < 4; t++) v[t] = src[min(x0 + kThreads * t, n8 - 1)];
#pragma unroll
    for (int t = 0; t < 4; t++) put(v[t], min(x0 + kThreads * t, n8 - 1));
  }
}

// Request i's raw bf16 query block (n8 16-byte chunks) into LDS.  Issued where no summary load
// is in flight, so that waiting for it waits for nothing else.
__device__ __forceinline__ void load_query_raw(const uint16_t* __restrict__ q, int i, int n8, const QueryPrefetch& pre,
                                               uint4* __restrict__ qraw) {
  stage_query_block(q, i, n8, pre, [&](uint4 w, int x) { qraw[x] = w; });
}

// Barrier over LDS only: the wave's LDS accesses complete, global loads stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Per-head kinds: the raw query block (LDS) as fp32 in each row's channel order,
// qs[(r * 16 + u) * E + e].  Ends with an LDS barrier.
template <int D, bool BF16>
__device__ __forceinline__ void convert_query(const uint4* __restrict__ qraw, int Hq, float* __restrict__ qs) {
  using M = RowMap<D, BF16>;
  constexpr int E = D / 16;
  const int n8 = Hq * D / 8;
  for (int x = threadIdx.x; x < n8; x += kThreads) {
    const uint4 w = qraw[x];
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int t = 0; t < 8; t++) {
      const int flat = 8 * x + t, r = flat / D, c = flat - r * D;
      const int chunk = c / M::kElemsPerChunk, e_in = c - chunk * M::kElemsPerChunk;
      const int uu = chunk % 16, cc = chunk / 16;              // inverse of RowMap::channel
      qs[(r * 16 + uu) * E + cc * M::kElemsPerChunk + e_in] = (t & 1) ? bf16hi(ws[t >> 1]) : bf16lo(ws[t >> 1]);
    }
  }
  lds_barrier();
}

// Group-mean query of every KV head from the raw query block (LDS): qbar[h][c] = (sum over
// r < g of q[h*g + r][c]) / g, the sum in fp64 in head order (exact for bf16 values), then
// finish_qbar's division; channels c >= qdims are zero (the content-channel score leaves the
// rope channels out).  Ends with an LDS barrier.
template <int D>
__device__ __forceinline__ void finish_qbar(const uint4* __restrict__ qraw, int Hq, int H, int qdims,
                                            double* __restrict__ qbar) {
  const int g = Hq / H;
  const uint16_t* qh = reinterpret_cast<const uint16_t*>(qraw);
  for (int t = threadIdx.x; t < H * D; t += kThreads) {
    const int h = t / D, c = t - h * D;
    double acc = 0.0;
    for (int r = 0; r < g; r++) acc += (double)bf16_to_f32(qh[(h * g + r) * D + c]);
    qbar[t] = c < qdims ? finish_qbar_one(acc, g) : 0.0;
  }
  lds_barrier();
}


// Float nearest to x in the given direction (x finite).
__device__ __forceinline__ float f64_to_f32_down(double x) {
  float f = (float)x;
  return (double)f > x ? nextafterf(f, -INFINITY) : f;
}
__device__ __forceinline__ float f64_to_f32_up(double x) {
  float f = (float)x;
  return (double)f < x ? nextafterf(f, INFINITY) : f;
}

// The four heads' per-lane partial sums p[0..3] over the 16 lanes of a row, scattered:
// lanes u and u ^ 8 (row rotation by 8) trade halves so that the lower half keeps heads 0
// and 1 and the upper half 2 and 3; lanes u and 7 - u (half-row mirror) then keep one head
// each; the quad sums the rest.  Lane u returns the total of head u / 4.
template <class T, int CTRL>
__device__ __forceinline__ T dpp_t(T x) {
  if constexpr (sizeof(T) == 8) return dpp_f64<CTRL>(x);
  else return dpp_f32<CTRL>(x);
}
template <class T>
__device__ __forceinline__ T reduce_scatter4(const T (&p)[4], int u) {
  const bool up = (u & 8) != 0;
  const T s0 = up ? p[0] : p[2], s1 = up ? p[1] : p[3];
  const T k0 = (up ? p[2] : p[0]) + dpp_t<T, 0x128>(s0);
  const T k1 = (up ? p[3] : p[1]) + dpp_t<T, 0x128>(s1);
  const bool odd = (u & 4) != 0;
  const T s = odd ? k0 : k1;
  T z = (odd ? k1 : k0) + dpp_t<T, 0x141>(s);
  z += dpp_t<T, 0x4E>(z);                          // quad lanes u ^ 2
  z += dpp_t<T, 0xB1>(z);                          // quad lanes u ^ 1
  return z;
}

// Exact score of an envelope kind for one (page, KV head) item held by a 16-lane row: lane u
// has the RowMap channels of the item's Max row in wa and Min row in wb (wa again when the kind
// reads no Min).  For each query head r of the group, the lane adds its channels' terms in
// channel order in fp64 (each term, a product of two bf16 values or its max / min / ReLU, is
// exact in fp32), the row reduces the sums, and the heads combine by max (head consensus: min).
// Every lane of the row returns the fp64 score.  qs holds the query rows as fp32 in row order:
// head h g + r at qs + ((h g + r) 16 + u) E.  The one-pass score kernel and the two-pass
// re-scoring both call this, so the two selections see bit-identical scores.
template <int KIND, int D>
__device__ __forceinline__ double env_exact(const float* qs, int h, int g, int u,
                                            const uint32_t (&wa)[RowWords<D, true>::W],
                                            const uint32_t (&wb)[RowWords<D, true>::W]) {
  constexpr int E = D / 16;
  if (g == 4) {
    // the four heads' sums reduced together, then the max (min) over the quads that hold them:
    // half-row mirror (quads 0 and 1, 2 and 3), then rotation by 8
    double p[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const float* qr = qs + ((h * 4 + r) * 16 + u) * E;
      double acc = 0.0;
#pragma unroll
      for (int e = 0; e < E; e++) {
        const float x = qr[e] * row_value<D, true>(wa, e);     // exact
        if constexpr (KIND == kQuestRectified) {
          acc += (double)fmaxf(x, 0.f);
        } else {
          const float y = qr[e] * row_value<D, true>(wb, e);   // exact
          acc += (double)(KIND == kEnvLower ? fminf(x, y) : fmaxf(x, y));
        }
      }
      p[r] = acc;
    }
    double z = reduce_scatter4(p, u);
    if constexpr (KIND == kQuestConsensus) {
      z = fmin(z, dpp_f64<0x141>(z));
      z = fmin(z, dpp_f64<0x128>(z));
    } else {
      z = fmax(z, dpp_f64<0x141>(z));
      z = fmax(z, dpp_f64<0x128>(z));
    }
    return z;
  }
  double s = KIND == kQuestConsensus ? INFINITY : -INFINITY;
  for (int r = 0; r < g; r++) {
    const float* qr = qs + ((h * g + r) * 16 + u) * E;
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const float x = qr[e] * row_value<D, true>(wa, e);     // exact
      if constexpr (KIND == kQuestRectified) {
        acc += (double)fmaxf(x, 0.f);
      } else {
        const float y = qr[e] * row_value<D, true>(wb, e);   // exact
        acc += (double)(KIND == kEnvLower ? fminf(x, y) : fmaxf(x, y));
      }
    }
    acc = row16_sum_f64(acc);
    if constexpr (KIND == kQuestConsensus) s = acc < s ? acc : s;
    else s = acc > s ? acc : s;
  }
  return s;
}

// Maximum over the 16 lanes of a DPP row; every lane of the row receives it.
__device__ __forceinline__ float row16_max_f32(float x) {
  x = fmaxf(x, dpp_f32<0x128>(x));
  x = fmaxf(x, dpp_f32<0x124>(x));
  x = fmaxf(x, dpp_f32<0x122>(x));
  x = fmaxf(x, dpp_f32<0x121>(x));
  return x;
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t row16_max_u32(uint32_t x) {
  x = max(x, dpp_u32<0x128>(x));
  x = max(x, dpp_u32<0x124>(x));
  x = max(x, dpp_u32<0x122>(x));
  x = max(x, dpp_u32<0x121>(x));
  return x;
}

// Packed pairs of bf16 values in a 32-bit word (channel 2k in the low half, 2k + 1 in the high).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
typedef short i16x2_t __attribute__((ext_vector_type(2)));
// a.lo b.lo + a.hi b.hi + c (v_dot2c_f32_bf16).  Its rounding is not that of an fp32 fma chain:
// the terms are aligned to the largest one and the sum rounded, which a probe of 4 M operand
// triples (products and accumulators from 2^-30 to 2^30, near cancellations, subnormals) measured
// at no more than 2.9 units of 2^-24 (|a.lo b.lo| + |a.hi b.hi| + |c|) per instruction, with
// subnormal products and results flushed to zero.
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}
// Per-half unsigned maximum of two packed words.
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a),
                                                                __builtin_bit_cast(u16x2_t, b)));
}
// 0xffff in each half whose sign bit is set, else 0.
__device__ __forceinline__ uint32_t pk_sign_mask(uint32_t a) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2_t, a) >> (i16x2_t)15);
}

// ------------------------------------------------------------------------------------
// Score policies.  MEAN_DOT / MAX_DOT: s_j = (mean_r q_r) . S_j (equal to the mean over the
// group's heads of q_r . S_j by linearity); the group-mean query is formed in fp64 from the
// staged query (exact for bf16 inputs) and kept in registers (a row always serves one head).
// QUEST: s_j = max_r sum_c max(q_rc Max_jc, q_rc Min_jc); each product of two bf16 values is
// exact in fp32, the per-head sums run in fp64, and q is read from LDS.
// ------------------------------------------------------------------------------------
template <int KIND, int D>
struct ScorePolicy {
  static constexpr bool kBf16 = !reads_mean(KIND);    // Max, Min, or the bf16 copy of Mean
  static constexpr int E = D / 16;
  static constexpr int U = items_per_stage<D, KIND>();
  static constexpr int W = RowWords<D, kBf16>::W;
  struct Stage {
    uint32_t a[U][W];                     // Mean / Max rows
    uint32_t b[needs_min(KIND) ? U : 1][needs_min(KIND) ? W : 1];   // Min rows
  };
  double qb[KIND == kMeanBound || per_head(KIND) ? 1 : E];  // the row's channels of qbar (exact, fp64)
  float qf[KIND == kMeanBound ? E : 1];   // kMeanBound: the same channels rounded to fp32
  float qabs;                             // kMeanBound: sum over the row of |qf_c|
  // bound kinds: the row's channels of the group's (at most four) query heads as packed bf16
  // pairs split by sign (qp: the channels with q >= 0, the others zero; qn: those with q < 0),
  // zero for heads past g, and the 1-norm over all D channels of this lane's head u / 4
  static constexpr bool kBound = is_env_bound(KIND);
  uint32_t qp[kBound ? 4 : 1][kBound ? E / 2 : 1], qn[kBound ? 4 : 1][kBound ? E / 2 : 1];
  float qnorm;

  // Bound kinds: the row's query registers and the head norms (qs: the request's query block in
  // LDS, fp32 in row order; g <= 4).
  __device__ __forceinline__ void on_new_request_bound(const float* qs, int h, int g, int u) {
    if constexpr (kBound) {
      float nrm[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < E / 2; k++) {
          uint32_t pos = 0u, neg = 0u;
#pragma unroll
          for (int half = 0; half < 2; half++) {
            const float x = r < g ? qs[((h * g + r) * 16 + u) * E + 2 * k + half] : 0.f;
            a += fabsf(x);
            const uint32_t bits = (__float_as_uint(x) >> 16) << (16 * half);   // x is a bf16 value
            if (x >= 0.f) pos |= bits;
            else neg |= bits;
          }
          qp[r][k] = pos;
          qn[r][k] = neg;
        }
        nrm[r] = row16_sum_f32(a);
      }
      const int mh = u >> 2;
      qnorm = mh == 0 ? nrm[0] : mh == 1 ? nrm[1] : mh == 2 ? nrm[2] : nrm[3];
    }
  }

  // The row's view of the group-mean query of KV head h (qbar: [H][D] fp64 in LDS).
  __device__ __forceinline__ void on_new_request(const double* qbar, int h, int u) {
    using MQ = RowMap<D, kBf16>;
    if constexpr (KIND == kMeanBound) {
      float a = 0.f;
#pragma unroll
      for (int c = 0; c < MQ::kChunks; c++)
#pragma unroll
        for (int e = 0; e < MQ::kElemsPerChunk; e++) {
          qf[c * MQ::kElemsPerChunk + e] = (float)qbar[h * D + MQ::channel(u, c, e)];
          a += fabsf(qf[c * MQ::kElemsPerChunk + e]);
        }
      qabs = row16_sum_f32(a);
    } else if constexpr (!per_head(KIND)) {
#pragma unroll
      for (int c = 0; c < MQ::kChunks; c++)
#pragma unroll
        for (int e = 0; e < MQ::kElemsPerChunk; e++)
          qb[c * MQ::kElemsPerChunk + e] = qbar[h * D + MQ::channel(u, c, e)];
    }
  }

  __device__ __forceinline__ void load(Stage& st, const float* __restrict__ mean, const uint16_t* __restrict__ maxs,
                                       const uint16_t* __restrict__ mins, const int* pid, int H, int h, int u,
                                       int j0, int slots, int nj) {
#pragma unroll
    for (int v = 0; v < U; v++) {
      // items past the chunk's end load nothing (compute skips them): every load costs the CU
      // an issue slot, cached or not.  The row's slot is the same for the wave's rows, so the
      // branch is uniform.
      const int jj = j0 + v * slots;
      if (jj >= nj) continue;
      const int64_t o = ((int64_t)pid[jj] * H + h) * D;
      if constexpr (reads_mean(KIND)) {
        load_row_words<D, false>(mean + o, u, st.a[v]);
      } else {
        load_row_words<D, true>(maxs + o, u, st.a[v]);      // Max, or the bf16 Mean copy
        if constexpr (needs_min(KIND)) load_row_words<D, true>(mins + o, u, st.b[v]);
      }
    }
  }

  // Scores of the stage's items; lane v of the row keeps item v's score, and one store per
  // plane writes them all: out[jj] (and, for the bounds, the upper one at out[plane + jj]).
  __device__ __forceinline__ void compute(const Stage& st, const float* qs, int h, int g, int u, int j0, int slots,
                                          int nj, float* __restrict__ out, int64_t plane) const {
    float mine = 0.f, mine_up = 0.f;
#pragma unroll
    for (int v = 0; v < U; v++) {
      const int jj = j0 + v * slots;
      if (jj < nj) {
        double s;
        if constexpr (is_env(KIND)) {
          double z;
          if constexpr (needs_min(KIND)) z = env_exact<KIND, D>(qs, h, g, u, st.a[v], st.b[v]);
          else z = env_exact<KIND, D>(qs, h, g, u, st.a[v], st.a[v]);
          if (u == v) mine = (float)z;
          continue;
        } else if constexpr (kBound) {
          // Per head, the sum of the exact terms t_c = q_c (q_c >= 0 ? a_c : b_c), with a, b = Max,
          // Min for Quest and the head consensus (max(q Max, q Min) is q Max for q >= 0, q Min
          // below), Min, Max for the pessimistic envelope, and max(Max, 0), min(Max, 0) for
          // rectified Quest: t_c = q+_c a_c + q-_c b_c with q+ = q where q >= 0 (else 0) and q- the
          // rest, two chains of bf16 pair dot products (dot2_bf16) per head, two channels per
          // step, added at the end; the row then reduces over 4 levels of fp32 additions.  Error:
          // each of a chain's n = E/2 steps is off by at most K 2^-24 (|its two products| + |the
          // running sum|); with K = 8 (the instruction measured at most 2.9) a chain is off by at
          // most n K 2^-24 sum |t_c| over its terms, so the fp32 sum differs from the exact one by
          // at most (4 K + 5) 2^-24 sum |t_c| < 2^-18.7 sum |t_c| (D = 128; less for D = 64), and
          // sum |t_c| <= |q_h|_1 m with m the largest |Max_c|, |Min_c| of the item.  The one-pass
          // fp64 sum is within 2^-40 sum |t_c| of the exact one, rounding the interval ends adds
          // at most 2^-23 |q_h|_1 m, and the fp32 norm and product fall short of |q_h|_1 m by a
          // factor of at most 1 - 2^-19: b = |q_h|_1 m 2^-18 covers all of these.  Subnormal
          // operands, products and sums flushed to zero lose at most 2^-126 (|q_h|_1 + D m) plus
          // 2^-126 per step over the row, which (|q_h|_1 + m) 2^-110 + 2^-110 covers.  So every
          // head's one-pass sum lies in [s_h - b, s_h + b].  The max (min) over the heads of the
          // ends then brackets the one-pass score, before and after its rounding to fp32
          // (monotone).  m is taken on the bf16 bit patterns (magnitudes order as integers).  A head
          // whose terms could leave the fp32 range, an infinite or NaN operand included (b then is
          // infinite, NaN or at least 2^100, and the fp32 sum may be NaN where the fp64 one is an
          // ordinary number), gets the interval (-inf, inf), so the exact score decides.
          float ax[4] = {0.f, 0.f, 0.f, 0.f}, ay[4] = {0.f, 0.f, 0.f, 0.f};
          uint32_t mb = 0u;
#pragma unroll
          for (int k = 0; k < E / 2; k++) {
            const uint32_t wa = st.a[v][k];
            uint32_t wb = wa;
            if constexpr (needs_min(KIND)) wb = st.b[v][k];
            mb = pk_max_u16(mb, wa & 0x7fff7fffu);
            if constexpr (needs_min(KIND)) mb = pk_max_u16(mb, wb & 0x7fff7fffu);
            uint32_t pa = wa, pb = wb;                   // paired with q >= 0, with q < 0
            if constexpr (KIND == kEnvLowerBound) {
              pa = wb;
              pb = wa;
            } else if constexpr (KIND == kRectifiedBound) {
              const uint32_t neg = pk_sign_mask(wa);
              pa = wa & ~neg;
              pb = wa & neg;
            }
#pragma unroll
            for (int r = 0; r < 4; r++) {
              ax[r] = dot2_bf16(qp[r][k], pa, ax[r]);
              ay[r] = dot2_bf16(qn[r][k], pb, ay[r]);
            }
          }
          float acc[4];
#pragma unroll
          for (int r = 0; r < 4; r++) acc[r] = ax[r] + ay[r];
          const float z = reduce_scatter4(acc, u);           // lane u: head u / 4
          const uint32_t mbits = row16_max_u32(max(mb << 16, mb & 0xffff0000u));
          const float m = __uint_as_float(mbits);
          const float b = qnorm * m * 0x1p-18f + (qnorm + m) * 0x1p-110f + 0x1p-110f;
          const bool finite = b < 0x1p100f;
          constexpr float kNone = KIND == kConsensusBound ? INFINITY : -INFINITY;
          float lo = (u >> 2) < g ? (finite ? z - b : -INFINITY) : kNone;
          float hi = (u >> 2) < g ? (finite ? z + b : INFINITY) : kNone;
          if constexpr (KIND == kConsensusBound) {
            lo = fminf(lo, dpp_f32<0x141>(lo));
            hi = fminf(hi, dpp_f32<0x141>(hi));
            lo = fminf(lo, dpp_f32<0x128>(lo));
            hi = fminf(hi, dpp_f32<0x128>(hi));
          } else {
            lo = fmaxf(lo, dpp_f32<0x141>(lo));
            hi = fmaxf(hi, dpp_f32<0x141>(hi));
            lo = fmaxf(lo, dpp_f32<0x128>(lo));
            hi = fmaxf(hi, dpp_f32<0x128>(hi));
          }
          if (u == v) {
            mine = lo;
            mine_up = hi;
          }
          continue;
        } else if constexpr (KIND == kMeanBound) {
          // In fp32: s' = qf . m and A' = sum |qf_c| |m_c| with m = bf16(Mean) and qf = fp32(qbar).
          // The exact score s (fp64 products of qbar and the fp32 Mean, one rounding to fp32)
          // differs from s' by at most
          //   2^-8 A    RNE to bf16 moves a normal channel by at most 2^-8 of its bf16 value
          //             (a subnormal one by 2^-134: the qabs * 2^-133 term)
          //   2^-24 A   rounding qbar to fp32
          //   40 u A    the fp32 evaluation (D/16 <= 36 fused steps per lane, 4 tree levels;
          //             u = 2^-24)
          //   2^-40 A   the fp64 evaluation of s, and its final rounding (monotone, so it keeps
          //             any fp32 bound on the fp64 value)
          // with A = sum |qbar_c m_c| <= A' (1 + 2^-18).  b = A' (2^-8 + 2^-16) covers all of
          // these plus the fp32 rounding of s' -/+ b itself (at most u (|s'| + b) <= 2^-23 A');
          // 2^-120 covers products that underflow.  So L = s' - b <= s <= s' + b = U.  Where A' is
          // infinite, NaN or near the end of the fp32 range, s' may be NaN while s is an ordinary
          // number: the interval is (-inf, inf) and the exact score decides.
          float acc = 0.f, aab = 0.f;
#pragma unroll
          for (int e = 0; e < E; e++) {
            const float x = row_value<D, true>(st.a[v], e);
            acc = fmaf(qf[e], x, acc);
            aab = fmaf(fabsf(qf[e]), fabsf(x), aab);
          }
          acc = row16_sum_f32(acc);
          aab = row16_sum_f32(aab);
          const float b = aab * (0x1p-8f + 0x1p-16f) + qabs * 0x1p-133f + 0x1p-120f;
          const bool finite = b < 0x1p100f;
          if (u == v) {
            mine = finite ? acc - b : -INFINITY;
            mine_up = finite ? acc + b : INFINITY;
          }
          continue;
        } else {
          s = exact_row_score<D, kBf16>(qb, st.a[v]);
        }
        if (u == v) mine = (float)s;
      }
    }
    const int jj = j0 + u * slots;
    if (u < U && jj < nj) {
      out[jj] = mine;
      if constexpr (has_bounds(KIND)) out[plane + jj] = mine_up;
    }
  }
};

// Byte offsets of the score kernel's dynamic LDS regions (16-byte aligned) and its size.
struct ScoreLds {
  int ind, raw, q, qbar, total;
};
template <int KIND, int D>
__host__ __device__ inline ScoreLds score_lds(int batch, int Hq, int H) {
  ScoreLds L;
  L.ind = 0;
  L.raw = batch <= kMaxLdsBatch ? ((2 * batch + 1) * 4 + 15) & ~15 : 0;   // page_indptr, seq_lens
  L.q = L.raw + Hq * D * 2;
  L.qbar = L.q + (per_head(KIND) ? Hq * D * 4 : 0);
  L.total = L.qbar + (per_head(KIND) ? 0 : H * D * 8);
  return L;
}

struct ScoreArgs {
  const uint16_t* q;
  const int32_t* indptr;
  const int32_t* indices;
  const int32_t* seq_lens;
  const float* mean;
  const uint16_t* maxs;
  const uint16_t* mins;
  float* scores;
  int64_t plane;                       // kMeanBound: floats per scores plane (H * B * stride);
                                       // kHeadDot: floats per query head's rows (B * stride)
  int Hq, H, ps, num_phys, max_pages, batch;   // ps: block size; max_pages: blocks per request
  int r;                               // blocks per page
  int qdims;                           // query channels that enter the group-mean scores
  int stride;                          // row stride of the scores table (max_pages rounded up to 4)
};

// Persistent score kernel following the sequence-local template (Appendix C): the page
// references of the whole batch, in page_indptr order, are split into one balanced
// contiguous range per workgroup.  A workgroup walks its range in chunks of up to 256 pages
// that never cross a request, with one barrier per chunk.  The next chunk's page ids load
// while the current chunk's summaries stream through each row's two-stage pipeline, and
// every row stores its own scores.  The query work of a new request runs while the chunk's
// first loads are in flight.
template <int KIND, int D, bool LDS_IND>
__global__ __launch_bounds__(kThreads) void score_kernel(const ScoreArgs a) {
  using P = ScorePolicy<KIND, D>;

  __shared__ int pid[2][kChunk];
  // dynamic LDS: page_indptr (batch <= kMaxLdsBatch), the raw bf16 query block of the next
  // request to stage, then the per-head kinds' fp32 query in row order [Hq][16][E], or the
  // other kinds' qbar [H][D] fp64
  extern __shared__ uint4 dyn_lds[];
  const ScoreLds L = score_lds<KIND, D>(a.batch, a.Hq, a.H);
  int* ind_lds = reinterpret_cast<int*>(reinterpret_cast<char*>(dyn_lds) + L.ind);
  uint4* qraw = reinterpret_cast<uint4*>(reinterpret_cast<char*>(dyn_lds) + L.raw);
  float* qs = reinterpret_cast<float*>(reinterpret_cast<char*>(dyn_lds) + L.q);
  double* qbar = reinterpret_cast<double*>(reinterpret_cast<char*>(dyn_lds) + L.qbar);
  const int tid = threadIdx.x;
  const int B = a.batch;
  if constexpr (LDS_IND) {
    for (int x = tid; x <= B; x += kThreads) ind_lds[x] = a.indptr[x];
    for (int x = tid; x < B; x += kThreads) ind_lds[B + 1 + x] = a.seq_lens[x];
  }
  __syncthreads();
  // block references: request i's blocks are [indptr[i] * r, indptr[i + 1] * r).  With the
  // page_indptr and the lengths in LDS, the cursor waits on LDS only, never on the summary loads
  // in flight (a wait for a global load issued after them would wait for them too).
  auto ind = [&](int x) -> int { return (LDS_IND ? ind_lds[x] : a.indptr[x]) * a.r; };
  auto len = [&](int i) -> int { return LDS_IND ? ind_lds[B + 1 + i] : a.seq_lens[i]; };
  const int T = ind(B);
  int k0, k1;
  {
    const int n = T, prog = (int)blockIdx.x, nprog = (int)gridDim.x;
    const int per = n / nprog, rem = n % nprog;
    k0 = prog * per + min(prog, rem);
    k1 = k0 + per + (prog < rem ? 1 : 0);
  }
  if (k0 >= k1) return;                                  // uniform over the block
  // request holding k0: the last i with ind(i) <= k0
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ind(mid) <= k0) lo = mid;
    else hi = mid - 1;
  }

  const int row = tid >> 4, u = tid & 15;
  const int h = row % a.H, slot = row / a.H, slots = kRows / a.H;
  const int g = a.Hq / a.H;

  // Chunk cursor: request ci, refs [ck, cend), of which the first cn are pages (logical pages
  // from cj).  A chunk's end needs only the page-list bounds; its page count needs the request's
  // length, a global load that is issued with the chunk's page ids and read after them.
  auto advance = [&](int& i, int k) {
    while (i < B - 1 && ind(i + 1) <= k) i++;
    return min(k1, min(k + kChunk, ind(i + 1)));
  };
  auto pages_in = [&](int i, int k, int end, int L, int& j0) {
    const int base = ind(i);
    const int P = num_pages(L, a.ps, ind(i + 1) - base, a.max_pages);
    j0 = k - base;
    return max(0, min(end, base + P) - k);               // refs past P_i are not pages
  };

  int ci = lo, ck = k0;
  int cend = advance(ci, ck);
  // The first request's query rows, the chunk's page ids and the request's length load
  // together: every reference of [ck, cend) lies in the request's page list, so the ids past its
  // last page are read (in bounds) and never used.  The raw query block reaches LDS before any
  // summary load is issued, so the staging below waits on LDS only (a wait for a query register
  // after the summary loads would wait for those too).
  const int n8 = a.Hq * D / 8;
  int cn, cj;
  {
    QueryPrefetch pre;
    query_prefetch(a.q, ci, n8, pre);
    if (tid < cend - ck) pid[0][tid] = (int)block_row(a.indices, ck + tid, a.r, a.num_phys);
    load_query_raw(a.q, ci, n8, pre, qraw);
    cn = pages_in(ci, ck, cend, len(ci), cj);
  }
  QueryPrefetch none;                                   // req -1: nothing prefetched
  int buf = 0, cur_req = -1, raw_req = ci;
  int next_raw = 0;                                      // the next chunk's page id (raw), per thread
  P pol;
  while (true) {
    __syncthreads();                                     // pid[buf] and qraw ready; last chunk's q reads done
    // the chunk's first stage is in flight while the query work below runs
    const bool active = cn > 0 && slot < cn;
    const int step = P::U * slots;
    const int* pc = pid[buf];
    typename P::Stage sa, sb;
    if (active) pol.load(sa, a.mean, a.maxs, a.mins, pc, a.H, h, u, slot, slots, cn);
    if (ci != cur_req && cn > 0) {                       // uniform over the block; qraw holds ci's block
      if constexpr (per_head(KIND)) {
        convert_query<D, P::kBf16>(qraw, a.Hq, qs);
        if constexpr (is_env_bound(KIND)) pol.on_new_request_bound(qs, h, g, u);
      } else {
        finish_qbar<D>(qraw, a.Hq, a.H, a.qdims, qbar);
        pol.on_new_request(qbar, h, u);
      }
      cur_req = ci;
    }
    // next chunk: its end, and its raw page ids into a register, consumed after this chunk's
    // summaries (the block rows are formed there, so nothing waits for the load before)
    int ni = ci, nk = cend, nend = cend;
    const bool more = nk < k1;
    if (more) {
      nend = advance(ni, nk);
      if (tid < nend - nk) next_raw = a.indices[(nk + tid) / a.r];
    }
    if (active) {
      float* out = a.scores + ((int64_t)h * B + ci) * a.stride + cj;    // this chunk's pages, head h
      int j0 = slot;
      while (true) {
        int jn = j0 + step;
        if (jn < cn) pol.load(sb, a.mean, a.maxs, a.mins, pc, a.H, h, u, jn, slots, cn);
        pol.compute(sa, qs, h, g, u, j0, slots, cn, out, a.plane);
        if (jn >= cn) break;
        j0 = jn;
        jn = j0 + step;
        if (jn < cn) pol.load(sa, a.mean, a.maxs, a.mins, pc, a.H, h, u, jn, slots, cn);
        pol.compute(sb, qs, h, g, u, j0, slots, cn, out, a.plane);
        if (jn >= cn) break;
        j0 = jn;
      }
    }
    if (!more) break;
    int nj0;
    const int nn = pages_in(ni, nk, nend, len(ni), nj0);
    // The empty asm consumes the raw id here, on every lane: the compiler can neither fold the
    // clamp into the load's branch nor leave the load pending into the next chunk, and either
    // would make it wait for the load, and for every summary load issued before it, ahead of
    // a chunk's work.
    asm volatile("" : "+v"(next_raw));
    if (tid < nn) {                                    // read after the next loop-top barrier
      const int jb = nk + tid, qb = jb / a.r;
      pid[buf ^ 1][tid] = (int)(clamp_page(next_raw, a.num_phys) * a.r + (jb - qb * a.r));
    }
    // the next request's raw query block, after this chunk's loads (no reader of qraw is left:
    // the staging above ended with a barrier)
    if (ni != raw_req) {                                 // uniform over the block
      load_query_raw(a.q, ni, n8, none, qraw);
      raw_req = ni;
    }
    buf ^= 1;
    ci = ni;
    ck = nk;
    cn = nn;
    cj = nj0;
    cend = nend;
  }
}

// ------------------------------------------------------------------------------------
// Per-query-head logits z_r = q_r . Mean_j (the NSA flow's first step): fp64 products and sums, one
// rounding to fp32, on the fp64 matrix cores.  The walk over the batch's page references is
// score_kernel's.  v_mfma_f64_4x4x4 multiplies four 4x4 blocks; here a wave takes four pages of
// one KV head (A rows i = lane & 3), four query heads of its group (B columns j = lane & 3) and
// splits the channels over k = lane >> 4 and the blocks b = (lane >> 2) & 3: a lane loads the
// 16-byte chunks 4k + b + 16c of its page's Mean row, one channel of which enters each MFMA, and the
// four blocks' sums meet in two DPP additions.  Groups of more than four heads take NS sets of four.
// The query takes 2 D/16 registers a set instead of four times as many per lane of a 16-lane row,
// and the row reductions fall away, so four waves fit per SIMD where the VALU form ran at two.
// KV heads: wave w of a workgroup takes H / 4 adjacent heads of H >= 4, one after the other over
// each stage's pages, so that a page's rows are read close together in time; with fewer heads the
// waves of one head share out the pages.
// Bound: the fp32 Mean stream.  Measured (64 requests of 8192 to 32768 tokens, 8 KV heads, groups of
// four, 325 MB), VALU form 84 us: one head at a time over a whole chunk of pages 87 us, heads w and
// w + 4 over each stage 74, adjacent heads 69 (4.7 TB/s).  Without the stores 8 us less; without the
// matrix instructions 2 us less; with cached instead of non-temporal loads 78.
template <int D, int NS, bool LDS_IND>
__global__ __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(NS == 1 ? 4 : NS == 2 ? 3 : 2))) void head_score_kernel(const ScoreArgs a) {
  constexpr int C = D / 64;                // 16-byte chunks of a row per lane
  constexpr int U = 8 / C;                 // pages per lane and stage: 128 bytes of loads
  constexpr int E = 4 * C;                 // channels per lane
  __shared__ int pid[2][kChunk];
  extern __shared__ uint4 dyn_lds[];
  const int B = a.batch, tid = (int)threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 3, b = (lane >> 2) & 3, k = lane >> 4;
  const int n8 = a.Hq * D / 8, g = a.Hq / a.H;
  uint4* qraw = dyn_lds;                   // two query blocks: the current chunk's and the next one's
  int* ind_lds = reinterpret_cast<int*>(dyn_lds + 2 * n8);
  if constexpr (LDS_IND) {
    for (int x = tid; x <= B; x += kThreads) ind_lds[x] = a.indptr[x];
    for (int x = tid; x < B; x += kThreads) ind_lds[B + 1 + x] = a.seq_lens[x];
  }
  __syncthreads();
  auto ind = [&](int x) -> int { return (LDS_IND ? ind_lds[x] : a.indptr[x]) * a.r; };
  auto len = [&](int x) -> int { return LDS_IND ? ind_lds[B + 1 + x] : a.seq_lens[x]; };
  int k0, k1;
  {
    const int n = ind(B), prog = (int)blockIdx.x, nprog = (int)gridDim.x;
    const int per = n / nprog, rem = n % nprog;
    k0 = prog * per + min(prog, rem);
    k1 = k0 + per + (prog < rem ? 1 : 0);
  }
  if (k0 >= k1) return;                    // uniform over the workgroup
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ind(mid) <= k0) lo = mid;
    else hi = mid - 1;
  }
  auto advance = [&](int& x, int kk) {
    while (x < B - 1 && ind(x + 1) <= kk) x++;
    return min(k1, min(kk + kChunk, ind(x + 1)));
  };
  auto pages_in = [&](int x, int kk, int end, int& j0) {
    const int base = ind(x);
    const int P = num_pages(len(x), a.ps, ind(x + 1) - base, a.max_pages);
    j0 = kk - base;
    return max(0, min(end, base + P) - kk);
  };
  // the wave's heads and its share of a chunk's pages
  const int passes = a.H >= 4 ? a.H / 4 : 1, slots = a.H >= 4 ? 4 : 16 / a.H;
  const int h0 = a.H >= 4 ? w * passes : w % a.H, slot0 = a.H >= 4 ? 0 : 4 * (w / a.H);

  QueryPrefetch none;
  int ci = lo, ck = k0, cend = advance(ci, ck), cj;
  if (tid < cend - ck) pid[0][tid] = (int)block_row(a.indices, ck + tid, a.r, a.num_phys);
  load_query_raw(a.q, ci, n8, none, qraw);
  int cn = pages_in(ci, ck, cend, cj);
  int buf = 0, qb = 0, next_raw = 0;
  uint4 sa[U][C], sb[U][C];
  double qv[NS][E];
  while (true) {
    __syncthreads();                       // pid[buf] and the query block ready
    const int* pc = pid[buf];
    // stage (pass, j0): pages j0 + i + slots v of the pass's head
    auto load = [&](int pass, int j0, uint4 (&st)[U][C]) {
      const int h = h0 + pass;
#pragma unroll
      for (int v = 0; v < U; v++) {
        if (j0 + v * slots >= cn) continue;                        // uniform over the wave
        const int j = min(j0 + v * slots + i, cn - 1);
        const float* src = a.mean + ((int64_t)pc[j] * a.H + h) * D + 4 * (4 * k + b);
#pragma unroll
        for (int c = 0; c < C; c++) st[v][c] = load_stream_u4(src + 64 * c);
      }
    };
    auto load_q = [&](int pass) {
      const int h = h0 + pass;
      const uint16_t* qh = reinterpret_cast<const uint16_t*>(qraw + qb * n8);
#pragma unroll
      for (int s = 0; s < NS; s++) {
        const int r = 4 * s + i;                                   // column j of B: query head 4 s + j
        const bool ok = r < g;
#pragma unroll
        for (int c = 0; c < C; c++) {
          const uint2 x = *reinterpret_cast<const uint2*>(qh + (h * g + (ok ? r : 0)) * D + 64 * c + 4 * (4 * k + b));
          qv[s][4 * c] = ok ? (double)bf16lo(x.x) : 0.0;
          qv[s][4 * c + 1] = ok ? (double)bf16hi(x.x) : 0.0;
          qv[s][4 * c + 2] = ok ? (double)bf16lo(x.y) : 0.0;
          qv[s][4 * c + 3] = ok ? (double)bf16hi(x.y) : 0.0;
        }
      }
    };
    auto compute = [&](int pass, int j0, const uint4 (&st)[U][C]) {
      // D row i, column j of block b sits in lane 16 i + 4 b + j
      const int jd = lane & 3, id = lane >> 4, bd = b;
      float mine = 0.f;
#pragma unroll
      for (int p = 0; p < U * NS; p++) {
        const int v = p / NS, s = p % NS;
        if (j0 + v * slots < cn) {
          double acc = 0.0;
#pragma unroll
          for (int c = 0; c < C; c++) {
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)__uint_as_float(st[v][c].x), qv[s][4 * c], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)__uint_as_float(st[v][c].y), qv[s][4 * c + 1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)__uint_as_float(st[v][c].z), qv[s][4 * c + 2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)__uint_as_float(st[v][c].w), qv[s][4 * c + 3], acc, 0, 0, 0);
          }
          acc += dpp_f64<0x128>(acc);                              // blocks b ^ 2, then b ^ 1 (row rotations)
          acc += dpp_f64<0x124>(acc);
          if (bd == p % 4) mine = (float)acc;
        }
        if (p % 4 == 3) {
          // lane (i, b, j) holds sum p - 3 + b: its page and head, one store for four sums
          const int pp = p - 3 + bd, pv = pp / NS, r = 4 * (pp % NS) + jd;
          const int jj = j0 + pv * slots + id, h = h0 + pass;
          if (r < g && jj < cn) a.scores[(int64_t)(h * g + r) * a.plane + (int64_t)ci * a.stride + cj + jj] = mine;
        }
      }
    };
    static_assert(U * NS % 4 == 0, "whole stores");
    auto step = [&](int& pass, int& j0) {  // the next stage; false past the last
      if (++pass == passes) {
        pass = 0;
        j0 += U * slots;
      }
      return j0 < cn;
    };
    int pa = 0, ja = slot0;
    const bool active = slot0 < cn;
    if (active) {
      load(pa, ja, sa);
      load_q(0);
    }
    // next chunk: its end, and its raw page ids into a register, consumed after this chunk's work
    int ni = ci, nk = cend, nend = cend;
    const bool more = nk < k1;
    if (more) {
      nend = advance(ni, nk);
      if (tid < nend - nk) next_raw = a.indices[(nk + tid) / a.r];
    }
    if (active) {
      int pb = pa, jb = ja;
      while (true) {
        bool go = step(pb, jb);
        if (go) load(pb, jb, sb);
        compute(pa, ja, sa);
        if (!go) break;
        if (pb != pa) load_q(pb);
        pa = pb;
        ja = jb;
        go = step(pa, ja);
        if (go) load(pa, ja, sa);
        compute(pb, jb, sb);
        if (!go) break;
        if (pa != pb) load_q(pa);
        pb = pa;
        jb = ja;
      }
    }
    if (!more) break;
    int nj0;
    const int nn = pages_in(ni, nk, nend, nj0);
    asm volatile("" : "+v"(next_raw));     // the load completes here, on every lane, not in a branch
    if (tid < nn) {
      const int jb = nk + tid, q = jb / a.r;
      pid[buf ^ 1][tid] = (int)(clamp_page(next_raw, a.num_phys) * a.r + (jb - q * a.r));
    }
    if (ni != ci) {                        // uniform: the next request's block, beside the one in use
      qb ^= 1;
      load_query_raw(a.q, ni, n8, none, qraw + qb * n8);
    }
    buf ^= 1;
    ci = ni;
    ck = nk;
    cn = nn;
    cj = nj0;
    cend = nend;
  }
}

// ------------------------------------------------------------------------------------
// top-K selection, one workgroup per (request, KV head)
// ------------------------------------------------------------------------------------
__device__ __forceinline__ bool is_forced(int j, int P, int n_sink, int n_local) {
  return j < n_sink || j >= P - n_local;
}

// Wave-wide inclusive scans in lane order through DPP moves, with no LDS round trip: shifts by 1,
// 2, 4 and 8 lanes within each row of 16, then the row totals carried forward by the broadcasts of
// lane 15 (into rows 1 and 3) and lane 31 (into rows 2 and 3).  A lane that a move leaves without
// a source takes the operation's identity.  Lane 63 ends with the whole wave's value.  The whole
// wave must be active.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x, uint32_t identity) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)x, CTRL, ROWS, 0xf, false);
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan_bits(uint32_t x, uint32_t identity, Op op) {
  x = op(x, dpp_move<0x111>(x, identity));          // row_shr:1
  x = op(x, dpp_move<0x112>(x, identity));          // row_shr:2
  x = op(x, dpp_move<0x114>(x, identity));          // row_shr:4
  x = op(x, dpp_move<0x118>(x, identity));          // row_shr:8
  x = op(x, dpp_move<0x142, 0xa>(x, identity));     // row_bcast:15
  x = op(x, dpp_move<0x143, 0xc>(x, identity));     // row_bcast:31
  return x;
}
__device__ __forceinline__ int wave_incl_sum(int x) {
  return (int)wave_scan_bits((uint32_t)x, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_last(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
__device__ __forceinline__ float wave_min_f32(float x) {
  return __uint_as_float(wave_last(wave_scan_bits(__float_as_uint(x), 0x7f800000u, [](uint32_t a, uint32_t b) {
    return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
  })));
}
__device__ __forceinline__ float wave_max_f32(float x) {
  return __uint_as_float(wave_last(wave_scan_bits(__float_as_uint(x), 0xff800000u, [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  })));
}

// Inclusive scan of one int per thread over the kThreads threads of the block, in thread order.
__device__ __forceinline__ int block_incl_scan(int x, int* wave_tot, int* total) {
  const int lane = lane_id(), w = threadIdx.x >> 6;
  x = wave_incl_sum(x);
  if (lane == kWave - 1) wave_tot[w] = x;
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kThreads / kWave; k++) {
    const int t = wave_tot[k];
    before += (k < w) ? t : 0;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return x + before;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  return wave_last(wave_scan_bits(x, 0xffffffffu, [](uint32_t a, uint32_t b) { return min(a, b); }));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  return wave_last(wave_scan_bits(x, 0u, [](uint32_t a, uint32_t b) { return max(a, b); }));
}

// Options of the radix selection beyond the exact one (Sec. 5.2 approximate top-k):
//   remap 1: keys are the affine map of the candidates' [min, max] onto 32-bit fixed point,
//            floor((s - min) * scale), scale = 4294967295 / (max - min) in fp64;
//   tau_q:   tolerate ratio in 16-bit fixed point; after a pass with key bits left, refinement
//            stops once certain * 65536 >= (65536 - tau_q) * K_free members lie in higher bins,
//            and the rest is a random sample of the threshold bin: its members ordered by the
//            8-bit hash h8(j) = lowbias32(z ^ j) >> 24, larger first, equal hashes by page,
//            z = lowbias32(seed ^ lowbias32(i * H + h)).  One more radix pass, over h8 instead
//            of the next key digit, finds the hash threshold.
// remap 0 and tau_q 0 is the exact selection.
struct TopkOptions {
  int remap, tau_q;
  uint32_t seed;
};

__device__ __forceinline__ uint32_t lowbias32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

// Block-wide min and max of one float per thread (NaN-free inputs; +inf/-inf when empty).
__device__ __forceinline__ void block_fminmax(float& mn, float& mx, float (*wave_fm)[kThreads / kWave]) {
  const int lane = lane_id(), w = threadIdx.x >> 6;
  mn = wave_min_f32(mn);
  mx = wave_max_f32(mx);
  if (lane == 0) {
    wave_fm[0][w] = mn;
    wave_fm[1][w] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kThreads / kWave; x++) {
    mn = fminf(mn, wave_fm[0][x]);
    mx = fmaxf(mx, wave_fm[1][x]);
  }
}

struct RadixState {
  uint32_t prefix, pmask;   // resolved high bits of the k-th largest key
  int top;                  // highest unresolved bit, -1 when done
  int remaining;            // rank of the target among keys that share the prefix
};

// Start from the candidates' smallest and largest keys: bits above the highest differing bit
// are common to every candidate.
__device__ __forceinline__ RadixState radix_init(uint32_t kmin, uint32_t kmax, int k) {
  RadixState r;
  const uint32_t diff = kmin ^ kmax;
  r.top = diff ? 31 - __clz((int)diff) : -1;
  r.pmask = r.top < 0 ? 0xffffffffu : (r.top >= 31 ? 0u : ~((2u << r.top) - 1u));
  r.prefix = kmin & r.pmask;
  r.remaining = k;
  return r;
}
// Digits of up to BITS bits, most significant first.
template <int BITS>
__device__ __forceinline__ int radix_shift(const RadixState& r) { return r.top >= BITS - 1 ? r.top - (BITS - 1) : 0; }
template <int BITS>
__device__ __forceinline__ uint32_t radix_dmask(const RadixState& r) {
  return r.top >= 0 ? (1u << (r.top - radix_shift<BITS>(r) + 1)) - 1u : 0u;
}

template <int BITS>
__device__ __forceinline__ void radix_advance(RadixState& r, const int* pick) {
  const int sh = radix_shift<BITS>(r);
  r.remaining -= pick[1];
  r.prefix |= (uint32_t)pick[0] << sh;
  r.pmask |= radix_dmask<BITS>(r) << sh;
  r.top = sh - 1;
}

// ------------------------------------------------------------------------------------
// Selection, one workgroup of T threads per (request, KV head), K pages per thread: thread t
// holds pages t, t + T, ..., so 64 consecutive pages lie in one wave's lanes of one slot, a ballot
// is a 64-bit word of page flags, and the words in slot and wave order are the pages in ascending
// order.  The chosen set is those words in LDS; compacting it takes one wave-wide prefix over
// their counts, which every wave forms for itself.  A few pairs wait for a chain of dependent round
// trips (geometry, bound rows, re-scored summaries) and barriers; a chip full of pairs is bound by
// instruction issue.  So slots past the request's pages are skipped by uniform branches, and the
// shape (T, K) follows the request bound and the number of pairs.
// ------------------------------------------------------------------------------------
template <int T, int K>
struct SelShape {
  static constexpr int W = T / kWave;                  // waves
  static constexpr int M = T * K;                      // pages
  static constexpr int kWords = M / kWave;             // flag words
  static constexpr int G = (kWords + kWave - 1) / kWave;   // words a lane holds in a prefix
  static_assert(kWave % W == 0, "a slot's words lie in one prefix group");
};

// Members and exclusive prefix counts of the flag words, as every wave holds them: lane l of
// group g has word 64 g + l.
template <int T, int K>
struct WordPrefix {
  using S = SelShape<T, K>;
  uint32_t lo[S::G], hi[S::G];
  int excl[S::G], total;
  __device__ __forceinline__ void load(const uint2* words, int nwords) {
    const int lane = lane_id();
    total = 0;
#pragma unroll
    for (int y = 0; y < S::G; y++) {
      const int wi = kWave * y + lane;
      const uint2 v = wi < nwords ? words[wi] : make_uint2(0u, 0u);
      lo[y] = v.x;
      hi[y] = v.y;
      const int c = __popc(v.x) + __popc(v.y);
      const int incl = wave_incl_sum(c);
      excl[y] = total + incl - c;
      total += (int)wave_last((uint32_t)incl);
    }
  }
  // This thread's page of slot x (a compile-time constant after unrolling) in wave w: whether it
  // is a member, and how many members lie below it.
  __device__ __forceinline__ bool at(int x, int w, int& rank) const {
    const int y = x * S::W / kWave, src = x * S::W % kWave + w;
    const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)lo[y], src);
    const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)hi[y], src);
    rank = __builtin_amdgcn_mbcnt_hi(u, __builtin_amdgcn_mbcnt_lo(l, (uint32_t)__builtin_amdgcn_readlane(excl[y], src)));
    return __builtin_amdgcn_inverse_ballot_w64((uint64_t)u << 32 | l);
  }
};
__device__ __forceinline__ uint2 word_of(uint64_t m) { return make_uint2((uint32_t)m, (uint32_t)(m >> 32)); }

// A wave's own words, one per slot: collected with lane x holding slot x's, stored at once.
template <int T, int K>
struct SlotWords {
  uint32_t lo = 0u, hi = 0u;
  __device__ __forceinline__ void put(int x, uint64_t m) {
    const bool mine = lane_id() == x;
    lo = mine ? (uint32_t)m : lo;
    hi = mine ? (uint32_t)(m >> 32) : hi;
  }
  __device__ __forceinline__ void add(int x, uint64_t m, int lane = lane_id()) {   // into slot x's word
    const bool mine = lane == x;
    lo |= mine ? (uint32_t)m : 0u;
    hi |= mine ? (uint32_t)(m >> 32) : 0u;
  }
  __device__ __forceinline__ void store(uint2* words, int w, int P) const {
    const int x = lane_id();
    if (x < K && x * T < P) words[x * SelShape<T, K>::W + w] = make_uint2(lo, hi);
  }
};

// The request's geometry and its share of the selection.
struct SelArgs {
  const float* lower;                  // [H][batch][stride] scores, or their lower bounds
  const float* upper;                  // upper bounds (two-pass kinds)
  const float* mean;                   // summaries of the re-scoring
  const uint16_t* maxs;
  const uint16_t* mins;
  const uint16_t* q;
  int Hq, H, qdims, ps, r, max_pages, stride, batch, num_phys;
  const int32_t* indptr;
  const int32_t* indices;
  const int32_t* seq_lens;
  const int32_t* items;                // page counts of the operator; nullptr: from seq_lens
  const int32_t* budget;
  int n_sink, n_local, max_sel;
  int32_t* sel_pages;
  int32_t* sel_count;
};
struct SelRow {
  int i, h, base, P, nS, nL, Kfree;
  bool all;
  int32_t* out;
};
__device__ __forceinline__ SelRow sel_row(const SelArgs& a, int b, int cap) {
  SelRow s;
  s.i = b / a.H;
  s.h = b - s.i * a.H;
  s.base = a.items ? 0 : a.indptr[s.i];
  s.P = a.items ? min(min(max(a.items[s.i], 0), a.stride), cap)
                : num_pages(a.seq_lens[s.i], a.ps, (a.indptr[s.i + 1] - s.base) * a.r, min(a.max_pages, cap));
  const int Ktot = max(min(a.budget[s.i], a.max_sel), 0);
  s.all = Ktot >= s.P;
  s.nS = min(a.n_sink, s.P);
  s.nL = min(a.n_local, s.P);
  const int nF = s.all ? s.P : s.nS + s.nL - max(0, s.nS - (s.P - s.nL));
  s.Kfree = s.all ? 0 : max(0, Ktot - nF);
  s.out = a.sel_pages + ((int64_t)s.i * a.H + s.h) * a.max_sel;
  return s;
}

// Ascending compaction of the chosen words (complete, behind a barrier) into the selection row.
template <int T, int K>
__device__ __forceinline__ void write_selection(const SelArgs& a, const SelRow& s, const uint2* words, int w) {
  using S = SelShape<T, K>;
  const int tid = (int)threadIdx.x;
  WordPrefix<T, K> wp;
  wp.load(words, (s.P + T - 1) / T * S::W);
#pragma unroll
  for (int x = 0; x < K; x++) {
    if (x * T < s.P) {                               // uniform
      int pos;
      if (wp.at(x, w, pos) && pos < a.max_sel) s.out[pos] = x * T + tid;
    }
  }
  for (int m = wp.total + tid; m < a.max_sel; m += T) s.out[m] = -1;
  if (s.h == 0 && tid == 0) a.sel_count[s.i] = min(wp.total, a.max_sel);
}

constexpr int kBins = 1024;            // histogram bins: 16 per lane of the wave that scans them

// One wave: the bin that holds the k-th largest entry of a histogram of kBins bins, the number of
// entries above it and its own count, in pick[0..2].  Lane l owns the bins 1023 - 16 l .. 1008 - 16 l.
__device__ __forceinline__ void wave_pick_bin(const int* hist, int k, int* pick) {
  constexpr int N = kBins / kWave;
  int lane = lane_id();
  asm volatile("" : "+v"(lane));                     // the bin numbers stay here, not in registers around a loop
  int c[N], tot = 0;
#pragma unroll
  for (int e = 0; e < N; e += 4) {
    const int4 v = *reinterpret_cast<const int4*>(&hist[kBins - N * lane - 4 - e]);
    c[e] = v.w;
    c[e + 1] = v.z;
    c[e + 2] = v.y;
    c[e + 3] = v.x;
    tot += (v.x + v.y) + (v.z + v.w);
  }
  int above = wave_incl_sum(tot) - tot;
  if (above < k && above + tot >= k) {               // one lane
#pragma unroll
    for (int e = 0; e < N; e++) {
      if (above < k && above + c[e] >= k) {
        pick[0] = kBins - 1 - N * lane - e;
        pick[1] = above;
        pick[2] = c[e];
      }
      above += c[e];
    }
  }
}

// The decode step's append inside the selection launch, by workgroups of its own ahead of the
// selection's: they write the step's K/V rows at token L - 1 and refresh that block's summaries
// with the cache stage's own task code (4 lanes per 8-channel task, as in the decode-step summary
// launch), so the cache and the summaries are bit-identical to a separate append.  The block is
// its request's last one, a forced local block, so the selection never reads its new summary.
struct AppendStep {
  summ::AppendArgs app;      // app.knew == nullptr: nothing to append
  const void* k;             // the K cache (read)
  float k_scale;
  int kt, ps, D, num_phys;
  int max_pages;             // blocks per request bound
  float* mean;
  uint16_t* mean_bf;
  uint16_t* maxo;
  uint16_t* mino;
};
// Append workgroups per request in a launch of T-thread workgroups: T / 4 tasks each.
template <int T>
__host__ __device__ constexpr int append_wgs(int H, int D) { return (H * (D / 8) + T / 4 - 1) / (T / 4); }

// Append workgroup a: its share of the tasks (KV head, 8-channel chunk) of its request's block
// L - 1.  A request whose token L - 1 lies in no listed block (L = 0, a short page list) appends
// nothing, as in the cache stage's own append launch.
template <int T, int KT, int KB>
__device__ __forceinline__ void append_tasks_kt(const AppendStep& ap, int a, int H, int bs, int r,
                                                const int32_t* __restrict__ indptr,
                                                const int32_t* __restrict__ indices,
                                                const int32_t* __restrict__ seq_lens) {
  const int wgs = append_wgs<T>(H, ap.D), i = a / wgs;
  const int L = seq_lens[i], base = indptr[i];
  const int P = num_pages(L, bs, (indptr[i + 1] - base) * r, ap.max_pages);
  if (L < 1 || (L - 1) / bs >= P) return;
  const int chunks = ap.D / 8;
  const int t = (a - i * wgs) * (T / 4) + (int)threadIdx.x / 4;          // the same for a quad's lanes
  const bool active = t < H * chunks;
  const int tk = active ? t : 0, h = tk / chunks;
  summ::task<4, KT, true, KB>(ap.k, ap.k_scale, ap.num_phys, H, ap.ps, bs, r, ap.D, indices, base, L, i,
                              (L - 1) / bs, h, tk - h * chunks, active, (int)threadIdx.x & 3, ap.mean, ap.mean_bf,
                              ap.maxo, ap.mino, ap.app);
}
// KB: token rows a lane loads per round trip (the order of the sums does not depend on it).
template <int T, int KB>
__device__ __forceinline__ void append_tasks(const AppendStep& ap, int a, int H, int bs, int r,
                                             const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                             const int32_t* __restrict__ seq_lens) {
  if (ap.kt == kKvFp8E4M3) append_tasks_kt<T, kKvFp8E4M3, KB>(ap, a, H, bs, r, indptr, indices, seq_lens);
  else if (ap.kt == kKvFp8E5M2) append_tasks_kt<T, kKvFp8E5M2, KB>(ap, a, H, bs, r, indptr, indices, seq_lens);
  else append_tasks_kt<T, kKvBf16, KB>(ap, a, H, bs, r, indptr, indices, seq_lens);
}

// ------------------------------------------------------------------------------------
// Exact selection.  For each (request, KV head), with K = K_free and B a monotone map of the
// bounds onto kBins bins of equal width between the smallest candidate lower bound and the
// largest candidate upper bound:
//   T_lo = K-th largest B(lower), T_hi = (K+1)-th largest B(upper) (over candidates);
//   B(upper) < T_lo  -> out: K candidates score strictly higher (their fp32 keys too);
//   B(lower) > T_hi  -> in:  at most K candidates, itself included, can score >= it;
//   otherwise undecided: ranked by its exact score; the best K - |in| of them by (score desc,
//   page asc) complete the set.
// B is non-decreasing, so the classification is as rigorous on bins as on the floats.  kBins bins are
// enough for the block mean, whose bounds leave the thresholds some three bins apart on spread-out
// scores (22 pages undecided on rows of 512 to 2048, 20 with 65536 bins); the envelope bounds are some 25
// times narrower than a bin, which leaves two to eight pages of the threshold's own to most rows of
// 4096, and one block that scores far above the others widens the bins for all.  So
// while both thresholds lie in one bin or in neighbours and more pages are undecided than one round of
// re-scoring takes, the undecided are binned again, between the extremes of the thresholds' own bins.
// Whole call, 64 pairs of 8192 blocks, one block scaled by 1 / 300 / 10^6: Quest 63.7 / 85.1 / 305 us with
// one histogram, 63.0 / 71.7 / 81 so; block mean 39.2 / 49.2 / 176 and 39.1 / 46.6 / 57.  Refining fewer
// pages than that costs more than re-scoring them (Quest 68.4 us without an outlier, 52.7 instead of
// 45.9 on 16 pairs of 16384 blocks).
// RK = kMeanDot: the two-pass block-mean selection (bounds in, fp32 Mean rows of D channels for
// the re-scoring with exact_row_score, the one-pass arithmetic).  RK = an envelope kind: the
// two-pass selection of that kind (bounds in, bf16 Max and Min rows of D channels for the
// re-scoring, g <= 4).  RK = kNoRescore: exact scores (lower == upper == the scores); the
// undecided pages are ranked by their own scores.
// Up to a wave of undecided pages is ranked by one wave; more (near-ties, or skewed scores such as
// the NSA softmax, which put most candidates in the lowest bins) by a radix select over the exact
// keys.  More than kMaxUndecided pages to re-score (bounds wider than the scores' spread): every page
// is re-scored, in batches whose rows and page ids load ahead of their use.  One workgroup then reads
// all of its row: 64 pairs of 8192 blocks whose Means differ by 2 % of their size, whole call 166 us with
// two dependent pages per lane row at a time, 144 so; 16 pairs of 16384 blocks 306 / 227.
// On 512 pairs instruction issue bounds it (the active-instruction counter covers 8 of the 12 us)
// behind a chain of five round trips.  Kernel trace, against 16-bit bucket keys found in two 256-bin passes by four waves of 16
// slots per thread, each appending its own head first: 512 pairs of up to 2048 pages, two-pass block
// mean 17.3 -> 12.6 us; 128 pairs of 4096 pages, two-pass Quest 15.9 -> 11.3; 1024 pairs of up to
// 4096 pages, Max 16.9 -> 12.1; 512 pairs of NSA scores 28.7 -> 12.5; 32 pairs of 2048 pages 10.1 ->
// 5.0.
// ------------------------------------------------------------------------------------
constexpr int kMaxUndecided = 1024;
constexpr int kBinRounds = 4;          // histograms of the re-scored kinds at most

// Bins per unit between lo and hi, 0 for an empty or infinite range.  A finite range that overflows
// fp32 is halved first (x - lo may then be infinite: the last bin).
__device__ __forceinline__ float bin_scale(float lo, float hi) {
  const float span = hi - lo;
  const bool fits = span < INFINITY;
  const float scale = (fits ? (float)kBins : (float)(kBins / 2)) / (fits ? span : 0.5f * hi - 0.5f * lo);
  return span > 0.f ? scale : 0.f;
}

// Six waves per SIMD (80 VGPRs) where the re-scoring allows it: the registers the compiler would
// otherwise take for the append workgroups' divisions cost the selection its residency, and a grid
// that is not resident at once leaves the dispatcher in the middle of a round over the CUs, which
// upsets the decode launch's pairing of long and short requests per CU (1024 pairs: decode 36.5 us
// after a selection at four waves per SIMD, 34.2 us at six).  1024 threads are alone on a CU at either;
// the block mean's take four for its batches of four rows, the envelope kinds' were slower so (64
// pairs of up to 8192 blocks with the append, kernel trace: 12.6 against 12.4 us).
template <int RK, int D, int T, int K>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(D > 128 ? 2 : (T > 512 && RK == kMeanDot) || (K > 8 && (T > 256 || RK != kNoRescore)) ? 4 : 6))) void topk_bucket_kernel(const SelArgs a, const AppendStep ap) {
  using S = SelShape<T, K>;
  constexpr bool kMeanRescore = RK == kMeanDot;
  constexpr bool kEnvRescore = is_env(RK);
  constexpr bool kRescore = kMeanRescore || kEnvRescore;
  constexpr int DD = kRescore ? D : 64;                      // shapes of the unused re-scoring parts
  using M = RowMap<DD, false>;                               // fp32 Mean rows
  using ME = RowMap<DD, true>;                               // bf16 Max / Min rows
  constexpr int E = DD / 16;
  // 16-byte query chunks of a group: g <= 16 heads (block mean), g <= 4 (envelope kinds)
  constexpr int kQChunks = kMeanRescore ? 16 * D / 8 : kEnvRescore ? 4 * D / 8 : 1;
  constexpr int kQRounds = (kQChunks + T - 1) / T;
  __shared__ __align__(16) int hist[2][kBins];
  __shared__ uint2 words[S::kWords];              // chosen pages
  __shared__ uint2 eq_words[S::kWords];           // radix select: the pages of the threshold key
  __shared__ uint32_t exact_keys[kRescore ? S::M : 1];   // re-scored keys by page (more than a wave of them)
  __shared__ int und[kRescore ? kMaxUndecided : kWave];  // undecided pages
  __shared__ uint32_t und_key[kWave];             // their exact keys (up to a wave of them)
  __shared__ uint4 qraw[kMeanRescore ? kQChunks : 1];   // the group's bf16 query rows
  __shared__ double qbar[kMeanRescore ? D : 1];   // group-mean query, channel order
  __shared__ float qs[kEnvRescore ? 4 * D : 1];   // the group's query rows, fp32 in row order
  __shared__ int pick[2][3];
  __shared__ uint32_t mm[2][S::W];
  __shared__ int counters[kRescore ? kBinRounds : 1][2];   // of each round: |in|, |undecided|

  const int n_app = ap.app.knew ? a.batch * append_wgs<T>(a.H, ap.D) : 0;
  if ((int)blockIdx.x < n_app) {                  // uniform: an append workgroup
    append_tasks<T, 4>(ap, (int)blockIdx.x, a.H, a.ps, a.r, a.indptr, a.indices, a.seq_lens);
    return;
  }
  const int tid = (int)threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SelRow s = sel_row(a, (int)blockIdx.x - n_app, S::M);
  const int P = s.P, g = a.Hq / a.H;
  auto is_cand = [&](int j) { return !s.all && j >= s.nS && j < P - s.nL; };

  if (s.Kfree > 0) {
    // every prologue load in one round trip: both bound rows and the group's query rows
    const int64_t row = ((int64_t)s.h * a.batch + s.i) * a.stride;
    float lf[K], uf[kRescore ? K : 1];
#pragma unroll
    for (int x = 0; x < K; x++) {
      if (x * T < P) {                               // uniform; lanes past P re-read the last page
        const int j = min(x * T + tid, P - 1);
        lf[x] = a.lower[row + j];
        if constexpr (kRescore) uf[x] = a.upper[row + j];
      }
    }
    const int nq = g * DD / 8;
    uint4 qv[kQRounds];
    if constexpr (kRescore) {
      const uint4* qsrc = reinterpret_cast<const uint4*>(a.q + ((int64_t)s.i * a.Hq + (int64_t)s.h * g) * D);
#pragma unroll
      for (int t = 0; t < kQRounds; t++) qv[t] = qsrc[min(tid + T * t, nq - 1)];
    }
    for (int x = tid; x < 2 * kBins / 4; x += T) reinterpret_cast<int4*>(&hist[0][0])[x] = make_int4(0, 0, 0, 0);
    if (tid < 2 * (kRescore ? kBinRounds : 1)) (&counters[0][0])[tid] = 0;
    uint32_t um = 0;                                 // bit x: the page of slot x is undecided
    SlotWords<T, K> sw;                              // this wave's chosen pages
    float lo_min = INFINITY, hi_max = -INFINITY;
#pragma unroll
    for (int x = 0; x < K; x++) {
      if (x * T < P) {
        const bool cand = is_cand(x * T + tid);
        if (cand) {
          if constexpr (kRescore) um |= 1u << x;
          lo_min = fminf(lo_min, lf[x]);
          if constexpr (kRescore) hi_max = fmaxf(hi_max, uf[x]);
          else hi_max = fmaxf(hi_max, lf[x]);
        }
        if constexpr (kRescore) {
          const int j0 = x * T + kWave * w;          // forced pages are chosen: in words at the row's ends
          if (j0 < s.nS || j0 + kWave > P - s.nL) sw.put(x, __ballot(x * T + tid < P && !cand));   // uniform
        }
      }
    }
    if constexpr (kMeanRescore) {
#pragma unroll
      for (int t = 0; t < kQRounds; t++)
        if (tid + T * t < nq) qraw[tid + T * t] = qv[t];
    } else if constexpr (kEnvRescore) {
      // the envelope scores' query layout: head r, channel c at (r 16 + u) E + e, c the RowMap
      // channel (u, cc, e)
#pragma unroll
      for (int t = 0; t < kQRounds; t++) {
        const int x = tid + T * t;
        if (x < nq) {
          const uint32_t ws[4] = {qv[t].x, qv[t].y, qv[t].z, qv[t].w};
#pragma unroll
          for (int k = 0; k < 8; k++) {
            const int flat = 8 * x + k, rr = flat / D, c = flat - rr * D;
            const int chunk = c / ME::kElemsPerChunk, e_in = c - chunk * ME::kElemsPerChunk;
            qs[(rr * 16 + chunk % 16) * E + (chunk / 16) * ME::kElemsPerChunk + e_in] =
                (k & 1) ? bf16hi(ws[k >> 1]) : bf16lo(ws[k >> 1]);
          }
        }
      }
    }
    // the range over the workgroup, behind a barrier
    auto block_range = [&]() {
      lo_min = wave_min_f32(lo_min);
      hi_max = wave_max_f32(hi_max);
      if (lane == 0) {
        mm[0][w] = __float_as_uint(lo_min);
        mm[1][w] = __float_as_uint(hi_max);
      }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < S::W; x++) {
        lo_min = fminf(lo_min, __uint_as_float(mm[0][x]));
        hi_max = fmaxf(hi_max, __uint_as_float(mm[1][x]));
      }
    };
    block_range();
    if constexpr (kMeanRescore) {
      // group-mean query: fp64 sums in head order, then finish_qbar's division (as one pass)
      const uint16_t* qh = reinterpret_cast<const uint16_t*>(qraw);
      for (int c = tid; c < D; c += T) {
        double acc = 0.0;
        for (int r = 0; r < g; r++) acc += (double)bf16lo(qh[r * D + c]);
        qbar[c] = c < a.qdims ? finish_qbar_one(acc, g) : 0.0;
      }
    }
    // exact scores take one round, which knows the candidates by their pages
    auto pending = [&](int x) -> bool {
      if constexpr (kRescore) return (um >> x) & 1u;
      else return is_cand(x * T + tid);
    };
    int need = s.Kfree, n_und;
#pragma clang loop unroll(disable)
    for (int round = 0;; round++) {
      int Pr = P, ln = lane;
      if constexpr (kRescore) {                      // the slots' tests are made in the round: kept around
        asm volatile("" : "+s"(Pr));                 // the loop they spill
        asm volatile("" : "+v"(ln));
      }
      const float origin = lo_min, scale = bin_scale(lo_min, hi_max);
      // NaN bounds (and any with scale 0) fall into bin 0
      auto bin_of = [&](float x) { return (int)fminf(fmaxf((x - origin) * scale, 0.f), (float)(kBins - 1)); };
      int bl[K], bu[kRescore ? K : 1];
#pragma unroll
      for (int x = 0; x < K; x++) {
        if (x * T < Pr) {
          bl[x] = bin_of(lf[x]);
          if constexpr (kRescore) bu[x] = bin_of(uf[x]);
          if (pending(x)) {
            atomicAdd(&hist[0][bl[x]], 1);
            if constexpr (kRescore) atomicAdd(&hist[1][bu[x]], 1);
          }
        }
      }
      __syncthreads();
      // at least need + 1 undecided pages exist (at first P > K_total)
      if (w == 0) wave_pick_bin(hist[0], need, pick[0]);
      if (w == S::W - 1) wave_pick_bin(hist[kRescore ? 1 : 0], need + 1, pick[1]);
      __syncthreads();
      const int t_lo = pick[0][0];                   // bin of the need-th largest lower bound
      const int t_hi = pick[1][0];                   // bin of the (need + 1)-th largest upper bound
      uint64_t mu[K];                                // this wave's undecided pages of slot x
      int n_in = 0, n_mine = 0;                      // this wave's counts
#pragma unroll
      for (int x = 0; x < K; x++) {
        mu[x] = 0;
        if (x * T < Pr) {
          const bool was = pending(x);
          bool u = bl[x] >= t_lo;
          if constexpr (kRescore) u = bu[x] >= t_lo;
          const bool in = was && bl[x] > t_hi;
          u = u && was && !in;
          if constexpr (kRescore) um = u ? um : um & ~(1u << x);
          else um |= u ? 1u << x : 0u;
          mu[x] = __ballot(u);
          const uint64_t mi = __ballot(in);
          n_in += __popcll(mi);
          n_mine += __popcll(mu[x]);
          if constexpr (kRescore) sw.add(x, mi, ln);
          else sw.put(x, __ballot(in || (x * T + tid < P && !was)));   // forced pages are chosen
        }
      }
      sw.store(words, w, Pr);
      // the undecided list (in any order), and the counts
      int at = 0;
      if (lane == 0) {
        if (n_in) atomicAdd(&counters[round][0], n_in);
        if (n_mine) at = atomicAdd(&counters[round][1], n_mine);
      }
      if (n_mine) {                                  // uniform over the wave
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int x = 0; x < K; x++) {
          if (mu[x]) {
            const int pos = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mu[x] >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)mu[x], 0u));
            if ((um >> x) & 1u) {
              if constexpr (kRescore) {
                if (pos < kMaxUndecided) und[pos] = x * T + tid;
              } else if (pos < kWave) {
                und[pos] = x * T + tid;
                und_key[pos] = float_key(lf[x]);
              }
            }
            at += __popcll(mu[x]);
          }
        }
      }
      __syncthreads();
      need -= counters[round][0];
      n_und = counters[round][1];
      if constexpr (!kRescore) break;
      // Both thresholds in one bin or in neighbours: the bins, not the bounds, leave the pages
      // undecided.
      if (round == kBinRounds - 1 || t_hi - t_lo > 1 || need == 0 || need >= n_und ||
          n_und <= min(kWave, T / 8))                // uniform
        break;
      lo_min = INFINITY;
      hi_max = -INFINITY;
#pragma unroll
      for (int x = 0; x < K; x++) {
        if ((um >> x) & 1u) {
          if (bin_of(lf[x]) == t_lo && fabsf(lf[x]) < INFINITY) {
            lo_min = fminf(lo_min, lf[x]);
            hi_max = fmaxf(hi_max, lf[x]);
          }
          if (bin_of(uf[x]) == t_hi && fabsf(uf[x]) < INFINITY) {
            lo_min = fminf(lo_min, uf[x]);
            hi_max = fmaxf(hi_max, uf[x]);
          }
        }
      }
      for (int x = tid; x < 2 * kBins / 4; x += T) reinterpret_cast<int4*>(&hist[0][0])[x] = make_int4(0, 0, 0, 0);
      block_range();
      if (!(hi_max > lo_min)) break;                 // one value, or none finite: uniform
    }
    if (need > 0 && need >= n_und) {                 // every undecided page is chosen
#pragma unroll
      for (int x = 0; x < K; x++)
        if (x * T < P) sw.add(x, __ballot((um >> x) & 1u));
      sw.store(words, w, P);
    } else if (need > 0) {
      // exact scores of the undecided pages (more than the list holds: of every page): rows of 16
      // lanes, kAt pages per row at a time, the next ones and the page ids after those on their way
      if constexpr (kRescore) {
        constexpr int kRowsT = T / 16, kAt = T > 512 && kMeanRescore ? 4 : 2;
        const bool listed = n_und <= kMaxUndecided;
        const int n_score = listed ? n_und : P;
        const int row16 = tid >> 4, u = tid & 15;
        double qb[kMeanRescore ? E : 1];
        if constexpr (kMeanRescore) {
#pragma unroll
          for (int c = 0; c < M::kChunks; c++)
#pragma unroll
            for (int e = 0; e < 4; e++) qb[4 * c + e] = qbar[M::channel(u, c, e)];
        }
        constexpr int WM = RowWords<DD, !kMeanRescore>::W;
        struct Rows {
          uint32_t a[kAt][WM];                         // Mean / Max rows
          uint32_t b[kAt][needs_min(RK) ? WM : 1];     // Min rows
        };
        // Batch b: pages row16 + (b kAt + v) kRowsT, v < N; past the last page, that page again.
        const int rsh = 31 - __clz(a.r);                           // blocks per page: 1, 2 or 4
        auto page_at = [&](int x) {
          const int y = min(x, n_score - 1), j = und[min(y, kMaxUndecided - 1)];
          return listed ? j : y;
        };
        struct Ids {
          int j[kAt], page[kAt];
        };
        auto load_ids = [&](int b, Ids& id, auto n) {
#pragma unroll
          for (int v = 0; v < decltype(n)::value; v++) {
            id.j[v] = page_at((b * kAt + v) * kRowsT + row16);
            id.page[v] = a.indices[s.base + (id.j[v] >> rsh)];
          }
        };
        auto load_rows = [&](const Ids& id, Rows& pr, auto n) {
#pragma unroll
          for (int v = 0; v < decltype(n)::value; v++) {
            const int64_t block = (clamp_page(id.page[v], a.num_phys) << rsh) + (id.j[v] & (a.r - 1));
            const int64_t at = (block * a.H + s.h) * D;
            if constexpr (kMeanRescore) load_row_words<DD, false>(a.mean + at, u, pr.a[v]);
            else load_row_words<DD, true>(a.maxs + at, u, pr.a[v]);
            if constexpr (needs_min(RK)) load_row_words<DD, true>(a.mins + at, u, pr.b[v]);
          }
        };
        auto score = [&](int b, const Rows& pr, auto n) {
#pragma unroll
          for (int v = 0; v < decltype(n)::value; v++) {
            float sc;
            if constexpr (kMeanRescore) sc = exact_row_score<DD, false>(qb, pr.a[v]);
            else if constexpr (needs_min(RK)) sc = (float)env_exact<RK, DD>(qs, 0, g, u, pr.a[v], pr.b[v]);
            else sc = (float)env_exact<RK, DD>(qs, 0, g, u, pr.a[v], pr.a[v]);
            const int x = (b * kAt + v) * kRowsT + row16;
            if (u == 0 && x < n_score) {
              if (n_und <= kWave) und_key[x] = float_key(sc);
              else exact_keys[page_at(x)] = float_key(sc);         // decided pages' keys are never read
            }
          }
        };
        const int batches = (n_score + kAt * kRowsT - 1) / (kAt * kRowsT);   // uniform
        if (n_score <= 2 * kRowsT) {                               // uniform: all at once
          auto once = [&](auto n) {
            if (row16 < n_score) {                                 // waves without a page have no work
              Ids id;
              Rows ra;
              load_ids(0, id, n);
              load_rows(id, ra, n);
              score(0, ra, n);
            }
          };
          if (n_score <= kRowsT) once(std::integral_constant<int, 1>{});
          else once(std::integral_constant<int, 2>{});
        } else {
          Ids id;
          Rows ra, rb;
          using All = std::integral_constant<int, kAt>;
          load_ids(0, id, All{});
          load_rows(id, ra, All{});
          load_ids(1, id, All{});
          for (int b = 0;; b += 2) {                               // uniform
            if (b + 1 < batches) load_rows(id, rb, All{});
            if (b + 2 < batches) load_ids(b + 2, id, All{});
            score(b, ra, All{});
            if (b + 1 >= batches) break;
            if (b + 2 < batches) load_rows(id, ra, All{});
            if (b + 3 < batches) load_ids(b + 3, id, All{});
            score(b + 1, rb, All{});
            if (b + 2 >= batches) break;
          }
        }
        __syncthreads();
      }
      if (n_und <= kWave) {
        // rank among the undecided by (key desc, page asc); the best `need` are chosen
        if (w == 0) {
          // composite (key, ~page): larger is better; the others' composites come as LDS
          // broadcasts, four per step, so the loads of a step are in flight together
          const bool mine = lane < n_und;
          const int jx = mine ? und[lane] : 0;
          const uint64_t cx = mine ? ((uint64_t)und_key[lane] << 32) | (uint32_t)~jx : 0ull;
          auto comp = [&](int y) { return ((uint64_t)und_key[y] << 32) | (uint32_t)~und[y]; };
          int rank = 0;
          int y = 0;
          for (; y + 4 <= n_und; y += 4) {
            const uint64_t c0 = comp(y), c1 = comp(y + 1), c2 = comp(y + 2), c3 = comp(y + 3);
            rank += (c0 > cx) + (c1 > cx) + (c2 > cx) + (c3 > cx);
          }
          for (; y < n_und; y++) rank += comp(y) > cx;
          if (mine && rank < need)
            atomicOr(reinterpret_cast<unsigned int*>(words) + (jx >> 5), 1u << (jx & 31));
        }
      } else {
        // radix select over the exact keys of the undecided pages, 10-bit digits from the highest
        // bit in which the extreme keys differ
        uint32_t ke[K];
        uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
        for (int x = 0; x < K; x++) {
          ke[x] = 0u;
          if ((um >> x) & 1u) {
            if constexpr (kRescore) ke[x] = exact_keys[x * T + tid];
            else ke[x] = float_key(lf[x]);
            kmin = min(kmin, ke[x]);
            kmax = max(kmax, ke[x]);
          }
        }
        kmin = wave_min_u32(kmin);
        kmax = wave_max_u32(kmax);
        if (lane == 0) {
          mm[0][w] = kmin;
          mm[1][w] = kmax;
        }
        for (int x = tid; x < kBins / 4; x += T) reinterpret_cast<int4*>(&hist[0][0])[x] = make_int4(0, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int x = 0; x < S::W; x++) {
          kmin = min(kmin, mm[0][x]);
          kmax = max(kmax, mm[1][x]);
        }
        RadixState rs = radix_init(kmin, kmax, need);
        int hb = 0;
        while (rs.top >= 0) {                        // uniform
          const int sh = radix_shift<10>(rs);
          const uint32_t dm = radix_dmask<10>(rs);
          for (int x = tid; x < kBins / 4; x += T)
            reinterpret_cast<int4*>(&hist[hb ^ 1][0])[x] = make_int4(0, 0, 0, 0);
#pragma unroll
          for (int x = 0; x < K; x++)
            if (((um >> x) & 1u) && (ke[x] & rs.pmask) == rs.prefix) atomicAdd(&hist[hb][(ke[x] >> sh) & dm], 1);
          __syncthreads();
          if (w == 0) wave_pick_bin(hist[hb], rs.remaining, pick[hb]);
          __syncthreads();
          radix_advance<10>(rs, pick[hb]);
          if (pick[hb][2] == rs.remaining) break;    // every key with this prefix is chosen
          hb ^= 1;
        }
        // above the threshold prefix: chosen; equal to it: the `remaining` lowest pages
#pragma unroll
        for (int x = 0; x < K; x++) {
          if (x * T < P) {
            const bool u = (um >> x) & 1u;
            const uint32_t mk = ke[x] & rs.pmask;
            const uint64_t gt = __ballot(u && mk > rs.prefix), eq = __ballot(u && mk == rs.prefix);
            if (lane == 0) {
              uint2& v = words[x * S::W + w];
              v = make_uint2(v.x | (uint32_t)gt, v.y | (uint32_t)(gt >> 32));
              eq_words[x * S::W + w] = word_of(eq);
            }
          }
        }
        __syncthreads();
        WordPrefix<T, K> ep;
        ep.load(eq_words, (P + T - 1) / T * S::W);
#pragma unroll
        for (int x = 0; x < K; x++) {
          if (x * T < P) {
            int rank;
            const bool e = ep.at(x, w, rank);
            const uint64_t m = __ballot(e && rank < rs.remaining);
            if (m && lane == 0) {
              uint2& v = words[x * S::W + w];
              v = make_uint2(v.x | (uint32_t)m, v.y | (uint32_t)(m >> 32));
            }
          }
        }
      }
    }
  } else {
    // every page, or the forced pages alone
    SlotWords<T, K> sw;
#pragma unroll
    for (int x = 0; x < K; x++) {
      if (x * T < P) {
        const int j = x * T + tid;
        sw.put(x, __ballot(j < P && !is_cand(j)));
      }
    }
    sw.store(words, w, P);
  }
  __syncthreads();
  write_selection<T, K>(a, s, words, w);
}

// ------------------------------------------------------------------------------------
// The radix selection with its options (TopkOptions; the approximate top-k and the remapped keys)
// on the same page slots.  The options define their result by 8-bit passes from the highest bit
// in which the candidates' extreme keys differ, so the passes stay; each costs one barrier: three
// histograms rotate (one filling, the next one cleared, the last one possibly still being read)
// and every wave finds the threshold bin for itself.  Latency-bound like the bucketed selection.
// Measured against 256 threads holding 32 contiguous pages each, one wave picking per pass behind a
// second barrier: 128 rows of 6000 to 8192 scores, remapped, tau 0.2, 25.5 -> 11.3 us a call; 37 rows
// of up to 3000 scores 19.3 -> 8.8.
// ------------------------------------------------------------------------------------
template <int T, int K>
__device__ __forceinline__ void radix_select_slots(const SelArgs a, const SelRow s, const TopkOptions opt) {
  using S = SelShape<T, K>;
  __shared__ __align__(16) int hist[3][256];
  __shared__ uint2 words[S::kWords];              // chosen pages
  __shared__ uint2 eq_words[S::kWords];           // pages of the tie class
  __shared__ uint32_t mm[2][S::W];
  const int tid = (int)threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = s.P;
  auto is_cand = [&](int j) { return !s.all && j >= s.nS && j < P - s.nL; };
  SlotWords<T, K> sw;
  if (s.Kfree > 0) {
    const float* row = a.lower + ((int64_t)s.h * a.batch + s.i) * a.stride;
    float sv[K];
#pragma unroll
    for (int x = 0; x < K; x++)
      if (x * T < P) sv[x] = row[min(x * T + tid, P - 1)];       // all loads issued before any use
    if (tid < kWave) *reinterpret_cast<int4*>(&hist[0][4 * tid]) = make_int4(0, 0, 0, 0);
    // Threshold prefix: a candidate is chosen when (key & pmask) > prefix, or when it equals the
    // prefix and its rank among equals (by page; after an early stop by (h8 desc, page)) is below
    // `remaining`.
    uint32_t key[K], kmin, kmax;
    if (opt.remap != 0) {
      // the candidates' score range (NaN excluded) fixes the affine map; NaN and the smallest
      // candidate both map to 0
      float mn = INFINITY, mx = -INFINITY;
#pragma unroll
      for (int x = 0; x < K; x++) {
        if (x * T < P && is_cand(x * T + tid) && sv[x] == sv[x]) {
          mn = fminf(mn, sv[x]);
          mx = fmaxf(mx, sv[x]);
        }
      }
      mn = wave_min_f32(mn);
      mx = wave_max_f32(mx);
      if (lane == 0) {
        mm[0][w] = __float_as_uint(mn);
        mm[1][w] = __float_as_uint(mx);
      }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < S::W; x++) {
        mn = fminf(mn, __uint_as_float(mm[0][x]));
        mx = fmaxf(mx, __uint_as_float(mm[1][x]));
      }
      const double rmin = (double)mn, rscale = mx > mn ? 4294967295.0 / ((double)mx - (double)mn) : 0.0;
      auto make_key = [&](float x) -> uint32_t {
        if (x != x) return 0u;
        return (uint32_t)fmin(fmax(floor(((double)x - rmin) * rscale), 0.0), 4294967295.0);
      };
#pragma unroll
      for (int x = 0; x < K; x++)
        if (x * T < P) key[x] = make_key(sv[x]);
      kmin = 0u;
      kmax = mx >= mn ? make_key(mx) : 0u;
    } else {
      kmin = 0xffffffffu;
      kmax = 0u;
#pragma unroll
      for (int x = 0; x < K; x++) {
        if (x * T < P) {
          key[x] = float_key(sv[x]);
          if (is_cand(x * T + tid)) {
            kmin = min(kmin, key[x]);
            kmax = max(kmax, key[x]);
          }
        }
      }
      kmin = wave_min_u32(kmin);
      kmax = wave_max_u32(kmax);
      if (lane == 0) {
        mm[0][w] = kmin;
        mm[1][w] = kmax;
      }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < S::W; x++) {
        kmin = min(kmin, mm[0][x]);
        kmax = max(kmax, mm[1][x]);
      }
    }
    // Every wave: the bin of histogram hb that holds the rs.remaining-th largest digit (lane l owns
    // the bins 255 - 4l .. 252 - 4l), the count above it and its own count.
    RadixState rs = radix_init(kmin, kmax, s.Kfree);
    int pk[3];
    auto pick_bin = [&](int hb) {
      const int4 v = *reinterpret_cast<const int4*>(&hist[hb][252 - 4 * lane]);
      const int c[4] = {v.w, v.z, v.y, v.x};
      const int tot = (v.x + v.y) + (v.z + v.w);
      int above = wave_incl_sum(tot) - tot, bin = -1, bin_above = 0, bin_n = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (above < rs.remaining && above + c[e] >= rs.remaining) {
          bin = 255 - 4 * lane - e;
          bin_above = above;
          bin_n = c[e];
        }
        above += c[e];
      }
      const int src = __builtin_ctzll(__ballot(bin >= 0));       // one lane
      pk[0] = __builtin_amdgcn_readlane(bin, src);
      pk[1] = __builtin_amdgcn_readlane(bin_above, src);
      pk[2] = __builtin_amdgcn_readlane(bin_n, src);
    };
    int hb = 0, certain = 0;
    int hthr = -1;                                   // stopped early: hash threshold h8
    const uint32_t hz = lowbias32(opt.seed ^ lowbias32((uint32_t)(s.i * a.H + s.h)));
    auto h8 = [&](int j) { return (int)(lowbias32(hz ^ (uint32_t)j) >> 24); };
    bool whole = false;                              // the whole tie class is chosen
    while (rs.top >= 0) {                            // uniform
      const int sh = radix_shift<8>(rs), nb = hb == 2 ? 0 : hb + 1;
      const uint32_t dm = radix_dmask<8>(rs);
      if (tid < kWave) *reinterpret_cast<int4*>(&hist[nb][4 * tid]) = make_int4(0, 0, 0, 0);
#pragma unroll
      for (int x = 0; x < K; x++)
        if (x * T < P && is_cand(x * T + tid) && (key[x] & rs.pmask) == rs.prefix)
          atomicAdd(&hist[hb][(key[x] >> sh) & dm], 1);
      __syncthreads();
      pick_bin(hb);
      radix_advance<8>(rs, pk);
      certain += pk[1];
      whole = pk[2] == rs.remaining;
      if (whole) break;
      hb = nb;
      if (rs.top >= 0 && (int64_t)certain * 65536 >= (int64_t)(65536 - opt.tau_q) * s.Kfree) {
        // early termination: one pass over the threshold bin's hashes orders the rest at random
#pragma unroll
        for (int x = 0; x < K; x++) {
          const int j = x * T + tid;
          if (x * T < P && is_cand(j) && (key[x] & rs.pmask) == rs.prefix) atomicAdd(&hist[hb][h8(j)], 1);
        }
        __syncthreads();
        pick_bin(hb);
        rs.remaining -= pk[1];
        hthr = pk[0];
        whole = pk[2] == rs.remaining;
        break;
      }
    }
    SlotWords<T, K> ew;
#pragma unroll
    for (int x = 0; x < K; x++) {
      if (x * T < P) {
        const int j = x * T + tid;
        const bool cand = is_cand(j);
        const uint32_t mk = key[x] & rs.pmask;
        bool eq = cand && mk == rs.prefix, in = cand && mk > rs.prefix;
        if (hthr >= 0) {                             // uniform
          const int hv = h8(j);
          in = in || (eq && hv > hthr);
          eq = eq && hv == hthr;
        }
        sw.put(x, __ballot(in || (whole && eq) || (j < P && !cand)));
        ew.put(x, __ballot(eq));
      }
    }
    if (!whole) {                                    // the tie class's `remaining` lowest pages
      ew.store(eq_words, w, P);
      __syncthreads();
      WordPrefix<T, K> ep;
      ep.load(eq_words, (P + T - 1) / T * S::W);
#pragma unroll
      for (int x = 0; x < K; x++) {
        if (x * T < P) {
          int rank;
          const bool e = ep.at(x, w, rank);
          sw.add(x, __ballot(e && rank < rs.remaining));
        }
      }
    }
  } else {
    // every page, or the forced pages alone
#pragma unroll
    for (int x = 0; x < K; x++) {
      if (x * T < P) {
        const int j = x * T + tid;
        sw.put(x, __ballot(j < P && !is_cand(j)));
      }
    }
  }
  sw.store(words, w, P);
  __syncthreads();
  write_selection<T, K>(a, s, words, w);
}

template <int T, int K>
__global__ __launch_bounds__(T) void topk_radix_kernel(const SelArgs a, const TopkOptions opt) {
  radix_select_slots<T, K>(a, sel_row(a, (int)blockIdx.x, T * K), opt);
}

// ------------------------------------------------------------------------------------
// The radix selection past the page slots.  Thread t owns the contiguous pages [t*R, t*R + R),
// R = ceil(P / kThreads), and every pass recomputes their keys from the scores (L2-resident after
// the first read).
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void radix_select_long(const SelArgs& a, const SelRow& row, const TopkOptions& opt) {
  __shared__ int hist[2][256];
  __shared__ int wave_tot[kThreads / kWave];
  __shared__ uint32_t wave_mm[2][kThreads / kWave];
  __shared__ float wave_fm[2][kThreads / kWave];
  __shared__ int pick[2][3];           // digit, count above the digit's bin, bin count

  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int i = row.i, h = row.h, P = row.P, nS = row.nS, nL = row.nL, Kfree = row.Kfree, max_sel = a.max_sel;
  const bool all = row.all;
  const float* s = a.lower + ((int64_t)h * a.batch + i) * a.stride;
  int32_t* out = row.out;
  const int R = (P + kThreads - 1) / kThreads;
  const int j_lo = min(P, tid * R), n_mine = min(P, j_lo + R) - j_lo;

  double rmin = 0.0, rscale = 0.0;                       // remap 1: min and scale of the affine map
  auto make_key = [&](float x) -> uint32_t {
    if (opt.remap == 0) return float_key(x);
    if (x != x) return 0u;
    // in [0, 2^32 - 1] for candidates; forced pages (never ranked) may fall outside: clamp
    return (uint32_t)fmin(fmax(floor(((double)x - rmin) * rscale), 0.0), 4294967295.0);
  };
  // f(j, key) for every candidate of this thread
  auto each_candidate = [&](auto&& f) {
    for (int j = j_lo; j < j_lo + n_mine; j++)
      if (!is_forced(j, P, nS, nL)) f(j, make_key(s[j]));
  };
  // Radix select over the candidates' keys.  Threshold prefix: a candidate is chosen when
  // (key & pmask) > prefix, or when it equals the prefix and its rank among equals (by page
  // index; after an early stop by (h8 desc, page)) is below `remaining`.
  uint32_t prefix = 0, pmask = 0;
  int remaining = Kfree;
  int hthr = -1;                                         // stopped early: hash threshold h8
  uint32_t hz = 0;                                       // hash salt z of this (request, head)
  // Wave 0 finds the bin of histogram hb holding the remaining-th largest digit (lane l owns
  // bins 255-4l .. 252-4l, descending): pick[hb] = {bin, count above it, bin count}.
  auto pick_bin = [&](int hb) {
    if (w == 0) {
      int c[4], tot = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        c[e] = hist[hb][255 - 4 * lane - e];
        tot += c[e];
      }
      int above = wave_incl_sum(tot) - tot;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (above < remaining && above + c[e] >= remaining) {
          pick[hb][0] = 255 - 4 * lane - e;
          pick[hb][1] = above;
          pick[hb][2] = c[e];
        }
        above += c[e];
      }
    }
    __syncthreads();
  };
  if (Kfree > 0) {
    if (opt.remap != 0) {
      // the candidates' score range (NaN excluded) fixes the affine map
      float fmn = INFINITY, fmx = -INFINITY;
      for (int j = j_lo; j < j_lo + n_mine; j++) {
        const float x = s[j];
        if (!is_forced(j, P, nS, nL) && x == x) {
          fmn = fminf(fmn, x);
          fmx = fmaxf(fmx, x);
        }
      }
      block_fminmax(fmn, fmx, wave_fm);
      rmin = (double)fmn;
      rscale = fmx > fmn ? 4294967295.0 / ((double)fmx - (double)fmn) : 0.0;
    }
    // bits above the highest bit where the smallest and largest candidate key differ are
    // common to every candidate and need no pass
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    each_candidate([&](int, uint32_t key) {
      kmin = min(kmin, key);
      kmax = max(kmax, key);
    });
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) {
      wave_mm[0][w] = kmin;
      wave_mm[1][w] = kmax;
    }
    hist[0][tid] = 0;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < kThreads / kWave; x++) {
      kmin = min(kmin, wave_mm[0][x]);
      kmax = max(kmax, wave_mm[1][x]);
    }
    const uint32_t diff = kmin ^ kmax;
    int top = diff ? 31 - __clz((int)diff) : -1;           // highest differing bit
    pmask = top >= 31 ? 0u : ~((2u << top) - 1u);           // common high bits
    if (top < 0) pmask = 0xffffffffu;                        // all candidate keys equal
    prefix = kmin & pmask;

    int hb = 0, certain = 0;
    while (top >= 0) {
      const int shift = top >= 7 ? top - 7 : 0;
      const uint32_t dmask = (1u << (top - shift + 1)) - 1u;   // 1..8 bits
      hist[hb ^ 1][tid] = 0;                                   // next pass's histogram
      each_candidate([&](int, uint32_t key) {
        if ((key & pmask) == prefix) atomicAdd(&hist[hb][(key >> shift) & dmask], 1);
      });
      __syncthreads();
      pick_bin(hb);
      remaining -= pick[hb][1];
      certain += pick[hb][1];
      prefix |= (uint32_t)pick[hb][0] << shift;
      pmask |= dmask << shift;
      const bool done = pick[hb][2] == remaining;   // every key with this prefix is chosen
      top = shift - 1;
      hb ^= 1;
      if (done) break;
      if (top >= 0 && (int64_t)certain * 65536 >= (int64_t)(65536 - opt.tau_q) * Kfree) {
        // early termination: one pass over the threshold bin's hashes (histogram hb was
        // cleared during the last pass) orders the rest at random
        hz = lowbias32(opt.seed ^ lowbias32((uint32_t)(i * a.H + h)));
        each_candidate([&](int j, uint32_t key) {
          if ((key & pmask) == prefix) atomicAdd(&hist[hb][lowbias32(hz ^ (uint32_t)j) >> 24], 1);
        });
        __syncthreads();
        pick_bin(hb);
        remaining -= pick[hb][1];
        hthr = pick[hb][0];
        break;
      }
    }
  }

  // Compaction: one scan gives each tied candidate its rank by page index, a second gives each
  // chosen page its slot.
  // After an early stop a bin member ranks above the tie class by its hash, else ties.
  auto hash_cmp = [&](int j) -> int {
    if (hthr < 0) return 0;
    const int hv = (int)(lowbias32(hz ^ (uint32_t)j) >> 24);
    return (hv > hthr) - (hv < hthr);
  };
  int n_eq = 0;
  if (Kfree > 0) {
    each_candidate([&](int j, uint32_t key) { n_eq += (key & pmask) == prefix && hash_cmp(j) == 0; });
  }
  int tot_eq;
  const int eq_rank = block_incl_scan(n_eq, wave_tot, &tot_eq) - n_eq;
  // the tie class's chosen members are its `remaining` lowest page indices
  auto chosen_at = [&](int j, uint32_t key, int& r) -> bool {
    if (all || is_forced(j, P, nS, nL)) return true;
    if (Kfree <= 0) return false;
    const uint32_t mk = key & pmask;
    if (mk != prefix) return mk > prefix;
    const int hc = hash_cmp(j);
    if (hc != 0) return hc > 0;
    const bool in = r < remaining;
    r++;
    return in;
  };
  int n_chosen = 0;
  {
    int r = eq_rank;
    for (int j = j_lo; j < j_lo + n_mine; j++) n_chosen += chosen_at(j, Kfree > 0 ? make_key(s[j]) : 0u, r);
  }
  int tot_sel;
  int pos = block_incl_scan(n_chosen, wave_tot, &tot_sel) - n_chosen;
  {
    int r = eq_rank;
    for (int j = j_lo; j < j_lo + n_mine; j++) {
      if (chosen_at(j, Kfree > 0 ? make_key(s[j]) : 0u, r)) {
        if (pos < max_sel) out[pos] = j;
        pos++;
      }
    }
  }
  for (int m = tot_sel + tid; m < max_sel; m += kThreads) out[m] = -1;
  if (h == 0 && tid == 0) a.sel_count[i] = min(tot_sel, max_sel);
}

// Requests of more than kTwoPassMaxPages blocks at the bound.  The bound is often a model's limit and
// the row far shorter, so a row that fits page slots still takes them.  Rows of up to 8192 / 2000 / 500
// scores in strides of 20000 / 20000 / 17000 (128 / 512 / 1024 pairs, exact): 59.2 / 18.2 / 8.8 us read
// again in each pass, 20.0 / 8.9 / 7.5 in slots; with 32 slots for all of them 20.7 / 14.3 / 15.7.
__global__ __launch_bounds__(kThreads) void topk_long_kernel(const SelArgs a, const TopkOptions opt) {
  const SelRow row = sel_row(a, (int)blockIdx.x, 1 << 30);
  if (row.P <= 8 * kThreads) radix_select_slots<kThreads, 8>(a, row, opt);               // uniform
  else if (row.P <= 32 * kThreads) radix_select_slots<kThreads, 32>(a, row, opt);
  else radix_select_long(a, row, opt);
}

// The same exact one-pass selection for requests of at most kWaveMaxPages blocks, by one wave per
// (request, KV head) and without workgroup barriers: lane l holds the score keys of blocks
// 8l .. 8l + 7, an MSB-first radix select over 8-bit digits (a 256-bin LDS histogram per pass,
// starting below the bits that every candidate key shares) finds the K_free-th largest
// candidate key, and a prefix over the lanes, which hold the blocks in ascending order, places
// the equal keys by block index and compacts the chosen blocks.  The decode step's append runs in
// workgroups of its own ahead of the selection's.
constexpr int kWaveMaxPages = 512;
constexpr int kWaveKeys = kWaveMaxPages / kWave;   // keys per lane

__device__ __forceinline__ int wave_excl_scan(int x, int* total) {
  const int incl = wave_incl_sum(x);
  *total = (int)wave_last((uint32_t)incl);
  return incl - x;
}

__global__ __launch_bounds__(kWave) void topk_wave_kernel(
    const float* __restrict__ scores, int H, int ps, int r, int max_pages, int stride, int batch,
    const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ budget, int n_sink, int n_local, int max_sel, int32_t* __restrict__ sel_pages,
    int32_t* __restrict__ sel_count, const AppendStep ap) {
  __shared__ __align__(16) int hist[256];
  const int n_app = ap.app.knew ? batch * append_wgs<kWave>(H, ap.D) : 0;
  if ((int)blockIdx.x < n_app) {           // uniform: an append workgroup
    // blocks of 64 tokens: a lane's 16 rows in one round trip, as in the append launch
    if (ps > 4 * summ::kBatch) append_tasks<kWave, 2 * summ::kBatch>(ap, (int)blockIdx.x, H, ps, r, indptr, indices, seq_lens);
    else append_tasks<kWave, summ::kBatch>(ap, (int)blockIdx.x, H, ps, r, indptr, indices, seq_lens);
    return;
  }
  const int lane = lane_id();
  const int pair = (int)blockIdx.x - n_app;
  const int i = pair / H, h = pair - i * H;
  // the score row loads with the request's geometry: lane l reads blocks 8l .. 8l + 7, clamped
  // into the row (stride >= 4 floats; entries past the request's blocks are never used)
  const float* row = scores + ((int64_t)h * batch + i) * stride;
  const float4 sa = *reinterpret_cast<const float4*>(row + min(kWaveKeys * lane, stride - 4));
  const float4 sb = *reinterpret_cast<const float4*>(row + min(kWaveKeys * lane + 4, stride - 4));
  const int base = indptr[i];
  const int P = num_pages(seq_lens[i], ps, (indptr[i + 1] - base) * r, min(max_pages, kWaveMaxPages));
  int Ktot = budget[i];
  Ktot = Ktot < max_sel ? Ktot : max_sel;
  Ktot = Ktot < 0 ? 0 : Ktot;
  int32_t* out = sel_pages + ((int64_t)i * H + h) * max_sel;
  const bool all = Ktot >= P;
  const int nS = min(n_sink, P), nL = min(n_local, P);
  const int nF = all ? P : nS + nL - max(0, nS - (P - nL));
  const int Kfree = all ? 0 : max(0, Ktot - nF);

  uint32_t key[kWaveKeys];
  uint32_t cand = 0;                       // bit x: block 8 lane + x is a candidate
  uint32_t kth = 0;                        // the K_free-th largest candidate key
  if (Kfree > 0) {                         // then P > Ktot >= 1
    const float f[kWaveKeys] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int x = 0; x < kWaveKeys; x++) {
      const int j = kWaveKeys * lane + x;
      key[x] = float_key(f[x]);
      if (j < P && !is_forced(j, P, nS, nL)) {
        cand |= 1u << x;
        kmin = min(kmin, key[x]);
        kmax = max(kmax, key[x]);
      }
    }
    RadixState s = radix_init(wave_min_u32(kmin), wave_max_u32(kmax), Kfree);
    while (s.top >= 0) {                   // uniform over the wave
      const int sh = radix_shift<8>(s);
      const uint32_t dm = radix_dmask<8>(s);
      *reinterpret_cast<int4*>(&hist[4 * lane]) = make_int4(0, 0, 0, 0);
      __syncthreads();
#pragma unroll
      for (int x = 0; x < kWaveKeys; x++)
        if (((cand >> x) & 1u) && (key[x] & s.pmask) == s.prefix) atomicAdd(&hist[(key[x] >> sh) & dm], 1);
      __syncthreads();
      // the bin that holds the remaining-th largest key (lane l: bins 255-4l .. 252-4l), found by
      // exactly one lane and read from its registers
      int c[4], tot = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        c[e] = hist[255 - 4 * lane - e];
        tot += c[e];
      }
      int above = wave_incl_sum(tot) - tot, bin = -1, bin_above = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (above < s.remaining && above + c[e] >= s.remaining) {
          bin = 255 - 4 * lane - e;
          bin_above = above;
        }
        above += c[e];
      }
      const int src = __builtin_ctzll(__ballot(bin >= 0));
      const int pk[2] = {__builtin_amdgcn_readlane(bin, src), __builtin_amdgcn_readlane(bin_above, src)};
      radix_advance<8>(s, pk);
      __syncthreads();                     // the histogram read before the next pass clears it
    }
    kth = s.prefix;
  }
  // candidates above the K_free-th key are in; equal keys go in by block order
  int n_gt = 0, n_eq = 0;
#pragma unroll
  for (int x = 0; x < kWaveKeys; x++) {
    if ((cand >> x) & 1u) {
      n_gt += key[x] > kth;
      n_eq += key[x] == kth;
    }
  }
  int tot_gt, tot_eq;
  wave_excl_scan(n_gt, &tot_gt);
  int eq_rank = wave_excl_scan(n_eq, &tot_eq);
  uint32_t chosen = 0;
#pragma unroll
  for (int x = 0; x < kWaveKeys; x++) {
    const int j = kWaveKeys * lane + x;
    bool c = false;
    if ((cand >> x) & 1u) c = key[x] > kth || (key[x] == kth && eq_rank++ < Kfree - tot_gt);
    else if (j < P) c = all || is_forced(j, P, nS, nL);
    chosen |= (uint32_t)c << x;
  }
  int tot_sel;
  int pos = wave_excl_scan(__popc(chosen), &tot_sel);
#pragma unroll
  for (int x = 0; x < kWaveKeys; x++) {
    if ((chosen >> x) & 1u) {
      if (pos < max_sel) out[pos] = kWaveKeys * lane + x;
      pos++;
    }
  }
  for (int m = tot_sel + lane; m < max_sel; m += kWave) out[m] = -1;
  if (h == 0 && lane == 0) sel_count[i] = min(tot_sel, max_sel);
}

// ------------------------------------------------------------------------------------
// Score flows over the operator table's Softmax, Conv1d and Sum, one workgroup per (request,
// KV head), in fp64 with one rounding to fp32:
//   NSA (its block top-k flow, Sec. 3.2: softmax, convolution, head sum, then top-K): for each query
//     head r of the group, p_rj = exp(z_rj - m_r) / l_r, the softmax over the request's pages of
//     the fp32 logits z_r (m_r their max, l_r = sum_j exp(z_rj - m_r), divided through the fp64
//     reciprocal of l_r); then the conv below; then the sum over the group's heads, in head order.
//   positional smoothing (Appendix G): the conv of the block-mean scores.
// Conv1d along the pages with taps (1/4, 1/2, 1/4) and zero padding:
//   y_j = x_{j-1} / 4 + x_j / 2 + x_{j+1} / 4,  x_{-1} = x_P = 0.
// in: [rows][batch][stride] (NSA: a row per query head; smoothing: a row per KV head).
// out: [H][batch][stride].
// ------------------------------------------------------------------------------------
constexpr int kFlowTile = 2048;      // pages of a row whose exponentials are in LDS at a time

__device__ __forceinline__ double conv3(double left, double mid, double right) {
  return 0.25 * left + 0.5 * mid + 0.25 * right;
}

// Sum over the wave; every lane receives it.
__device__ __forceinline__ double wave_sum_f64(double x) {
  x = row16_sum_f64(x);
  x += __shfl_xor(x, 16, kWave);
  x += __shfl_xor(x, 32, kWave);
  return x;
}

// NSA: the waves take four query heads of the group at a time, one each, so a head's max and sum are
// wave reductions; where a round has two heads or one, two or four waves share a head's row (kShare: the
// log2 of the waves per head of every round, -1: by the round) and join their max and sum in LDS.  The
// exponentials of the round's heads (a row of up to kTile pages, longer rows tile by tile, with the two
// neighbours) meet in LDS, where every thread convolves and sums its pages' heads.  Two barriers per
// four heads where one workgroup per head row needed six each: the kernel waits on its chain of barriers
// and fp64 exponentials, and on the waves in flight, so kTile follows the request bound (a row of 2048
// pages in registers takes 208 of them) and the LDS the group.  Measured, us with all threads on one head
// after the other / one wave per head always, 2048 pages at most / now: 512 rows of 2048 pages in groups of
// 1: 7.4 / 10.0 / 6.5, of 4: 20.1 / 13.7 / 13.6, of 5: 24.1 / 20.5 / 18.0; 1600 rows of 600 pages in groups of
// 1: 7.4 / 22.6 / 7.0, of 4: 18.5 / 25.3 / 13.5; 128 rows of 8192 pages (16 loads of a lane in flight, where it
// had one) in groups of 1: 31.8 / 61.9 / 19.1, of 4: 110 / 75.8 / 54.8.
template <bool kNsa, int kTile, int kShare>
__global__ __launch_bounds__(kThreads) void flow_kernel(const float* __restrict__ in, float* __restrict__ out, int H,
                                                        int g, int ps, int r, int max_pages, int stride, int batch,
                                                        const int32_t* __restrict__ indptr,
                                                        const int32_t* __restrict__ seq_lens,
                                                        const int32_t* __restrict__ items) {
  constexpr int W = kThreads / kWave;
  extern __shared__ double e_lds[];                  // NSA: [min(g, W)][row], row = tile + 2: e_j at 1 + j - tile start
  __shared__ double inv_of[16];
  __shared__ float max_of[16];
  __shared__ double part_sum[W];
  __shared__ float part_max[W];
  const int tid = threadIdx.x;
  const int i = blockIdx.x / H, h = blockIdx.x % H;
  const int P = items ? max(0, min(items[i], stride))
                      : num_pages(seq_lens[i], ps, (indptr[i + 1] - indptr[i]) * r, max_pages);
  float* y = out + ((int64_t)h * batch + i) * stride;
  if constexpr (!kNsa) {
    const float* x = in + ((int64_t)h * batch + i) * stride;
    for (int j = tid; j < P; j += kThreads) {
      const double left = j > 0 ? (double)x[j - 1] : 0.0;
      const double right = j + 1 < P ? (double)x[j + 1] : 0.0;
      y[j] = (float)conv3(left, (double)x[j], right);
    }
    return;
  }
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = min(max_pages, kTile), row = tile + 2;
  const bool staged = P <= tile;                     // uniform: one tile, its sums taken on the way
  auto logits = [&](int rr) { return in + ((int64_t)(h * g + rr) * batch + i) * stride; };
  // A round of n heads: 1 << sh waves share a head's row, 64 pages by 64 pages in turn.
  auto share = [&](int n) { return kShare >= 0 ? kShare : n >= 3 ? 0 : n == 2 ? 1 : 2; };
  constexpr int kRound = kTile / kWave >> (kShare > 0 ? kShare : 0);   // a wave's pages of a staged row, by lanes
  // the max or sum of a head from its waves' parts (behind a barrier when they are several)
  auto joint = [&](auto x, auto* part, int sh, auto op) {
    if (sh == 0) return x;                           // uniform
    if (lane == 0) part[w] = x;
    __syncthreads();
    const int w0 = w >> sh << sh;
    x = part[w0];
    for (int k = 1; k < 1 << sh; k++) x = op(x, part[w0 + k]);
    __syncthreads();                                 // part free
    return x;
  };
  auto max_op = [](float a, float b) { return fmaxf(a, b); };
  auto sum_op = [](double a, double b) { return a + b; };
  if (!staged) {
    for (int r0 = 0; r0 < g; r0 += W) {
      const int sh = share(g - r0), rr = r0 + (w >> sh), part = w & ((1 << sh) - 1);
      const bool mine = rr < g;                      // uniform over the wave
      const float* z = logits(mine ? rr : 0);
      const int step = kWave << sh;
      constexpr int N = 16;                          // loads in flight
      float mx = -INFINITY;
      if (mine)
        for (int j0 = part * kWave + lane; j0 < P; j0 += N * step) {
          float v[N];
#pragma unroll
          for (int x = 0; x < N; x++) v[x] = z[min(j0 + x * step, P - 1)];
#pragma unroll
          for (int x = 0; x < N; x++) mx = fmaxf(mx, v[x]);
        }
      mx = joint(wave_max_f32(mx), part_max, sh, max_op);
      double l = 0.0;
      if (mine)
        for (int j0 = part * kWave + lane; j0 < P; j0 += N * step) {
          float v[N];
#pragma unroll
          for (int x = 0; x < N; x++) v[x] = z[min(j0 + x * step, P - 1)];
#pragma unroll
          for (int x = 0; x < N; x++)
            if (j0 + x * step < P) l += exp((double)v[x] - (double)mx);
        }
      l = joint(wave_sum_f64(l), part_sum, sh, sum_op);
      if (mine && lane == 0 && part == 0) {
        max_of[rr] = mx;
        inv_of[rr] = 1.0 / l;
      }
    }
    __syncthreads();
  }
  for (int t0 = 0; t0 < P; t0 += tile) {
    const int t1 = min(P, t0 + tile);
    double acc[kTile / kThreads];
#pragma unroll
    for (int x = 0; x < kTile / kThreads; x++) acc[x] = 0.0;
    for (int r0 = 0; r0 < g; r0 += W) {
      const int n = min(W, g - r0), sh = share(n), slot = w >> sh, rr = r0 + slot, part = w & ((1 << sh) - 1);
      const bool mine = slot < n;                    // uniform over the wave
      const float* z = logits(mine ? rr : 0);
      const int first = part * kWave + lane, step = kWave << sh;
      double* e = e_lds + slot * row;
      if (staged) {
        float zr[kRound];
        float mx = -INFINITY;
        if (mine) {
#pragma unroll
          for (int x = 0; x < kRound; x++)
            if (x * step < P) zr[x] = z[min(x * step + first, P - 1)];    // one round trip
#pragma unroll
          for (int x = 0; x < kRound; x++)
            if (x * step < P) mx = fmaxf(mx, zr[x]);
        }
        mx = joint(wave_max_f32(mx), part_max, sh, max_op);
        double l = 0.0;
        if (mine) {
#pragma unroll
          for (int x = 0; x < kRound; x++) {
            if (x * step < P) {
              const int j = x * step + first;
              const double v = exp((double)zr[x] - (double)mx);
              if (j < P) {
                e[1 + j] = v;
                l += v;
              }
            }
          }
        }
        l = joint(wave_sum_f64(l), part_sum, sh, sum_op);
        if (mine && lane == 0 && part == 0) inv_of[rr] = 1.0 / l;
      } else if (mine) {
        const double mx = (double)max_of[rr];
        for (int j = max(0, t0 - 1) + first; j < min(P, t1 + 1); j += step) e[1 + j - t0] = exp((double)z[j] - mx);
      }
      if (mine && lane == 0 && part == 0) {          // zero padding at the ends of the row
        if (t0 == 0) e[0] = 0.0;
        if (t1 == P) e[1 + P - t0] = 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < kTile / kThreads; x++) {
        const int j = t0 + x * kThreads + tid;
        if (j < t1) {
          const double* q = e_lds + 1 + j - t0;
          for (int s = 0; s < n; s++, q += row) acc[x] += conv3(q[-1], q[0], q[1]) * inv_of[r0 + s];
        }
      }
      __syncthreads();                               // e free for the next heads or tile
    }
#pragma unroll
    for (int x = 0; x < kTile / kThreads; x++) {
      const int j = t0 + x * kThreads + tid;
      if (j < t1) y[j] = (float)acc[x];
    }
  }
}

// Persistent grid: as many workgroups as can be resident at once, but no more than give each
// about kMinItemsPerWg (page, KV head) items (at least one per CU): a workgroup stages its
// request's query block (up to 18 KiB for the MLA geometry) before it streams, which only pays
// off over enough items.  The item count is bounded on the host by batch x max blocks x H.
// Measured on the MLA workload (16384 items; score + top-K): 30.0 us with every resident slot,
// 25.1 us at 32 items per workgroup, 27.1 us at 64 and 27.0 us at 128.
constexpr int kMinItemsPerWg = 32;
int score_grid(const void* fn, size_t lds, const ScoreArgs& a) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kThreads, lds) != hipSuccess || per_cu < 1)
    per_cu = 1;
  // a persistent grid must be resident at once: also bound it by the CU's LDS
  hipFuncAttributes fa;
  if (hipFuncGetAttributes(&fa, fn) == hipSuccess) {
    const int by_lds = (int)(kLdsPerCu / (fa.sharedSizeBytes + lds));
    per_cu = std::max(1, std::min(per_cu, by_lds));
  }
  const int cus = device_cus();
  const long long items = (long long)a.batch * a.max_pages * a.H;
  const long long by_items = (items + kMinItemsPerWg - 1) / kMinItemsPerWg;
  return (int)std::max<long long>(cus, std::min<long long>((long long)per_cu * cus * kScoreGridFactor, by_items));
}
template <int KIND, int D>
void launch_score(const ScoreArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)score_lds<KIND, D>(a.batch, a.Hq, a.H).total;
  // page_indptr in LDS up to kMaxLdsBatch requests, read from global memory beyond
  const bool lds_ind = a.batch <= kMaxLdsBatch;
  const void* fn = lds_ind ? reinterpret_cast<const void*>(score_kernel<KIND, D, true>)
                           : reinterpret_cast<const void*>(score_kernel<KIND, D, false>);
  const int grid = score_grid(fn, lds, a);
  if (lds_ind) hipLaunchKernelGGL((score_kernel<KIND, D, true>), dim3(grid), dim3(kThreads), lds, stream, a);
  else hipLaunchKernelGGL((score_kernel<KIND, D, false>), dim3(grid), dim3(kThreads), lds, stream, a);
}
template <int D, int NS>
void launch_head_score_sets(const ScoreArgs& a, hipStream_t stream) {
  const bool lds_ind = a.batch <= kMaxLdsBatch;
  const size_t lds = (size_t)2 * a.Hq * D * 2 + (lds_ind ? (size_t)(2 * a.batch + 1) * 4 : 0);
  const void* fn = lds_ind ? reinterpret_cast<const void*>(head_score_kernel<D, NS, true>)
                           : reinterpret_cast<const void*>(head_score_kernel<D, NS, false>);
  const int grid = score_grid(fn, lds, a);
  if (lds_ind) hipLaunchKernelGGL((head_score_kernel<D, NS, true>), dim3(grid), dim3(kThreads), lds, stream, a);
  else hipLaunchKernelGGL((head_score_kernel<D, NS, false>), dim3(grid), dim3(kThreads), lds, stream, a);
}
template <int D>
void launch_head_score(const ScoreArgs& a, hipStream_t stream) {
  const int g = a.Hq / a.H;
  if (g <= 4) launch_head_score_sets<D, 1>(a, stream);
  else if (g <= 8) launch_head_score_sets<D, 2>(a, stream);
  else launch_head_score_sets<D, 4>(a, stream);
}

// The bucketed selection's shape: as many threads as keep a request's pages at four slots each
// while the batch's (request, KV head) pairs leave CUs idle; fewer and longer waves when the pairs
// fill the chip by themselves, because every wave repeats the prefixes and reductions.  Kernel
// trace, us at T = 1024 / 512 / 256: 32 pairs of 2048 pages 5.3 / 5.8 / 6.6, 128 pairs of 4096 pages
// 11.1 / 11.7 / 15.0, 512 pairs of 2048 pages 21.8 / 13.8 / 14.0, 1024 pairs of 4096 pages 22.9 /
// 13.3 / 12.9.  Unused slots cost too: 512 pairs of up to 2048 pages of NSA scores at T = 512 take
// 13.0 us with four slots, 14.2 with eight.  Past 4096 pages (up to kTwoPassMaxPages) the selection
// stays here because the two-pass kinds then read half the summary bytes and the general radix
// kernel re-reads the scores: block mean of eight requests of 6000 to 8192 pages, score + selection
// 42.2 + 25.6 us in one pass with the radix kernel, 22 + 11 here (the whole call 66.8 -> 37.5 us).
template <int RK, int D, int T, int K>
void launch_bucket_shape(const SelArgs& a, const AppendStep& ap, hipStream_t stream) {
  const int grid = a.batch * a.H + (ap.app.knew ? a.batch * append_wgs<T>(a.H, ap.D) : 0);
  hipLaunchKernelGGL((topk_bucket_kernel<RK, D, T, K>), dim3(grid), dim3(T), 0, stream, a, ap);
}
template <int RK, int D>
void launch_bucket(const SelArgs& a, const AppendStep& ap, hipStream_t stream) {
  const long long pairs = (long long)a.batch * a.H, cus = device_cus();
  if (a.max_pages <= 1024) launch_bucket_shape<RK, D, 256, 4>(a, ap, stream);
  else if (a.max_pages <= 2048 && pairs <= 2 * cus) launch_bucket_shape<RK, D, 512, 4>(a, ap, stream);
  else if (D <= 128 && a.max_pages <= 4096 && 2 * pairs <= cus)
    launch_bucket_shape<RK, D <= 128 ? D : 64, 1024, 4>(a, ap, stream);
  else if (a.max_pages <= 4096 && pairs <= 2 * cus) launch_bucket_shape<RK, D, 512, 8>(a, ap, stream);
  else if (a.max_pages <= 4096) launch_bucket_shape<RK, D, 256, 16>(a, ap, stream);
  else if constexpr (D > 128) {          // 1024 threads leave too few registers for the re-scoring
    if (a.max_pages <= 8192) launch_bucket_shape<RK, D, 512, 16>(a, ap, stream);
    else launch_bucket_shape<RK, D, 512, 32>(a, ap, stream);
  } else {
    if (a.max_pages <= 8192) launch_bucket_shape<RK, D, 1024, 8>(a, ap, stream);
    else launch_bucket_shape<RK, D, 1024, 16>(a, ap, stream);
  }
}

// The radix selection's shape: as the bucketed one's, but long rows take 512 threads once there is more
// than a pair per CU.  us a call (remapped, tau 0.2) at 32 / 128 / 512 / 1024 pairs, rows of up to 1000:
// 256 threads 4.9 / 5.1 / 5.7 / 7.3, 512 4.9 / 5.1 / 6.4 / 9.0; 2000: 512 x 4 slots 5.8 / 5.6 / 7.7 / 10.8, 256 x
// 8 6.7 / 6.7 / 8.1 / 10.1; 4000: 1024 x 4 7.8 / 8.0 / 11.3 / 19.9, 512 x 8 8.1 / 8.2 / 10.7 / 16.8, 256 x 16 10.9 /
// 11.3 / 12.5 / 17.0; 8000: 1024 x 8 11.5 / 11.6 / 20.1 / 38.1, 512 x 16 13.0 / 13.1 / 17.8 / 28.3, 256 x 32 19.6 /
// 19.7 / 22.3 / 30.3; 16000: 1024 x 16 18.1 / 19.1 / 35.5 / 67.4, 512 x 32 20.2 / 21.3 / 30.2 / 57.0.
template <int T, int K>
void launch_radix_shape(const SelArgs& a, const TopkOptions& opt, hipStream_t stream) {
  hipLaunchKernelGGL((topk_radix_kernel<T, K>), dim3(a.batch * a.H), dim3(T), 0, stream, a, opt);
}
void launch_radix(const SelArgs& a, const TopkOptions& opt, hipStream_t stream) {
  const long long pairs = (long long)a.batch * a.H, cus = device_cus();
  if (a.max_pages <= 1024) launch_radix_shape<256, 4>(a, opt, stream);
  else if (a.max_pages <= 2048 && pairs <= 2 * cus) launch_radix_shape<512, 4>(a, opt, stream);
  else if (a.max_pages <= 2048) launch_radix_shape<256, 8>(a, opt, stream);
  else if (a.max_pages <= 4096 && 2 * pairs <= cus) launch_radix_shape<1024, 4>(a, opt, stream);
  else if (a.max_pages <= 4096 && pairs <= 2 * cus) launch_radix_shape<512, 8>(a, opt, stream);
  else if (a.max_pages <= 4096) launch_radix_shape<256, 16>(a, opt, stream);
  else if (a.max_pages <= 8192 && pairs <= cus) launch_radix_shape<1024, 8>(a, opt, stream);
  else if (a.max_pages <= 8192) launch_radix_shape<512, 16>(a, opt, stream);
  else if (pairs <= cus) launch_radix_shape<1024, 16>(a, opt, stream);
  else launch_radix_shape<512, 32>(a, opt, stream);
}

// Selection from scores in a.lower: exact and unmapped by the bucketed kernel, else by radix
// passes; rows past the page slots of both by the general radix kernel.
void launch_select(const SelArgs& a, const TopkOptions& opt, const AppendStep& ap, hipStream_t stream) {
  if (a.max_pages > kTwoPassMaxPages)
    hipLaunchKernelGGL(topk_long_kernel, dim3(a.batch * a.H), dim3(kThreads), 0, stream, a, opt);
  else if (opt.remap != 0 || opt.tau_q != 0) launch_radix(a, opt, stream);
  else launch_bucket<kNoRescore, 0>(a, ap, stream);
}

}  // namespace

int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 0;
  return cus > 0 ? cus : 256;
}

size_t score_workspace_bytes(int batch, int num_kv_heads, int num_q_heads, int max_pages) {
  const size_t planes = std::max(2 * num_kv_heads, num_q_heads + num_kv_heads);
  size_t b = planes * (size_t)batch * (size_t)score_stride(max_pages) * sizeof(float);
  return (b + 255) & ~(size_t)255;
}

// One-pass scores of an ABI score kind (NSA: its per-head logits; smoothing: the block mean it
// smooths): the block mean for D in {64, 128, 576}, every other kind for D in {64, 128} (the
// host rejects the rest).
void launch_one_pass_score(int abi_kind, int Dqk, const ScoreArgs& a, hipStream_t stream) {
#define VX_ENV(K)                                   \
  do {                                              \
    if (Dqk == 64) launch_score<K, 64>(a, stream);  \
    else launch_score<K, 128>(a, stream);           \
  } while (0)
  switch (internal_kind(abi_kind)) {
    case kMeanDot:
      if (Dqk == 64) launch_score<kMeanDot, 64>(a, stream);
      else if (Dqk == 128) launch_score<kMeanDot, 128>(a, stream);
      else launch_score<kMeanDot, 576>(a, stream);
      break;
    case kQuest: VX_ENV(kQuest); break;
    case kQuestConsensus: VX_ENV(kQuestConsensus); break;
    case kEnvLower: VX_ENV(kEnvLower); break;
    case kQuestRectified: VX_ENV(kQuestRectified); break;
    case kHeadDot:
      if (Dqk == 64) launch_head_score<64>(a, stream);
      else launch_head_score<128>(a, stream);
      break;
    default: VX_ENV(kMaxDot); break;
  }
#undef VX_ENV
}

hipError_t launch_score_topk(const Geometry& g, const uint16_t* q, int Hq, int kind, const float* mean,
                             const uint16_t* mean_bf, const uint16_t* maxs, const uint16_t* mins,
                             const int32_t* budget, int n_sink, int n_local, int max_sel, int32_t* sel_pages,
                             int32_t* sel_count, void* ws, int remap, int tau_q, uint32_t seed, hipStream_t stream,
                             const StepAppend& sa) {
  if (g.batch == 0) return hipSuccess;
  float* scores = reinterpret_cast<float*>(ws);
  const bool approx = remap != 0 || tau_q != 0;           // one-pass scores, then the radix select
  const int ik = internal_kind(kind);
  // the selection paths: the block mean's two passes, the envelope kinds' two passes, else one
  // pass of scores (through a flow for NSA and smoothing) selected by the one-wave kernel up to
  // kWaveMaxPages blocks per request, the bucketed kernel up to kTwoPassMaxPages, else the radix kernel
  const bool mean_two_pass = (kind == kMeanDot || kind == kAbiContent) && mean_bf && !approx;
  const bool env_two_pass =
      is_env(ik) && !approx && g.max_pages <= kTwoPassMaxPages && Hq <= 4 * g.H && (g.Dqk == 64 || g.Dqk == 128);
  const bool flow = kind == kAbiNsa || kind == kAbiSmooth;
  const bool wave = !approx && !mean_two_pass && !env_two_pass && g.max_pages <= kWaveMaxPages;
  // The step's append: workgroups of its own inside the selection launch, or a launch ahead of
  // everything when the selection reads every block's score (the flows couple the pages; the
  // radix path is not fused).
  AppendStep ap{};
  if (sa.k_new) {
    if (approx || g.max_pages > kTwoPassMaxPages || flow) {
      const hipError_t e =
          launch_kv_append_summarize(g, sa.k_new, sa.v_new, sa.mean, sa.mean_bf, sa.maxo, sa.mino, stream);
      if (e != hipSuccess) return e;
    } else {
      ap.app = summ::AppendArgs{sa.k_new, sa.v_new, const_cast<void*>(g.k), const_cast<void*>(g.v)};
      ap.k = g.k;
      ap.k_scale = g.k_scale;
      ap.kt = g.kv_dtype;
      ap.ps = g.ps;
      ap.D = g.Dqk;
      ap.num_phys = g.num_phys_pages;
      ap.mean = sa.mean;
      ap.mean_bf = sa.mean_bf;
      ap.maxo = sa.maxo;
      ap.mino = sa.mino;
      ap.max_pages = g.max_pages;
    }
  }
  ScoreArgs a;
  a.q = q;
  a.indptr = g.indptr;
  a.indices = g.indices;
  a.seq_lens = g.seq_lens;
  a.mean = mean;
  a.maxs = maxs;
  a.mins = mins;
  a.scores = scores;
  a.Hq = Hq;
  a.H = g.H;
  a.ps = g.bs;                               // scores are per block
  a.r = g.r;
  a.num_phys = g.num_phys_pages;
  a.max_pages = g.max_pages;
  a.batch = g.batch;
  a.stride = score_stride(g.max_pages);
  a.plane = (int64_t)g.H * g.batch * a.stride;
  a.qdims = kind == kAbiContent ? g.Dv : g.Dqk;
  SelArgs t{};
  t.lower = t.upper = scores;
  t.mean = mean;
  t.maxs = maxs;
  t.mins = mins;
  t.q = q;
  t.Hq = Hq;
  t.H = g.H;
  t.qdims = a.qdims;
  t.ps = g.bs;
  t.r = g.r;
  t.max_pages = g.max_pages;
  t.stride = a.stride;
  t.batch = g.batch;
  t.num_phys = g.num_phys_pages;
  t.indptr = g.indptr;
  t.indices = g.indices;
  t.seq_lens = g.seq_lens;
  t.budget = budget;
  t.n_sink = n_sink;
  t.n_local = n_local;
  t.max_sel = max_sel;
  t.sel_pages = sel_pages;
  t.sel_count = sel_count;
  if (mean_two_pass || env_two_pass) {
    // a bound pass, then re-scoring of the undecided pages in the bucketed select
    t.upper = scores + a.plane;
    if (mean_two_pass) a.maxs = mean_bf;
#define VX_TWO_PASS(BK, RK, DD)          \
  do {                                   \
    launch_score<BK, DD>(a, stream);     \
    const hipError_t e = hipGetLastError(); \
    if (e != hipSuccess) return e;       \
    launch_bucket<RK, DD>(t, ap, stream); \
  } while (0)
#define VX_ENV_TWO_PASS(K)                                             \
  case K:                                                              \
    if (g.Dqk == 64) VX_TWO_PASS(bound_of_env(K), K, 64);              \
    else VX_TWO_PASS(bound_of_env(K), K, 128);                         \
    break;
    switch (ik) {
      case kMeanDot:
        if (g.Dqk == 64) VX_TWO_PASS(kMeanBound, kMeanDot, 64);
        else if (g.Dqk == 128) VX_TWO_PASS(kMeanBound, kMeanDot, 128);
        else VX_TWO_PASS(kMeanBound, kMeanDot, 576);
        break;
      VX_ENV_TWO_PASS(kQuest)
      VX_ENV_TWO_PASS(kQuestConsensus)
      VX_ENV_TWO_PASS(kEnvLower)
      VX_ENV_TWO_PASS(kQuestRectified)
      default: break;
    }
#undef VX_ENV_TWO_PASS
#undef VX_TWO_PASS
    return hipGetLastError();
  }
  if (kind == kAbiNsa || kind == kAbiSmooth) {
    // the flow's first step into the planes after the first H, its last step into plane 0
    float* first = scores + (int64_t)g.H * g.batch * a.stride;
    a.scores = first;
    a.plane = (int64_t)g.batch * a.stride;
    launch_one_pass_score(kind, g.Dqk, a, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_score_flow(kind, first, scores, a.stride, g.H, Hq, g.batch, nullptr, g.bs, g.r, g.max_pages,
                          g.indptr, g.seq_lens, stream);
    if (e != hipSuccess) return e;
  } else {
    launch_one_pass_score(kind, g.Dqk, a, stream);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (wave) {
    const int grid = g.batch * g.H + (ap.app.knew ? g.batch * append_wgs<kWave>(g.H, g.Dqk) : 0);
    hipLaunchKernelGGL(topk_wave_kernel, dim3(grid), dim3(kWave), 0, stream, scores, g.H, g.bs, g.r,
                       g.max_pages, a.stride, g.batch, g.indptr, g.indices, g.seq_lens, budget, n_sink, n_local,
                       max_sel, sel_pages, sel_count, ap);
    return hipGetLastError();
  }
  launch_select(t, TopkOptions{remap, tau_q, seed}, ap, stream);
  return hipGetLastError();
}

hipError_t launch_score(const Geometry& g, const uint16_t* q, int Hq, int kind, const float* mean,
                        const uint16_t* maxs, const uint16_t* mins, float* scores, int stride, hipStream_t stream) {
  if (g.batch == 0) return hipSuccess;
  ScoreArgs a;
  a.q = q;
  a.indptr = g.indptr;
  a.indices = g.indices;
  a.seq_lens = g.seq_lens;
  a.mean = mean;
  a.maxs = maxs;
  a.mins = mins;
  a.scores = scores;
  a.Hq = Hq;
  a.H = g.H;
  a.ps = g.bs;                               // scores are per block
  a.r = g.r;
  a.num_phys = g.num_phys_pages;
  a.max_pages = g.max_pages;
  a.batch = g.batch;
  a.stride = stride;
  a.plane = (int64_t)g.batch * stride;       // NSA logits: the rows of query head r start at r * plane
  a.qdims = kind == kAbiContent ? g.Dv : g.Dqk;
  launch_one_pass_score(kind, g.Dqk, a, stream);
  return hipGetLastError();
}

hipError_t launch_score_flow(int kind, const float* in, float* out, int stride, int H, int Hq, int batch,
                             const int32_t* items, int ps, int r, int max_pages, const int32_t* indptr,
                             const int32_t* seq_lens, hipStream_t stream) {
  if (batch == 0) return hipSuccess;
  if (kind == kAbiNsa) {
    const int rows = std::min(Hq / H, kThreads / kWave);
    auto launch = [&](auto tile, auto share) {
      constexpr int T = decltype(tile)::value, S = decltype(share)::value;
      hipLaunchKernelGGL((flow_kernel<true, T, S>), dim3(batch * H), dim3(kThreads),
                         sizeof(double) * rows * (std::min(max_pages, T) + 2), stream, in, out, H, Hq / H, ps, r,
                         max_pages, stride, batch, indptr, seq_lens, items);
    };
    auto with_tile = [&](auto share) {
      if (max_pages <= kFlowTile / 4) launch(std::integral_constant<int, kFlowTile / 4>{}, share);
      else if (max_pages <= kFlowTile / 2) launch(std::integral_constant<int, kFlowTile / 2>{}, share);
      else launch(std::integral_constant<int, kFlowTile>{}, share);
    };
    const int g = Hq / H;
    if (g == 1) with_tile(std::integral_constant<int, 2>{});
    else if (g == 2) with_tile(std::integral_constant<int, 1>{});
    else if (g % 4 == 0 || g % 4 == 3) with_tile(std::integral_constant<int, 0>{});
    else with_tile(std::integral_constant<int, -1>{});
  } else {
    hipLaunchKernelGGL((flow_kernel<false, kThreads, 0>), dim3(batch * H), dim3(kThreads), 0, stream, in, out, H, Hq / H,
                       ps, r, max_pages, stride, batch, indptr, seq_lens, items);
  }
  return hipGetLastError();
}

hipError_t launch_topk_select(const float* scores, int stride, int H, int batch, const int32_t* items,
                              const int32_t* budget, int n_sink, int n_local, int max_sel, int remap, int tau_q,
                              uint32_t seed, int32_t* sel_pages, int32_t* sel_count, hipStream_t stream) {
  if (batch == 0) return hipSuccess;
  SelArgs t{};
  t.lower = t.upper = scores;
  t.Hq = t.H = H;
  t.ps = 16;
  t.r = 1;
  t.max_pages = t.stride = stride;
  t.batch = batch;
  t.items = items;
  t.budget = budget;
  t.n_sink = n_sink;
  t.n_local = n_local;
  t.max_sel = max_sel;
  t.sel_pages = sel_pages;
  t.sel_count = sel_count;
  launch_select(t, TopkOptions{remap, tau_q, seed}, AppendStep{}, stream);
  return hipGetLastError();
}

}  // namespace vx
