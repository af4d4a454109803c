// Construction of the main + residual cache of one layer (App. D, Algorithm 1
// with the residual count r given per (b, kv head)).
//
// Per (b, kv head), in launch order:
//   lse_partial    MFMA logits of the G*w observation-window rows against a
//                  chunk of 256-key groups (each wave owns 64 keys of a group
//                  and runs over its rows); per row the max and sum of exp
//                  (base 2) over the keys it can see (causal in the window)
//   lse_final      merges the chunk partials into one log-sum-exp per row
//   score_accum    recomputes the logits; raw[p] = sum over rows of the
//                  normalised weight of key p, for the scored positions
//   pool_scores    centred zero-padded sum (5 taps by default) over the
//                  scored positions, and the selection's first radix pass
//   [adakv_alloc]  with cross-head allocation only: moves top-k budget
//                  between the KV heads of a sequence (one ranking of all
//                  heads' scores, per-head safeguard floor and slot cap) and
//                  rewrites each head's sizes before the selection
//   select_hist x2 radix select (11, 11 and 10 bits of the fp32 bit pattern)
//  [select_count]  of the k_top-th and (k_top + r')-th largest score over blocks
//   select_write   of 8192 scores, counted per block first where the list is
//                  long; ties at a threshold go to the lower position. Stable
//                  compaction writes main_idx (top-k, then the protected
//                  window), the evicted list E and the Lloyd seeds, all
//                  ascending
//  [select_one]    pooling and selection in one launch on short lists
//   gather_init    copies the main rows into slots [r, r + m), clears the
//                  residual slots, seeds the Lloyd centres with K[seed] (fp32,
//                  bf16 hi + lo and the squared norm)
//   T x { lloyd_assign   MFMA distances ||mu||^2 - 2 k.mu with mu = hi + lo,
//                        argmin with ties to the lower centre, and per-block
//                        group histograms
//         lloyd_offsets  group starts and per-block offsets (counting sort),
//                        and the update's pieces
//         lloyd_scatter  stable placement of E by group
//        [lloyd_sort     both in one launch where E is short]
//         lloyd_update   fp64 sums of the members in fixed order -> new
//                        centres; in the last round also the mean values,
//                        counts and log-counts written to the cache }
// Scores follow the SnapKV rule (App. B.2.2), selection the main-selection
// equation (Sec. 5.2), the partition objective and summaries Sec. 5.3 and
// App. B.3.
#include <math.h>

#include <vector>

#include <type_traits>

#include "common.h"
#include "internal.h"

namespace reskv {

namespace {

constexpr int kThreads = 256;
constexpr int kKeyGroups = 4;     // 256-key groups per lse chunk (at least) and per score-pass block
// Score-pass blocks of four key groups up to which the pass takes one group per
// block instead: more blocks for short passes, but each stages every window row.
// Whole scoring constructions (d = 128, bf16), four groups / one: 128 rows, 128
// blocks 89 / 80 us, 256 95 / 91, 384 107 / 109, 480 113 / 118; more rows, whose
// blocks of eight waves leave four without keys: 256 rows, 128 blocks 103 / 98, 192
// 107 / 112, 256 111 / 122, 480 144 / 169. fp32 passes are longer per row and
// gain up to 384 blocks at any count (256 rows 784 / 746 us, 480 blocks 921 / 952).
constexpr int kFewScoreBlocks = 384;
constexpr int kFewScoreBlocksWide = 128;  // bf16, more than kRowChunk rows
// fp32 lse chunks up to which their rows are dealt to blocks 16 at a time: each
// such block reads the chunk's keys again. A whole scoring construction (d = 128,
// 128 window rows), undealt / dealt: 4 chunks 135 / 75 us, 64 156 / 118, 128 174 /
// 176, 160 200 / 218, 256 228 / 302, 384 334 / 426; 64 to 1024 rows cross there too
constexpr int kDealtChunks = 128;
// window rows staged in LDS per scoring step: 128, or 256 when there are
// more than 128 (each key group is then loaded once for all of them)
constexpr int kRowChunk = 128;
constexpr int kRowChunkWide = 256;
// s_waitcnt immediate: vector-memory count 0, export and LDS/scalar counts
// left at their maximum (no wait on them)
constexpr int kWaitVmcnt0 = 0x0F70;
constexpr int kTokBlock = 256;     // evicted tokens per counting-sort block (histograms, scatter)
constexpr int kSelThreads = 1024;
constexpr int kSelPer = 8;                          // scores per selection thread
constexpr int kSelChunk = kSelPer * kSelThreads;   // scores per selection block
constexpr int kSelUncounted = 8;                   // blocks up to which the placement counts the scores before a block itself
constexpr int kSelBins = 2048;                     // digits of the wider selection passes
constexpr int kAdaHist = kSelBins + 1024;          // cross-head search histograms per head (second and third pass)
constexpr int kSelHist = 4 * kSelBins;             // selection pass histograms per head (sel_at)
constexpr int kPieceMin = 4096;                     // update pieces of 1024 members from which they are not cut smaller

struct BuildArgs {
  const void* k;
  const void* v;
  const void* q_obs;
  void* kc;
  void* vc;
  float* logc;
  int32_t* main_idx;
  int32_t* res_len;
  int32_t* main_len;
  float* dbg_scores;
  int32_t* dbg_assign;
  float* dbg_centers;  // [T][BH][Rcap][D] or NULL
  const HeadMeta* meta;
  float2* lse_part;    // [BH][NCH][R] (max, sum) in base 2, one per lse block
  float* lse2;         // [BH][R]
  float* raw;          // [BH][S]
  float* score;        // [BH][S]
  int32_t* elist;      // [BH][S]   evicted positions, ascending
  int32_t* seeds;      // [BH][Rcap]
  float* cent;         // [BH][Rcap][D]
  uint16_t* cent_hi;   // [BH][Rcap][D]
  uint16_t* cent_lo;   // [BH][Rcap][D]
  float* cnorm;        // [BH][Rcap]
  int32_t* assign;     // [BH][S]   group of evicted token i
  int32_t* hist;       // [BH][NBLK][Rcap] block histograms -> block offsets
  int32_t* order;      // [BH][S]   evicted positions grouped by centre
  int4* items;         // [BH][NIT] update pieces: group | piece << 12, partial slot or -1, first entry of order, group size
  int32_t* nitem;      // [BH]
  int32_t* parrive;    // [BH][Rcap] pieces of a split group that have left their sums
  double* part;        // [BH][NPART][2][D] key and value sums of split groups' pieces
  int32_t* sel_hist;   // [BH][kSelHist] selection pass histograms (zeroed by lse_final and, for the next candidate, gather_init), or NULL
  bool more;           // another candidate's selection follows (gather_init zeroes sel_hist)
  int32_t* ada_hist;   // [BH][kAdaHist] cross-head search histograms (zeroed by pool_scores), or NULL
  uint32_t* ada_state; // [2][B][kAdaState] per sequence: prefix, then the heads' tokens above its range
  uint32_t* sel_state; // [BH][2][4] thresholds' prefixes and remaining ranks after the first and second pass
  uint4* sel_cnt;      // [BH][NSEL] per selection block: scores above / equal to each threshold (select_count), or NULL
  int NC;              // candidates built in one batch
  int SBH;             // heads with keys and values of their own, B * Hkv of one candidate
  int B, Hq, Hkv, G, C, Rcap, S, w, R, LG, KG, NCH, NBLK, NSEL, T;
  int lpiece, NIT, NPART;  // log2 of the members per update piece, pieces and partial slots per head
  int wr;              // leading window rows per query head that score (R = G * wr)
  int pool_half;       // pooling taps on each side of a position
  int cap_slots;       // slots a head may fill at construction (C minus the decode reserve)
  float scale2;        // log2(e) / sqrt(d)
};

// (b, kv head) of a block from blockIdx.y / .z; with rev set the heads are
// walked in the opposite order, so a kernel that re-reads the keys of the
// kernel before it starts with the heads that kernel read last (still in the
// memory-side cache) instead of the ones it read first.
__device__ __forceinline__ void block_head(const BuildArgs& a, int rev, int& b, int& kvh, int& bh) {
  bh = blockIdx.z * a.Hkv + blockIdx.y;
  if (rev) bh = a.B * a.Hkv - 1 - bh;
  b = bh / a.Hkv;
  kvh = bh - b * a.Hkv;
}

// Head whose keys, values and raw scores head bh reads: with several candidate
// constructions in one batch (the proxy's), heads bh, bh + SBH, ... are copies.
__device__ __forceinline__ int source_head(const BuildArgs& a, int bh) { return bh % a.SBH; }

__device__ __forceinline__ float to_f32(uint16_t x) { return __uint_as_float((uint32_t)x << 16); }
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ void store_elem(uint16_t* p, float x) { *p = f32_to_bf16_rne(x); }
__device__ __forceinline__ void store_elem(float* p, float x) { *p = x; }

// Scoring row t = h*wr + i of the group: query head kvh*G + h, window row i
// (position s-w+i); only the leading wr rows of each head's window score.
// Rows [r0, r0 + nrows) are copied into LDS, rows at or past R as zeros. The
// 16-byte pieces of a row are permuted by the row's low bits, which keeps the
// MFMA fragment reads free of bank conflicts without padding the rows.
template <typename T, int D>
struct WindowRows {
  static constexpr int kRowB = D * (int)sizeof(T);
  static constexpr int kPieces = kRowB / 16;  // 8 or more
  static __device__ __forceinline__ int at(int row, int pc) { return row * kRowB + (pc ^ (row & 7)) * 16; }
  static __device__ __forceinline__ void stage(unsigned char* s_q, const BuildArgs& a, int b, int kvh, int r0,
                                               int nrows) {
    for (int x = threadIdx.x; x < nrows * kPieces; x += blockDim.x) {
      const int rr = x / kPieces, pc = x % kPieces, t = r0 + rr;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (t < a.R) {
        const int h = t / a.wr, i = t % a.wr;
        const T* q = static_cast<const T*>(a.q_obs) + (((size_t)b * a.Hq + kvh * a.G + h) * a.w + i) * D;
        v = reinterpret_cast<const uint4*>(q)[pc];
      }
      *reinterpret_cast<uint4*>(s_q + at(rr, pc)) = v;
    }
  }
  // Fragment of row 16 rt + col: its pieces grp + 4 i lie at
  // (grp ^ col % 4) + 4 (i ^ (col / 4) % 2), so two addresses (even and odd
  // i) and constant offsets reach them all.
  static __device__ __forceinline__ int lane_at(int col, int grp, int odd) {
    return col * kRowB + ((grp ^ (col & 3)) + 4 * (odd ^ ((col >> 2) & 1))) * 16;
  }
  static __device__ __forceinline__ void load(Frag<T, D>& f, const unsigned char* even, const unsigned char* odd) {
#pragma unroll
    for (int i = 0; i < Frag<T, D>::kSteps; ++i)
      f.w[i] = *reinterpret_cast<const typename Frag<T, D>::Word*>((i & 1 ? odd : even) + 128 * (i >> 1));
  }
};

// ---------------------------------------------------------------- scoring

// Scoring blocks stream groups of 256 keys one after the other (the lse pass
// 4, 8 or 16 groups per chunk, the score pass 4 or 1 per block, as the plan
// chooses); in each group a wave owns 64 keys and runs over every window row.
// The window rows are staged in LDS once per block, RC at a time: every row
// chunk loads the block's keys again, so with more than 128 rows (G w = 224,
// 256) the wide chunk of 256 rows reads each key once per pass.

// Key fragments of the 64 keys from kw (clamped to the sequence).
template <typename T, int D>
__device__ __forceinline__ void load_score_keys(Frag<T, D> (&f)[4], const T* K, int kw, int s, int col, int grp) {
#pragma unroll
  for (int t = 0; t < 4; ++t) f[t].load(K + (size_t)min(kw + 16 * t + col, s - 1) * D, grp);
}

// lse pass: the MFMA is oriented keys x rows, C[key][row]: a lane holds 16
// keys of one row, so a row's max and sum need only two cross-lane steps.
// A chunk is four waves, each keeping a running (max, sum) per row over its
// key groups, one 64-key group at a time (no second key buffer): the other
// waves of the SIMD hide its key loads and the chain max -> exponentials ->
// sum of a row tile. Bound by issue: MFMA and VALU instructions take turns on
// a SIMD here, and a row tile of 64 keys costs 16 MFMAs (17 cycles each), 17
// exponentials (9) and about 60 other VALU operations (4). Variants, none of
// which changes a row's arithmetic:
//   kRQ = 2, wide row chunk: two copies of a chunk's waves deal its row tiles
//   between them, so two blocks of eight waves share a CU's LDS and 128
//   registers give four waves per SIMD (28 query heads, 64 ragged contexts of
//   4K-64K tokens, window 32: 239 -> 214 us);
//   kRQ = 1, up to 128 rows: three waves per SIMD;
//   kSplit: a block takes one of the chunk's row chunks, for fp32 where the
//   chunks alone leave most CUs idle (2 heads of 1024 tokens, 64 rows: 28 ->
//   14 us; bf16 passes that short gained nothing from it).
template <typename T, int D, int RC, int kRQ, bool kSplit>
__global__ __launch_bounds__(256 * kRQ, (sizeof(T) == 4 ? 2 : kRQ > 1 ? 4 : 3)) void lse_partial(BuildArgs a) {
  constexpr int NT = 256 * kRQ;
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int span = 256 * a.LG;  // keys per chunk
  const int nrs = kSplit ? (a.R + RC - 1) / RC : 1;  // blocks that share a chunk's row chunks
  const int ch = blockIdx.x / nrs, rs = blockIdx.x - ch * nrs;
  if (hm.all_main || ch * span >= hm.s) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int vw = wave & 3, rq = wave >> 2;  // wave of the chunk, its share of the row tiles
  const int k0 = ch * span + 64 * vw;       // this wave's first key
  using Rows = WindowRows<T, D>;
  __shared__ __align__(16) unsigned char s_q[RC * Rows::kRowB];
  __shared__ float2 s_ml[4][RC];
  const unsigned char *q_even = s_q + Rows::lane_at(col, grp, 0), *q_odd = s_q + Rows::lane_at(col, grp, 1);
  const T* K = static_cast<const T*>(a.k) + (size_t)bh * a.S * D;
  for (int r0 = rs * RC; r0 < a.R; r0 += nrs * RC) {
    const int nrt = (min(RC, a.R - r0) + 15) / 16;
    if (r0 >= nrs * RC) __syncthreads();  // the previous chunk's rows and records are consumed
    Frag<T, D> kf[4];
    load_score_keys<T, D>(kf, K, k0, hm.s, col, grp);
    Rows::stage(s_q, a, b, kvh, r0, 16 * nrt);
    __syncthreads();
    // running (max, sum) of row 16 rt + col over this wave's keys, kept in
    // LDS so the row-tile loop need not be unrolled; the four lane groups
    // hold the same reduced values and each lane reads back its own writes
    for (int rt = rq; rt < nrt; rt += kRQ) s_ml[vw][16 * rt + col] = make_float2(kNegInf, 0.f);
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // the first group's keys have landed
    const int last = min(a.LG, (hm.s - k0 + 255) / 256);  // this wave's groups that hold keys (may be none)
#pragma unroll 1
    for (int gi = 0; gi < last; ++gi) {
      const int kw = k0 + 256 * gi;  // this wave's keys in group gi
      if (gi > 0) load_score_keys<T, D>(kf, K, kw, hm.s, col, grp);
      __builtin_amdgcn_sched_barrier(0);  // the group's key loads go out before its work
      // keys up to s - w are visible to every window row (and lie below s):
      // such waves skip the per-element masks
      auto rows = [&](auto full_tag) {
        constexpr bool kFull = decltype(full_tag)::value;
#pragma unroll 1
        for (int rt = rq; rt < nrt; rt += kRQ) {
          const int row = 16 * rt + col;  // window row of this lane's column
          const float2 st = s_ml[vw][row];
          Frag<T, D> qf;
          Rows::load(qf, q_even + rt * 16 * Rows::kRowB, q_odd + rt * 16 * Rows::kRowB);
          int pos = 0;
          if constexpr (!kFull) pos = r0 + row < a.R ? hm.s - a.w + (r0 + row) % a.wr : -1;
          // raw logits; the scale is positive, so the max commutes with it
          float v[16];
          float m = kNegInf;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const f32x4_t c = mma<D>(kf[t], qf, zero4());
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int p = kw + 16 * t + 4 * grp + i;
              const float x = (kFull || (p < hm.s && p <= pos)) ? c[i] : kNegInf;
              v[4 * t + i] = x;
              m = fmaxf(m, x);
            }
          }
          m = rows4_max(m);
          m = m == kNegInf ? kNegInf : m * a.scale2;
          const float m_new = fmaxf(st.x, m);
          const bool none = m_new == kNegInf;  // no key seen yet: the state stays
          const float ref = none ? 0.f : m_new;
          float l = 0.f;
#pragma unroll
          for (int j = 0; j < 16; ++j) l += fast_exp2(fmaf(v[j], a.scale2, -ref));
          l = rows4_sum(l);
          s_ml[vw][row] = make_float2(m_new, none ? st.y : fmaf(st.y, fast_exp2(st.x - ref), l));
        }
      };
      if (kw + 64 <= hm.s - a.w + 1) rows(std::true_type{});
      else rows(std::false_type{});
    }
    __syncthreads();
    // per row, the four waves' states into one record
    for (int t = threadIdx.x; t < min(RC, a.R - r0); t += NT) {
      float M = kNegInf;
#pragma unroll
      for (int w = 0; w < 4; ++w) M = fmaxf(M, s_ml[w][t].x);
      float L = 0.f;
      if (M != kNegInf) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float2 e = s_ml[w][t];
          if (e.x != kNegInf) L = fmaf(e.y, exp2f(e.x - M), L);
        }
      }
      a.lse_part[((size_t)bh * a.NCH + ch) * a.R + r0 + t] = make_float2(M, L);
    }
  }
}

// The head's selection histograms start from zero (where there are any).
__device__ __forceinline__ void zero_sel_hist(const BuildArgs& a, int bh, int i, int step) {
  if (a.sel_hist == nullptr) return;
  for (int4* h = reinterpret_cast<int4*>(a.sel_hist + (size_t)bh * kSelHist); i < kSelHist / 4; i += step)
    h[i] = make_int4(0, 0, 0, 0);
}

// One thread per row: the chunk records merged in chunk order, requested 16 at
// a time (bound by their latency: one at a time, 32 chunks took 15 us).
__global__ __launch_bounds__(kThreads) void lse_final(BuildArgs a) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int t = blockIdx.x * kThreads + threadIdx.x;
  for (int c = 0; c < a.NC; ++c) zero_sel_hist(a, c * a.SBH + bh, t, gridDim.x * kThreads);
  if (hm.all_main || t >= a.R) return;
  const int nch = (hm.s + 256 * a.LG - 1) / (256 * a.LG);
  const float2* pp = a.lse_part + (size_t)bh * a.NCH * a.R + t;
  constexpr int kB = 16;
  float2 e[kB];
  auto read = [&](int c0) {
#pragma unroll
    for (int u = 0; u < kB; ++u) e[u] = c0 + u < nch ? pp[(size_t)(c0 + u) * a.R] : make_float2(kNegInf, 0.f);
  };
  float M = kNegInf;
  for (int c0 = 0; c0 < nch; c0 += kB) {
    read(c0);
#pragma unroll
    for (int u = 0; u < kB; ++u) M = fmaxf(M, e[u].x);
  }
  float L = 0.f;
  for (int c0 = 0; c0 < nch; c0 += kB) {
    if (nch > kB) read(c0);
#pragma unroll
    for (int u = 0; u < kB; ++u)
      if (e[u].x != kNegInf) L = fmaf(e[u].y, exp2f(e[u].x - M), L);
  }
  a.lse2[(size_t)bh * a.R + t] = M + log2f(L);
}

// Score pass: C[row][key]: a lane holds one key of 4 rows, so the per-key
// sums stay in registers until two final cross-lane steps, and no cross-wave
// merge is needed. One key group per wave at a time and a rolled row-tile
// loop keep it at four waves per SIMD (bf16); with the wide row chunk two
// blocks of eight waves (NT = 512) share a CU (32 heads of 128K tokens, 256
// rows: 413 -> 323 us with four waves per SIMD instead of two). Bound by issue
// like the lse pass: 16 MFMAs, 16 exponentials and about 45 other VALU
// operations per row tile of 64 keys, and by the keys' HBM reads at 128 rows.
template <typename T, int D, int RC, int NT>
__global__ __launch_bounds__(NT, (sizeof(T) == 2 ? 4 : 2)) void score_accum(BuildArgs a, int rev) {
  int b, kvh, bh;
  block_head(a, rev, b, kvh, bh);
  const HeadMeta hm = a.meta[bh];
  const int k0 = blockIdx.x * 256 * a.KG;
  if (hm.all_main || k0 >= hm.n_sc) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  using Rows = WindowRows<T, D>;
  __shared__ __align__(16) unsigned char s_q[RC * Rows::kRowB];
  __shared__ __align__(16) float s_lse[RC];
  const unsigned char *q_even = s_q + Rows::lane_at(col, grp, 0), *q_odd = s_q + Rows::lane_at(col, grp, 1);
  const T* K = static_cast<const T*>(a.k) + (size_t)bh * a.S * D;
  for (int r0 = 0; r0 < a.R; r0 += RC) {
    const int nrt = (min(RC, a.R - r0) + 15) / 16;
    if (r0 > 0) __syncthreads();  // the previous chunk's rows are consumed
    Frag<T, D> kf[4];
    load_score_keys<T, D>(kf, K, k0 + 64 * wave, hm.s, col, grp);
    Rows::stage(s_q, a, b, kvh, r0, 16 * nrt);
    // padded rows carry lse = +inf and add 0
    for (int t = threadIdx.x; t < 16 * nrt; t += NT)
      s_lse[t] = r0 + t < a.R ? a.lse2[(size_t)bh * a.R + r0 + t] : __builtin_huge_valf();
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // the first group's keys have landed
#pragma unroll 1
    for (int kg = 0; kg < 256 * a.KG; kg += NT) {
      const int kw = k0 + kg + 64 * wave;  // this wave's keys
      if (kw >= hm.n_sc || kg + 64 * wave >= 256 * a.KG) break;  // wave-uniform
      if (kg > 0) load_score_keys<T, D>(kf, K, kw, hm.s, col, grp);
      __builtin_amdgcn_sched_barrier(0);  // the group's key loads go out before its work
      float ksum[4] = {0.f, 0.f, 0.f, 0.f};
      // keys up to s - w are visible to every window row: such waves skip the
      // per-element causal test
      auto rows = [&](auto full_tag) {
        constexpr bool kFull = decltype(full_tag)::value;
#pragma unroll 1
        for (int rt = 0; rt < nrt; ++rt) {
          Frag<T, D> qf;
          Rows::load(qf, q_even + rt * 16 * Rows::kRowB, q_odd + rt * 16 * Rows::kRowB);
          const float4 l4 = *reinterpret_cast<const float4*>(s_lse + 16 * rt + 4 * grp);
          const float lse[4] = {l4.x, l4.y, l4.z, l4.w};
          int pos[4];
          if constexpr (!kFull)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int t = r0 + 16 * rt + 4 * grp + i;
              pos[i] = t < a.R ? hm.s - a.w + t % a.wr : -1;  // padded rows see no key
            }
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const f32x4_t c = mma<D>(qf, kf[t], zero4());
            const int p = kw + 16 * t + col;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float e = fast_exp2(fmaf(c[i], a.scale2, -lse[i]));
              ksum[t] += (kFull || p <= pos[i]) ? e : 0.f;
            }
          }
        }
      };
      if (kw + 64 <= hm.s - a.w + 1) rows(std::true_type{});
      else rows(std::false_type{});
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float v = rows4_sum(ksum[t]);
        const int p = kw + 16 * t + col;
        if (grp == 0 && p < hm.n_sc) {
          float* dst = a.raw + (size_t)bh * a.S + p;
          if (r0 == 0) *dst = v;
          else *dst += v;  // later row chunks add to this lane's own sums
        }
      }
    }
  }
}

// Centred (2 * pool_half + 1)-tap sum with zero padding over the scored
// positions (5 taps for the SnapKV rule, 1 for H2O and TOVA). A thread pools
// kPoolPer consecutive positions from one window of raw scores held in
// registers (zeros outside [0, n)), adding the taps in ascending position
// order as the one-position form does.
constexpr int kPoolPer = 4;
constexpr int kPoolHalfMax = 15;  // pool_half <= 15 (pool_kernel <= 31)
constexpr int kPoolThreads = 1024;

// Histogram increment of bin `dig` by the lanes with `act` set. Scores share
// their leading digits (sign and exponent), so the lanes of a wave often hit
// one bin: up to two leader rounds count the lanes that share the leader's
// bin with one atomic each; the remaining lanes add their own. Called by
// every lane of the wave (act false where a lane has nothing to count).
__device__ __forceinline__ void wave_hist_add(int* hist, int dig, bool act, int lane) {
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const unsigned long long m = __ballot(act);
    if (m == 0ull) return;  // wave-uniform
    const int leader = __ffsll((long long)m) - 1;
    const int d = __shfl(dig, leader, 64);
    const unsigned long long same = __ballot(act && dig == d);
    if (lane == leader) atomicAdd(&hist[d], __popcll(same));
    act = act && dig != d;
  }
  if (act) atomicAdd(&hist[dig], 1);
}

// Radix passes of the selection: 11, 11 and 10 bits of the fp32 bit pattern,
// most significant first. A pass's histograms in the head's sel_hist: one for
// both thresholds in the first pass, one each in the others.
__host__ __device__ constexpr int sel_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }
__host__ __device__ constexpr int sel_bins(int pass) { return pass == 2 ? 1024 : kSelBins; }
__device__ __forceinline__ int sel_at(int pass, int q) {
  return pass == 0 ? 0 : pass == 1 ? kSelBins * (1 + q) : 3 * kSelBins + 1024 * q;
}

// Pooled scores of positions p0 .. p0 + kN - 1 (those below n).
template <int kN>
__device__ __forceinline__ void pool_run(const BuildArgs& a, const float* raw, int p0, int n, float (&v)[kN]) {
  const int ph = a.pool_half;
  float w[kN + 2 * kPoolHalfMax];  // raw[p0 - kPoolHalfMax + i]
#pragma unroll
  for (int i = 0; i < kN + 2 * kPoolHalfMax; ++i) {
    const int q = p0 - kPoolHalfMax + i;
    const bool tap = q >= p0 - ph && q < p0 + kN + ph;
    w[i] = tap && q >= 0 && q < n ? raw[q] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    v[k] = 0.f;
#pragma unroll
    for (int j = -kPoolHalfMax; j <= kPoolHalfMax; ++j)
      if (j >= -ph && j <= ph) v[k] += w[k + kPoolHalfMax + j];
  }
}

// The block also counts its scores' leading digits into the head's first
// selection histogram.
__global__ __launch_bounds__(kPoolThreads) void pool_scores(BuildArgs a) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int n = hm.all_main ? 0 : hm.n_sc;
  const int b0 = blockIdx.x * kPoolThreads * kPoolPer;
  if (a.ada_hist && blockIdx.x == 0)
    for (int i = threadIdx.x; i < kAdaHist; i += kPoolThreads) a.ada_hist[(size_t)bh * kAdaHist + i] = 0;
  if (b0 >= n && !a.dbg_scores) return;  // block-uniform
  __shared__ int s_hist[kSelBins];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < kSelBins; i += kPoolThreads) s_hist[i] = 0;
  const int p0 = b0 + tid * kPoolPer;
  float pooled[kPoolPer];
  pool_run(a, a.raw + (size_t)source_head(a, bh) * a.S, p0, n, pooled);
  __syncthreads();  // the histogram is cleared
#pragma unroll
  for (int k = 0; k < kPoolPer; ++k) {
    const int p = p0 + k;
    const float v = p < n ? pooled[k] : -1.f;
    if (p < n) a.score[(size_t)bh * a.S + p] = v;
    if (a.dbg_scores && p < a.S) a.dbg_scores[(size_t)bh * a.S + p] = v;
    wave_hist_add(s_hist, __float_as_uint(v) >> sel_shift(0), p < n, lane);
  }
  __syncthreads();
  int* gh = a.sel_hist + (size_t)bh * kSelHist;
  for (int i = tid; i < kSelBins; i += kPoolThreads)
    if (s_hist[i]) atomicAdd(&gh[i], s_hist[i]);
}

// -------------------------------------------------------------- selection

// Exclusive scan of one whole number per thread over a block of NT threads.
template <int NT, typename I>
__device__ __forceinline__ I block_excl_scan(I v, I* s_tmp, I& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  I x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const I y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_tmp[wave] = x;
  __syncthreads();
  I off = 0, tot = 0;
#pragma unroll
  for (int w2 = 0; w2 < NT / 64; ++w2) {
    const I t = s_tmp[w2];
    if (w2 < wave) off += t;
    tot += t;
  }
  __syncthreads();
  total = tot;
  return off + x - v;
}

// Selection runs over blocks of kSelChunk consecutive scores per head, so a
// head's long score list is spread over many CUs: three radix passes (the
// first inside pool_scores) each add the block's digit histogram of the scores
// still matching a threshold's prefix into the head's pass histogram; the
// blocks of the next kernel find the digits from the completed histogram.
// Finally each block places its scores: the counts of the scores before the
// block above and equal to each threshold, taken by the block itself or on long
// lists by a launch of their own, give its output offsets and the tie
// ranks of its equal scores (ties are taken lowest position first). Short
// lists are bound by the launches and the chain of digits: 8 heads of 32K
// scores took 52 us in seven launches (8-bit passes, a count of their own) and
// take 34 us in these four, 256 heads 185 and 137 us.

// Threshold state: prefixes of the k1-th and k2-th largest score's bits and
// the ranks that remain among the scores matching them.
struct SelState {
  uint32_t pref[2];
  int krem[2];
};

// Both thresholds' digits of pass `pass` from the head's completed histograms
// (laid out as sel_at says):
// every thread holds two bins in descending digit order, a block scan counts
// the scores above them, and the bin that reaches the remaining rank is the
// digit. While the thresholds share their prefix one histogram serves both.
// Called by every thread of a kSelThreads block.
__device__ __forceinline__ void sel_digit(const int* gh, int pass, SelState& st) {
  __shared__ unsigned long long s_scan[kSelThreads / 64];
  __shared__ int s_dig[2], s_above[2];
  const int tid = threadIdx.x, top = sel_bins(pass) - 1 - 2 * tid;
  const bool shared = pass == 0 || (st.krem[0] > 0 && st.krem[1] > 0 && st.pref[0] == st.pref[1]);
  int c[2][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int* h = gh + sel_at(pass, shared ? 0 : q);
    const int2 w = top >= 1 ? *reinterpret_cast<const int2*>(h + top - 1) : make_int2(0, 0);
    c[q][0] = w.y;
    c[q][1] = w.x;
  }
  if (tid < 2) s_dig[tid] = s_above[tid] = 0;
  unsigned long long total;
  const unsigned long long ex = block_excl_scan<kSelThreads>(
      (unsigned)(c[0][0] + c[0][1]) | (unsigned long long)(unsigned)(c[1][0] + c[1][1]) << 32, s_scan, total);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int above = q == 0 ? (int)(ex & 0xffffffffu) : (int)(ex >> 32), k = st.krem[q];
    if (k > above && k <= above + c[q][0] + c[q][1]) {  // one thread
      const bool first = k <= above + c[q][0];
      s_dig[q] = first ? top : top - 1;
      s_above[q] = first ? above : above + c[q][0];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (st.krem[q] > 0) {
      st.pref[q] |= (uint32_t)s_dig[q] << sel_shift(pass);
      st.krem[q] -= s_above[q];
    }
}

// Four consecutive scores at any position (4-byte aligned).
__device__ __forceinline__ void load4(uint32_t* u, const uint32_t* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
  const u32x4 w = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) u[e] = w[e];
}

// State after pass 0 or 1, as the kernel after that pass left it.
__device__ __forceinline__ SelState sel_load(const BuildArgs& a, int bh, int pass) {
  const uint4 w = *reinterpret_cast<const uint4*>(a.sel_state + ((size_t)bh * 2 + pass) * 4);
  return SelState{{w.x, w.y}, {(int)w.z, (int)w.w}};
}

// Radix pass 1 or 2 over one block's scores: the previous pass's digits, then
// the digit histograms of the scores matching each threshold's prefix, added
// into the head's pass histogram.
template <int kPass>
__global__ __launch_bounds__(kSelThreads) void select_hist(BuildArgs a) {
  const int bh = blockIdx.z * a.Hkv + blockIdx.y;
  const HeadMeta hm = a.meta[bh];
  const int i0 = blockIdx.x * kSelChunk, n = hm.n_sc;
  if (hm.all_main || i0 >= n) return;  // block-uniform
  constexpr int kBins = sel_bins(kPass), kShift = sel_shift(kPass);
  constexpr uint32_t kMask = ~0u << sel_shift(kPass - 1);
  __shared__ int s_hist[2][kBins];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t* key = reinterpret_cast<const uint32_t*>(a.score + (size_t)bh * a.S);
  uint32_t u[kSelPer];
#pragma unroll
  for (int v = 0; v < kSelPer; ++v) {  // coalesced, all loads in flight together
    const int i = i0 + v * kSelThreads + tid;
    u[v] = i < n ? key[i] : 0u;
  }
  for (int i = tid; i < 2 * kBins; i += kSelThreads) (&s_hist[0][0])[i] = 0;
  SelState st = kPass == 1 ? SelState{{0u, 0u}, {hm.k_top, hm.k_top + hm.r_eff}} : sel_load(a, bh, 0);
  sel_digit(a.sel_hist + (size_t)bh * kSelHist, kPass - 1, st);  // synchronises the block
  if (blockIdx.x == 0 && tid == 0)
    *reinterpret_cast<uint4*>(a.sel_state + ((size_t)bh * 2 + kPass - 1) * 4) =
        make_uint4(st.pref[0], st.pref[1], (uint32_t)st.krem[0], (uint32_t)st.krem[1]);
  if (st.krem[0] <= 0 && st.krem[1] <= 0) return;  // block-uniform
  const bool shared = st.krem[0] > 0 && st.krem[1] > 0 && st.pref[0] == st.pref[1];
#pragma unroll
  for (int v = 0; v < kSelPer; ++v) {
    const bool in = i0 + v * kSelThreads + tid < n;
    const int dig = (u[v] >> kShift) & (kBins - 1);
    wave_hist_add(s_hist[0], dig, in && st.krem[0] > 0 && (u[v] & kMask) == st.pref[0], lane);
    if (!shared) wave_hist_add(s_hist[1], dig, in && st.krem[1] > 0 && (u[v] & kMask) == st.pref[1], lane);
  }
  __syncthreads();
  int* gh = a.sel_hist + (size_t)bh * kSelHist + sel_at(kPass, 0);
  for (int x = tid; x < 2 * kBins; x += kSelThreads) {
    const int c = (&s_hist[0][0])[x];
    if (c) atomicAdd(&gh[x], c);
  }
}

// Lengths of the outputs, the main list of a head that keeps every token, and
// the protected recent window behind the top-scored tokens, by block blk of
// the head.
__device__ __forceinline__ void sel_fixed(const BuildArgs& a, const HeadMeta& hm, int bh, int blk) {
  const int tid = threadIdx.x;
  int32_t* main_idx = a.main_idx + (size_t)bh * a.C;
  if (blk == 0 && tid == 0) {
    a.res_len[bh] = hm.r;
    a.main_len[bh] = hm.main_len;
  }
  if (hm.all_main) {
    for (int i = blk * kSelChunk + tid; i < min(hm.s, (blk + 1) * kSelChunk); i += kSelThreads) main_idx[i] = i;
    return;
  }
  // the protected recent window follows the top-scored tokens
  if (blk == 0)
    for (int i = tid; i < hm.P; i += kSelThreads) main_idx[hm.k_top + i] = hm.n_sc + i;
}

// Placement: main_idx (top-scored, ascending, then the protected recent
// window), elist (every other scored position, ascending) and seeds (ranks
// k1 .. k2 - 1, ascending). Each thread owns kSelPer consecutive positions
// of the block's chunk and ranks them; the block's three runs are gathered
// in LDS and stored with consecutive lanes on consecutive entries.
// Scores of a block's chunk (per consecutive positions per thread in seg, at
// most kSelPer) into the lists, given the thresholds, how many scores equal
// to each are taken, and the counts of the blocks before.
struct SelBase {
  int e1, e2, top, seed;  // equal to the thresholds, top-scored, seeds
};
__device__ __forceinline__ void sel_place(const BuildArgs& a, const HeadMeta& hm, int bh, int blk,
                                          const uint32_t (&seg)[kSelPer], int per, const SelState& st, const SelBase& base) {
  __shared__ int s_tmp[kSelThreads / 64];
  const int n = hm.n_sc, i0 = blk * kSelChunk, tid = threadIdx.x, lo = i0 + tid * per;
  int32_t* main_idx = a.main_idx + (size_t)bh * a.C;
  const uint32_t T1 = st.pref[0], T2 = st.pref[1];
  const int need1 = st.krem[0], need2 = st.krem[1];
  const bool on1 = hm.k_top > 0, on2 = hm.k_top + hm.r_eff > 0;
  const int base_e1 = base.e1, base_e2 = base.e2, base_top = base.top, base_seed = base.seed;
  const int base_ev = blk * kSelChunk - base_top;
  // equal-to-threshold counts per thread, scanned: the tie ranks
  int e1 = 0, e2 = 0;
#pragma unroll
  for (int v = 0; v < kSelPer; ++v)
    if (v < per && lo + v < n) { e1 += (seg[v] == T1); e2 += (seg[v] == T2); }
  // both counts in one scan (each block total is at most kSelChunk < 2^16)
  int tot;
  const int eb12 = block_excl_scan<kSelThreads>(e1 | (e2 << 16), s_tmp, tot);
  const int eb1 = base_e1 + (eb12 & 0xffff), eb2 = base_e2 + (eb12 >> 16);
  auto classify = [&](uint32_t u, int& r1, int& r2, bool& top, bool& sel2) {
    top = on1 && (u > T1 || (u == T1 && r1 < need1));
    sel2 = on2 && (u > T2 || (u == T2 && r2 < need2));
    r1 += (u == T1);
    r2 += (u == T2);
  };
  int c_top = 0, c_seed = 0;
  {
    int r1 = eb1, r2 = eb2;
#pragma unroll
    for (int v = 0; v < kSelPer; ++v) {
      if (v < per && lo + v < n) {
        bool top, sel2;
        classify(seg[v], r1, r2, top, sel2);
        c_top += top;
        c_seed += (sel2 && !top);
      }
    }
  }
  // block-local run offsets: top-scored from the front of s_run, evicted
  // after them (the two partition the chunk), seeds in their own buffer
  // (the evicted count of the threads before this one is their positions
  // minus their top-scored ones: every earlier thread holds per)
  int nts;
  const int ots = block_excl_scan<kSelThreads>(c_top | (c_seed << 16), s_tmp, nts);
  const int n_top = nts & 0xffff, n_seed = nts >> 16;
  const int n_valid = min(kSelChunk, n - i0);
  const int n_ev = n_valid - n_top;
  int ob_top = ots & 0xffff;
  int ob_seed = ots >> 16;
  int ob_ev = n_top + min(tid * per, n_valid) - ob_top;
  __shared__ uint16_t s_run[kSelChunk];  // positions within the block's chunk
  __shared__ uint16_t s_seed[kSelChunk];
  int r1 = eb1, r2 = eb2;
#pragma unroll
  for (int v = 0; v < kSelPer; ++v) {
    if (v < per && lo + v < n) {
      bool top, sel2;
      classify(seg[v], r1, r2, top, sel2);
      const uint16_t at = (uint16_t)(tid * per + v);
      if (top) s_run[ob_top++] = at;
      else s_run[ob_ev++] = at;
      if (sel2 && !top) s_seed[ob_seed++] = at;
    }
  }
  __syncthreads();
  int32_t* elist = a.elist + (size_t)bh * a.S;
  int32_t* seeds = a.seeds + (size_t)bh * a.Rcap;
  for (int i = tid; i < n_top + n_ev; i += kSelThreads) {
    if (i < n_top) main_idx[base_top + i] = i0 + s_run[i];
    else elist[base_ev + i - n_top] = i0 + s_run[i];
  }
  for (int i = tid; i < n_seed; i += kSelThreads) seeds[base_seed + i] = i0 + s_seed[i];
}

// Block sums of the four counts (above and equal to each threshold), above in
// the low half and equal in the high half. Called by every thread of a
// kSelThreads block.
__device__ __forceinline__ void sel_block_counts(int g1, int q1, int g2, int q2, unsigned long long& c1,
                                                 unsigned long long& c2) {
  __shared__ unsigned long long s_cnt[2][kSelThreads / 64];
  const int tid = threadIdx.x;
  c1 = (unsigned)g1 | (unsigned long long)(unsigned)q1 << 32;
  c2 = (unsigned)g2 | (unsigned long long)(unsigned)q2 << 32;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { c1 += __shfl_xor(c1, o, 64); c2 += __shfl_xor(c2, o, 64); }
  if ((tid & 63) == 0) { s_cnt[0][tid >> 6] = c1; s_cnt[1][tid >> 6] = c2; }
  __syncthreads();
  c1 = c2 = 0;
#pragma unroll
  for (int w = 0; w < kSelThreads / 64; ++w) { c1 += s_cnt[0][w]; c2 += s_cnt[1][w]; }
}

// Counts of one block's scores above and equal to the thresholds, for the
// placement of the blocks after it. Long lists only (kSelUncounted): a block of
// the placement that counts the scores before it itself saves this launch, but
// reads 32 KB per block before it through one CU, in all quadratic in the list.
// Whole constructions without residuals, 8 heads, uncounted / counted: 32K
// tokens 93 / 98 us, 64K 120 / 120, 128K 181 / 177, 512K 584 / 526, 1M 1172 / 979 (one
// head 328 / 262); other head counts cross at 64K too.
__global__ __launch_bounds__(kSelThreads) void select_count(BuildArgs a) {
  const int bh = blockIdx.z * a.Hkv + blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
  const HeadMeta hm = a.meta[bh];
  const int i0 = blk * kSelChunk, n = hm.n_sc;
  if (hm.all_main || i0 >= n) return;  // block-uniform
  const uint32_t* key = reinterpret_cast<const uint32_t*>(a.score + (size_t)bh * a.S);
  uint32_t u[kSelPer];
#pragma unroll
  for (int v = 0; v < kSelPer; ++v) {
    const int i = i0 + v * kSelThreads + tid;
    u[v] = i < n ? key[i] : 0u;
  }
  SelState st = sel_load(a, bh, 1);
  sel_digit(a.sel_hist + (size_t)bh * kSelHist, 2, st);  // synchronises the block
  int g1 = 0, q1 = 0, g2 = 0, q2 = 0;
#pragma unroll
  for (int v = 0; v < kSelPer; ++v)
    if (i0 + v * kSelThreads + tid < n) {
      g1 += u[v] > st.pref[0]; q1 += u[v] == st.pref[0];
      g2 += u[v] > st.pref[1]; q2 += u[v] == st.pref[1];
    }
  unsigned long long c1, c2;
  sel_block_counts(g1, q1, g2, q2, c1, c2);
  if (tid == 0)
    a.sel_cnt[(size_t)bh * a.NSEL + blk] =
        make_uint4((uint32_t)c1, (uint32_t)(c1 >> 32), (uint32_t)c2, (uint32_t)(c2 >> 32));
}

__global__ __launch_bounds__(kSelThreads) void select_write(BuildArgs a) {
  const int bh = blockIdx.z * a.Hkv + blockIdx.y;
  const HeadMeta hm = a.meta[bh];
  const int tid = threadIdx.x, blk = blockIdx.x;
  sel_fixed(a, hm, bh, blk);
  if (hm.all_main) return;
  if (blk * kSelChunk >= hm.n_sc) return;  // block-uniform
  const int n = hm.n_sc, i0 = blk * kSelChunk;
  const uint32_t* key = reinterpret_cast<const uint32_t*>(a.score + (size_t)bh * a.S);
  const int lo = i0 + tid * kSelPer;
  uint32_t seg[kSelPer];
  if (lo + kSelPer <= n) {
#pragma unroll
    for (int v = 0; v < kSelPer; v += 4) load4(seg + v, key + lo + v);
  } else {
#pragma unroll
    for (int v = 0; v < kSelPer; ++v) seg[v] = lo + v < n ? key[lo + v] : 0u;
  }
  // Thresholds T_q = the final prefixes; krem[q] = how many scores equal to
  // T_q are taken (lowest positions first); a threshold with k = 0 takes none.
  SelState st = sel_load(a, bh, 1);
  sel_digit(a.sel_hist + (size_t)bh * kSelHist, 2, st);  // synchronises the block
  const uint32_t T1 = st.pref[0], T2 = st.pref[1];
  // scores before this block (full chunks) above and equal to each threshold
  SelBase base{0, 0, 0, 0};
  if (blk > 0) {  // block-uniform
    int g1 = 0, q1 = 0, g2 = 0, q2 = 0;
    if (a.sel_cnt) {
      const uint4* cnt = a.sel_cnt + (size_t)bh * a.NSEL;
      for (int x = tid; x < blk; x += kSelThreads) {
        const uint4 c = cnt[x];
        g1 += (int)c.x; q1 += (int)c.y;
        g2 += (int)c.z; q2 += (int)c.w;
      }
    } else {
      constexpr int kV = 8;  // 16-byte requests in flight
      for (int x0 = 4 * tid; x0 < i0; x0 += 4 * kV * kSelThreads) {
        uint32_t u[kV][4];
#pragma unroll
        for (int v = 0; v < kV; ++v)
          if (x0 + 4 * v * kSelThreads < i0) load4(u[v], key + x0 + 4 * v * kSelThreads);
#pragma unroll
        for (int v = 0; v < kV; ++v)
          if (x0 + 4 * v * kSelThreads < i0)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              g1 += u[v][e] > T1; q1 += u[v][e] == T1;
              g2 += u[v][e] > T2; q2 += u[v][e] == T2;
            }
      }
    }
    unsigned long long c1, c2;  // above in the low half, equal in the high half
    sel_block_counts(g1, q1, g2, q2, c1, c2);
    base.e1 = (int)(c1 >> 32);
    base.e2 = (int)(c2 >> 32);
    // top scores taken, and those of ranks k1 .. k2 - 1 (the top ones are among the first k2)
    base.top = hm.k_top > 0 ? (int)(c1 & 0xffffffffu) + min(st.krem[0], base.e1) : 0;
    base.seed = (hm.k_top + hm.r_eff > 0 ? (int)(c2 & 0xffffffffu) + min(st.krem[1], base.e2) : 0) - base.top;
  }
  sel_place(a, hm, bh, blk, seg, kSelPer, st, base);
}

// Pooling and the whole selection of a head with at most kSelChunk scores in
// one block: the scores stay in registers, the passes' histograms in LDS. Such
// lists are bound by launches (2 heads of 1008 scores: 24 us in the four
// launches of the general path, 13 us here; a
// construction of 8 or 256 heads of 8100 tokens 6 or 14 us less).
__global__ __launch_bounds__(kSelThreads) void select_one(BuildArgs a) {
  const int bh = blockIdx.z * a.Hkv + blockIdx.y;
  const HeadMeta hm = a.meta[bh];
  const int tid = threadIdx.x, lane = tid & 63, n = hm.all_main ? 0 : hm.n_sc;
  const int per = (n + kSelThreads - 1) / kSelThreads, lo = tid * per;  // short lists spread over all waves
  sel_fixed(a, hm, bh, 0);
  if (a.dbg_scores)
    for (int p = n + tid; p < a.S; p += kSelThreads) a.dbg_scores[(size_t)bh * a.S + p] = -1.f;
  if (hm.all_main) return;
  __shared__ int s_hist[kSelHist];
  float v[kSelPer];
  const float* raw = a.raw + (size_t)source_head(a, bh) * a.S;
  if (per == 1) {
    float v1[1];
    pool_run(a, raw, lo, n, v1);
    v[0] = v1[0];
#pragma unroll
    for (int i = 1; i < kSelPer; ++i) v[i] = 0.f;
  } else {
    pool_run(a, raw, lo, n, v);
  }
  uint32_t seg[kSelPer];
#pragma unroll
  for (int i = 0; i < kSelPer; ++i) {
    seg[i] = __float_as_uint(v[i]);
    if (a.dbg_scores && i < per && lo + i < n) a.dbg_scores[(size_t)bh * a.S + lo + i] = v[i];
  }
  for (int i = tid; i < kSelHist; i += kSelThreads) s_hist[i] = 0;
  __syncthreads();  // the histograms are cleared
  SelState st{{0u, 0u}, {hm.k_top, hm.k_top + hm.r_eff}};
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = sel_shift(pass), bins = sel_bins(pass);
    const uint32_t mask = pass == 0 ? 0u : ~0u << sel_shift(pass > 0 ? pass - 1 : 0);
    const bool shared = pass == 0 || (st.krem[0] > 0 && st.krem[1] > 0 && st.pref[0] == st.pref[1]);
#pragma unroll
    for (int i = 0; i < kSelPer; ++i) {
      if (i >= per) break;  // block-uniform
      const bool in = lo + i < n;
      const int dig = (seg[i] >> shift) & (bins - 1);
      wave_hist_add(s_hist + sel_at(pass, 0), dig, in && (pass == 0 || (st.krem[0] > 0 && (seg[i] & mask) == st.pref[0])),
                    lane);
      if (!shared) wave_hist_add(s_hist + sel_at(pass, 1), dig, in && st.krem[1] > 0 && (seg[i] & mask) == st.pref[1], lane);
    }
    __syncthreads();
    sel_digit(s_hist, pass, st);
    __syncthreads();  // the digit scratch is free again
  }
  sel_place(a, hm, bh, 0, seg, per, st, SelBase{0, 0, 0, 0});
}

// ------------------------------------- AdaKV cross-head budget allocation

// Per sequence b (one block): the KV heads that are not all-main share their
// top-k budgets (the compared method AdaKV of App. B.2.2, which allocates
// the kept budget across heads from SnapKV scores with a safeguard
// coefficient). Head h keeps floor(safeguard * k_top_h) of its own best
// tokens; the other sum(k_top) - sum(floor) slots follow one ranking of every
// head's remaining tokens (score descending, then head, then position), a
// head taking tokens only while it holds fewer than
// cap_h = min(n_sc_h, C - r_h - P_h). A head's tokens in that ranking come
// in its own (score, position) order, so its final set is its own top-k'_h:
// only the counts k'_h are found here, and the selection then takes each
// head's top k'_h exactly as for a uniform split.
//
// With N_h(x) = the head's scored tokens above x, the ranking reaches head
// h's tokens above x after taking min(room_h, max(0, N_h(x) - floor_h)) of
// them (room_h = cap_h - floor_h). A radix search over the fp32 bit pattern
// (non-negative floats order as unsigned integers) finds the score x* of the
// last slot handed out from per-head digit histograms, in the selection's
// three passes: the first histogram is the one the pooling counted, the other
// two count the scores matching the sequence's prefix over blocks of
// kSelChunk scores, each kernel resolving the digit before it; the tokens tied
// at x* then go to the heads in ascending order. (One block per sequence
// reading every score four times took 143 us at 16 sequences of 4 heads and
// 4K-64K tokens, the three launches 50 us.)
constexpr int kAdaState = 1 + kAdaMaxHeads;  // per sequence: prefix, then the heads' tokens above its range

struct AdaShared {
  int floor[kAdaMaxHeads], room[kAdaMaxHeads], above[kAdaMaxHeads];
  int live[kAdaMaxHeads];              // 0 for heads that keep every token and take no part
  int higher[kAdaMaxHeads], equal[kAdaMaxHeads];  // of the current prefix range: tokens in higher digits, in the digit
  unsigned long long scan[kSelThreads / 64];
  int extra, total_room;
};

// The sequence's floors, rooms and slots to hand out; whether a search is
// needed. Called by every thread of a kSelThreads block.
__device__ __forceinline__ bool ada_setup(const BuildArgs& a, double safeguard, int b, AdaShared& s) {
  const int tid = threadIdx.x;
  if (tid < 64) {
    int fl = 0, room = 0, k = 0, live = 0;
    if (tid < a.Hkv) {
      const HeadMeta hm = a.meta[b * a.Hkv + tid];
      if (!hm.all_main) {
        live = 1;
        k = hm.k_top;
        fl = (int)floor(safeguard * (double)k);
        room = min(hm.n_sc, a.cap_slots - hm.r - hm.P) - fl;
      }
      s.floor[tid] = fl;
      s.room[tid] = room;
      s.above[tid] = 0;
      s.live[tid] = live;
    }
    int extra = k - fl, total = room;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { extra += __shfl_xor(extra, o, 64); total += __shfl_xor(total, o, 64); }
    if (tid == 0) { s.extra = extra; s.total_room = total; }
  }
  __syncthreads();
  return s.extra > 0 && s.total_room > s.extra;
}

// Digit of pass `pass` for the whole sequence, and each head's tokens in
// higher digits and in it. Slots handed out down to digit d are non-increasing
// in d, so the digits reaching `extra` are a prefix 0 .. d*; their count gives
// d*. Called by every thread of a kSelThreads block.
__device__ __forceinline__ int ada_digit(const BuildArgs& a, int b, int pass, AdaShared& s) {
  const int H = a.Hkv, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bins = sel_bins(pass), top = bins - 1 - 2 * tid;  // this thread's two bins, descending
  auto hist = [&](int h) {
    const size_t bh = (size_t)b * H + h;
    return pass == 0 ? a.sel_hist + bh * kSelHist : a.ada_hist + bh * kAdaHist + (pass == 2 ? kSelBins : 0);
  };
  auto load2 = [&](int h) {
    return h < H && s.live[h] && top >= 1 ? *reinterpret_cast<const int2*>(hist(h) + top - 1) : make_int2(0, 0);
  };
  long long f0 = 0, f1 = 0;  // slots handed out down to the two bins
  for (int h = 0; h < H; h += 2) {  // two heads per scan
    const int2 x = load2(h), y = load2(h + 1);
    unsigned long long all;
    const unsigned long long ex = block_excl_scan<kSelThreads>(
        (unsigned)(x.x + x.y) | (unsigned long long)(unsigned)(y.x + y.y) << 32, s.scan, all);
    auto add = [&](int hh, int e, const int2& c) {
      if (hh >= H) return;
      const int base = s.above[hh] + e - s.floor[hh];
      f0 += min(s.room[hh], max(0, base + c.y));
      f1 += min(s.room[hh], max(0, base + c.y + c.x));
    };
    add(h, (int)(ex & 0xffffffffu), x);
    add(h + 1, (int)(ex >> 32), y);
  }
  const int n0 = __syncthreads_count(top >= 1 && f0 >= s.extra), n1 = __syncthreads_count(top >= 1 && f1 >= s.extra);
  const int digit = n0 + n1 > 0 ? n0 + n1 - 1 : 0;
  for (int h = wave; h < H; h += kSelThreads / 64) {
    int hi = 0;
    if (s.live[h])
      for (int d = digit + 1 + lane; d < bins; d += 64) hi += hist(h)[d];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hi += __shfl_xor(hi, o, 64);
    if (lane == 0) {
      s.higher[h] = hi;
      s.equal[h] = s.live[h] ? hist(h)[digit] : 0;
    }
  }
  __syncthreads();
  return digit;
}

// Pass 1 or 2 of the search over one block of a head's scores.
template <int kPass>
__global__ __launch_bounds__(kSelThreads) void adakv_hist(BuildArgs a, double safeguard) {
  const int b = blockIdx.z, h = blockIdx.y, bh = b * a.Hkv + h, tid = threadIdx.x, lane = tid & 63;
  constexpr int kBins = sel_bins(kPass), kShift = sel_shift(kPass);
  constexpr uint32_t kMask = ~0u << sel_shift(kPass - 1);
  const HeadMeta hm = a.meta[bh];
  const int i0 = blockIdx.x * kSelChunk, n = hm.all_main ? 0 : hm.n_sc;
  const bool first = blockIdx.x == 0 && h == 0;  // leaves the sequence's state
  if (i0 >= n && !first) return;  // block-uniform
  __shared__ AdaShared s;
  __shared__ int s_hist[kBins];
  const uint32_t* key = reinterpret_cast<const uint32_t*>(a.score + (size_t)bh * a.S);
  uint32_t u[kSelPer];
#pragma unroll
  for (int v = 0; v < kSelPer; ++v) {
    const int i = i0 + v * kSelThreads + tid;
    u[v] = i < n ? key[i] : 0u;
  }
  for (int i = tid; i < kBins; i += kSelThreads) s_hist[i] = 0;
  if (!ada_setup(a, safeguard, b, s)) return;
  uint32_t* state = a.ada_state + (size_t)b * kAdaState;
  uint32_t prefix = 0u;
  if (kPass == 2) {
    prefix = state[0];
    if (tid < a.Hkv) s.above[tid] = (int)state[1 + tid];
    __syncthreads();
  }
  // the second pass's state goes to its own slot: blocks still read the first's
  uint32_t* next = kPass == 2 ? state + (size_t)a.B * kAdaState : state;
  prefix |= (uint32_t)ada_digit(a, b, kPass - 1, s) << sel_shift(kPass - 1);
  if (first) {
    if (tid == 0) next[0] = prefix;
    if (tid < a.Hkv) next[1 + tid] = (uint32_t)(s.above[tid] + s.higher[tid]);
  }
#pragma unroll
  for (int v = 0; v < kSelPer; ++v)
    wave_hist_add(s_hist, (u[v] >> kShift) & (kBins - 1),
                  i0 + v * kSelThreads + tid < n && (u[v] & kMask) == prefix, lane);
  __syncthreads();
  int* gh = a.ada_hist + (size_t)bh * kAdaHist + (kPass == 2 ? kSelBins : 0);
  for (int i = tid; i < kBins; i += kSelThreads)
    if (s_hist[i]) atomicAdd(&gh[i], s_hist[i]);
}

// The last digit, the counts, and the heads' sizes rewritten. One block per
// sequence.
__global__ __launch_bounds__(kSelThreads) void adakv_alloc(BuildArgs a, HeadMeta* meta, double safeguard) {
  const int b = blockIdx.x, H = a.Hkv, tid = threadIdx.x;
  __shared__ AdaShared s;
  __shared__ int s_take[kAdaMaxHeads];
  const bool search = ada_setup(a, safeguard, b, s);  // block-uniform
  if (search) {
    const uint32_t* state = a.ada_state + (size_t)(a.B + b) * kAdaState;
    if (tid < H) s.above[tid] = (int)state[1 + tid];
    __syncthreads();
    ada_digit(a, b, 2, s);
    if (tid == 0) {
      // slots above x*, then the tokens tied at x* to the heads in order
      int rem = s.extra;
      for (int h = 0; h < H; ++h) {
        s_take[h] = min(s.room[h], max(0, s.above[h] + s.higher[h] - s.floor[h]));
        rem -= s_take[h];
      }
      for (int h = 0; h < H; ++h) {
        const int gt = s.above[h] + s.higher[h], ge = gt + s.equal[h];
        const int tied = max(0, ge - s.floor[h]) - max(0, gt - s.floor[h]);
        const int t = min(min(s.room[h] - s_take[h], tied), rem);
        s_take[h] += t;
        rem -= t;
      }
    }
    __syncthreads();
  }
  if (tid >= H) return;
  HeadMeta hm = meta[b * H + tid];
  if (hm.all_main) return;
  hm.k_top = s.floor[tid] + (search ? s_take[tid] : s.extra == 0 ? 0 : s.room[tid]);
  hm.m = hm.P + hm.k_top;
  hm.main_len = hm.m;
  hm.nE = hm.s - hm.m;
  hm.r_eff = hm.r < hm.nE ? hm.r : hm.nE;
  meta[b * H + tid] = hm;
}

// ------------------------------------------------ gather + centre seeding

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void gather_init(BuildArgs a) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  constexpr int kChunks = D * (int)sizeof(T) / 16;  // 16-byte chunks per row
  const T* K = static_cast<const T*>(a.k) + (size_t)source_head(a, bh) * a.S * D;
  const T* V = static_cast<const T*>(a.v) + (size_t)source_head(a, bh) * a.S * D;
  T* kc = static_cast<T*>(a.kc) + (size_t)bh * a.C * D;
  T* vc = static_cast<T*>(a.vc) + (size_t)bh * a.C * D;
  const int32_t* main_idx = a.main_idx + (size_t)bh * a.C;
  const int rows = hm.main_len + hm.r;
  for (int x = blockIdx.x * kThreads + threadIdx.x; x < rows * kChunks; x += gridDim.x * kThreads) {
    const int row = x / kChunks, ck = x % kChunks;
    uint4 kv = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
    int dst;
    if (row < hm.main_len) {
      const int src = main_idx[row];
      kv = reinterpret_cast<const uint4*>(K + (size_t)src * D)[ck];
      vv = reinterpret_cast<const uint4*>(V + (size_t)src * D)[ck];
      dst = hm.r + row;
    } else {
      dst = row - hm.main_len;  // residual slot, cleared
    }
    reinterpret_cast<uint4*>(kc + (size_t)dst * D)[ck] = kv;
    reinterpret_cast<uint4*>(vc + (size_t)dst * D)[ck] = vv;
  }
  if (a.more) zero_sel_hist(a, bh, blockIdx.x * kThreads + threadIdx.x, gridDim.x * kThreads);
  // every log-count starts empty
  for (int j = blockIdx.x * kThreads + threadIdx.x; j < a.Rcap; j += gridDim.x * kThreads)
    a.logc[(size_t)bh * a.Rcap + j] = kNegInf;
  // seeds become the first centres, one wave per centre: the fp32 copy, the
  // bf16 hi + lo split and the squared norm, summed as the update sums it (an
  // fp64 butterfly over each 64 elements, then those partials in order)
  static_assert(D % 64 == 0, "whole waves per centre row");
  const int32_t* seeds = a.seeds + (size_t)bh * a.Rcap;
  const int lane = threadIdx.x & 63;
  const int nw = gridDim.x * (kThreads / 64);
  for (int j = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); j < hm.r_eff; j += nw) {
    const T* kr = K + (size_t)seeds[j] * D;
    const size_t ci = (size_t)bh * a.Rcap + j;
    double t = 0.0;
#pragma unroll
    for (int e0 = 0; e0 < D; e0 += 64) {
      const float x = to_f32(kr[e0 + lane]);
      const uint16_t h = f32_to_bf16_rne(x);
      a.cent[ci * D + e0 + lane] = x;
      a.cent_hi[ci * D + e0 + lane] = h;
      a.cent_lo[ci * D + e0 + lane] = f32_to_bf16_rne(x - to_f32(h));
      double sq = (double)x * x;
#pragma unroll
      for (int msk = 1; msk < 64; msk <<= 1) sq += __shfl_xor(sq, msk, 64);
      t += sq;
    }
    if (lane == 0) a.cnorm[ci] = (float)t;
  }
}

// hi = bf16(mu), lo = bf16(mu - hi), norm = ||mu||^2 (fp64 sum in a fixed
// order: a butterfly within each wave, then the waves' partials in order)
template <int D>
__device__ void prep_center(const BuildArgs& a, size_t ci, const float* mu, double* s_red) {
  static_assert(D <= kThreads, "one element per thread");
  const int tid = threadIdx.x;
  double sq = 0.0;
  if (tid < D) {
    const float x = mu[tid];
    const uint16_t h = f32_to_bf16_rne(x);
    a.cent_hi[ci * D + tid] = h;
    a.cent_lo[ci * D + tid] = f32_to_bf16_rne(x - to_f32(h));
    sq = (double)x * x;
  }
#pragma unroll
  for (int msk = 1; msk < 64; msk <<= 1) sq += __shfl_xor(sq, msk, 64);
  if ((tid & 63) == 0) s_red[tid >> 6] = sq;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < (D + 63) / 64; ++w) t += s_red[w];
    a.cnorm[ci] = (float)t;
  }
  __syncthreads();
}


// ------------------------------------------------------------------ Lloyd

// One MFMA k-step of an fp32 centre tile against one token tile, 1 element per
// lane.
template <int D>
__device__ __forceinline__ f32x4_t mma_step(const Frag<float, D>& c, const Frag<float, D>& t, int k, f32x4_t acc) {
  const float4 x = c.w[k >> 2], y = t.w[k >> 2];
  const int e = k & 3;
  return __builtin_amdgcn_mfma_f32_16x16x4f32(e == 0 ? x.x : e == 1 ? x.y : e == 2 ? x.z : x.w,
                                              e == 0 ? y.x : e == 1 ? y.y : e == 2 ? y.z : y.w, acc, 0, 0, 0);
}

// Tiling of the assignment. Each wave holds kTiles 16-token tiles of keys in
// registers and streams the centres from LDS; every centre fragment read from
// LDS feeds kTiles MFMAs per part (hi and lo for bf16), so LDS traffic per
// MFMA falls as 1 / kTiles. bf16: 4 tiles (64 tokens per wave) in blocks of 4
// waves at four waves per SIMD, so four blocks share a CU and drift out of
// step: some load keys while others run MFMAs. At d = 128 the kernel with the
// lo part stages 16 centres at a time, which keeps it within the 128
// registers of that occupancy. fp32 (twice the key registers): 2 tiles,
// 8 waves, four waves per SIMD. Histograms stay per 256-token block of the
// evicted list.
template <typename T, int D, bool kLo>
struct AssignShape {
  static constexpr bool kBf = sizeof(T) == 2;
  static constexpr int kTiles = kBf ? 4 : 2;
  static constexpr int kWaves = kBf ? 4 : 8;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kWavesPerSimd = 4;
  static constexpr int kCenters = kBf ? (kLo && D == 128 ? 16 : 32) : 64;  // centres staged in LDS per step
  static constexpr int kTokens = kWaves * 16 * kTiles;                    // evicted tokens per block
  static constexpr int kSubs = kTokens / kTokBlock;                       // histogram blocks per block
  static_assert(kTokens % kTokBlock == 0, "assignment tiling");
};

// Assignment of AssignShape::kTokens evicted tokens to the nearest centre:
// C[centre][token] = mu.k on MFMA with mu = hi + lo (bf16 pair) or fp32,
// dist = ||mu||^2 - 2 mu.k, argmin with ties to the lower centre. All token
// tiles of a wave advance through each k-step together, so the MFMA chains
// are independent. Centres past r' are staged with an infinite norm and
// never win. kLo = false drops the lo part: the first round's centres are
// bf16 key rows, so for finite keys lo is exactly zero there and the
// distances are the same bit for bit with half the MFMAs.
template <typename T, int D, bool kLo = true>
__global__ __launch_bounds__((AssignShape<T, D, kLo>::kThreads), (AssignShape<T, D, kLo>::kWavesPerSimd)) void lloyd_assign(BuildArgs a, int iter) {
  using Shape = AssignShape<T, D, kLo>;
  constexpr bool kBf = sizeof(T) == 2;
  constexpr int kTT = Shape::kTiles;
  constexpr int kSubs = Shape::kSubs;
  constexpr int kNT = Shape::kThreads;
  constexpr int kCC = Shape::kCenters;
  constexpr int kRowB = kBf ? D * 2 + 16 : D * 4 + 16;   // padded LDS row bytes
  constexpr int kSteps = kBf ? D / 32 : D / 4;           // MFMA k-steps over the lane's share of a row
  const int blk = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int t0 = blk * Shape::kTokens;
  if (hm.r_eff == 0 || t0 >= hm.nE) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;
  __shared__ __align__(16) unsigned char s_c[kCC * kRowB * (kBf ? 2 : 1)];
  __shared__ float s_norm[kCC];
  extern __shared__ int s_hist[];  // [r_eff]: one 256-token histogram block at a time

  const T* K = static_cast<const T*>(a.k) + (size_t)source_head(a, bh) * a.S * D;
  const int32_t* elist = a.elist + (size_t)bh * a.S;
  const int tw = t0 + wave * 16 * kTT;  // this wave's first token
  Frag<T, D> tk[kTT];
#pragma unroll
  for (int tt = 0; tt < kTT; ++tt) {
    const int i = min(tw + 16 * tt + col, hm.nE - 1);
    tk[tt].load(K + (size_t)elist[i] * D, grp);
  }
  // per token tile: the lane's best distance and centre (over the centres of
  // its lane group, merged across the groups at the end)
  float best[kTT];
  int bidx[kTT];
#pragma unroll
  for (int tt = 0; tt < kTT; ++tt) { best[tt] = __builtin_huge_valf(); bidx[tt] = 0x7fffffff; }

  const size_t cbase = (size_t)bh * a.Rcap;
  // centre chunks are staged through one LDS buffer; the next chunk's global
  // loads are issued before this chunk's MFMAs and written after a barrier
  constexpr int kPieces = (kBf ? D * 2 : D * 4) / 16;       // 16-byte pieces per row
  constexpr int kPer = kCC * kPieces / kNT;   // pieces per thread
  static_assert(kCC * kPieces % kNT == 0, "staging split");
  uint4 ph[kPer], pl[kPer];
  float pn = 0.f;
  auto fetch = [&](int j0) {
    const int nj = min(kCC, hm.r_eff - j0);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int x = tid + u * kNT, jj = x / kPieces, pc = x % kPieces;
      ph[u] = pl[u] = make_uint4(0, 0, 0, 0);
      if (jj < nj) {
        if (kBf) {
          ph[u] = reinterpret_cast<const uint4*>(a.cent_hi + (cbase + j0 + jj) * D)[pc];
          if (kLo) pl[u] = reinterpret_cast<const uint4*>(a.cent_lo + (cbase + j0 + jj) * D)[pc];
        } else {
          ph[u] = reinterpret_cast<const uint4*>(a.cent + (cbase + j0 + jj) * D)[pc];
        }
      }
    }
    if (tid < kCC) pn = tid < nj ? a.cnorm[cbase + j0 + tid] : __builtin_huge_valf();
  };
  auto commit = [&]() {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int x = tid + u * kNT, jj = x / kPieces, pc = x % kPieces;
      *reinterpret_cast<uint4*>(s_c + jj * kRowB + pc * 16) = ph[u];
      if (kBf && kLo) *reinterpret_cast<uint4*>(s_c + (kCC + jj) * kRowB + pc * 16) = pl[u];
    }
    if (tid < kCC) s_norm[tid] = pn;
  };
  fetch(0);
  commit();
  for (int j0 = 0; j0 < hm.r_eff; j0 += kCC) {
    const int nj = min(kCC, hm.r_eff - j0);
    __syncthreads();  // the chunk in LDS is complete
    if (j0 + kCC < hm.r_eff) fetch(j0 + kCC);
    const int nct = (nj + 15) / 16;
    for (int ct = 0; ct < nct; ++ct) {  // block-uniform
      const int crow = 16 * ct + col;
      f32x4_t acc[kTT];
#pragma unroll
      for (int tt = 0; tt < kTT; ++tt) acc[tt] = zero4();
      if constexpr (kBf) {
        // one k-step of the hi and lo centre rows at a time: 8 elements per
        // lane, the same pieces as the token fragments (Frag layout)
        const unsigned char* rh = s_c + crow * kRowB + 16 * grp;
        const unsigned char* rl = s_c + (kCC + crow) * kRowB + 16 * grp;
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
          const uint4 ch = *reinterpret_cast<const uint4*>(rh + 64 * k);
          const uint4 cl = kLo ? *reinterpret_cast<const uint4*>(rl + 64 * k) : make_uint4(0, 0, 0, 0);
#pragma unroll
          for (int tt = 0; tt < kTT; ++tt)
            acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ch), as_bf16x8(tk[tt].w[k]), acc[tt], 0, 0, 0);
          if constexpr (kLo) {
#pragma unroll
            for (int tt = 0; tt < kTT; ++tt)
              acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(cl), as_bf16x8(tk[tt].w[k]), acc[tt], 0, 0, 0);
          }
        }
      } else {
        Frag<T, D> ch;
        ch.load(reinterpret_cast<const T*>(s_c + crow * kRowB), grp);
#pragma unroll
        for (int k = 0; k < kSteps; ++k)
#pragma unroll
          for (int tt = 0; tt < kTT; ++tt) acc[tt] = mma_step<D>(ch, tk[tt], k, acc[tt]);
      }
      float nrm[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) nrm[i] = s_norm[16 * ct + 4 * grp + i];
      const int jb = j0 + 16 * ct + 4 * grp;
      // the lane's 4 centres in ascending order, then against earlier
      // tiles; each step runs for all token tiles before the next, so the
      // tiles' independent compare-select chains interleave
      float bv[kTT];
      int bi[kTT];
#pragma unroll
      for (int tt = 0; tt < kTT; ++tt) {
        bv[tt] = fmaf(-2.f, acc[tt][0], nrm[0]);
        bi[tt] = jb;
      }
#pragma unroll
      for (int i = 1; i < 4; ++i)
#pragma unroll
        for (int tt = 0; tt < kTT; ++tt) {
          const float dist = fmaf(-2.f, acc[tt][i], nrm[i]);
          const bool lt = dist < bv[tt];
          bi[tt] = lt ? jb + i : bi[tt];
          bv[tt] = lt ? dist : bv[tt];
        }
#pragma unroll
      for (int tt = 0; tt < kTT; ++tt) {
        const bool lt = bv[tt] < best[tt];
        bidx[tt] = lt ? bi[tt] : bidx[tt];
        best[tt] = lt ? bv[tt] : best[tt];
      }
    }
    if (j0 + kCC < hm.r_eff) {  // block-uniform
      __syncthreads();  // every wave is done with this chunk
      commit();
    }
  }
  // argmin across the 4 lane groups (centres interleave across them): ties
  // to the lower index
#pragma unroll
  for (int tt = 0; tt < kTT; ++tt) {
    float bv = best[tt];
    int bi = bidx[tt];
#pragma unroll
    for (int msk = 16; msk < 64; msk <<= 1) {
      const float ov = __shfl_xor(bv, msk, 64);
      const int oi = __shfl_xor(bi, msk, 64);
      if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (bi >= hm.r_eff) bi = 0;  // only reachable with non-finite keys
    bidx[tt] = bi;
    const int i = tw + 16 * tt + col;
    if (grp == 0 && i < hm.nE) {
      a.assign[(size_t)bh * a.S + i] = bi;
      if (a.dbg_assign) a.dbg_assign[((size_t)iter * a.B * a.Hkv + bh) * a.S + elist[i]] = bi;
    }
  }
  // group histograms of the 256-token blocks of the evicted list that this
  // block covers and that hold tokens, one at a time through LDS (none where
  // one block sorts the head)
  if (a.hist == nullptr) return;
  for (int q = 0; q < kSubs && t0 + q * kTokBlock < hm.nE; ++q) {  // block-uniform
    for (int j = tid; j < hm.r_eff; j += kNT) s_hist[j] = 0;
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < kTT; ++tt) {
      const int i = tw + 16 * tt + col;
      if (grp == 0 && i < hm.nE && (i - t0) / kTokBlock == q) atomicAdd(&s_hist[bidx[tt]], 1);
    }
    __syncthreads();
    int32_t* hist = a.hist + ((size_t)bh * a.NBLK + blk * kSubs + q) * a.Rcap;
    for (int j = tid; j < hm.r_eff; j += kNT) hist[j] = s_hist[j];
    __syncthreads();
  }
}

// First sorted position of group j (cnt members), and its update pieces: a
// group of up to 2^lpiece members is one piece, a larger one is cut into
// pieces that leave partial sums (parrive counts them). Called by every
// thread of an NT-thread block, in group order, `on` where it holds a group;
// the scan carries members, pieces (bits 32..47) and split groups' pieces
// (bits 48..63), each below its field's limit, from earlier calls in `carry`
// to `all`.
template <int NT>
__device__ __forceinline__ int emit_pieces(const BuildArgs& a, int bh, int j, bool on, int cnt, unsigned long long carry,
                                           unsigned long long* s_tmp, unsigned long long& all) {
  const int np = max(1, (cnt + (1 << a.lpiece) - 1) >> a.lpiece);
  const unsigned long long own =
      on ? (unsigned)cnt | (unsigned long long)np << 32 | (unsigned long long)(np > 1 ? np : 0) << 48 : 0ull;
  const unsigned long long at = carry + block_excl_scan<NT>(own, s_tmp, all);
  const int start = (int)(at & 0xffffffffu);
  if (on) {
    a.parrive[(size_t)bh * a.Rcap + j] = 0;
    int4* it = a.items + (size_t)bh * a.NIT + (int)(at >> 32 & 0xffff);
    for (int q = 0; q < np; ++q)
      it[q] = make_int4(j | q << 12, np > 1 ? (int)(at >> 48) + q : -1, start + (q << a.lpiece), cnt);
  }
  return start;
}

// Group sizes and counting-sort offsets: hist[blk][j] becomes the first
// output position of block blk's members of group j. One 1024-thread block
// per head; the groups take `cols` threads (r' rounded up to a power of two,
// at most 1024) and the histogram rows are split among the 1024 / cols row
// groups, so a head with few groups still has every thread walking rows.
constexpr int kOffThreads = 1024;
__global__ __launch_bounds__(kOffThreads) void lloyd_offsets(BuildArgs a) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  if (hm.r_eff == 0) return;
  __shared__ int s_part[kOffThreads];   // per (row group, group) row sums
  __shared__ int s_start[kOffThreads];  // first output position of each group
  __shared__ unsigned long long s_tmp[kOffThreads / 64];
  const int nblk = (hm.nE + kTokBlock - 1) / kTokBlock;
  int32_t* hist = a.hist + (size_t)bh * a.NBLK * a.Rcap;
  int lc = 0;  // log2 of cols
  while ((1 << lc) < hm.r_eff && (1 << lc) < kOffThreads) ++lc;
  const int cols = 1 << lc, ngrp = kOffThreads >> lc;
  const int c = threadIdx.x & (cols - 1), rg = threadIdx.x >> lc;
  const int per = (nblk + ngrp - 1) >> (10 - lc);
  static_assert(kOffThreads == 1 << 10, "row group split");
  const int q_lo = min(nblk, rg * per), q_hi = min(nblk, q_lo + per);
  // the rows of this thread's range are read in batches of kBatch independent
  // loads so the walk is not a chain of memory round trips
  constexpr int kBatch = 16;
  unsigned long long carry = 0;  // running totals of the passes before (emit_pieces)
  for (int j0 = 0; j0 < hm.r_eff; j0 += cols) {
    const int j = j0 + c;
    const bool act = j < hm.r_eff;
    int tot = 0;
    auto read = [&](int (&v)[kBatch], int q0) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v[u] = q0 + u < q_hi ? hist[(size_t)(q0 + u) * a.Rcap + j] : 0;
    };
    if (act)
      for (int q0 = q_lo; q0 < q_hi; q0 += kBatch) {
        int v[kBatch];
        read(v, q0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) tot += v[u];
      }
    s_part[threadIdx.x] = tot;
    __syncthreads();
    int before = 0, col_tot = 0;  // rows of lower row groups come first
    for (int g2 = 0; g2 < ngrp; ++g2) {
      const int v = s_part[g2 * cols + c];
      before += g2 < rg ? v : 0;
      col_tot += v;
    }
    unsigned long long all;
    const int start = emit_pieces<kOffThreads>(a, bh, j, rg == 0 && act, col_tot, carry, s_tmp, all);
    if (rg == 0) s_start[c] = start;  // the row-group-0 threads come first in the scan
    __syncthreads();
    if (act) {
      int run = s_start[c] + before;
      for (int q0 = q_lo; q0 < q_hi; q0 += kBatch) {
        int v[kBatch];
        read(v, q0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          if (q0 + u < q_hi) hist[(size_t)(q0 + u) * a.Rcap + j] = run;
          run += v[u];
        }
      }
    }
    carry += all;
    __syncthreads();  // s_part and s_start are rewritten by the next pass
  }
  if (threadIdx.x == 0) a.nitem[bh] = (int)(carry >> 32 & 0xffff);
}

// Rank of this lane's token among the earlier lanes' tokens of the same group
// (r_eff groups, one ballot per bit of the group index); peers = the lanes of
// that group. Called by every lane of the wave, `live` where it holds a token.
__device__ __forceinline__ int wave_group_rank(int g, bool live, int r_eff, int lane, uint64_t& peers) {
  peers = __ballot(live);
  const int nbits = r_eff > 1 ? 32 - __clz(r_eff - 1) : 0;
  for (int bit = 0; bit < nbits; ++bit) {
    const bool on = (g >> bit) & 1;
    const uint64_t set = __ballot(live && on);
    peers &= on ? set : ~set;
  }
  return __popcll(peers & ((1ull << lane) - 1));
}

// The whole counting sort of a head with few evicted tokens in one block: the
// tokens in 64-token batches (up to kSortBatches per wave), a table of the
// batches' group counts in LDS, prefixes over the batches and the groups, then
// the stable placement. It takes the place of the per-block histograms, the
// offsets and the scatter where those are bound by their launches (2 heads of
// 928 tokens: 8.4 + 3.2 -> 5.2 us a round). The table and the batches per wave
// set the line: 16384 entries of 16 bits, 128 batches (8192 tokens), 1024
// groups.
constexpr int kSortThreads = 1024;
constexpr int kSortBatches = 8;
constexpr int kSortTable = 16384;
__global__ __launch_bounds__(kSortThreads) void lloyd_sort(BuildArgs a) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int r = hm.r_eff;
  if (r == 0) return;
  __shared__ __align__(4) uint16_t s_cnt[kSortTable];  // [batch][group] counts, then prefixes over the batches
  __shared__ int s_start[kSortThreads];
  __shared__ unsigned long long s_tmp[kSortThreads / 64];
  constexpr int kNW = kSortThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = (hm.nE + 63) / 64;
  int g[kSortBatches], src[kSortBatches], rank[kSortBatches];
#pragma unroll
  for (int k = 0; k < kSortBatches; ++k) {
    const int i = (k * kNW + wave) * 64 + lane;
    g[k] = i < hm.nE ? a.assign[(size_t)bh * a.S + i] : 0;
    src[k] = i < hm.nE ? a.elist[(size_t)bh * a.S + i] : 0;
  }
  for (int x = tid; x < (nb * r + 1) / 2; x += kSortThreads) reinterpret_cast<uint32_t*>(s_cnt)[x] = 0;
  __syncthreads();  // the table is cleared
#pragma unroll
  for (int k = 0; k < kSortBatches; ++k) {
    const int q = k * kNW + wave;
    if (q >= nb) break;  // wave-uniform
    const bool live = q * 64 + lane < hm.nE;
    uint64_t peers;
    rank[k] = wave_group_rank(g[k], live, r, lane, peers);
    if (live && rank[k] == 0) s_cnt[q * r + g[k]] = (uint16_t)__popcll(peers);
  }
  __syncthreads();
  int run = 0;
  if (tid < r)
    for (int q0 = 0; q0 < nb; q0 += 8) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = q0 + u < nb ? s_cnt[(q0 + u) * r + tid] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (q0 + u < nb) s_cnt[(q0 + u) * r + tid] = (uint16_t)run;
        run += v[u];
      }
    }
  unsigned long long all;
  s_start[tid] = emit_pieces<kSortThreads>(a, bh, tid, tid < r, run, 0ull, s_tmp, all);
  if (tid == 0) a.nitem[bh] = (int)(all >> 32 & 0xffff);
  __syncthreads();  // starts and prefixes are complete
#pragma unroll
  for (int k = 0; k < kSortBatches; ++k) {
    const int q = k * kNW + wave;
    if (q >= nb) break;
    if (q * 64 + lane < hm.nE) a.order[(size_t)bh * a.S + s_start[g[k]] + s_cnt[q * r + g[k]] + rank[k]] = src[k];
  }
}

// Stable placement: members of a group keep ascending evicted order. A
// token's rank inside its 256-token block is the number of earlier tokens
// there in the same group: within a wave, the lanes sharing its group come
// from one ballot per bit of the group index; across the block's waves, from
// a per-wave count table in LDS (dynamic, kTokBlock / 64 rows of r' ints).
__global__ __launch_bounds__(kTokBlock) void lloyd_scatter(BuildArgs a) {
  const int blk = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const HeadMeta hm = a.meta[bh];
  const int t0 = blk * kTokBlock;
  if (hm.r_eff == 0 || t0 >= hm.nE) return;
  constexpr int kNW = kTokBlock / 64;
  extern __shared__ int s_cnt[];  // [kNW][r_eff]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = t0 + tid;
  const bool live = i < hm.nE;
  const int g = live ? a.assign[(size_t)bh * a.S + i] : 0;
  const int src = live ? a.elist[(size_t)bh * a.S + i] : 0;
  for (int j = tid; j < kNW * hm.r_eff; j += kTokBlock) s_cnt[j] = 0;
  uint64_t peers;
  const int in_wave = wave_group_rank(g, live, hm.r_eff, lane, peers);
  __syncthreads();  // the table is cleared
  if (live && in_wave == 0) s_cnt[wave * hm.r_eff + g] = __popcll(peers);
  __syncthreads();
  if (!live) return;
  int rank = in_wave;
  for (int w = 0; w < wave; ++w) rank += s_cnt[w * hm.r_eff + g];
  const int dst = a.hist[((size_t)bh * a.NBLK + blk) * a.Rcap + g] + rank;
  a.order[(size_t)bh * a.S + dst] = src;
}

// Member indices q, q + NG, q + 2NG, q + 3NG of a piece's sorted list of cnt
// members (past its end the last member's).
__device__ __forceinline__ void load_ids(int (&id)[4], const int32_t* mem, int q, int NG, int cnt) {
#pragma unroll
  for (int u = 0; u < 4; ++u) id[u] = mem[min(q + u * NG, cnt - 1)];
}

// acc += the 8 elements of one row piece (zeros where the row is past the end)
__device__ __forceinline__ void add_row(double (&acc)[8], uint4 w, bool in) {
  const uint32_t pw[4] = {in ? w.x : 0u, in ? w.y : 0u, in ? w.z : 0u, in ? w.w : 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[2 * e] += (double)bf16_lo(pw[e]);
    acc[2 * e + 1] += (double)bf16_hi(pw[e]);
  }
}

// New centre of a group = fp64 mean of its members' keys, summed in a fixed
// order; an empty group keeps its centre. The last round also writes the
// entry: mean key and mean value in the cache dtype, and log c_j. One block
// per piece: a group of up to 2^lpiece members, or that many members of a
// larger one, whose pieces leave their sums and whose last piece to arrive
// adds them in piece order. Bound by the gathered rows' HBM traffic once no
// block runs long: the first round's groups, grown around single seed keys,
// run from a few members to tens of thousands, and with one block per group
// the largest one set the time (32 heads of 130K tokens, 0 to 256 groups:
// first round 519 -> 172 us, later rounds 191-213 -> 174 us; 8 heads of 32K
// tokens: 78 -> 16 us and 18-30 -> 15 us).
// Each thread keeps four member rows in flight and requests the next four
// members' indices right behind them; the last step is padded with the last
// member (added as zeros), so a group of 64 members or fewer costs one round
// trip for the indices and one for the rows. bf16 rows stay packed until they
// are added (seven blocks per CU).
// kKV (last round, bf16): each member's key and value rows are read in the
// same loop, twice the rows in flight of two passes one after the other.
template <typename T, int D, bool kKV = false>
__global__ __launch_bounds__(kThreads, (kKV && sizeof(T) == 2 ? 4 : sizeof(T) == 2 ? 7 : 4)) void lloyd_update(BuildArgs a, int last, int rev) {
  int b, kvh, bh;
  block_head(a, rev, b, kvh, bh);
  const HeadMeta hm = a.meta[bh];
  if (hm.r_eff == 0 || (int)blockIdx.x >= a.nitem[bh]) return;
  constexpr int CPR = D / 8;            // lanes per row, 8 elements each
  constexpr int NG = kThreads / CPR;    // member groups
  __shared__ double s_sum[NG][D];
  __shared__ float s_mu[D];
  __shared__ double s_red[D];
  __shared__ int s_last;
  const int tid = threadIdx.x, c = tid % CPR, g = tid / CPR;
  const int4 item = a.items[(size_t)bh * a.NIT + blockIdx.x];
  const int j = item.x & 0xfff, piece = item.x >> 12, total = item.w;
  const size_t ci = (size_t)bh * a.Rcap + j;
  const int cnt = min(1 << a.lpiece, total - (piece << a.lpiece));  // members of this piece
  const int32_t* mem = a.order + (size_t)bh * a.S + item.z;
  const T* K = static_cast<const T*>(a.k) + (size_t)source_head(a, bh) * a.S * D;
  const T* V = static_cast<const T*>(a.v) + (size_t)source_head(a, bh) * a.S * D;
  double sk = 0.0, sv = 0.0;  // key and value sums of column tid (threads tid < D)
  // the member groups' sums of one column in ascending order
  auto reduce = [&](const double (&acc)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s_sum[g][8 * c + e] = acc[e];
    __syncthreads();
    double t = 0.0;
    if (tid < D)
      for (int gg = 0; gg < NG; ++gg) t += s_sum[gg][tid];
    __syncthreads();
    return t;
  };
  int id[4];
  if constexpr (kKV && sizeof(T) == 2) {
    // last round: the key and value rows of each member are read together
    // (twice the rows in flight), each summed in member order as below
    double ak[8], av[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) ak[e] = av[e] = 0.0;
    if (g < cnt) load_ids(id, mem, g, NG, cnt);
    for (int q = g; q < cnt; q += 4 * NG) {
      uint4 wk[4], wv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t off = (size_t)id[u] * D + 8 * c;
        wk[u] = *reinterpret_cast<const uint4*>(K + off);
        wv[u] = *reinterpret_cast<const uint4*>(V + off);
      }
      if (q + 4 * NG < cnt) load_ids(id, mem, q + 4 * NG, NG, cnt);  // the next rows' indices
#pragma unroll
      for (int u = 0; u < 4; ++u) add_row(ak, wk[u], q + u * NG < cnt);
#pragma unroll
      for (int u = 0; u < 4; ++u) add_row(av, wv[u], q + u * NG < cnt);
    }
    sk = reduce(ak);
    sv = reduce(av);
  } else {
    for (int pass = 0; pass < (last ? 2 : 1); ++pass) {
      const T* X = pass == 0 ? K : V;
      double acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.0;
      // members g, g + NG, g + 2NG, ... in order
      if (g < cnt) load_ids(id, mem, g, NG, cnt);
      for (int q = g; q < cnt; q += 4 * NG) {
        if constexpr (sizeof(T) == 2) {  // rows stay packed until added: 4 registers each
          uint4 w[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] = *reinterpret_cast<const uint4*>(X + (size_t)id[u] * D + 8 * c);
          if (q + 4 * NG < cnt) load_ids(id, mem, q + 4 * NG, NG, cnt);
#pragma unroll
          for (int u = 0; u < 4; ++u) add_row(acc, w[u], q + u * NG < cnt);
        } else {
          float x[4][8];
#pragma unroll
          for (int u = 0; u < 4; ++u) load8_f32(X + (size_t)id[u] * D + 8 * c, x[u]);
          if (q + 4 * NG < cnt) load_ids(id, mem, q + 4 * NG, NG, cnt);
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += q + u * NG < cnt ? (double)x[u][e] : 0.0;
        }
      }
      const double t = reduce(acc);
      if (pass == 0) sk = t;
      else sv = t;
    }
  }
  if (item.y >= 0) {  // block-uniform: a piece of a split group
    // Partial sums and arrivals go through agent-scope accesses (the pieces
    // run on several XCDs, whose L2s do not see each other's plain stores);
    // every store has completed before the block counts itself in, so the
    // block that counts last reads complete sums. That order rests on the
    // wait and on stores that write through and loads that bypass, not on
    // the language's release and acquire: at agent scope those write back and
    // invalidate the whole L2 (a split-K merge ordered that way ran 7 times
    // slower).
    const int np = (total + (1 << a.lpiece) - 1) >> a.lpiece;
    unsigned long long* part = reinterpret_cast<unsigned long long*>(a.part) + (size_t)bh * a.NPART * 2 * D;
    auto slot = [&](int p, int q) { return &part[((size_t)p * 2 + q) * D + tid]; };
    if (tid < D) {
      __hip_atomic_store(slot(item.y, 0), (unsigned long long)__double_as_longlong(sk), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      if (last)
        __hip_atomic_store(slot(item.y, 1), (unsigned long long)__double_as_longlong(sv), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(&a.parrive[ci], 1) == np - 1;
    __syncthreads();
    if (!s_last) return;
    asm volatile("" ::: "memory");
    auto gather = [&](int q) {
      double t = 0.0;
      for (int p0 = 0; p0 < np; p0 += 8) {  // 8 partial sums in flight, added in piece order
        unsigned long long v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          v[u] = __hip_atomic_load(slot(item.y - piece + min(p0 + u, np - 1), q), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < 8; ++u) t += p0 + u < np ? __longlong_as_double((long long)v[u]) : 0.0;
      }
      return t;
    };
    if (tid < D) {
      sk = gather(0);
      if (last) sv = gather(1);
    }
  }
  if (tid < D) {
    const float mu = total > 0 ? (float)(sk / total) : a.cent[ci * D + tid];  // empty group keeps its centre
    a.cent[ci * D + tid] = mu;
    s_mu[tid] = mu;
    if (last) {
      store_elem(static_cast<T*>(a.kc) + ((size_t)bh * a.C + j) * D + tid, mu);
      store_elem(static_cast<T*>(a.vc) + ((size_t)bh * a.C + j) * D + tid, total > 0 ? (float)(sv / total) : 0.f);
    }
  }
  if (last) {
    if (tid == 0) a.logc[ci] = total > 0 ? logf((float)total) : kNegInf;
    return;
  }
  __syncthreads();
  prep_center<D>(a, ci, s_mu, s_red);
}

__global__ void fill_i32(int32_t* p, size_t n, int32_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Debug export of the centres round `iter` assigns against: rows j < r' of
// the fp32 centres, zero rows after them.
__global__ __launch_bounds__(kThreads) void export_centres(BuildArgs a, int iter, int D) {
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int bh = b * a.Hkv + kvh;
  const int r_eff = a.meta[bh].r_eff;
  const size_t n = (size_t)a.Rcap * D;
  const float* src = a.cent + (size_t)bh * n;
  float* dst = a.dbg_centers + ((size_t)iter * a.B * a.Hkv + bh) * n;
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads)
    dst[i] = (int)(i / D) < r_eff ? src[i] : 0.f;
}

// Sizes of one (b, kv head) from its context length s, residual count r and
// budget b (main-selection equation, Sec. 5.2; reading R4 for |P|).
__host__ __device__ inline HeadMeta make_meta(int s, int r, int budget, int recent) {
  HeadMeta m{};
  m.s = s;
  m.r = r;
  m.m = budget - r;
  m.all_main = s <= m.m;
  m.P = m.all_main ? 0 : (recent < m.m ? recent : m.m);
  if (m.P > s) m.P = s;
  m.n_sc = m.all_main ? 0 : s - m.P;
  m.k_top = m.all_main ? 0 : m.m - m.P;
  m.nE = m.all_main ? 0 : s - m.m;
  m.r_eff = r < m.nE ? r : m.nE;
  m.main_len = m.all_main ? s : m.m;
  return m;
}

// Per-head sizes travel as kernel arguments (copied at launch), in chunks.
constexpr int kMetaChunk = 256;
struct MetaChunk {
  int first, count, recent;
  int s[kMetaChunk], r[kMetaChunk], budget[kMetaChunk];
};

__global__ void meta_kernel(HeadMeta* meta, MetaChunk c) {
  const int i = threadIdx.x;
  if (i < c.count) meta[c.first + i] = make_meta(c.s[i], c.r[i], c.budget[i], c.recent);
}

// Arguments of every construction kernel; `meta` and the outputs belong to
// the candidate being built, the scratch to the plan's workspace.
BuildArgs make_args(const BuildPlan& pl, const void* k, const void* v, const void* q_obs, const HeadMeta* meta,
                    const BuildOut& out, float* dbg_scores, int32_t* dbg_assign, float* dbg_centers,
                    void* workspace) {
  char* ws = static_cast<char*>(workspace);
  BuildArgs a{};
  a.k = k; a.v = v; a.q_obs = q_obs;
  a.kc = out.kc; a.vc = out.vc; a.logc = out.logc; a.main_idx = out.main_idx;
  a.res_len = out.res_len; a.main_len = out.main_len;
  a.dbg_scores = dbg_scores; a.dbg_assign = dbg_assign; a.dbg_centers = dbg_centers;
  a.meta = meta;
  a.lse_part = reinterpret_cast<float2*>(ws + pl.off_lsep);
  a.lse2 = reinterpret_cast<float*>(ws + pl.off_lse);
  a.raw = reinterpret_cast<float*>(ws + pl.off_raw);
  a.score = reinterpret_cast<float*>(ws + pl.off_score);
  a.elist = reinterpret_cast<int32_t*>(ws + pl.off_elist);
  a.seeds = reinterpret_cast<int32_t*>(ws + pl.off_seeds);
  a.cent = reinterpret_cast<float*>(ws + pl.off_cent);
  a.cent_hi = reinterpret_cast<uint16_t*>(ws + pl.off_chi);
  a.cent_lo = reinterpret_cast<uint16_t*>(ws + pl.off_clo);
  a.cnorm = reinterpret_cast<float*>(ws + pl.off_cnorm);
  a.assign = reinterpret_cast<int32_t*>(ws + pl.off_assign);
  a.hist = pl.one_sort ? nullptr : reinterpret_cast<int32_t*>(ws + pl.off_hist);
  a.order = reinterpret_cast<int32_t*>(ws + pl.off_order);
  a.items = reinterpret_cast<int4*>(ws + pl.off_items);
  a.nitem = reinterpret_cast<int32_t*>(ws + pl.off_nitem);
  a.parrive = reinterpret_cast<int32_t*>(ws + pl.off_parrive);
  a.part = reinterpret_cast<double*>(ws + pl.off_part);
  a.lpiece = pl.lpiece; a.NIT = pl.NIT; a.NPART = pl.NPART;
  a.sel_hist = pl.sel_multi ? reinterpret_cast<int32_t*>(ws + pl.off_selh) : nullptr;
  a.sel_state = reinterpret_cast<uint32_t*>(ws + pl.off_sels);
  a.sel_cnt = pl.count_sel ? reinterpret_cast<uint4*>(ws + pl.off_selc) : nullptr;
  a.NC = pl.NC; a.SBH = pl.B * pl.Hkv;
  a.B = pl.B; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.G = pl.G; a.C = pl.C; a.Rcap = pl.Rcap; a.S = pl.S; a.w = pl.w;
  a.wr = pl.wr; a.pool_half = pl.pool_half; a.R = pl.R; a.LG = pl.LG; a.KG = pl.KG; a.NCH = pl.NCH; a.NBLK = pl.NBLK;
  a.NSEL = pl.NSEL; a.T = pl.T;
  a.cap_slots = pl.C;
  a.scale2 = kLog2e / sqrtf((float)pl.D);
  return a;
}

#define RESKV_CHECK() do { e = hipGetLastError(); if (e != hipSuccess) return e; } while (0)

// Raw window scores of every scored position: the log-sum-exp per window row,
// then the normalised weights summed. Which shapes: up to 128 rows one chunk
// of rows; more than 128 the wide chunk, at bf16 rows or rows of 64 (fp32 rows
// of 128 would hold one block per CU); and for fp32 the lse pass's rows dealt
// to blocks 16 at a time where the chunks alone give a CU under two blocks.
template <typename T, int D>
hipError_t launch_scores_typed(const BuildPlan& pl, const BuildArgs& a, hipStream_t st) {
  auto grid = [&](int x) { return dim3(x < 1 ? 1 : x, pl.Hkv, pl.B); };
  hipError_t e;
  const dim3 gf = grid((pl.R + kThreads - 1) / kThreads);
  constexpr bool kBf = sizeof(T) == 2;
  const bool wide = (kBf || D == 64) && pl.R > kRowChunk, few = pl.deal_rows;
  if constexpr (!kBf)
    if (few)
      hipLaunchKernelGGL((lse_partial<T, D, 16, 1, true>), grid(pl.NCH * ((pl.R + 15) / 16)), dim3(256), 0, st, a);
  if constexpr (kBf || D == 64)
    if (wide && (kBf || !few))
      hipLaunchKernelGGL((lse_partial<T, D, kRowChunkWide, 2, false>), grid(pl.NCH), dim3(512), 0, st, a);
  if (!wide && (kBf || !few))
    hipLaunchKernelGGL((lse_partial<T, D, kRowChunk, 1, false>), grid(pl.NCH), dim3(256), 0, st, a);
  RESKV_CHECK();
  hipLaunchKernelGGL(lse_final, gf, dim3(kThreads), 0, st, a); RESKV_CHECK();
  // the second pass over the keys walks the heads in reverse (cache reuse)
  if constexpr (kBf || D == 64)
    if (wide) {
      hipLaunchKernelGGL((score_accum<T, D, kRowChunkWide, 512>), grid(pl.NSC), dim3(512), 0, st, a, 1);
      RESKV_CHECK();
      return hipSuccess;
    }
  hipLaunchKernelGGL((score_accum<T, D, kRowChunk, 256>), grid(pl.NSC), dim3(256), 0, st, a, 1); RESKV_CHECK();
  return hipSuccess;
}

// Pooling, selection, gather and the Lloyd rounds of one candidate.
template <typename T, int D>
hipError_t launch_candidate_typed(const BuildPlan& pl, const BuildArgs& a, hipStream_t st,
                                  HeadMeta* alloc_meta = nullptr, double safeguard = 1.0) {
  const dim3 bhg(1, pl.Hkv, a.B);
  auto grid = [&](int x) { return dim3(x < 1 ? 1 : x, pl.Hkv, a.B); };
  hipError_t e;
  if (a.dbg_assign) {
    hipLaunchKernelGGL(fill_i32, dim3(1024), dim3(256), 0, st, a.dbg_assign,
                       (size_t)pl.T * pl.B * pl.Hkv * pl.S, -1);
    RESKV_CHECK();
  }
  constexpr int kPoolChunk = kPoolThreads * kPoolPer;
  if (!pl.sel_multi) {
    hipLaunchKernelGGL(select_one, bhg, dim3(kSelThreads), 0, st, a); RESKV_CHECK();
  } else {
    hipLaunchKernelGGL(pool_scores, grid((pl.S + kPoolChunk - 1) / kPoolChunk), dim3(kPoolThreads), 0, st, a);
    RESKV_CHECK();
    if (alloc_meta) {
      hipLaunchKernelGGL(adakv_hist<1>, grid(pl.NSEL), dim3(kSelThreads), 0, st, a, safeguard); RESKV_CHECK();
      hipLaunchKernelGGL(adakv_hist<2>, grid(pl.NSEL), dim3(kSelThreads), 0, st, a, safeguard); RESKV_CHECK();
      hipLaunchKernelGGL(adakv_alloc, dim3(pl.B), dim3(kSelThreads), 0, st, a, alloc_meta, safeguard);
      RESKV_CHECK();
    }
    hipLaunchKernelGGL(select_hist<1>, grid(pl.NSEL), dim3(kSelThreads), 0, st, a); RESKV_CHECK();
    hipLaunchKernelGGL(select_hist<2>, grid(pl.NSEL), dim3(kSelThreads), 0, st, a); RESKV_CHECK();
    if (pl.count_sel) {
      hipLaunchKernelGGL(select_count, grid(pl.NSEL), dim3(kSelThreads), 0, st, a); RESKV_CHECK();
    }
    hipLaunchKernelGGL(select_write, grid(pl.NSEL), dim3(kSelThreads), 0, st, a); RESKV_CHECK();
  }
  const int rows = pl.max_main + pl.Rcap;
  const int gblocks = (rows * (D * (int)sizeof(T) / 16) + kThreads - 1) / kThreads;
  hipLaunchKernelGGL((gather_init<T, D>), grid(gblocks < 64 ? gblocks : 64), dim3(kThreads), 0, st, a);
  RESKV_CHECK();
  if (pl.max_reff > 0) {
    const size_t hist_lds = (size_t)pl.max_reff * sizeof(int);
    using S1 = AssignShape<T, D, false>;
    using S2 = AssignShape<T, D, true>;
    for (int it = 0; it < pl.T; ++it) {
      if (a.dbg_centers) {
        hipLaunchKernelGGL(export_centres, grid((pl.Rcap * D + kThreads * 8 - 1) / (kThreads * 8)), dim3(kThreads),
                           0, st, a, it, D);
        RESKV_CHECK();
      }
      if (sizeof(T) == 2 && it == 0)  // centres are the seeds' bf16 keys: lo = 0
        hipLaunchKernelGGL((lloyd_assign<T, D, false>), grid((pl.max_E + S1::kTokens - 1) / S1::kTokens),
                           dim3(S1::kThreads), hist_lds, st, a, it);
      else
        hipLaunchKernelGGL((lloyd_assign<T, D>), grid((pl.max_E + S2::kTokens - 1) / S2::kTokens), dim3(S2::kThreads),
                           hist_lds, st, a, it);
      RESKV_CHECK();
      if (pl.one_sort) {
        hipLaunchKernelGGL(lloyd_sort, bhg, dim3(kSortThreads), 0, st, a); RESKV_CHECK();
      } else {
        hipLaunchKernelGGL(lloyd_offsets, bhg, dim3(kOffThreads), 0, st, a); RESKV_CHECK();
        hipLaunchKernelGGL(lloyd_scatter, grid(pl.NBLK), dim3(kTokBlock), (kTokBlock / 64) * hist_lds, st, a);
        RESKV_CHECK();
      }
      // the update walks the heads in reverse of the assignment before and
      // after it, so each starts on the keys the other read last
      const int last = it == pl.T - 1 ? 1 : 0;
      if (last)
        hipLaunchKernelGGL((lloyd_update<T, D, true>), grid(pl.NIT), dim3(kThreads), 0, st, a, last, 1);
      else
        hipLaunchKernelGGL((lloyd_update<T, D>), grid(pl.NIT), dim3(kThreads), 0, st, a, last, 1);
      RESKV_CHECK();
    }
  }
  return hipSuccess;
}

#undef RESKV_CHECK

}  // namespace

void head_meta(const BuildPlan& pl, const int32_t* seq_len, const int32_t* budget, const int32_t* res_count,
               int recent, std::vector<HeadMeta>& out) {
  out.resize((size_t)pl.B * pl.Hkv);
  for (int b = 0; b < pl.B; ++b)
    for (int h = 0; h < pl.Hkv; ++h)
      out[(size_t)b * pl.Hkv + h] = make_meta(seq_len[b], res_count[b * pl.Hkv + h], budget[b], recent);
}

void init_build_plan(const reskv_shape_t& s, const reskv_build_params_t& p, BuildPlan* plan) {
  BuildPlan& pl = *plan;
  pl = BuildPlan{};
  pl.B = s.batch; pl.Hq = s.num_q_heads; pl.Hkv = s.num_kv_heads; pl.G = s.num_q_heads / s.num_kv_heads;
  pl.D = s.head_dim; pl.C = s.slot_cap; pl.Rcap = s.res_cap; pl.S = p.max_seq_len; pl.w = p.obs_window;
  pl.wr = p.fit_rows > 0 ? p.fit_rows : p.obs_window;
  pl.pool_half = (p.pool_kernel > 0 ? p.pool_kernel : 5) / 2;
  pl.NC = 1;
  pl.R = pl.G * pl.wr; pl.T = p.lloyd_iters; pl.dtype = s.dtype;
}

bool fold_build_plan(const std::vector<HeadMeta>& hm, BuildPlan* plan) {
  BuildPlan& pl = *plan;
  for (const HeadMeta& m : hm) {
    if (m.s > pl.max_s) pl.max_s = m.s;
    if (m.main_len > pl.max_main) pl.max_main = m.main_len;
    if (m.r_eff > pl.max_reff) pl.max_reff = m.r_eff;
    if (m.nE > pl.max_E) pl.max_E = m.nE;
    if (m.main_len + m.r > pl.C) return false;
  }
  return true;
}

bool layout_build_plan(BuildPlan* plan) {
  BuildPlan& pl = *plan;
  if (pl.R > 1024 || pl.Rcap > 4096) return false;
  const size_t BH = (size_t)pl.B * pl.Hkv;
  const size_t CH = BH * pl.NC;  // heads the candidates build at a time
  // the lse pass takes 16, 8 or 4 key groups per block: the longest chunks
  // that still give at least 1024 blocks (fewer blocks write fewer partial
  // records and stage the window rows fewer times)
  pl.LG = kKeyGroups;
  for (int lg = 16; lg > kKeyGroups; lg /= 2)
    if (BH * (size_t)((pl.max_s + 256 * lg - 1) / (256 * lg)) >= 1024) {
      pl.LG = lg;
      break;
    }
  pl.NCH = (pl.max_s + 256 * pl.LG - 1) / (256 * pl.LG);
  pl.deal_rows = pl.dtype == RESKV_F32 && BH * pl.NCH <= kDealtChunks;
  const size_t score_blocks = BH * (size_t)((pl.max_s + 256 * kKeyGroups - 1) / (256 * kKeyGroups));
  const int few_blocks = pl.dtype == RESKV_BF16 && pl.R > kRowChunk ? kFewScoreBlocksWide : kFewScoreBlocks;
  pl.KG = score_blocks <= (size_t)few_blocks ? 1 : kKeyGroups;
  pl.NSC = (pl.max_s + 256 * pl.KG - 1) / (256 * pl.KG);
  pl.NBLK = (pl.max_E + kTokBlock - 1) / kTokBlock;
  if (pl.NBLK < 1) pl.NBLK = 1;
  pl.NSEL = (pl.max_s + kSelChunk - 1) / kSelChunk;
  if (pl.NSEL < 1) pl.NSEL = 1;
  pl.sel_multi = pl.cross_head || pl.NSEL > 1;
  pl.count_sel = pl.NSEL > kSelUncounted;
  const int nb64 = (pl.max_E + 63) / 64;
  pl.one_sort = nb64 <= kSortBatches * (kSortThreads / 64) && pl.max_reff <= kSortThreads &&
                (long long)nb64 * pl.max_reff <= kSortTable;
  // update pieces of 256 members while the whole construction has fewer than
  // kPieceMin of 1024 (short chains where few blocks are in flight), else 1024.
  // Whole constructions of 128K tokens, pieces of 1024 / 256: one head, 256
  // groups of like size 347 / 336 us, one of them large 358 / 334; 8 heads 999 / 989
  // and 1010 / 975; 30 heads 3205 / 3252. A group that holds all tokens has 512
  // pieces to add: 8 heads in one group 830 / 1073 (one block per group: 6416).
  pl.lpiece = CH * (size_t)((pl.max_E + 1023) / 1024) < kPieceMin ? 8 : 10;
  while (pl.max_E >> pl.lpiece > 16384) ++pl.lpiece;  // piece counts stay below 2^16 (lloyd_offsets packs them)
  const int pieces = pl.max_reff > 0 ? pl.max_E >> pl.lpiece : 0;
  pl.NIT = pl.max_reff + pieces;  // sum over groups of max(1, ceil(count / piece))
  pl.NPART = 2 * pieces;        // groups above one piece: ceil(c / piece) <= 2 c / piece
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = align_up(off + bytes, 256); return o; };
  pl.off_meta = take(BH * sizeof(HeadMeta));
  pl.off_lsep = take(BH * pl.NCH * pl.R * sizeof(float2));
  pl.off_lse = take(BH * pl.R * sizeof(float));
  pl.off_raw = take(BH * pl.S * sizeof(float));
  pl.off_score = take(CH * pl.S * sizeof(float));
  pl.off_elist = take(CH * pl.S * sizeof(int32_t));
  pl.off_seeds = take(CH * pl.Rcap * sizeof(int32_t));
  pl.off_cent = take(CH * pl.Rcap * pl.D * sizeof(float));
  pl.off_chi = take(CH * pl.Rcap * pl.D * sizeof(uint16_t));
  pl.off_clo = take(CH * pl.Rcap * pl.D * sizeof(uint16_t));
  pl.off_cnorm = take(CH * pl.Rcap * sizeof(float));
  pl.off_assign = take(CH * pl.S * sizeof(int32_t));
  pl.off_hist = take(pl.one_sort ? 0 : CH * pl.NBLK * pl.Rcap * sizeof(int32_t));
  pl.off_order = take(CH * pl.S * sizeof(int32_t));
  pl.off_items = take(CH * pl.NIT * sizeof(int4));
  pl.off_nitem = take(CH * sizeof(int32_t));
  pl.off_parrive = take(CH * pl.Rcap * sizeof(int32_t));
  pl.off_part = take(CH * pl.NPART * 2 * pl.D * sizeof(double));
  pl.off_selh = take(pl.sel_multi ? CH * kSelHist * sizeof(int32_t) : 0);
  pl.off_sels = take(CH * 8 * sizeof(uint32_t));
  pl.off_selc = take(pl.count_sel ? CH * pl.NSEL * sizeof(uint4) : 0);
  pl.bytes = off;
  return true;
}

bool make_build_plan_adakv(const reskv_shape_t& s, const reskv_build_params_t& p, double safeguard,
                           int decode_reserve, const int32_t* seq_len, const int32_t* budget,
                           const int32_t* res_count, BuildPlan* plan) {
  init_build_plan(s, p, plan);
  plan->cross_head = true;
  std::vector<HeadMeta> hm;
  head_meta(*plan, seq_len, budget, res_count, p.recent_window, hm);
  const int cslots = s.slot_cap - decode_reserve;
  for (HeadMeta& m : hm) {  // widest sizes the allocation can give each head
    if (m.all_main) continue;
    const int fl = (int)floor(safeguard * (double)m.k_top);
    const int cap = m.n_sc < cslots - m.r - m.P ? m.n_sc : cslots - m.r - m.P;
    m.main_len = m.P + cap;
    m.nE = m.s - m.P - fl;
    m.r_eff = m.r < m.nE ? m.r : m.nE;
  }
  if (!fold_build_plan(hm, plan) || !layout_build_plan(plan)) return false;
  plan->off_adah = plan->bytes;
  plan->off_adas = align_up(plan->off_adah + (size_t)plan->B * plan->Hkv * kAdaHist * sizeof(int32_t), 256);
  plan->bytes = align_up(plan->off_adas + (size_t)2 * plan->B * kAdaState * sizeof(uint32_t), 256);
  return true;
}

bool make_build_plan(const reskv_shape_t& s, const reskv_build_params_t& p, const int32_t* seq_len,
                     const int32_t* budget, const int32_t* res_count, BuildPlan* plan) {
  init_build_plan(s, p, plan);
  std::vector<HeadMeta> hm;
  head_meta(*plan, seq_len, budget, res_count, p.recent_window, hm);
  return fold_build_plan(hm, plan) && layout_build_plan(plan);
}

hipError_t upload_meta(const BuildPlan& pl, const int32_t* seq_len, const int32_t* budget,
                       const int32_t* res_count, int sets, int recent, HeadMeta* meta, hipStream_t stream) {
  const int SBH = pl.B * pl.Hkv, BH = sets * SBH;
  for (int first = 0; first < BH; first += kMetaChunk) {
    MetaChunk c;
    c.first = first;
    c.count = BH - first < kMetaChunk ? BH - first : kMetaChunk;
    c.recent = recent;
    for (int i = 0; i < c.count; ++i) {
      const int bh = first + i, b = bh % SBH / pl.Hkv;
      c.s[i] = seq_len[b];
      c.r[i] = res_count[bh];
      c.budget[i] = budget[b];
    }
    hipLaunchKernelGGL(meta_kernel, dim3(1), dim3(kMetaChunk), 0, stream, meta, c);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_build_scores(const BuildPlan& pl, const void* k, const void* q_obs, const HeadMeta* meta,
                               void* workspace, hipStream_t stream) {
  const BuildArgs a = make_args(pl, k, nullptr, q_obs, meta, BuildOut{}, nullptr, nullptr, nullptr, workspace);
  const bool bf = pl.dtype == RESKV_BF16;
  if (pl.D == 128) return bf ? launch_scores_typed<uint16_t, 128>(pl, a, stream) : launch_scores_typed<float, 128>(pl, a, stream);
  if (pl.D == 64) return bf ? launch_scores_typed<uint16_t, 64>(pl, a, stream) : launch_scores_typed<float, 64>(pl, a, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_build_adakv(const reskv_shape_t& s, const reskv_build_params_t& p, double safeguard,
                              int decode_reserve, const BuildPlan& pl, const void* k, const void* v,
                              const int32_t* seq_len, const void* q_obs, const int32_t* budget,
                              const int32_t* res_count, void* kc, void* vc, float* logc, int32_t* main_idx,
                              int32_t* res_len, int32_t* main_len, float* dbg_scores, int32_t* dbg_assign,
                              float* dbg_centers, void* workspace, hipStream_t stream) {
  (void)s;
  HeadMeta* meta = reinterpret_cast<HeadMeta*>(static_cast<char*>(workspace) + pl.off_meta);
  hipError_t e = upload_meta(pl, seq_len, budget, res_count, 1, p.recent_window, meta, stream);
  if (e != hipSuccess) return e;
  e = launch_build_scores(pl, k, q_obs, meta, workspace, stream);
  if (e != hipSuccess) return e;
  const BuildOut out{kc, vc, logc, main_idx, res_len, main_len};
  BuildArgs a = make_args(pl, k, v, nullptr, meta, out, dbg_scores, dbg_assign, dbg_centers, workspace);
  a.cap_slots = pl.C - decode_reserve;
  a.ada_hist = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + pl.off_adah);
  a.ada_state = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + pl.off_adas);
  const bool bf = pl.dtype == RESKV_BF16;
  if (pl.D == 128)
    return bf ? launch_candidate_typed<uint16_t, 128>(pl, a, stream, meta, safeguard)
              : launch_candidate_typed<float, 128>(pl, a, stream, meta, safeguard);
  if (pl.D == 64)
    return bf ? launch_candidate_typed<uint16_t, 64>(pl, a, stream, meta, safeguard)
              : launch_candidate_typed<float, 64>(pl, a, stream, meta, safeguard);
  return hipErrorInvalidValue;
}

hipError_t launch_build_candidate(const BuildPlan& pl, const void* k, const void* v, const HeadMeta* meta,
                                  const BuildOut& out, float* dbg_scores, int32_t* dbg_assign, float* dbg_centers,
                                  bool more, void* workspace, hipStream_t stream) {
  BuildArgs a = make_args(pl, k, v, nullptr, meta, out, dbg_scores, dbg_assign, dbg_centers, workspace);
  a.B = pl.B * pl.NC;
  a.more = more;
  const bool bf = pl.dtype == RESKV_BF16;
  if (pl.D == 128) return bf ? launch_candidate_typed<uint16_t, 128>(pl, a, stream) : launch_candidate_typed<float, 128>(pl, a, stream);
  if (pl.D == 64) return bf ? launch_candidate_typed<uint16_t, 64>(pl, a, stream) : launch_candidate_typed<float, 64>(pl, a, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_build(const reskv_shape_t& s, const reskv_build_params_t& p, const BuildPlan& pl,
                        const void* k, const void* v, const int32_t* seq_len, const void* q_obs,
                        const int32_t* budget, const int32_t* res_count, void* kc, void* vc,
                        float* logc, int32_t* main_idx, int32_t* res_len, int32_t* main_len,
                        float* dbg_scores, int32_t* dbg_assign, float* dbg_centers, void* workspace,
                        hipStream_t stream) {
  (void)s;
  HeadMeta* meta = reinterpret_cast<HeadMeta*>(static_cast<char*>(workspace) + pl.off_meta);
  hipError_t e = upload_meta(pl, seq_len, budget, res_count, 1, p.recent_window, meta, stream);
  if (e != hipSuccess) return e;
  e = launch_build_scores(pl, k, q_obs, meta, workspace, stream);
  if (e != hipSuccess) return e;
  const BuildOut out{kc, vc, logc, main_idx, res_len, main_len};
  return launch_build_candidate(pl, k, v, meta, out, dbg_scores, dbg_assign, dbg_centers, false, workspace, stream);
}

}  // namespace reskv
