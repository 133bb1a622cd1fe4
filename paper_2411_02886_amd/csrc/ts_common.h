// Shared device helpers and workspace layout for the TokenSelect gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "tokenselect.h"

namespace ts {

constexpr int kWave = 64;
constexpr int kScoreTileTokens = 32;   // tokens per wave tile in the score pass
constexpr int kScoreLdsStride = 36;    // floats per head row of the staged score tile (16 B aligned)
constexpr int kScoreMaxWg = 1024;      // upper bound on workgroups per sequence in the score pass
constexpr int kScoreFlatWg = 512;      // two workgroups per CU: from more one-tile work on the sequences of a batch share a grid in the score pass
constexpr int kScoreFlatMaxBatch = 64; // ... that is, so many sequences: one per lane
constexpr int kTopkBins = 2048;        // 11-bit radix digit
constexpr int kTopkChunk = 2048;       // keys per workgroup in the top-k passes
constexpr int kBoundHistCopies = 8;    // replicas of the lower-bound histogram (same-address atomics are what its flush costs)
constexpr int kAttnChunk = 64;         // selected tokens per workgroup in sparse attention
constexpr int kAttnWhole = 256;        // list entries that one workgroup of sixteen waves attends by itself
constexpr int kAttnMaxRun = 4;        // chunks one attention workgroup folds into its partial, at most (256 list entries: one per thread)
constexpr int kAttnMaxSplit = 512;     // splits the merge kernel can stage (k <= 32768)

constexpr int kStreamTile = 32;        // keys per wave tile
constexpr int kStreamMaxSpan = 3584;   // the run's rows in LDS beside the tiles, two workgroups per CU
constexpr int kStreamMinSpan = 4 * kStreamTile;   // shorter runs leave a wave without a tile
// List entries per run (split) of a (sequence, KV head) pair.  The CUs share the work evenly only where the workgroups fill
// whole rounds of 256; a round costs the run's length plus about 160 keys of start, a merge of n runs about 200 + 5 n
// keys.  (H 32/8, D 128, 2048 tokens each: 12 sequences in 288 workgroups 30.6 us, in 192 24.9, in 480 24.2; 36 sequences
// in 288 70.4, in 864 59.7; H 16/16, D 64: 20 sequences in 320 44.6, in 960 37.8.  Over 110 shapes of 4 to 640 pairs the
// choice is 0.5 % above the best split on average, 6 % at most.)
inline int stream_span(long pairs, int total) {
  int best = 0;
  long best_cost = 0;
  for (int n = (total + kStreamMaxSpan - 1) / kStreamMaxSpan; ; ++n) {
    const int span = ((total + n - 1) / n + kStreamTile - 1) / kStreamTile * kStreamTile;
    const int runs = (total + span - 1) / span;          // rounded up, the runs may be fewer
    if (best != 0 && (span < kStreamMinSpan || pairs * runs > 2048)) break;
    const long cost = (pairs * runs + 255) / 256 * (span + 160) + (runs > 1 ? 200 + 5 * runs : 0);
    if (best == 0 || cost < best_cost) { best = span; best_cost = cost; }
  }
  return best;
}

// bf16: whether the attention streams long runs (sparse_attn_stream.hip) instead of taking 64-token chunks, `wgs` of them
// (sparse_attn_decode.hip).  The more query heads a KV head has, the more the vector kernel has to do per row, and the
// earlier the line.  Three heads and more: a list that is one run needs no merge, and streaming it is the faster way whatever
// the rest (73 shapes of 1 to 21 sequences, 2 to 2016 chunks: 1.12 to 2.24 times, 54 of one to seven pairs and 257 to 300 entries:
// 1.09 to 1.26; us, chunks and streamed: H 8/2, D 64, 1 x 256 tokens 9.2 and 5.9, 3 x 300 7.3 and 5.8; H 16/4, D 128, 1 x 300 8.1 and
// 7.3; H 24/8, D 64, 15 x 287 10.0 and 6.9; H 64/8, D 128, 21 x 748 33.6 and 15.0; the log-sum-exp's error against 64 bits 1.3 to
// 1.9e-7 instead of 1.9 to 3.1e-7, the output's own rounding in both).  With splits it starts later and merges, which short calls feel
// (74 shapes; us, just below and above the lines): H 64/8, D 128, 1 x 1429 9.7 and 10.0, 3 x 915 11.8 and 10.0; H 28/4, D 128, 2 x
// 2228 11.2 and 12.1, 10 x 679 12.4 and 10.4; H 40/8, D 128, 1 x 3072 10.3 and 12.1, 6 x 1565 16.3 and 13.2; H 32/8, D 128, 2 x
// 1291 9.6 and 11.0, 3 x 3385 15.8 and 14.1; D 64, 3 x 3055 11.6 and 11.8, 2 x 5637 13.3 and 11.6; H 24/8, D 64, 3 x 3636 10.8 and
// 12.0, 13 x 960 12.2 and 11.8.
// With one or two heads the vector kernel keeps up with the memory until its partials are many (2048 tokens of H 16/8:
// D 128 with 9216 workgroups 61 and 60, with 10496 74 and 66; D 64 with 18432 63 and 68, with 23040 83 and 74).  Before
// that streaming pays for short lists that need no splits (H 16/8, D 128, 47 x 700 tokens 33 and 29), with one head if they
// also fill the rounds (H 16/16, D 128, 700 tokens: 480 pairs 35 and 33, 528 pairs in their three rounds 39 and 44).
inline bool attn_streams(int G, int D, long pairs, int total) {
  const long wgs = (total + kAttnChunk - 1) / kAttnChunk * pairs;
  if (G >= 3) return stream_span(pairs, total) >= total || wgs >= (G >= 7 ? 352 : G >= 5 ? 768 : G == 3 ? 1536 : D == 128 ? 1152 : 1280);
  if (wgs < 4096) return false;
  if (wgs >= (D == 128 ? 10240 : 22528)) return true;
  if (total > (G == 2 ? 1536 : 1024) || stream_span(pairs, total) < total) return false;
  return G == 2 || 5 * pairs >= 4 * ((pairs + 255) / 256 * 256);
}

// Whether one workgroup of sixteen waves attends a pair's whole list: up to kAttnWhole entries, a pair per CU, head counts that the waves
// have registers and LDS for.  (fp32, D 64, eight heads: 8 pairs of 64 entries 8.1 us in chunks, 8.5 so; 128 pairs 9.4 and 8.7.
// bf16 lists of three and more heads stream.)
constexpr bool attn_whole_supported(int dtype, int D, int G) { return dtype == TS_F32 ? (D == 64 || G <= 3) : G < 3; }
inline bool attn_whole(int dtype, int D, int G, long pairs, int total) {
  return attn_whole_supported(dtype, D, G) && total <= kAttnWhole && pairs <= 256 && (dtype != TS_F32 || G < 8 || pairs >= 64);
}

// Workgroups per sequence that re-evaluate the candidates of the compact selection: two per CU over the batch (what the LDS for the scores of
// 256 candidates, up to 58 KiB, allows from 29 heads on, and the registers of float rows at head size 128; narrower layers would
// hold more, but a candidate's chain of loads bounds the kernel and not the work of a CU).  How many candidates there are is known on the device only -- a little more than k when votes
// are peaked, every token when they are flat, whatever k is -- so the number does not fall with k (k 64 of 1048576 flat
// votes: 12.9 ms with k / 4 workgroups, 1.7 ms with 512); those that would get fewer than kEvalMinShare candidates leave at once.
// Large batches: 512 / batch may leave a good part of the round empty; more rounds of smaller shares do not, and a round
// more costs about 0.08 of a sequence, with a small k more (300 sequences of up to 4000 tokens, H 8/2, k 256: peaked votes
// 45 -> 43 us, flat 205 -> 123).
constexpr int kEvalMinShare = 4;
inline int eval_workgroups(int batch, int max_seq_len, int k) {
  const int most = (max_seq_len + kEvalMinShare - 1) / kEvalMinShare;
  int best = 512 / batch;
  if (best < 4) {
    double best_cost = 0.0;
    for (int n = 1; n <= 8; ++n) {
      const double cost = (double)((n * (long)batch + 511) / 512) * (1.0 / n + 0.08 + 4.0 / (k > 32 ? k : 32));
      if (n == 1 || cost < best_cost) { best = n; best_cost = cost; }
    }
  }
  return best < most ? best : most;
}

// ---------------------------------------------------------------- workspace layout (host + device)
struct WsLayout {
  size_t topk_hist;        // uint32 [B][2][kTopkBins] : histograms of the first two radix passes (must start zeroed)
  size_t bound_hist;       // uint32 [B][kBoundHistCopies][kTopkBins] : compact selection, histogram of the vote lower bounds
                           // (must start zeroed too; decode only)
  size_t topk_state;       // uint32 [B][8] : digits and remaining ranks fixed so far
  size_t hdr;              // uint32 [B][8] : left by the score pass for the calls that follow it
  size_t score_partials;   // float [B][kScoreMaxWg][H][2]
  size_t topk_blk;         // uint32 [B][nblk] : per-chunk counts
  size_t topk_list;        // uint2 [B][nblk][kTopkChunk] : compacted (key, token) entries of the short top-k path
  size_t topk_dense;       // uint2 [B][nblk * kTopkChunk] : compact selection, (vote key, token) of the candidates without gaps (decode only)
  size_t blk_max;          // float [B][score_nblk][H] : compact score pass, per-block head maxima (decode only)
  int score_nblk;          // ceil(max_seq_len / kScoreTileTokens)
  size_t attn_out;         // float [B][H][nsplit][D]
  size_t attn_ml;          // float [B][H][nsplit][2]
  size_t pf_stat_part;     // float [B][TS][C][H][2]            (chunk > 1 only; sized for prefill_max_token_splits)
  size_t pf_vote_part;     // float [B][RB * H_kv][max_seq_len] (chunk > 1 only)
  size_t attn_chunk_o;     // float [B][C][H][nsplit][D]        (chunk > 1 with key-list splits)
  size_t attn_chunk_ml;    // float [B][C][H][nsplit][2]
  int attn_chunk_nsplit;
  size_t total;
  int pf_rb, pf_ts;
  int topk_nblk;
  int attn_nsplit;
};

inline int ilog2(int x) { int s = 0; while ((1 << s) < x) ++s; return s; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Key-list splits of the chunk-form attention: a workgroup owns 128 rows and fills a CU, so the key list
// is split until there is about one workgroup per CU; every split keeps at least four 64-key tiles (two per key group).
inline int chunk_attn_splits(const ts_problem* p, int k) {
  const int G = p->num_q_heads / p->num_kv_heads;
  const long wgs = (long)((p->chunk * G + 127) / 128) * p->num_kv_heads * p->batch;
  const int ntile = (k + p->num_initial + p->num_local + p->chunk + 63) / 64;
  int s = (int)((256 + wgs / 2) / wgs);
  if (s > 8) s = 8;
  if (s > ntile / 4) s = ntile / 4;
  if (s < 1) s = 1;
  return s;
}

// workgroups of a chunked-prefill sweep whose token range is split t ways
inline long prefill_sweep_workgroups(const ts_problem* p, int row_blocks, int t) {
  return ((long)p->batch * p->num_kv_heads * t + 7) / 8 * 8 * row_blocks;
}
// The most token splits that may be chosen: grows with max_seq_len, as the choice below does not.  The workspace is sized by
// this one, so that a workspace for the longest prompt serves every shorter one.
inline int prefill_max_token_splits(const ts_problem* p, int row_blocks) {
  const int ntile = (p->max_seq_len + 63) / 64;
  int t = 1;
  while (t < 64 && t < ntile && prefill_sweep_workgroups(p, row_blocks, t + 1) <= 2048) ++t;
  return t;
}
// Token splits of the chunked-prefill sweeps.  The chip holds 512 workgroups at a time (two per CU), so the splits are
// those whose workgroups fill whole rounds: a workgroup costs its tiles plus about 2.5 tiles of start (query fragments,
// row statistics, first loads), and a single round leaves the chip waiting for its slowest workgroup -- the more so when
// the sequences of a batch have different lengths.  (2 x 300 queries of H 28/4 over 12007 and 30011 tokens: 28 splits in
// four rounds 121 + 140 us, 14 in two 114 + 129, 7 in one 129 + 141; 512 queries of H 32/8 over 262144: 16 and 32 the same.)
inline int prefill_token_splits(const ts_problem* p, int row_blocks) {
  const int ntile = (p->max_seq_len + 63) / 64, most = prefill_max_token_splits(p, row_blocks);
  const double uneven = p->batch > 1 ? 0.15 : 0.03;
  int best = 1;
  double best_cost = 0.0;
  for (int t = 1; t <= most; ++t) {
    const long rounds = (prefill_sweep_workgroups(p, row_blocks, t) + 511) / 512;
    const double cost = (double)rounds * ((ntile + t - 1) / t + 2.5) * (1.0 + uneven / (double)rounds);
    if (t == 1 || cost < best_cost) { best = t; best_cost = cost; }
  }
  return best;
}

inline WsLayout ws_layout(const ts_problem* p, int k) {
  WsLayout w{};
  const size_t B = (size_t)p->batch, H = (size_t)p->num_q_heads, D = (size_t)p->head_dim;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  w.topk_nblk = (p->max_seq_len + kTopkChunk - 1) / kTopkChunk;
  if (w.topk_nblk < 1) w.topk_nblk = 1;
  w.attn_nsplit = (k + p->num_initial + p->num_local + kAttnChunk - 1) / kAttnChunk;   // forced tokens join the list
  if (w.attn_nsplit < 1) w.attn_nsplit = 1;
  // the histograms come first: they are the part that must start (and is left) zeroed
  w.topk_hist = take(B * 2 * kTopkBins * 4);
  if (p->chunk == 1) w.bound_hist = take(B * kBoundHistCopies * kTopkBins * 4);
  w.topk_state = take(B * 8 * 4);
  w.hdr = take(B * 8 * 4);
  w.score_partials = take(B * kScoreMaxWg * H * 2 * 4);
  w.topk_blk = take(B * (size_t)w.topk_nblk * 4);
  w.topk_list = take(B * (size_t)w.topk_nblk * kTopkChunk * 8);
  w.score_nblk = (p->max_seq_len + kScoreTileTokens - 1) / kScoreTileTokens;
  if (p->chunk == 1) {
    w.topk_dense = take(B * (size_t)w.topk_nblk * kTopkChunk * 8);
    w.blk_max = take(B * (size_t)w.score_nblk * H * 4);
  }
  if (p->chunk > 1) {
    const int G = p->num_q_heads / p->num_kv_heads;
    w.pf_rb = (p->chunk * G + 255) / 256;
    w.pf_ts = prefill_token_splits(p, w.pf_rb);
    w.pf_stat_part = take(B * (size_t)prefill_max_token_splits(p, w.pf_rb) * p->chunk * H * 2 * 4);
    w.pf_vote_part = take(B * (size_t)w.pf_rb * p->num_kv_heads * (size_t)p->max_seq_len * 4);
  }
  // the sections that depend on k come last, so that every other offset is the same for any k
  w.attn_out = take(B * H * (size_t)w.attn_nsplit * D * 4);
  w.attn_ml = take(B * H * (size_t)w.attn_nsplit * 2 * 4);
  if (p->chunk > 1) {
    w.attn_chunk_nsplit = chunk_attn_splits(p, k);
    if (w.attn_chunk_nsplit > 1) {
      w.attn_chunk_o = take(B * p->chunk * H * (size_t)w.attn_chunk_nsplit * D * 4);
      w.attn_chunk_ml = take(B * p->chunk * H * (size_t)w.attn_chunk_nsplit * 2 * 4);
    }
  }
  w.total = off;
  return w;
}

#ifdef __HIPCC__
// ---------------------------------------------------------------- device helpers
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// round-to-nearest-even float -> bf16 bits (finite inputs)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// sum over the 8 lanes of an aligned lane group; every lane of the group gets the total
__device__ __forceinline__ float group8_sum(float v) {
  v += dpp_f32<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_f32<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f32<0x141>(v);   // row_half_mirror
  return v;
}
__device__ __forceinline__ float group16_sum(float v) {
  v = group8_sum(v);
  v += dpp_f32<0x140>(v);   // row_mirror
  return v;
}
__device__ __forceinline__ float group8_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  return v;
}

// inclusive prefix sum over the 64 lanes of a wave, on the DPP network (row shifts, then the rows' last lanes broadcast):
// six dependent additions instead of six trips through the LDS permute unit
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add_u32(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  v = dpp_add_u32<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add_u32<0x112, 0xf>(v);   // row_shr:2
  v = dpp_add_u32<0x114, 0xf>(v);   // row_shr:4
  v = dpp_add_u32<0x118, 0xf>(v);   // row_shr:8
  v = dpp_add_u32<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add_u32<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// order-preserving key of a float: larger float <=> larger unsigned key; -0.0 maps onto +0.0
__device__ __forceinline__ uint32_t float_key(float v) {
  uint32_t u = __float_as_uint(v);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inverse of float_key
__device__ __forceinline__ float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// exp(x) for x <= 0 (larger x also fine up to ~700); result below 1e-300 flushes to 0
__device__ __forceinline__ double exp_f64(double x) {
  const bool tiny = x < -690.0;
  x = tiny ? -690.0 : x;
  const double n = rint(x * 1.44269504088896340736);
  double r = fma(n, -6.93147180369123816490e-01, x);
  r = fma(n, -1.90821492927058770002e-10, r);
  // Taylor series on |r| <= 0.347, degree 11: truncation below 3e-14 relative
  double p = 1.0 / 39916800.0;
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  const long long bits = ((long long)n + 1023LL) << 52;   // 2^n, n >= -996 here
  return tiny ? 0.0 : p * __longlong_as_double(bits);
}

#endif  // __HIPCC__

}  // namespace ts
