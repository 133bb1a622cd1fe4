// Matrix-core score pass: which calls take it, its launch shape, and how the workgroups of a grid that a batch shares are handed out.
// Plain C++ beside the kernel that uses it, so that the arithmetic can be gone through without a GPU.
#pragma once
#include "ts_kernels.h"

#ifdef __HIPCC__
#define TS_HD __host__ __device__ __forceinline__
#else
#define TS_HD inline
#endif

namespace ts {

enum Scan { kScanTested, kScanMasked, kScanWhole };   // the cache test runs in the launch; a skip mask; every sequence

// Shapes the matrix-core form covers: bf16, two column blocks per wave tile.  Wave tiles of 8 KV heads (G 3 and 4) or of 4 (G 5
// to 8), and no more of them side by side than a workgroup has waves (five to eight heads over 8 or 16 KV heads, score pass, us, vector
// kernel and this one: 64/8, 4 x 20011 to 40009 tokens 63.0 and 46.4, 6000 18.4 and 8.6, 200000 93.5 and 77.6; 40/8, 2500 tokens
// 14.5 and 7.6, 100000 45.5 and 45.5).
inline bool score_codes_mfma_supported(int dtype, int D, int G, int H_kv) {
  if (dtype != TS_BF16 || (D != 64 && D != 128)) return false;
  if (G >= 3 && G <= 4) return H_kv >= 8;
  if (G >= 5 && G <= 8) return H_kv >= 4 && H_kv <= 16;
  return false;
}

// Whether the matrix-core kernel covers a call and is the faster one.
// Five to seven heads over 8 and 16 KV heads: a wave's piece of a row of the score matrix is 80 to 112 bytes, not whole lines, and the
// vector kernel, whose workgroups write whole rows, is the faster one for large matrices.  Over 150 shapes the two cross between 104 and
// 130 MiB of K; the line lies where no shape is slower by it: up to 96 MiB the matrix cores take 0.76 to 0.92 of the vector kernel's time.  us,
// vector and matrix cores: 40/8, D 128, 49152 tokens (96 MiB) 24.5 and 22.4, 57344 25.4 and 25.1, 81920 35.3 and 37.1; 8 x 7168 (112
// MiB) 24.6 and 25.7; 56/8 28.1 and 23.9, 28.4 and 26.2, 37.4 and 39.3; 28.2 and 27.1; 80/16, D 64, 49152 (96 MiB) 27.4 and 22.7, 81920
// 39.0 and 40.1.  Eight heads' pieces are lines (64/8, D 128, 300000 138 and 122, D 64 83 and 69), and the compact form's bytes stay
// in the L2 (40/8, D 128, 300000 115 and 107; D 64 80 and 57).  With a mask or a test a sequence's scores are those of a call of
// its own, and so its own length counts, however many are scanned: of batches of 100 to 350 MiB together all scanned take 0.83 to 1.17
// of the vector kernel's time (median 1.01; 40/8, D 64, 2 x 81920, the worst), half of them 0.64 to 1.10, one 0.50 to 0.92.
inline bool score_takes_matrix_cores(const ts_problem* p, bool dense, Scan scan) {
  const int G = p->num_q_heads / p->num_kv_heads;
  if ((p->num_q_heads % 4) != 0 || !score_codes_mfma_supported(p->dtype, p->head_dim, G, p->num_kv_heads)) return false;
  if (!dense || G < 5 || G == 8 || p->num_kv_heads == 4) return true;
  const double k_bytes = (double)p->max_seq_len * p->num_kv_heads * p->head_dim * 2 * (scan == kScanWhole ? p->batch : 1);
  return k_bytes <= 96.0 * 1048576.0;
}

// dense: the run's fp32 rows are staged instead of its bytes
inline size_t score_codes_mfma_lds_bytes(int D, int G, int RR, bool dense) {
  const int HB = G <= 4 ? 8 : 4;
  const size_t per_wave = (size_t)32 * (D * 2 + 16) + (size_t)RR * kScoreTileTokens * HB * G * (dense ? 4 : 1) +
                          (size_t)RR * HB * G * 4;
  return 4 * per_wave;
}

// x / d for the tiles of a unit of the shared grid, x up to 2^26: powers of two and 6, 12 and 24, where the rounded-up factor is
// off by 16 / 2^31 at most, exact to 2^27.
TS_HD uint32_t score_unit_mul(uint32_t d) { return (uint32_t)((((uint64_t)1 << 31) + d - 1) / d); }
TS_HD uint32_t score_unit_div(uint32_t x, uint32_t mul) { return (uint32_t)(((uint64_t)x * mul) >> 31); }

// Launch shape of the matrix-core score kernel (both forms): fills the wave-tile fields and a.RR, returns the
// workgroups per sequence.  A wave owns one run of consecutive tiles where the sequence is short enough, so that
// its output leaves in one burst at the end of its life; about 2048 waves per sequence (measured on MI355X:
// 131072 tokens 49 us with one tile per wave, 45.7 us with two).
// forced_rr, forced_wg: tuning knobs, 0 = automatic.
inline void score_codes_mfma_shape(const ts_problem* p, int G, bool dense, Scan scan, int forced_rr, int forced_wg, ScoreArgs* a, long* wg_out) {
  const bool whole_batch = scan == kScanWhole;
  a->HB = G <= 4 ? 8 : 4; a->hb_shift = ilog2(a->HB); a->NU = p->num_kv_heads / a->HB;
  a->uniform_page = p->page_size >= (8 / a->HB);
  const long ntt = (p->max_seq_len + kScoreTileTokens - 1) / kScoreTileTokens;
  const int NU = a->NU;
  auto wgs_of = [&](int r) -> long {
    long n = ((ntt + r - 1) / r * NU + 3) / 4;
    return n > kScoreMaxWg ? (long)kScoreMaxWg : n;
  };
  int rr = forced_rr;
  if (rr <= 0 && dense && G >= 5 && NU > 1) {
    // The score matrix of several wave tiles side by side leaves in pieces of rows, which long runs do not join, and the LDS of
    // four tiles costs workgroups (H 64/8, D 64, 300000 tokens 69 us with one, 73 with two, 105 with four).  One tile per wave
    // up to one round of three workgroups per CU; then a second one that is nearly empty takes longer than two tiles per
    // wave in the first (D 128, 50000 tokens 26.7 and 22.6, 65000 31.2 and 27.9; D 64 16.6 and 15.9).  Between the most
    // workgroups of a launch and two full rounds D 128 has the shorter runs again (80000 37.7 and 38.8, 90000 39.2 and
    // 42.3, D 64 23.5 and 22.5), beyond it the longer ones and D 64 the shorter (120000 53.8 and 50.3, D 64 30.3 and 33.3).
    const long one = (ntt * NU + 3) / 4;               // workgroups of one tile per wave
    rr = one <= 768 ? 1 : one > 1536 ? (p->head_dim == 64 ? 1 : 2) : one <= kScoreMaxWg || p->head_dim == 64 ? 2 : 1;
  } else if (rr <= 0) {
    // Longest run that still gives every CU two workgroups, among those the one whose workgroups fill the
    // rounds best: the CU holds floor(160 KiB / LDS) workgroups, three at most (registers), and a last round
    // that is half empty costs as much as a full one (786432 tokens of H 28/4: 8-tile runs 151 us, 6-tile runs
    // two full rounds).
    rr = 1;
    double best = -1.0;
    for (int r = 8; r >= 1; r -= (r > 2 ? 2 : 1)) {     // 8, 6, 4, 2, 1: odd run lengths measured slower throughout
      const long n = wgs_of(r);
      if (r > 1 && n < 512) continue;
      long per_cu = (long)(163840 / score_codes_mfma_lds_bytes(p->head_dim, G, r, dense));
      if (per_cu > 3) per_cu = 3;
      if (per_cu < 1) continue;
      const long slots = 256 * per_cu, rounds = (n + slots - 1) / slots;
      const double fill = (double)n / (double)(rounds * slots);
      if (fill > best + 0.05) { best = fill; rr = r; }
    }
    // A batch of shorter sequences fills the machine with runs of four tiles too, and the compact form's bytes then leave
    // in fewer, longer bursts (score pass alone: 32 sequences of 1031 to 16001 tokens, H 32/8, 117 -> 114 us; 16 of 4000
    // to 16000, H 28/4, 40 -> 37; 8 of 65536, H 32/8, 190 -> 188).  Not where a skip mask or the Selection Cache's test may leave
    // one or two of them to fill it (one of the 32: 15 us with runs of one tile, 38 of four; one of the 8: 28 and 43), and not
    // for the score matrix's rows, four times as many bytes (the 32: 118.8 -> 147.5).
    if (!dense && whole_batch && rr < 4 && p->batch >= 4 && wgs_of(4) * p->batch >= 512) rr = 4;
  }
  // A batch whose lengths and mask are known when the launch starts shares one grid (shared_share) from more work on than a tile for
  // each wave of two workgroups per CU: up to there every wave of the other grid has its tile at once, and sharing costs up
  // to a microsecond (score matrix, us, the other grid and shared: 8 sequences of 3000 to 6000 tokens, H 32/8, 18.6 and 19.5; 4 of 5000
  // to 10000 18.5 and 19.3; 16 of 683 to 2048 13.4 and 13.3; beyond the line 16 of 1533 to 4600 25.5 and 20.3).
  // Beyond one round of a tile per wave two workgroups per CU share the work, at head size 64, with its rows of half the length,
  // three (32 of 1031 to 16001 tokens of 32/8, D 128, 97.6 us, with three per CU 105; D 64, 112 batches of 3 to 32 sequences
  // 1.05 times as fast as in a grid of their own, 1.01 with two per CU; D 128, 56 batches 1.06).  The staged runs are as long as
  // a wave's tiles can be, while two workgroups' LDS allows.  With a mask the statistics keep the runs found above.  Not with a mask for the
  // score matrix of five to seven heads with several wave tiles side by side: its rows leave in pieces, and several tiles per
  // workgroup at a time make it worse (us, shared and in a grid of its own: 40/8, D 64, 8 x 40960 tokens, all of them 88 and 76,
  // half 43.8 and 41.9, one 12.9 and 14.1; 56/8, D 64, 103 and 84, 52 and 46, 16.1 and 15.0; D 128, 8 x 10240, 41.8 and
  // 38.1, 22.5 and 21.9, 10.7 and 10.1).
  const int groups = 4 / NU;
  const long slots = kScoreFlatWg - p->batch, sr = rr;
  a->SR = rr;
  const bool in_pieces = dense && G >= 5 && G <= 7 && NU > 1;
  bool shares = scan != kScanTested && !(scan == kScanMasked && in_pieces) && p->batch >= 2 && p->batch <= kScoreFlatMaxBatch && forced_rr <= 0 && forced_wg <= 0 &&
                wgs_of(1) * p->batch > kScoreFlatWg;
  if (shares && scan == kScanMasked) {
    const long units = (p->batch * ((ntt + groups * sr - 1) / (groups * sr)) + slots - 1) / slots;   // of a workgroup, at most
    a->run_stat_bytes = (int)(units * groups * p->num_q_heads * sizeof(float2));
    shares = wgs_of(rr) < kScoreMaxWg && units <= 64 && a->run_stat_bytes <= 16384;   // one run per wave of a call of its own
    if (shares) rr = (int)(units * sr < 8 ? units * sr : 8);
    else a->run_stat_bytes = 0;
  } else if (shares) {
    const long most = (p->batch * ntt / slots * NU + 3) / 4 + 1;   // tiles of a wave
    rr = (int)(most < 8 ? most : 8);
  }
  if (shares) {
    if (dense) rr = rr >= 4 ? 2 : 1;                       // rows of floats: four times the LDS
    while (rr > 1 && score_codes_mfma_lds_bytes(p->head_dim, G, rr, dense) + a->run_stat_bytes > 81920) --rr;
  }
  if (rr > 8) rr = 8;
  while (rr > 1 && score_codes_mfma_lds_bytes(p->head_dim, G, rr, dense) > 163840) --rr;
  a->RR = rr;
  long wgl = wgs_of(rr);
  if (forced_wg > 0) wgl = forced_wg;
  if (shares) {
    const long lds = (long)score_codes_mfma_lds_bytes(p->head_dim, G, rr, dense) + a->run_stat_bytes;
    long per_cu = 163840 / lds, most = p->head_dim == 64 ? 4 : 3;            // registers
    if (per_cu > most) per_cu = most;
    a->flat_batch = p->batch; wgl = 256 * per_cu;
    a->flat_grid = (int)wgl; a->nu_shift = ilog2(NU); a->grain_mul = score_unit_mul((uint32_t)(groups * a->SR));
    a->flat_wgs = p->head_dim == 64 && wgl > 512 ? 768 : kScoreFlatWg;
  }
  *wg_out = wgl;
}

// What a wave scans: run n of its tiles starts at tile base + n * stride of sequence b, whose x-th of n workgroups this is.
// uw: units of a workgroup, whose statistics leave one by one (masked calls).
struct ScoreShare { int b, x, n, N, indptr, base, stride, tiles, uw; };

// ---- the shared grid (see shared_share): what a lane reckons for its sequence, and a wave for its tiles
TS_HD int score_share_groups(const ScoreArgs& a) { return 4 >> a.nu_shift; }                            // waves that share a tile range
TS_HD int score_share_grain(const ScoreArgs& a, bool masked) { return masked ? score_share_groups(a) * a.SR : 1; }   // tiles of a unit
TS_HD uint32_t score_share_units(const ScoreArgs& a, bool masked, int ntt) {
  return masked ? score_unit_div((uint32_t)(ntt + score_share_grain(a, true) - 1), a.grain_mul) : (uint32_t)ntt;
}
TS_HD uint32_t score_share_least(const ScoreArgs& a, bool masked) { return masked ? 1u : (uint32_t)score_share_groups(a); }   // units of a workgroup
TS_HD uint32_t score_share_least_count(const ScoreArgs& a, bool masked, uint32_t units) {
  const uint32_t n = masked ? units : (units + score_share_least(a, false) - 1) >> (2 - a.nu_shift);
  return n > 1u ? n : 1u;
}
TS_HD uint32_t score_share_upw(const ScoreArgs& a, bool masked, uint32_t total) {
  const uint32_t slots = (uint32_t)(a.flat_wgs - a.flat_batch), least = score_share_least(a, masked);   // the sequences' counts are rounded up
  const uint32_t n = ((total + slots - 1) / slots + least - 1) & ~(least - 1);                           // the waves' parts are equal
  return n > least ? n : least;
}
TS_HD uint32_t score_share_count(uint32_t units, uint32_t upw) {
  const uint32_t n = (units + upw - 1) / upw;
  return n > 1u ? n : 1u;
}
TS_HD void score_share_tiles(const ScoreArgs& a, bool masked, int wave, int upw, int ntt, ScoreShare& s) {   // of workgroup s.x
  const int part = wave >> a.nu_shift, groups_shift = 2 - a.nu_shift;
  s.stride = a.RR; s.uw = upw;
  if (masked) {
    const int per = upw * a.SR, left = ntt - (s.x * upw * score_share_grain(a, true) + part * per);
    s.base = ntt - left;
    s.tiles = left < 0 ? 0 : left < per ? left : per;
  } else {
    const int t0 = s.x * upw, have = upw < ntt - t0 ? upw : ntt - t0;
    const int lo = (have * part) >> groups_shift, hi = (have * (part + 1)) >> groups_shift;
    s.base = t0 + lo; s.tiles = hi - lo;
  }
}

}  // namespace ts
