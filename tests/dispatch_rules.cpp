/* The host rules of csrc/ts_common.h behind C names, compiled by tests/rules_util.py: what a launch would be, without a GPU. */
#include "ts_score_shape.h"
#include <string.h>

static ts_problem score_problem(int B, int H, int H_kv, int D, int max_seq_len) {
  ts_problem p{};
  p.batch = B; p.chunk = 1; p.num_q_heads = H; p.num_kv_heads = H_kv; p.head_dim = D; p.page_size = 16; p.max_seq_len = max_seq_len; p.dtype = TS_BF16;
  return p;
}

extern "C" {
int rule_attn_streams(int G, int D, long pairs, int total) { return ts::attn_streams(G, D, pairs, total) ? 1 : 0; }
int rule_eval_workgroups(int batch, int max_seq_len, int k) { return ts::eval_workgroups(batch, max_seq_len, k); }
int rule_chunk_splits(int chunk, int H, int H_kv, int D, int k, int num_initial) {
  ts_problem p{};
  p.batch = 1; p.chunk = chunk; p.num_q_heads = H; p.num_kv_heads = H_kv; p.head_dim = D; p.num_initial = num_initial;
  return ts::chunk_attn_splits(&p, k);
}
long rule_zeroed_bytes(int batch, int max_seq_len) {      // of a decode workspace: the histograms, which come first
  ts_problem p{};
  p.batch = batch; p.chunk = 1; p.num_q_heads = 1; p.num_kv_heads = 1; p.head_dim = 64; p.max_seq_len = max_seq_len;
  return (long)ts::ws_layout(&p, 1).topk_state;
}
int rule_topk_scratch_fits(int batch, int max_seq_len) {   // the table and the third histogram of flat votes in the list's memory
  ts_problem p{};
  p.batch = batch; p.chunk = 1; p.num_q_heads = 1; p.num_kv_heads = 1; p.head_dim = 64; p.max_seq_len = max_seq_len;
  const ts::WsLayout w = ts::ws_layout(&p, 1);
  return (size_t)batch * w.topk_nblk * 1024 * 2 + (size_t)batch * 1024 * 4 <= w.topk_dense - w.topk_list ? 1 : 0;
}
unsigned rule_unit_div(unsigned x, unsigned d) { return ts::score_unit_div(x, ts::score_unit_mul(d)); }
int rule_stream_span(long pairs, int total) { return ts::stream_span(pairs, total); }
int rule_score_cores(int B, int H, int H_kv, int D, int max_seq_len, int dense, int scan) {
  const ts_problem p = score_problem(B, H, H_kv, D, max_seq_len);
  return ts::score_takes_matrix_cores(&p, dense != 0, (ts::Scan)scan) ? 1 : 0;
}
/* out: whether the batch shares the grid, workgroups, RR, SR, NU, LDS bytes, run_stat_bytes */
void rule_score_shape(int B, int H, int H_kv, int D, int max_seq_len, int dense, int scan, long* out) {
  const ts_problem p = score_problem(B, H, H_kv, D, max_seq_len);
  ts::ScoreArgs a{};
  long wgl = 0;
  ts::score_codes_mfma_shape(&p, H / H_kv, dense != 0, (ts::Scan)scan, 0, 0, &a, &wgl);
  const long v[7] = {a.flat_batch > 0, wgl, a.RR, a.SR, a.NU, (long)ts::score_codes_mfma_lds_bytes(D, H / H_kv, a.RR, dense != 0) + a.run_stat_bytes, a.run_stat_bytes};
  memcpy(out, v, sizeof v);
}
/* What shared_share gives every wave of a shared grid: out[workgroup][wave] = sequence (-1: the workgroup leaves), x, n, first tile, tiles, uw.
 * The scans over the lanes are loops here, everything else is what the kernel calls. */
void rule_score_share(int B, int H, int H_kv, int D, int max_seq_len, int dense, int masked, const int* lens, const uint8_t* skip, int* out) {
  const ts_problem p = score_problem(B, H, H_kv, D, max_seq_len);
  ts::ScoreArgs a{};
  long grid = 0;
  const bool m = masked != 0;
  ts::score_codes_mfma_shape(&p, H / H_kv, dense != 0, m ? ts::kScanMasked : ts::kScanWhole, 0, 0, &a, &grid);
  int ntt[64];
  uint32_t units[64], cnt[64], total = 0, wgs = 0, upw = ts::score_share_least(a, m);
  for (int b = 0; b < B; ++b) {
    const bool scanned = !m || skip[b] == 0;
    ntt[b] = scanned ? (lens[b] + ts::kScoreTileTokens - 1) / ts::kScoreTileTokens : 0;
    units[b] = ts::score_share_units(a, m, ntt[b]);
    cnt[b] = scanned ? ts::score_share_least_count(a, m, units[b]) : 0u;
    total += units[b]; wgs += cnt[b];
  }
  if (wgs > (uint32_t)a.flat_grid) {
    upw = ts::score_share_upw(a, m, total);
    for (int b = 0; b < B; ++b) cnt[b] = m && skip[b] != 0 ? 0u : ts::score_share_count(units[b], upw);
  }
  for (long w = 0; w < grid; ++w) {
    int b = 0;
    uint32_t first = 0;
    while (b < B && first + cnt[b] <= (uint32_t)w) first += cnt[b++];
    for (int wave = 0; wave < 4; ++wave) {
      int* o = out + (w * 4 + wave) * 6;
      o[0] = b < B ? b : -1;
      if (b >= B) continue;
      ts::ScoreShare s{};
      s.x = (int)(w - first);
      ts::score_share_tiles(a, m, wave, (int)upw, ntt[b], s);
      o[1] = s.x; o[2] = (int)cnt[b]; o[3] = s.base; o[4] = s.tiles; o[5] = s.uw;
    }
  }
}
}
