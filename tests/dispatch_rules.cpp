/* The host rules of csrc/ts_common.h behind C names, compiled by tests/rules_util.py: what a launch would be, without a GPU. */
#include "ts_common.h"

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
}
