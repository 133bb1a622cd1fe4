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
int rule_stream_span(long pairs, int total) { return ts::stream_span(pairs, total); }
}
