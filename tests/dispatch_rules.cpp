/* The host rules of csrc/ts_common.h behind C names, compiled by tests/rules_util.py: what a launch would be, without a GPU. */
#include "ts_common.h"

extern "C" {
int rule_attn_streams(int G, int D, long pairs, int total) { return ts::attn_streams(G, D, pairs, total) ? 1 : 0; }
int rule_eval_workgroups(int batch, int max_seq_len, int k) { return ts::eval_workgroups(batch, max_seq_len, k); }
int rule_stream_span(long pairs, int total) { return ts::stream_span(pairs, total); }
}
