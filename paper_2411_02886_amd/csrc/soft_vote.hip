// Eq. 5 (head soft vote): votes[t] = sum_h exp(c * (S[h][t] - max_h)) / sumexp_h.
//
// Up to eight lanes share one token; its H scores are one contiguous row, read as 16-byte pieces
// (a wave load covers whole consecutive rows).  The subtraction of the row maximum, the scaling and the
// argument reduction are double precision (exact difference, no loss to a large argument), the fractional
// power of two is the hardware float exponential, the weighted sum over heads is double again and is rounded
// to float once: a vote carries about 1e-7 relative error on top of what the float scores' own rounding gives.
#include "ts_kernels.h"

namespace ts {


// Merges the per-workgroup (max, sum-exp) partials of one (sequence, head) into row_stats.
// One workgroup per (head, sequence); every partial is loaded at once (one memory round trip), the
// rescaling exponentials and the sum are double precision.
__global__ __launch_bounds__(256) void score_stats_merge_kernel(VoteArgs a) {
  __shared__ float s_m[4];
  __shared__ double s_l[4];
  const int h = blockIdx.x, b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b] : 0;   // checked after the partials' loads have been issued
  // The partial count is what the score launch recorded in the workspace, whatever the host believes now; the slots that
  // the host expects are loaded at once (one memory round trip, the slots all exist), unused ones are masked afterwards,
  // and in the rare case that there are more (a tuning knob changed in between) the rest follows.  (Always loading all
  // 1024 slots, a batch of 32 sequences of 16001 tokens took 12.1 us instead of 5.1.)
  const int nparts = min((int)a.hdr[b * 8 + 0], kScoreMaxWg);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int PER = kScoreMaxWg / 256;
  float mp[PER], lp[PER];
  auto load_slot = [&](int i) {
    const int p = threadIdx.x + 256 * i;
    const float2 v = *reinterpret_cast<const float2*>(a.partials + (((size_t)b * kScoreMaxWg + p) * a.H + h) * 2);
    mp[i] = v.x; lp[i] = v.y;
  };
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    mp[i] = -INFINITY; lp[i] = 0.f;
    if (256 * i < a.parts_hint) load_slot(i);
  }
  if (nparts > a.parts_hint) {
#pragma unroll
    for (int i = 0; i < PER; ++i) load_slot(i);
  }
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if ((int)threadIdx.x + 256 * i >= nparts) { mp[i] = -INFINITY; lp[i] = 0.f; }
  if (skip_flag != 0) return;
  float m = mp[0];
#pragma unroll
  for (int i = 1; i < PER; ++i) m = fmaxf(m, mp[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if (lane == 0) s_m[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
  const double sc = (double)a.scale;
  double l = 0.0;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (mp[i] != -INFINITY) l += (double)lp[i] * exp_f64(sc * ((double)mp[i] - (double)m));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
  if (lane == 0) s_l[wave] = l;
  __syncthreads();
  if (threadIdx.x == 0) {
    a.row_stats_out[((size_t)b * a.H + h) * 2] = m;
    a.row_stats_out[((size_t)b * a.H + h) * 2 + 1] = (float)(s_l[0] + s_l[1] + s_l[2] + s_l[3]);
  }
}

// exp(c * d) for the vote, d = score - row maximum (exact in double), c2 = c * log2(e): the argument is reduced in
// double (t = n + f, |f| <= 1/2, so nothing of the float scores' precision is lost to a large argument), 2^f comes
// from the hardware float exponential (1 ulp) and is scaled by 2^n.  Relative error about 1e-7, the size of the
// rounding of the float vote itself and well below what the float scores' own rounding does to a vote.
__device__ __forceinline__ float vote_exp(double d, double c2) {
  const double t = fmax(d * c2, -1000.0);
  const double n = rint(t);
  const float f = (float)(t - n);
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// LPT lanes share one token row of H scores (stored [token][head]); a lane owns CPL 16-byte chunks.
// A workgroup takes NP passes of 256 / LPT tokens, all score loads issued up front (NP > 1 for long sequences:
// fewer, fatter workgroups, as the dispatch rate of tiny workgroups is what limits the kernel there).
template <int CPL, bool VEC, int NP>
__global__ __launch_bounds__(256) void soft_vote_kernel(VoteArgs a, int lpt_shift) {
  __shared__ double s_m[128];
  __shared__ double s_inv[128];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b] : 0;   // issued together with the length
  const int N = min(max(a.seq_lens[b], 0), a.max_seq_len);
  if (skip_flag != 0) return;
  const int LPT = 1 << lpt_shift;
  const int tpp = 256 >> lpt_shift;                 // tokens per pass
  const int tok0 = blockIdx.x * (tpp * NP);
  if (tok0 >= N) return;
  const int jv = threadIdx.x & (LPT - 1);
  const double c2 = (double)a.scale * 1.44269504088896340736;
  const int H = a.H;
  // statistics of every head: issued together with the score loads
  const float2 stv = *reinterpret_cast<const float2*>(a.row_stats + ((size_t)b * H + min((int)threadIdx.x, H - 1)) * 2);
  float s[NP][CPL][4];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int tc = min(tok0 + p * tpp + (int)(threadIdx.x >> lpt_shift), N - 1);   // out-of-range threads shadow the last token
    const float* sp = a.scores + ((size_t)b * a.max_seq_len + tc) * H;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int h0 = (jv + i * LPT) * 4;
      if (VEC) {
        const float4 v = *reinterpret_cast<const float4*>(sp + min(h0, H - 4));   // clamped: no branch between loads
        s[p][i][0] = v.x; s[p][i][1] = v.y; s[p][i][2] = v.z; s[p][i][3] = v.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[p][i][e] = sp[min(h0 + e, H - 1)];
      }
    }
  }
  if (threadIdx.x < H) { s_m[threadIdx.x] = (double)stv.x; s_inv[threadIdx.x] = 1.0 / (double)stv.y; }
  __syncthreads();
  const int r_lo = min(a.n_init, N), r_hi = max(r_lo, N - a.n_local);
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int t = tok0 + p * tpp + (int)(threadIdx.x >> lpt_shift);
    double vote = 0.0;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int h0 = (jv + i * LPT) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // lanes past the last head hold a shadow of heads H-4..H-1: they are skipped, not weighted by zero
        // (a shadowed score can lie far above the maximum of the head it would be compared with: inf * 0)
        if (h0 + e < H) vote = fma((double)vote_exp((double)s[p][i][e] - s_m[h0 + e], c2), s_inv[h0 + e], vote);
      }
    }
    for (int off = 1; off < LPT; off <<= 1) vote += __shfl_xor(vote, off);
    if (t < N && jv == 0) a.votes[(size_t)b * a.max_seq_len + t] = (t >= r_lo && t < r_hi) ? (float)vote : 0.f;
  }
}

// Eq. 5 and the start of the TopK in one launch.  A workgroup of T threads owns T / 2 consecutive tokens:
// it computes their votes as soft_vote_kernel does (same arithmetic, LPT lanes per token row, four passes of loads in
// flight), counts the top 11 key bits of the ranked tokens' votes in an LDS histogram and adds the non-empty bins to
// one of the replicated global histograms -- one flush per workgroup, spread over kBoundHistCopies copies, so the
// same-address atomics stay few.  (Measured and dropped: merging the score pass's statistics partials inside this
// kernel as well, every workgroup for itself.  At 128K tokens that is 128 KiB of partials per workgroup, 32 MiB of
// L2 reads per launch, and costs the kernel 4.7 us -- what the merge launch costs.)
// MERGE: a sequence whose score launch leaves few partials (kMergeParts a head, kMergeInVote in all: short sequences) has them merged
// here after all, by every workgroup for itself -- the partials' loads go out with the scores', the same sums otherwise --
// and the merge launch disappears.  (4096 tokens, 8 heads, 32 partials: 3.3 + 4.2 -> 5.4 us.)
// The line: with up to 256 partials a head (30000 tokens of 12 heads, five sequences) the step took 62 us instead of 55.
constexpr int kMergeInVote = 1024;   // partials x heads
constexpr int kMergeParts = 64;      // partials per head: two per thread
// T: 512 where eight lanes share a token (from 17 heads on: a round of four passes), 1024 for narrower rows.  Smaller workgroups
// fill the rounds of the machine better and start and end beside each other; each flushes a histogram of its own, though, which is
// what counts for narrow rows (statistics merge and vote, 1024 and 512 threads, us: 4 x 20011 to 40009 tokens of 64 heads 18.6 and
// 14.7; 5 x 20000 to 60000 of 12 heads 9.4 and 9.8).  Up to 32 heads, between half a round and a round of large workgroups (129 to
// 256), 1024: each has a CU to itself, and there are half as many histograms for the compaction.  Inside (12 shapes; vote, then the step):
// 66000 x 1 of 28 heads 10.3 and 10.6, 51.0 and 51.5; 80000 x 1 of 32 10.5 and 11.1, 65.8 and 67.3; 131072 x 1 of 32 11.2 and 11.3,
// 86.2 and 86.9; 65536 x 2 of 28 10.8 and 11.3, 64.0 and 64.5; 20000 x 4 of 32 10.0 and 10.4; 16000 x 8 of 32 10.3 and 10.7, steps the
// same.  Outside: 65000 x 1 of 32 10.0 and 9.8, steps the same; 30000 x 2 of 32 9.9 and 9.4; 20000 x 1 of 32 9.6 and 8.8, 43.0 and 42.2;
// 131500 x 1 of 32 13.6 and 12.1, 87.7 and 87.1; 17000 x 8 of 32 12.7 and 11.9, 99.7 and 98.6; 180000 x 1 of 28 13.2 and 12.5;
// 262144 x 1 of 32 14.7 and 15.1, but 132.0 and 129.8.

template <int T, int CPL, bool VEC, bool MERGE>
__global__ __launch_bounds__(T) void soft_vote_ranked_kernel(VoteArgs a, int lpt_shift) {
  __shared__ double s_m[128];
  __shared__ double s_inv[128];
  __shared__ uint32_t hist[kTopkBins];
  constexpr int NP = 4, kRankTokens = T / 2;
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b] : 0;   // issued together with the length
  const int N = min(max(a.seq_lens[b], 0), a.max_seq_len);
  if (skip_flag != 0) return;
  const int tok0 = blockIdx.x * kRankTokens;
  if (tok0 >= N) {
    // an empty sequence has statistics too: those of no score
    if (MERGE && tok0 == 0 && (int)threadIdx.x < a.H)
      *reinterpret_cast<float2*>(a.row_stats_out + ((size_t)b * a.H + threadIdx.x) * 2) = make_float2(-INFINITY, 0.f);
    return;
  }
  const int H = a.H;
  const double c2 = (double)a.scale * 1.44269504088896340736;
  const int LPT = 1 << lpt_shift;
  const int tpp = T >> lpt_shift;                 // tokens per pass
  const int jv = threadIdx.x & (LPT - 1);
  const int npass = (kRankTokens + tpp - 1) / tpp;   // LPT / 2 passes, one for the narrowest rows
  float s[NP][CPL][4];
  // the scores of a round of NP passes: all loads issued up front
  auto load_round = [&](int p0) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int tc = min(tok0 + (p0 + p) * tpp + (int)(threadIdx.x >> lpt_shift), N - 1);   // out-of-range threads shadow the last token
      const float* sp = a.scores + ((size_t)b * a.max_seq_len + tc) * H;
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const int h0 = (jv + i * LPT) * 4;
        if (VEC) {
          const float4 v = *reinterpret_cast<const float4*>(sp + min(h0, H - 4));   // clamped: no branch between loads
          s[p][i][0] = v.x; s[p][i][1] = v.y; s[p][i][2] = v.z; s[p][i][3] = v.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) s[p][i][e] = sp[min(h0 + e, H - 1)];
        }
      }
    }
  };
  load_round(0);
  const bool counts = a.max_seq_len > kTopkOneWg;      // shorter sequences are ranked without a histogram
  if (counts) for (int i = threadIdx.x; i < kTopkBins; i += T) hist[i] = 0u;
  if (MERGE) {
    // 32 threads per head, T / 32 heads per round.  Thread pl stands in for the threads pl + 32 * i of the merge kernel and adds
    // in that kernel's order, so that the statistics are the same bit for bit.
    const int nparts = min((int)a.hdr[b * 8 + 0], kScoreMaxWg);
    const int pl = threadIdx.x & 31;
    const double sc = (double)a.scale;
    for (int h0 = 0; h0 < H; h0 += T / 32) {
      const int h = h0 + (int)(threadIdx.x >> 5), hc = min(h, H - 1);
      auto slot = [&](int p) { return *reinterpret_cast<const float2*>(a.partials + (((size_t)b * kScoreMaxWg + p) * H + hc) * 2); };
      float2 v[2];                                     // all slots exist; unused ones are masked
#pragma unroll
      for (int i = 0; i < 2; ++i) v[i] = slot(pl + 32 * i);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (pl + 32 * i >= nparts) v[i] = make_float2(-INFINITY, 0.f);
      float m = fmaxf(v[0].x, v[1].x);
      for (int p = pl + kMergeParts; p < nparts; p += 32) m = fmaxf(m, slot(p).x);   // more than expected: a tuning knob changed in between
#pragma unroll
      for (int o = 1; o < 32; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
      auto term = [&](float2 x) { return x.x != -INFINITY ? (double)x.y * exp_f64(sc * ((double)x.x - (double)m)) : 0.0; };
      double l = 0.0;
      for (int w = 0; w == 0 || (w < 4 && 64 * w < nparts); ++w) {                   // the merge kernel's wave w
        double t[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int p0 = pl + 64 * w + 32 * i;
          t[i] = w == 0 ? term(v[i]) : p0 < nparts ? term(slot(p0)) : 0.0;
          for (int p = p0 + 256; p < nparts; p += 256) t[i] += term(slot(p));
        }
        double tw = t[0] + t[1];
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) tw += __shfl_xor(tw, o);
        l += tw;
      }
      if (pl == 0 && h < H) {
        const float lf = (float)l;
        s_m[h] = (double)m; s_inv[h] = 1.0 / (double)lf;
        if (blockIdx.x == 0) { a.row_stats_out[((size_t)b * H + h) * 2] = m; a.row_stats_out[((size_t)b * H + h) * 2 + 1] = lf; }
      }
    }
  } else if (threadIdx.x < H) {
    const float2 stv = *reinterpret_cast<const float2*>(a.row_stats + ((size_t)b * H + threadIdx.x) * 2);
    s_m[threadIdx.x] = (double)stv.x; s_inv[threadIdx.x] = 1.0 / (double)stv.y;
  }
  __syncthreads();
  const int r_lo = min(a.n_init, N), r_hi = max(r_lo, N - a.n_local);
  for (int p0 = 0; p0 < npass; p0 += NP) {
    if (tok0 + p0 * tpp >= N) break;
    if (p0 != 0) load_round(p0);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p0 + p >= npass) break;
      const int tl = (p0 + p) * tpp + (int)(threadIdx.x >> lpt_shift);   // token inside the workgroup's range
      const int t = tl < kRankTokens ? tok0 + tl : N;                     // (a pass of the narrowest rows is wider than the range)
      double vote = 0.0;
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const int h0 = (jv + i * LPT) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (h0 + e < H) vote = fma((double)vote_exp((double)s[p][i][e] - s_m[h0 + e], c2), s_inv[h0 + e], vote);
      }
      for (int off = 1; off < LPT; off <<= 1) vote += __shfl_xor(vote, off);
      if (t < N && jv == 0) {
        const bool ranked = t >= r_lo && t < r_hi;
        const float vf = ranked ? (float)vote : 0.f;
        a.votes[(size_t)b * a.max_seq_len + t] = vf;
        if (ranked && counts) atomicAdd(&hist[float_key(vf) >> 21], 1u);
      }
    }
  }
  if (!counts) return;
  __syncthreads();
  uint32_t* gh = a.rank_hist + ((size_t)b * kBoundHistCopies + (blockIdx.x & (kBoundHistCopies - 1))) * kTopkBins;
  for (int i = threadIdx.x; i < kTopkBins; i += T)
    if (hist[i] != 0u) atomicAdd(&gh[i], hist[i]);
}

hipError_t launch_soft_vote_ranked(const VoteArgs& a, int B, hipStream_t s) {
  const int hq = (a.H + 3) / 4;                     // 16-byte chunks per token row
  int lpt_shift = 0;
  while ((1 << lpt_shift) < hq && lpt_shift < 3) ++lpt_shift;
  const int cpl = (hq + (1 << lpt_shift) - 1) >> lpt_shift;   // 1, 2 or 4 for H <= 128
  const bool vec = (a.H % 4 == 0) && (((uintptr_t)a.scores & 15) == 0);
  const bool merge_in_vote = a.parts_hint <= kMergeParts && a.parts_hint * a.H <= kMergeInVote;
  if (!merge_in_vote) hipLaunchKernelGGL(score_stats_merge_kernel, dim3(a.H, B), dim3(256), 0, s, a);
  const long wgs = ((long)a.max_seq_len + 511) / 512 * B;
  const int threads = lpt_shift < 3 || (cpl == 1 && wgs > 128 && wgs <= 256) ? 1024 : 512, tokens = threads / 2;
  dim3 grid((a.max_seq_len + tokens - 1) / tokens, B);
#define TS_RV(T, C, V) do { if (merge_in_vote) hipLaunchKernelGGL((soft_vote_ranked_kernel<T, C, V, true>), grid, dim3(T), 0, s, a, lpt_shift); \
    else hipLaunchKernelGGL((soft_vote_ranked_kernel<T, C, V, false>), grid, dim3(T), 0, s, a, lpt_shift); } while (0)
  if (threads == 1024) { if (vec) TS_RV(1024, 1, true); else TS_RV(1024, 1, false); }
  else if (cpl <= 1) { if (vec) TS_RV(512, 1, true); else TS_RV(512, 1, false); }
  else if (cpl <= 2) { if (vec) TS_RV(512, 2, true); else TS_RV(512, 2, false); }
  else { if (vec) TS_RV(512, 4, true); else TS_RV(512, 4, false); }
#undef TS_RV
  return hipGetLastError();
}

hipError_t launch_stats_merge(const VoteArgs& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(score_stats_merge_kernel, dim3(a.H, B), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_soft_vote(const VoteArgs& a, int B, hipStream_t s) {
  const int hq = (a.H + 3) / 4;                     // 16-byte chunks per token row
  int lpt_shift = 0;
  while ((1 << lpt_shift) < hq && lpt_shift < 3) ++lpt_shift;
  const int cpl = (hq + (1 << lpt_shift) - 1) >> lpt_shift;   // 1, 2 or 4 for H <= 128
  const bool vec = (a.H % 4 == 0) && (((uintptr_t)a.scores & 15) == 0);
  hipLaunchKernelGGL(score_stats_merge_kernel, dim3(a.H, B), dim3(256), 0, s, a);
  const int tpp = 256 >> lpt_shift;
  const long nwg1 = ((long)a.max_seq_len * B + tpp - 1) / tpp;
  const int np = nwg1 >= 16384 ? 4 : (nwg1 >= 2048 ? 2 : 1);   // passes per workgroup (measured: 1 M tokens 42 -> 32 us with 4)
  dim3 grid((a.max_seq_len + tpp * np - 1) / (tpp * np), B);
#define TS_VOTE(C, V) do { if (np == 4) hipLaunchKernelGGL((soft_vote_kernel<C, V, 4>), grid, dim3(256), 0, s, a, lpt_shift); \
    else if (np == 2) hipLaunchKernelGGL((soft_vote_kernel<C, V, 2>), grid, dim3(256), 0, s, a, lpt_shift); \
    else hipLaunchKernelGGL((soft_vote_kernel<C, V, 1>), grid, dim3(256), 0, s, a, lpt_shift); } while (0)
  if (cpl <= 1) { if (vec) TS_VOTE(1, true); else TS_VOTE(1, false); }
  else if (cpl <= 2) { if (vec) TS_VOTE(2, true); else TS_VOTE(2, false); }
  else { if (vec) TS_VOTE(4, true); else TS_VOTE(4, false); }
#undef TS_VOTE
  return hipGetLastError();
}

}  // namespace ts
