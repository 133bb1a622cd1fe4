// Compact form of the decode selection (Algorithm 2 + Eq. 5 + TopK without the score matrix in memory).
//
// The score pass leaves one byte per score -- its distance below the head's maximum inside a block of
// tokens, in quarter octaves of softmax weight, rounded towards the maximum -- the block maxima, and the
// usual per-workgroup softmax statistics.  After the statistics merge (soft_vote.hip):
//   vote_bounds_kernel   turns the bytes into an upper and a lower bound of every token's vote (they differ
//                        by 2^(1/4) plus guards) and histograms the lower bounds;
//   topk_compact_kernel  (topk.hip) lists every token whose upper bound reaches the histogram bin of the k-th
//                        largest lower bound -- a superset of the top-k, usually 1.05-1.5 k tokens;
//   topk_eval_kernel     recomputes their scores from K (exact products, double accumulation) and their votes as
//                        Eq. 5 defines them, and lists (vote key, token) in token order.
// The finishing workgroup of the radix select (topk.hip) then picks the k largest of those votes.  Why the
// candidates are a superset: k tokens have votes >= their lower bounds >= the k-th largest lower bound L_k,
// so the k-th largest vote is >= L_k, and a token of the top-k has upper bound >= its vote >= L_k.
#include "ts_kernels.h"
#include "ts_score_math.h"

namespace ts {

// Guards that keep the bounds valid under rounding.  The byte was formed from the float score of the score pass
// (a few ulp of the largest score away from the exact one that the candidates are re-evaluated with) through a
// float product; the exponent offset of a block is rounded to float; the hardware exponential has 1 ulp; the
// sum over heads rounds H times.
constexpr float kCodeGuard = 1e-3f;               // octaves added to the decoded upper end of a byte ...
constexpr float kScoreGuard = 1.0f / 262144.0f;   // ... plus c2 * |largest maximum| * 2^-18 for the score's own rounding
constexpr float kBoundUp = 1.0002f;               // factor on the summed upper bound
constexpr float kBoundDown = 0.9998f;             // factor on the summed lower bound

// One lane per token: a lane reads its token's H bytes (a wave reads 64 consecutive rows) and sums, head by head,
// weight(block, head) * 2^((byte - 255) / 4): the weight of a byte-255 score of each 32-token block this workgroup
// meets (2^(c2 * (block max - max_h)) / sumexp_h, exponent formed in double) from an LDS table, the power from the
// hardware exponential.  The next 256 tokens' bytes are in flight while the current ones are summed.  The
// workgroup's histogram of the lower bounds is flushed once.
template <int HW>                                // dwords per token row (H / 4); 0 = any H, byte loads
__global__ __launch_bounds__(256) void vote_bounds_kernel(BoundArgs a, int tokens_per_wg) {
  constexpr int BT = kScoreTileTokens;          // tokens per block of the byte form
  constexpr int NW = HW > 0 ? HW : 1;
  __shared__ double s_km[128];                  // c2 * max_h + log2(sumexp_h)
  __shared__ float s_absmax[4];
  __shared__ uint32_t hist[kTopkBins];
  extern __shared__ float s_off[];              // [blocks of this workgroup][H]
  const int b = blockIdx.y;
  const int H = a.H;
  const int tbeg = blockIdx.x * tokens_per_wg;
  uint32_t qn[NW];
  auto load_codes = [&](int t0) {               // rows past the sequence are read too (they exist) and ignored
    if (HW > 0) {
      const int tc = min(t0 + (int)threadIdx.x, a.max_seq_len - 1);
      const uint32_t* cp = reinterpret_cast<const uint32_t*>(a.codes + ((size_t)b * a.max_seq_len + tc) * H);
#pragma unroll
      for (int w = 0; w < NW; ++w) qn[w] = cp[w];
    }
  };
  if (tbeg < a.max_seq_len) load_codes(tbeg);
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b] : 0;
  const int N = min(max(a.seq_lens[b], 0), a.max_seq_len);
  if (skip_flag != 0) return;
  if (tbeg >= N) return;
  const int tend = min(N, tbeg + tokens_per_wg);
  const double c2d = (double)a.scale * 1.44269504088896340736;
  float am = 0.f;
  if (threadIdx.x < H) {
    const float2 st = *reinterpret_cast<const float2*>(a.row_stats + ((size_t)b * H + threadIdx.x) * 2);
    s_km[threadIdx.x] = c2d * (double)st.x + log2((double)st.y);
    am = fabsf(st.x);
  }
  const int blk0 = tbeg / BT, nblk_wg = (tend - 1) / BT - blk0 + 1;
  // block maxima of this workgroup's tokens: loaded before the barrier, turned into weights after it
  float mxb[4];
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const int i = threadIdx.x + i4 * 256;
    mxb[i4] = i < nblk_wg * H ? a.blk_max[((size_t)b * a.nblk + min(blk0 + i / H, a.nblk - 1)) * H + i % H] : 0.f;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) am = fmaxf(am, __shfl_xor(am, off));
  if ((threadIdx.x & 63) == 0) s_absmax[threadIdx.x >> 6] = am;
  for (int i = threadIdx.x; i < kTopkBins; i += 256) hist[i] = 0u;
  __syncthreads();
  am = fmaxf(fmaxf(s_absmax[0], s_absmax[1]), fmaxf(s_absmax[2], s_absmax[3]));
  const float guard = kCodeGuard + (float)c2d * am * kScoreGuard;
  const float lo_scale = kBoundDown * __builtin_amdgcn_exp2f(-0.25f - 2.f * guard);
  for (int i = threadIdx.x; i < nblk_wg * H; i += 256) {
    const int i4 = i >> 8;                      // the first 1024 entries were loaded above
    float m;
    if (i4 < 4) m = i4 == 0 ? mxb[0] : i4 == 1 ? mxb[1] : i4 == 2 ? mxb[2] : mxb[3];
    else m = a.blk_max[((size_t)b * a.nblk + min(blk0 + i / H, a.nblk - 1)) * H + i % H];
    s_off[i] = __builtin_amdgcn_exp2f((float)(c2d * (double)m - s_km[i % H]) + guard);   // exponent <= guard; 0 for an empty block
  }
  __syncthreads();
  // Byte 0 is open towards minus infinity: a head with byte 0 gives no lower bound.  Instead of leaving such heads out
  // of the sum one by one (a compare, a select and an add per score), the most they can have put into the upper sum
  // is taken off once per token: 2^(-255/4) times the sum of the block's weights over the heads, and a weight is at
  // most 2^guard / sumexp_h <= 2^guard.
  const float zero_byte_total = __builtin_amdgcn_exp2f(-63.75f) * (float)H * __builtin_amdgcn_exp2f(guard) * 1.00001f;
  const int r_lo = min(a.n_init, N), r_hi = max(r_lo, N - a.n_local);
  for (int t0 = tbeg; t0 < tend; t0 += 256) {
    uint32_t qc[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) qc[w] = qn[w];
    if (t0 + 256 < tend) load_codes(t0 + 256);
    const int t = t0 + (int)threadIdx.x;
    const int tblk = min(t, tend - 1) / BT - blk0;
    const float* offp = s_off + tblk * H;
    float up = 0.f;
    if (HW > 0) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float4 o4 = *reinterpret_cast<const float4*>(offp + w * 4);
        const uint32_t c0 = qc[w] & 255u, c1 = (qc[w] >> 8) & 255u, c2b = (qc[w] >> 16) & 255u, c3 = qc[w] >> 24;
        // 2^((byte - 255) / 4) from the hardware exponential: a 256-entry LDS table read at random addresses by 64 lanes
        // conflicts on its banks and was what bounded the kernel (1M tokens: 15.2 us with the table, 14.2 us without)
        const float p2 = __builtin_amdgcn_exp2f(fmaf((float)c2b, 0.25f, -63.75f));
        const float p3 = __builtin_amdgcn_exp2f(fmaf((float)c3, 0.25f, -63.75f));
        const float p1 = __builtin_amdgcn_exp2f(fmaf((float)c1, 0.25f, -63.75f));
        const float p0 = __builtin_amdgcn_exp2f(fmaf((float)c0, 0.25f, -63.75f));
        up = fmaf(o4.x, p0, up); up = fmaf(o4.y, p1, up);
        up = fmaf(o4.z, p2, up); up = fmaf(o4.w, p3, up);
      }
    } else {
      const uint8_t* cp = a.codes + ((size_t)b * a.max_seq_len + min(t, N - 1)) * H;
      for (int h = 0; h < H; ++h) {
        const uint32_t c = cp[h];
        up = fmaf(offp[h], __builtin_amdgcn_exp2f(fmaf((float)c, 0.25f, -63.75f)), up);
      }
    }
    float lo = fmaxf(up - zero_byte_total, 0.f) * lo_scale;
    up *= kBoundUp;
    if (t < tend) {
      const bool ranked = t >= r_lo && t < r_hi;
      a.vote_hi[(size_t)b * a.max_seq_len + t] = ranked ? up : 0.f;
      if (a.vote_lo != nullptr) a.vote_lo[(size_t)b * a.max_seq_len + t] = ranked ? lo : 0.f;
      if (ranked) atomicAdd(&hist[float_key(lo) >> 21], 1u);
    }
  }
  __syncthreads();
  uint32_t* gh = a.hist + ((size_t)b * kBoundHistCopies + (blockIdx.x % kBoundHistCopies)) * kTopkBins;
  for (int i = threadIdx.x; i < kTopkBins; i += 256)
    if (hist[i] != 0u) atomicAdd(&gh[i], hist[i]);
}

hipError_t launch_vote_bounds(const BoundArgs& a, int B, hipStream_t s) {
  // a workgroup flushes one histogram: 256 tokens each for short sequences, at most about 1024 workgroups per
  // sequence for long ones
  int tpw = (a.max_seq_len + 1023) / 1024;
  if (tpw < 256) tpw = 256;
  tpw = (tpw + 255) / 256 * 256;
  // the table of block factors has to fit beside 11 KiB of static LDS without asking for more than the default 64 KiB
  while (tpw > 256 && (size_t)(tpw / kScoreTileTokens + 1) * a.H * sizeof(float) > 49152) tpw -= 256;
  const int nwg = (a.max_seq_len + tpw - 1) / tpw;
  const size_t lds = (size_t)(tpw / kScoreTileTokens + 1) * a.H * sizeof(float);
  const dim3 grid(nwg, B);
  const int hw = a.vec ? a.H / 4 : 0;
#define TS_VB(W) case W: hipLaunchKernelGGL((vote_bounds_kernel<W>), grid, dim3(256), lds, s, a, tpw); break;
  switch (hw) {
    TS_VB(1) TS_VB(2) TS_VB(3) TS_VB(4) TS_VB(5) TS_VB(6) TS_VB(7) TS_VB(8) TS_VB(10) TS_VB(12) TS_VB(14) TS_VB(16) TS_VB(24) TS_VB(32)
    default: hipLaunchKernelGGL((vote_bounds_kernel<0>), grid, dim3(256), lds, s, a, tpw); break;
  }
#undef TS_VB
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The candidates (listed per 2048-token chunk by topk_compact_kernel over the upper bounds) re-evaluated from K.
//
// What bounds it: for one sequence the chain of dependent loads (chunk counts -> token -> page id -> K row).  For a batch
// the gather of the rows, with the chain before it and the votes behind it, which all workgroups pass through at the same time: 32
// sequences of 1031 to 16001 tokens, H 32/8, are about 70 thousand candidates and 140 MB of K rows, 24 us at the rate of a
// gather, in 35 us.  The candidates of a sequence are numbered through and every workgroup takes an equal share of them,
// whatever chunk they come from.  (When the workgroup that had compacted a chunk also evaluated it, a short sequence -- all
// of its tokens candidates, in one or two chunks -- was one workgroup's serial tail: 277 us for the 32 sequences.)
// The products run on v_mfma_f64_4x4x4 (four blocks of 4 candidates x 4 query heads, one KV head each, 4 elements a step).  The
// double-precision matrix instructions are no faster than v_fma_f64, and both occupy the vector ALU; what goes is everything
// around the products: a lane converts its quarter of a row once for four heads, no sums travel across lanes, and the query
// takes 64 registers, so that the next step's loads leave as the current pieces are converted.  (A row on eight lanes, products by
// v_fma_f64, sums by DPP: the 32 sequences 45.5 us; 32 of 4000 to 12500, H 28/4, k 4000 80.6, now 51.  Eight waves
// instead of four a workgroup: the same for batches, 0.5 to 1 us more for one sequence; where a wave of four has two units to go
// through, 4 x 20000 to 40000, H 64/32, D 64, k 2000, 18.2 and
// 14.5, 16.0 before.)
// One query head per KV head (ONE) would use a quarter of the matrix instruction's columns: v_fma_f64, and the sums of the four lanes of a row
// by the swaps of half and quarter waves (one sequence of 200000 tokens, k 2048: H 8/8, D 128, 6.7 -> 6.1 us, fp32 7.6 ->
// 7.0; 16/16, D 64, 6.7 -> 6.2; 32 of 1031 to 16001, H 1/1, D 128, 37.4 -> 34.2).  Two heads the same way: 4/2, D 128, 6.6 -> 6.8, fp32
// 6.8 -> 7.0, for want of registers.  (Eight lanes to a row are still faster there for a single sequence: 16/8, D 128, 6.6, with
// four 6.9; fp32 7.2 and 7.9; batches 35.6 and 33.6.)
// The scores of up to CB candidates meet in LDS, where the softmax weights are formed with every lane at work.

// exp(c * d) as ts_soft_vote forms it: argument reduced in double, 2^fraction from the float hardware exponential
__device__ __forceinline__ float refine_vote_exp(double d, double c2) {
  const double t = fmax(d * c2, -1000.0);
  const double n = rint(t);
  const float f = (float)(t - n);
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffLL), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppRor8 = 0x128;

// sum over the four lanes of a wave that are 16 apart
__device__ __forceinline__ double quarter_sum_f64(double v) {
  auto sum = [](auto lo, auto hi) {
    return __longlong_as_double(((long long)hi[0] << 32) | (unsigned int)lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | (unsigned int)lo[1]);
  };
  unsigned long long u = (unsigned long long)__double_as_longlong(v);
  v = sum(__builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false), __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false));
  u = (unsigned long long)__double_as_longlong(v);
  return sum(__builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false), __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false));
}

// the elements of a 16-byte piece as doubles
template <int DT>
__device__ __forceinline__ void unpack_f64(uint4 w, double* f) {
  const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (DT == TS_BF16) { f[2 * c] = (double)bf16_lo(x[c]); f[2 * c + 1] = (double)bf16_hi(x[c]); }
    else f[c] = (double)__uint_as_float(x[c]);
  }
}

constexpr int kEvalMaxBatch = 256;        // candidates whose scores a workgroup holds in LDS at a time, at most

// CS: sets of four query heads of a KV head.  ONE: one query head per KV head.  WAVES: eight where that many (set, four KV heads) pairs are, else four.
template <int DT, int D, int CS, int WAVES, bool ONE>
__global__ __launch_bounds__(64 * WAVES, 2) void topk_eval_kernel(RefineArgs a, int cb) {
  constexpr int T = 64 * WAVES;
  constexpr int ES = Elt<DT>::size;
  constexpr int RB = D * ES;
  constexpr int EPP = 16 / ES;            // elements of a 16-byte piece
  constexpr int NP = RB / 64;             // pieces per lane: four lanes share a K row
  __shared__ uint32_t wave_sum[WAVES];
  __shared__ int ctok[kEvalMaxBatch];
  __shared__ long long cslot[kEvalMaxBatch];
  __shared__ double s_m[128];
  __shared__ double s_inv[128];
  extern __shared__ double sc[];          // [cb][H] scores of the batch, then uint32 [nblk + 1] prefix of the chunk counts
  const TopkArgs& ta = a.t;
  const int b = blockIdx.y;
  const int H = a.H, G = H / a.H_kv;
  uint32_t* off = reinterpret_cast<uint32_t*>(sc + (size_t)cb * H);
  const int skip_flag = ta.skip != nullptr ? (int)ta.skip[b] : 0;
  const int Nb = min(max(ta.seq_lens[b], 0), ta.max_seq_len);
  const int indptr = a.page_indptr[b];
  if (skip_flag != 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Operand lanes: row (query head) c of block bl, elements of pieces kk, kk + 4, ...; result lanes: row kk, column c of block bl.
  // A block is four candidates and one KV head; with fewer than four KV heads the blocks are different candidates.
  const int c = lane & 3, bl = (lane >> 2) & 3, kk = lane >> 4;
  const int HB = min(a.H_kv, 4), hb_shift = 31 - __clz(HB);
  const int NU = a.H_kv >> hb_shift;                  // groups of HB KV heads
  const int tps = 16 >> hb_shift;                     // candidates of a wave step
  const int units = NU * CS;                          // 1, 2, 4 or, with eight waves, 8: a wave stays with one
  const int unit = wave & (units - 1), wsub = wave / units, wstep = WAVES / units;
  const int kvh = (unit & (NU - 1)) * HB + (bl & (HB - 1));
  const int g = unit / NU * 4 + c;                    // this lane's query head of the KV head
  const int cand = (bl >> hb_shift) * 4;              // first candidate of the block in a step
  // Loads come back in the order they were asked for, and a load waits for the stores before it: the counts, which the chain goes on
  // with, are asked for first; the query is converted and the histogram cleared behind the loads of the first rows.  (One
  // sequence of 200000 tokens, k 2048, D 128, us, query and clearing first and so: fp32, H 28/4 8.3 and 7.8, 12/2 7.9 and 7.1, 40/8 9.7
  // and 9.0; bf16, 64/8 8.3 and 7.9; of 20000, k 512, 64/8 7.2 and 6.1.  Batches the same.)
  constexpr int CPT = 4;                              // consecutive chunks per thread and round: T * CPT chunks (1024 or 2048) at a time
  uint32_t cnt[CPT];
  auto load_counts = [&](int c0) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int ch = c0 + (int)threadIdx.x * CPT + i;
      cnt[i] = ch < ta.nblk ? ta.blk[(size_t)b * ta.nblk + ch] : 0u;
    }
  };
  load_counts(0);
  float2 stat = make_float2(0.f, 1.f);
  if (threadIdx.x < H) stat = *reinterpret_cast<const float2*>(a.row_stats + ((size_t)b * H + threadIdx.x) * 2);
  uint4 qw[NP];
  double qd[NP * EPP];
  {
    const uint8_t* qp = a.q + ((size_t)b * H + (size_t)kvh * G + (ONE ? 0 : min(g, G - 1))) * RB + kk * 16;
#pragma unroll
    for (int i = 0; i < NP; ++i) qw[i] = *reinterpret_cast<const uint4*>(qp + i * 64);
  }
  auto convert_q = [&]() {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if (!ONE && g >= G) qw[i] = make_uint4(0u, 0u, 0u, 0u);
      unpack_f64<DT>(qw[i], qd + i * EPP);
    }
  };
  // the lower bounds' histogram has been consumed by the compaction: leave it zeroed, a share per workgroup
  auto clear = [&]() {
    uint4* g0 = reinterpret_cast<uint4*>(ta.rep_hist + (size_t)b * kBoundHistCopies * kTopkBins);   // 256-byte aligned section
    for (int i = (int)(blockIdx.x * T + threadIdx.x); i < kBoundHistCopies * kTopkBins / 4; i += (int)gridDim.x * T)
      g0[i] = make_uint4(0u, 0u, 0u, 0u);
  };
  // ---- prefix of the chunks' candidate counts
  uint32_t carry = 0;
  for (int c0 = 0; c0 < ta.nblk; c0 += T * CPT) {
    const int ch = c0 + (int)threadIdx.x * CPT;
    if (c0 != 0) load_counts(c0);
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < CPT; ++i) sum += cnt[i];
    const uint32_t incl = wave_inclusive_scan(sum);
    __syncthreads();
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t base = carry + incl - sum;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const uint32_t x = wave_sum[w];
      if (w < wave) base += x;
      carry += x;
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i) { if (ch + i < ta.nblk) off[ch + i] = base; base += cnt[i]; }
  }
  if (threadIdx.x == 0) off[ta.nblk] = carry;
  if (threadIdx.x < H) { s_m[threadIdx.x] = (double)stat.x; s_inv[threadIdx.x] = 1.0 / (double)stat.y; }
  const uint32_t total = carry;
  if (blockIdx.x == 0 && threadIdx.x == 0) ta.state[b * 8 + kStTotal] = total;
  __syncthreads();
  const uint32_t groups = min((uint32_t)gridDim.x, (total + kEvalMinShare - 1) / kEvalMinShare);   // that have work
  if (blockIdx.x >= groups) { clear(); return; }
  const uint32_t c_begin = (uint32_t)((unsigned long long)total * blockIdx.x / groups);
  const uint32_t c_end = (uint32_t)((unsigned long long)total * (blockIdx.x + 1) / groups);
  const double c2d = (double)a.scale * 1.44269504088896340736;
  const int npages = (Nb + a.P - 1) >> a.p_shift;
  uint2* dense = ta.dense + (size_t)b * ta.nblk * kTopkChunk;
  for (uint32_t c0 = c_begin; c0 < c_end; c0 += cb) {
    const int n = (int)min((uint32_t)cb, c_end - c0);
    if ((int)threadIdx.x < n) {                        // one thread per candidate: its token and its row in the pool
      const uint32_t i = c0 + threadIdx.x;
      int lo = 0, hi = ta.nblk;                        // off[lo] <= i < off[hi]
      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (off[mid] <= i) lo = mid; else hi = mid; }
      const int t = (int)ta.list[((size_t)b * ta.nblk + lo) * kTopkChunk + (i - off[lo])].y;
      const int pid = a.page_indices[indptr + min(t >> a.p_shift, npages - 1)];
      ctok[threadIdx.x] = t;
      cslot[threadIdx.x] = ((long long)pid << a.p_shift) + (t & (a.P - 1));
    }
    __syncthreads();
    const int nsteps = (n + tps - 1) / tps;
    // steps of this wave: wsub, wsub + wstep, ...; a piece of the next step's rows is asked for as soon as one has been converted
    auto row_of = [&](int st) -> const uint8_t* {
      return a.k_pool + ((size_t)cslot[min(st * tps + cand + c, n - 1)] * a.H_kv + kvh) * RB + kk * 16;
    };
    uint4 buf[NP];
    auto step = [&](int st, bool more) {
      const uint8_t* kn = more ? row_of(st + wstep) : nullptr;
      double acc[2] = {0.0, 0.0};
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        double kd[EPP];
        unpack_f64<DT>(buf[i], kd);
        if (more) buf[i] = *reinterpret_cast<const uint4*>(kn + i * 64);
        // products of two floats are exact in double
#pragma unroll
        for (int e = 0; e < EPP; ++e)
          acc[e & 1] = ONE ? fma(kd[e], qd[i * EPP + e], acc[e & 1]) : __builtin_amdgcn_mfma_f64_4x4x4f64(kd[e], qd[i * EPP + e], acc[e & 1], 0, 0, 0);
      }
      const double sum = ONE ? quarter_sum_f64(acc[0] + acc[1]) : acc[0] + acc[1];
      const int ci = st * tps + cand + (ONE ? c : kk);
      if (ci < n && (ONE ? kk == 0 : g < G)) sc[(size_t)ci * H + (ONE ? kvh : kvh * G + g)] = sum;
    };
    int st = wsub;
    if (st < nsteps) {
      const uint8_t* kp = row_of(st);
#pragma unroll
      for (int i = 0; i < NP; ++i) buf[i] = *reinterpret_cast<const uint4*>(kp + i * 64);
    }
    if (c0 == c_begin) { convert_q(); clear(); }
    if (st < nsteps) {
      for (; st + wstep < nsteps; st += wstep) step(st, true);
      step(st, false);
    }
    __syncthreads();
    // ---- votes: 16 lanes per candidate
    for (int ci = (int)threadIdx.x >> 4; ci < ((n + 15) & ~15); ci += T / 16) {
      const int cc = min(ci, n - 1);
      double vote = 0.0;
      for (int h = (int)threadIdx.x & 15; h < H; h += 16)
        vote += (double)refine_vote_exp(sc[(size_t)cc * H + h] - s_m[h], c2d) * s_inv[h];
      vote += dpp_f64<kDppXor1>(vote);
      vote += dpp_f64<kDppXor2>(vote);
      vote += dpp_f64<kDppHalfMirror>(vote);
      vote += dpp_f64<kDppRor8>(vote);
      if (ci < n && (threadIdx.x & 15) == 0) dense[c0 + ci] = make_uint2(float_key((float)vote), (uint32_t)ctok[ci]);
    }
    __syncthreads();
  }
}

template <int DT, int D>
static hipError_t eval_g(int G, const RefineArgs& a, dim3 grid, hipStream_t s) {
  // the scores of a batch and the prefix of the chunk counts (8192 at most) fit 64 KiB beside 6 KiB of static LDS
  const size_t off_bytes = (size_t)(a.t.nblk + 1) * sizeof(uint32_t);
  int cb = (int)((59392 - off_bytes) / ((size_t)a.H * sizeof(double)));
  if (cb > kEvalMaxBatch) cb = kEvalMaxBatch;
  const size_t lds = (size_t)cb * a.H * sizeof(double) + off_bytes;
  const int units = (a.H_kv + 3) / 4 * (G > 4 ? 2 : 1);
#define TS_EVAL(CS, WAVES, ONE) hipLaunchKernelGGL((topk_eval_kernel<DT, D, CS, WAVES, ONE>), grid, dim3(64 * WAVES), lds, s, a, cb)
  if (G > 4) { if (units > 4) TS_EVAL(2, 8, false); else TS_EVAL(2, 4, false); }
  else if (G > 1) { if (units > 4) TS_EVAL(1, 8, false); else TS_EVAL(1, 4, false); }
  else { if (units > 4) TS_EVAL(1, 8, true); else TS_EVAL(1, 4, true); }
#undef TS_EVAL
  return hipGetLastError();
}

hipError_t launch_topk_eval(int dtype, int D, int G, const RefineArgs& a, int B, hipStream_t s) {
  const dim3 grid(a.parts, B);
  if (dtype == TS_F32) return D == 64 ? eval_g<TS_F32, 64>(G, a, grid, s) : eval_g<TS_F32, 128>(G, a, grid, s);
  return D == 64 ? eval_g<TS_BF16, 64>(G, a, grid, s) : eval_g<TS_BF16, 128>(G, a, grid, s);
}

}  // namespace ts
