// TopK of Eq. 3-5 as an exact radix select over 32-bit order-preserving keys.
//
// Three histogram passes (11 + 11 + 10 bits) find the key of the k-th largest value: every
// workgroup histograms its 2048-key chunk in LDS and adds the non-empty bins to a global histogram;
// the next kernel's workgroups each walk that (8 KiB, cache-resident) histogram from the top and fix
// the digit for themselves, so no kernel waits on another workgroup and nothing but the kernel
// boundary orders the passes.  The emit pass writes the winners in token order: all keys above
// the threshold plus the first (k - #above) keys equal to it.  How many of both the earlier chunks hold it reads from a
// table that the third pass leaves, a chunk's number of keys at or above every value of the last digit (kTableChunks); for
// longer sequences a counting pass in between records them per chunk.  That is the "lower token index wins ties" rule and yields
// ascending indices without a sort.
#include "ts_kernels.h"

namespace ts {


// exclusive prefix sum over the 256 threads of a workgroup; *total receives the sum
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total, uint32_t* lds /* >= 5 words */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) lds[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t x = lds[w];
    if (w < wave) base += x;
    tot += x;
  }
  *total = tot;
  return base + incl - v;
}

// Walks a global histogram from its top bin down and finds the bin holding the k_rem-th largest key.
// All 256 threads call it and all get the result: digit and the rank remaining inside that bin.
// An empty selection (k_rem == 0) returns digit = NB (no key can match it).
template <int NB>
__device__ __forceinline__ void find_digit(const uint32_t* gh, uint32_t k_rem, uint32_t* digit, uint32_t* k_next,
                                           uint32_t* lds /* >= 8 words */) {
  constexpr int PER = NB / 256;
  uint32_t c[PER];
  uint32_t sum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {   // thread 0 owns the top PER bins, in descending order
    c[e] = gh[NB - 1 - (threadIdx.x * PER + e)];
    sum += c[e];
  }
  uint32_t total;
  uint32_t above = block_exclusive_scan(sum, &total, lds);
  __syncthreads();
  if (threadIdx.x == 0) { lds[5] = NB; lds[6] = 0u; }
  __syncthreads();
  if (k_rem != 0) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (above < k_rem && k_rem <= above + c[e]) { lds[5] = NB - 1 - (threadIdx.x * PER + e); lds[6] = k_rem - above; }
      above += c[e];
    }
  }
  __syncthreads();
  *digit = lds[5];
  *k_next = lds[6];
  __syncthreads();
}

// find_digit over a histogram kept as kBoundHistCopies replicas (the vote kernel's flush spreads its atomics
// over them): the copies are summed on the way in.  Votes are not negative, their keys lie in the upper half of the bins: the
// lower half is only read where that does not hold k_rem entries.  (Every workgroup reads the copies, 32 KiB instead of 64:
// topk_compact_kernel, us, compact form, 1048576 tokens of H 28/4, k 4096, 5.6 and 4.8; 32 sequences of 1031 to 16001, 32/8, k 2048, 6.6 and
// 5.7, five-call form 6.4 and 5.3; 131072 4.8 and 4.4.  A whole step gains less than two runs of it differ.)
template <int NB>
__device__ __forceinline__ void find_digit_rep(const uint32_t* gh, uint32_t k_rem, uint32_t* digit, uint32_t* k_next,
                                               uint32_t* lds /* >= 8 words */) {
  constexpr int HALF = NB / 2;
  static_assert(HALF == 4 * 256, "four bins per thread, one 16-byte load per copy");
  uint32_t seen = 0;                          // entries of the halves gone through
  for (int half = 1; half >= 0; --half) {
    // the thread's bins are consecutive in memory (descending bin order = ascending address from `lowest`)
    const int lowest = half * HALF + HALF - 4 - (int)threadIdx.x * 4;
    uint4 w[kBoundHistCopies];
#pragma unroll
    for (int r = 0; r < kBoundHistCopies; ++r) w[r] = *reinterpret_cast<const uint4*>(gh + r * NB + lowest);
    uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < kBoundHistCopies; ++r) { c[0] += w[r].w; c[1] += w[r].z; c[2] += w[r].y; c[3] += w[r].x; }
    uint32_t total;
    if (threadIdx.x == 0) { lds[5] = NB; lds[6] = 0u; }      // the scan's barriers stand between this and the writes below
    uint32_t above = seen + block_exclusive_scan(c[0] + c[1] + c[2] + c[3], &total, lds);
    if (k_rem != 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (above < k_rem && k_rem <= above + c[e]) { lds[5] = (uint32_t)(lowest + 3 - e); lds[6] = k_rem - above; }
        above += c[e];
      }
    }
    seen += total;
    if (k_rem <= seen) break;                 // the same in all threads
    __syncthreads();
  }
  __syncthreads();
  *digit = lds[5];
  *k_next = lds[6];
  __syncthreads();
}

// The counting pass read all votes once more for a launch's latency.  ts_topk on flat votes, five launches and four: 20000 tokens 21.0
// and 18.4 us, 131072 22.3 and 19.4, 8 x 262144 33.1 and 30.0, 1048576, the last length with the table, 39.0 and 36.5.  Beyond, the
// emit pass' reads, a piece of the table for every pair of chunks, grow with the square of their number.
constexpr int kTableChunks = 512;

// state words per sequence
enum { ST_PREFIX0 = 0, ST_KREM0 = 1, ST_KEFF = 2, ST_PREFIX1 = 3, ST_KREM1 = 4, ST_THR = 5, ST_NEED_EQ = 6 };

// tokens [LO, N) of a sequence take part: forced initial tokens, the chunk's own tokens and forced recent
// tokens do not
// (b is the virtual sequence: a.heads of them share one real sequence's length)
__device__ __forceinline__ int ranked_lo(const TopkArgs& a, int b) {
  return min(a.head, min(max(a.seq_lens[b / a.heads], 0), a.max_seq_len));
}
__device__ __forceinline__ int ranked_hi(const TopkArgs& a, int b, int lo) {
  return max(lo, min(max(a.seq_lens[b / a.heads], 0), a.max_seq_len) - a.tail);
}

__device__ __forceinline__ void load_keys(const float* v, int base, int LO, int N, uint32_t* key, bool* valid) {
#pragma unroll
  for (int i = 0; i < kTopkChunk / 256; ++i) {
    const int t = base + i * 256 + threadIdx.x;
    valid[i] = t >= LO && t < N;
    key[i] = valid[i] ? float_key(v[t]) : 0u;
  }
}

__device__ __forceinline__ void flush_hist(const uint32_t* h, uint32_t* gh, int nb) {
  for (int i = threadIdx.x; i < nb; i += 256)
    if (h[i] != 0) atomicAdd(&gh[i], h[i]);
}

// pass 0: histogram of the top 11 key bits.  A workgroup walks every gridDim.x-th chunk and flushes its LDS
// histogram once: the flush is atomics on a few hundred hot bins, so fewer, fatter workgroups contend less.
__global__ __launch_bounds__(256) void topk_hist0_kernel(TopkArgs a) {
  __shared__ uint32_t h[kTopkBins];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  if ((int)blockIdx.x * kTopkChunk >= N) return;
  for (int i = threadIdx.x; i < kTopkBins; i += 256) h[i] = 0;
  __syncthreads();
  for (int base = blockIdx.x * kTopkChunk; base < N; base += gridDim.x * kTopkChunk) {
    uint32_t key[kTopkChunk / 256]; bool valid[kTopkChunk / 256];
    load_keys(a.votes + (size_t)b * a.max_seq_len, base, LO, N, key, valid);
#pragma unroll
    for (int i = 0; i < kTopkChunk / 256; ++i)
      if (valid[i]) atomicAdd(&h[key[i] >> 21], 1u);
  }
  __syncthreads();
  flush_hist(h, a.hist + ((size_t)b * 2 + 0) * kTopkBins, kTopkBins);
}

// pass 1: fix digit 0 from histogram 0 (or the vote kernel's copies of it, whose fold into one took a launch more), histogram
// the next 11 bits of the keys that carry it; histogram 2, which lies in scratch memory because all of the emit pass' workgroups
// may read it, so that none can leave it zeroed, is cleared for pass 2
__global__ __launch_bounds__(256) void topk_hist1_kernel(TopkArgs a) {
  __shared__ uint32_t h[kTopkBins];
  __shared__ uint32_t lds[8];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  const int base = blockIdx.x * kTopkChunk;
  if (base >= N && blockIdx.x != 0) return;
  uint32_t key[kTopkChunk / 256]; bool valid[kTopkChunk / 256];
  load_keys(a.votes + (size_t)b * a.max_seq_len, base, LO, N, key, valid);
  for (int i = threadIdx.x; i < kTopkBins; i += 256) h[i] = 0;
  const uint32_t k_eff = (uint32_t)min(a.k, N - LO);
  uint32_t d0, krem0;
  if (a.rep_hist != nullptr) find_digit_rep<kTopkBins>(a.rep_hist + (size_t)b * kBoundHistCopies * kTopkBins, k_eff, &d0, &krem0, lds);
  else find_digit<kTopkBins>(a.hist + ((size_t)b * 2 + 0) * kTopkBins, k_eff, &d0, &krem0, lds);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.state[b * 8 + ST_PREFIX0] = d0 << 21; a.state[b * 8 + ST_KREM0] = krem0; a.state[b * 8 + ST_KEFF] = k_eff;
  }
  if (blockIdx.x == 0) {
    uint32_t* g2 = a.hist2 + (size_t)b * 1024;
    for (int i = threadIdx.x; i < 1024; i += 256) g2[i] = 0u;
  }
#pragma unroll
  for (int i = 0; i < kTopkChunk / 256; ++i)
    if (valid[i] && (key[i] >> 21) == d0) atomicAdd(&h[(key[i] >> 10) & 2047u], 1u);
  __syncthreads();
  flush_hist(h, a.hist + ((size_t)b * 2 + 1) * kTopkBins, kTopkBins);
}

// pass 2: fix digit 1, histogram the last 10 bits; histogram 0 is no longer needed and is cleared.  TABLE: also the chunk's
// row of the table, for every value of the last digit the number of its keys there or above (at most 2048), and apart the
// number above all of them.
template <bool TABLE>
__global__ __launch_bounds__(256) void topk_hist2_kernel(TopkArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t h[1024];
  __shared__ uint32_t lds[8];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  const int base = blockIdx.x * kTopkChunk;
  if (base >= N && blockIdx.x != 0) return;
  uint32_t key[kTopkChunk / 256]; bool valid[kTopkChunk / 256];
  load_keys(a.votes + (size_t)b * a.max_seq_len, base, LO, N, key, valid);
  for (int i = threadIdx.x; i < 1024; i += 256) h[i] = 0;
  const uint32_t prefix0 = a.state[b * 8 + ST_PREFIX0], krem0 = a.state[b * 8 + ST_KREM0];
  uint32_t d1, krem1;
  find_digit<kTopkBins>(a.hist + ((size_t)b * 2 + 1) * kTopkBins, krem0, &d1, &krem1, lds);
  // an empty selection keeps an impossible prefix so that nothing matches below
  const bool none = krem0 == 0;
  const uint32_t prefix1 = prefix0 | ((d1 & 2047u) << 10);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) { a.state[b * 8 + ST_PREFIX1] = prefix1; a.state[b * 8 + ST_KREM1] = none ? 0u : krem1; }
    if (a.rep_hist != nullptr) {
      uint4* g0 = reinterpret_cast<uint4*>(a.rep_hist + (size_t)b * kBoundHistCopies * kTopkBins);
      for (int i = threadIdx.x; i < kBoundHistCopies * kTopkBins / 4; i += 256) g0[i] = make_uint4(0u, 0u, 0u, 0u);
    } else {
      uint32_t* g0 = a.hist + ((size_t)b * 2 + 0) * kTopkBins;
      for (int i = threadIdx.x; i < kTopkBins; i += 256) g0[i] = 0u;
    }
  }
#pragma unroll
  for (int i = 0; i < kTopkChunk / 256; ++i)
    if (valid[i] && !none && (key[i] >> 10) == (prefix1 >> 10)) atomicAdd(&h[key[i] & 1023u], 1u);
  __syncthreads();
  flush_hist(h, a.hist2 + (size_t)b * 1024, 1024);
  if (TABLE) {
    uint32_t gt = 0;
#pragma unroll
    for (int i = 0; i < kTopkChunk / 256; ++i) gt += valid[i] && !none && (key[i] >> 10) > (prefix1 >> 10);
    const int lowest = 1020 - 4 * (int)threadIdx.x;             // thread 0 owns the top four values
    const uint4 c = *reinterpret_cast<const uint4*>(&h[lowest]);
    uint32_t total;
    const uint32_t ex = block_exclusive_scan((c.x + c.y + c.z + c.w) | (gt << 16), &total, lds);
    const uint32_t w3 = (total >> 16) + (ex & 0xffffu) + c.w, w2 = w3 + c.z, w1 = w2 + c.y, w0 = w1 + c.x;
    const size_t chunk = (size_t)b * a.nblk + blockIdx.x;
    *reinterpret_cast<uint2*>(a.table + chunk * 1024 + lowest) = make_uint2(w0 | (w1 << 16), w2 | (w3 << 16));
    if (threadIdx.x == 0) a.blk[chunk] = total >> 16;
  }
}

// fix the last digit (the threshold key is now exact) and count, per chunk, the keys above / equal to it
__global__ __launch_bounds__(256) void topk_count_kernel(TopkArgs a) {
  __shared__ uint32_t lds[8];
  __shared__ uint32_t red[4];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  const int base = blockIdx.x * kTopkChunk;
  uint32_t key[kTopkChunk / 256]; bool valid[kTopkChunk / 256];
  load_keys(a.votes + (size_t)b * a.max_seq_len, base, LO, N, key, valid);
  const uint32_t prefix1 = a.state[b * 8 + ST_PREFIX1], krem1 = a.state[b * 8 + ST_KREM1];
  uint32_t d2, need_eq;
  find_digit<1024>(a.hist2 + (size_t)b * 1024, krem1, &d2, &need_eq, lds);
  const bool none = krem1 == 0;
  const uint32_t thr = none ? 0xffffffffu : (prefix1 | (d2 & 1023u));
  if (none) need_eq = 0;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      a.state[b * 8 + ST_THR] = thr; a.state[b * 8 + ST_NEED_EQ] = need_eq;
    }
    uint32_t* g1 = a.hist + ((size_t)b * 2 + 1) * kTopkBins;
    for (int i = threadIdx.x; i < kTopkBins; i += 256) g1[i] = 0u;
  }
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int i = 0; i < kTopkChunk / 256; ++i) {
    gt += valid[i] && !none && key[i] > thr;
    eq += valid[i] && !none && key[i] == thr;
  }
  uint32_t packed = gt | (eq << 16);   // a chunk holds 2048 keys: both counts fit in 16 bits
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) packed += __shfl_xor(packed, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = packed;
  __syncthreads();
  if (threadIdx.x == 0) a.blk[(size_t)b * a.nblk + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// winners of a chunk, in token order; every workgroup sums the counts of the chunks before it.  TABLE: it fixes the last
// digit for itself and looks the counts up in the table of pass 2.
template <bool TABLE>
__global__ __launch_bounds__(256) void topk_emit_kernel(TopkArgs a) {
  __shared__ uint32_t scan_lds[8];
  __shared__ uint32_t red[2][4];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  uint32_t thr = a.state[b * 8 + (TABLE ? ST_PREFIX1 : ST_THR)];
  uint32_t need_eq = TABLE ? 0u : a.state[b * 8 + ST_NEED_EQ];
  const uint32_t krem1 = a.state[b * 8 + ST_KREM1];
  const bool none = krem1 == 0;
  const int k_eff = (int)a.state[b * 8 + ST_KEFF];
  const bool as_votes = a.vote_acc != nullptr;      // Eq. 4: winners are counted per token, not listed
  int32_t* out = as_votes ? nullptr : a.idx + (size_t)b * a.k;
  float* acc = as_votes ? a.vote_acc + (size_t)(b / a.heads) * a.max_seq_len : nullptr;
  if (blockIdx.x == 0) {
    if (!as_votes) {
      for (int i = k_eff + threadIdx.x; i < a.k; i += 256) out[i] = -1;
      if (threadIdx.x == 0) a.count[b] = k_eff;
    }
    if (TABLE) {
      uint32_t* g1 = a.hist + ((size_t)b * 2 + 1) * kTopkBins;
      for (int i = threadIdx.x; i < kTopkBins; i += 256) g1[i] = 0u;
    }
  }
  const int base = blockIdx.x * kTopkChunk;
  if (base >= N || none) return;
  const float* v = a.votes + (size_t)b * a.max_seq_len;
  constexpr int PER = kTopkChunk / 256;
  const int t0 = base + threadIdx.x * PER;   // PER consecutive tokens per thread: order is preserved
  uint32_t key[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) key[e] = ((t0 + e) >= LO && (t0 + e) < N) ? float_key(v[t0 + e]) : 0u;
  // counts of all earlier chunks
  uint32_t pg = 0, pe = 0;
  const uint32_t* blk = a.blk + (size_t)b * a.nblk;
  if (TABLE) {
    uint32_t d2;
    find_digit<1024>(a.hist2 + (size_t)b * 1024, krem1, &d2, &need_eq, scan_lds);
    d2 &= 1023u;
    thr |= d2;
    const uint16_t* row = a.table + (size_t)b * a.nblk * 1024 + d2;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) {
      const uint32_t ge = row[(size_t)i * 1024], g = d2 == 1023u ? blk[i] : (uint32_t)row[(size_t)i * 1024 + 1];
      pg += g; pe += ge - g;
    }
  } else {       // gt in the low half is too narrow for a sum: add the halves apart
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) { const uint32_t x = blk[i]; pg += x & 0xffffu; pe += x >> 16; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { pg += __shfl_xor(pg, off); pe += __shfl_xor(pe, off); }
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = pg; red[1][threadIdx.x >> 6] = pe; }
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const bool valid = (t0 + e) >= LO && (t0 + e) < N;
    gt += valid && key[e] > thr;
    eq += valid && key[e] == thr;
  }
  uint32_t total;
  const uint32_t ex = block_exclusive_scan(gt | (eq << 16), &total, scan_lds);   // has the barriers red[] needs
  uint32_t gt_before = red[0][0] + red[0][1] + red[0][2] + red[0][3] + (ex & 0xffffu);
  uint32_t eq_before = red[1][0] + red[1][1] + red[1][2] + red[1][3] + (ex >> 16);
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int t = t0 + e;
    if (t >= LO && t < N) {
      if (key[e] > thr) {
        if (as_votes) atomicAdd(&acc[t], 1.0f);      // small integers: exact and order-independent in float
        else out[gt_before + min(eq_before, need_eq)] = t;
        ++gt_before;
      } else if (key[e] == thr) {
        if (eq_before < need_eq) {
          if (as_votes) atomicAdd(&acc[t], 1.0f);
          else out[gt_before + eq_before] = t;
        }
        ++eq_before;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Short path (3 launches): after pass 0 every chunk compacts, in token order, the keys that fall in or above
// the bin of the k-th key (the winners for sure plus the few candidates that share its bin; typically k plus a
// few hundred entries in all), and one workgroup per sequence finishes the job on that list: two more radix
// digits over the candidates in LDS histograms, then the ordered emit.  Same result as the passes over all votes.

constexpr int kFinalThreads = 1024;        // many threads, few entries each: the per-entry chain of a thread is the latency
                                           // that counts (256 threads x 32 entries measured 1.7x slower)
constexpr int kFinalMaxBlk = 8192;         // chunks per sequence the short path handles (16 Mi tokens)
constexpr int kTieMax = 256;               // entries of one 2^13-key bin that the finish ranks among themselves

// pass 1 of the short path: fix digit 0, compact the entries with (key >> 21) >= digit 0
__global__ __launch_bounds__(256) void topk_compact_kernel(TopkArgs a) {
  __shared__ uint32_t lds[8];
  __shared__ uint32_t scan_lds[8];
  const int b = blockIdx.y;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the length
  const int LO = ranked_lo(a, b), N = ranked_hi(a, b, LO);
  if (skip_flag != 0) return;
  const uint32_t k_eff = (uint32_t)min(a.k, N - LO);
  constexpr int PER = kTopkChunk / 256;
  const int base = blockIdx.x * kTopkChunk;
  const int t0 = base + threadIdx.x * PER;   // PER consecutive tokens per thread: order is preserved
  const float* v = a.votes + (size_t)b * a.max_seq_len;
  // the votes are loaded before the histogram is walked: the two round trips overlap
  uint32_t key[PER];
  bool valid[PER];
  if (((reinterpret_cast<uintptr_t>(v) & 15) == 0) && base + kTopkChunk <= a.max_seq_len) {
    // the usual case: 16-byte loads (the row exists up to max_seq_len)
#pragma unroll
    for (int q4 = 0; q4 < PER / 4; ++q4) {
      const float4 w = *reinterpret_cast<const float4*>(v + t0 + q4 * 4);
      const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = q4 * 4 + i;
        valid[e] = (t0 + e) >= LO && (t0 + e) < N;
        key[e] = valid[e] ? float_key(x[i]) : 0u;
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      valid[e] = (t0 + e) >= LO && (t0 + e) < N;
      key[e] = valid[e] ? float_key(v[t0 + e]) : 0u;
    }
  }
  uint32_t d0, krem0;
  if (a.rep_hist != nullptr) find_digit_rep<kTopkBins>(a.rep_hist + (size_t)b * kBoundHistCopies * kTopkBins, k_eff, &d0, &krem0, lds);
  else find_digit<kTopkBins>(a.hist + ((size_t)b * 2 + 0) * kTopkBins, k_eff, &d0, &krem0, lds);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.state[b * 8 + ST_PREFIX0] = d0 << 21; a.state[b * 8 + ST_KREM0] = krem0; a.state[b * 8 + ST_KEFF] = k_eff;
  }
  uint32_t n = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) n += valid[e] && (key[e] >> 21) >= d0;      // d0 == kTopkBins (empty selection) matches nothing
  uint32_t total;
  uint32_t pos = block_exclusive_scan(n, &total, scan_lds);
  uint2* list = a.list + ((size_t)b * a.nblk + blockIdx.x) * kTopkChunk;
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (valid[e] && (key[e] >> 21) >= d0) list[pos++] = make_uint2(key[e], (uint32_t)(t0 + e));
  if (threadIdx.x == 0) a.blk[(size_t)b * a.nblk + blockIdx.x] = total;
}

// exclusive prefix sum over the kFinalThreads threads of the final workgroup
__device__ __forceinline__ uint32_t final_exclusive_scan(uint32_t v, uint32_t* total, uint32_t* lds /* >= 16 words */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) lds[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kFinalThreads / 64; ++w) {
    const uint32_t x = lds[w];
    if (w < wave) base += x;
    tot += x;
  }
  *total = tot;
  return base + incl - v;
}

// digit of the k_rem-th largest key in an LDS histogram of NB bins (all threads get the result)
template <int NB>
__device__ __forceinline__ void final_find_digit(const uint32_t* h, uint32_t k_rem, uint32_t* digit, uint32_t* k_next,
                                                 uint32_t* scan_lds, uint32_t* res /* 2 words */) {
  constexpr int PER = NB / kFinalThreads;
  uint32_t c[PER];
  uint32_t sum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) { c[e] = h[NB - 1 - (threadIdx.x * PER + e)]; sum += c[e]; }
  uint32_t total;
  uint32_t above = final_exclusive_scan(sum, &total, scan_lds);
  if (threadIdx.x == 0) { res[0] = NB; res[1] = 0u; }
  __syncthreads();
  if (k_rem != 0) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (above < k_rem && k_rem <= above + c[e]) { res[0] = NB - 1 - (threadIdx.x * PER + e); res[1] = k_rem - above; }
      above += c[e];
    }
  }
  __syncthreads();
  *digit = res[0];
  *k_next = res[1];
  __syncthreads();
}

// passes 2, 3 and the emit of the short path: one workgroup per (virtual) sequence
// FULL: the entries are the re-evaluated candidates of the compact selection, listed without gaps (a.dense); their
// keys are exact votes, of which only the lower edge of the k-th largest lower bound's bin is known.
// SHORT: no list at all: a sequence of at most kFinalThreads * kFinalPer tokens whose votes this workgroup reads itself;
// digit 0 is counted here.
enum { FINAL_LIST = 0, FINAL_FULL = 1, FINAL_SHORT = 2 };
template <int kFinalPer, int MODE>         // consecutive entries per thread and batch
__global__ __launch_bounds__(kFinalThreads) void topk_final_kernel(TopkArgs a) {
  constexpr bool FULL = MODE == FINAL_FULL, SHORT = MODE == FINAL_SHORT;
  __shared__ uint32_t off[MODE != FINAL_LIST ? 1 : kFinalMaxBlk + 1];   // exclusive prefix of the chunks' entry counts
  __shared__ uint32_t h[kTopkBins];
  __shared__ uint32_t tie[FULL ? kTieMax : 1];            // keys that share the k-th key's bin
  __shared__ uint32_t n_tie;
  __shared__ uint32_t scan_lds[16];
  __shared__ uint32_t res[2];
  const int b = blockIdx.x;
  const int skip_flag = a.skip != nullptr ? (int)a.skip[b / a.heads] : 0;   // issued together with the state words
  const int tid = threadIdx.x;
  const int LO = SHORT ? ranked_lo(a, b) : 0, N = SHORT ? ranked_hi(a, b, LO) : 0;
  uint32_t d0 = MODE != FINAL_LIST ? 0u : a.state[b * 8 + ST_PREFIX0] >> 21, krem0 = MODE != FINAL_LIST ? 0u : a.state[b * 8 + ST_KREM0];
  const int k_eff = SHORT ? min(a.k, N - LO) : (int)a.state[b * 8 + ST_KEFF];
  // What the list's loads can be given before the lengths, the counts and the state are known leaves beside those: of the
  // candidates the first 1 1/8 k, which are there as a rule (the section holds a.nblk * kTopkChunk; the others follow when their
  // number is known), of the chunks their counts.  The clearing stores below stand behind them: a load waits for the stores
  // before it.  (This kernel, compact form, us, before and so: 131072 tokens, H 32/8, k 2048, 5.4 and 5.2; 1048576 of 28/4, k 4096, 7.6 and
  // 7.3; 32 of 1031 to 16001 7.0 and 6.2.  A whole batch of places loaded early is more than the list: k 4096 7.9; k places 7.5.)
  uint2 e[kFinalPer];
  const uint2* dense = FULL ? a.dense + (size_t)b * a.nblk * kTopkChunk : nullptr;
  auto load_dense = [&](uint32_t p0) {
#pragma unroll
    for (int i = 0; i < kFinalPer; i += 2) {
      uint4 w = make_uint4(0u, 0u, 0u, 0u);
      if (p0 + i < (uint32_t)a.nblk * kTopkChunk) w = *reinterpret_cast<const uint4*>(dense + p0 + i);   // whole pairs
      e[i] = make_uint2(w.x, w.y);
      e[i + 1] = make_uint2(w.z, w.w);
    }
  };
  const uint32_t early = (uint32_t)a.k + (uint32_t)a.k / 8;
  if (FULL && (uint32_t)tid * kFinalPer < early) load_dense((uint32_t)tid * kFinalPer);
  const uint32_t n_first = MODE == FINAL_LIST && tid < a.nblk ? a.blk[(size_t)b * a.nblk + tid] : 0u;
  if (skip_flag != 0) return;
  if (SHORT) {                               // the votes' loads go out first
    const float* v = a.votes + (size_t)b * a.max_seq_len;
    const int t0 = tid * kFinalPer;
    if ((reinterpret_cast<uintptr_t>(v) & 15) == 0 && t0 + kFinalPer <= a.max_seq_len) {     // 16-byte loads (the row exists up to max_seq_len)
#pragma unroll
      for (int q4 = 0; q4 < kFinalPer / 4; ++q4) {
        const float4 w = *reinterpret_cast<const float4*>(v + t0 + q4 * 4);
        const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = t0 + q4 * 4 + i;
          e[q4 * 4 + i] = (t >= LO && t < N) ? make_uint2(float_key(x[i]), (uint32_t)t) : make_uint2(0u, 0xffffffffu);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < kFinalPer; ++i) {
        const int t = t0 + i;
        e[i] = (t >= LO && t < N) ? make_uint2(float_key(v[t]), (uint32_t)t) : make_uint2(0u, 0xffffffffu);
      }
    }
    for (int i = tid; i < kTopkBins; i += kFinalThreads) h[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFinalPer; ++i)
      if (e[i].y != 0xffffffffu) atomicAdd(&h[e[i].x >> 21], 1u);
    __syncthreads();
    final_find_digit<kTopkBins>(h, (uint32_t)k_eff, &d0, &krem0, scan_lds, res);
  }
  const bool as_votes = a.vote_acc != nullptr;
  int32_t* out = as_votes ? nullptr : a.idx + (size_t)b * a.k;
  float* acc = as_votes ? a.vote_acc + (size_t)(b / a.heads) * a.max_seq_len : nullptr;
  auto clear = [&]() {
    if (!as_votes) {
      // FULL: the candidates come from float comparisons; with NaN among the votes fewer than k_eff of them may
      // arrive, and the slots that then stay empty must not keep an older selection's ids (finite votes fill them all)
      for (int i = (FULL ? 0 : k_eff) + tid; i < a.k; i += kFinalThreads) out[i] = -1;
      if (FULL && a.sel_votes != nullptr)
        for (int i = k_eff + tid; i < a.k; i += kFinalThreads) a.sel_votes[(size_t)b * a.k + i] = 0.f;
      if (tid == 0) a.count[b] = k_eff;
    }
    if (FULL || SHORT) {         // the lower bounds' histogram was cleared by the re-evaluation; short sequences have none
    } else if (a.rep_hist != nullptr) {   // the vote kernel's replicated histogram has been consumed by the compact pass
      uint4* g0 = reinterpret_cast<uint4*>(a.rep_hist + (size_t)b * kBoundHistCopies * kTopkBins);
      for (int i = tid; i < kBoundHistCopies * kTopkBins / 4; i += kFinalThreads) g0[i] = make_uint4(0u, 0u, 0u, 0u);
    } else {     // histogram 0 has been consumed by the compact pass: leave it zeroed for the next call
      uint32_t* g0 = a.hist + ((size_t)b * 2 + 0) * kTopkBins;
      for (int i = tid; i < kTopkBins; i += kFinalThreads) g0[i] = 0u;
    }
  };
  uint32_t total;
  if (SHORT) {
    total = (uint32_t)N;
  } else if (FULL) {
    total = min(a.state[b * 8 + kStTotal], (uint32_t)a.nblk * kTopkChunk);
  } else {
    // ---- chunk offsets
    uint32_t carry = 0;
    for (int c0 = 0; c0 < a.nblk; c0 += kFinalThreads) {
      const int c = c0 + tid;
      const uint32_t n = c0 == 0 ? n_first : c < a.nblk ? a.blk[(size_t)b * a.nblk + c] : 0u;
      uint32_t tot;
      const uint32_t ex = final_exclusive_scan(n, &tot, scan_lds);
      if (c < a.nblk) off[c] = carry + ex;
      carry += tot;
      __syncthreads();
    }
    total = carry;
    if (tid == 0) off[a.nblk] = total;
    __syncthreads();
  }
  if (total == 0 || k_eff == 0) { clear(); return; }
  const uint2* list = SHORT ? nullptr : a.list + (size_t)b * a.nblk * kTopkChunk;

  // entries of a batch: thread tid owns the kFinalPer consecutive positions from p0
  const bool single = SHORT || total <= (uint32_t)kFinalThreads * kFinalPer;   // the usual case: the list sits in registers
  auto load_batch = [&](uint32_t base) {
    const uint32_t p0 = base + (uint32_t)tid * kFinalPer;
    if (FULL) {
      if (base != 0u || !single || (p0 >= early && p0 < total)) load_dense(p0);
#pragma unroll
      for (int i = 0; i < kFinalPer; ++i)
        if (p0 + i >= total) e[i] = make_uint2(0u, 0xffffffffu);
      return;
    }
    int c = 0;
    if (p0 < total) {                         // chunk with off[c] <= p0 < off[c + 1]
      int lo = 0, hi = a.nblk;                // invariant: off[lo] <= p0 < off[hi]
      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (off[mid] <= p0) lo = mid; else hi = mid; }
      c = lo;
    }
    uint32_t cur = off[c], next = off[c + 1];
#pragma unroll
    for (int i = 0; i < kFinalPer; ++i) {
      const uint32_t p = p0 + i;
      e[i] = make_uint2(0u, 0xffffffffu);
      if (p < total) {
        while (p >= next) { ++c; cur = next; next = off[c + 1]; }   // ends: p < total = off[nblk]
        e[i] = list[(size_t)c * kTopkChunk + (p - cur)];
      }
    }
  };
  if (!SHORT && single) load_batch(0);
  clear();

  uint32_t thr, need_eq;
  bool fixed = false;                         // thr and need_eq are known (the same in all threads)
  if (FULL) {
    // The k-th vote lies at or above the lower edge of the bin that the k-th largest lower bound fell into, and
    // within the width of the bounds above it: 2048 bins of 2^13 keys from that edge on (two octaves) hold it, and a
    // bin of 2^13 keys (a thousandth of the vote) a few entries, which are ranked among themselves.  One histogram
    // pass instead of two or three (with the list dense and its scans on the DPP network, 1048576 tokens, k 4096: 14.5 -> 7.6 us).  Votes spread otherwise (the last bin also
    // takes everything above, or a bin holds more entries than can be ranked at once) go the general way below.
    const uint32_t edge = a.state[b * 8 + ST_PREFIX0];
    auto bin_of = [&](uint32_t key) -> uint32_t { return min((key - edge) >> 13, (uint32_t)kTopkBins - 1u); };
    for (int i = tid; i < kTopkBins; i += kFinalThreads) h[i] = 0u;
    if (tid == 0) n_tie = 0u;
    uint32_t above = 0u;
    __syncthreads();
    for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
      if (!single) load_batch(base);
#pragma unroll
      for (int i = 0; i < kFinalPer; ++i)
        if (e[i].y != 0xffffffffu && e[i].x >= edge) {
          const uint32_t d = bin_of(e[i].x);
          if (d < (uint32_t)kTopkBins - 1u) atomicAdd(&h[d], 1u);
          else ++above;                        // most entries: one addition per wave below instead of one each
        }
    }
    above = wave_inclusive_scan(above);
    if ((tid & 63) == 63 && above != 0u) atomicAdd(&h[kTopkBins - 1], above);
    __syncthreads();
    uint32_t d, krem;
    final_find_digit<kTopkBins>(h, (uint32_t)k_eff, &d, &krem, scan_lds, res);
    if (d < (uint32_t)kTopkBins - 1u && h[d] <= (uint32_t)kTieMax) {
      const int n = (int)h[d];
      for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
        if (!single) load_batch(base);
#pragma unroll
        for (int i = 0; i < kFinalPer; ++i)
          if (e[i].y != 0xffffffffu && e[i].x >= edge && bin_of(e[i].x) == d) tie[atomicAdd(&n_tie, 1u)] = e[i].x;
      }
      __syncthreads();
      if (tid < n) {
        const uint32_t mine = tie[tid];
        uint32_t gt = 0, eq = 0;
        for (int i = 0; i < n; ++i) { gt += tie[i] > mine; eq += tie[i] == mine; }
        if (gt < krem && krem <= gt + eq) { res[0] = mine; res[1] = krem - gt; }   // equal keys write equal values
      }
      __syncthreads();
      thr = res[0]; need_eq = res[1];
      fixed = true;
    }
    __syncthreads();
  }
  if (!fixed) {
    if (FULL) {   // ---- digit 0: bits 31..21 over all entries
      for (int i = tid; i < kTopkBins; i += kFinalThreads) h[i] = 0u;
      __syncthreads();
      for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
        if (!single) load_batch(base);
#pragma unroll
        for (int i = 0; i < kFinalPer; ++i)
          if (e[i].y != 0xffffffffu) atomicAdd(&h[e[i].x >> 21], 1u);
      }
      __syncthreads();
      final_find_digit<kTopkBins>(h, (uint32_t)k_eff, &d0, &krem0, scan_lds, res);
    }
    // ---- digit 1: bits 20..10 of the candidates (entries of bin d0)
    for (int i = tid; i < kTopkBins; i += kFinalThreads) h[i] = 0u;
    __syncthreads();
    for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
      if (!single) load_batch(base);
#pragma unroll
      for (int i = 0; i < kFinalPer; ++i)
        if (e[i].y != 0xffffffffu && (e[i].x >> 21) == d0) atomicAdd(&h[(e[i].x >> 10) & 2047u], 1u);
    }
    __syncthreads();
    uint32_t d1, krem1;
    final_find_digit<kTopkBins>(h, krem0, &d1, &krem1, scan_lds, res);
    const uint32_t prefix1 = (d0 << 21) | ((d1 & 2047u) << 10);
    // ---- digit 2: the last 10 bits -- unless every entry that shares the threshold's 22-bit prefix is a winner (the
    // usual case: a few thousand entries over 2^22 prefixes leave the threshold's bin with one or two), when the
    // prefix alone decides
    const uint32_t cnt1 = d1 < (uint32_t)kTopkBins ? h[d1] : 0xffffffffu;
    if (krem1 == cnt1 && prefix1 != 0u) {
      thr = prefix1 - 1u; need_eq = 0u;          // "above thr" = "prefix at least prefix1"; nothing equals thr among the winners
    } else {
      __syncthreads();                            // every thread has read cnt1 before the histogram is cleared
      for (int i = tid; i < 1024; i += kFinalThreads) h[i] = 0u;
      __syncthreads();
      for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
        if (!single) load_batch(base);
#pragma unroll
        for (int i = 0; i < kFinalPer; ++i)
          if (e[i].y != 0xffffffffu && (e[i].x >> 10) == (prefix1 >> 10)) atomicAdd(&h[e[i].x & 1023u], 1u);
      }
      __syncthreads();
      uint32_t d2;
      final_find_digit<1024>(h, krem1, &d2, &need_eq, scan_lds, res);
      thr = prefix1 | (d2 & 1023u);
    }
  }
  // ---- emit in token order: every key above the threshold, and the first need_eq keys equal to it
  uint32_t gt_done = 0, eq_done = 0;
  for (uint32_t base = 0; base < total; base += kFinalThreads * kFinalPer) {
    if (!single) load_batch(base);
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int i = 0; i < kFinalPer; ++i) {
      const bool valid = e[i].y != 0xffffffffu;
      gt += valid && e[i].x > thr;
      eq += valid && e[i].x == thr;
    }
    uint32_t tot;
    const uint32_t ex = final_exclusive_scan(gt | (eq << 16), &tot, scan_lds);   // a batch holds at most 8192 entries: 14 bits each half
    uint32_t gt_before = gt_done + (ex & 0xffffu), eq_before = eq_done + (ex >> 16);
#pragma unroll
    for (int i = 0; i < kFinalPer; ++i) {
      if (e[i].y == 0xffffffffu) continue;
      const int t = (int)e[i].y;
      if (e[i].x > thr) {
        if (as_votes) atomicAdd(&acc[t], 1.0f);
        else {
          out[gt_before + min(eq_before, need_eq)] = t;
          if (FULL && a.sel_votes != nullptr) a.sel_votes[(size_t)b * a.k + gt_before + min(eq_before, need_eq)] = key_float(e[i].x);
        }
        ++gt_before;
      } else if (e[i].x == thr) {
        if (eq_before < need_eq) {
          if (as_votes) atomicAdd(&acc[t], 1.0f);
          else {
            out[gt_before + eq_before] = t;
            if (FULL && a.sel_votes != nullptr) a.sel_votes[(size_t)b * a.k + gt_before + eq_before] = key_float(e[i].x);
          }
        }
        ++eq_before;
      }
    }
    gt_done += tot & 0xffffu; eq_done += tot >> 16;
    __syncthreads();
  }
}

hipError_t launch_topk(const TopkArgs& args, int B, hipStream_t s) {
  TopkArgs a = args;
  // behind the table, in the list's memory: 2 of its 16 KiB a chunk and 4 KiB a sequence
  a.hist2 = reinterpret_cast<uint32_t*>(a.table + (size_t)B * a.nblk * 1024);
  dim3 grid(a.nblk, B);
  const bool short_path = a.list != nullptr && a.nblk <= kFinalMaxBlk;
  static_assert(kTopkOneWg == kFinalThreads * 8, "8 votes per thread");
  if (a.one_wg && a.max_seq_len <= kTopkOneWg) {
    // the whole sequence fits one workgroup's registers: one launch instead of two, three or (flat votes) four, whatever
    // the distribution.  4096 tokens, k 256: 4.6 + 5.1 -> 5.5 us (and no histogram in the vote kernel).  The line lies at
    // 8 votes per thread: a decode step of 8000 tokens 42 -> 37 us; with 16 votes per thread 16000 tokens took 45 us
    // instead of 43, and five sequences of them 72 instead of 68
    if (a.max_seq_len <= kFinalThreads * 4) hipLaunchKernelGGL((topk_final_kernel<4, FINAL_SHORT>), dim3(B), dim3(kFinalThreads), 0, s, a);
    else hipLaunchKernelGGL((topk_final_kernel<8, FINAL_SHORT>), dim3(B), dim3(kFinalThreads), 0, s, a);
    return hipGetLastError();
  }
  if (a.rep_hist == nullptr)
    hipLaunchKernelGGL(topk_hist0_kernel, dim3(a.nblk < 128 ? a.nblk : 128, B), dim3(256), 0, s, a);
  if (short_path) {
    hipLaunchKernelGGL(topk_compact_kernel, grid, dim3(256), 0, s, a);
    // the list holds about k entries plus the few that share the k-th key's bin: one batch in the usual case
    if (a.k <= 3072) hipLaunchKernelGGL((topk_final_kernel<4, FINAL_LIST>), dim3(B), dim3(kFinalThreads), 0, s, a);
    else hipLaunchKernelGGL((topk_final_kernel<8, FINAL_LIST>), dim3(B), dim3(kFinalThreads), 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(topk_hist1_kernel, grid, dim3(256), 0, s, a);
  if (a.nblk <= kTableChunks) {
    hipLaunchKernelGGL(topk_hist2_kernel<true>, grid, dim3(256), 0, s, a);
    hipLaunchKernelGGL(topk_emit_kernel<true>, grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(topk_hist2_kernel<false>, grid, dim3(256), 0, s, a);
    hipLaunchKernelGGL(topk_count_kernel, grid, dim3(256), 0, s, a);
    hipLaunchKernelGGL(topk_emit_kernel<false>, grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// the candidates of the compact selection: votes = upper bounds, rep_hist = the lower bounds' histogram
hipError_t launch_topk_compact(const TopkArgs& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(topk_compact_kernel, dim3(a.nblk, B), dim3(256), 0, s, a);
  return hipGetLastError();
}

// finishing workgroup over a list of exact votes (compact selection)
hipError_t launch_topk_final_full(const TopkArgs& a, int B, hipStream_t s) {
  // entries per thread: a list of up to 5/4 k sits in registers (the candidates are usually 1.03 to 1.2 k)
  const int per = (int)(((long)a.k * 5 / 4 + kFinalThreads - 1) / kFinalThreads);
  if (per <= 2) hipLaunchKernelGGL((topk_final_kernel<2, FINAL_FULL>), dim3(B), dim3(kFinalThreads), 0, s, a);
  else if (per <= 4) hipLaunchKernelGGL((topk_final_kernel<4, FINAL_FULL>), dim3(B), dim3(kFinalThreads), 0, s, a);
  else if (per <= 6) hipLaunchKernelGGL((topk_final_kernel<6, FINAL_FULL>), dim3(B), dim3(kFinalThreads), 0, s, a);
  else hipLaunchKernelGGL((topk_final_kernel<8, FINAL_FULL>), dim3(B), dim3(kFinalThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace ts
