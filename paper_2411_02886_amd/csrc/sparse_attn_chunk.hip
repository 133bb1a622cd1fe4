// Eq. 2 (selective sparse attention), chunk form: each of the C queries of a prefill chunk attends
// over the shared selected tokens plus the chunk's own tokens up to and including itself, in one
// joint softmax ([K_select, K_current] of Eq. 2 with a causal mask inside the chunk).
//
// The kernel here serves head size 64; head size 128 takes sparse_attn_chunk_wide.hip, whose four waves of 64 rows were 0.76 to
// 0.94 of this kernel's speed at head size 64 (12 shapes): with half the products per weight the vector ALU is the bound, and two
// waves a SIMD fill it better than one.  The merge of the splits serves both.
//
// Matrix-core flash attention over a gathered key list.  The G query heads x C queries of one KV head are rows that
// all meet the same keys.  A workgroup of eight waves owns 128 rows: four waves of 32 rows take the even 64-key tiles
// of its share of the list, four the odd ones, and the two halves meet in LDS at the end, so that half as many
// partials have to travel through memory.
//
// What bounds it: phases of a wave (scores, weights, output) that follow each other, and the LDS, where eight waves read every
// fragment for 32 rows only.  What was taken out of the loop:
//   * Scores are formed transposed (K as A operand, Q as B): a lane then holds 32 keys of ONE row, so the running
//     softmax is two registers per lane, and the weights, rounded to bf16, are the B operand of O^T += V^T P^T
//     as they stand -- which key sits at which k of the product is free as long as V^T is read the same way.
//   * V^T is read from the row-major V tile by the transposing LDS read (16 columns x 4 keys per 16 lanes).
//   * K and V rows go from memory to LDS directly, 16 bytes per lane, each lane fetching the piece that belongs at its
//     place: pieces are exchanged inside a row (piece ^ swz(key)) so that both reads are free of bank conflicts.
//   * No maximum over the scores: weights are formed against the row's reference exponent, 2^8 above the largest when it was
//     set; only if a weight comes out as 2 or more (or not a number) the reference is raised and the tile's weights are formed again.
//   * The weights' sums come from the matrix cores: v_dot2_f32_bf16 with a pair of ones runs on their multipliers (6 cycles
//     alone, 22 beside another wave's products).
//   * The key list is resolved in the loop, a step per tile ahead: token id, page id, rows; a lane resolves one key, and the
//     lanes that stage its row take it from there on the DPP network.
// (The last two: 1 to 4 % of a call, 12 shapes of 497 to 2687 selected keys: 2 x 512 queries of H 16/16 23.1 -> 22.2 us, 300 of
// H 32/8 20.0 -> 19.6.  A register limit for four waves a SIMD: 0.83 to 1.03 of that, with scratch.)
#include "ts_kernels.h"
#include <limits.h>
#include <type_traits>

namespace ts {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kCaRows = 128;     // rows per workgroup (four waves of 32)
constexpr int kCaGroups = 2;     // key groups per workgroup
constexpr int kCaTile = 64;      // keys per tile
constexpr float kCaUnset = -3.40282347e38f;   // reference exponent of a row that has seen no key: no finite logit lies below it
constexpr uint32_t kCaTwo = 0x40004000u;      // bits that only bf16 numbers of 2 and more have (and infinities and NaN): such a weight raises the reference ...
constexpr float kCaHead = 8.f;                // ... to this far above the largest exponent so far
constexpr float kCaBig = 1048576.f;  // references beyond this: the logits are rounded before it is taken off them

// place of a row's 16-byte pieces in LDS: 16 rows x one piece (K fragments) and 4 rows x 4 pieces (V^T) each
// fall on all banks
__device__ __forceinline__ int ca_swz(int key) { return (((key >> 1) & 1) << 2) | ((key >> 2) & 3); }

__global__ __launch_bounds__(512, 2) void chunk_attn_kernel(ChunkAttnArgs a) {
  constexpr int D = 64;
  constexpr int KS = D / 16;                     // k-steps of Q K^T
  constexpr int NBO = D / 32;                    // 32-row blocks of the transposed output
  constexpr int RBYTES = D * 2;
  constexpr int PPR = RBYTES / 16;               // 16-byte pieces per K/V row
  constexpr int KPI = 64 / PPR;                  // keys per wave load
  constexpr int NLD = 16 / KPI;                  // loads per wave, tile and pool: a wave stages 16 keys
  constexpr int TILE_B = kCaTile * RBYTES;
  // [buffer][key group][K tile, V tile]
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave >> 2, rg = wave & 3;       // key group, row group
  const int half = lane >> 5, col = lane & 31;
  // Workgroups that gather the same rows (sequence, KV head, split) sit on one XCD, next to each other in launch order,
  // so that its L2 fetches the rows once (workgroup L runs on XCD L % 8); the row blocks of a group are dealt to
  // a.xsplit XCDs where the groups alone would leave some of them idle.
  const int nrb = (a.C * a.G + kCaRows - 1) / kCaRows, rbs = (nrb + a.xsplit - 1) / a.xsplit;
  const int vg = ((int)(blockIdx.x >> 3) / rbs) * 8 + (int)(blockIdx.x & 7);
  const int rb = (vg % a.xsplit) * rbs + (int)(blockIdx.x >> 3) % rbs, group = vg / a.xsplit;
  if (rb >= nrb) return;
  const int split = group % a.nsplit, kvh = group / a.nsplit % a.H_kv, b = group / a.nsplit / a.H_kv;
  const int C = a.C, G = a.G, H = a.H;
  const int nrows = C * G;
  const int N = min(max(a.seq_lens[b], 0), a.max_seq_len);
  const int r0 = rb * kCaRows;
  if (N < C) {
    // a sequence shorter than the chunk holds no chunk (an idle slot of the batch): its rows are zero, and nothing is
    // read through its page table, which may be empty
    for (int i = threadIdx.x; i < kCaRows * D; i += 512) {
      const int row = r0 + i / D, d = i % D;
      if (row >= nrows) break;
      const size_t hb = ((size_t)b * C + row / G) * H + kvh * G + row % G;
      if (a.nsplit == 1) {
        reinterpret_cast<uint16_t*>(a.out)[hb * D + d] = 0;
        if (d == 0 && a.lse != nullptr) a.lse[hb] = -INFINITY;
      } else {
        a.part_o[(hb * a.nsplit + split) * D + d] = 0.f;
        if (d == 0) { float* pm = a.part_ml + (hb * a.nsplit + split) * 2; pm[0] = -INFINITY; pm[1] = 0.f; }
      }
    }
    return;
  }
  // key list: forced initial block, selected tokens, forced block before the chunk (seen by every query), then the
  // chunk's own tokens
  const int Nc = N - C;                                         // cached tokens before the chunk
  const int f_lo = min(a.n_init, Nc), f_hi = max(f_lo, Nc - a.n_local);
  const int csel = min(max(a.count[b], 0), a.idx_stride);
  const int cnt = f_lo + csel + (Nc - f_hi);
  const int c_last = min(C - 1, (r0 + kCaRows - 1) / G);       // last query of this row block
  const int nkeys = cnt + c_last + 1;                           // keys any row of the block may see
  const int ntile_all = (nkeys + kCaTile - 1) / kCaTile;
  // this workgroup's share of the key list (tiles [tile0, tile0 + ntile)); may be empty
  const int tps = (ntile_all + a.nsplit - 1) / a.nsplit;
  const int tile0 = min(split * tps, ntile_all);
  const int ntile = min(tps, ntile_all - tile0);
  const int niter = (ntile + kCaGroups - 1) / kCaGroups;
  const int32_t* sel = a.idx + (size_t)b * a.idx_stride;
  const int32_t* pages = a.page_indices + a.page_indptr[b];
  float c2 = a.sm_scale * 1.44269504088896340736f;
  if (c2 == 0.f) c2 = 1e-37f;                                   // the same weights (all 1), and a hidden key still gets 0
  const float hidden = c2 > 0.f ? -INFINITY : INFINITY;         // c2 * hidden = -inf

  // ---- query fragments (B operand of K Q^T): lane holds row = col, k = 16 * ks + 8 * half .. + 8
  const int row = r0 + rg * 32 + col;
  const int qc = row / G;                                       // query of this lane's row
  const int vis = min(qc, c_last);                              // last token of the chunk that it sees
  bf16x8_t qfrag[KS];
  {
    const bool valid = row < nrows;
    const int c = valid ? qc : 0, g = valid ? row % G : 0;
    const uint8_t* qp = a.q + ((((size_t)b * C + c) * H + (size_t)kvh * G + g) * D + 8 * half) * 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (valid) v = *reinterpret_cast<const uint4*>(qp + ks * 32);
      qfrag[ks] = __builtin_bit_cast(bf16x8_t, v);
    }
  }
  float ref = kCaUnset;                                         // the row's reference exponent
  // Sums of the rounded weights, by the matrix cores: rows 0 and 1 of the result are the sums of the weights' rows col and
  // 16 + col (col = lane % 16), the lanes of the operand that hold them picked out by ones
  f32x4_t lacc = {0.f, 0.f, 0.f, 0.f};
  bf16x8_t pick;
  {
    const uint32_t one = (lane & 15) == ((lane >> 4) & 1) ? 0x3f803f80u : 0u;
    pick = __builtin_bit_cast(bf16x8_t, make_uint4(one, one, one, one));
  }
  // The weights' exponents are one fma, c2 * score - reference.  Its exact product differs from the rounded one that the
  // reference came from by up to 2^-24 of the logit, and with logits of 2^31 that alone would over- or underflow the
  // exponential.  A wave that meets such a reference rounds the logits first from then on: `factor` is 1 and every tile takes
  // the way of the masked ones, where the scores are multiplied (0.5 to 1.1 of 60 us; a test of its own in the loop 0.7 to 1.2).
  float factor = c2;
  int plain_below = cnt - kCaTile + 1;                          // tiles that begin below this need no look at their scores
  f32x16_t oacc[NBO];                                           // O^T: d = 32 * nb + 8 * (e / 4) + 4 * half + e % 4
#pragma unroll
  for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[nb][e] = 0.f;

  // ---- staging: this wave's 16 keys of its group's tile, load i covering keys 16 * rg + i * KPI + lane / PPR.  A list
  // entry becomes a row in three steps, one iteration apart: token id (raw_*), page id (page_*), rows.  What an
  // iteration consumes was loaded in the one before and has been waited for at its top, so nothing waits behind the rows.
  // A lane looks one key up, the m-th (m = lane % 4) of those that the 16 lanes of its row stage; a load's lanes take its row from
  // there on the DPP network (the look-ups and addresses of every lane for itself were a third of the loop's vector instructions).
  const int st_key = lane / PPR, st_pos = lane % PPR;
  const int my_key = rg * 16 + ((lane & 2) >> 1) * KPI + (lane >> 4) * 2 + (lane & 1);
  int raw_id = 0, page_id = 0, page_off = 0;
  auto key_of = [&](int it) { return min((tile0 + it * kCaGroups + kg) * kCaTile + my_key, nkeys - 1); };   // past the end: the last key
  auto fetch_ids = [&](int it) { raw_id = sel[min(max(key_of(it) - f_lo, 0), a.idx_stride - 1)]; };
  auto token_of = [&](int it) -> int {
    const int j = key_of(it);
    int t = (j < f_lo) ? j : raw_id;
    t = (j < f_lo + csel) ? t : f_hi + (j - f_lo - csel);
    t = (j < cnt) ? t : Nc + (j - cnt);
    return min(max(t, 0), N - 1);                               // a stale or corrupt index must not leave the page table
  };
  auto fetch_pages = [&](int t) { page_id = pages[t >> a.p_shift]; page_off = t & (a.P - 1); };
  const int row_shift = 31 - __builtin_clz((uint32_t)(a.H_kv * RBYTES));   // H_kv is a power of two
  uint32_t piece[NLD];                                          // this lane's piece of load i's rows
#pragma unroll
  for (int i = 0; i < NLD; ++i) piece[i] = (uint32_t)kvh * RBYTES + (uint32_t)((st_pos ^ ca_swz(i * KPI + st_key)) * 16);   // the swizzle looks at the low four bits only
  // Memory to LDS, 16 bytes per lane: the wave's 64 lanes fill 1 KiB from the (uniform) LDS address.  Written in
  // assembly because the compiler, which cannot tell the two buffers apart, makes every later LDS read wait for the
  // builtin form; completion is awaited by the vmcnt(0) before the barrier at the top of the loop.
  auto load_rows = [&](int buf) {
    const uint32_t kt = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem +
                        (uint32_t)((buf * kCaGroups + kg) * 2 * TILE_B + rg * 16 * RBYTES);
    const uint32_t row = ((uint32_t)page_id << a.p_shift) + (uint32_t)page_off;
    const uint32_t lo = row << row_shift, hi = row >> (32 - row_shift);
    auto load = [&](auto i_c) __attribute__((always_inline)) {
      constexpr int I = decltype(i_c)::value;
      auto of = [&](uint32_t v) __attribute__((always_inline)) -> uint32_t {      // row_newbcast: lanes 2 I and 2 I + 1 of each 16
        const uint32_t v0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + 2 * I, 0xf, 0xf, true);
        const uint32_t v1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x151 + 2 * I, 0xf, 0xf, true);
        return (lane & 8) != 0 ? v1 : v0;
      };
      const uint64_t o = ((uint64_t)of(hi) << 32) | (of(lo) | piece[I]);
      const uint32_t dst = __builtin_amdgcn_readfirstlane(kt + I * KPI * RBYTES), dst_v = dst + TILE_B;
      const uint8_t *k_row = a.k_pool + o, *v_row = a.v_pool + o;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(dst), "v"(k_row) : "memory", "m0");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(dst_v), "v"(v_row) : "memory", "m0");
    };
    static_assert(NLD == 2, "the loads are written out");
    load(std::integral_constant<int, 0>{});
    load(std::integral_constant<int, 1>{});
  };

  if (niter > 0) {
    fetch_ids(0);
    fetch_pages(token_of(0));
    fetch_ids(1);
    load_rows(0);
    fetch_pages(token_of(1));
    fetch_ids(2);
  }
  const int ka_swz = ca_swz(col);                            // K fragment: key 32 * kb + col
  // V^T: 16 lanes read 4 keys x 16 columns; lane i of them reads key i / 4, columns 4 * (i % 4) ..
  const int vt_key = 4 * half + ((lane & 15) >> 2), vt_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  for (int it = 0; it < niter; ++it) {
    const int buf = it & 1;
    __builtin_amdgcn_s_waitcnt(0x0f70);                         // vmcnt(0): this wave's rows of the tile (and the ids behind them) are there
    __syncthreads();                                            // ... everybody's; and the other buffer has been read
    if (it + 1 < niter) {
      const int t = token_of(it + 2);
      load_rows(buf ^ 1);
      fetch_pages(t);
      fetch_ids(it + 3);
    }
    const int tile = tile0 + it * kCaGroups + kg;
    if (it * kCaGroups + kg >= ntile) continue;                 // the last round of the odd group may be empty
    const uint8_t* kt = smem + (size_t)((buf * kCaGroups + kg) * 2) * TILE_B;
    const uint8_t* vt = kt + TILE_B;
    // ---- S^T for 64 keys x 32 rows, two independent chains
    f32x16_t s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[kb][e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const uint4 av = *reinterpret_cast<const uint4*>(kt + (kb * 32 + col) * RBYTES + (((ks * 2 + half) ^ ka_swz) * 16));
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av), qfrag[ks], s[kb], 0, 0, 0);
      }
    // ---- weights against the reference; keys the row may not see get none
    const int j0 = tile * kCaTile;
    auto round_logits = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) s[kb][e] *= c2;
    };
    if (j0 >= plain_below) {                                    // the same for the whole wave
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int cq = j0 + kb * 32 + 8 * (e >> 2) + 4 * half + (e & 3) - cnt;   // >= 0: the chunk's token cq
          s[kb][e] = cq <= vis ? s[kb][e] : hidden;
        }
      if (__builtin_expect(plain_below == INT_MIN, 0)) round_logits();
    }
    uint32_t pk[2][8];
    for (int tries = 0; tries < 2; ++tries) {
      uint32_t any = 0u;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const bf16x2_t p = {(__bf16)__builtin_amdgcn_exp2f(fmaf(factor, s[kb][e], -ref)), (__bf16)__builtin_amdgcn_exp2f(fmaf(factor, s[kb][e + 1], -ref))};
          pk[kb][e >> 1] = __builtin_bit_cast(uint32_t, p);
          any |= pk[kb][e >> 1];
        }
      if (__builtin_amdgcn_ballot_w64((any & kCaTwo) != 0u) == 0) break;
      // first visible key of a row, or a logit far above the reference.  Straight-line code: a branch per lane here
      // makes the compiler copy the accumulators on the common path too.
      float m = ref;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) m = fmaxf(m, factor * s[kb][e] + kCaHead);
      m = fmaxf(m, __shfl_xor(m, 32));                          // both halves of a row raise its reference together
      const float f = __builtin_amdgcn_exp2f(ref - m);          // 1 where nothing changes, 0 while the reference is unset
      const float fo = __shfl(f, (lane & 15) + 16);
      lacc[0] *= f; lacc[1] *= fo;                              // lanes 0 to 15 hold them
#pragma unroll
      for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[nb][e] *= f;
      ref = m;
      if (__builtin_expect(plain_below != INT_MIN && __builtin_amdgcn_ballot_w64(fabsf(m) > kCaBig && m != kCaUnset) != 0, 0)) {
        factor = 1.f; plain_below = INT_MIN;
        round_logits();
      }
    }
    // ---- O^T += V^T P^T: k-step ks2 of a block takes keys 16 * ks2 + 4 * half + {0..3, 8..11}, the keys of s[8 * ks2 ..]
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) {
      const uint32_t (&pw)[8] = pk[k4 >> 1];
      const int o = 4 * (k4 & 1);
      const uint4 pb = make_uint4(pw[o], pw[o + 1], pw[o + 2], pw[o + 3]);
      lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick, __builtin_bit_cast(bf16x8_t, pb), lacc, 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < NBO; ++nb) {
        s16x4_t v[2];
#pragma unroll
        for (int h8 = 0; h8 < 2; ++h8) {
          const int key = k4 * 16 + h8 * 8 + vt_key, c = nb * 32 + vt_col;
          const uint8_t* p = vt + key * RBYTES + (((c >> 3) ^ ca_swz(key)) * 16) + (c & 7) * 2;
          v[h8] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)p);
        }
        const uint2 v0 = __builtin_bit_cast(uint2, v[0]), v1 = __builtin_bit_cast(uint2, v[1]);
        oacc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, make_uint4(v0.x, v0.y, v1.x, v1.y)),
                                                            __builtin_bit_cast(bf16x8_t, pb), oacc[nb], 0, 0, 0);
      }
    }
  }

  // ---- the two key groups meet: the odd group's rows through LDS
  const float sum_lo = __shfl(lacc[0], lane & 15), sum_hi = __shfl(lacc[1], lane & 15);
  const float lsum = (lane & 16) != 0 ? sum_hi : sum_lo;
  __syncthreads();
  float* xo = reinterpret_cast<float*>(smem) + (size_t)rg * (NBO * 16 + 2) * 64 + lane;   // [row group][register][lane]
  if (kg == 1) {
#pragma unroll
    for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) xo[(nb * 16 + e) * 64] = oacc[nb][e];
    xo[(NBO * 16) * 64] = ref; xo[(NBO * 16 + 1) * 64] = lsum;
  }
  __syncthreads();
  if (kg == 1 || row >= nrows) return;
  const float ref1 = xo[(NBO * 16) * 64], l1 = xo[(NBO * 16 + 1) * 64];
  const float m = fmaxf(ref, ref1);
  const float w0 = __builtin_amdgcn_exp2f(ref - m), w1 = __builtin_amdgcn_exp2f(ref1 - m);
  const float l = fmaf(w1, l1, w0 * lsum);
  const size_t hb = ((size_t)b * C + qc) * H + kvh * G + row % G;
  auto merged = [&](int nb, int q4) -> float4 {                 // O[row][d .. d + 3], d = 32 * nb + 8 * q4 + 4 * half
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = fmaf(w1, xo[(nb * 16 + q4 * 4 + e) * 64], w0 * oacc[nb][q4 * 4 + e]);
    return make_float4(o[0], o[1], o[2], o[3]);
  };
  if (a.nsplit == 1) {
    const float inv = l > 0.f ? 1.f / l : 0.f;
    uint8_t* po = a.out + (hb * D + half * 4) * 2;
#pragma unroll
    for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float4 o = merged(nb, q4);
        *reinterpret_cast<uint2*>(po + (nb * 32 + q4 * 8) * 2) =
            make_uint2(f32_to_bf16_bits(o.x * inv) | (f32_to_bf16_bits(o.y * inv) << 16), f32_to_bf16_bits(o.z * inv) | (f32_to_bf16_bits(o.w * inv) << 16));
      }
    if (half == 0 && a.lse != nullptr) a.lse[hb] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * 0.69314718055994530942f : -INFINITY;
  } else {
    float* po = a.part_o + (hb * a.nsplit + split) * D + half * 4;
#pragma unroll
    for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) *reinterpret_cast<float4*>(po + nb * 32 + q4 * 8) = merged(nb, q4);
    if (half == 0) {
      float* pm = a.part_ml + (hb * a.nsplit + split) * 2;
      pm[0] = l > 0.f ? m : -INFINITY; pm[1] = l;
    }
  }
}

// Merges the key-list splits of one row: with M = max_s ref_s (base-2 exponents),
// out = sum_s 2^(ref_s - M) O_s / sum_s 2^(ref_s - M) l_s.  D / 4 lanes per row, 16 bytes of every split's partial each.
template <int D>
__global__ __launch_bounds__(256) void chunk_attn_merge_kernel(ChunkAttnArgs a, int nrow) {
  constexpr int LPR = D / 4;
  const int hb = blockIdx.x * (256 / LPR) + (int)threadIdx.x / LPR, d = ((int)threadIdx.x % LPR) * 4;
  if (hb >= nrow) return;
  const float* pm = a.part_ml + (size_t)hb * a.nsplit * 2;
  float M = -INFINITY;
  for (int s = 0; s < a.nsplit; ++s) M = fmaxf(M, pm[2 * s]);
  float L = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < a.nsplit; ++s) {
    const float r = pm[2 * s];
    const float w = (r == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(r - M);
    const float4 x = *reinterpret_cast<const float4*>(a.part_o + ((size_t)hb * a.nsplit + s) * D + d);
    L = fmaf(w, pm[2 * s + 1], L);
    o.x = fmaf(w, x.x, o.x); o.y = fmaf(w, x.y, o.y); o.z = fmaf(w, x.z, o.z); o.w = fmaf(w, x.w, o.w);
  }
  const bool any = L > 0.f;
  const uint2 w = make_uint2(f32_to_bf16_bits(any ? o.x / L : 0.f) | (f32_to_bf16_bits(any ? o.y / L : 0.f) << 16),
                             f32_to_bf16_bits(any ? o.z / L : 0.f) | (f32_to_bf16_bits(any ? o.w / L : 0.f) << 16));
  *reinterpret_cast<uint2*>(a.out + ((size_t)hb * D + d) * 2) = w;
  if (a.lse != nullptr && d == 0) a.lse[hb] = any ? (M + __builtin_amdgcn_logf(L)) * 0.69314718055994530942f : -INFINITY;
}

hipError_t launch_sparse_attn_chunk(const ChunkAttnArgs& args, int B, hipStream_t s) {
  ChunkAttnArgs a = args;
  const int nrb = (a.C * a.G + kCaRows - 1) / kCaRows;                 // both kernels own 128 rows a workgroup
  const int groups = B * a.H_kv * a.nsplit;                            // times xsplit: a multiple of 8
  a.xsplit = groups % 8 == 0 ? 1 : groups % 4 == 0 ? 2 : groups % 2 == 0 ? 4 : 8;
  const int rbs = (nrb + a.xsplit - 1) / a.xsplit;
  const unsigned grid = (unsigned)(groups * a.xsplit * rbs);
  if (a.D == 128) {
    const hipError_t e = launch_chunk_attn_wide(a, grid, s);
    if (e != hipSuccess) return e;
  } else {
    const size_t lds = (size_t)2 * kCaGroups * 2 * kCaTile * 64 * 2;   // 64 KiB: two workgroups per CU
    hipLaunchKernelGGL(chunk_attn_kernel, dim3(grid), dim3(512), lds, s, a);
  }
  if (a.nsplit > 1) {
    const int rows = B * a.C * a.H, rpw = 256 / (a.D / 4);
    if (a.D == 128) hipLaunchKernelGGL(chunk_attn_merge_kernel<128>, dim3((rows + rpw - 1) / rpw), dim3(256), 0, s, a, rows);
    else hipLaunchKernelGGL(chunk_attn_merge_kernel<64>, dim3((rows + rpw - 1) / rpw), dim3(256), 0, s, a, rows);
  }
  return hipGetLastError();
}

}  // namespace ts
