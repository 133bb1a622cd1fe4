// Eq. 2 (selective sparse attention), decode form for batches (bf16): the gather as a stream.
//
// With hundreds of (sequence, KV head) pairs the step is a gather of 2 * k * H_kv * D * 2 bytes per sequence, and what
// counts is how many bytes are in flight.  A workgroup takes a long run of one pair's list; each of its four waves walks
// 32-key tiles of its own, without any barrier: K and V rows go from memory to the wave's part of the LDS directly
// (16 bytes per lane, whole rows), K is fetched again as soon as its scores are formed, V as soon as it has been
// multiplied, and the other seven waves of the CU (two workgroups of 64 KiB) keep the memory busy meanwhile.  A plain
// random gather of 256-byte pieces runs at 5.9 TB/s on this part.
// The products run on the matrix cores (the G query heads are columns of a 16-column operand, D / 32 + 3 * D / 16
// MFMAs per 16 and 32 keys): on the vector ALU they were 470 instructions per wave and 8 KiB, and the registers for them
// left one or two waves per SIMD.  The weights keep their 24 bits: each is the sum of three bf16 numbers, and V is
// multiplied with each of them.
// Measured (H 32/8, D 128, 2048 of each): 64 sequences 113 + 15 (merge) -> 90 us;
// H 28/4, 48 sequences, 4736 of each: 134 + 12 -> 80 + 5 us.
#include "ts_kernels.h"

namespace ts {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr float kStUnset = -3.40282347e38f;   // reference logit before the first key: no finite logit lies below it
constexpr float kStHead = 4.f;                // a raised reference lies this far above the largest logit so far ...
constexpr float kStRaise = 1.f;               // ... and is raised again when a lane's eight weights exceed this: no weight is above 1
constexpr float kStBig = 1048576.f;           // references beyond this: the logits are rounded before it is taken off them
constexpr float kLog2e = 1.44269504088896340736f;

// place of a row's 16-byte pieces in LDS: 16 rows x one piece (K fragments) and 8 rows x 2 pieces (V^T) each fall on
// all banks
template <int D> __device__ __forceinline__ int st_swz(int key) {
  return D == 128 ? (((key & 7) << 1) | ((key >> 3) & 1)) : ((((key >> 1) & 3) << 1) | ((key >> 3) & 1));
}

template <int D, int G>
__global__ __launch_bounds__(256, 2) void sparse_attn_stream_kernel(AttnArgs a) {
  constexpr int RB = D * 2;                   // bytes per row
  constexpr int PPR = RB / 16;                // 16-byte pieces per row
  constexpr int RPI = 64 / PPR;               // rows per wave load
  constexpr int NLD = kStreamTile / RPI;      // wave loads per tile and pool
  constexpr int KS = D / 32;                  // MFMAs per 16 keys, scores
  constexpr int DB = D / 16;                  // 16-row blocks of the transposed output
  constexpr int TILE_B = kStreamTile * RB;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // [wave][K tile, V tile], then uint32 slots [span]
  __shared__ float s_ml[4][16][2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kvh = blockIdx.x, split = blockIdx.y, b = blockIdx.z;
  const int H = a.H;
  // attended list = forced initial tokens [0, f_lo), the cnt selected tokens, forced recent tokens [f_hi, nb)
  const int nb = min(max(a.seq_lens[b], 0), a.max_seq_len);
  const int f_lo = min(a.n_init, nb), f_hi = max(f_lo, nb - a.n_local);
  const int cnt = nb > 0 ? min(max(a.count[b], 0), a.idx_stride) : 0;   // an empty sequence attends nothing, whatever count says
  const int total = f_lo + cnt + (nb - f_hi);
  const int j0 = split * a.span;
  const int nj = min(max(total - j0, 0), a.span);
  const size_t hb0 = (size_t)b * H + kvh * G;
  if (nj <= 0) {                              // nothing attended in this split
    if (a.nsplit > 1) {
      if (threadIdx.x < G) { float* ml = a.part_ml + ((hb0 + threadIdx.x) * a.nsplit + split) * 2; ml[0] = -INFINITY; ml[1] = 0.f; }
    } else {
      for (int i = threadIdx.x; i < G * D; i += 256) reinterpret_cast<uint16_t*>(a.out)[hb0 * D + i] = 0;
      if (threadIdx.x < G && a.lse != nullptr) a.lse[hb0 + threadIdx.x] = -INFINITY;
    }
    return;
  }
  uint32_t* slots = reinterpret_cast<uint32_t*>(smem + 4 * 2 * TILE_B);
  // the list of the run as pool rows; the tail of the last tile repeats the run's first token (weight 0)
  const int ntile = (nj + kStreamTile - 1) / kStreamTile;
  const int32_t* pages = a.page_indices + a.page_indptr[b];
  constexpr int UL = 8;                       // list entries of a thread in flight: ids, then pages, are two round trips for 2048 entries
  for (int i0 = threadIdx.x; i0 < ntile * kStreamTile; i0 += 256 * UL) {
    int t[UL];
    uint32_t page[UL];
#pragma unroll
    for (int u = 0; u < UL; ++u) {
      const int i = i0 + u * 256, jj = j0 + (i < nj ? i : 0);
      const int sel = a.idx[(size_t)b * a.idx_stride + min(max(jj - f_lo, 0), a.idx_stride - 1)];
      t[u] = jj < f_lo ? jj : jj < f_lo + cnt ? sel : f_hi + (jj - f_lo - cnt);
      t[u] = min(max(t[u], 0), nb - 1);       // a stale or corrupt index must not leave the page table
    }
#pragma unroll
    for (int u = 0; u < UL; ++u) page[u] = (uint32_t)pages[t[u] >> a.p_shift];
#pragma unroll
    for (int u = 0; u < UL; ++u)
      if (i0 + u * 256 < ntile * kStreamTile) slots[i0 + u * 256] = (page[u] << a.p_shift) + (uint32_t)(t[u] & (a.P - 1));
  }
  // query fragments (B operand): column = head (zero past G), k = 32 * ks + 8 * (lane / 16) .. + 8
  const int col = lane & 15, kgrp = lane >> 4;
  bf16x8_t qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (col < G) v = *reinterpret_cast<const uint4*>(a.q + (hb0 + col) * RB + ks * 64 + kgrp * 16);
    qf[ks] = __builtin_bit_cast(bf16x8_t, v);
  }
  const float sm = a.sm_scale;
  __builtin_amdgcn_s_waitcnt(0x0f70);         // vmcnt(0): from here on only the row loads are outstanding
  __syncthreads();

  uint8_t* kt = smem + wave * 2 * TILE_B;
  uint8_t* vt = kt + TILE_B;
  const uint32_t lds_k = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)kt;
  const int st_row = lane / PPR, st_pos = lane % PPR;
  uint64_t off[NLD];                          // of the rows of a tile in the pools, this lane's piece
  auto rows_of = [&](int tile) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int row = i * RPI + st_row;
      off[i] = ((uint64_t)slots[tile * kStreamTile + row] * (uint32_t)a.H_kv + (uint32_t)kvh) * RB + (uint32_t)((st_pos ^ st_swz<D>(row & 15)) * 16);
    }
  };
  // 1 KiB per load: the wave's lanes fill LDS from `dst` on.  In assembly, so that the compiler does not make every LDS
  // read wait for it; the waits stand below.  Non-temporal: the rows are read once (102 -> 89 us with 64 sequences).
  auto load_rows = [&](const uint8_t* pool, uint32_t dst) {
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" :: "s"(dst + i * 1024), "v"(pool + off[i]) : "memory", "m0");
  };
  float ref = kStUnset, lsum = 0.f;           // of head `col`: reference logit (the same in its four lanes), this lane's keys' sum
  bool big = false;                           // some head's reference is large (the same for the whole wave)
  f32x4_t o[DB];                              // O^T: row d = 16 * db + 4 * kgrp + r, column = head
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  const int vt_key = 4 * kgrp + (col >> 2), vt_c = (col & 3) >> 1, vt_b = (col & 1) * 8;   // V^T read: key, piece of the pair, half

  if (wave < ntile) { rows_of(wave); load_rows(a.k_pool, lds_k); load_rows(a.v_pool, lds_k + TILE_B); }
  for (int tile = wave; tile < ntile; tile += 4) {
    const bool more = tile + 4 < ntile;
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NLD) : "memory");            // this tile's K rows (its V rows follow them)
    // ---- scores: two blocks of 16 keys, element r is key 16 * kb + 4 * kgrp + r.  The products of each MFMA are added up on
    // their own: handed from one to the next the sums lose more than the vector form's (root mean square error of the
    // log-sum-exp, 1500 keys at four times 1 / sqrt(D): 5.8e-7 against 4.6e-7 of the vector form; this way 4.4e-7)
    f32x4_t part[KS][2], s[2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const uint4 av = *reinterpret_cast<const uint4*>(kt + (kb * 16 + col) * RB + (((ks * 4 + kgrp) ^ st_swz<D>(col)) * 16));
        part[ks][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av), qf[ks], (f32x4_t){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[kb][r] = part[0][kb][r] + part[1][kb][r];
        if (KS == 4) s[kb][r] += part[KS - 2][kb][r] + part[KS - 1][kb][r];
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                     // the K tile has been read
    if (more) { rows_of(tile + 4); load_rows(a.k_pool, lds_k); }
    // ---- weights against the reference: exp(logit - reference).  One fma forms the difference, which loses least; its
    // exact product differs from the rounded one that the reference came from by up to 2^-24 of the logit, though, and with
    // logits of 2^31 that alone would over- or underflow the exponential
    const int left = nj - tile * kStreamTile;                              // keys of this tile that exist
    float p[8];
    float sum;
    for (int tries = 0; tries < 2; ++tries) {
      sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = s[e >> 2][e & 3];
        p[e] = __builtin_amdgcn_exp2f((big ? x * sm - ref : fmaf(x, sm, -ref)) * kLog2e);
        if (16 * (e >> 2) + 4 * kgrp + (e & 3) >= left) p[e] = 0.f;
        sum += p[e];
      }
      if (__builtin_amdgcn_ballot_w64(!(sum <= kStRaise)) == 0) break;
      float m = ref;                                                       // first keys, or a logit far above the reference
#pragma unroll
      for (int e = 0; e < 8; ++e) m = fmaxf(m, s[e >> 2][e & 3] * sm + kStHead);   // (a repeated key past the end is a real one)
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      big = __builtin_amdgcn_ballot_w64(fabsf(m) > kStBig) != 0;
      const float f = __builtin_amdgcn_exp2f((ref - m) * kLog2e);          // 0 while the reference is unset
      lsum *= f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[db][r] *= f;
      ref = m;
    }
    lsum += sum;
    // each weight as three bf16 numbers whose sum is the weight; k-slot 8 * kgrp + e of the product is p[e]'s key.  The
    // parts are cut off, not rounded, and the lower two are kept above 2^-30 of the weight: all three have its sign and none
    // is zero beside it, so that an infinite V row comes out infinite (inf - inf and 0 * inf would make it NaN).
    uint32_t w[3][4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const float q0 = p[e] * 9.3132257e-10f, q1 = p[e + 1] * 9.3132257e-10f;
      float x0 = p[e], x1 = p[e + 1];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        w[c][e >> 1] = __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);   // the high halves
        if (c < 2) {
          x0 = fmaxf(x0 - bf16_lo(w[c][e >> 1]), q0);                      // the differences are exact
          x1 = fmaxf(x1 - bf16_hi(w[c][e >> 1]), q1);
        }
      }
    }
    // ---- O^T += V^T P^T
    if (more) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NLD) : "memory");  // this tile's V rows (the next K rows follow them)
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      uint2 v[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const uint8_t* vp = vt + (kb * 16 + vt_key) * RB + (((db * 2 + vt_c) ^ st_swz<D>(vt_key)) * 16) + vt_b;
        v[kb] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)vp));
      }
      const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, make_uint4(v[0].x, v[0].y, v[1].x, v[1].y));
#pragma unroll
      for (int c = 0; c < 3; ++c)
        o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8_t, make_uint4(w[c][0], w[c][1], w[c][2], w[c][3])), o[db], 0, 0, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                     // the V tile has been read
    if (more) load_rows(a.v_pool, lds_k + TILE_B);
  }

  // ---- the four waves meet: head `col`'s sums over its four lanes, then over the waves
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  __syncthreads();                                                         // every wave is done with its tiles
  float* so = reinterpret_cast<float*>(smem);                              // [wave][head][D + 4]
  if (col < G) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<float4*>(so + (wave * G + col) * (D + 4) + db * 16 + kgrp * 4) = make_float4(o[db][0], o[db][1], o[db][2], o[db][3]);
    if (kgrp == 0) { s_ml[wave][col][0] = ref; s_ml[wave][col][1] = lsum; }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < G * D; i += 256) {
    const int g = i / D, d = i % D;
    const float m = fmaxf(fmaxf(s_ml[0][g][0], s_ml[1][g][0]), fmaxf(s_ml[2][g][0], s_ml[3][g][0]));
    float x = 0.f, l = 0.f;
#pragma unroll
    for (int w4 = 0; w4 < 4; ++w4) {
      const float f = __builtin_amdgcn_exp2f((s_ml[w4][g][0] - m) * kLog2e);   // a wave without keys: 0
      x = fmaf(f, so[(w4 * G + g) * (D + 4) + d], x);
      l = fmaf(f, s_ml[w4][g][1], l);
    }
    if (a.nsplit > 1) {
      a.part_out[((hb0 + g) * a.nsplit + split) * D + d] = x;
      if (d == 0) { float* ml = a.part_ml + ((hb0 + g) * a.nsplit + split) * 2; ml[0] = m; ml[1] = l; }
    } else {
      reinterpret_cast<uint16_t*>(a.out)[(hb0 + g) * D + d] = (uint16_t)f32_to_bf16_bits(l > 0.f ? x / l : 0.f);
      if (d == 0 && a.lse != nullptr) a.lse[hb0 + g] = l > 0.f ? m + logf(l) : -INFINITY;
    }
  }
}

// Merges the splits of a row (few: long runs): out = sum_s e^{m_s - M} o_s / sum_s e^{m_s - M} l_s.  D / 4 lanes per row,
// 16 bytes of every split's partial each.
template <int D>
__global__ __launch_bounds__(256) void stream_merge_kernel(AttnArgs a, int nrow) {
  constexpr int LPR = D / 4;
  const int hb = (int)blockIdx.x * (256 / LPR) + (int)threadIdx.x / LPR, d = ((int)threadIdx.x % LPR) * 4;
  if (hb >= nrow) return;
  const int b = hb / a.H;
  const int nb = min(max(a.seq_lens[b], 0), a.max_seq_len);
  const int f_lo = min(a.n_init, nb), f_hi = max(f_lo, nb - a.n_local);
  const int total = f_lo + (nb > 0 ? min(max(a.count[b], 0), a.idx_stride) : 0) + (nb - f_hi);
  const int ns = min(a.nsplit, (total + a.span - 1) / a.span);   // splits that hold tokens
  const float* ml = a.part_ml + (size_t)hb * a.nsplit * 2;
  const float* po = a.part_out + (size_t)hb * a.nsplit * D + d;
  constexpr int US = 8;                       // splits whose partials are in flight together
  float M = -INFINITY, L = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < ns; s0 += US) {
    float2 v[US];
    float4 x[US];
#pragma unroll
    for (int u = 0; u < US; ++u) {
      const int s = min(s0 + u, ns - 1);
      v[u] = *reinterpret_cast<const float2*>(ml + 2 * s);
      x[u] = *reinterpret_cast<const float4*>(po + (size_t)s * D);
    }
    float m = M;
#pragma unroll
    for (int u = 0; u < US; ++u) m = fmaxf(m, v[u].x);
    if (m == -INFINITY) continue;             // nothing but empty splits so far
    const float f = expf(M - m);
    L *= f; o.x *= f; o.y *= f; o.z *= f; o.w *= f;
#pragma unroll
    for (int u = 0; u < US; ++u) {
      const float w = s0 + u < ns ? expf(v[u].x - m) : 0.f;
      L = fmaf(w, v[u].y, L);
      o.x = fmaf(w, x[u].x, o.x); o.y = fmaf(w, x[u].y, o.y); o.z = fmaf(w, x[u].z, o.z); o.w = fmaf(w, x[u].w, o.w);
    }
    M = m;
  }
  const bool any = L > 0.f;
  *reinterpret_cast<uint2*>(a.out + ((size_t)hb * D + d) * 2) =
      make_uint2(f32_to_bf16_bits(any ? o.x / L : 0.f) | (f32_to_bf16_bits(any ? o.y / L : 0.f) << 16),
                 f32_to_bf16_bits(any ? o.z / L : 0.f) | (f32_to_bf16_bits(any ? o.w / L : 0.f) << 16));
  if (a.lse != nullptr && d == 0) a.lse[hb] = any ? M + logf(L) : -INFINITY;
}

template <int D, int G>
static hipError_t stream_one(const AttnArgs& a, dim3 grid, hipStream_t s) {
  const size_t lds = (size_t)4 * 2 * kStreamTile * D * 2 + (size_t)a.span * sizeof(uint32_t);
  if (lds > 65536 - 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sparse_attn_stream_kernel<D, G>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((sparse_attn_stream_kernel<D, G>), grid, dim3(256), lds, s, a);
  return hipGetLastError();
}

static hipError_t stream_runs(int D, int G, const AttnArgs& a, int B, hipStream_t s) {
  if (a.span < kStreamTile || a.span % kStreamTile != 0 || a.span > kStreamMaxSpan) return hipErrorInvalidValue;
  const dim3 grid(a.H_kv, a.nsplit, B);
  switch (G) {
#define TS_CASE(g) case g: return D == 64 ? stream_one<64, g>(a, grid, s) : stream_one<128, g>(a, grid, s);
    TS_CASE(1) TS_CASE(2) TS_CASE(3) TS_CASE(4) TS_CASE(5) TS_CASE(6) TS_CASE(7) TS_CASE(8)
#undef TS_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_sparse_attn_stream(int D, int G, const AttnArgs& a, int B, hipStream_t s) {
  const hipError_t e = stream_runs(D, G, a, B, s);
  if (e != hipSuccess || a.nsplit == 1) return e;
  const int rows = B * a.H, rpw = 256 / (D / 4);
  if (D == 64) hipLaunchKernelGGL(stream_merge_kernel<64>, dim3((rows + rpw - 1) / rpw), dim3(256), 0, s, a, rows);
  else hipLaunchKernelGGL(stream_merge_kernel<128>, dim3((rows + rpw - 1) / rpw), dim3(256), 0, s, a, rows);
  return hipGetLastError();
}

}  // namespace ts
