// Eq. 2, chunk form, head size 128 (sparse_attn_chunk.hip has the kernel for head size 64, the merge of the splits, and how the
// scores and weights are laid out).
//
// What bounded the eight-wave form of that file here: its waves of 32 rows read every K and V fragment for 32 rows only, 256 KiB of LDS a
// pair of 64-key tiles beside the 64 KiB that arrive, and their phases (scores, weights, output) follow each other.  Here a workgroup
// of four waves, one per SIMD, owns the same 128 rows: two of them 64 rows each on the even 64-key tiles of its share, two on the
// odd ones.  A fragment serves 64 rows, and in one piece of straight-line code a wave forms the weights of one block of 32
// keys on the vector ALU while the matrix cores form the scores of the next and add the output of the last one.
//   * A wave issues in order, so the vector instructions are shared out behind every single product: behind two products
//     in a row they wait for the first to leave the matrix cores.  (Two products and fma, fma, exp, exp, cvt: 68 to 75
//     cycles, the products alone 64; every vector instruction beyond four a product costs 5.)
//   * The weights' sums come from the matrix cores too: v_dot2_f32_bf16 with a pair of ones runs on their multipliers (6
//     cycles alone, 22 beside them).
//   * No sum in the loop means that the reference is raised by a look at the bits of the packed weights.
//   * A list entry becomes a row on the way (token id, page id, place, a tile apart); it passes through LDS, fetched like
//     the rows, because a register's load would be waited for together with all rows behind it.
//   * Tiles that every row sees in full have a loop of their own without masks.
// Measured, 512 queries of H 32/8, 4096 selected + 512 own keys: 58.9 -> 51.3 us a call (launch, list, start, end and merge are 20 of them
// in both); 3 x 777 queries of H 28/4, 1666 + 640 + 777 keys 184 -> 148; 3 x 300 of H 40/8 85 -> 68; with 64 to 512 keys the
// same to 1.1 times as fast (35 shapes, 0.98 at the worst).  Of a wave's cycles the matrix
// core is busy 40 %, the vector ALU 43 %; a tile of 64 keys takes a wave 3900 cycles, 2180 of them products.  Tried on the way: the eight waves' two
// key groups taking turns, one at the products, one at the weights, 51.8 us; reads further ahead no faster; four-key look-ups
// by ds_bpermute 1.5 us slower.
#include "ts_kernels.h"
#include <limits.h>
#include <type_traits>

namespace ts {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kCwThreads = 256;  // four waves: two groups of 64 rows x two key groups
constexpr int kCwRows = 128;     // rows per workgroup
constexpr int kCwGroups = 2;     // key groups per workgroup
constexpr int kCwTile = 64;      // keys per tile
constexpr float kCwUnset = -3.40282347e38f;   // reference exponent of a row that has seen no key: no finite logit lies below it
constexpr uint32_t kCwTwo = 0x40004000u;      // bits that only bf16 numbers of 2 and more have (and infinities and NaN): such a weight raises the reference ...
constexpr float kCwHead = 8.f;                // ... to this far above the largest exponent so far
constexpr float kCwBig = 1048576.f;           // references beyond this: the logits are rounded before it is taken off them

// place of a row's 16-byte pieces in LDS: 16 rows x one piece (K fragments) and 4 rows x 4 pieces (V^T) each
// fall on all banks
__device__ __forceinline__ int cw_swz(int key) { return ((key & 3) << 2) | ((key >> 2) & 3); }

__global__ __launch_bounds__(kCwThreads, 1) void chunk_attn_wide_kernel(ChunkAttnArgs a) {
  constexpr int D = 128;
  constexpr int KS = D / 16;                     // k-steps of Q K^T
  constexpr int NBO = D / 32;                    // 32-row blocks of the transposed output
  constexpr int RBYTES = D * 2;
  constexpr int PPR = RBYTES / 16;               // 16-byte pieces per K/V row
  constexpr int KPI = 64 / PPR;                  // keys per wave load
  constexpr int WK = kCwTile / 2;                // keys of a tile that a wave stages
  constexpr int NLD = WK / KPI;                  // loads per wave, tile and pool
  static_assert(NLD == 8, "the loads are written out below");
  constexpr int TILE_B = kCwTile * RBYTES;
  // [buffer][key group][K tile, V tile]
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave >> 1, rg = wave & 1;       // key group, row group
  const int half = lane >> 5, col = lane & 31;
  // Workgroups that gather the same rows (sequence, KV head, split) sit on one XCD, next to each other in launch order,
  // so that its L2 fetches the rows once (workgroup L runs on XCD L % 8); the row blocks of a group are dealt to
  // a.xsplit XCDs where the groups alone would leave some of them idle.
  const int nrb = (a.C * a.G + kCwRows - 1) / kCwRows, rbs = (nrb + a.xsplit - 1) / a.xsplit;
  const int vg = ((int)(blockIdx.x >> 3) / rbs) * 8 + (int)(blockIdx.x & 7);
  const int rb = (vg % a.xsplit) * rbs + (int)(blockIdx.x >> 3) % rbs, group = vg / a.xsplit;
  if (rb >= nrb) return;
  const int split = group % a.nsplit, kvh = group / a.nsplit % a.H_kv, b = group / a.nsplit / a.H_kv;
  const int C = a.C, G = a.G, H = a.H;
  const int nrows = C * G;
  const int N = min(max(a.seq_lens[b], 0), a.max_seq_len);
  const int r0 = rb * kCwRows;
  if (N < C) {
    // a sequence shorter than the chunk holds no chunk (an idle slot of the batch): its rows are zero, and nothing is
    // read through its page table, which may be empty
    for (int i = threadIdx.x; i < kCwRows * D; i += kCwThreads) {
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
  const int c_last = min(C - 1, (r0 + kCwRows - 1) / G);       // last query of this row block
  const int nkeys = cnt + c_last + 1;                           // keys any row of the block may see
  const int ntile_all = (nkeys + kCwTile - 1) / kCwTile;
  // this workgroup's share of the key list (tiles [tile0, tile0 + ntile)); may be empty
  const int tps = (ntile_all + a.nsplit - 1) / a.nsplit;
  const int tile0 = min(split * tps, ntile_all);
  const int ntile = min(tps, ntile_all - tile0);
  const int niter = (ntile + kCwGroups - 1) / kCwGroups;
  const int32_t* sel = a.idx + (size_t)b * a.idx_stride;
  const int32_t* pages = a.page_indices + a.page_indptr[b];
  float c2 = a.sm_scale * 1.44269504088896340736f;
  if (c2 == 0.f) c2 = 1e-37f;                                   // the same weights (all 1), and a hidden key still gets 0
  const float hidden = c2 > 0.f ? -INFINITY : INFINITY;         // c2 * hidden = -inf

  // ---- query fragments (B operand of K Q^T): of the wave's two blocks of 32 rows, lane holds row = col, k = 16 * ks + 8 * half .. + 8
  int row[2], vis[2];                                           // vis: last token of the chunk that the row sees
  bf16x8_t qfrag[2][KS];
#pragma unroll
  for (int rb2 = 0; rb2 < 2; ++rb2) {
    row[rb2] = r0 + rg * 64 + rb2 * 32 + col;
    vis[rb2] = min(row[rb2] / G, c_last);
    const bool valid = row[rb2] < nrows;
    const int c = valid ? row[rb2] / G : 0, g = valid ? row[rb2] % G : 0;
    const uint8_t* qp = a.q + ((((size_t)b * C + c) * H + (size_t)kvh * G + g) * D + 8 * half) * 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (valid) v = *reinterpret_cast<const uint4*>(qp + ks * 32);
      qfrag[rb2][ks] = __builtin_bit_cast(bf16x8_t, v);
    }
  }
  float ref[2] = {kCwUnset, kCwUnset};                          // the rows' reference exponents
  // Sums of the rounded weights, by the matrix cores: rows 0 and 1 of the result are the sums of the weights' rows col and
  // 16 + col (col = lane % 16), the lanes of the operand that hold them picked out by ones.  (v_dot2_f32_bf16 with a pair
  // of ones runs on the matrix cores' multipliers: 6 cycles alone, 22 beside MFMAs.)
  f32x4_t lacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  bf16x8_t pick;
  {
    const uint32_t one = (lane & 15) == ((lane >> 4) & 1) ? 0x3f803f80u : 0u;
    pick = __builtin_bit_cast(bf16x8_t, make_uint4(one, one, one, one));
  }
  // The weights' exponents are one fma, c2 * score - reference.  Its exact product differs from the rounded one that the
  // reference came from by up to 2^-24 of the logit, and with logits of 2^31 that alone would over- or underflow the
  // exponential.  A wave that meets such a reference rounds the logits first from then on: `factor` is 1, and the loop without masks
  // ends after the second block of its pair; every later block takes the way of the masked ones, where the scores are multiplied.
  float factor = c2;
  int plain_below = cnt - kCwTile + 1;                          // tiles that begin below this need no look at their scores
  f32x16_t oacc[2][NBO];                                        // O^T: d = 32 * nb + 8 * (e / 4) + 4 * half + e % 4
#pragma unroll
  for (int rb2 = 0; rb2 < 2; ++rb2)
#pragma unroll
    for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[rb2][nb][e] = 0.f;

  // ---- staging: this wave's 32 keys of its group's tile, load i covering keys 32 * rg + i * KPI + lane / PPR.  An entry of the
  // list becomes a row of the pool in three steps a tile apart (token id, page id, row), and what a step consumes was
  // loaded in the one before and has been waited for.  A lane looks one key up, the m-th (m = lane % 8) of those that the 16
  // lanes of its row stage; a load's lanes take its row from there on the DPP network.
  const int st_key = lane / PPR, st_pos = lane % PPR;
  const int my_key = rg * WK + (lane & 7) * KPI + st_key;
  auto key_of = [&](int it) { return min((tile0 + it * kCwGroups + kg) * kCwTile + my_key, nkeys - 1); };   // past the end: the last key
  auto id_of = [&](int it) -> const int32_t* { return sel + min(max(key_of(it) - f_lo, 0), a.idx_stride - 1); };
  auto token_of = [&](int it, int id) -> int {
    const int j = key_of(it);
    int t = (j < f_lo) ? j : id;
    t = (j < f_lo + csel) ? t : f_hi + (j - f_lo - csel);
    t = (j < cnt) ? t : Nc + (j - cnt);
    return min(max(t, 0), N - 1);                               // a stale or corrupt index must not leave the page table
  };
  struct Place { uint32_t lo, hi; };                            // of a row in the pools
  const int row_shift = 31 - __builtin_clz((uint32_t)(a.H_kv * RBYTES));   // H_kv is a power of two
  auto row_of = [&](int token, int page) -> Place {
    const uint32_t row = ((uint32_t)page << a.p_shift) + (uint32_t)(token & (a.P - 1));
    return Place{row << row_shift, row >> (32 - row_shift)};
  };
  uint32_t piece[4];                                            // this lane's piece of load i's rows: i % 4 decides
#pragma unroll
  for (int i = 0; i < 4; ++i) piece[i] = (uint32_t)kvh * RBYTES + (uint32_t)((st_pos ^ cw_swz(i * KPI + st_key)) * 16);   // the swizzle looks at the low four bits only
  // Memory to LDS, 16 bytes per lane: the wave's 64 lanes fill 1 KiB from the (uniform) LDS address.  Written in
  // assembly because the compiler, which cannot tell the buffers apart, makes every later LDS read wait for the
  // builtin form; completion is awaited by the vmcnt(0) before a tile's barrier.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem + (uint32_t)(rg * WK * RBYTES);
  auto load_row = [&](const uint8_t* pool, Place rows, int tile_slot, auto i_c) __attribute__((always_inline)) {
    constexpr int I = decltype(i_c)::value;
    // row_newbcast: lane I of each 16
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rows.lo, 0x150 + I, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rows.hi, 0x150 + I, 0xf, 0xf, true);
    const uint64_t off = ((uint64_t)hi << 32) | (lo | piece[I & 3]);
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(tile_slot * TILE_B + I * KPI * RBYTES));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(dst), "v"(pool + off) : "m0");
  };
  auto k_slot = [&](int buf) { return (buf * kCwGroups + kg) * 2; };   // tile slots of the LDS: [buffer][group][K, V]

  typedef const __attribute__((address_space(3))) bf16x8_t lds_bf16x8;
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  // K fragment ks of key block kb: row 32 * kb + col, piece (2 * ks + half) ^ swz(col) -- ks flips bits of the address only
  const uint32_t ka0 = lds_base + (uint32_t)(col * RBYTES + ((half ^ cw_swz(col)) * 16));
  // V^T: 16 lanes read 4 keys x 16 columns; lane i of them reads key i / 4, columns 4 * (i % 4) ..; the output block nb and
  // the upper eight keys of a k-step flip bits of the piece
  const int vt_key = 4 * half + ((lane & 15) >> 2), vt_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const uint32_t va0 = lds_base + (uint32_t)(vt_key * RBYTES + (((vt_col >> 3) ^ cw_swz(vt_key)) * 16) + (vt_col & 7) * 2);
  // An entry on its way to a row passes through LDS (two places per lane behind the tiles), fetched like the rows: the
  // compiler would wait for a register's load with a count that knows nothing of the rows in flight.
  const uint32_t look = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)(4 * kCwGroups * TILE_B + wave * 512));
  auto fetch_look = [&](const int32_t* p, int place) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(look + place * 256), "v"(p) : "m0");
  };
  auto read_look = [&](int place) -> int { return *(const volatile __attribute__((address_space(3))) int*)(look + (uint32_t)(place * 256 + lane * 4)); };
  Place rows_k = {}, rows_v = {};                               // rows of the K tile and of the V tile that are requested next
  int token = 0;                                                // of the tile after that K tile
  // K tile `next` - 1 has been requested: rows of tile `next`, page ids of the one after, token ids of the one after that
  auto look_up = [&](int next) __attribute__((always_inline)) {
    const int page = read_look(0), id = read_look(1);
    rows_v = rows_k;
    rows_k = row_of(token, page);
    token = token_of(next + 1, id);
    fetch_look(pages + (token >> a.p_shift), 0);
    fetch_look(id_of(next + 2), 1);
  };

  // ---- The list is worked on in blocks of 32 keys, two to a tile.  While the vector ALU forms the weights of block j, the
  // matrix cores form the scores of block j + 1 and add the output of block j - 1: one piece of straight-line code.
  f32x16_t s[2][2];                                             // [block parity][row block] S^T: key 8 * (e / 4) + 4 * half + e % 4
  uint32_t pk[2][2][8];                                         // the weights, rounded to bf16
  auto round_logits = [&](f32x16_t (&x)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int rb2 = 0; rb2 < 2; ++rb2)
#pragma unroll
      for (int e = 0; e < 16; ++e) x[rb2][e] *= c2;
  };
  constexpr int AHEAD = 3;
  bf16x8_t carry[AHEAD];
  auto body = [&](auto half_c, int it, auto with_scores, auto with_output, auto with_loads, auto masked) __attribute__((always_inline)) {
    constexpr int CUR = decltype(half_c)::value, NXT = 1 - CUR; // this block is half CUR of tile `it`
    constexpr bool SC = decltype(with_scores)::value, OUT = decltype(with_output)::value, LD = decltype(with_loads)::value;
    f32x16_t (&x)[2] = s[CUR];
    // keys the row may not see get no weight
    const int lt = it * kCwGroups + kg;                         // tile of this workgroup's share; the last round of the odd group may be empty
    const int j0 = (tile0 + lt) * kCwTile;
    if (decltype(masked)::value && (j0 >= plain_below || lt >= ntile)) {   // the same for the whole wave
#pragma unroll
      for (int rb2 = 0; rb2 < 2; ++rb2) {
        const int see = lt < ntile ? vis[rb2] : INT_MIN;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int cq = j0 + CUR * 32 + 8 * (e >> 2) + 4 * half + (e & 3) - cnt;   // >= 0: the chunk's token cq
          x[rb2][e] = cq <= see ? x[rb2][e] : hidden;
        }
      }
      if (__builtin_expect(plain_below == INT_MIN, 0)) round_logits(x);
    }
    const uint32_t kt = ka0 + (uint32_t)(k_slot((it + CUR) & 1) * TILE_B + NXT * 32 * RBYTES);
    const uint32_t vt = va0 + (uint32_t)((k_slot((it + CUR + 1) & 1) + 1) * TILE_B + NXT * 32 * RBYTES);
    constexpr int NS = KS + 2 * NBO, T0 = SC ? 0 : KS, T1 = OUT ? NS : KS; // steps: scores, then output; two MFMAs each
    constexpr bool CIN = CUR == 0 && OUT;                       // this block's first fragments were read at the end of the one before
    bf16x8_t frag[NS];                                          // of step t: K rows of the next block (t < KS), V^T of the last one
    auto fetch = [&](int t) __attribute__((always_inline)) {
      if (t < KS) { frag[t] = *(lds_bf16x8*)(kt ^ (uint32_t)(t * 32)); return; }
      const int k2 = (t - KS) / NBO, nb = (t - KS) % NBO;       // k-step k2 takes keys 16 * k2 + 4 * half + {0..3, 8..11}, the keys of x[8 * k2 ..]
      s16x4_t v[2];
#pragma unroll
      for (int h8 = 0; h8 < 2; ++h8)
        v[h8] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((vt ^ (uint32_t)(nb * 64 + h8 * 32)) + (uint32_t)((k2 * 16 + h8 * 8) * RBYTES)));
      const uint2 v0 = __builtin_bit_cast(uint2, v[0]), v1 = __builtin_bit_cast(uint2, v[1]);
      frag[t] = __builtin_bit_cast(bf16x8_t, make_uint4(v0.x, v0.y, v1.x, v1.y));
    };
    auto weights_of = [&](int rb2, int k2) __attribute__((always_inline)) -> bf16x8_t {
      const uint32_t (&pw)[8] = pk[NXT][rb2];
      return __builtin_bit_cast(bf16x8_t, make_uint4(pw[4 * k2], pw[4 * k2 + 1], pw[4 * k2 + 2], pw[4 * k2 + 3]));
    };
    uint32_t any = 0u;
    float y[16][2], w[16][2];
    // pair i of the 16 pairs of weights, in three stages a step apart: none of a step's instructions waits for another of them
    auto exponent = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2; ++u) y[i][u] = fmaf(factor, x[i >> 3][2 * (i & 7) + u], -ref[i >> 3]);
    };
    auto power = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2; ++u) w[i][u] = __builtin_amdgcn_exp2f(y[i][u]);
    };
    auto pack = [&](int i) __attribute__((always_inline)) {
      const bf16x2_t p = {(__bf16)w[i][0], (__bf16)w[i][1]};
      pk[CUR][i >> 3][i & 7] = __builtin_bit_cast(uint32_t, p);
      any |= pk[CUR][i >> 3][i & 7];
    };
#pragma unroll
    for (int t = T0; t < T1 && t < T0 + AHEAD; ++t) { if (CIN) frag[t] = carry[t - T0]; else fetch(t); }
    // A step: a fragment read AHEAD steps before its use, a row load, two products, a pair of weights.  Kept in this order, the
    // vector instructions shared out behind every single product: a wave issues in order, and what stands behind two
    // products in a row waits for the first to leave the matrix cores.
    auto product = [&](int t, int rb2) __attribute__((always_inline)) {
      if (t < T0 || t >= T1) return;
      if (t < KS) s[NXT][rb2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[t], qfrag[rb2][t < KS ? t : 0], t == 0 ? (f32x16_t){} : s[NXT][rb2], 0, 0, 0);
      else oacc[rb2][(t - KS) % NBO] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[t], weights_of(rb2, (t - KS) / NBO), oacc[rb2][(t - KS) % NBO], 0, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      product(t, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (t >= T0 && t + AHEAD < T1) fetch(t + AHEAD);
      if (CUR == 1 && SC && t + AHEAD >= NS)                    // of K tile it + 1, second half
        carry[t + AHEAD - NS] = *(lds_bf16x8*)((ka0 + (uint32_t)(k_slot((it + 1) & 1) * TILE_B + 32 * RBYTES)) ^ (uint32_t)((t + AHEAD - NS) * 32));
#pragma unroll
      for (int i = t * 16 / NS; i < (t + 1) * 16 / NS; ++i) { if (i > 1) pack(i - 2); exponent(i); }
      __builtin_amdgcn_sched_barrier(0);
      product(t, 1);
      __builtin_amdgcn_sched_barrier(0);
      if (LD && t < NLD) {                                      // rows of K tile it + 2 and V tile it + 1
        switch (t) {
#define TS_ROW(I) case I: load_row(a.k_pool, rows_k, k_slot(it & 1), std::integral_constant<int, I>{}); \
                          load_row(a.v_pool, rows_v, k_slot((it + 1) & 1) + 1, std::integral_constant<int, I>{}); break;
          TS_ROW(0) TS_ROW(1) TS_ROW(2) TS_ROW(3) TS_ROW(4) TS_ROW(5) TS_ROW(6) TS_ROW(7)
#undef TS_ROW
        }
      }
      if (LD && t == NLD) look_up(it + 3);
#pragma unroll
      for (int i = t * 16 / NS; i < (t + 1) * 16 / NS; ++i) if (i > 0) power(i - 1);
      if (OUT && t < 4) lacc[t >> 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick, weights_of(t >> 1, t & 1), lacc[t >> 1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    power(15); pack(14); pack(15);
    if (__builtin_amdgcn_ballot_w64((any & kCwTwo) != 0u) != 0) {
      // first visible key of a row, or a logit far above the reference.  Straight-line code: a branch per lane here
      // makes the compiler copy the accumulators on the common path too.
#pragma unroll
      for (int rb2 = 0; rb2 < 2; ++rb2) {
        float m = ref[rb2];
#pragma unroll
        for (int e = 0; e < 16; ++e) m = fmaxf(m, factor * x[rb2][e] + kCwHead);
        // the first block: the second one's scores are there too, and a reference from all keys of the tile leaves more rows
        // with a largest weight that is a power of two, exact in bf16 (error of `out` against 64 bits, 256 to 2048 keys: 1 to
        // 2 % more without)
        if (CUR == 0 && !OUT) {
          const int see = lt < ntile ? vis[rb2] : INT_MIN;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int cq = j0 + 32 + 8 * (e >> 2) + 4 * half + (e & 3) - cnt;
            m = fmaxf(m, factor * (cq <= see ? s[NXT][rb2][e] : hidden) + kCwHead);
          }
        }
        m = fmaxf(m, __shfl_xor(m, 32));                        // both halves of a row raise its reference together
        const float f = __builtin_amdgcn_exp2f(ref[rb2] - m);   // 1 where nothing changes, 0 while the reference is unset
        const float fo = __shfl(f, (lane & 15) + 16);
        lacc[rb2][0] *= f; lacc[rb2][1] *= fo;                  // lanes 0 to 15 hold them
#pragma unroll
        for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[rb2][nb][e] *= f;
        ref[rb2] = m;
      }
      const bool big = (fabsf(ref[0]) > kCwBig && ref[0] != kCwUnset) || (fabsf(ref[1]) > kCwBig && ref[1] != kCwUnset);
      if (__builtin_expect(plain_below != INT_MIN && __builtin_amdgcn_ballot_w64(big) != 0, 0)) {
        factor = 1.f; plain_below = INT_MIN;
        round_logits(x);
        // the loop without masks takes one more block as it is, whose scores are there already; a masked block rounds its own
        if (CUR == 1 && SC && !decltype(masked)::value) round_logits(s[NXT]);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) { exponent(i); power(i); pack(i); }
    }
  };
  // Buffers: the barrier between the blocks of tile `it` says that K tile it + 1 and V tile `it` have arrived and that K tile
  // `it` and V tile it - 1 have been read, whose places K tile it + 2 and V tile it + 1 then take.
  auto tile_barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;
  if (niter > 0) {
    // four dependent round trips: lengths, ids of four tiles, pages of three, rows
    int ids[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) ids[n] = *id_of(n);
    const int tok0 = token_of(0, ids[0]), tok1 = token_of(1, ids[1]), tok2 = token_of(2, ids[2]);
    const int pg0 = pages[tok0 >> a.p_shift], pg1 = pages[tok1 >> a.p_shift], pg2 = pages[tok2 >> a.p_shift];
    token = token_of(3, ids[3]);
    fetch_look(pages + (token >> a.p_shift), 0);
    fetch_look(id_of(4), 1);
    const Place rows0 = row_of(tok0, pg0);
    rows_v = row_of(tok1, pg1); rows_k = row_of(tok2, pg2);
#define TS_ROW(I) load_row(a.k_pool, rows0, k_slot(0), std::integral_constant<int, I>{});
    TS_ROW(0) TS_ROW(1) TS_ROW(2) TS_ROW(3) TS_ROW(4) TS_ROW(5) TS_ROW(6) TS_ROW(7)
#undef TS_ROW
#define TS_ROW(I) load_row(a.k_pool, rows_v, k_slot(1), std::integral_constant<int, I>{});
    TS_ROW(0) TS_ROW(1) TS_ROW(2) TS_ROW(3) TS_ROW(4) TS_ROW(5) TS_ROW(6) TS_ROW(7)
#undef TS_ROW
#define TS_ROW(I) load_row(a.v_pool, rows0, k_slot(0) + 1, std::integral_constant<int, I>{});
    TS_ROW(0) TS_ROW(1) TS_ROW(2) TS_ROW(3) TS_ROW(4) TS_ROW(5) TS_ROW(6) TS_ROW(7)
#undef TS_ROW
    tile_barrier();
    // tile -1's second half, without weights: the scores of the first block
#pragma unroll
    for (int rb2 = 0; rb2 < 2; ++rb2)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[0][rb2][e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t av = *(lds_bf16x8*)((ka0 + (uint32_t)(k_slot(0) * TILE_B)) ^ (uint32_t)(ks * 32));
#pragma unroll
      for (int rb2 = 0; rb2 < 2; ++rb2) s[0][rb2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, qfrag[rb2][ks], s[0][rb2], 0, 0, 0);
    }
    body(B0{}, 0, Yes{}, No{}, No{}, Yes{});
    int it = 0;
    // rounds of tiles that every row sees in full; the reference of large logits ends them early
    const int full = (ntile + 1 - kg) / kCwGroups;              // of this key group's tiles
    for (; it + 1 < niter; ++it) {
      if (it + 1 >= full || (tile0 + (it + 1) * kCwGroups + kg) * kCwTile >= plain_below) break;
      tile_barrier();
      body(B1{}, it, Yes{}, Yes{}, Yes{}, No{});
      body(B0{}, it + 1, Yes{}, Yes{}, No{}, No{});
    }
    for (; it + 1 < niter; ++it) {
      tile_barrier();
      body(B1{}, it, Yes{}, Yes{}, Yes{}, Yes{});
      body(B0{}, it + 1, Yes{}, Yes{}, No{}, Yes{});
    }
    tile_barrier();
    body(B1{}, niter - 1, No{}, Yes{}, No{}, Yes{});
    // the output of the last block
    const uint32_t vt = va0 + (uint32_t)((k_slot((niter - 1) & 1) + 1) * TILE_B + 32 * RBYTES);
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
      for (int rb2 = 0; rb2 < 2; ++rb2) {
        const uint32_t (&pw)[8] = pk[1][rb2];
        const bf16x8_t w = __builtin_bit_cast(bf16x8_t, make_uint4(pw[4 * k2], pw[4 * k2 + 1], pw[4 * k2 + 2], pw[4 * k2 + 3]));
        lacc[rb2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick, w, lacc[rb2], 0, 0, 0);
#pragma unroll
        for (int nb = 0; nb < NBO; ++nb) {
          s16x4_t v[2];
#pragma unroll
          for (int h8 = 0; h8 < 2; ++h8)
            v[h8] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((vt ^ (uint32_t)(nb * 64 + h8 * 32)) + (uint32_t)((k2 * 16 + h8 * 8) * RBYTES)));
          const uint2 v0 = __builtin_bit_cast(uint2, v[0]), v1 = __builtin_bit_cast(uint2, v[1]);
          oacc[rb2][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, make_uint4(v0.x, v0.y, v1.x, v1.y)), w, oacc[rb2][nb], 0, 0, 0);
        }
      }
  }

  // ---- the two key groups meet through LDS: the even one finishes the waves' first 32 rows, the odd one the second
  constexpr int XR = NBO * 16 + 2;
  float* xo = reinterpret_cast<float*>(smem) + lane;            // [row group][key group][register][lane]: what that key group finishes
  auto exchange = [&](auto mine_c) __attribute__((always_inline)) {
    constexpr int M = decltype(mine_c)::value;                  // this wave's key group, and the row block that it finishes
    float* give = xo + (size_t)(rg * 2 + 1 - M) * XR * 64;
    const float* take = xo + (size_t)(rg * 2 + M) * XR * 64;
    float lsum[2];
#pragma unroll
    for (int rb2 = 0; rb2 < 2; ++rb2) {
      const float lo = __shfl(lacc[rb2][0], lane & 15), hi = __shfl(lacc[rb2][1], lane & 15);
      lsum[rb2] = (lane & 16) != 0 ? hi : lo;
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NBO; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) give[(nb * 16 + e) * 64] = oacc[1 - M][nb][e];
    give[(NBO * 16) * 64] = ref[1 - M]; give[(NBO * 16 + 1) * 64] = lsum[1 - M];
    __syncthreads();
    if (row[M] >= nrows) return;
    const float ref1 = take[(NBO * 16) * 64], l1 = take[(NBO * 16 + 1) * 64];
    const float m = fmaxf(ref[M], ref1);
    const float w0 = __builtin_amdgcn_exp2f(ref[M] - m), w1 = __builtin_amdgcn_exp2f(ref1 - m);
    const float l = fmaf(w1, l1, w0 * lsum[M]);
    const size_t hb = ((size_t)b * C + row[M] / G) * H + kvh * G + row[M] % G;
    auto merged = [&](int nb, int q4) -> float4 {               // O[row][d .. d + 3], d = 32 * nb + 8 * q4 + 4 * half
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(w1, take[(nb * 16 + q4 * 4 + e) * 64], w0 * oacc[M][nb][q4 * 4 + e]);
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
  };
  if (kg == 0) exchange(B0{});
  else exchange(B1{});
}

hipError_t launch_chunk_attn_wide(const ChunkAttnArgs& a, unsigned grid, hipStream_t s) {
  const size_t lds = (size_t)4 * kCwGroups * kCwTile * 128 * 2 + kCwThreads * 8;      // 130 KiB: one workgroup per CU
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&chunk_attn_wide_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chunk_attn_wide_kernel, dim3(grid), dim3(kCwThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace ts
