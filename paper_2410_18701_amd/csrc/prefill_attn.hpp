// Causal attention of the queries prefilled inside the batch, for a step
// without prefill/decode separation: a new query's prompt of p tokens sits at
// input positions T - p .. T - 1 of its row (q [batch][T][n_q_heads][D],
// k_new / v_new [batch][T][n_kv_heads][D]); prompt position i attends over
// prompt positions 0 .. i -- the rest of its row is masked -- and every prompt
// position's key and value is appended to the cache as column L + T - p + i.
// The other rows of the step are decoded by the work-item kernels.
//
// Work: one workgroup per (tile of prompt positions, query head); the tiles
// of the prefilled queries are numbered consecutively, a query's longest
// tiles (the last positions, which see the most keys) first.  Keys and values
// come straight from k_new / v_new (the prompt is read by every tile of a
// head, through the caches).  The appends to the cache run in workgroups of
// their own, one per (tile, kv-head), after all the attention workgroups in
// the grid of prefill_fa_kernel (bf16, on the matrix cores): short ones, they
// fill the end of the launch instead of lengthening every attention
// workgroup by a load and a store of its tile; in prefill_f32_kernel (fp32)
// the first query head of each kv-head appends its tile.
#pragma once

#include "common.hpp"
#include "decode_attn.hpp"
#include "decode_attn_mfma.hpp"   // bf16x8, f32x4, as_bf16x8

namespace baton {

constexpr int kMaxPrefill = 64;   // == BATON_MAX_PREFILL

struct PrefillArgs {
  uint32_t* k;              // the layer's ring rows [batch][n_kv_heads][cap][D] (appended to)
  uint32_t* v;
  const uint32_t* q;        // [batch][T][n_q_heads][D]
  const uint32_t* knew;     // [batch][T][n_kv_heads][D]
  const uint32_t* vnew;
  uint32_t* out;            // [batch][T][n_q_heads][D]
  int64_t cap, base, L;
  int32_t T, batch, n_kv_heads, n_ins;
  int32_t n_tiles;          // tiles over all prefilled queries (per query head)
  int32_t unit_heads;       // query heads that read the same keys (G), or 1
  int32_t xcd_map;          // 1: keep each unit's workgroups on one XCD (units % 8 == 0)
  int32_t n_attn;           // attention workgroups (n_tiles x query heads); the matrix-core
                            // kernel's grid then has n_tiles x n_kv_heads append workgroups
  float qscale;             // scale * log2(e)
  int32_t slot[kMaxPrefill];
  int32_t plen[kMaxPrefill];
  int32_t tile_end[kMaxPrefill];   // inclusive prefix of tiles over the prefilled queries
};

// The work of this workgroup: query head hq, prefilled query ins, tile.  The
// grid is one-dimensional over n_tiles x query heads, tile-major: all query
// heads of one tile are dealt before the next tile, and the tiles run from
// the longest (a query's last positions, which see the most keys; the queries
// are ordered by prompt length, longest first) to the shortest, so that the
// workgroups that start last are short.  Workgroups are dealt to the XCDs
// round-robin by index, and each XCD has its own L2; with xcd_map the heads
// are numbered so that all workgroups reading one kv-head's keys (a unit: its
// G query heads) run on the same XCD.
__device__ __forceinline__ void prefill_work(const PrefillArgs& a, int& hq, int32_t& ins,
                                             int32_t& tile) {
  const int32_t nq = a.n_attn / a.n_tiles;   // query heads
  const int32_t g = blockIdx.x / nq, j = blockIdx.x % nq;
  if (a.xcd_map) {
    const int32_t xcd = j % 8, k = j / 8;
    const int32_t u = xcd + 8 * (k / a.unit_heads);
    hq = u * a.unit_heads + k % a.unit_heads;
  } else {
    hq = j;
  }
  ins = 0;
  while (ins < a.n_ins - 1 && g >= a.tile_end[ins]) ++ins;
  tile = a.tile_end[ins] - 1 - g;   // the query's tiles, counted from its last one
}

// Appends prompt positions [t0, t0 + n) of kv-head h (threads tid of nthr).
template <int VPT>
__device__ __forceinline__ void prefill_append(const PrefillArgs& a, int b, int h, int32_t p,
                                               int64_t row0, int32_t t0, int32_t n, int tid, int nthr) {
  const int64_t ring_row = (int64_t)b * a.n_kv_heads + h;   // within the layer's rows
  u32x4* rk = reinterpret_cast<u32x4*>(a.k) + ring_row * a.cap * VPT;
  u32x4* rv = reinterpret_cast<u32x4*>(a.v) + ring_row * a.cap * VPT;
  const u32x4* kin = reinterpret_cast<const u32x4*>(a.knew);
  const u32x4* vin = reinterpret_cast<const u32x4*>(a.vnew);
  const int64_t c0 = a.base + a.L + a.T - p;   // < 2 * cap: base < cap, L + T <= cap
  for (int idx = tid; idx < n * VPT; idx += nthr) {
    const int32_t t = t0 + idx / VPT;
    const int e = idx % VPT;
    int64_t col = c0 + t;
    col = col >= a.cap ? col - a.cap : col;
    const int64_t src = ((row0 + t) * a.n_kv_heads + h) * VPT + e;
    rk[col * VPT + e] = kin[src];
    rv[col * VPT + e] = vin[src];
  }
}

// fp32, on the fp32 matrix operation (v_mfma_f32_16x16x4_f32: fp32 products
// and sums).  A workgroup of four
// waves takes 16 positions of one query head; wave w takes every fourth
// block of 16 keys from block w on, and the waves' softmax states merge through
// LDS at the end.  What bounds it is, for short prompts, the chain of blocks a
// wave walks -- hence the split of the keys over the waves instead of the
// positions, and no barrier on the way -- and for long ones the loads of K in
// the operand's layout (16 rows of 64 bytes, a quarter of the L1's rate).  The
// registers are capped for four workgroups a CU at head_dim 64 (123 used) and two
// at 128 (236): the compiler then gives the operations' results to the vector ALUs
// directly, where without a cap it took 164 and 284, accumulators among them, that
// every addition had to read back.  (32 positions per workgroup, which halve the
// loads per operation but run one or two workgroups a CU, take 1.05 to 2.0 times
// as long at every size measured: 3 to 19,456 workgroups, prompts of 20 to 4,096.)
//  * QK^T: A = 16 key rows, B = 16 positions.  The contraction's order is free,
//    so step (i, e) takes element e of the 16-byte vectors at 16 i + 4 (l / 16):
//    both operands are loaded 16 bytes per lane.  Lane l, register r holds the
//    score of key 4 (l / 16) + r for position l % 16.
//  * PV, transposed: O^T = V^T P^T.  Step r takes keys 4 (l / 16) + r, so B is
//    the lane's own weight r; A = V^T of those keys, where tile (h, e) covers
//    the columns 64 h + 4 c + e, c < 16: the V rows are loaded whole, 16 bytes
//    per lane.  Lane l holds columns 64 h + 16 (l / 16) + 4 r + e of position
//    l % 16: its outputs are 16-byte vectors over e.
// us per layer, one prompt, 8 query heads over 4 kv-heads, head_dim 64, against a
// kernel that walked the keys one at a time on the vector ALUs: 40 tokens 14.4 ->
// 6.4, 300 81 -> 10.5, 1024 276 -> 27; 32 heads of 128: 300 tokens 93 -> 24.6, 1024
// 550 -> 127 (68 TFLOP/s of the matrix operation's 157).
template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2)))
prefill_f32_kernel(const PrefillArgs a) {
  constexpr int VPT = D / 4, DI = D / 16, DH = D / 64, NW = 4;
  __shared__ __attribute__((aligned(16))) f32x4 so[NW][DH * 4][kWave];
  __shared__ float sm[NW][16], sl[NW][16];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, g4 = lane / 16, c16 = lane % 16;
  int hq;
  int32_t ins, tile;
  prefill_work(a, hq, ins, tile);
  const int nkv = a.n_kv_heads, nq = a.n_attn / a.n_tiles, group = nq / nkv, h = hq / group;
  const int b = a.slot[ins];
  const int32_t p = a.plen[ins];
  const int32_t i0 = tile * 16;
  const int64_t row0 = (int64_t)b * a.T + (a.T - p);
  const u32x4* kin = reinterpret_cast<const u32x4*>(a.knew);
  const u32x4* vin = reinterpret_cast<const u32x4*>(a.vnew);

  // The positions as B operands, pre-scaled; positions past the prompt: zeros.
  const int32_t qi = i0 + c16;
  f32x4 qf[DI];
#pragma unroll
  for (int i = 0; i < DI; ++i) {
    const u32x4 x = qi < p ? reinterpret_cast<const u32x4*>(a.q)[((row0 + qi) * nq + hq) * VPT + 4 * i + g4]
                           : u32x4{0, 0, 0, 0};
    qf[i] = __builtin_bit_cast(f32x4, x) * a.qscale;
  }
  float m = -INFINITY, l = 0.f;
  f32x4 o[DH][4];
#pragma unroll
  for (int hh = 0; hh < DH; ++hh)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[hh][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The prompt's keys and values of head h as raw buffers; a token past the
  // prompt gets an offset beyond the range, which loads zeros.
  const uint32_t tok_bytes = (uint32_t)nkv * VPT * 16;
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(kin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(vin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  auto load = [](__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  };
  f32x4 kf[DI], vf[4][DH];
  auto load_k = [&](int32_t kb) {
    const int32_t t = kb + c16;
    const uint32_t off = t < p ? (uint32_t)t * tok_bytes + 16u * g4 : 0x80000000u;
#pragma unroll
    for (int i = 0; i < DI; ++i) kf[i] = load(rk, off + 64u * i);
  };
  auto load_v = [&](int32_t kb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t t = kb + 4 * g4 + r;
      const uint32_t off = t < p ? (uint32_t)t * tok_bytes + 16u * c16 : 0x80000000u;
#pragma unroll
      for (int hh = 0; hh < DH; ++hh) vf[r][hh] = load(rv, off + 256u * hh);
    }
  };
  const int32_t last = min(i0 + 16, p) - 1;   // the last position, and the last key it sees
  int32_t kb = 16 * w;
  if (kb <= last) {
    load_k(kb);
    load_v(kb);
  }
  for (; kb <= last; kb += 16 * NW) {               // wave-uniform
    // Every matrix operation starts from zero, four products, and the 4 DI of
    // them are added as a tree: a score's rounding error is that of a lane's own
    // sum of four products and a tree over the lanes (2-norm against float64 where
    // scores dominate, of that: chains of four operations 1.04 to 1.24, of two 1.00
    // to 1.10, this 0.97 to 1.03).  Eight operations at a time, with the additions of
    // the eight before placed between them, in the operations' shadow; left alone
    // the compiler issues all of them first and spills.
    constexpr int NE = DI / 2;                      // eights of a score's operations
    f32x4 pr[2][8], part[NE];
#pragma unroll
    for (int x = 0; x <= NE; ++x) {
      if (x < NE) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int i = 2 * x + j / 4;
          pr[x % 2][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][j % 4], qf[i][j % 4], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
      }
      if (x > 0) {
        f32x4(&q)[8] = pr[(x - 1) % 2];
        f32x4& t = part[x - 1];
        t = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
        asm volatile("" : "+v"(t));                 // added here, not where the loads of the next keys end the block
      }
      if (x > 0 && x < NE) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a matrix operation
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // and four vector ones
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int n = NE / 2; n > 0; n /= 2)
#pragma unroll
      for (int e = 0; e < n; ++e) part[e] += part[e + n];
    f32x4 s = part[0];
    const bool more = kb + 16 * NW <= last;
    if (more) load_k(kb + 16 * NW);
    if (kb + 15 > i0) {                             // some position does not see the whole block
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = kb + 4 * g4 + r <= qi ? s[r] : -INFINITY;
    }
    const float mx = max_over_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
    const float mn = fmaxf(m, mx);
    const float ref = mn == -INFINITY ? 0.f : mn;
    const float alpha = exp2f(m - ref);             // m = -inf before the first visible key: 0
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = exp2f(s[r] - ref);
      sum += s[r];
    }
    l = l * alpha + sum;                            // this lane's keys
    m = mn;
#pragma unroll
    for (int hh = 0; hh < DH; ++hh)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[hh][e] *= alpha;
    // A weight of 0 does not hide a value that is not finite: where a position
    // may not see the whole block and some value of it is inf or NaN (rare),
    // each position adds its visible keys' values one by one.
    bool odd = false;
    if (kb + 15 > i0) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int hh = 0; hh < DH; ++hh)
#pragma unroll
          for (int e = 0; e < 4; ++e) odd = odd || (__float_as_uint(vf[r][hh][e]) & 0x7F800000u) == 0x7F800000u;
    }
    if (__ballot(odd)) {
      for (int j = 0; j < 16 && kb + j <= last; ++j) {
        // key j's weight for position c16: register j % 4 of lane group j / 4
        const float wj = __shfl(j % 4 == 0 ? s[0] : j % 4 == 1 ? s[1] : j % 4 == 2 ? s[2] : s[3],
                                16 * (j / 4) + c16, kWave);
        if (kb + j > qi) continue;
#pragma unroll
        for (int hh = 0; hh < DH; ++hh)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const f32x4 v = load(rv, (uint32_t)(kb + j) * tok_bytes + 256u * hh + 64u * g4 + 16u * r);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[hh][e][r] = fmaf(wj, v[e], o[hh][e][r]);
          }
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int hh = 0; hh < DH; ++hh)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            o[hh][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][hh][e], s[r], o[hh][e], 0, 0, 0);
    }
    if (more) load_v(kb + 16 * NW);
  }
  // Merge the waves: wave w finishes the vectors of register r = w.
  const float lw = sum_over_groups(l);
  if (g4 == 0) {
    sm[w][c16] = m;
    sl[w][c16] = lw;
  }
#pragma unroll
  for (int hh = 0; hh < DH; ++hh)
#pragma unroll
    for (int r = 0; r < 4; ++r) so[w][hh * 4 + r][lane] = f32x4{o[hh][0][r], o[hh][1][r], o[hh][2][r], o[hh][3][r]};
  __syncthreads();
  float mm = -INFINITY;
#pragma unroll
  for (int q = 0; q < NW; ++q) mm = fmaxf(mm, sm[q][c16]);
  float lt = 0.f, f[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const float mq = sm[q][c16];
    f[q] = mq == -INFINITY ? 0.f : exp2f(mq - mm);
    lt += f[q] * sl[q][c16];
  }
  const float inv = 1.f / lt;
  if (qi < p) {
#pragma unroll
    for (int hh = 0; hh < DH; ++hh) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NW; ++q) v += so[q][hh * 4 + w][lane] * f[q];
      v *= inv;
      reinterpret_cast<f32x4*>(a.out)[((row0 + qi) * nq + hq) * VPT + 16 * hh + 4 * g4 + w] = v;
    }
  }
  if (hq % group == 0) prefill_append<VPT>(a, b, h, p, row0, i0, min(16, p - i0), tid, 256);
}

// bf16 on the matrix cores, flash-attention style: a workgroup of 4*S waves
// takes kPrefillTile prompt positions of one query head; four waves cover the
// positions (16 each) and S such quartets split the keys, each
// walking every S-th tile of KT keys (S tiles staged in LDS per iteration, K
// and V both as rows, 16-byte stores), and the quartets' softmax states merge
// through LDS at the end -- S shortens the longest causal tile's chain of
// iterations.  What bounds it is that chain: the waves wait 0.58 of their cycles
// (prompts of 64 to 1,018 tokens, 32 heads of 128) on the staging and its barriers
// and on the dependent products and softmax steps.  Each 32-key block costs a
// wave 16 KB of LDS reads (prefill_fa32_kernel halves that per position).
//  * QK^T: A = 16 key rows (lane l: key l % 16 of the half tile), B = 16 of
//    the wave's positions; the score of key 4*(l/16) + r (first 16 keys) and
//    16 + 4*(l/16) + r (next 16) for position l % 16 lands in
//    lane l, register r.
//  * PV, transposed: O^T = V^T P^T.  B = P^T with k = 8*(l/16) + e standing
//    for key 4*(l/16) + e (e < 4) and 16 + 4*(l/16) + e - 4 (e >= 4) -- the
//    lane's own scores, in place; A = V^T in that key order, read with the
//    LDS transpose load (ds_read_b64_tr_b16): within a group of 16 lanes,
//    lane i receives element i % 4 of the 8-byte block addressed by lane
//    i / 4 + 4e, for e = 0..3; lane m of group g addresses key 4g + m / 4 at
//    columns 16*dt + 4*(m % 4), so lane i gets V[4g + e][16*dt + i].  Lane l
//    then holds output columns 16*dt + 4*(l/16) + r of position l % 16 of the
//    group: a position's rescale and normalisation stay in its own lanes, and
//    the max over the four lane groups uses the gfx950 row swaps.
//  * The weights' sum: one more operation per block, a column of ones as A
//    and the same P^T as B, so the sum is of the bf16 weights P·V was made
//    of, and every lane of a position holds it whole.
// Rows are padded to 8 dwords past a multiple of 32, so that the 16 rows of a
// transpose load spread over all banks.
// Keys per LDS tile and key stream: 32 (a stage of 64 keys with two streams,
// 37 KB of LDS) rather than 64, so that a workgroup's first stage arrives
// sooner and its last stage carries fewer keys past its diagonal.
#ifndef BATON_PREFILL_KT
#define BATON_PREFILL_KT 32
#endif
#ifndef BATON_PREFILL_LAZY
#define BATON_PREFILL_LAZY 8.0f
#endif
constexpr float kPrefillLazy = BATON_PREFILL_LAZY;
constexpr int kPrefillTile = 64;             // positions per workgroup

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ s16x4 lds_read_tr16(const uint8_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(__attribute__((address_space(3))) void*)(p));
}

// Registers capped so that two workgroups share a CU (128 per lane, four waves
// per SIMD).
template <int D, int G, int S>
__global__ void __launch_bounds__(256 * S) __attribute__((amdgpu_waves_per_eu(4)))
prefill_fa_kernel(const PrefillArgs a) {
  constexpr int VPT = D / 8, KK = D / 32, DT = D / 16;
  constexpr int TILE = kPrefillTile;
  constexpr int KT = BATON_PREFILL_KT;       // keys per LDS tile and key stream
  constexpr int ROW = D * 2 + 32;            // bytes per staged key / value row
  constexpr int NT = 256 * S;                // threads
  constexpr int NLD = KT * VPT / 256;        // 16-byte vectors per thread per stage, K and V each
  constexpr int REC = DT * 4 + 2;            // floats of a lane's softmax state
  static_assert((ROW / 4) % 32 == 8, "row padding");
  static_assert(S == 1 || (S - 1) * 4 * kWave * REC * 4 <= 2 * S * KT * ROW, "merge area");
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * S * KT * ROW];
  uint8_t* const ldsK = lds;
  uint8_t* const ldsV = lds + S * KT * ROW;
  const int tid = threadIdx.x;
  if ((int32_t)blockIdx.x >= a.n_attn) {
    // An append workgroup (after every attention workgroup in the grid, so
    // that these short ones fill the end of the launch): tile g of the
    // prefilled queries' prompt positions, kv-head h, into the ring.
    const int32_t j = (int32_t)blockIdx.x - a.n_attn;
    const int32_t g = j / a.n_kv_heads, h = j % a.n_kv_heads;
    int32_t ins = 0;
    while (ins < a.n_ins - 1 && g >= a.tile_end[ins]) ++ins;
    const int32_t tile = a.tile_end[ins] - 1 - g, p = a.plen[ins], b = a.slot[ins];
    const int64_t row0 = (int64_t)b * a.T + (a.T - p);
    prefill_append<VPT>(a, b, h, p, row0, tile * TILE, min(TILE, p - tile * TILE), tid, NT);
    return;
  }
  const int wave = tid / kWave, lane = tid % kWave;
  const int ks = wave / 4;                             // key stream of this wave
  const int g4 = lane / 16, c16 = lane % 16;
  int hq;
  int32_t ins, tile;
  prefill_work(a, hq, ins, tile);
  const int h = hq / G;
  const int b = a.slot[ins];
  const int32_t p = a.plen[ins];
  const int32_t wg0 = tile * TILE;                     // first position of the workgroup
  const int32_t i0 = wg0 + (wave % 4) * 16;       // first position of this wave
  const int64_t row0 = (int64_t)b * a.T + (a.T - p);
  const int nkv = a.n_kv_heads, nq = nkv * G;
  const u32x4* qin = reinterpret_cast<const u32x4*>(a.q);
  const u32x4* kin = reinterpret_cast<const u32x4*>(a.knew);
  const u32x4* vin = reinterpret_cast<const u32x4*>(a.vnew);
  const u32x4 zero = {0, 0, 0, 0};

  // A negative scale's sign is folded into q (negating a bf16 value is
  // exact), so that the softmax below always works with a positive factor:
  // the largest scaled score is then the scale times the largest score.
  const float qscale = fabsf(a.qscale);
  const uint32_t qsw = a.qscale < 0.f ? 0x80008000u : 0u;
  const u32x4 qsign = {qsw, qsw, qsw, qsw};
  const int32_t qi = i0 + c16;
  bf16x8 qb[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qb[kk] = as_bf16x8(qi < p ? qin[((row0 + qi) * nq + hq) * VPT + kk * 4 + g4] ^ qsign : zero);

  // Running max, the sums of the weights (ol: the weights as rounded to bf16
  // for the matrix operation, times a column of ones, on the matrix cores --
  // the output is then normalized by exactly the weights it was made of) and
  // the output accumulators.
  float m = -INFINITY;
  f32x4 ol = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[DT];
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int32_t wg_last = min(wg0 + TILE - 1, p - 1);
  // the wave's last position; a wave wholly past the prompt computes nothing
  const int32_t w_last = i0 < p ? min(i0 + 15, p - 1) : -1;
  // This lane's transpose-load address within a value row block: key offset
  // 4*g4 + c16/4, columns 4*(c16 % 4).
  const int tr_off = (4 * g4 + c16 / 4) * ROW + (c16 % 4) * 8;
  // The prompt's keys and values of head h as raw buffers: token t's row at
  // byte t * nkv * D * 2; a token past the prompt gets an offset beyond the
  // range, which loads zeros (no branch, no wait per load).
  const uint32_t tok_bytes = (uint32_t)nkv * VPT * 16;
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(kin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(vin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  u32x4 kr[NLD], vr[NLD];
  auto fetch = [&](int32_t kt, u32x4 (&kr)[NLD], u32x4 (&vr)[NLD]) {
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int v = tid + NT * u;
      const int32_t t = kt + v / VPT;
      const uint32_t off = t < p ? (uint32_t)t * tok_bytes + (uint32_t)(v % VPT) * 16u : 0x80000000u;
      kr[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0));
      vr[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0));
    }
  };
  auto compute = [&](int32_t k0) {
#pragma unroll
    for (int half = 0; half < KT / 32; ++half) {
      const int kb = ks * KT + 32 * half;              // key row of the block in the stage
      const int32_t tt = k0 + kb;
      if (tt > w_last) break;                          // wave-uniform
      f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = sa;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const u32x4 ka = *reinterpret_cast<const u32x4*>(ldsK + (kb + c16) * ROW + (kk * 4 + g4) * 16);
        const u32x4 kc = *reinterpret_cast<const u32x4*>(ldsK + (kb + 16 + c16) * ROW + (kk * 4 + g4) * 16);
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ka), qb[kk], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kc), qb[kk], sb, 0, 0, 0);
      }
      // Unscaled scores; masked keys -inf.  A block whose 32 keys all come
      // before the wave's first position is visible to all of its positions
      // and needs no mask (positions past the prompt are never written).
      float s[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] = sa[r];
        s[4 + r] = sb[r];
      }
      if (tt + 31 > i0) {                            // wave-uniform
        const int32_t lim = qi < p ? qi - tt : -1;   // keys tt .. tt + lim are visible
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[r] = 4 * g4 + r <= lim ? s[r] : -INFINITY;
          s[4 + r] = 16 + 4 * g4 + r <= lim ? s[4 + r] : -INFINITY;
        }
      }
      float mx = s[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = fmaxf(mx, s[e]);
      mx = max_over_groups(mx) * qscale;             // qscale >= 0: the max of the scaled scores
      // The reference the weights are taken against moves only when the
      // block's maximum passes it by more than kPrefillLazy (base 2):
      // softmax does not depend on the reference, the weights stay below
      // 2^kPrefillLazy (well inside bf16's and fp32's range, at bf16's
      // relative precision), and the accumulators are rescaled -- this
      // lane's position by its own factor -- only when some position's
      // reference moved, which after the first keys is rare.
      if (__ballot(mx > m + kPrefillLazy)) {     // wave-uniform
        const float mn = mx > m + kPrefillLazy ? mx : m;
        const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
        ol *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
        m = mn;
      }
      const float ref = m == -INFINITY ? 0.f : m;
      // exponents are <= kPrefillLazy here: the hardware exp2 (results below
      // the smallest normal flush to 0, which a softmax weight may); the
      // scale is applied in the exponent's multiply-add
      bf16x8 pa;
#pragma unroll
      for (int e = 0; e < 8; ++e) pa[e] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[e], qscale, -ref));
      const uint8_t* vblk = ldsV + kb * ROW + tr_off;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const s16x4 lo = lds_read_tr16(vblk + dt * 32);
        const s16x4 hi = lds_read_tr16(vblk + 16 * ROW + dt * 32);
        const s16x4 w2[2] = {lo, hi};
        const bf16x8 vb = __builtin_bit_cast(bf16x8, w2);
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, pa, o[dt], 0, 0, 0);
      }
      ol = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pa, ol, 0, 0, 0);
    }
  };
  // The next stage's loads are in flight while the current one is computed.
  fetch(0, kr, vr);
  for (int32_t k0 = 0; k0 <= wg_last; k0 += S * KT) {   // bounds are workgroup-uniform
    __syncthreads();                                   // the previous stage is consumed
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int v = tid + NT * u;
      const int off = (v / VPT) * ROW + (v % VPT) * 16;
      *reinterpret_cast<u32x4*>(ldsK + off) = kr[u];
      *reinterpret_cast<u32x4*>(ldsV + off) = vr[u];
    }
    __syncthreads();
    if (k0 + S * KT <= wg_last) fetch(k0 + S * KT, kr, vr);
    compute(k0);
  }

  // Every lane of a position holds its whole sum (the operation summed over
  // the 32 keys of each block).
  float lsum = ol[0];
  if constexpr (S > 1) {
    // Key streams 1.. hand their states to stream 0 (same positions, same lane).
    __syncthreads();                                   // the stage buffers are free
    float* mrg = reinterpret_cast<float*>(lds) + ((ks - 1) * 4 + wave % 4) * kWave * REC + lane * REC;
    if (ks > 0) {
      mrg[0] = m;
      mrg[1] = lsum;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mrg[2 + dt * 4 + r] = o[dt][r];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int k = 1; k < S; ++k) {
        const float* src = reinterpret_cast<const float*>(lds) + ((k - 1) * 4 + wave % 4) * kWave * REC + lane * REC;
        const float m2 = src[0];
        const float mm = fmaxf(m, m2);
        const float fa = m == -INFINITY ? 0.f : exp2f(m - mm);
        const float fb = m2 == -INFINITY ? 0.f : exp2f(m2 - mm);
        lsum = lsum * fa + src[1] * fb;
        m = mm;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) o[dt][r] = o[dt][r] * fa + src[2 + dt * 4 + r] * fb;
      }
    }
  }
  if (ks == 0 && qi < p) {
    // Lane l holds columns 16 dt + 4 (l / 16) + r of position l % 16.
    const float inv = 1.f / lsum;
    uint16_t* o16 = reinterpret_cast<uint16_t*>(a.out) + ((row0 + qi) * nq + hq) * D + 4 * g4;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *reinterpret_cast<uint2*>(o16 + 16 * dt) =
          make_uint2(f32_to_bf16_rne(o[dt][0] * inv) | (f32_to_bf16_rne(o[dt][1] * inv) << 16),
                     f32_to_bf16_rne(o[dt][2] * inv) | (f32_to_bf16_rne(o[dt][3] * inv) << 16));
  }
}

// bf16 for long prompts, on v_mfma_f32_32x32x16_bf16: four waves of 32 prompt
// positions of one query head, the keys in blocks of 32.  In the kernel above
// every 32 x 16 block of scores reads its 16 KB of keys and values from LDS; here
// the same 16 KB serve 32 positions, the loads go to LDS without registers two blocks ahead, and the block loop is
// pipelined in software so that a wave's matrix and vector work overlap:
// iteration t multiplies the values of block t - 1 and takes the maximum of block
// t's scores, then computes the scores of block t + 1 and the weights of block t.
//  * scores: A = 32 key rows, B = 32 positions; lane l, register r: position
//    l % 32, key 8 (r / 4) + 4 (l / 32) + r % 4.
//  * values: O^T = V^T P^T; step j takes registers 8 j .. 8 j + 7 of the lane's
//    own weights as B, so A's k = 8 (l / 32) + e stands for key 16 j + 4 (l / 32)
//    + e (e < 4) and 16 j + 8 + 4 (l / 32) + e - 4: two transposing LDS loads.
//  * the weights' sum is of the bf16 weights P.V is made of.
// 64 query heads over 8 kv-heads of 128, 4096 tokens: 390 -> 325 us (0.70 -> 0.85
// PFLOP/s over the visible pairs).  What bounds it now: two waves per SIMD (173
// registers) that wait for their own chain 0.34 of their cycles (the matrix cores
// busy 0.46 of the time, no LDS conflicts), and the clock, 1.88 GHz under this
// load; before its first block each wave also waits for its query fragments, whose
// loads the compiler takes one after the other.  Capped for three waves it spills,
// and two accumulators per score or a raised wave priority changed nothing.
constexpr int kPrefillTile32 = 128;
// How far (base 2) a block's maximum may pass the reference before it moves.
// The weight of the key a reference was taken from is exactly 1; the further a
// later maximum may pass it, the more often the largest weight is one that bf16
// rounds.  Error against float64 (prompts of 1,500 to 2,600 tokens, 2-norm
// relative; the kernel above, with two references per position, 0.00205) and
// time at 4096 tokens of 64 heads: 0 0.00200, 327 us; 1 0.00204, 325; 1.5 0.00205,
// 322; 8 0.00208, 298.
constexpr float kPrefillLazy32 = 1.0f;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// LDS rows are filled by LDS-direct loads (no registers hold keys or values on
// their way), so they cannot be padded; the 16-byte chunks of a row are placed
// by the row instead, so that reads of many rows spread over all banks:
//  * keys (a chunk of 32 rows per read, lane half hh reading chunk 2 kk + hh):
//    the halves in different halves of the row, xor the row;
//  * values (transposing loads, 64 bytes of 4 + 4 rows): 64-byte units xor the
//    row.
// (Chunks xor the row for both cost 60% of the LDS cycles in conflicts.)
template <int CH>   // chunks per row: 16 (head_dim 128) or 8
__device__ __forceinline__ int key_place(int chunk, int row) {
  return ((chunk % 2) * (CH / 2) + chunk / 2) ^ (CH == 16 ? row % 16 : row / 2 % 8);
}
template <int CH>
__device__ __forceinline__ int key_chunk(int place, int row) {   // the inverse in `chunk`
  const int y = place ^ (CH == 16 ? row % 16 : row / 2 % 8);
  return (y % (CH / 2)) * 2 + y / (CH / 2);
}
template <int CH>
__device__ __forceinline__ int value_place(int chunk, int row) {   // its own inverse
  return chunk ^ (4 * (CH == 16 ? row % 4 : row / 2 % 2));
}
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t off) {
#if defined(__HIP_DEVICE_COMPILE__)
  // lane l's 16 bytes land at dst + 16 l
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
#endif
}

// This wave's LDS reads and all but its last VM loads have finished, then the
// barrier.  __syncthreads() does not promise that another wave's loads into LDS
// have landed.
template <int VM>
__device__ __forceinline__ void wait_and_barrier() {
  static_assert(VM < 16, "vmcnt's low four bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070 | VM);       // vmcnt <= VM, lgkmcnt 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int D, int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2)))
prefill_fa32_kernel(const PrefillArgs a) {
  constexpr int VPT = D / 8, KK = D / 16, DT = D / 32, TILE = kPrefillTile32;
  constexpr int ROW = D * 2;
  constexpr int RPI = kWave / VPT, NI = 32 / RPI / 4;   // rows per load; loads per wave and block
  // a buffer each, not an array of three: reads of one must not wait for the loads into the other
  __shared__ __attribute__((aligned(1024))) uint8_t ldsK0[32 * ROW], ldsK1[32 * ROW], ldsK2[32 * ROW];
  __shared__ __attribute__((aligned(1024))) uint8_t ldsV0[32 * ROW], ldsV1[32 * ROW], ldsV2[32 * ROW];
  const int tid = threadIdx.x;
  if ((int32_t)blockIdx.x >= a.n_attn) {
    const int32_t j = (int32_t)blockIdx.x - a.n_attn;
    const int32_t g = j / a.n_kv_heads, h = j % a.n_kv_heads;
    int32_t ins = 0;
    while (ins < a.n_ins - 1 && g >= a.tile_end[ins]) ++ins;
    const int32_t tile = a.tile_end[ins] - 1 - g, p = a.plen[ins], b = a.slot[ins];
    const int64_t row0 = (int64_t)b * a.T + (a.T - p);
    prefill_append<VPT>(a, b, h, p, row0, tile * TILE, min(TILE, p - tile * TILE), tid, 256);
    return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int c32 = lane % 32, hh = lane / 32, g4 = lane / 16, m16 = lane % 16;
  int hq;
  int32_t ins, tile;
  prefill_work(a, hq, ins, tile);
  const int h = hq / G;
  const int b = a.slot[ins];
  const int32_t p = a.plen[ins];
  const int32_t wg0 = tile * TILE, i0 = wg0 + 32 * wave;
  const int64_t row0 = (int64_t)b * a.T + (a.T - p);
  const int nkv = a.n_kv_heads, nq = nkv * G;
  const u32x4* qin = reinterpret_cast<const u32x4*>(a.q);
  const u32x4* kin = reinterpret_cast<const u32x4*>(a.knew);
  const u32x4* vin = reinterpret_cast<const u32x4*>(a.vnew);
  const float qscale = fabsf(a.qscale);
  const uint32_t qsw = a.qscale < 0.f ? 0x80008000u : 0u;
  const u32x4 qsign = {qsw, qsw, qsw, qsw};
  const int32_t qi = i0 + c32;
  bf16x8 qb[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qb[kk] = as_bf16x8(qi < p ? qin[((row0 + qi) * nq + hq) * VPT + kk * 2 + hh] ^ qsign : u32x4{0, 0, 0, 0});

  const uint32_t tok_bytes = (uint32_t)nkv * VPT * 16;
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(kin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(vin + (row0 * nkv + h) * VPT), 0, (uint32_t)p * tok_bytes, kBufferWord3);
  // Block t's rows into buf: load i of this wave brings rows (4 i + wave) RPI ..
  const int lr = wave * RPI + lane / VPT;
  uint32_t off_k[NI], off_v[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = 4 * RPI * i + lr;
    off_k[i] = (uint32_t)row * tok_bytes + (uint32_t)key_chunk<VPT>(lane % VPT, row) * 16u;
    off_v[i] = (uint32_t)row * tok_bytes + (uint32_t)value_place<VPT>(lane % VPT, row) * 16u;
  }
  auto fetch = [&](__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[NI], int32_t t, uint8_t* buf) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      lds_load16(r, buf + (4 * i + wave) * 1024,
                 32 * t + 4 * RPI * i < p - lr ? off[i] + (uint32_t)(32 * t) * tok_bytes : 0x80000000u);
  };
  const int k_off = c32 * ROW + key_place<VPT>(hh, c32) * 16;   // chunk 2 kk + hh: xor 16 kk
  auto scores = [&](const uint8_t* buf) {
    f32x16 s = {};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*reinterpret_cast<const u32x4*>(buf + (k_off ^ (16 * kk)))),
                                                  qb[kk], s, 0, 0, 0);
    return s;
  };
  // Transposing load (j, e, dt): key 16 j + 8 e + 4 hh + m / 4, columns 32 dt +
  // 16 (g % 2) + 4 (m % 4), m = lane % 16, g = lane / 16.
  const int v_row = 4 * hh + m16 / 4;              // key 16 j + 8 e more: the same place
  const int v_off = v_row * ROW + value_place<VPT>(2 * (g4 % 2) + (m16 % 4) / 2, v_row) * 16 + 8 * (m16 % 2);

  const int32_t last_t = (min(wg0 + TILE, p) - 1) / 32;                    // the workgroup's last block
  const int32_t my_t = i0 < p ? (min(i0 + 32, p) - 1) / 32 : -1;           // this wave's
  float m = -INFINITY, lsum = 0.f;
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x16{};
  bf16x8 pw[2] = {as_bf16x8(u32x4{0, 0, 0, 0}), as_bf16x8(u32x4{0, 0, 0, 0})};   // weights of block t - 1

  // Iteration t, with block t's scores in s: the loads of V block t + 1 and K
  // block t + 3 go where V block t - 2 and K block t were last read before the
  // barrier that began it; V block t - 1 and K block t + 1 are read.  Its
  // barrier comes after every load but this iteration's own 2 NI (and every
  // LDS read) of the wave has finished, so a load has two iterations.
  f32x16 s;
  auto step = [&](int32_t t, const uint8_t* kbuf, const uint8_t* vbuf, uint8_t* kfree, uint8_t* vfree) {
    fetch(rv, off_v, t + 1, vfree);
    fetch(rk, off_k, t + 3, kfree);
    if (t <= my_t + 1) {                         // wave-uniform; iteration my_t + 1 only adds block my_t's values
      if (32 * t + 31 > i0) {                    // not every position sees the whole block
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int32_t key = 32 * t + 8 * (r / 4) + 4 * hh + r % 4;
          s[r] = key <= qi && qi < p ? s[r] : -INFINITY;
        }
      }
      float mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
      if (t > 0) {                               // the values of block t - 1
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            s16x4 w2[2];
#pragma unroll
            for (int e = 0; e < 2; ++e)
              w2[e] = lds_read_tr16(vbuf + (16 * j + 8 * e) * ROW + (v_off ^ (64 * dt)));
            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w2), pw[j], o[dt], 0, 0, 0);
          }
      }
      {
        const uint32_t u = __float_as_uint(mx);
        const auto x = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        mx = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])) * qscale;
      }
      if (__ballot(mx > m + kPrefillLazy32)) {   // the reference moves, see above
        const float mn = mx > m + kPrefillLazy32 ? mx : m;
        const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
        lsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
        m = mn;
      }
      const float ref = m == -INFINITY ? 0.f : m;
      const f32x16 sn = scores(kbuf);            // of block t + 1, beside the weights of block t
#pragma unroll
      for (int r = 0; r < 16; ++r) pw[r / 8][r % 8] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[r], qscale, -ref));
      const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);
#pragma unroll
      for (int r = 0; r < 16; r += 2)
        lsum = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pw[r / 8][r % 8], pw[r / 8][r % 8 + 1]}, ones, lsum, false);
      s = sn;
    }
    wait_and_barrier<2 * NI>();
  };
  fetch(rk, off_k, 0, ldsK0);
  fetch(rk, off_k, 1, ldsK1);
  fetch(rk, off_k, 2, ldsK2);
  fetch(rv, off_v, 0, ldsV0);
  wait_and_barrier<0>();
  s = scores(ldsK0);
  wait_and_barrier<0>();                         // K block 0 is read: iteration 0 loads over it
  for (int32_t t = 0;; t += 3) {                 // bounds are workgroup-uniform; iteration last_t + 1 is the last
    step(t, ldsK1, ldsV2, ldsK0, ldsV1);
    if (t > last_t) break;
    step(t + 1, ldsK2, ldsV0, ldsK1, ldsV2);
    if (t + 1 > last_t) break;
    step(t + 2, ldsK0, ldsV1, ldsK2, ldsV0);
    if (t + 2 > last_t) break;
  }
  {
    const uint32_t u = __float_as_uint(lsum);
    const auto x = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    lsum = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  }
  if (qi < p) {
    const float inv = 1.f / lsum;
    uint16_t* o16 = reinterpret_cast<uint16_t*>(a.out) + ((row0 + qi) * nq + hq) * D + 4 * hh;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; r += 4)
        *reinterpret_cast<uint2*>(o16 + 32 * dt + 2 * r) =
            make_uint2(f32_to_bf16_rne(o[dt][r] * inv) | (f32_to_bf16_rne(o[dt][r + 1] * inv) << 16),
                       f32_to_bf16_rne(o[dt][r + 2] * inv) | (f32_to_bf16_rne(o[dt][r + 3] * inv) << 16));
  }
}

}  // namespace baton
