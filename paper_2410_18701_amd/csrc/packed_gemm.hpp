// GEMM kernels of the decode-layer projections: y[m][n] (+)= sum_k x[m][k]
// w[n][k] for m < rows <= 256, a linear layer at a decode step's batch, on a
// packed copy of the weight.  bf16 storage, fp32 sums, outputs rounded to
// nearest even.
//
// The packed weight, made once per weight by pack_weight_kernel: 16-row slices
// of w, each a run of 1 KB blocks, one per step of 32 along k, block (s, t)
// holding at byte 16 l the eight elements w[16 s + l % 16][32 t + 8 (l / 16)
// ..] (zeros past N or K) -- exactly the A operand of
// v_mfma_f32_16x16x32_bf16 for lane l.  A wave streams a slice with one
// contiguous 1 KB load per block, so every weight row is read in long bursts
// (in the stored row-major layout a wave would touch 16 rows 64 bytes at a
// time, which the DRAM serves at a fraction of its bandwidth).  x's rows are
// the B operand, 16 at a time (lane l: row 16 j + l % 16, the same k group);
// lane l then holds outputs (n0 + 4 (l / 16) + r, 16 j + l % 16), r < 4.
// Loads are raw buffer loads whose out-of-range offsets return zeros: x rows
// past `rows` and k past K need no branch.
//
// Three kernels, chosen by the rows (packed_gemm_plan in gemm_plan.hpp):
//  * up to 8 rows, row_gemm_kernel: no barrier, no LDS until the end; where it
//    is not the faster one, skinny_gemm_kernel;
//  * 9 to 64 rows, skinny_gemm_kernel: one slice per wave; with the gated
//    activation only where its workgroups make one round;
//  * past 64 rows, and with the gated activation from 9 rows otherwise,
//    tile_gemm_kernel: one to three slices per wave, the LDS reads of the
//    activations pipelined ahead of the matrix operations.
// Unsplit, the kernels that a row count may take add along k in the same order
// -- up to 8 rows the sums of four ranges of k, past that one chain of 32-wide
// matrix operations per output -- so either gives the same bits, and a gated
// product those of the plain one and the activation.
#pragma once

#include "gemm_plan.hpp"
#include "layer_ops.hpp"

namespace baton {
namespace {

typedef __bf16 gemm_bf16x8 __attribute__((ext_vector_type(8)));
typedef float gemm_f32x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
  const uint16_t* x;     // [rows][K]
  const uint16_t* wp;    // packed weight: [ceil(N / 16)][ceil(K / 32)] blocks of 512 elements
  uint16_t* y;           // [rows][N]
  float* part;           // [S][rows][N] fp32, when S > 1
  int32_t rows, N, K;    // rows <= 256
  int32_t chunks;        // row chunks (tile_gemm_kernel past 64 rows), or 1
  int32_t groups;        // slice groups (workgroups per chunk)
  int32_t kt;            // blocks per slice, ceil(K / 32)
  int32_t tc;            // blocks per split
  int32_t accumulate;    // 1: y += x . w^T
  int32_t gated;         // F > 0: w is [gate; up] (2F rows), y [rows][F] = silu(x . gate^T) * (x . up^T)
};

constexpr uint32_t kGemmOob = 0x80000000u;   // an offset past every buffer's range
constexpr int32_t kGemmBufWord3 = 0x00020000;

template <int AUX>   // 2: non-temporal
__device__ __forceinline__ u32x4 gemm_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX));
}

// A raw buffer resource over [p, p + bytes), held in scalar registers: base and
// size are uniform, but a select between them may otherwise be left in vector
// registers, and every load through it would then run a loop over its values.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const uint16_t* p, int32_t bytes) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)hi << 32 | lo), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), kGemmBufWord3);
}

__device__ __forceinline__ gemm_f32x4 gemm_mfma(const u32x4& a, const u32x4& b, const gemm_f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(gemm_bf16x8, a), __builtin_bit_cast(gemm_bf16x8, b),
                                                 c, 0, 0, 0);
}

// One thread per 16-byte piece of the packed weight.
__global__ void __launch_bounds__(256) pack_weight_kernel(const u32x4* __restrict__ w, u32x4* __restrict__ wp,
                                                          int32_t N, int32_t K, int32_t kt, int64_t n_pieces) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_pieces) return;
  const int32_t l = (int32_t)(i % kWave);
  const int64_t blk = i / kWave;
  const int32_t t = (int32_t)(blk % kt);
  const int32_t n = (int32_t)(blk / kt) * 16 + l % 16, k = 32 * t + 8 * (l / 16);
  wp[i] = (n < N && k < K) ? w[((int64_t)n * K + k) / 8] : u32x4{0, 0, 0, 0};
}

// Up to 8 rows the sum over `blocks` 32-wide blocks is of four ranges of k added
// in order; this is a range's length in batches of four blocks (the last ranges
// may be shorter or empty).
__device__ __forceinline__ int32_t four_ranges(int32_t blocks) { return ((blocks + 3) / 4 + 3) / 4; }

// The four outputs (m, n .. n + 3) of a lane: the split's partial sum, or y.
__device__ __forceinline__ void gemm_store(const GemmArgs& a, int32_t m, int32_t n, gemm_f32x4 v) {
  if (gridDim.y > 1) {
    *reinterpret_cast<gemm_f32x4*>(a.part + ((int64_t)blockIdx.y * a.rows + m) * a.N + n) = v;
    return;
  }
  uint2* yp = reinterpret_cast<uint2*>(a.y + (int64_t)m * a.N + n);
  if (a.accumulate) {
    const uint2 old = *yp;
    v[0] += bf16_lo(old.x); v[1] += bf16_hi(old.x); v[2] += bf16_lo(old.y); v[3] += bf16_hi(old.y);
  }
  *yp = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}

__device__ __forceinline__ uint2 pack_bf16x4(const gemm_f32x4& v) {
  return make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}

// The gated epilogue of a workgroup whose waves w and w + 2 (w < 2) hold a gate
// slice set and the up slices of the same columns, the same (row, column) places
// in each: every wave finishes every other tile, the gate wave the even ones, the
// up wave the odd ones, the other's outputs (rounded to bf16) reaching it through
// lds.  gs0 is the pair's first gate slice; rows row0 .. row0 + rows - 1 are written.
template <int NS, int MT>
__device__ __forceinline__ void gemm_gated_store(const GemmArgs& a, uint8_t* lds, const gemm_f32x4 (&acc)[NS][MT], int w,
                                                 int lane, int32_t gs0, int32_t row0, int32_t rows) {
  uint2* ex = reinterpret_cast<uint2*>(lds) + (w % 2) * NS * MT * kWave + lane;
  const int up = w / 2, c16 = lane % 16, g4 = lane / 16;
#pragma unroll
  for (int q = 0; q < NS * MT; ++q)
    if (q % 2 != up) ex[q * kWave] = pack_bf16x4(acc[q / MT][q % MT]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NS * MT; ++q) {
    if (q % 2 != up) continue;
    const int32_t n = 16 * (gs0 + q / MT) + 4 * g4, m = 16 * (q % MT) + c16;
    if (n >= a.gated || m >= rows) continue;
    const uint2 own = pack_bf16x4(acc[q / MT][q % MT]), other = ex[q * kWave];
    *reinterpret_cast<uint2*>(a.y + (int64_t)(row0 + m) * a.gated + n) = up ? silu_mul4(other, own) : silu_mul4(own, other);
  }
}

// ---------------------------------------------------------- up to 8 rows --
// What bounds it: the weight's bytes from HBM; each byte is used for at most
// eight rows.  A workgroup of four waves owns NS slices (1; gated 2, a gate
// slice and the up slice of the same columns) and each wave a quarter of the
// k range, kRowDepth pairs of blocks in flight per wave, so that the loop has
// neither a barrier nor LDS and 256 slices already fill the GPU: the
// projections that used to split along k need no partial sums in HBM and no
// second launch.  The waves' sums meet in LDS at the end, added in wave order.
// The activations are loaded straight in the B operand's layout, 16 rows of 64
// bytes per load, which costs the L1 four times a contiguous load: lanes of
// rows past `rows` cost nothing, so this is right for a few rows and too slow
// for many (llama2-7b's QKV product takes 19.2 us at 1 row, 20.3 at 8, 23.3 at
// 16 against 20.8, 21.1 and 21.3 of the staged kernel below).  Measured at 1
// row (us, staged kernel with its reductions first; a plain read of the weight
// last): QKV 20.8 -> 19.2 (16.2), output 12.5 -> 8.9 (6.6), gate/up with the
// activation 36.5 -> 31.8 (27.8), down 18.9 -> 18.4 (15.0).
constexpr int kRowDepth = 8;
constexpr uint32_t kRowOob = 0x40000000u;   // past a slice (at most 2^29 bytes) and the rows of x (2^29)

template <bool GATED>
__global__ void __launch_bounds__(kWave * kGemmWaves) row_gemm_kernel(const GemmArgs a) {
  constexpr int NS = GATED ? 2 : 1, P = kRowDepth;
  __shared__ __attribute__((aligned(16))) gemm_f32x4 red[kGemmWaves][NS][kWave];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, c16 = lane % 16, g4 = lane / 16;
  const int32_t grp = blockIdx.x;
  const int32_t t_begin = blockIdx.y * a.tc, t_end = min(a.kt, t_begin + a.tc);
  // this wave's pairs of blocks, an even number of them (whole batches of the staged kernel)
  const int32_t np = (t_end - t_begin + 1) / 2, per = 2 * four_ranges(t_end - t_begin);
  const int32_t p0 = min(w * per, np), p1 = min(p0 + per, np);
  const uint32_t row_bytes = (uint32_t)a.K * 2u;
  __amdgpu_buffer_rsrc_t rw[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i)
    rw[i] = uniform_rsrc(a.wp + ((int64_t)(grp + i * (a.gated / 16)) * a.kt + t_begin) * 512, (t_end - t_begin) * 1024);
  const __amdgpu_buffer_rsrc_t rx = uniform_rsrc(a.x, (int32_t)(a.rows * row_bytes));
  // blocks of this wave whose k group of this lane lies inside [0, K)
  const int32_t tl = min(min(t_end, t_begin + 2 * p1), (a.K - 8 * g4 + 31) / 32);
  const uint32_t x0 = (uint32_t)c16 * row_bytes + 16u * g4, w0 = 16u * lane;
  const bool row_in = c16 < a.rows;
  u32x4 wr[P][NS][2], xr[P][2];
  auto issue = [&](int32_t p, u32x4 (&wv)[NS][2], u32x4 (&xv)[2]) {
    const int32_t t = t_begin + 2 * p;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool in = t + u < tl;
      const uint32_t wo = in ? w0 + 1024u * (uint32_t)(t + u - t_begin) : kRowOob;
#pragma unroll
      for (int i = 0; i < NS; ++i) wv[i][u] = gemm_load<2>(rw[i], wo);
      xv[u] = gemm_load<0>(rx, in && row_in ? x0 + 64u * (uint32_t)(t + u) : kRowOob);
    }
  };
  gemm_f32x4 acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i] = gemm_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < P; ++q) issue(p0 + q, wr[q], xr[q]);
  for (int32_t p = p0; p < p1; p += P) {
#pragma unroll
    for (int q = 0; q < P; ++q) {   // past p1: zeros
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < NS; ++i) acc[i] = gemm_mfma(wr[q][i][u], xr[q][u], acc[i]);
      __builtin_amdgcn_sched_barrier(0);
      issue(p + q + P, wr[q], xr[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) red[w][i][lane] = acc[i];
  __syncthreads();
  const int32_t n = 16 * grp + 4 * g4;
  if (w > 0 || !row_in || n >= (GATED ? a.gated : a.N)) return;
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int q = 1; q < kGemmWaves; ++q) acc[i] += red[q][i][lane];
  if constexpr (GATED)
    *reinterpret_cast<uint2*>(a.y + (int64_t)c16 * a.gated + n) = silu_mul4(pack_bf16x4(acc[0]), pack_bf16x4(acc[1]));
  else
    gemm_store(a, c16, n, acc[0]);
}

// ------------------------- 9 to 64 rows, and up to 8 where it is faster --
// A wave owns one slice (four per workgroup; gated: two gate slices and their
// up slices), the workgroup all the rows.  The
// activation rows are staged in LDS per batch of four blocks, each row padded
// by 16 bytes so that the 16 rows one B-operand read spans fall in different
// banks; when there are too few slices to occupy the GPU the blocks are also
// split into S ranges whose fp32 partial sums gemm_reduce_kernel adds up.
// tile_gemm_kernel with one slice per wave is no faster here (llama2-7b at 64
// rows: QKV 25.6 against 25.4 us, output 14.1 against 14.8, down 23.7 against
// 23.8; at 16 rows QKV 22.5 against 21.4, down 20.4 against 19.4).
template <int MG, bool GATED, bool FOUR>
__global__ void __launch_bounds__(kWave * kGemmWaves) skinny_gemm_kernel(const GemmArgs a) {
  constexpr int KU = 4, P = 4;                     // blocks per batch; register sets of the load pipeline
  constexpr int kRows = 64;                        // staged rows (past `rows`: zeros)
  constexpr int kRow = 64 * KU + 16;               // bytes per staged row
  constexpr int kBuf = kRows * kRow, kPieces = 4 * KU;   // 16-byte pieces per row and batch
  constexpr int kXPer = kRows * kPieces / (kWave * kGemmWaves);   // activation pieces per thread and batch
  __shared__ __attribute__((aligned(16))) uint8_t xs[2][kBuf];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, c16 = lane % 16, g4 = lane / 16;
  // Gated: waves 0 and 1 take two gate slices, waves 2 and 3 their up slices.
  static_assert(kGemmWaves == 4, "the gated epilogue pairs two gate and two up waves");
  const int32_t gate = 2 * (int32_t)blockIdx.x + w % 2;
  const int32_t slice = GATED ? gate + (w < 2 ? 0 : a.gated / 16) : (int32_t)blockIdx.x * kGemmWaves + w;
  const int32_t s_end = GATED && w < 2 ? a.gated / 16 : (a.N + 15) / 16;   // this wave's slices end here
  const int32_t t_begin = blockIdx.y * a.tc, t_end = min(a.kt, t_begin + a.tc);
  const uint32_t row_bytes = (uint32_t)a.K * 2u;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(   // empty past N (loads zeros, writes nothing)
      const_cast<uint16_t*>(a.wp) + ((int64_t)min(slice, s_end - 1) * a.kt + t_begin) * 512, 0,
      slice < s_end ? (t_end - t_begin) * 1024 : 0, kGemmBufWord3);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(a.x), 0, (int32_t)(a.rows * row_bytes), kGemmBufWord3);

  gemm_f32x4 acc[1][MG];
#pragma unroll
  for (int j = 0; j < MG; ++j) acc[0][j] = gemm_f32x4{0.f, 0.f, 0.f, 0.f};

  // Loads of batch b (blocks t_begin + KU b ...): the workgroup's activation
  // pieces (thread tid: pieces tid + 256 i -- row p / (4 KU), 16 bytes at
  // 16 (p % (4 KU)) of the batch) and this wave's weight blocks, both issued
  // unconditionally (past the end they return zeros).
  auto issue = [&](int32_t b, u32x4 (&xr)[kXPer], u32x4 (&wr)[KU]) {
    const int32_t tb = t_begin + KU * b;
#pragma unroll
    for (int i = 0; i < kXPer; ++i) {
      const int32_t p = tid + kWave * kGemmWaves * i;
      const int32_t m = p / kPieces, c = p % kPieces;
      const int32_t k = 32 * tb + 8 * c;
      xr[i] = gemm_load<0>(rx, (m < a.rows && k < a.K && tb + c / 4 < t_end)
                                   ? (uint32_t)m * row_bytes + (uint32_t)k * 2u : kGemmOob);
    }
#pragma unroll
    for (int u = 0; u < KU; ++u)
      wr[u] = gemm_load<2>(rw, tb + u < t_end ? (uint32_t)(tb + u - t_begin) * 1024u + (uint32_t)lane * 16u : kGemmOob);
  };
  auto stage = [&](int buf, const u32x4 (&xr)[kXPer]) {
#pragma unroll
    for (int i = 0; i < kXPer; ++i) {
      const int32_t p = tid + kWave * kGemmWaves * i;
      *reinterpret_cast<u32x4*>(&xs[buf][(p / kPieces) * kRow + (p % kPieces) * 16]) = xr[i];
    }
  };
  // FOUR: the sum of each of the four ranges of k that row_gemm_kernel's waves
  // take by itself, the ranges added in the waves' order (the same bits).
  const int32_t range = four_ranges(t_end - t_begin);   // batches
  int32_t next = range, passed = 0;
  gemm_f32x4 tot[MG];
  auto mult = [&](int32_t b, const u32x4 (&wr)[KU]) {
    if (FOUR && b == next) {   // the same for the whole workgroup
#pragma unroll
      for (int j = 0; j < MG; ++j) {
        tot[j] = passed ? tot[j] + acc[0][j] : acc[0][j];
        acc[0][j] = gemm_f32x4{0.f, 0.f, 0.f, 0.f};
      }
      next += range;
      ++passed;
    }
    const int buf = b & 1;
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      u32x4 xb[MG];
#pragma unroll
      for (int j = 0; j < MG; ++j)
        xb[j] = *reinterpret_cast<const u32x4*>(&xs[buf][(16 * j + c16) * kRow + (32 * u + 8 * g4) * 2]);
#pragma unroll
      for (int j = 0; j < MG; ++j) acc[0][j] = gemm_mfma(wr[u], xb[j], acc[0][j]);
    }
  };
  // P register sets: while batch b is multiplied, batches b + 1 .. b + P - 1
  // are in flight (every batch's activation loads are issued ahead of its
  // weight loads, so waiting for activations never waits for weights), and
  // batch b + 1's activations, issued P - 2 batches earlier, go to LDS at the
  // end of the step.  Batch b's activations are in LDS buffer b & 1.  Sets are
  // indexed by constants only (the steps are unrolled), so they stay in
  // registers.
  const int32_t n_batch = (t_end - t_begin + KU - 1) / KU;   // the same for the whole workgroup
  if (n_batch > 0) {
    u32x4 xr[P][kXPer], wr[P][KU];
#pragma unroll
    for (int q = 0; q < P - 1; ++q) issue(q, xr[q], wr[q]);
    stage(0, xr[0]);
    __syncthreads();
#define BATON_GEMM_STEP(S)                                               \
  issue(b + (S) + P - 1, xr[((S) + P - 1) % P], wr[((S) + P - 1) % P]); \
  __builtin_amdgcn_sched_barrier(0);                                     \
  mult(b + (S), wr[(S) % P]);                                            \
  stage((b + (S) + 1) & 1, xr[((S) + 1) % P]);                           \
  __syncthreads();
    // A counted loop with no exit inside its body (an exit between the steps
    // makes the compiler drain every load in flight at the loop head), then
    // the last n_batch % P steps.
    int32_t b = 0;
    for (; b + P <= n_batch; b += P) {
#pragma unroll
      for (int q = 0; q < P; ++q) {
        BATON_GEMM_STEP(q)
      }
    }
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
      if (b + q >= n_batch) break;
      BATON_GEMM_STEP(q)
    }
#undef BATON_GEMM_STEP
  }
  if constexpr (FOUR) {
#pragma unroll
    for (int j = 0; j < MG; ++j) {
      if (passed) acc[0][j] = tot[j] + acc[0][j];
      if (passed < 3) acc[0][j] += gemm_f32x4{0.f, 0.f, 0.f, 0.f};   // the empty ranges
    }
  }
  if constexpr (GATED) {
    gemm_gated_store<1, MG>(a, &xs[0][0], acc, w, lane, gate, 0, a.rows);
    return;
  }
  const int32_t n = 16 * slice + 4 * g4;
  if (n >= a.N) return;
#pragma unroll
  for (int j = 0; j < MG; ++j) {
    const int32_t m = 16 * j + c16;
    if (m < a.rows) gemm_store(a, m, n, acc[0][j]);
  }
}

// ------------------------- past 64 rows, and gated from 9 rows if faster --
// The (slice group, row chunk) of a workgroup.  One chunk: the group is the
// workgroup index.  Several: workgroups are dealt to the GPU's eight XCDs in
// turn (index mod 8), so the chunks of one group go to indices 8 apart -- the
// same XCD, dispatched one after the other -- and the weight blocks they all
// read come from that XCD's L2 after the first read; the grid is padded to
// whole sets of 8 groups, the padding workgroups doing nothing.
__device__ __forceinline__ bool gemm_tile(const GemmArgs& a, int32_t& grp, int32_t& chunk) {
  if (a.chunks == 1) {
    grp = (int32_t)blockIdx.x;
    chunk = 0;
    return true;
  }
  const int32_t b = (int32_t)blockIdx.x, j = b / 8;
  chunk = j % a.chunks;
  grp = (j / a.chunks) * 8 + b % 8;
  return grp < a.groups;
}

// A workgroup's tile is 16 MT rows by 64 NS columns (gated: 32 NS gate and the
// same 32 NS up columns): four waves, each MT row tiles by NS slices, the
// activations shared through LDS, each wave's weights straight to registers.
// Per 64-wide step a workgroup brings 2 MT KB of activations and 8 NS KB of
// weights into its CU for 2 MT NS matrix operations per wave; a CU takes about
// 64 bytes of activations and 73 of weights per ns (the fit in gemm_plan.hpp)
// whatever the pipeline (register- and LDS-direct-staged activations, one and
// two waves per SIMD: the same times), so what counts is the bytes per
// operation: tiles as large as still give every CU a workgroup.  Both staging
// and fragments run ahead:
//  * three LDS buffers, one barrier per step: while step b is multiplied, step
//    b + 2's activations go from registers to LDS, and step b + 1's first
//    fragments are read from the buffer that the last barrier completed;
//  * the fragments of half a step (32 of k) are read during the matrix
//    operations of the half before it, placed between them by the scheduling
//    groups (left alone the compiler reads one fragment, waits for it and
//    multiplies, some 120 cycles per three operations);
//  * activations are in flight for two to three steps, weights as well.
// llama2-7b, us, against 64-row chunks of two slices per wave without the
// read-ahead: gate/up with the activation at 256 rows 87-89 -> 65-71 (0.71
// PFLOP/s), at 128 66 -> 51, at 96 62 -> 47, at 64 46.6 -> 41.4, at 16 37 ->
// 34; QKV at 256 56.5 -> 41.5; down at 256 44 -> 40.
constexpr uint32_t kTileOob = 0x40000000u;   // past a slice (2^29 bytes) and 32 rows of x (2^30)

// sched_group_barrier classes
constexpr int kSgMfma = 0x008, kSgVmemRead = 0x020, kSgDsRead = 0x100, kSgDsWrite = 0x200;

// WAUX: the weight loads' cache policy, 2 (non-temporal) when each block is
// read once (one row chunk), 0 when another chunk reads it again from L2.
template <int MT, int NS, int WAUX, bool GATED>
__global__ void __launch_bounds__(256) tile_gemm_kernel(const GemmArgs a) {
  constexpr int KU = 2;
  constexpr int kXPer = (MT + 1) / 2;             // 32-row groups of the tile: one 16-byte piece per thread each
  constexpr int kRow = 64 * KU + 16;              // bytes per staged row
  constexpr int kBuf = 32 * kXPer * kRow;
  constexpr int kRows = 16 * MT;
  constexpr int kGate = GATED ? 2 * NS * MT * 512 : 0;
  static_assert(kGate <= 3 * kBuf, "gated exchange area");
  __shared__ __attribute__((aligned(16))) uint8_t lds[3 * kBuf];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, c16 = lane % 16, g4 = lane / 16;
  int32_t grp, chunk;
  if (!gemm_tile(a, grp, chunk)) return;
  const int32_t slice0 = GATED ? (w < 2 ? 2 * NS * grp + NS * w : a.gated / 16 + 2 * NS * grp + NS * (w - 2))
                               : (grp * 4 + w) * NS;
  const int32_t s_end = GATED ? (w < 2 ? a.gated / 16 : a.N / 16) : (a.N + 15) / 16;
  const int32_t t_begin = blockIdx.y * a.tc, t_end = min(a.kt, t_begin + a.tc);
  const uint32_t row_bytes = (uint32_t)a.K * 2u;
  __amdgpu_buffer_rsrc_t rw[NS], rx[kXPer];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int32_t slice = slice0 + i;
    rw[i] = uniform_rsrc(a.wp + ((int64_t)min(slice, s_end - 1) * a.kt + t_begin) * 512, slice < s_end ? (t_end - t_begin) * 1024 : 0);
  }
  const int32_t row0 = kRows * chunk, rows = min(kRows, a.rows - row0);
#pragma unroll
  for (int i = 0; i < kXPer; ++i) {
    const int32_t nr = max(0, min(32, rows - 32 * i));
    rx[i] = uniform_rsrc(a.x + (int64_t)(nr ? row0 + 32 * i : 0) * a.K, (int32_t)(nr * row_bytes));
  }
  gemm_f32x4 acc[NS][MT];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = gemm_f32x4{0.f, 0.f, 0.f, 0.f};

  const uint32_t xo = (uint32_t)(tid / 8) * row_bytes + (uint32_t)(tid % 8) * 16u + (uint32_t)t_begin * 64u;
  const int32_t xlim = min(4 * t_end, a.K / 8) - 4 * t_begin - tid % 8;   // batch b's piece is inside while 8 b < xlim
  const uint32_t wo = (uint32_t)lane * 16u;
  const int32_t nt = t_end - t_begin;
  auto issue_x = [&](int32_t b, u32x4 (&xr)[kXPer]) {
    const uint32_t off = 8 * b < xlim ? xo + 128u * (uint32_t)b : kTileOob;
#pragma unroll
    for (int i = 0; i < kXPer; ++i) xr[i] = gemm_load<0>(rx[i], off);
  };
  auto issue_w = [&](int32_t b, int u, u32x4 (&wr)[KU][NS]) {
    const int32_t t = KU * b + u;
    const uint32_t off = t < nt ? wo + 1024u * (uint32_t)t : kTileOob;
#pragma unroll
    for (int i = 0; i < NS; ++i) wr[u][i] = gemm_load<WAUX>(rw[i], off);
  };
  uint8_t* const st = lds + (tid / 8) * kRow + (tid % 8) * 16;
  auto stage = [&](int buf, const u32x4 (&xr)[kXPer]) {
#pragma unroll
    for (int i = 0; i < kXPer; ++i) *reinterpret_cast<u32x4*>(st + buf * kBuf + 32 * i * kRow) = xr[i];
  };
  const uint8_t* const ld = lds + c16 * kRow + g4 * 16;
  auto frag = [&](int buf, int u, u32x4 (&xb)[MT]) {
#pragma unroll
    for (int j = 0; j < MT; ++j) xb[j] = *reinterpret_cast<const u32x4*>(ld + buf * kBuf + 16 * j * kRow + 64 * u);
  };
  auto mult = [&](const u32x4 (&wv)[NS], const u32x4 (&xb)[MT]) {
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int i = 0; i < NS; ++i)
        acc[i][j] = gemm_mfma(wv[i], xb[j], acc[i][j]);
  };
  const int32_t n_batch = (nt + KU - 1) / KU;
  u32x4 xr[3][kXPer], wr[3][KU][NS], fa[MT], fb[MT];
  issue_x(0, xr[0]);
  issue_x(1, xr[1]);
  issue_w(0, 0, wr[0]);
  issue_w(0, 1, wr[0]);
  issue_x(2, xr[2]);
  issue_w(1, 0, wr[1]);
  issue_w(1, 1, wr[1]);
  issue_w(2, 0, wr[2]);
  stage(0, xr[0]);
  issue_x(3, xr[0]);
  stage(1, xr[1]);
  __syncthreads();
  frag(0, 0, fa);
#define BATON_TILE_STEP(B, Q)                                     \
  {                                                               \
    __builtin_amdgcn_sched_barrier(0);                            \
    frag((Q), 1, fb);                                             \
    issue_x((B) + 4, xr[((Q) + 1) % 3]);                          \
    issue_w((B) + 2, 1, wr[((Q) + 2) % 3]);                       \
    mult(wr[(Q)][0], fa);                                         \
    _Pragma("unroll") for (int z = 0; z < MT; ++z) {              \
      __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2, 0);      \
      __builtin_amdgcn_sched_group_barrier(kSgMfma, NS, 0);       \
      __builtin_amdgcn_sched_group_barrier(kSgVmemRead, 1, 0);    \
    }                                                             \
    __builtin_amdgcn_sched_barrier(0);                            \
    frag(((Q) + 1) % 3, 0, fa);                                   \
    stage(((Q) + 2) % 3, xr[((Q) + 2) % 3]);                      \
    issue_w((B) + 3, 0, wr[(Q)]);                                 \
    mult(wr[(Q)][1], fb);                                         \
    _Pragma("unroll") for (int z = 0; z < MT; ++z) {              \
      __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2, 0);      \
      if (z < kXPer) __builtin_amdgcn_sched_group_barrier(kSgDsWrite, 1, 0); \
      __builtin_amdgcn_sched_group_barrier(kSgMfma, NS, 0);       \
      if (z < NS) __builtin_amdgcn_sched_group_barrier(kSgVmemRead, 1, 0);  \
    }                                                             \
    __builtin_amdgcn_sched_barrier(0);                            \
    __syncthreads();                                              \
  }
  int32_t b = 0;
  for (; b + 3 <= n_batch; b += 3) {
    BATON_TILE_STEP(b, 0)
    BATON_TILE_STEP(b + 1, 1)
    BATON_TILE_STEP(b + 2, 2)
  }
  if (b < n_batch) BATON_TILE_STEP(b, 0)
  if (b + 1 < n_batch) BATON_TILE_STEP(b + 1, 1)
#undef BATON_TILE_STEP
  if constexpr (GATED) {
    gemm_gated_store<NS, MT>(a, lds, acc, w, lane, 2 * NS * grp + NS * (w % 2), row0, rows);
    return;
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int32_t n = 16 * (slice0 + i) + 4 * g4;
    if (n >= a.N) continue;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      const int32_t m = 16 * j + c16;
      if (m >= rows) continue;
      gemm_store(a, row0 + m, n, acc[i][j]);
    }
  }
}

// y[m][n] (+)= sum over the S splits of part[s][m][n], 4 outputs per thread,
// the splits added in order.
__global__ void __launch_bounds__(256) gemm_reduce_kernel(const float* __restrict__ part, uint16_t* __restrict__ y,
                                                          int32_t S, int64_t n_out, int32_t accumulate) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n_out) return;
  float4 v = *reinterpret_cast<const float4*>(part + i);
  for (int32_t s = 1; s < S; ++s) {
    const float4 p = *reinterpret_cast<const float4*>(part + s * n_out + i);
    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
  }
  uint2* yp = reinterpret_cast<uint2*>(y + i);
  if (accumulate) {
    const uint2 old = *yp;
    v.x += bf16_lo(old.x); v.y += bf16_hi(old.x); v.z += bf16_lo(old.y); v.w += bf16_hi(old.y);
  }
  *yp = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
}

// The split sums of a projection's output added up (and to the residual y
// with accumulate) as gemm_reduce_kernel does, then each row's RMS norm as
// rmsnorm_kernel does, element for element and in the same order: one
// workgroup per row, thread t owning the row's 8-element groups t, t +
// kRowThreads, ...  The result is bit-identical to the two launches, without
// the second one's read of y.
__global__ void __launch_bounds__(kRowThreads) reduce_rmsnorm_kernel(
    const float* __restrict__ part, uint16_t* __restrict__ y, int32_t S, int64_t n_out, int32_t accumulate,
    const u32x4* __restrict__ g, u32x4* __restrict__ yn, int32_t vec_per_row, float inv_dim, float eps) {
  __shared__ float psum[kRowThreads / kWave];
  const int64_t row = blockIdx.x;
  u32x4* yr = reinterpret_cast<u32x4*>(y) + row * vec_per_row;
  float ss = 0.f;
  u32x4 w0 = {0, 0, 0, 0};   // the thread's first group
  for (int i = threadIdx.x; i < vec_per_row; i += kRowThreads) {
    const int64_t e0 = (row * vec_per_row + i) * 8;   // the group's first element
    const u32x4 old = accumulate ? yr[i] : u32x4{0, 0, 0, 0};
    float4 v[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) v[hf] = *reinterpret_cast<const float4*>(part + e0 + 4 * hf);
    // the splits in order, four splits' loads in flight (past the last: the last again, not added)
    for (int32_t s0 = 1; s0 < S; s0 += 4) {
      float4 q[4][2];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
          q[u][hf] = *reinterpret_cast<const float4*>(part + min(s0 + u, S - 1) * n_out + e0 + 4 * hf);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (s0 + u >= S) break;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          v[hf].x += q[u][hf].x; v[hf].y += q[u][hf].y; v[hf].z += q[u][hf].z; v[hf].w += q[u][hf].w;
        }
      }
    }
    u32x4 w;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if (accumulate) {
        v[hf].x += bf16_lo(old[2 * hf]); v[hf].y += bf16_hi(old[2 * hf]);
        v[hf].z += bf16_lo(old[2 * hf + 1]); v[hf].w += bf16_hi(old[2 * hf + 1]);
      }
      w[2 * hf] = pack_bf16(v[hf].x, v[hf].y);
      w[2 * hf + 1] = pack_bf16(v[hf].z, v[hf].w);
    }
    if (i == (int)threadIdx.x) w0 = w;
    yr[i] = w;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = bf16_lo(w[j]), b = bf16_hi(w[j]);
      ss = fmaf(a, a, fmaf(b, b, ss));
    }
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) ss += __shfl_xor(ss, off, kWave);
  if (threadIdx.x % kWave == 0) psum[threadIdx.x / kWave] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kRowThreads / kWave; ++w) tot += psum[w];
  const float inv = 1.0f / sqrtf(tot * inv_dim + eps);
  for (int i = threadIdx.x; i < vec_per_row; i += kRowThreads) {
    const u32x4 w = i == (int)threadIdx.x ? w0 : yr[i], gw = g[i];   // this thread's own stores above
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = pack_bf16(bf16_lo(w[j]) * inv * bf16_lo(gw[j]), bf16_hi(w[j]) * inv * bf16_hi(gw[j]));
    yn[row * vec_per_row + i] = o;
  }
}

}  // namespace
}  // namespace baton
