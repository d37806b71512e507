// Row and elementwise kernels of a decode layer around the attention: RMS
// normalisation, the fused projection's split with rotary embedding of
// queries and keys, and the gated activation.  bf16 storage, fp32
// arithmetic, outputs rounded to nearest even.
#pragma once

#include "common.hpp"

namespace baton {
namespace {   // internal linkage: the kernels are included by two translation units

// Threads of a row's workgroup in the norms.  What bounds them is latency, one
// workgroup per row: with 512 a row of 4096 is one 16-byte vector per thread, read
// (in reduce_rmsnorm_kernel with all its split sums) in one round and kept in
// registers for the second pass.  Against 256
// threads reading twice, whole llama2-7b layers: 585.0 -> 580.0 us for two at 64
// rows, 206.9 -> 203.5 at one; the feed-forward block at 256 rows 113.9 -> 110.3.
// (rmsnorm_kernel alone takes 256 for many short rows, norm_threads.)
constexpr int kRowThreads = 512;

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
}

// y[r] = x[r] / sqrt(mean(x[r]^2) + eps) * g, one workgroup of NT threads per
// row; dim a multiple of 8 (16-byte vectors).  Rows of at most 256 vectors have
// the same bits with 256 threads as with more, whose sums are zeros.
template <int NT>
__global__ void __launch_bounds__(NT) rmsnorm_kernel(const u32x4* __restrict__ x, const u32x4* __restrict__ g,
                                                     u32x4* __restrict__ y, int32_t vec_per_row, float inv_dim,
                                                     float eps) {
  __shared__ float part[NT / kWave];
  const int64_t row = blockIdx.x;
  const u32x4* xr = x + row * vec_per_row;
  float ss = 0.f;
  u32x4 w0 = {0, 0, 0, 0};   // the thread's first vector
  for (int i = threadIdx.x; i < vec_per_row; i += NT) {
    const u32x4 w = xr[i];
    if (i == (int)threadIdx.x) w0 = w;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = bf16_lo(w[j]), b = bf16_hi(w[j]);
      ss = fmaf(a, a, fmaf(b, b, ss));
    }
  }
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) ss += __shfl_xor(ss, off, kWave);
  if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) tot += part[w];
  const float inv = 1.0f / sqrtf(tot * inv_dim + eps);
  for (int i = threadIdx.x; i < vec_per_row; i += NT) {
    const u32x4 w = i == (int)threadIdx.x ? w0 : xr[i], gw = g[i];
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = pack_bf16(bf16_lo(w[j]) * inv * bf16_lo(gw[j]), bf16_hi(w[j]) * inv * bf16_hi(gw[j]));
    y[row * vec_per_row + i] = o;
  }
}

// Split of the fused projection qkv [B][(Hq + 2 Hkv) D] into q [B][Hq][D],
// k [B][Hkv][D] (both rotated) and v [B][Hkv][D].  One wave per (row, head):
// lane i < D/2 rotates pair (i, i + D/2) by pos_b * theta^(-2i/D).  The angle
// is formed and reduced modulo 2 pi in double precision, its sine and cosine
// then taken in single precision on [-pi, pi].
struct RopeArgs {
  const uint16_t* qkv;
  uint16_t* q;
  uint16_t* k;
  uint16_t* v;
  int32_t n_q_heads, n_kv_heads, head_dim;
  double log2_theta;
  int32_t pos[512];
};

__global__ void __launch_bounds__(kWave) rope_qkv_kernel(const RopeArgs a) {
  const int hq = a.n_q_heads, hkv = a.n_kv_heads, D = a.head_dim, half = D / 2;
  const int heads = hq + 2 * hkv;
  const int b = blockIdx.x / heads, head = blockIdx.x - b * heads;
  const uint16_t* src = a.qkv + ((int64_t)b * heads + head) * D;
  const int i = threadIdx.x;
  if (head >= hq + hkv) {                      // a value head: copied
    uint16_t* dst = a.v + ((int64_t)b * hkv + (head - hq - hkv)) * D;
    for (int e = i; e < D; e += kWave) dst[e] = src[e];
    return;
  }
  if (i >= half) return;
  const double inv = exp2(-(double)(2 * i) / D * a.log2_theta);
  const double two_pi = 6.283185307179586;
  double ang = (double)a.pos[b] * inv;
  ang -= two_pi * rint(ang / two_pi);
  float s, c;
  sincosf((float)ang, &s, &c);
  const float x0 = __uint_as_float((uint32_t)src[i] << 16);
  const float x1 = __uint_as_float((uint32_t)src[i + half] << 16);
  uint16_t* dst = head < hq ? a.q + ((int64_t)b * hq + head) * D : a.k + ((int64_t)b * hkv + (head - hq)) * D;
  dst[i] = (uint16_t)f32_to_bf16_rne(x0 * c - x1 * s);
  dst[i + half] = (uint16_t)f32_to_bf16_rne(x0 * s + x1 * c);
}

// silu(gate) * up of four packed bf16 pairs, rounded to bf16.
__device__ __forceinline__ uint2 silu_mul4(uint2 g, uint2 u) {
  const uint32_t gw[2] = {g.x, g.y}, uw[2] = {u.x, u.y};
  uint32_t o[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float g0 = bf16_lo(gw[q]), g1 = bf16_hi(gw[q]);
    const float s0 = g0 / (1.f + expf(-g0)), s1 = g1 / (1.f + expf(-g1));
    o[q] = pack_bf16(s0 * bf16_lo(uw[q]), s1 * bf16_hi(uw[q]));
  }
  return make_uint2(o[0], o[1]);
}

// out[r][j] = silu(gate_up[r][j]) * gate_up[r][F + j], 8 elements per thread.
__global__ void __launch_bounds__(256) silu_mul_kernel(const u32x4* __restrict__ gu, u32x4* __restrict__ out,
                                                       int32_t vec_per_row, int64_t n_vec) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_vec) return;
  const int64_t r = i / vec_per_row, c = i - r * vec_per_row;
  const u32x4 g = gu[r * 2 * vec_per_row + c], u = gu[r * 2 * vec_per_row + vec_per_row + c];
  const uint2 lo = silu_mul4(make_uint2(g[0], g[1]), make_uint2(u[0], u[1]));
  const uint2 hi = silu_mul4(make_uint2(g[2], g[3]), make_uint2(u[2], u[3]));
  out[i] = u32x4{lo.x, lo.y, hi.x, hi.y};
}

}  // namespace
}  // namespace baton
