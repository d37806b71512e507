// Host side of the decode-layer operations around the attention: the
// projections on the library's weight-streaming GEMM over packed weights (up
// to 256 rows), launches of the row and elementwise kernels.
// The C ABI is documented in include/baton.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>

#include "baton.h"
#include "layer_ops.hpp"
#include "packed_gemm.hpp"

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// How a product runs: the kernel, its tile, and the split along k.
enum GemmKind { kRowGemm, kSkinnyGemm, kTileGemm };
struct GemmPlan {
  GemmKind kind;
  int32_t mt, ns;       // row tiles of 16 per workgroup, weight slices per wave
  int32_t chunks;       // row chunks
  int32_t groups;       // slice groups
  int32_t tc, splits;   // 32-wide blocks per split, splits along k
};

// The plan of a product of `rows` rows with `slices` 16-row weight slices
// (gated: of gate slices, each with its up slice) of kt blocks, `max_splits`
// the most the workspace holds partial sums for.  The plan depends on the
// sizes alone, and gated products follow the same rule as ungated ones with
// one split where their sums must be the same bits: up to 8 rows every product
// divides k over its workgroup's waves alike, past that unsplit sums run along
// k in one chain in either kernel.
GemmPlan packed_gemm_plan(int32_t rows, int32_t slices, int32_t kt, bool gated, int32_t max_splits) {
  GemmPlan p;
  p.chunks = 1;
  p.splits = 1;
  if (rows <= 8) {
    // A workgroup per slice already divides k over its four waves; with fewer
    // than 64 slices (a quarter of the CUs) k is split further, at least 64
    // blocks each.  1 row, us, 1 / 2 / 4 splits: 512 x 8192 9.8 / 8.5 / 7.6,
    // but 1024 x 4096 6.6 / 7.1 / 7.8 and 2048 x 2048 5.4 / 7.3 / 9.6.
    p.kind = kRowGemm;
    p.mt = p.ns = 1;
    p.groups = slices;
    if (!gated && slices < 64) p.splits = std::min(4, kt / 64);
  } else if (rows <= 64 && !gated) {
    // With fewer than 512 slices (one per wave: two waves per SIMD), split
    // into about 1024 / slices ranges of at least 8 blocks each: at 64 rows
    // the split's partial sums and second launch cost more than they gain once
    // the slices alone give two waves per SIMD.
    p.kind = kSkinnyGemm;
    p.mt = (rows + 15) / 16;
    p.ns = 1;
    p.groups = (slices + baton::kGemmWaves - 1) / baton::kGemmWaves;
    if (slices < 512) p.splits = std::min((1024 + slices - 1) / slices, kt / 8);
  } else {
    // The tile (slices per wave) and the split that the measured costs favour:
    // a workgroup's step of 64 along k takes its CU about (2 mt + 8 ns) KB of
    // loads at 0.022 us a KB, the workgroups run in rounds of 256, and a split
    // costs a launch (4 us) and writes and reads its partial sums (5 TB/s).
    // llama2-7b, modelled / measured us: QKV at 256 rows 3 slices, 2 splits
    // 43 / 42 (2 slices, 1 split 46 / 46), down at 256 rows 2 slices, 4 splits
    // 41 / 40 (3 and 5: 44 / 45), QKV at 128 rows 2 and 2 31 / 33 (1 and 1
    // 34 / 34), gate/up at 128 rows 2 slices 45 / 51 (3: 56 / 62, 1: 67 / 61).
    p.kind = kTileGemm;
    p.chunks = rows > 128 ? 2 : 1;
    p.mt = (rows + 16 * p.chunks - 1) / (16 * p.chunks);
    double best = 0;
    p.ns = 0;
    const int32_t n_out = 16 * slices;
    for (int32_t ns = 1; ns <= (rows > 64 ? 3 : 2); ++ns) {
      const int32_t per = gated ? 2 * ns : 4 * ns, groups = (slices + per - 1) / per;
      for (int32_t s = 1; s <= (gated ? 1 : std::min(8, std::max(1, max_splits))); ++s) {
        const int32_t tc = (kt + s - 1) / s, sn = (kt + tc - 1) / tc;
        const int64_t rounds = ((int64_t)groups * p.chunks * sn + 255) / 256;
        const double us = 0.022 * rounds * ((tc + 1) / 2) * (2 * p.mt + 8 * ns) +
                          (sn > 1 ? 4 + 8e-6 / 5 * sn * rows * (double)n_out : 0);
        if (p.ns == 0 || us < best) {
          best = us;
          p.ns = ns;
          p.groups = groups;
          p.splits = sn;
        }
      }
    }
  }
  p.splits = std::max(1, std::min(p.splits, max_splits));
  p.tc = (kt + p.splits - 1) / p.splits;
  p.splits = (kt + p.tc - 1) / p.tc;
  return p;
}

template <int MT, int NS, bool GATED>
void launch_tile_ns(const baton::GemmArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(baton::kWave * baton::kGemmWaves);
  if constexpr (MT > 4) {
    if (a.chunks > 1) {
      hipLaunchKernelGGL((baton::tile_gemm_kernel<MT, NS, 0, GATED>), grid, block, 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((baton::tile_gemm_kernel<MT, NS, 2, GATED>), grid, block, 0, s, a);
}

template <int MT, bool GATED>
void launch_tile_mt(const baton::GemmArgs& a, int32_t ns, dim3 grid, hipStream_t s) {
  if constexpr (MT > 4 || GATED) {   // up to 64 rows gated products only
    if (ns == 1) return launch_tile_ns<MT, 1, GATED>(a, grid, s);
    if (ns == 2) return launch_tile_ns<MT, 2, GATED>(a, grid, s);
    if constexpr (MT > 4) launch_tile_ns<MT, 3, GATED>(a, grid, s);
  }
}

template <bool GATED>
void launch_tile(const baton::GemmArgs& a, const GemmPlan& p, dim3 grid, hipStream_t s) {
  switch (p.mt) {
    case 1: return launch_tile_mt<1, GATED>(a, p.ns, grid, s);
    case 2: return launch_tile_mt<2, GATED>(a, p.ns, grid, s);
    case 3: return launch_tile_mt<3, GATED>(a, p.ns, grid, s);
    case 4: return launch_tile_mt<4, GATED>(a, p.ns, grid, s);
    case 5: return launch_tile_mt<5, GATED>(a, p.ns, grid, s);
    case 6: return launch_tile_mt<6, GATED>(a, p.ns, grid, s);
    case 7: return launch_tile_mt<7, GATED>(a, p.ns, grid, s);
    default: return launch_tile_mt<8, GATED>(a, p.ns, grid, s);
  }
}

// Launches the product; a.x .. a.K, a.part, a.accumulate and a.gated are set.
// Returns the number of splits whose partial sums are still to be added.
int32_t launch_packed_gemm(baton::GemmArgs& a, int32_t max_splits, hipStream_t s) {
  const bool gated = a.gated > 0;
  a.kt = (a.K + 31) / 32;
  const GemmPlan p = packed_gemm_plan(a.rows, gated ? a.gated / 16 : (a.N + 15) / 16, a.kt, gated, max_splits);
  a.chunks = p.chunks;
  a.groups = p.groups;
  a.tc = p.tc;
  // with several chunks, whole sets of 8 groups (the kernel's XCD-aware dealing)
  const int64_t blocks = p.chunks == 1 ? p.groups : (int64_t)(p.groups + 7) / 8 * 8 * p.chunks;
  const dim3 grid((unsigned)blocks, (unsigned)p.splits), block(baton::kWave * baton::kGemmWaves);
  if (p.kind == kRowGemm) {
    if (gated) hipLaunchKernelGGL(baton::row_gemm_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(baton::row_gemm_kernel<false>, grid, block, 0, s, a);
  } else if (p.kind == kSkinnyGemm) {
    switch (p.mt) {
      case 1: hipLaunchKernelGGL(baton::skinny_gemm_kernel<1>, grid, block, 0, s, a); break;
      case 2: hipLaunchKernelGGL(baton::skinny_gemm_kernel<2>, grid, block, 0, s, a); break;
      case 3: hipLaunchKernelGGL(baton::skinny_gemm_kernel<3>, grid, block, 0, s, a); break;
      default: hipLaunchKernelGGL(baton::skinny_gemm_kernel<4>, grid, block, 0, s, a);
    }
  } else if (gated) {
    launch_tile<true>(a, p, grid, s);
  } else {
    launch_tile<false>(a, p, grid, s);
  }
  return p.splits;
}

}  // namespace

extern "C" {

size_t baton_linear_packed_bytes(int32_t out_dim, int32_t in_dim) {
  if (out_dim < 1 || in_dim < 1) return 0;
  return (size_t)((out_dim + 15) / 16) * 16 * (size_t)((in_dim + 31) / 32) * 32 * 2;
}

baton_status baton_linear_pack(int32_t dtype, const void* w, void* wp, int32_t out_dim, int32_t in_dim,
                               hipStream_t stream) {
  if (!w || !wp || out_dim < 1 || in_dim < 1 || in_dim % 8 || out_dim % 8) return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(w) || !aligned16(wp) || in_dim > (1 << 24)) return BATON_EINVAL;
  const int32_t kt = (in_dim + 31) / 32;
  const int64_t n_pieces = (int64_t)((out_dim + 15) / 16) * kt * baton::kWave;
  hipLaunchKernelGGL(baton::pack_weight_kernel, dim3((unsigned)((n_pieces + 255) / 256)), dim3(256), 0, stream,
                     static_cast<const baton::u32x4*>(w), static_cast<baton::u32x4*>(wp), out_dim, in_dim, kt,
                     n_pieces);
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

}  // extern "C"

namespace {

// baton_linear_packed, and with gain the RMS norm of its output rows into
// y_norm (the split sums added and each row normalised by one kernel when the
// product splits along k).
baton_status linear_packed(int32_t dtype, const void* x, const void* wp, void* y, int32_t rows, int32_t out_dim,
                           int32_t in_dim, int32_t accumulate, const void* gain, float eps, void* y_norm, void* ws,
                           size_t ws_bytes, hipStream_t stream) {
  if (!x || !wp || !y || rows < 1 || rows > BATON_GEMM_MAX_ROWS || out_dim < 1 || in_dim < 1 || (ws_bytes && !ws))
    return BATON_EINVAL;
  if (gain && (!y_norm || !aligned16(gain) || !aligned16(y_norm) || !(eps >= 0.f) || !std::isfinite(eps)))
    return BATON_EINVAL;
  if (accumulate != 0 && accumulate != 1) return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(x) || !aligned16(wp) || !aligned16(y) || in_dim % 8 || out_dim % 8 || in_dim > (1 << 24))
    return BATON_EINVAL;
  baton::GemmArgs a;
  a.x = static_cast<const uint16_t*>(x);
  a.wp = static_cast<const uint16_t*>(wp);
  a.y = static_cast<uint16_t*>(y);
  a.part = static_cast<float*>(ws);
  a.rows = rows;
  a.N = out_dim;
  a.K = in_dim;
  a.accumulate = accumulate;
  a.gated = 0;
  // as many splits along k as the workspace holds partial sums for
  const size_t per_split = (size_t)rows * out_dim * sizeof(float);
  const int32_t max_splits = ws && aligned16(ws) ? (int32_t)std::min<size_t>(ws_bytes / per_split, 1024) : 1;
  const int32_t S = launch_packed_gemm(a, max_splits, stream);
  const int64_t n_out = (int64_t)rows * out_dim;
  if (S > 1 && gain) {
    hipLaunchKernelGGL(baton::reduce_rmsnorm_kernel, dim3(rows), dim3(baton::kRowThreads), 0, stream, a.part, a.y, S,
                       n_out, accumulate, static_cast<const baton::u32x4*>(gain),
                       static_cast<baton::u32x4*>(y_norm), out_dim / 8, 1.0f / out_dim, eps);
  } else {
    if (S > 1)
      hipLaunchKernelGGL(baton::gemm_reduce_kernel, dim3((unsigned)((n_out / 4 + 255) / 256)), dim3(256), 0, stream,
                         a.part, a.y, S, n_out, accumulate);
    if (gain)
      hipLaunchKernelGGL(baton::rmsnorm_kernel, dim3(rows), dim3(baton::kRowThreads), 0, stream,
                         static_cast<const baton::u32x4*>(y), static_cast<const baton::u32x4*>(gain),
                         static_cast<baton::u32x4*>(y_norm), out_dim / 8, 1.0f / out_dim, eps);
  }
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

}  // namespace

extern "C" {

baton_status baton_linear_packed(int32_t dtype, const void* x, const void* wp, void* y, int32_t rows,
                                 int32_t out_dim, int32_t in_dim, int32_t accumulate, void* ws, size_t ws_bytes,
                                 hipStream_t stream) {
  return linear_packed(dtype, x, wp, y, rows, out_dim, in_dim, accumulate, nullptr, 0.f, nullptr, ws, ws_bytes,
                       stream);
}

baton_status baton_linear_packed_rmsnorm(int32_t dtype, const void* x, const void* wp, void* y, int32_t rows,
                                         int32_t out_dim, int32_t in_dim, int32_t accumulate, const void* gain,
                                         float eps, void* y_norm, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (!gain) return BATON_EINVAL;
  return linear_packed(dtype, x, wp, y, rows, out_dim, in_dim, accumulate, gain, eps, y_norm, ws, ws_bytes,
                       stream);
}

baton_status baton_linear_packed_silu(int32_t dtype, const void* x, const void* wp, void* y, int32_t rows,
                                      int32_t out_dim, int32_t in_dim, hipStream_t stream) {
  if (!x || !wp || !y || rows < 1 || rows > BATON_GEMM_MAX_ROWS || out_dim < 32 || out_dim % 32 || in_dim < 8 ||
      in_dim % 8 || in_dim > (1 << 24))
    return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(x) || !aligned16(wp) || !aligned16(y)) return BATON_EINVAL;
  baton::GemmArgs a;
  a.x = static_cast<const uint16_t*>(x);
  a.wp = static_cast<const uint16_t*>(wp);
  a.y = static_cast<uint16_t*>(y);
  a.part = nullptr;
  a.rows = rows;
  a.N = out_dim;
  a.K = in_dim;
  a.accumulate = 0;
  a.gated = out_dim / 2;   // never split along k: the epilogue needs the whole sum
  launch_packed_gemm(a, 1, stream);
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

baton_status baton_rmsnorm(int32_t dtype, const void* x, const void* gain, void* y, int32_t rows, int32_t dim,
                           float eps, hipStream_t stream) {
  if (!x || !gain || !y || rows < 1 || dim < 8 || dim % 8 || !(eps >= 0.f) || !std::isfinite(eps)) return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(x) || !aligned16(gain) || !aligned16(y)) return BATON_EINVAL;
  hipLaunchKernelGGL(baton::rmsnorm_kernel, dim3(rows), dim3(baton::kRowThreads), 0, stream,
                     static_cast<const baton::u32x4*>(x), static_cast<const baton::u32x4*>(gain),
                     static_cast<baton::u32x4*>(y), dim / 8, 1.0f / dim, eps);
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

baton_status baton_silu_mul(int32_t dtype, const void* gate_up, void* out, int32_t rows, int32_t dim,
                            hipStream_t stream) {
  if (!gate_up || !out || rows < 1 || dim < 8 || dim % 8) return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(gate_up) || !aligned16(out)) return BATON_EINVAL;
  const int64_t n_vec = (int64_t)rows * (dim / 8);
  hipLaunchKernelGGL(baton::silu_mul_kernel, dim3((unsigned)((n_vec + 255) / 256)), dim3(256), 0, stream,
                     static_cast<const baton::u32x4*>(gate_up), static_cast<baton::u32x4*>(out), dim / 8, n_vec);
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

}  // extern "C"
