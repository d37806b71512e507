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

// Launches of one form; false: the form does not exist, nothing is launched.
template <int MT, int NS, bool GATED>
bool launch_tile_ns(const baton::GemmArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(baton::kWave * baton::kGemmWaves);
  if (a.chunks > 1) {
    if constexpr (baton::tile_gemm_built(MT, NS, 2, GATED)) {
      hipLaunchKernelGGL((baton::tile_gemm_kernel<MT, NS, 0, GATED>), grid, block, 0, s, a);
      return true;
    }
  } else if constexpr (baton::tile_gemm_built(MT, NS, 1, GATED)) {
    hipLaunchKernelGGL((baton::tile_gemm_kernel<MT, NS, 2, GATED>), grid, block, 0, s, a);
    return true;
  }
  return false;
}

template <int MT, bool GATED>
bool launch_tile_mt(const baton::GemmArgs& a, int32_t ns, dim3 grid, hipStream_t s) {
  switch (ns) {
    case 1: return launch_tile_ns<MT, 1, GATED>(a, grid, s);
    case 2: return launch_tile_ns<MT, 2, GATED>(a, grid, s);
    case 3: return launch_tile_ns<MT, 3, GATED>(a, grid, s);
    default: return false;
  }
}

template <bool GATED>
bool launch_tile(const baton::GemmArgs& a, const baton::GemmPlan& p, dim3 grid, hipStream_t s) {
  switch (p.mt) {
    case 1: return launch_tile_mt<1, GATED>(a, p.ns, grid, s);
    case 2: return launch_tile_mt<2, GATED>(a, p.ns, grid, s);
    case 3: return launch_tile_mt<3, GATED>(a, p.ns, grid, s);
    case 4: return launch_tile_mt<4, GATED>(a, p.ns, grid, s);
    case 5: return launch_tile_mt<5, GATED>(a, p.ns, grid, s);
    case 6: return launch_tile_mt<6, GATED>(a, p.ns, grid, s);
    case 7: return launch_tile_mt<7, GATED>(a, p.ns, grid, s);
    case 8: return launch_tile_mt<8, GATED>(a, p.ns, grid, s);
    default: return false;
  }
}

template <bool GATED>
bool launch_skinny(const baton::GemmArgs& a, const baton::GemmPlan& p, dim3 grid, hipStream_t s) {
  const dim3 block(baton::kWave * baton::kGemmWaves);
  if (a.rows <= 8) {
    hipLaunchKernelGGL((baton::skinny_gemm_kernel<1, GATED, true>), grid, block, 0, s, a);
    return true;
  }
  switch (p.mt) {
    case 1: hipLaunchKernelGGL((baton::skinny_gemm_kernel<1, GATED, false>), grid, block, 0, s, a); return true;
    case 2: hipLaunchKernelGGL((baton::skinny_gemm_kernel<2, GATED, false>), grid, block, 0, s, a); return true;
    case 3: hipLaunchKernelGGL((baton::skinny_gemm_kernel<3, GATED, false>), grid, block, 0, s, a); return true;
    case 4: hipLaunchKernelGGL((baton::skinny_gemm_kernel<4, GATED, false>), grid, block, 0, s, a); return true;
    default: return false;
  }
}

// Launches the product; a.x .. a.K, a.part, a.accumulate and a.gated are set.
// Returns the number of splits whose partial sums are still to be added (1:
// none), 0 if the plan's form of the kernel does not exist.
int32_t launch_packed_gemm(baton::GemmArgs& a, int32_t max_splits, hipStream_t s) {
  const bool gated = a.gated > 0;
  a.kt = (a.K + 31) / 32;
  const baton::GemmPlan p =
      baton::packed_gemm_plan(a.rows, gated ? a.gated / 16 : (a.N + 15) / 16, a.K, gated, max_splits);
  a.chunks = p.chunks;
  a.groups = p.groups;
  a.tc = p.tc;
  // with several chunks, whole sets of 8 groups (the kernel's XCD-aware dealing)
  const int64_t blocks = p.chunks == 1 ? p.groups : (int64_t)(p.groups + 7) / 8 * 8 * p.chunks;
  const dim3 grid((unsigned)blocks, (unsigned)p.splits), block(baton::kWave * baton::kGemmWaves);
  bool built = true;
  if (p.kind == baton::kRowGemm) {
    if (gated) hipLaunchKernelGGL(baton::row_gemm_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(baton::row_gemm_kernel<false>, grid, block, 0, s, a);
  } else if (p.kind == baton::kSkinnyGemm) {
    built = gated ? launch_skinny<true>(a, p, grid, s) : launch_skinny<false>(a, p, grid, s);
  } else {
    built = gated ? launch_tile<true>(a, p, grid, s) : launch_tile<false>(a, p, grid, s);
  }
  return built ? p.splits : 0;
}

void launch_rmsnorm(const void* x, const void* gain, void* y, int32_t rows, int32_t dim, float eps, hipStream_t s) {
  auto launch = [&](auto kernel, int32_t threads) {
    hipLaunchKernelGGL(kernel, dim3(rows), dim3(threads), 0, s, static_cast<const baton::u32x4*>(x),
                       static_cast<const baton::u32x4*>(gain), static_cast<baton::u32x4*>(y), dim / 8, 1.0f / dim, eps);
  };
  static_assert(baton::kRowThreads == 512, "norm_threads' larger choice");
  if (baton::norm_threads(rows, dim) == 256) launch(baton::rmsnorm_kernel<256>, 256);
  else launch(baton::rmsnorm_kernel<baton::kRowThreads>, baton::kRowThreads);
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
  if (S < 1) return BATON_EINVAL;
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
      launch_rmsnorm(y, gain, y_norm, rows, out_dim, eps, stream);
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
  if (launch_packed_gemm(a, 1, stream) < 1) return BATON_EINVAL;
  return hipGetLastError() == hipSuccess ? BATON_OK : BATON_EHIP;
}

baton_status baton_rmsnorm(int32_t dtype, const void* x, const void* gain, void* y, int32_t rows, int32_t dim,
                           float eps, hipStream_t stream) {
  if (!x || !gain || !y || rows < 1 || dim < 8 || dim % 8 || !(eps >= 0.f) || !std::isfinite(eps)) return BATON_EINVAL;
  if (dtype != BATON_BF16) return BATON_EDTYPE;
  if (!aligned16(x) || !aligned16(gain) || !aligned16(y)) return BATON_EINVAL;
  launch_rmsnorm(x, gain, y, rows, dim, eps, stream);
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
