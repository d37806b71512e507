// How a packed product (packed_gemm.hpp) runs -- the kernel, its tile and the
// split along k -- and a row norm, from the sizes alone.  Host code without a GPU header, so that
// the rule can be evaluated on its own.
#pragma once

#include <algorithm>
#include <cstdint>

namespace baton {

constexpr int32_t kGemmWaves = 4;   // waves per workgroup

enum GemmKind { kRowGemm, kSkinnyGemm, kTileGemm };
struct GemmPlan {
  GemmKind kind;
  int32_t mt, ns;       // row tiles of 16 per workgroup, weight slices per wave
  int32_t chunks;       // row chunks
  int32_t groups;       // slice groups
  int32_t tc, splits;   // 32-wide blocks per split, splits along k
};

// The tile_gemm_kernel forms that exist: with one row chunk of up to 64 rows
// gated products only, of one or two slices per wave; chunks of 48 rows or more
// otherwise.
constexpr bool tile_gemm_built(int32_t mt, int32_t ns, int32_t chunks, bool gated) {
  return mt >= 1 && mt <= 8 && ns >= 1 && ns <= 3 && (mt > 4 || (chunks > 1 ? mt > 2 : gated && ns <= 2));
}

// Up to 8 rows: row_gemm_kernel (a workgroup per slice, k over its four waves)
// or skinny_gemm_kernel (a wave per slice).  Both sides measured over outputs
// of 192 .. 128,256 and in of 64 .. 20,480 at 1 and 8 rows; us below at 1 row,
// the row kernel first, outputs x in (gated: rows of [gate; up]).
inline bool row_kernel(int32_t rows, int32_t slices, int32_t kt, bool gated) {
  // Its launch has a workgroup, 256 threads, per slice, of less than 2^32 in all.
  if (slices >= 1 << 24) return false;
  const int32_t groups = gated ? (slices + 1) / 2 : (slices + kGemmWaves - 1) / kGemmWaves;   // of the staged kernel
  // Short k leaves a wave a fraction of its eight pairs of loads, all of which
  // it issues: 4096 x 256 4.2 / 3.4, x 512 4.4 / 4.3, x 1024 4.7 / 5.7; 8192 x
  // 512 6.5 / 4.7, x 1536 8.4 / 8.1, x 2048 9.3 / 9.8; gated 4096 x 512 5.9 /
  // 5.0, x 1024 6.3 / 6.3, x 2048 7.3 / 9.3, 8192 x 1024 7.3 / 7.0, x 1536
  // 8.4 / 8.7.
  if (groups <= 64) return kt >= (gated ? 30 : 16);
  if (groups <= 128) return kt >= (gated ? 40 : 50);
  // Few rows, plain, slices an odd multiple of 128 KB apart, which the staged
  // kernel reads 8% slower than its neighbours and this one, in whole rounds of
  // its loads, does not: 12288 x 4096 19.1 / 20.7, x 4064 20.9 / 19.9, x 4160
  // 21.8 / 19.4, x 8192 35.3 / 33.6, x 12288 48.5 / 51.4, 32000 x 4096 0.92 of
  // the time; but gated 12288 x 4096 21.8 / 19.5, and at 8 rows 20.2 / 20.5.
  if (!gated && rows <= 4 && kt % 256 == 128) return true;
  // One round of the staged kernel on more than half of the CUs: 10240 x 2048
  // 12.0 / 10.3, x 8192 32.2 / 29.7, 16384 x 512 11.0 / 5.7, x 11008 58.8 /
  // 56.0; gated 10240 x 4096 20.8 / 17.7.
  if (groups <= 256) return false;
  // Several rounds, the last of them poorly filled: 18432 x 2048 18.3 / 20.2, x
  // 4096 28.7 / 38.0, 22016 x 4096 33.1 / 38.2, x 8192 60.7 / 68.7, gated 58.9 /
  // 68.3; 36864 x 4096 0.82 of the time, 40960 0.86.  Well filled: 32768 x 2048
  // 1.13 times, x 8192 1.00, 65536 x 5120 1.10.  Short k: 18432 x 1536 16.7 /
  // 15.9, 22016 x 1024 17.2 / 11.9, x 2048 20.7 / 20.4.
  const int64_t room = (int64_t)(groups + 255) / 256 * 256;
  return 2 * room >= 3 * (int64_t)groups ? kt >= 64 : 5 * room >= 6 * (int64_t)groups && kt >= 128;
}

// Splits along k of row_gemm_kernel with a few slices.  A wave runs its quarter
// of the range in rounds of 16 blocks, about 1.6 us each; a second launch and
// the partial sums cost about 1.5, with many slices more.  So up to one round
// per wave and one workgroup per CU, the fewest ranges that give that many
// rounds, and only where that saves enough of them.  1 row, us, 1 / 2 / 3 / 4 /
// 8 splits: 512 x 4096 5.8 / 5.9 / 6.0 / 6.3 / 7.0, x 6144 7.7 / 7.6 / 6.1 / 6.5
// / 7.2, x 16384 15.3 / 11.0 / 9.9 / 8.7 / 8.7; 1024 x 16384 16.2 / 12.3 / 11.2
// / 11.5 / 13.4; 2048 x 8192 10.6 / 10.6, x 11008 14.0 / 12.3 / 14.5; 192 x 4096
// 5.8 / 5.8, at 8 rows 6.8 / 6.4.
inline int32_t row_splits(int32_t slices, int32_t kt, int32_t max_splits) {
  auto rounds = [&](int32_t s) {
    const int32_t pairs = ((kt + s - 1) / s + 1) / 2;
    return ((pairs + kGemmWaves - 1) / kGemmWaves + 7) / 8;
  };
  const int32_t most = std::min({(kt + 63) / 64, 256 / slices, 8, max_splits});
  if (most < 2 || rounds(1) - rounds(most) < (slices <= 24 ? 1 : slices < 128 ? 2 : 3)) return 1;
  int32_t s = 1;
  while (rounds(s) > rounds(most)) ++s;
  return s;
}

// The plan of a product of `rows` rows with `slices` 16-row weight slices
// (gated: of gate slices, each with its up slice), `max_splits` the most the
// workspace holds partial sums for.  The plan depends on the
// sizes alone.  Any kernel it may take for a row count sums an unsplit product
// in the same order, gated or not, so the choice never changes its bits.
inline GemmPlan packed_gemm_plan(int32_t rows, int32_t slices, int32_t in_dim, bool gated, int32_t max_splits) {
  const int32_t kt = (in_dim + 31) / 32;   // 32-wide blocks
  GemmPlan p;
  p.chunks = 1;
  p.splits = 1;
  if (rows <= 8) {
    p.mt = p.ns = 1;
    p.kind = row_kernel(rows, slices, kt, gated) ? kRowGemm : kSkinnyGemm;
    if (p.kind == kRowGemm && !gated && max_splits > 1) {
      if (slices > 256 && slices <= 384 && kt >= 96 && (kt >= 160 || kt % 64)) {
        // Up to 1.5 workgroups per CU of the kernel with a slice per
        // workgroup: the second round is half empty.  The staged kernel in two
        // ranges of k, 1 row, us, row kernel / this: 5120 x 3072 11.1 / 10.8,
        // 6144 x 5120 16.2 / 15.4, 6144 x 16384 41.9 / 35.5; but 6144 x 4096
        // (whole rounds of the row kernel's loads) 12.5 / 14.7, and 7168 x 8192
        // 23.0 / 24.9.
        p.kind = kSkinnyGemm;
        p.splits = 2;
      } else if (slices <= 128) {
        p.splits = row_splits(slices, kt, max_splits);
      }
    }
    p.groups = p.kind == kRowGemm ? slices : gated ? (slices + 1) / 2 : (slices + kGemmWaves - 1) / kGemmWaves;
  } else if (rows <= 64 && !gated) {
    // With fewer than 512 slices (one per wave: two waves per SIMD), split
    // into about 1024 / slices ranges of at least 8 blocks each: at 64 rows
    // the split's partial sums and second launch cost more than they gain once
    // the slices alone give two waves per SIMD.
    p.kind = kSkinnyGemm;
    p.mt = (rows + 15) / 16;
    p.ns = 1;
    p.groups = (slices + kGemmWaves - 1) / kGemmWaves;
    if (slices < 512) p.splits = std::min((1024 + slices - 1) / slices, kt / 8);
  } else if (rows <= 64) {
    // Gated.  As long as the staged kernel's workgroups make one round, its four
    // blocks per barrier against the tile's two, one slice per wave in both: 16
    // rows, us, staged / tile, gate and up rows x in: 1024 x 8192 26.5 / 32.1,
    // 8192 x 4096 17.2 / 20.0, x 896 7.0 / 7.4 (14144), x 512 5.1 / 5.0, 16384 x 4096
    // 24.6 / 24.8; 64 rows, whose activations the tile reads ahead, 4096 x 8192
    // 40.2 / 42.1, x 2048 13.4 / 13.2, x 1024 8.9 / 8.7.
    p.groups = (slices + 1) / 2;
    p.mt = (rows + 15) / 16;
    p.ns = 1;
    if (p.groups <= 256 && kt >= (rows <= 48 ? 24 : 128)) {
      p.kind = kSkinnyGemm;
    } else {
      // Two slices per wave where that makes one round of two and a workgroup
      // has enough work: one / two, us, 22016 x 4096 at 9 rows 32.8 / 34.1, 32
      // 37.2 / 36.1, 64 44.9 / 40.9, x 8192 at 16 65.2 / 63.3, at 32 70.9 / 66.2;
      // 26304 x 3216 at 48 40.7 / 35.3; two over one at 64 rows of 512 in 1.00 to
      // 1.10, of 1024 0.95 to 0.99; 30720 x 4096 at 64 1.01, x 8192 0.89; more
      // rounds, 36864 and up, 1.02 to 1.24 at any k.
      p.kind = kTileGemm;
      if (p.groups > 256 && p.groups <= 512 &&
          (rows > 32 ? kt >= (p.groups <= 430 ? 24 : 200) : rows > 16 && kt >= 200)) {
        p.ns = 2;
        p.groups = (slices + 3) / 4;
      }
    }
  } else {
    // The row chunks, slices per wave and split that the measured costs favour.
    // The workgroups run in rounds of one per CU: 256, or 32 per XCD where the
    // chunks of a group share one.  A workgroup takes 0.13 mt ns us for its start
    // and outputs and, for each step of 64 along k (2 mt KB of activations, 8 ns KB
    // of weights), 0.021 + 0.032 mt + 0.112 ns, with rows of x that do not start on
    // 128 bytes 0.041 mt, and 0.02 more where chunks share the weights; a split
    // costs a launch, 0.37 us per range and its partial sums (at 10 TB/s: they stay
    // in the caches).  Fitted to 60,000 launches (65 to 256 rows, 192 to 32,768
    // outputs of 64 to 16,384, all chunks, slices and splits), of which the choice
    // is within 1.1% of the best on average.  us, chunks of up to 128 rows and up
    // to 8 splits / this: 128 rows 1024 x 16384 22.8 / 19.1, 512 x 16384 21.8 /
    // 17.8, 256 rows 1536 x 4096 19.3 / 16.3, 256 rows 2592 x 8368 43.9 / 29.8,
    // gated 160 rows 10240 x 4096 39.7 / 34.5.
    p.kind = kTileGemm;
    double best = -1;
    const double n_out = 16.0 * slices * rows, x_cost = in_dim % 64 ? 0.041 : 0.032;
    // A step or two of k: the launch is its start and its outputs, and many small
    // workgroups overlap them: 256 rows 16384 x 64 8.3 / 6.8 us.
    const bool short_k = kt <= 4 && slices < 1 << 20;
    const int32_t c_lo = short_k ? (rows + 63) / 64 : (rows + 127) / 128, c_hi = short_k ? c_lo : (rows + 47) / 48;
    for (int32_t c = c_lo; c <= c_hi; ++c) {
      const int32_t mt = (rows + 16 * c - 1) / (16 * c);
      if ((c - 1) * mt * 16 >= rows) continue;   // the last chunk would be empty
      for (int32_t ns = 1; ns <= (short_k ? 1 : 3); ++ns) {
        const int32_t per = gated ? 2 * ns : kGemmWaves * ns, groups = (slices + per - 1) / per;
        for (const int32_t s : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20}) {
          if (s > 1 && (gated || short_k || s > max_splits || s > kt / 4 || (int64_t)groups * c * s > 768)) break;
          const int32_t tc = (kt + s - 1) / s, sn = (kt + tc - 1) / tc;
          const int64_t rounds = c == 1 ? ((int64_t)groups * sn + 255) / 256 : ((int64_t)(groups + 7) / 8 * c * sn + 31) / 32;
          const double step = (c > 1 ? 0.041 : 0.021) + x_cost * mt + 0.112 * ns;
          const double us = rounds * (0.13 * mt * ns + (tc + 1) / 2 * step) +
                            (sn > 1 ? 1.6 + 0.37 * sn + 8.3e-7 * sn * n_out : 0);
          if (best < 0 || us < best) {
            best = us;
            p.chunks = c;
            p.mt = mt;
            p.ns = ns;
            p.groups = groups;
            p.splits = sn;
          }
        }
      }
    }
  }
  p.splits = std::max(1, std::min(p.splits, max_splits));
  p.tc = (kt + p.splits - 1) / p.splits;
  p.splits = (kt + p.tc - 1) / p.tc;
  return p;
}

// Threads of rmsnorm_kernel's workgroups, one per row: 512 read a row of 4096 in
// one round, but where rows fill the GPU and leave half of them idle 256 let more
// rows run at once.  512 / 256 threads, us: 1024 rows of 2048 3.79 / 3.71, of 512
// 3.09 / 2.89, 16,384 of 512 15.2 / 11.0, of 2048 26.4 / 23.4; but 256 rows of 2048
// 2.83 / 2.90, 1024 of 4096 5.00 / 5.13.  And a launch has less than 2^32 threads.
inline int32_t norm_threads(int32_t rows, int32_t dim) {
  return rows > 512 && (dim <= 2048 || rows >= 1 << 23) ? 256 : 512;
}

}  // namespace baton
