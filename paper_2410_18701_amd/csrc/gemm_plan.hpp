// How a packed product (packed_gemm.hpp) runs: the kernel, its tile and the
// split along k, from the sizes alone.  Host code without a GPU header, so that
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

// The tile_gemm_kernel forms that exist: up to 64 rows gated products only, of
// one or two slices per wave and one row chunk.
constexpr bool tile_gemm_built(int32_t mt, int32_t ns, int32_t chunks, bool gated) {
  return mt >= 1 && mt <= 8 && ns >= 1 && (mt > 4 ? ns <= 3 : gated && ns <= 2 && chunks == 1);
}

// The plan of a product of `rows` rows with `slices` 16-row weight slices
// (gated: of gate slices, each with its up slice) of kt blocks, `max_splits`
// the most the workspace holds partial sums for.  The plan depends on the
// sizes alone, and gated products follow the same rule as ungated ones with
// one split where their sums must be the same bits: up to 8 rows every product
// divides k over its workgroup's waves alike, past that unsplit sums run along
// k in one chain in either kernel.
inline GemmPlan packed_gemm_plan(int32_t rows, int32_t slices, int32_t kt, bool gated, int32_t max_splits) {
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
    p.groups = (slices + kGemmWaves - 1) / kGemmWaves;
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

}  // namespace baton
