"""The library's rule for packed products (csrc/gemm_plan.hpp, host code without
a GPU header), compiled as it stands and called from the tests."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_18701_amd", "csrc")
SHIM = """
#include "gemm_plan.hpp"
extern "C" void plan(int rows, int slices, int in_dim, int gated, int max_splits, int* o) {
  const baton::GemmPlan p = baton::packed_gemm_plan(rows, slices, in_dim, gated != 0, max_splits);
  const int v[] = {p.kind, p.mt, p.ns, p.chunks, p.groups, p.tc, p.splits};
  for (int i = 0; i < 7; ++i) o[i] = v[i];
}
extern "C" int tile_built(int mt, int ns, int chunks, int gated) {
  return baton::tile_gemm_built(mt, ns, chunks, gated != 0);
}
"""
ROW, STAGED, TILE = 0, 1, 2
Plan = collections.namedtuple("Plan", "kind mt ns chunks groups tc splits")


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
        return ctypes.CDLL(so)


def plan(rows, out_dim, in_dim, gated=False, ws_bytes=32 << 20):
    """The plan of baton_linear_packed (gated: baton_linear_packed_silu, out_dim the
    rows of [gate; up]) with a workspace of ws_bytes."""
    o = (ctypes.c_int * 7)()
    slices = out_dim // 32 if gated else -(-out_dim // 16)
    splits = 1 if gated or not ws_bytes else min(ws_bytes // (4 * rows * out_dim), 1024)
    lib().plan(rows, slices, in_dim, int(gated), splits, o)
    return Plan(*o)


def tile_built(mt, ns, chunks, gated):
    return bool(lib().tile_built(mt, ns, chunks, int(gated)))
