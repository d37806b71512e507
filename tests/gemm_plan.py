"""The library's rules for packed products and for a step's bf16 prompts
(csrc/gemm_plan.hpp, csrc/prefill_plan.hpp: host code without a GPU header), compiled as
they stand and called from the tests."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_18701_amd", "csrc")
SHIM = """
#include "gemm_plan.hpp"
#include "prefill_plan.hpp"
extern "C" void plan(int rows, int slices, int in_dim, int gated, int max_splits, int* o) {
  const baton::GemmPlan p = baton::packed_gemm_plan(rows, slices, in_dim, gated != 0, max_splits);
  const int v[] = {p.kind, p.mt, p.ns, p.chunks, p.groups, p.tc, p.splits};
  for (int i = 0; i < 7; ++i) o[i] = v[i];
}
extern "C" int tile_built(int mt, int ns, int chunks, int gated) {
  return baton::tile_gemm_built(mt, ns, chunks, gated != 0);
}
extern "C" int norm_threads(int rows, int dim) { return baton::norm_threads(rows, dim); }
extern "C" int prefill_long(int head_dim, const int* plen, int n, int wgs) {
  return baton::prefill_long(head_dim, plen, n, wgs);
}
"""
ROW, STAGED, TILE = 0, 1, 2
kWaves = 4   # per workgroup
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


# (rows, out, in) whose plans past 64 rows -- plain without a workspace, plain with one,
# gated where out allows -- reach every tile form the rule can choose, with outputs that
# leave part of a wave's slices and of a workgroup empty.
PAST_64 = [
    (65, 32, 136), (65, 8480, 136), (65, 16448, 2056), (65, 32896, 136), (81, 8480, 136), (81, 16448, 2056),
    (81, 24608, 136), (81, 32896, 136), (97, 8256, 136), (97, 10280, 136), (97, 10400, 136), (97, 16448, 136),
    (97, 16448, 2056), (97, 32896, 136), (113, 5128, 2056), (113, 10272, 136), (113, 13664, 192), (113, 24608, 136),
    (113, 32896, 136), (129, 5344, 136), (129, 16448, 136), (150, 4128, 2056), (161, 12512, 136), (161, 16448, 136),
    (192, 5408, 192), (193, 6240, 136), (193, 9280, 136), (193, 12512, 136), (193, 16448, 136), (225, 16448, 136),
    (244, 1040, 4104), (256, 1032, 2056), (256, 12512, 136), (256, 22016, 72)]


def past_64(rows, out_dim, in_dim):
    """The tile forms (mt, ns, several chunks, gated) that the product's three calls take and
    that leave part of a workgroup empty."""
    forms = set()
    for gated, ws in [(False, 0), (False, 32 << 20)] + [(True, 0)] * (out_dim % 32 == 0):
        p = plan(rows, out_dim, in_dim, gated, ws)
        if (out_dim // 32 if gated else -(-out_dim // 16)) % ((2 if gated else kWaves) * p.ns):
            forms.add((p.mt, p.ns, p.chunks > 1, gated))
    return forms


def prefill_long(heads, head_dim, lens):
    """Whether prompts of these lengths take the kernel of 128 positions per workgroup."""
    wgs = heads * sum(-(-p // 128) for p in lens)
    return bool(lib().prefill_long(head_dim, (ctypes.c_int * len(lens))(*lens), len(lens), wgs))
