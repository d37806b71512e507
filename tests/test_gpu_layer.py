"""The decode layer around the attention on the GPU (through the C ABI) against
the layer oracle: each operation on the GPU's own inputs, then whole layers
over several decode steps with evictions and insertions, on a small model and
on llama2-7b's shapes.

Tolerances: an operation's output is stored in bf16 (8 significant bits), so
one operation may differ from the float64 definition by half a unit in the
last place, 2^-9 relative, plus the fp32 accumulation of a GEMM; bound used:
2^-7 |ref| + 1e-3.  Whole layers are compared with the oracle storing every
intermediate in bf16 where the GPU does; a bf16 tie that the two round apart
propagates, so the bound there is 2^-5 |ref| + 2e-2, checked at the end of
every layer."""
import os

import numpy as np
import pytest
import torch

import oracle.baton_oracle as O
import oracle.llama_layer as LL
from paper_2410_18701_amd import layer as PL
from paper_2410_18701_amd.cache import BatonCache
from tests import gemm_plan as G
from tests import parity
from workload import driver, gen
from workload import model as M
from workload.configs import Workload

pytestmark = pytest.mark.gpu


def _bits(rng, shape, scale_exp=0):
    x = rng.standard_normal(shape).astype(np.float32) * np.float32(2.0 ** -scale_exp)
    return LL.to_bits(x.astype(np.float64), O.BF16)


def _dev(bits):
    return torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


def _val(t):
    return O.widen(parity.host_bits(t), O.BF16)


# Whole-layer bound: the residual stream after a layer against the oracle's
# layer with the same bf16 roundings, each side going on from the GPU's stream.
LAYER_REL, LAYER_ATOL = 2.0 ** -5, 2e-2
_LAYER_WORST = {}


def _note_layer_margin(got, want, what):
    """Keeps the worst whole-layer error of the test (written with the other margins)."""
    err = np.abs(got - want)
    frac = float((err / (LAYER_REL * np.abs(want) + LAYER_ATOL)).max())
    rel = float((err / np.maximum(np.abs(want), 1e-3)).max())
    test = os.environ.get("PYTEST_CURRENT_TEST", "").split(" (")[0]
    old = _LAYER_WORST.get(test)
    if old is None or frac > old["frac_of_tol"]:
        rec = {"test": test, "what": "whole layer " + what, "dtype": "bf16", "max_abs_err": float(err.max()),
               "max_rel_err": rel, "tol": f"2^-5 |ref| + 2e-2", "frac_of_tol": round(frac, 4)}
        if old is not None:
            parity.MARGINS.remove(old)
        parity.MARGINS.append(rec)
        _LAYER_WORST[test] = rec


def _close(got, want, rel=2.0 ** -7, atol=1e-3, what=""):
    err = np.abs(got - want) - (rel * np.abs(want) + atol)
    assert np.all(err <= 0), f"{what}: worst excess {err.max():.3g} at {np.unravel_index(err.argmax(), err.shape)}"


def _pack_reference(wb):
    """The packed weight layout written out from its definition (include/baton.h):
    16-row slices, 1 KB blocks per 32 columns, lane l's 8 elements at 16 l."""
    N, K = wb.shape
    S, T = -(-N // 16), -(-K // 32)
    pad = np.zeros((S * 16, T * 32), wb.dtype)
    pad[:N, :K] = wb
    out = np.zeros((S, T, 64, 8), wb.dtype)
    for lane in range(64):
        g, r = lane // 16, lane % 16
        for t in range(T):
            out[:, t, lane, :] = pad[r::16, 32 * t + 8 * g:32 * t + 8 * g + 8]
    return out.reshape(-1)


# (rows, out_dim, in_dim, workspace bytes): one split along in_dim (many
# outputs, or no workspace), several splits and their reduction (64 x 4096 x
# 4096, 8 x 4096 x 11008), a partial 16-row slice and a column tail shorter
# than 32 (17 x 1000 x 1000), every group of 16 rows; past 64 rows, one or more
# chunks (128 and 256 rows at llama2-7b's shapes, a partial last row tile at 100
# and 200 rows, with and without splits).
@pytest.mark.parametrize("rows,out_dim,in_dim,ws", [
    (1, 64, 64, 32 << 20), (5, 520, 136, 32 << 20), (64, 4096, 4096, 32 << 20), (8, 4096, 11008, 32 << 20),
    (17, 1000, 1000, 32 << 20), (33, 12288, 4096, 32 << 20), (64, 4096, 4096, 0), (48, 22016, 4096, 32 << 20),
    (128, 4096, 4096, 64 << 20), (256, 12288, 4096, 64 << 20), (100, 256, 512, 32 << 20),
    (200, 1000, 1000, 32 << 20), (256, 4096, 11008, 0), (129, 4096, 4096, 64 << 20)])
def test_linear_packed(rows, out_dim, in_dim, ws):
    rng = np.random.default_rng(rows + out_dim + 7)
    k = round(np.log2(in_dim) / 2)
    xb, wb, yb = _bits(rng, (rows, in_dim)), _bits(rng, (out_dim, in_dim), k), _bits(rng, (rows, out_dim))
    g = PL.Gemm(ws_bytes=ws)
    wp = g.pack(_dev(wb))
    assert np.array_equal(parity.host_bits(wp.data), _pack_reference(wb)), "packed layout"
    y = torch.empty((rows, out_dim), dtype=torch.bfloat16, device="cuda")
    g.linear_packed(_dev(xb), wp, y)
    want = LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16))
    _close(_val(y), want, what="linear_packed")
    y2 = _dev(yb)
    g.linear_packed(_dev(xb), wp, y2, accumulate=True)
    _close(_val(y2), O.widen(yb, O.BF16) + want, what="linear_packed accumulate")
    g.close()


# The fused projection + RMS norm against the two calls it replaces, bit for
# bit, on shapes that split along in_dim (the output and down projections of
# llama2-7b at 64 and 8 rows, 17 rows of a smaller one) and ones that do not
# (many output slices, or no workspace), with and without accumulate; and
# against the oracle's norm of the oracle's product.
@pytest.mark.parametrize("rows,out_dim,in_dim,ws", [
    (64, 4096, 4096, 32 << 20), (8, 4096, 11008, 32 << 20), (17, 1024, 1000, 32 << 20),
    (33, 12288, 4096, 32 << 20), (64, 4096, 4096, 0), (128, 4096, 11008, 64 << 20), (256, 4096, 4096, 64 << 20),
    (200, 1024, 1000, 0)])
def test_linear_packed_rmsnorm(rows, out_dim, in_dim, ws):
    rng = np.random.default_rng(rows + out_dim + 13)
    k = round(np.log2(in_dim) / 2)
    xb, wb, yb, gb = (_bits(rng, (rows, in_dim)), _bits(rng, (out_dim, in_dim), k), _bits(rng, (rows, out_dim)),
                      _bits(rng, (out_dim,)))
    g = PL.Gemm(ws_bytes=ws)
    wp = g.pack(_dev(wb))
    x, gain = _dev(xb), _dev(gb)
    for acc in (False, True):
        y_ref, y = _dev(yb), _dev(yb)
        n_ref = torch.empty_like(y)
        n = torch.full_like(y, float("nan"))
        g.linear_packed(x, wp, y_ref, accumulate=acc)
        PL.rmsnorm(y_ref, gain, n_ref, 1e-5)
        g.linear_packed_rmsnorm(x, wp, y, gain, 1e-5, n, accumulate=acc)
        torch.cuda.synchronize()
        assert np.array_equal(parity.host_bits(y), parity.host_bits(y_ref)), f"y (accumulate={acc})"
        assert np.array_equal(parity.host_bits(n), parity.host_bits(n_ref)), f"y_norm (accumulate={acc})"
        want = LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16)) + (O.widen(yb, O.BF16) if acc else 0.0)
        _close(_val(y), want, what="linear_packed_rmsnorm y")
        _close(_val(n), LL.rmsnorm(_val(y), O.widen(gb, O.BF16), 1e-5), atol=1e-6, what="y_norm")
    g.close()


# The gate/up projection with the gated activation in its epilogue against
# linear_packed (unsplit) into a [gate; up] buffer then silu_mul, bit for bit
# (33 x 2048 x 1000 is a product linear_packed would split): llama2-7b's
# gate/up at 64 and 8 rows, an odd number of 16-column gate slices (48 columns:
# the last workgroup's second gate wave has none), rows not a multiple of 16;
# and against the oracle.
@pytest.mark.parametrize("rows,F,in_dim", [(64, 11008, 4096), (8, 11008, 4096), (17, 48, 136), (33, 1024, 1000),
                                            (128, 11008, 4096), (256, 1024, 1000), (150, 48, 136)])
def test_linear_packed_silu(rows, F, in_dim):
    rng = np.random.default_rng(rows + F + 17)
    k = round(np.log2(in_dim) / 2)
    xb, wb = _bits(rng, (rows, in_dim)), _bits(rng, (2 * F, in_dim), k)
    g = PL.Gemm()
    g0 = PL.Gemm(ws_bytes=0)   # the reference product unsplit, as the fused kernel sums it
    wp = g.pack(_dev(wb))
    x = _dev(xb)
    gu = torch.empty((rows, 2 * F), dtype=torch.bfloat16, device="cuda")
    ref = torch.empty((rows, F), dtype=torch.bfloat16, device="cuda")
    g0.linear_packed(x, wp, gu)
    PL.silu_mul(gu, ref)
    out = torch.full((rows, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    g.linear_packed_silu(x, wp, out)
    torch.cuda.synchronize()
    assert np.array_equal(parity.host_bits(out), parity.host_bits(ref)), "fused against linear_packed + silu_mul"
    guv = _val(gu)
    _close(guv, LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16)), what="gate_up")
    _close(_val(out), LL.silu(guv[:, :F]) * guv[:, F:], atol=1e-6, what="silu(gate) * up")
    g.close()
    g0.close()


def _packed_products(rows, in_dim, out_dim, ws):
    """linear_packed, with accumulate, and linear_packed_silu (out_dim in whole pairs of
    slices) against the oracle, in buffers of NaN past the last row."""
    rng = np.random.default_rng(rows * 131 + in_dim + out_dim)
    k = round(np.log2(in_dim) / 2)
    xb, wb = _bits(rng, (rows, in_dim)), _bits(rng, (out_dim, in_dim), k)
    g = PL.Gemm(ws_bytes=ws)
    wp = g.pack(_dev(wb))
    nan = lambda n: torch.full((rows + 16, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    F = out_dim // 2 if out_dim % 32 == 0 else 0
    xp, yp, ap = nan(in_dim), nan(out_dim), nan(F)
    xp[:rows] = _dev(xb)
    g.linear_packed(xp[:rows], wp, yp[:rows])
    if F:
        g.linear_packed_silu(xp[:rows], wp, ap[:rows])
    y2 = yp.clone()
    g.linear_packed(xp[:rows], wp, y2[:rows], accumulate=True)
    torch.cuda.synchronize()
    want = LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16))
    _close(_val(yp[:rows].contiguous()), want, what="linear_packed")
    _close(_val(y2[:rows].contiguous()), _val(yp[:rows].contiguous()) + want, what="accumulate")
    if F:
        # gate and up are rounded to bf16 before the activation: half a unit of each
        # (2^-9) and of the result, and the activation's slope (at most 1.1 times |gate|'s)
        _close(_val(ap[:rows].contiguous()), LL.silu(want[:, :F]) * want[:, F:], rel=2.0 ** -6, atol=4e-3, what="gated")
    for t in (yp, y2, ap):
        assert torch.isnan(t[rows:]).all(), "written past the last row"
    g.close()


# The products' kernels at the edges of their ranges and tiles: 1 and 8 rows
# (a workgroup per slice or staged rows), 9 and 64 (staged rows), 65 .. 256 (row
# chunks of three to eight tiles, one slice per wave: these products are too small
# for the rule to take more), k of one 16-byte piece, of an odd number of 32-wide
# blocks and with a tail shorter than 32, outputs that leave part of a slice and of
# a workgroup empty, with and without splits along k.  The rows of x past the last
# one and the outputs past the last row are NaN: neither may be read into a result
# or written.
@pytest.mark.parametrize("in_dim,out_dim,ws", [(8, 32, 0), (72, 96, 32 << 20), (200, 1056, 32 << 20),
                                               (2056, 416, 32 << 20), (4104, 32, 32 << 20)])
@pytest.mark.parametrize("rows", [1, 7, 8, 9, 16, 33, 64, 65, 80, 81, 112, 128, 129, 161, 192, 225, 256])
def test_packed_products_edges(rows, in_dim, out_dim, ws):
    _packed_products(rows, in_dim, out_dim, ws)


# Past 64 rows, every tile form the rule can choose -- three to eight row tiles, one to
# three slices per wave, one chunk or several, gated or not, with splits or without --
# at outputs that leave part of a wave's slices, of a workgroup and, with several chunks,
# of the grid empty.
@pytest.mark.parametrize("ws", [0, 32 << 20])
@pytest.mark.parametrize("rows,out_dim,in_dim", G.PAST_64)
def test_tile_forms(rows, out_dim, in_dim, ws):
    _packed_products(rows, in_dim, out_dim, ws)


def _gated_against_plain(rows, F, in_dim):
    """linear_packed_silu bit for bit linear_packed without a workspace then silu_mul, and the product against the oracle."""
    rng = np.random.default_rng(rows + F + in_dim)
    xb, wb = _bits(rng, (rows, in_dim)), _bits(rng, (2 * F, in_dim), round(np.log2(in_dim) / 2))
    g = PL.Gemm(ws_bytes=0)
    x, wp = _dev(xb), g.pack(_dev(wb))
    gu, out = (torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (2 * F, F))
    ref = torch.empty_like(out)
    g.linear_packed(x, wp, gu)
    PL.silu_mul(gu, ref)
    g.linear_packed_silu(x, wp, out)
    torch.cuda.synchronize()
    assert np.array_equal(parity.host_bits(out), parity.host_bits(ref)), "fused against linear_packed + silu_mul"
    _close(_val(gu), LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16)), what="gate_up")
    g.close()


# Up to 8 rows either of two kernels, by the sizes: the choice for a gated product
# and for the plain one of the same weight need not be the same, the bits are
# (12288 x 4096 at 1 row and 2048 x 600 take one each).  The products that split
# along k: ranges of the kernel with a workgroup per slice (few outputs, long k),
# and two ranges of the staged one (5200 x 3080).
@pytest.mark.parametrize("rows,F,in_dim,kinds", [
    (1, 6144, 4096, (G.ROW, G.STAGED)), (3, 1024, 600, (G.ROW, G.STAGED)), (8, 5120, 520, (G.STAGED, G.STAGED)),
    (7, 48, 200, (G.STAGED, G.STAGED)), (8, 8176, 2056, (G.STAGED, G.STAGED)), (2, 16384, 72, (G.STAGED, G.STAGED)),
    (8, 11008, 1032, (G.STAGED, G.STAGED)), (5, 1040, 1096, (G.ROW, G.ROW))])
def test_kernels_of_up_to_8_rows_agree(rows, F, in_dim, kinds):
    assert (G.plan(rows, 2 * F, in_dim, False, 0).kind, G.plan(rows, 2 * F, in_dim, True).kind) == kinds
    _gated_against_plain(rows, F, in_dim)


# The gated product at 9 to 64 rows: the staged kernel at one to four row tiles with
# a last gate slice alone, and the tile kernel with one and two slices per wave, the
# last workgroup with one gate slice of its four.
@pytest.mark.parametrize("rows,F,in_dim,kind,ns", [
    (9, 1040, 1032, G.STAGED, 1), (17, 48, 2056, G.STAGED, 1), (48, 528, 1096, G.STAGED, 1), (64, 48, 4104, G.STAGED, 1),
    (32, 11024, 1000, G.TILE, 1), (33, 11024, 1000, G.TILE, 2), (64, 11024, 1096, G.TILE, 2), (17, 8240, 6408, G.TILE, 2), (10, 11024, 8, G.TILE, 1)])
def test_gated_kernels_of_9_to_64_rows(rows, F, in_dim, kind, ns):
    p = G.plan(rows, 2 * F, in_dim, True)
    assert (p.kind, p.ns) == (kind, ns)
    _gated_against_plain(rows, F, in_dim)


@pytest.mark.parametrize("rows,out_dim,in_dim,kind,splits", [
    (8, 192, 16384, G.ROW, 8), (1, 2048, 11008, G.ROW, 2), (5, 1024, 5128, G.ROW, 3), (3, 5200, 3080, G.STAGED, 2)])
def test_split_products_of_up_to_8_rows(rows, out_dim, in_dim, kind, splits):
    p = G.plan(rows, out_dim, in_dim)
    assert (p.kind, p.splits) == (kind, splits)
    rng = np.random.default_rng(rows + out_dim + in_dim)
    xb, yb = _bits(rng, (rows, in_dim)), _bits(rng, (rows, out_dim))
    wb = _bits(rng, (out_dim, in_dim), round(np.log2(in_dim) / 2))
    g = PL.Gemm()
    x, wp, y, y2 = _dev(xb), g.pack(_dev(wb)), torch.empty((rows, out_dim), dtype=torch.bfloat16, device="cuda"), _dev(yb)
    g.linear_packed(x, wp, y)
    g.linear_packed(x, wp, y2, accumulate=True)
    want = LL.linear(O.widen(xb, O.BF16), O.widen(wb, O.BF16))
    _close(_val(y), want, what="linear_packed")
    _close(_val(y2), O.widen(yb, O.BF16) + want, what="accumulate")
    g.close()


def test_rmsnorm_and_silu_mul():
    rng = np.random.default_rng(11)
    xb, gb = _bits(rng, (7, 4096)), _bits(rng, (4096,))
    y = torch.empty((7, 4096), dtype=torch.bfloat16, device="cuda")
    PL.rmsnorm(_dev(xb), _dev(gb), y, 1e-5)
    _close(_val(y), LL.rmsnorm(O.widen(xb, O.BF16), O.widen(gb, O.BF16), 1e-5), atol=1e-6, what="rmsnorm")
    gub = _bits(rng, (7, 2 * 11008))
    out = torch.empty((7, 11008), dtype=torch.bfloat16, device="cuda")
    PL.silu_mul(_dev(gub), out)
    gu = O.widen(gub, O.BF16)
    _close(_val(out), LL.silu(gu[:, :11008]) * gu[:, 11008:], atol=1e-6, what="silu_mul")


@pytest.mark.parametrize("rows,dim", [(513, 8), (600, 520), (1030, 2048), (520, 2056)])
def test_rmsnorm_of_many_rows(rows, dim):
    """More rows than a decode step has (another workgroup size up to 2048 elements): the
    oracle's values, and each row's bits do not depend on how many there are."""
    rng = np.random.default_rng(rows + dim)
    xb, gb = _bits(rng, (rows, dim)), _bits(rng, (dim,))
    y, y8 = (torch.full((n, dim), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (rows, 8))
    PL.rmsnorm(_dev(xb), _dev(gb), y, 1e-5)
    PL.rmsnorm(_dev(xb[:8]), _dev(gb), y8, 1e-5)
    _close(_val(y), LL.rmsnorm(O.widen(xb, O.BF16), O.widen(gb, O.BF16), 1e-5), atol=1e-6, what="rmsnorm")
    assert np.array_equal(parity.host_bits(y8), parity.host_bits(y)[:8])


def test_rope_at_token_counts():
    """Positions are the slots' token counts: holes from an in-batch prefill
    do not count, free slots are rotated at 0."""
    B, Hq, Hkv, D = 4, 8, 2, 128
    cache = BatonCache(1, B, Hq, Hkv, D, capacity=256, dtype="bf16")
    w = Workload("r", "bf16", 1, B, Hq, Hkv, D, 1, 0, seed=9)
    dev = driver.DeviceInputs(w)
    srcs = [dev.prefill(q, n) for q, n in zip([0, 1], [30, 5])]
    cache.embed([0, 1], [30, 5], [s[0] for s in srcs], [s[1] for s in srcs])
    cache.shape_insert([2], [12])
    q, kn, vn = dev.prefill_step(0, 0, 12, [(2, 2, 12)])
    cache.decode_attn(0, q, kn, vn)
    cache.advance()
    toks = cache.tokens()
    assert toks == [31, 6, 12, 0]
    rng = np.random.default_rng(12)
    qkvb = _bits(rng, (B, (Hq + 2 * Hkv) * D))
    qo = torch.empty((B, Hq, D), dtype=torch.bfloat16, device="cuda")
    ko = torch.empty((B, Hkv, D), dtype=torch.bfloat16, device="cuda")
    vo = torch.empty((B, Hkv, D), dtype=torch.bfloat16, device="cuda")
    PL.rope_qkv(cache, _dev(qkvb), qo, ko, vo, 10000.0)
    qr, kr, vr = LL.split_qkv(O.widen(qkvb, O.BF16), Hq, Hkv, D)
    pos = np.array(toks, np.float64)[:, None]
    _close(_val(qo), LL.rope(qr, pos, 1e4), atol=2e-3, what="rope q")
    _close(_val(ko), LL.rope(kr, pos, 1e4), atol=2e-3, what="rope k")
    assert np.array_equal(parity.host_bits(vo), LL.split_qkv(qkvb, Hq, Hkv, D)[2])
    cache.close()


def _run_layers(m, NL, B, steps_ops, seed=21, capacity=128):
    """GPU layers and the oracle in lockstep; returns the worst relative excess."""
    w = Workload("layer", "bf16", NL, B, m.n_q_heads, m.n_kv_heads, m.head_dim, 1, 0, seed=seed)
    dev = driver.DeviceInputs(w)
    cache = BatonCache(NL, B, m.n_q_heads, m.n_kv_heads, m.head_dim, capacity=capacity, dtype="bf16")
    pb = O.PaddedBatch(NL, B, m.n_q_heads, m.n_kv_heads, m.head_dim, O.BF16, fill_bits=cache.fill_bits)
    wd = [M.weights_device(seed, m, l) for l in range(NL)]
    wh = [M.weights_host(seed, m, l) for l in range(NL)]
    gemm = PL.Gemm()
    layers = PL.DecodeLayers(cache, wd, gemm, m.theta, m.eps)
    step = 0
    for op in steps_ops:
        if op[0] == "embed":
            _, slots, lens, qids = op
            srcs = [dev.prefill(q, n) for q, n in zip(qids, lens)]
            cache.embed(slots, lens, [s[0] for s in srcs], [s[1] for s in srcs])
            pb.embed(slots, lens, [gen.prefill_host(seed, "k", q, NL, m.n_kv_heads, n, m.head_dim, "bf16")
                                   for q, n in zip(qids, lens)],
                     [gen.prefill_host(seed, "v", q, NL, m.n_kv_heads, n, m.head_dim, "bf16")
                      for q, n in zip(qids, lens)])
        elif op[0] == "evict":
            cache.evict(op[1], release=True)
            pb.evict(op[1], release=True)
        else:
            x = M.x_device(seed, step, B, m.hidden)
            xh = M.bf16_value(M.x_host(seed, step, B, m.hidden))
            assert np.array_equal(_val(x), xh)
            pos = cache.tokens()
            live = [b for b in range(B) if pb.lens[b] > 0]
            for layer in range(NL):
                layers.layer(layer, x)
                xh = LL.decode_layer(pb, layer, xh, wh[layer], pos, m.theta, m.eps, stored=O.BF16)
                got = _val(x)
                _close(got[live], xh[live], rel=LAYER_REL, atol=LAYER_ATOL, what=f"step {step} layer {layer}")
                _note_layer_margin(got[live], xh[live], f"{m.name if hasattr(m, 'name') else 'layer'} B={B}")
                xh = got   # both sides go on from the GPU's stream
            cache.advance()
            pb.advance()
            step += 1
    torch.cuda.synchronize()
    L, _, lens = cache.query()
    assert (L, lens) == (pb.L, pb.lens)
    gemm.close()
    cache.close()


def test_layers_small_model():
    m = M.ModelShape(256, 4, 2, 64, 512)
    ops = [("embed", [0, 1, 2], [9, 30, 4], [0, 1, 2]), ("step",), ("step",),
           ("evict", [1]), ("embed", [3, 1], [12, 40], [3, 4]), ("step",), ("evict", [0]), ("step",)]
    _run_layers(m, 2, 4, ops)


def test_layers_small_model_128_slots():
    """Past 64 slots the projections take the tile kernel."""
    m = M.ModelShape(256, 4, 2, 64, 512)
    lens = [(7 * b) % 50 + 1 for b in range(128)]
    ops = [("embed", list(range(128)), lens, list(range(128))), ("step",),
           ("evict", [3, 70, 127]), ("embed", [70, 3], [60, 2], [128, 129]), ("step",)]
    _run_layers(m, 1, 128, ops)


def test_layers_llama2_7b_shape():
    ops = [("embed", [0, 1, 2, 3], [100, 7, 33, 64], [0, 1, 2, 3]), ("step",),
           ("evict", [2]), ("embed", [2], [20], [4]), ("step",)]
    _run_layers(M.LLAMA2_7B, 2, 4, ops, capacity=192)
