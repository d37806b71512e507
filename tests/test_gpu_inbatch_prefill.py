"""Baton without prefill/decode separation on the GPU (sec. 4.1): new queries
prefilled inside the batch (baton_shape_insert), holes left in the other rows,
the holey mask, causal prefill attention and later decode steps over holey
rows -- in lockstep with the materialized oracle: ring bit for bit, mask bit
for bit, token counts, every output within tolerance, and positions that hold
no token left untouched."""
import json
import os

import numpy as np
import pytest

from tests import gemm_plan as G
from tests import oracle_pins, parity

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 1, 4, 4, 4, 64), ("f32", 2, 5, 8, 2, 128), ("bf16", 2, 6, 8, 8, 128),
          ("bf16", 1, 5, 16, 2, 128), ("bf16", 1, 4, 4, 2, 64)]


def _sid(s):
    return f"{s[0]}-{s[1]}x{s[2]}-{s[3]}/{s[4]}x{s[5]}"


def _golden_ops():
    """The hand-derived replay's operations (tests/golden/inbatch_prefill_replay.json)."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "inbatch_prefill_replay.json")
    ops, s = [], 0
    for op in json.load(open(path))["ops"]:
        if op["op"] in ("embed", "shape"):
            ops.append((op["op"], op["slots"], op["lens"], op["qids"]))
        elif op["op"] == "evict":
            ops.append(("evict", op["slots"]))
        else:
            ops.append(("step", s))
            s += 1
    return ops


def _random_ops(seed, B, steps, max_len):
    rng = np.random.default_rng(seed)
    ops, qid, s = [], 0, 0
    for op in oracle_pins._random_ops_shaped(rng, B, steps, max_len):
        if op[0] in ("embed", "shape"):
            qids = list(range(qid, qid + len(op[1])))
            qid += len(op[1])
            ops.append((op[0], op[1], op[2], qids))
            if op[0] == "shape":
                ops.append(("step", s))
                s += 1
        elif op[0] == "evict":
            ops.append(op)
        else:
            ops.append(("step", s))
            s += 1
    return ops


@pytest.mark.parametrize("shape", SHAPES, ids=_sid)
def test_golden_story(shape):
    dtype, NL, _, Hq, Hkv, D = shape
    err = parity.run_script((dtype, NL, 3, Hq, Hkv, D), _golden_ops(), capacity=64)
    print(f"[inbatch golden] {shape}: max abs error {err:.3g}", flush=True)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[1] > 1], ids=_sid)
def test_random_sequences_separate_buffers(shape):
    """Prefill steps with K and V in two allocations of their own (packed layers)."""
    dtype, NL, B, Hq, Hkv, D = shape
    ops = _random_ops(7, B, steps=10, max_len=70)
    err = parity.run_script(shape, ops, capacity=2048, split=64, layout="separate")
    print(f"[inbatch random] {shape} separate buffers: {len(ops)} ops, max abs error {err:.3g}", flush=True)


@pytest.mark.parametrize("shape", SHAPES, ids=_sid)
@pytest.mark.parametrize("seed", [0, 1])
def test_random_sequences(shape, seed):
    dtype, NL, B, Hq, Hkv, D = shape
    ops = _random_ops(seed * 10 + len(shape[0]), B, steps=14, max_len=70)
    err = parity.run_script(shape, ops, capacity=2048, split=64)
    print(f"[inbatch random] {shape} seed {seed}: {len(ops)} ops, max abs error {err:.3g}", flush=True)


def test_long_prompts_and_wrap():
    """Prompts spanning many tiles and key blocks (up to 300 tokens), several
    prefills in one step with different lengths, a ring that wraps."""
    ops = [("embed", [0, 1, 2], [100, 40, 7], [0, 1, 2]), ("step", 0),
           ("evict", [1]), ("shape", [1], [300], [3]), ("step", 1), ("step", 2),
           ("evict", [0, 2]), ("shape", [2, 0], [129, 33], [4, 5]), ("step", 3),
           ("evict", [1]), ("embed", [1], [60], [6]), ("step", 4),
           ("evict", [2]), ("shape", [2], [250], [7]), ("step", 5), ("step", 6)]
    for shape in (("bf16", 1, 3, 8, 8, 128), ("bf16", 1, 3, 16, 2, 64), ("f32", 1, 3, 4, 2, 128)):
        err = parity.run_script(shape, ops, capacity=800, split=64)
        print(f"[inbatch long] {shape}: max abs error {err:.3g}", flush=True)


def test_extract_with_holes():
    """A query with holes stored aside and re-inserted: its tokens come back in
    order without the holes, and it decodes on as the oracle says."""
    ops = [("embed", [0, 1], [20, 9], [0, 1]), ("step", 0),
           ("shape", [2], [12], [2]), ("step", 1), ("step", 2),
           ("evict", [1]), ("shape", [1], [5], [3]), ("step", 3),
           ("extract", [0, 2], "holey"), ("evict", [0, 2]), ("step", 4),
           ("embed_saved", [3, 0], "holey"), ("step", 5), ("step", 6)]
    for shape in (("bf16", 2, 4, 8, 2, 128), ("f32", 1, 4, 4, 4, 64)):
        err = parity.run_script(shape, ops, capacity=256, split=64)
        print(f"[inbatch extract] {shape}: max abs error {err:.3g}", flush=True)


@pytest.mark.parametrize("scale", [1.0, -0.5])
def test_peaked_and_negative_scale(scale):
    """Prompts and decode rows with a peaked softmax (scale 1 at head_dim 128)
    and with a negative scale, whose sign the prefill kernel folds into q."""
    ops = [("embed", [0, 1, 2], [100, 40, 7], [0, 1, 2]), ("step", 0),
           ("evict", [1]), ("shape", [1], [200], [3]), ("step", 1), ("step", 2),
           ("evict", [0, 2]), ("shape", [2, 0], [129, 33], [4, 5]), ("step", 3), ("step", 4)]
    for shape in (("bf16", 1, 3, 8, 8, 128), ("bf16", 1, 3, 16, 2, 64), ("f32", 1, 3, 4, 2, 128)):
        err = parity.run_script(shape, ops, capacity=600, split=64, scale=scale)
        print(f"[inbatch scale {scale}] {shape}: max abs error {err:.3g}", flush=True)


def test_holes_with_unscrubbed_evictions():
    """In-batch prefill and holes after evictions that leave stale tokens
    (no BATON_SCRUB) and do not release: live tokens, mask and outputs as the
    oracle says."""
    ops = [("embed", [0, 1, 2], [30, 12, 50], [0, 1, 2]), ("step", 0),
           ("evict", [1], False, False), ("shape", [1], [20], [3]), ("step", 1),
           ("evict", [2], False, False), ("embed", [2], [9], [4]), ("step", 2),
           ("evict", [0], True, False), ("shape", [0], [6], [5]), ("step", 3), ("step", 4),
           ("evict", [], True, False), ("step", 5)]
    for shape in (("bf16", 2, 3, 8, 2, 128), ("f32", 1, 3, 4, 4, 64)):
        err = parity.run_script(shape, ops, capacity=256, split=64)
        print(f"[inbatch stale] {shape}: max abs error {err:.3g}", flush=True)


@pytest.mark.parametrize("shape", [("f32", 1, 3, 4, 4, 128), ("bf16", 1, 3, 8, 8, 128), ("bf16", 1, 3, 4, 4, 64),
                                   ("bf16", 1, 3, 16, 2, 128), ("bf16", 1, 3, 8, 4, 64)], ids=_sid)
def test_gathered_items(shape):
    """A row that lives through many prefill steps keeps a short run (the
    tokens it decoded since the last one) behind each hole; the attention
    kernels read such runs as gathered items of at most one pass of a
    workgroup (VALU: 32, 64 and 128 tokens for the first three shapes, more
    than the split at head_dim 64; matrix cores, grouped heads: 64):
    slot 0 ends with some 70 tokens in short runs behind 19 holes (several
    gathered items, the last with the current token), slot 1 (a 10-token
    prompt) is short runs only, slot 2 is prefilled again and again with
    prompts of 3-40 tokens."""
    prompts = [5, 23, 40, 7, 31, 12, 3, 37]
    ops = [("embed", [0], [100], [0]), ("shape", [1], [10], [1]), ("step", 0)]
    s, qid = 1, 2
    for c in range(18):
        if c:
            ops.append(("evict", [2]))
        ops += [("shape", [2], [prompts[c % len(prompts)]], [qid]), ("step", s)]
        qid, s = qid + 1, s + 1
        for _ in range(c % 5 + 1):
            ops.append(("step", s))
            s += 1
    err = parity.run_script(shape, ops, capacity=1024, split=64)
    print(f"[inbatch gathered] {shape}: {s} steps, max abs error {err:.3g}", flush=True)


@pytest.mark.parametrize("shape", [("bf16", 1, 4, 8, 2, 128), ("bf16", 1, 4, 4, 4, 64), ("f32", 1, 4, 4, 4, 128)],
                         ids=_sid)
def test_many_holes_rows_of_different_ages(shape):
    """Sixty holes held by rows of different ages: slot 0 lives through every
    prefill step, slot 1 is prefilled again and again, slot 2 is embedded
    (prefilled elsewhere) after 20 of them and slot 3 prefilled in the batch
    after 40, so each row holds its own suffix of the hole list.  The run
    behind a hole is the prefill step's one token and up to two decode steps,
    or (twice) 66 decode steps: listed runs, runs cut into a piece of the
    split (64) and a remainder, and back-to-back short runs in one work list
    (66 tokens are listed at head_dim 64, whose gathered items hold 128)."""
    prompts = [5, 23, 40, 7, 31, 12, 3, 37, 2, 18]
    ops = [("embed", [0], [150], [0]), ("step", 0)]
    s, qid = 1, 1
    for c in range(60):
        if c:
            ops.append(("evict", [1]))
        if c == 20:
            ops.append(("embed", [2], [90], [qid]))
            qid += 1
        slots, lens = [1], [prompts[c % len(prompts)]]
        if c == 40:
            slots, lens = [1, 3], [lens[0], 25]
        ops += [("shape", slots, lens, list(range(qid, qid + len(slots)))), ("step", s)]
        qid, s = qid + len(slots), s + 1
        for _ in range(66 if c in (10, 35) else c % 3):
            ops.append(("step", s))
            s += 1
    err = parity.run_script(shape, ops, capacity=2048, split=64)
    print(f"[inbatch many holes] {shape}: {s} steps, max abs error {err:.3g}", flush=True)


# The fp32 prefill kernel at the edges of its tiles: prompts of one token, one
# short of, exactly and one past a 16-key block and a round of the four waves'
# blocks, several prompts in one step, more workgroups than run at once (64 heads of
# 64 and 32 of 128 at 300 tokens) and the launch of one workgroup per CU (8 heads of
# 128 at 601 tokens); then the same prompt with a value that is not finite near its
# end, which the positions before it must not see.
@pytest.mark.parametrize("heads,kv,D,lens", [(4, 4, 64, [1, 15, 16, 17]), (4, 2, 128, [63, 64, 65, 2]),
                                             (8, 1, 64, [33, 130]), (64, 8, 64, [300]), (32, 32, 128, [300, 49]),
                                             (8, 2, 128, [601, 20])])
def test_f32_prefill_edges(heads, kv, D, lens):
    import torch
    from paper_2410_18701_amd.cache import BatonCache
    B, T = len(lens), max(lens)
    g = torch.Generator().manual_seed(sum(lens) + heads)
    q, k, v = (torch.randn((B, T, h, D), generator=g) for h in (heads, kv, kv))

    def run(v):
        cache = BatonCache(1, B, heads, kv, D, capacity=T + 64, dtype="f32")
        cache.shape_insert(list(range(B)), lens)
        out = torch.full((B, T, heads, D), float("nan"), device="cuda")
        cache.decode_attn(0, q.cuda(), k.cuda(), v.cuda(), out=out)
        cache.advance()
        ks, vs = cache.extract(list(range(B)))
        for b, p in enumerate(lens):
            assert torch.equal(ks[b][0].cpu(), k[b, T - p:].transpose(0, 1).contiguous()), "appended keys"
            assert torch.equal(vs[b][0].cpu().view(torch.int32),
                               v[b, T - p:].transpose(0, 1).contiguous().view(torch.int32)), "appended values"
        cache.close()
        return out.cpu()

    out = run(v)
    for b, p in enumerate(lens):
        assert torch.isnan(out[b, :T - p]).all(), "a position without a token was written"
        hide = torch.ones(p, p, dtype=torch.bool).triu(1)
        for h in range(heads):
            kk, vv = (x[b, T - p:, h // (heads // kv)].double() for x in (k, v))
            s = (q[b, T - p:, h].double() @ kk.T * D ** -0.5).masked_fill(hide, -np.inf)
            err = (out[b, T - p:, h].double() - torch.softmax(s, -1) @ vv).abs().max()
            assert err <= 1e-5, f"slot {b} head {h}: {err}"
    for bad in (float("inf"), float("nan")):
        vb = v.clone()
        vb[:, T - 1] = bad
        ob = run(vb)
        for b, p in enumerate(lens):
            rows = slice(T - p, T - 1)
            assert (ob[b, rows] - out[b, rows]).abs().max() <= 1e-5 if p > 1 else True
            assert not torch.isfinite(ob[b, T - 1]).any()


def _scores_by_four(q, k, scale):
    """base-2 scores of q [n][D] against k [m][D] in float32 as a lane group adds them: each
    lane four products in a chain of fused multiply-adds, then a tree over the lanes."""
    f32 = np.float32
    qs = (q.astype(f32) * f32(f32(scale) * f32(1.4426950408889634))).astype(f32)
    n, m, lanes = q.shape[0], k.shape[0], q.shape[1] // 4
    acc = np.zeros((n, m, lanes), f32)
    for e in range(4):   # exact products in float64, one rounding per multiply-add
        acc = (acc + qs[:, None, e::4].astype(np.float64) * k[None, :, e::4].astype(np.float64)).astype(f32)
    while acc.shape[2] > 1:
        acc = acc[:, :, 0::2] + acc[:, :, 1::2]
    return acc[:, :, 0]


# fp32 prompts whose rounding error is mostly the scores': no larger against float64
# than with scores added four products at a time and then as a tree, and the softmax
# and the products in float32.  With that order the kernel has 0.97 to 1.02 times the
# reference's error, with chains of four matrix operations 1.15 to 1.22; the bound
# leaves 3% for the sample (3,800 rows and more, about 1%) and the later sums' order.
@pytest.mark.parametrize("D,scale,p", [(64, 1.0, 40), (64, 4.0, 100), (128, 1.0, 100), (128, 2.0, 100)])
def test_f32_prefill_score_rounding(D, scale, p):
    import torch
    from paper_2410_18701_amd.cache import BatonCache
    H, B = 16, 6
    g = torch.Generator().manual_seed(D + p)
    q, k, v = (torch.randn((B, p, H, D), generator=g) for _ in range(3))
    cache = BatonCache(1, B, H, H, D, capacity=p + 64, dtype="f32")
    cache.shape_insert(list(range(B)), [p] * B)
    out = torch.empty((B, p, H, D), device="cuda")
    cache.decode_attn(0, q.cuda(), k.cuda(), v.cuda(), out=out, scale=scale)
    cache.advance()
    out = out.cpu().numpy()
    cache.close()
    hide = np.triu(np.ones((p, p), bool), 1)
    err = [0.0, 0.0]
    for b in range(B):
        for h in range(H):
            qh, kh, vh = (x[b, :, h].numpy() for x in (q, k, v))
            exact = np.where(hide, -np.inf, qh.astype(np.float64) @ kh.astype(np.float64).T * scale)
            w = np.exp(exact - exact.max(1, keepdims=True))
            want = w @ vh.astype(np.float64) / w.sum(1, keepdims=True)
            s = np.where(hide, np.float32(-np.inf), _scores_by_four(qh, kh, scale))
            w = np.exp2(s - s.max(1, keepdims=True))   # in float32 like what follows
            err[0] += ((out[b, :, h] - want) ** 2).sum()
            err[1] += ((w @ vh / w.sum(1, keepdims=True) - want) ** 2).sum()
    ratio = (err[0] / err[1]) ** 0.5
    print(f"[f32 score rounding] D {D} scale {scale} p {p}: {ratio:.3f}", flush=True)
    assert ratio <= 1.05, ratio


# Bound of a position's outputs against float64, 2-norm over 2-norm: the weights and the
# outputs are rounded to bf16, 2^-9 each at worst (the kernel's mean is 0.002).  A key
# too many or too few near position 1,024 is about 0.03, a missing block of 32 keys 0.1.
POSITION_REL = 6e-3


def _check_prompt(out, q, k, v, p, scale, what):
    """Causal attention outputs out [p][heads][D] of a prompt against float64, on three
    heads, a position at a time."""
    import torch
    heads, kv = q.shape[1], k.shape[1]
    hide = torch.ones(p, p, dtype=torch.bool).triu(1)
    for h in (0, heads // 2 - 1, heads - 1):
        kk, vv = (x[:, h // (heads // kv)].double() for x in (k, v))
        want = torch.softmax((q[:, h].double() @ kk.T * scale).masked_fill(hide, -np.inf), -1) @ vv
        err = (out[:, h].double() - want).norm(dim=1) / want.norm(dim=1)
        assert err.max() <= POSITION_REL, f"{what} head {h} position {int(err.argmax())}: {err.max()}"


# The long-prompt bf16 kernel (128 positions per workgroup) at its edges: one token past
# and one short of a 32-key block, a wave's positions and a tile, prompts of a few tokens
# beside a long one (tiles of waves with nothing to do), every grouping, both head sizes,
# a negative scale; against float64 on a few heads, the appended rows bit for bit on all.
@pytest.mark.parametrize("heads,kv,D,lens,scale", [
    (64, 8, 128, [1025, 1, 31, 513], 0.0), (64, 64, 128, [1055, 129, 640], 0.0),
    (64, 16, 64, [1030, 1025, 992, 895], 0.0), (64, 32, 128, [1119, 33, 700], -0.2),
    (64, 8, 64, [1535, 700, 641, 2], 1.0)])
def test_long_prompt_kernel_edges(heads, kv, D, lens, scale):
    import torch
    from paper_2410_18701_amd.cache import BatonCache
    B, T = len(lens), max(lens)
    g = torch.Generator().manual_seed(sum(lens) + heads)
    q, k, v = (torch.randn((B, T, h, D), generator=g).bfloat16() for h in (heads, kv, kv))
    for b, p in enumerate(lens):          # positions without a token: not read into a result
        for x in (q, k, v):
            x[b, :T - p] = float("nan")
    assert G.prefill_long(heads, D, lens)
    cache = BatonCache(1, B, heads, kv, D, capacity=T + 64, dtype="bf16")
    cache.shape_insert(list(range(B)), lens)
    out = torch.full((B, T, heads, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    cache.decode_attn(0, q.cuda(), k.cuda(), v.cuda(), out=out, scale=scale)
    cache.advance()
    ks, vs = cache.extract(list(range(B)))
    out = out.cpu()
    for b, p in enumerate(lens):
        assert torch.equal(ks[b][0].cpu(), k[b, T - p:].transpose(0, 1).contiguous()), "appended keys"
        assert torch.equal(vs[b][0].cpu(), v[b, T - p:].transpose(0, 1).contiguous()), "appended values"
        assert torch.isnan(out[b, :T - p]).all(), "a position without a token was written"
        _check_prompt(out[b, T - p:], q[b, T - p:], k[b, T - p:], v[b, T - p:], p, scale or D ** -0.5, f"slot {b}")
    cache.close()


# The same kernel in a running batch: two rows decode beside the prompts, and the ring,
# which a query before them has moved on, ends in the middle of the prompts' columns.
@pytest.mark.parametrize("heads,kv,D,lens", [(64, 8, 128, [1055, 1030]), (64, 64, 64, [1290, 1313, 900])])
def test_long_prompts_beside_decoding_rows_over_the_rings_end(heads, kv, D, lens):
    import torch
    from paper_2410_18701_amd.cache import BatonCache
    assert G.prefill_long(heads, D, lens)
    rows, T, cap = [37, 90], max(lens), max(lens) + 250
    B = 3 + len(lens)
    g = torch.Generator().manual_seed(sum(lens))
    src = [tuple(torch.randn((1, kv, n, D), generator=g).bfloat16() for _ in range(2)) for n in rows]
    q, k, v = (torch.randn((B, T, h, D), generator=g).bfloat16() for h in (heads, kv, kv))
    cache = BatonCache(1, B, heads, kv, D, capacity=cap, dtype="bf16")
    cache.shape_insert([2], [300])
    cache.decode_attn(0, *(x[:, :300].contiguous().cuda() for x in (q, k, v)))
    cache.advance()
    cache.embed([0, 1], rows, [s[0].cuda() for s in src], [s[1].cuda() for s in src])
    cache.evict([2], release=True)
    slots = list(range(3, B))
    cache.shape_insert(slots, lens)
    L, base, _ = cache.query()
    first = (base + L) % cap
    assert L == max(rows) and 0 < first < cap < first + T, (base, L, T, cap)   # the step's columns wrap
    out = torch.full((B, T, heads, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    cache.decode_attn(0, q.cuda(), k.cuda(), v.cuda(), out=out)
    cache.advance()
    out = out.cpu()
    ks, vs = cache.extract([0, 1] + slots)
    for b, p in zip(slots, lens):
        for got, x in ((ks, k), (vs, v)):
            assert torch.equal(got[b - 1][0].cpu(), x[b, T - p:].transpose(0, 1).contiguous()), "appended rows"
        assert torch.isnan(out[b, :T - p]).all(), "a position without a token was written"
        _check_prompt(out[b, T - p:], q[b, T - p:], k[b, T - p:], v[b, T - p:], p, D ** -0.5, f"slot {b}")
    for b in (0, 1):
        kk, vv = (torch.cat([src[b][i][0], (k, v)[i][b, 0].unsqueeze(1)], 1) for i in (0, 1))   # [kv][n + 1][D]
        assert torch.equal(ks[b][0].cpu(), kk) and torch.equal(vs[b][0].cpu(), vv), "the decoding row's tokens"
        kk, vv = (x.double().repeat_interleave(heads // kv, 0) for x in (kk, vv))
        s = (q[b, 0].double().unsqueeze(1) @ kk.transpose(1, 2)).squeeze(1) * D ** -0.5
        want = (torch.softmax(s, -1).unsqueeze(1) @ vv).squeeze(1)
        err = (out[b, 0].double() - want).norm(dim=1) / want.norm(dim=1)
        assert err.max() <= POSITION_REL, f"row {b}: {err.max()}"
        assert torch.isnan(out[b, 1:]).all(), "a position without a token was written"
    cache.close()
