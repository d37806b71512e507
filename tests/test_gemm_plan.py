"""The rule that chooses a packed product's kernel, tile and split (host code):
over the range of sizes every plan covers the product and names a kernel form
that exists."""
import random

import pytest

from tests import gemm_plan as G

SIZES = [16, 32, 96, 208, 512, 1024, 1040, 2048, 4096, 5120, 6160, 8192, 10240, 12288, 14336, 16384, 18432, 22016,
         22048, 24576, 32000, 36864, 65536, 128256]
INS = [8, 64, 200, 512, 1024, 1536, 2048, 3072, 4096, 4104, 5120, 8192, 11008, 12288, 16384, 28672]


@pytest.mark.parametrize("gated", [False, True])
def test_every_plan_covers_the_product(gated):
    rng = random.Random(5)
    for rows in range(1, 257):
        for out_dim in SIZES + [16 * rng.randint(1, 4096) for _ in range(8)]:
            out_dim = (out_dim + 31) // 32 * 32 if gated else out_dim
            for in_dim in INS:
                for ws in ([0] if gated else [0, 32 << 20]):
                    what = (rows, out_dim, in_dim, gated, ws)
                    p = G.plan(rows, out_dim, in_dim, gated, ws)
                    kt, slices = -(-in_dim // 32), out_dim // 32 if gated else -(-out_dim // 16)
                    assert p.splits >= 1 and p.splits * p.tc >= kt > (p.splits - 1) * p.tc, what   # no empty split
                    assert p.splits == 1 or p.splits * rows * out_dim * 4 <= ws, what
                    per = {G.ROW: 1, G.STAGED: 2 if gated else 4, G.TILE: (2 if gated else 4) * p.ns}[p.kind]
                    assert p.groups * per >= slices > (p.groups - 1) * per, what
                    assert p.chunks * p.mt * 16 >= rows > (p.chunks - 1) * p.mt * 16, what
                    if p.kind == G.TILE:
                        assert G.tile_built(p.mt, p.ns, p.chunks, gated), what
                    else:
                        assert p.ns == 1 and p.chunks == 1 and p.mt <= (1 if p.kind == G.ROW else 4), what
                        assert rows <= (8 if p.kind == G.ROW else 64), what


def test_forms_that_do_not_exist_are_known():
    """The launcher asks the same predicate and returns an error for a form that was not built."""
    for mt, ns, chunks, gated in [(4, 1, 1, False), (1, 1, 1, False), (1, 1, 2, True), (2, 1, 2, False), (2, 3, 1, True), (9, 1, 2, True),
                                  (5, 4, 1, False), (0, 1, 1, True), (8, 0, 1, True)]:
        assert not G.tile_built(mt, ns, chunks, gated), (mt, ns, chunks, gated)
    assert G.tile_built(8, 3, 2, False) and G.tile_built(3, 3, 2, False) and G.tile_built(4, 2, 1, True) and G.tile_built(5, 1, 1, False)


# (rows, out, in, gated, kind, least workgroups): sizes at which the wrong kernel or
# too few workgroups measured 1.1 to 1.9 times the time of the right one, up to 8 rows.
@pytest.mark.parametrize("rows,out_dim,in_dim,gated,kind,least", [
    (1, 8192, 512, False, G.STAGED, 128), (8, 16384, 512, False, G.STAGED, 256), (1, 16384, 2048, False, G.STAGED, 256),
    (1, 32768, 512, True, G.STAGED, 512), (8, 1024, 512, True, G.STAGED, 16), (4, 16384, 1024, True, G.STAGED, 256),
    (8, 10240, 16384, True, G.STAGED, 160), (1, 10240, 2048, False, G.STAGED, 160),
    (1, 22016, 4096, True, G.ROW, 688), (8, 18432, 8192, False, G.ROW, 1152), (1, 4096, 4096, False, G.ROW, 256),
    (1, 512, 16384, False, G.ROW, 256), (8, 1024, 16384, False, G.ROW, 256), (1, 192, 16384, False, G.ROW, 96),
    (1, 2048, 11008, False, G.ROW, 256), (1, 512, 4096, False, G.ROW, 32), (8, 6144, 16384, False, G.STAGED, 192)])
def test_up_to_8_rows(rows, out_dim, in_dim, gated, kind, least):
    p = G.plan(rows, out_dim, in_dim, gated)
    assert p.kind == kind and p.groups * p.splits >= least, p


# The gated product at 9 to 64 rows: the staged kernel measured 0.79 to 0.95 of the
# tile's time where its workgroups make one round (not with short k at 64 rows).
@pytest.mark.parametrize("rows,out_dim,in_dim,kind", [
    (9, 1024, 8192, G.STAGED), (16, 8192, 4096, G.STAGED), (32, 2048, 8192, G.STAGED), (48, 12288, 4096, G.STAGED),
    (64, 4096, 8192, G.STAGED), (9, 10240, 1024, G.STAGED), (64, 4096, 1024, G.TILE), (16, 22016, 4096, G.TILE),
    (64, 22016, 4096, G.TILE)])
def test_gated_9_to_64_rows(rows, out_dim, in_dim, kind):
    assert G.plan(rows, out_dim, in_dim, True).kind == kind


# Past 64 rows: the plan of chunks of up to 128 rows and 8 splits left most of the GPU
# idle where outputs are few (64 to 160 workgroups), and 160 rows in two chunks took
# one and a quarter rounds where three chunks make one.
@pytest.mark.parametrize("rows,out_dim,in_dim,gated,least,most", [
    (128, 512, 16384, False, 120, 256), (65, 512, 11008, False, 96, 256), (128, 1024, 16384, False, 160, 256),
    (256, 512, 16384, False, 160, 256), (256, 1024, 8192, True, 48, 256), (160, 10240, 4096, True, 200, 256)])
def test_past_64_rows_fills_the_gpu(rows, out_dim, in_dim, gated, least, most):
    p = G.plan(rows, out_dim, in_dim, gated)
    assert least <= p.groups * p.chunks * p.splits <= most, p


def test_the_edge_products_reach_every_tile_form():
    """Guards the GPU tests of G.PAST_64: a change of the rule that drops a form from them fails here."""
    forms = set().union(*(G.past_64(*a) for a in G.PAST_64))
    every = {(mt, ns, chunks, gated) for mt in range(3, 9) for ns in (1, 2, 3) for chunks in (False, True)
             for gated in (False, True) if chunks or mt > 4}
    # one slice per wave of 128-row chunks, gated: four chunks of 64 rows are always the cheaper choice
    assert every - forms == {(8, 1, True, True)}
    assert any(G.plan(*a).splits > 1 and G.plan(*a).chunks > 1 for a in G.PAST_64)


def test_launches_stay_below_2_to_the_32_threads():
    """Weights of 2^28 outputs and more, which a workgroup per slice cannot launch."""
    for rows in (1, 8, 9, 64, 65, 256):
        for out_dim in ((1 << 28) - 16, 1 << 28, 1 << 29):
            for in_dim in (32, 96, 2048, 4096):
                for gated in (False, True):
                    p = G.plan(rows, out_dim, in_dim, gated)
                    assert p.groups * p.chunks * p.splits * 256 < 1 << 32, (rows, out_dim, in_dim, gated, p)


@pytest.mark.parametrize("rows,dim,threads", [
    (4096, 512, 256), (1024, 2048, 256), (16384, 64, 256), (513, 1024, 256), (512, 512, 512), (64, 2048, 512),
    (256, 512, 512), (4096, 4096, 512), (1, 64, 512)])
def test_norm_threads(rows, dim, threads):
    """512 threads took up to 1.45 times the time over many short rows."""
    assert G.lib().norm_threads(rows, dim) == threads


@pytest.mark.parametrize("rows", [(1 << 23) - 1, 1 << 23, (1 << 24) - 1])
@pytest.mark.parametrize("dim", [8, 2048, 2056, 4096])
def test_norm_launches_fit(rows, dim):
    assert rows * G.lib().norm_threads(rows, dim) < 1 << 32
