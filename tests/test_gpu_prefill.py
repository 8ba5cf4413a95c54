"""GPU parity of the tiled kernel.  Calls of more than 2048 tokens always run on it, so the shapes
here stay small; every test asks the library which kernel and tile its call takes."""
import numpy as np
import pytest
import torch

import paper_2603_25385_amd as G
from glowq_inputs import UnitShape
from oracle import glowq_oracle as O
from gpu_util import DeviceUnit, Workspace, stream
from util import add_stored_projection, check_with_infinities, overflow_one_rank, recipe_unit, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-3                     # the forward's bar: fp32 accumulation, R rounded once
ULP = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}
LARGE, HALF = 0, 1


def route_of(du, slabs=True):
    r = G.glowq_debug_route([du.desc], slabs)[0]
    assert r.kernel == G.GLOWQ_ROUTE_TILED
    return r


def make(T, d_in, d_outs, act, Gs=128, r=24, seed=None):
    return recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=Gs, method="alg1", qr="none", seed=seed)


def check(ys, refs, tol):
    for y, ref in zip(ys, refs):
        assert y.shape == ref.shape and np.isfinite(y).all()
        e = rel_err(y, ref)
        assert e <= tol, e


def check_infinite_rank(T, d_in, d_outs, act, r):
    u = make(T, d_in, d_outs, act, 128, r)
    overflow_one_rank(O, u, r - 3)
    du = DeviceUnit(u)
    ws = Workspace([du.desc])
    G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, stream())
    for got, want in zip(du.outputs(), add_stored_projection(O, u, O.group_forward(u, False))):
        check_with_infinities(got, want, TOL)
    return du


def test_one_workspace_for_calls_of_different_sizes():
    # a long prompt whose projection runs in K parts (their arrival counters lie past the first 256
    # bytes of the workspace), and short calls that leave partial sums there, in turn through one
    # buffer that was cleared once: the same bits every time, no wait expired
    units = [make(T, 4352, (64, 40), "f16", seed=60 + T) for T in (2056, 1, 40, 130)]
    dus = [DeviceUnit(u) for u in units]
    route_of(dus[0])
    nbytes = max(G.glowq_workspace_bytes([d.desc]) for d in dus)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    G.glowq_workspace_init(ws.data_ptr(), nbytes, stream())
    failed = torch.zeros(1, dtype=torch.int32, device="cuda")
    first = {}
    for k in (0, 1, 0, 2, 0, 3, 0, 1, 2, 3, 0) * 3:
        dus[k].clear()
        G.glowq_group_forward(dus[k].desc, True, ws.data_ptr(), nbytes, stream())
        G.glowq_workspace_status([dus[k].desc], ws.data_ptr(), nbytes, failed.data_ptr(), stream())
        ys = dus[k].outputs()
        assert int(failed.item()) == 0
        if k not in first:
            check(ys, O.group_forward(units[k], True), TOL)
            first[k] = ys
        assert all(np.array_equal(a, b) for a, b in zip(first[k], ys)), k


# (T, d_in, d_outs, types, tile): half-size tiles and large ones, a last token tile of one and of two
# blocks, one K tile, ragged row blocks that straddle modules
CASES = [(2056, 128, (264, 96, 40), ("f16", "bf16"), HALF), (2070, 640, (264, 96, 40), ("f16", "bf16"), HALF),
         (2056, 128, (1000,), ("f16", "bf16"), HALF), (2070, 128, (3000, 3000, 3000), ("f16",), LARGE),
         (2056, 128, (4008,), ("bf16",), LARGE), (2070, 256, (6008,), ("bf16",), LARGE)]


@pytest.mark.parametrize("Gs,r", [(128, 72), (64, 16), (64, 128)])
@pytest.mark.parametrize("T,d_in,d_outs,act,tile", [(T, d, o, a, t) for T, d, o, acts, t in CASES for a in acts])
def test_tiles_match_the_oracle(T, d_in, d_outs, act, tile, Gs, r):
    u = make(T, d_in, d_outs, act, Gs, r)
    for restore, out in ((True, "act"), (True, "f32"), (False, "f32")):
        du = DeviceUnit(u, out, 8)
        assert route_of(du).tile == tile
        ws = Workspace([du.desc])
        G.glowq_group_forward(du.desc, restore, ws.ptr, ws.bytes, stream())
        check(du.outputs(), O.group_forward(u, restore), TOL + (ULP[act] if out == "act" else 0.0))
        ws.assert_idle()


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("r", [8, 24, 64, 120, 128])
def test_every_rank_with_k_parts_of_the_projection(r, act):
    # three parts of unequal length that the last one to finish adds; twice through one workspace
    u = make(2056, 4352, (136, 40), act, r=r)
    du = DeviceUnit(u)
    route_of(du)
    ws = Workspace([du.desc])
    for _ in range(2):
        du.clear()
        G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, stream())
        check(du.outputs(), O.group_forward(u, True), TOL)
        ws.assert_idle()


@pytest.mark.parametrize("T,d_in,d_outs,act,out,tile,slices", [
    (2056, 8320, (264, 40), "f16", "f32", HALF, 2), (2056, 8320, (264, 40), "bf16", "act", HALF, 2),
    (2056, 12288, (72,), "f16", "act", HALF, 3), (257, 16384, (2008,), "bf16", "f32", HALF, 4),
    (257, 12288, (4008,), "f16", "act", LARGE, 3), (520, 8192, (4008,), "bf16", "f32", LARGE, 2)])
def test_k_slices(T, d_in, d_outs, act, out, tile, slices):
    # two to four slices of unequal length (65 tiles: 32 + 33), each leaves an fp32 slab in the
    # workspace, the first carries the correction, a second kernel adds them in slice order; ragged
    # rows (40: a slab row of 40 floats), padded output rows, restored and not, the same bits every
    # time, and against a call that cannot cut (no workspace)
    u = make(T, d_in, d_outs, act)
    du = DeviceUnit(u, out, 8)
    r = route_of(du)
    assert (r.tile, r.k_slices) == (tile, slices)
    ws = Workspace([du.desc])
    refs = {f: O.group_forward(u, f) for f in (True, False)}
    tol = TOL + (ULP[act] if out == "act" else 0.0)
    seen = {}
    for restore in (True, False, True):
        du.clear()
        G.glowq_group_forward(du.desc, restore, ws.ptr, ws.bytes, stream())
        ys = du.outputs()
        check(ys, refs[restore], tol)
        ws.assert_idle()
        if restore in seen:
            assert all(np.array_equal(a, b) for a, b in zip(seen[restore], ys))
        seen[restore] = ys
    du.clear()
    G.glowq_group_forward(du.desc, False, 0, 0, stream())
    check(du.outputs(), refs[False], tol)


def test_k_slices_and_a_full_module_table():
    # seven units in one launch, five of them long enough for K slices (four at 16384 channels, two at
    # 8192): the table of 16 module entries has room for some of the slices only, so units cut four
    # ways, two ways and not at all and ordinary units share it; masked and restored ones, called
    # longest not first, twice through one workspace
    shapes = [(256, (64, 40)), (16384, (40,)), (8192, (40, 24)), (16384, (24,)), (384, (136,)), (16384, (40,)), (8192, (72,))]
    mask = [1, 1, 0, 1, 1, 0, 1]
    units = [make(2056, d, o, "f16", r=16, seed=30 + i) for i, (d, o) in enumerate(shapes)]
    dus = [DeviceUnit(u) for u in units]
    routes = G.glowq_debug_route([d.desc for d in dus])
    assert all(r.launch == 0 and r.kernel == G.GLOWQ_ROUTE_TILED for r in routes)
    assert [r.k_slices for r in routes] == [1, 4, 2, 1, 1, 1, 2]
    ws = Workspace([d.desc for d in dus])
    refs = [O.group_forward(u, bool(f)) for u, f in zip(units, mask)]
    for _ in range(2):
        for d in dus:
            d.clear()
        G.glowq_block_forward([d.desc for d in dus], bytes(mask), ws.ptr, ws.bytes, stream())
        for d, ref in zip(dus, refs):
            check(d.outputs(), ref, TOL)
        ws.assert_idle()


@pytest.mark.parametrize("Gs", [128, 64])
@pytest.mark.parametrize("act,d_out,tile", [("f16", 48, HALF), ("bf16", 48, HALF), ("f16", 9000, LARGE), ("bf16", 4008, LARGE)])
def test_multiplies_with_the_stored_weight(act, d_out, tile, Gs):
    # rows of the identity (and zeros up to the kernel's token count): every output is one weight as the
    # kernel's own dequantiser made it, which must be round_act((q - z) s) bit for bit
    T, d_in = 2056, 128
    rng = np.random.default_rng(3)
    q = rng.integers(0, 16, size=(d_out, d_in)).astype(np.uint8)
    s_bits = rng.integers(1, 0x6C00, size=(d_out, d_in // Gs)).astype(np.uint16)
    z_bits = O.f64_to_bits(rng.integers(0, 16, size=(d_out, d_in // Gs)).astype(np.float64), "f16")
    X = np.zeros((T, d_in), np.uint16)
    X[np.arange(d_in) * 16, np.arange(d_in)] = O.f64_to_bits(np.ones(1), act)[0]     # in every token tile
    du = DeviceUnit(dict(act=act, G=Gs, r=0, d_in=d_in, B=None, X=X,
                         modules=[dict(wq=O.pack_int4(q), scales=s_bits, zeros=z_bits, A=None)]))
    assert route_of(du).tile == tile
    ws = Workspace([du.desc])
    G.glowq_group_forward(du.desc, False, ws.ptr, ws.bytes, stream())
    y = du.outputs()[0]
    seen = y[np.arange(d_in) * 16].T
    ref = O.bits_to_f64(O.dequant_bits(q, s_bits, z_bits, Gs, act), act)
    bad = np.argwhere(seen != ref)
    assert bad.size == 0, (bad[:5], seen[tuple(bad[0])], ref[tuple(bad[0])])
    rest = np.ones(T, bool)
    rest[np.arange(d_in) * 16] = False
    assert not y[rest].any()


@pytest.mark.parametrize("Gs", [128, 64])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_wide_tiles_multiply_with_the_stored_weight(act, Gs):
    # the identity: every output is one weight as k_wide's dequantiser made it; 25 K tiles, ragged rows and tokens
    d_in, d_out = 3200, 4104
    rng = np.random.default_rng(4)
    q = rng.integers(0, 16, size=(d_out, d_in)).astype(np.uint8)
    s_bits = rng.integers(1, 0x6C00, size=(d_out, d_in // Gs)).astype(np.uint16)
    z_bits = O.f64_to_bits(rng.integers(0, 16, size=(d_out, d_in // Gs)).astype(np.float64), "f16")
    X = np.zeros((d_in, d_in), np.uint16)
    np.fill_diagonal(X, O.f64_to_bits(np.ones(1), act)[0])
    du = DeviceUnit(dict(act=act, G=Gs, r=0, d_in=d_in, B=None, X=X,
                         modules=[dict(wq=O.pack_int4(q), scales=s_bits, zeros=z_bits, A=None)]))
    route_of(du)
    assert G.glowq_debug_tile_tokens([du.desc]) == [256]
    ws = Workspace([du.desc])
    G.glowq_group_forward(du.desc, False, ws.ptr, ws.bytes, stream())
    seen = du.outputs()[0].T
    ref = O.bits_to_f64(O.dequant_bits(q, s_bits, z_bits, Gs, act), act)
    bad = np.argwhere(seen != ref)
    assert bad.size == 0, (bad[:5], seen[tuple(bad[0])], ref[tuple(bad[0])])


@pytest.mark.parametrize("T,d_in,d_outs,tokens", [(2056, 2304, (72, 40), 128), (1025, 4352, (10248,), 256)])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_handoff_in_a_row_and_in_graphs(act, T, d_in, d_outs, tokens):
    # the projection's parts, its flags and their consumers back to back: 200 launches, half of them
    # replays of a captured call with eager calls in between, every result equal to the first one's bits
    u = make(T, d_in, d_outs, act)
    du = DeviceUnit(u)
    route_of(du)
    assert G.glowq_debug_tile_tokens([du.desc]) == [tokens]
    ws = Workspace([du.desc])
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, stream())
    first = du.outputs()
    check(first, O.group_forward(u, True), TOL)
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, torch.cuda.current_stream().cuda_stream)
        for it in range(20):
            du.clear()
            for k in range(5):
                graph.replay()
                G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, side.cuda_stream)
            side.synchronize()
            assert all(np.array_equal(a, b) for a, b in zip(first, du.outputs())), it
    ws.assert_idle()


# the wide tiles (256 x 256): one row block and one token more than a tile, a last token tile of one 128-token
# projection tile, ragged rows of several modules, both group sizes, one and two stages of ranks.  Tiles and
# projection workgroups stay within the chip's 256 places (6136 and 10248 rows in place of 5624 and 9224 are one tile
# too many: 106 to 123 us on wide tiles, 90 to 104 on the smaller ones that such calls take)
@pytest.mark.parametrize("T,d_in,d_outs,act,Gs,r", [
    (1025, 3328, (6152, 5624), "f16", 64, 128), (1025, 3328, (6152, 5624), "bf16", 128, 72),
    (1281, 3328, (9224,), "f16", 128, 8), (1281, 3328, (9224,), "bf16", 64, 120)])
def test_wide_tiles_match_the_oracle(T, d_in, d_outs, act, Gs, r):
    u = make(T, d_in, d_outs, act, Gs, r)
    refs = {f: O.group_forward(u, f) for f in (True, False)}
    for restore, out in ((True, "act"), (True, "f32"), (False, "act")):
        du = DeviceUnit(u, out, 8)
        route_of(du)
        assert G.glowq_debug_tile_tokens([du.desc]) == [256]
        ws = Workspace([du.desc])
        G.glowq_group_forward(du.desc, restore, ws.ptr, ws.bytes, stream())
        check(du.outputs(), refs[restore], TOL + (ULP[act] if out == "act" else 0.0))
        ws.assert_idle()


# a rank of R past the activation type's range: infinite outputs of that token's and no NaN from the operand words past
# the last rank, one stage of ranks and two
@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("T,d_in,d_outs,r,tile", [(300, 1024, (8200,), 72, 1), (300, 1024, (8200,), 8, 1), (1100, 512, (16392,), 24, 0)])
def test_infinite_rank_on_large_and_half_tiles(T, d_in, d_outs, act, r, tile):
    route = route_of(check_infinite_rank(T, d_in, d_outs, act, r))
    assert (route.kernel, route.tile) == (G.GLOWQ_ROUTE_TILED, tile)


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("T,d_in,d_outs,r", [(1025, 3328, (6152, 5624), 72), (1281, 3328, (9224,), 8)])
def test_infinite_rank_on_wide_tiles(T, d_in, d_outs, act, r):
    du = check_infinite_rank(T, d_in, d_outs, act, r)
    assert G.glowq_debug_tile_tokens([du.desc]) == [256]


def test_wide_tiles_with_k_slices():
    # a long contraction in three slices beside an ordinary unit, group size 64; twice through one workspace
    units = [make(512, 3072, (12288, 12296), "bf16", 64, 24, seed=71), make(512, 12288, (1000,), "bf16", 64, 72, seed=72)]
    dus = [DeviceUnit(u) for u in units]
    descs = [d.desc for d in dus]
    assert G.glowq_debug_tile_tokens(descs) == [256, 256]
    assert [r.k_slices for r in G.glowq_debug_route(descs)] == [1, 3]
    ws = Workspace(descs)
    refs = [O.group_forward(u, True) for u in units]
    for _ in range(2):
        for d in dus:
            d.clear()
        G.glowq_block_forward(descs, bytes([1, 1]), ws.ptr, ws.bytes, stream())
        for d, ref in zip(dus, refs):
            check(d.outputs(), ref, TOL + ULP["bf16"])
        ws.assert_idle()


# fewer slices beside other units than the unit's shapes ask for (one per 4096 channels, four at most), or none; ragged rows, a
# last token tile of one
@pytest.mark.parametrize("act,T,short,d_in,d_outs,slices", [
    ("f16", 500, (3072, (9896, 8056)), 12416, (2832, 4112), 2), ("bf16", 513, (3200, (9328, 11560)), 16512, (2216, 2080), 2),
    ("bf16", 513, (3200, (11840, 7456, 13112)), 8192, (1488, 1928), 1)])
def test_wide_tiles_with_fewer_k_slices(act, T, short, d_in, d_outs, slices):
    units = [make(T, *short, act, seed=74), make(T, d_in, d_outs, act, seed=75)]
    dus = [DeviceUnit(u, "act", 8) for u in units]
    descs = [d.desc for d in dus]
    assert G.glowq_debug_tile_tokens(descs) == [256, 256]
    assert [r.k_slices for r in G.glowq_debug_route(descs)] == [1, slices]
    wider = [DeviceUnit(u, "f32", 8) for u in units]              # 32-bit outputs keep them
    assert [r.k_slices for r in G.glowq_debug_route([d.desc for d in wider])] == [1, min(4, d_in // 4096)]
    ws = Workspace(descs)
    for mask in ((1, 1), (0, 1), (1, 0)):
        for d in dus:
            d.clear()
        G.glowq_block_forward(descs, bytes(mask), ws.ptr, ws.bytes, stream())
        for d, u, m in zip(dus, units, mask):
            check(d.outputs(), O.group_forward(u, bool(m)), TOL + ULP[act])
        ws.assert_idle()


def long_units(act, Gs):
    # an odd number of K tiles, a unit of one K tile, fewer tokens (a last token tile of 188 of 256), two stages of ranks
    return [make(1025, 5248, (6152, 4360), act, Gs, 72, seed=81), make(1025, 128, (264, 40), act, Gs, 8, seed=82),
            make(700, 3328, (2056,), act, Gs, 128, seed=83)]


@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_wide_tiles_with_units_of_several_lengths(act):
    units = long_units(act, 128)
    dus = [DeviceUnit(u) for u in units]
    refs = {f: [O.group_forward(u, f) for u in units] for f in (True, False)}
    for order, mask in (((0, 1, 2), (1, 1, 1)), ((2, 1, 0), (1, 1, 1)), ((0, 1, 2), (1, 0, 1)), ((2, 1, 0), (0, 1, 1))):
        descs = [dus[k].desc for k in order]
        assert G.glowq_debug_tile_tokens(descs) == [256] * 3
        assert all(r.launch == 0 for r in G.glowq_debug_route(descs))
        ws = Workspace(descs)
        for k in order:
            dus[k].clear()
        G.glowq_block_forward(descs, bytes(mask), ws.ptr, ws.bytes, stream())
        for k, f in zip(order, mask):
            check(dus[k].outputs(), refs[bool(f)][k], TOL)
        ws.assert_idle()


@pytest.mark.parametrize("Gs", [128, 64])
@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_wide_tiles_give_the_bits_of_the_128_token_tiles(act, Gs):
    # the same units beside one of a single K tile that moves the launch to the smaller tiles; R's partial sums, both
    # output types, one unit masked
    units = long_units(act, Gs)
    extra = make(1025, 128, (12288,), act, Gs, 8, seed=84)
    for out in ("act", "f32"):
        dus = [DeviceUnit(u, out) for u in units]
        short = DeviceUnit(extra, out)
        seen = []
        for descs, tokens in (([d.desc for d in dus], 256), ([d.desc for d in dus] + [short.desc], 128)):
            assert G.glowq_debug_tile_tokens(descs) == [tokens] * len(descs)
            ws = Workspace(descs)
            for d in dus:
                d.clear()
            G.glowq_block_forward(descs, bytes([1, 0, 1, 1][:len(descs)]), ws.ptr, ws.bytes, stream())
            seen.append([y for d in dus for y in d.outputs()])
            ws.assert_idle()
        assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(*seen))


# Tiles of 80, 96, 112 and 128 tokens (a call's tokens dealt evenly to as many tiles as tiles of 128 would be), first and
# last of each height, in one, two and three token tiles: the second tile of 140 tokens takes its R from both of the
# projection's tiles of 128
@pytest.mark.parametrize("T,d_in,d_outs,act,tile,height", [
    (70, 1152, (10008, 10008), "f16", HALF, 80), (80, 1152, (10008, 10008), "bf16", HALF, 80), (81, 768, (12008, 12008), "f16", HALF, 96),
    (96, 768, (12008, 12008), "bf16", HALF, 96), (97, 768, (12008, 12008), "bf16", HALF, 112), (112, 768, (12008, 12008), "f16", HALF, 112),
    (113, 768, (12008, 12008), "f16", HALF, 128), (140, 768, (12008, 12008), "f16", HALF, 80), (157, 768, (12008, 12008), "bf16", HALF, 80),
    (200, 768, (8232, 8232), "bf16", HALF, 112), (300, 768, (8232, 8232), "f16", HALF, 112), (90, 256, (26008,) * 3, "bf16", LARGE, 96),
    (140, 256, (26008,) * 3, "f16", LARGE, 80), (200, 256, (20008, 20008), "bf16", LARGE, 112), (260, 256, (26008, 26008), "f16", LARGE, 96)])
def test_tile_heights(T, d_in, d_outs, act, tile, height):
    for Gs, r in ((128, 72), (64, 128)):
        u = make(T, d_in, d_outs, act, Gs, r)
        du = DeviceUnit(u, "act", 8)
        assert route_of(du).tile == tile and G.glowq_debug_tile_height([du.desc]) == [height]
        ws = Workspace([du.desc])
        for restore in (True, False):
            du.clear()
            G.glowq_group_forward(du.desc, restore, ws.ptr, ws.bytes, stream())
            check(du.outputs(), O.group_forward(u, restore), TOL + ULP[act])
            ws.assert_idle()


# A third slice of K (binary16, one token tile, several units in a launch) keeps its partial results behind all slices of the
# workspace; without that room the call runs in two slices
def test_a_third_slice_and_its_room():
    shapes = [((20008, 20008), 1024), ((2056,), 9984), ((520, 264), 10112)]
    units = [make(100, d, outs, "f16", r=24, seed=95 + i) for i, (outs, d) in enumerate(shapes)]
    dus = [DeviceUnit(u) for u in units]
    descs = [d.desc for d in dus]
    routes = G.glowq_debug_route(descs)
    assert [r.k_slices for r in routes] == [1, 3, 3] and {(r.launch, r.kernel) for r in routes} == {(0, G.GLOWQ_ROUTE_TILED)}
    slices, need = sum(G.glowq_workspace_bytes([d]) for d in descs), G.glowq_workspace_bytes(descs)
    assert need >= slices + 3 * 100 * (2056 + 784) * 4
    failed = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for nbytes, third in ((need, True), (need - 256, False), (slices, False), (need, True)):
        buf = torch.zeros(need + 4096, dtype=torch.uint8, device="cuda")
        buf[slices:] = 0xA5
        for restore in (1, 0):
            for d in dus:
                d.clear()
            G.glowq_block_forward(descs, bytes([restore] * 3), buf.data_ptr(), nbytes, stream())
            for u, d in zip(units, dus):
                check(d.outputs(), O.group_forward(u, bool(restore)), TOL)
        G.glowq_workspace_status(descs, buf.data_ptr(), nbytes, failed.data_ptr(), stream())
        torch.cuda.synchronize()
        assert int(failed.item()) == 0
        assert bool((buf[slices:need] != 0xA5).any()) == third and bool((buf[need:] == 0xA5).all())


def test_units_of_several_token_counts_share_tiles_of_one_height():
    # 70, 200 and 330 tokens in one launch: the most blocks that a unit asks for (seven) hold for all
    units = [make(T, 768, (12008, 4008), "f16", r=24, seed=90 + T) for T in (70, 330, 200)]
    dus = [DeviceUnit(u) for u in units]
    routes = G.glowq_debug_route([d.desc for d in dus])
    assert {(r.launch, r.kernel) for r in routes} == {(0, G.GLOWQ_ROUTE_TILED)}
    assert G.glowq_debug_tile_height([d.desc for d in dus]) == [112] * 3
    ws = Workspace([d.desc for d in dus])
    G.glowq_block_forward([d.desc for d in dus], bytes([1, 1, 1]), ws.ptr, ws.bytes, stream())
    for u, d in zip(units, dus):
        check(d.outputs(), O.group_forward(u, True), TOL)
    ws.assert_idle()
