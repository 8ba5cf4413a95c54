"""GPU parity of the batched kernel (more than four tokens): edges of tiles, token blocks, K tiles and
wave groups, and (test_every_tile) each workgroup tile that its rule chooses, asked of the library."""
import numpy as np
import pytest
import torch

import paper_2603_25385_amd as G
from glowq_inputs import UnitShape
from oracle import glowq_oracle as O
from gpu_util import DeviceUnit, Workspace, run_group, stream
from util import recipe_unit, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-3                     # the forward's bar: fp32 accumulation, R rounded once
ULP = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}

# (T, d_in, d_outs): one K tile for four wave groups; wave groups with unequal shares of K; ragged
# row blocks that straddle modules; token tiles of 16, 32 and 64 with ragged last ones; from a
# workgroup or two to several per compute unit; more than 64 tokens
SHAPES = [(16, 128, (40, 264, 96)), (5, 1152, (40, 264, 96)), (9, 1024, (4096, 4120)), (17, 640, (2000, 2008)),
          (32, 384, (12000,)), (20, 2048, (8000,)), (33, 128, (40, 264)), (45, 1024, (1000,)), (64, 640, (6000,)),
          (64, 512, (20000,)), (65, 1152, (40, 264)), (79, 1152, (1960, 1960)), (129, 640, (520,)),
          (200, 384, (4000,)), (300, 256, (264,))]


@pytest.mark.parametrize("act,Gs", [("f16", 128), ("f16", 64), ("bf16", 128), ("bf16", 64)])
@pytest.mark.parametrize("T,d_in,d_outs", SHAPES)
def test_tiles_match_the_oracle(T, d_in, d_outs, act, Gs):
    r = 72 if Gs == 128 else 16             # two whole correction steps and a ragged one; half a step
    u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=Gs, method="alg1", qr="none")
    for restore, out in ((True, "act"), (True, "f32"), (False, "f32")):
        ys, _, _ = run_group(u, restore, out=out, ldy_pad=8)
        tol = TOL + (ULP[act] if out == "act" else 0.0)
        for y, ref in zip(ys, O.group_forward(u, restore)):
            assert np.isfinite(y).all() and rel_err(y, ref) <= tol


# (T, d_in, rows, tile): binary16 up to 32 tokens, where the sums are scaled; beyond, where the weights
# are rounded; bfloat16
TILE_SHAPES = {
    "exact": [(5, 256, (40, 264), 0), (5, 128, (40, 264), 1), (5, 768, (5000,), 2), (18, 896, (10008,), 3),
              (18, 4352, (10008,), 4), (5, 1536, (5000,), 7), (5, 8320, (4440, 4440), 8)],
    "f16": [(33, 256, (40, 264), 0), (33, 128, (40, 264), 1), (33, 768, (2008,), 2), (70, 128, (10008,), 3),
            (33, 4352, (6008,), 4), (33, 3200, (12008,), 5), (50, 128, (20008,), 6), (33, 1536, (2008,), 7)],
    "bf16": [(5, 384, (40, 264), 0), (5, 128, (40, 264), 1), (5, 1536, (10008,), 2), (18, 128, (10008,), 3),
             (131, 6272, (4008,), 5), (131, 128, (10008,), 6), (5, 2176, (5000,), 7), (5, 8320, (4440, 4440), 8)]}


@pytest.mark.parametrize("kind,T,d_in,d_outs,tile", [(k, *s) for k, shapes in TILE_SHAPES.items() for s in shapes])
def test_every_tile(kind, T, d_in, d_outs, tile):
    act = "bf16" if kind == "bf16" else "f16"
    for Gs, r in ((128, 72), (64, 128)):
        u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=Gs, method="alg1", qr="none")
        for restore, out in ((True, "act"), (False, "f32")):
            ys, du, _ = run_group(u, restore, out=out, ldy_pad=8)
            got = G.glowq_debug_route([du.desc])[0]
            assert (got.kernel, got.tile) == (G.GLOWQ_ROUTE_BATCHED, tile)
            tol = TOL + (ULP[act] if out == "act" else 0.0)
            for y, ref in zip(ys, O.group_forward(u, restore)):
                assert np.isfinite(y).all() and rel_err(y, ref) <= tol


# R small enough that the consumers add the projection's slices themselves, at its limits (512 ranks
# of all tokens, 8192 channels) and right beyond; one K tile (four slices of 32 channels) and
# slices of unequal length; several tokens tiles
@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("T,r,d_in", [(64, 8, 128), (32, 16, 2176), (5, 96, 4096), (8, 64, 8192), (8, 64, 8320), (9, 64, 1152),
                                      (16, 32, 640), (43, 8, 1024)])
def test_small_projections(T, r, d_in, act):
    u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, (200, 72)), act=act, G=128, method="alg1", qr="none")
    ys, _, _ = run_group(u, True)
    for y, ref in zip(ys, O.group_forward(u, True)):
        assert np.isfinite(y).all() and rel_err(y, ref) <= TOL


@pytest.mark.parametrize("T", [7, 24, 50, 90])
def test_units_of_one_call_share_a_launch(T):
    # units of different widths, ranks and gating in one call (more than one launch holds), called
    # longest last, twice through one workspace: every unit's result is its own
    shapes = [UnitShape("a", 256, (64, 40)), UnitShape("b", 128, (48,)), UnitShape("c", 2176, (136, 16)),
              UnitShape("d", 384, (24, 24, 24))] * 5
    mask = [(i % 3) != 1 for i in range(len(shapes))]
    units = [recipe_unit(O, 1, 0, T, seed=50 + i, r=(8, 40, 24, 64)[i % 4], shape=s, G=128) for i, s in enumerate(shapes)]
    dus = [DeviceUnit(u) for u in units]
    ws = Workspace([d.desc for d in dus])
    refs = [O.group_forward(u, f) for u, f in zip(units, mask)]
    for _ in range(2):
        for d in dus:
            d.clear()
        G.glowq_block_forward([d.desc for d in dus], bytes(mask), ws.ptr, ws.bytes, stream())
        for d, ref in zip(dus, refs):
            for y, yr in zip(d.outputs(), ref):
                assert rel_err(y, yr) <= TOL
        ws.assert_idle()


# Contractions cut across workgroups: slices of unequal length, two to four of them, one K tile per wave group, ragged
# row blocks that straddle modules, ragged token tiles; with the correction (the first slice's) and without; one unit
# alone and two of a kind
@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("T,d_in,d_outs,n,r", [
    (9, 13696, (1000, 600), 2, 16), (11, 13568, (1168,), 2, 16), (17, 14336, (40, 264, 96), 2, 16), (20, 13824, (1768, 2080), 2, 72),
    (27, 14208, (3304,), 2, 72), (9, 13696, (2600, 1512), 1, 72), (32, 14208, (4096,), 1, 72)])
def test_contractions_cut_across_workgroups(T, d_in, d_outs, n, r, act):
    u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=128, method="alg1", qr="none")
    dus = [DeviceUnit(u) for _ in range(n)]
    descs = [d.desc for d in dus]
    assert all(2 <= r.k_slices <= 4 for r in G.glowq_debug_route(descs))
    assert all(r.k_slices == 1 for r in G.glowq_debug_route(descs, False))
    ws = Workspace(descs)
    for restore in (True, False):
        refs, first = O.group_forward(u, restore), None
        for _ in range(3):                  # the counts of the call before are in the workspace
            for d in dus:
                d.clear()
            G.glowq_block_forward(descs, bytes([restore] * n), ws.ptr, ws.bytes, stream())
            ys = [y for d in dus for y in d.outputs()]
            for y, ref in zip(ys, refs * n):
                assert np.isfinite(y).all() and rel_err(y, ref) <= TOL + ULP[act]
            first = first or ys
            assert all(np.array_equal(a, b) for a, b in zip(first, ys))      # whichever slice comes last
            ws.assert_idle()


# A unit with a correction alone in its launch is cut from 4096 rows and nine tokens on
@pytest.mark.parametrize("T,rows,cut", [(9, 4096, True), (8, 4096, False), (9, 4080, False), (11, 1168, False)])
def test_lone_units_are_cut_from_a_size_on(T, rows, cut):
    u = recipe_unit(O, 1, 0, T, r=16, shape=UnitShape("g", 13568, (rows,)), act="bf16", G=128, method="alg1", qr="none")
    assert (G.glowq_debug_route([DeviceUnit(u).desc])[0].k_slices > 1) == cut


@pytest.mark.parametrize("act", ["f16", "bf16"])
def test_cut_and_whole_contractions_share_a_launch(act):
    shapes = [UnitShape("a", 1024, (1024, 256, 256)), UnitShape("b", 1024, (1024,)), UnitShape("c", 1024, (2048, 2048)),
              UnitShape("d", 14208, (1024,))] * 2
    units = [recipe_unit(O, 1, 0, 14, seed=70 + i, r=(64, 16)[i % 2], shape=s, act=act, G=128, method="alg1", qr="none")
             for i, s in enumerate(shapes)]
    mask = [i != 3 for i in range(len(shapes))]
    dus = [DeviceUnit(u) for u in units]
    routes = G.glowq_debug_route([d.desc for d in dus])
    assert {r.launch for r in routes} == {0} and [r.k_slices > 1 for r in routes] == [False, False, False, True] * 2
    ws = Workspace([d.desc for d in dus])
    for _ in range(2):
        for d in dus:
            d.clear()
        G.glowq_block_forward([d.desc for d in dus], bytes(mask), ws.ptr, ws.bytes, stream())
        for u, d, on in zip(units, dus, mask):
            for y, ref in zip(d.outputs(), O.group_forward(u, on)):
                assert rel_err(y, ref) <= TOL + ULP[act]
        ws.assert_idle()


def test_cut_contractions_in_a_graph():
    u = recipe_unit(O, 1, 0, 11, r=64, shape=UnitShape("g", 13568, (4176,)), act="bf16", G=128, method="alg1", qr="none")
    du = DeviceUnit(u)
    ws = Workspace([du.desc])
    assert G.glowq_debug_route([du.desc])[0].k_slices > 1
    refs = O.group_forward(u, True)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        G.glowq_group_forward(du.desc, True, ws.ptr, ws.bytes, torch.cuda.current_stream().cuda_stream)
    for _ in range(4):
        du.clear()
        graph.replay()
        torch.cuda.synchronize()
        for y, ref in zip(du.outputs(), refs):
            assert rel_err(y, ref) <= TOL + ULP["bf16"]


# The room for the slices' partial results lies behind the units' slices of the workspace and is not required
@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("T,d_in,d_outs,n,r", [(24, 14208, (4096,), 1, 72), (9, 13696, (1000, 600), 2, 16)])
def test_room_for_partial_results_is_optional(T, d_in, d_outs, n, r, act):
    u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=128, method="alg1", qr="none")
    dus = [DeviceUnit(u) for _ in range(n)]
    descs = [d.desc for d in dus]
    need, slices = G.glowq_workspace_bytes(descs), 0
    for d in descs:
        bare = G.glowq_unit.from_buffer_copy(d)
        bare.modules = None
        slices += G.glowq_workspace_bytes([bare])
    assert need > slices and all(r.k_slices > 1 for r in G.glowq_debug_route(descs))
    refs, failed = O.group_forward(u, True), torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for nbytes, cut in ((need, True), (need - 256, False), (slices, False), (need, True)):
        buf = torch.zeros(need + 4096, dtype=torch.uint8, device="cuda")
        buf[slices:] = 0xA5
        for _ in range(2):
            for d in dus:
                d.clear()
            G.glowq_block_forward(descs, bytes([1] * n), buf.data_ptr(), nbytes, stream())
            for y, ref in zip([y for d in dus for y in d.outputs()], refs * n):
                assert np.isfinite(y).all() and rel_err(y, ref) <= TOL + ULP[act]
        G.glowq_workspace_status(descs, buf.data_ptr(), nbytes, failed.data_ptr(), stream())
        torch.cuda.synchronize()
        assert int(failed.item()) == 0
        assert bool((buf[slices:need] != 0xA5).any()) == cut and bool((buf[need:] == 0xA5).all())
    with pytest.raises(G.GlowqError) as e:
        G.glowq_block_forward(descs, bytes([1] * n), buf.data_ptr(), slices - 1, stream())
    assert e.value.status == G.GLOWQ_ERR_WORKSPACE


def test_a_workspace_for_64_tokens_serves_fewer():
    u = recipe_unit(O, 1, 0, 64, r=72, shape=UnitShape("g", 14208, (4096,)), act="bf16", G=128, method="alg1", qr="none")
    du = DeviceUnit(u)
    ws = Workspace([du.desc])
    for T in (64, 32, 24, 11, 5):
        du.clear()
        G.glowq_group_forward(du.describe(T=T), True, ws.ptr, ws.bytes, stream())
        for y, ref in zip(du.outputs(T), O.group_forward(dict(u, X=u["X"][:T]), True)):
            assert rel_err(y, ref) <= TOL + ULP["bf16"]


# Tiles of 64 tokens that hold 48 of them: the last call that fits and the first that does not, in one, two and three token tiles
@pytest.mark.parametrize("T,d_in,d_outs,act,tile", [
    (48, 2688, (12008,), "f16", 5), (49, 2688, (10008,), "f16", 5), (96, 2688, (6008,), "f16", 5), (97, 2688, (6008,), "f16", 5),
    (48, 640, (20008,), "f16", 6), (49, 128, (20008,), "f16", 6), (96, 128, (12008,), "f16", 6), (145, 128, (8008,), "f16", 6),
    (144, 5888, (4008,), "bf16", 5), (145, 5888, (4008,), "bf16", 5), (144, 128, (10008,), "bf16", 6), (145, 128, (10008,), "bf16", 6)])
def test_tiles_of_three_token_blocks(T, d_in, d_outs, act, tile):
    u = recipe_unit(O, 1, 0, T, r=72, shape=UnitShape("g", d_in, d_outs), act=act, G=64, method="alg1", qr="none")
    for restore in (True, False):
        ys, du, _ = run_group(u, restore, out="act", ldy_pad=8)
        r = G.glowq_debug_route([du.desc])[0]
        assert (r.kernel, r.tile) == (G.GLOWQ_ROUTE_BATCHED, tile)
        assert G.glowq_debug_tile_height([du.desc]) == [48 if T % 48 == 0 else 64]
        for y, ref in zip(ys, O.group_forward(u, restore)):
            assert np.isfinite(y).all() and rel_err(y, ref) <= TOL + ULP[act]


# tiles of 128 rows, which launches of several units take: rows that end inside a workgroup and straddle modules, ragged
# tokens, whole contractions and cut ones, both kinds of dequantisation
@pytest.mark.parametrize("act,T,d_in,d_outs,n,r,slices", [
    ("f16", 21, 1152, (4096, 2056), 12, 16, 1), ("bf16", 21, 1152, (6152,), 12, 72, 1), ("f16", 21, 8320, (520, 512), 8, 72, 3),
    ("bf16", 31, 8320, (1032,), 12, 16, 2), ("f16", 45, 4224, (4104,), 8, 72, 1), ("bf16", 61, 4224, (3072, 8), 12, 16, 1)])
def test_tiles_of_128_rows(act, T, d_in, d_outs, n, r, slices):
    for Gs in (128, 64):
        u = recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=Gs, method="alg1", qr="none")
        dus = [DeviceUnit(u) for _ in range(n)]
        descs = [d.desc for d in dus]
        assert {(q.kernel, q.tile, q.k_slices, q.launch) for q in G.glowq_debug_route(descs)} == {(G.GLOWQ_ROUTE_BATCHED, 9, slices, 0)}
        ws = Workspace(descs)
        for mask in ([True] * n, [i % 3 == 1 for i in range(n)]):
            for d in dus:
                d.clear()
            G.glowq_block_forward(descs, bytes(mask), ws.ptr, ws.bytes, stream())
            refs = {on: O.group_forward(u, on) for on in set(mask)}
            for d, on in zip(dus, mask):
                for y, ref in zip(d.outputs(), refs[on]):
                    assert np.isfinite(y).all() and rel_err(y, ref) <= TOL
            ws.assert_idle()
