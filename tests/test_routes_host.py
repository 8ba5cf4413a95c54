"""Which kernel serves a forward call, asked of the library on the host (no GPU): the limits of the
classes, what shares a launch, K slices and what waits inside a launch."""
import pytest

import paper_2603_25385_amd as G


def unit(T, d_in, d_outs, r=16, Gs=128, act=G.GLOWQ_F16, out=G.GLOWQ_F32):
    mods = [G.make_module(0, 0, 0, d, d) for d in d_outs]
    return G.make_unit(0, 0, mods, T, d_in, r, Gs, act, out)


def route(*args, slabs=True, **kw):
    return G.glowq_debug_route([unit(*args, **kw)], slabs)[0]


def test_classes_by_token_count():
    K = [(T, route(T, 4096, (4096,)).kernel) for T in (1, 4, 5, 64, 65, 2048, 2049)]
    assert K == [(1, G.GLOWQ_ROUTE_FEW), (4, G.GLOWQ_ROUTE_FEW), (5, G.GLOWQ_ROUTE_BATCHED), (64, G.GLOWQ_ROUTE_BATCHED),
                 (65, G.GLOWQ_ROUTE_BATCHED), (2048, G.GLOWQ_ROUTE_TILED), (2049, G.GLOWQ_ROUTE_TILED)]
    assert route(2049, 256, (64,)).kernel == G.GLOWQ_ROUTE_TILED      # never batched past 2048 tokens
    M = [(T, G.glowq_debug_mx_route(unit(T, 4096, (4096,))).kernel) for T in (1, 4, 5, 16, 17)]
    assert M == [(1, G.GLOWQ_ROUTE_MX_ONE), (4, G.GLOWQ_ROUTE_MX_ONE), (5, G.GLOWQ_ROUTE_MX_SMALL),
                 (16, G.GLOWQ_ROUTE_MX_SMALL), (17, G.GLOWQ_ROUTE_MX_TILED)]


def test_every_batched_tile_is_chosen_for_some_call():
    tiles = {route(T, d_in, (rows,), r=64, act=act).tile
             for act in (G.GLOWQ_F16, G.GLOWQ_BF16) for T in (5, 9, 18, 33, 50, 131)
             for d_in in (128, 256, 384, 768, 1536, 3200, 4352, 8320) for rows in (304, 2008, 5000, 9000, 12008, 20008)
             if route(T, d_in, (rows,), r=64, act=act).kernel == G.GLOWQ_ROUTE_BATCHED}
    assert tiles == set(range(9))


def test_units_that_share_a_launch():
    few = [unit(T, 256, (64,)) for T in (1, 1, 2, 1)]
    assert [r.launch for r in G.glowq_debug_route(few)] == [0, 0, 1, 2]
    batched = [unit(T, 256, (64,)) for T in (9, 16, 17, 32, 33, 64)] + [unit(64, 256, (64,), act=G.GLOWQ_BF16)]
    assert [r.launch for r in G.glowq_debug_route(batched)] == [0, 0, 1, 1, 2, 2, 3]
    assert [r.launch for r in G.glowq_debug_route([unit(24, 256, (64,))] * 17)] == [0] * 16 + [1]
    tiled = [unit(512, 4096, (4096,) * 8)] * 3                        # sixteen module entries per launch
    assert [r.launch for r in G.glowq_debug_route(tiled)] == [0, 0, 1]


def test_k_slices_need_their_slabs():
    assert route(512, 14336, (4096,)).k_slices == 3
    assert route(512, 14336, (4096,), slabs=False).k_slices == 1
    assert route(512, 4096, (4096,)).k_slices == 1


def test_the_choice_knows_whether_k_can_be_cut():
    # without slabs (no workspace, glowq_group_forward_static) a long contraction stays in one piece, and
    # the estimate must be that of one piece: 512 tokens x 2048 rows x 16384 on the tiled kernel's few
    # workgroups take twice the batched kernel's time and more
    assert route(512, 16384, (2048,)).k_slices == 4
    for T, d_in, d_out in ((512, 16384, 2048), (300, 14336, 4096), (257, 16384, 2008)):
        assert route(T, d_in, (d_out,)).kernel == G.GLOWQ_ROUTE_TILED
        assert route(T, d_in, (d_out,), slabs=False).kernel == G.GLOWQ_ROUTE_BATCHED
    # likewise where the module table of a launch has no room for the slices
    full = [unit(700, 16384, (1000,))] + [unit(700, 256, (64,) * 5)] * 3
    assert [r.k_slices for r in G.glowq_debug_route(full)] == [1] * 4


def test_only_consumers_of_r_wait():
    # the projection's own workgroups wait for nothing, so launches whose consumers come in a launch of
    # their own have no wait at all, whether the projection is cut into K slices (past 4096 channels) or not
    for d_in in (4096, 4352, 8192, 16384):
        for T in (17, 130, 2048):
            assert G.glowq_debug_mx_route(unit(T, d_in, (4096,), r=64)).wait_polls == 0, (T, d_in)
        assert G.glowq_debug_mx_route(unit(16, d_in, (4096,), r=64)).wait_polls == 0


def test_the_wait_for_r_is_as_long_on_small_tiles():
    # whichever kernel a call of more than four tokens takes, its consumers look for R a million times
    # (a second and more) before they leave the correction out: a call must not lose it sooner
    # because its tiles are small
    tiled = route(2048, 4096, (14336,))
    assert tiled.kernel == G.GLOWQ_ROUTE_TILED and tiled.wait_polls >= 1 << 20
    for T in (5, 16, 32, 33, 64, 65, 300, 1000):
        small = route(T, 512, (264,))
        assert small.kernel == G.GLOWQ_ROUTE_BATCHED and small.wait_polls >= tiled.wait_polls, T


def test_the_smallest_calls_start_four_waves():
    # two or three K tiles on few rows: a workgroup of eight waves (tiles 2 and 4) takes longer to start
    # and to meet than its second wave group saves
    for T, d_in, d_outs, Gs in [(16, 256, (256,) * 3, 64), (13, 256, (1408,), 128), (9, 384, (512, 512), 128),
                                (24, 256, (256,), 128)]:
        for act in (G.GLOWQ_F16, G.GLOWQ_BF16):
            assert route(T, d_in, d_outs, Gs=Gs, act=act).tile not in (2, 4), (T, d_in, d_outs)


# Calls that cost rules of fewer constants sent to slower tiles than they had run on before those
# rules (us).  Routes that are not slower: B<n> batched tile n, L / H the tiled kernel's large / half-size tiles
NOT_SLOWER = [
    (672, 256, (2512,) * 3, "f16", "act", 128, 128, "L H"),      # 11.2 before, 17.6 then
    (326, 256, (3736,) * 3, "bf16", "act", 16, 64, "L H"),      # 10.1 before, 15.4 then
    (456, 640, (2944,) * 3, "f16", "act", 72, 128, "L H"),      # 16.6 before, 21.2 then
    (7, 1920, (6288,), "f16", "f32", 64, 128, "B7"),      # 7.1 before, 9.1 then
    (6, 1408, (8456,), "f16", "f32", 32, 128, "B2"),      # 6.6 before, 8.4 then
    (9, 1408, (4632,), "f16", "f32", 16, 128, "B2 B7"),      # 6.6 before, 8.4 then
    (8, 1152, (1096,) * 3, "f16", "act", 16, 128, "B0 B2 B7"),      # 6.3 before, 7.8 then
    (891, 512, (5344,), "f16", "f32", 64, 64, "L H"),      # 19.3 before, 23.8 then
    (871, 640, (4632,), "f16", "f32", 64, 128, "L H"),      # 19.5 before, 24.0 then
    (24, 10112, (4960,) * 2, "f16", "act", 16, 64, "B4"),      # 24.2 before, 29.3 then
    (427, 9728, (4032,) * 2, "f16", "f32", 16, 128, "B6 L"),      # 98.9 before, 118.9 then
    (830, 768, (5856,), "f16", "f32", 72, 128, "H"),      # 19.3 before, 23.2 then
    (7, 1536, (1224,), "f16", "act", 32, 64, "B0 B2 B7"),      # 6.9 before, 8.1 then
    (26, 12672, (5008,) * 2, "f16", "act", 64, 64, "B4"),      # 31.0 before, 36.4 then
    (971, 2304, (2656,) * 3, "f16", "act", 72, 128, "L"),      # 61.1 before, 70.8 then
    (10, 1408, (4160,) * 2, "bf16", "act", 64, 64, "B1 B2 B8"),      # 7.9 before, 9.0 then
    (10, 4224, (8608,), "bf16", "act", 32, 128, "B2 B8"),      # 12.6 before, 14.4 then
    (263, 1280, (8912,) * 3, "f16", "act", 128, 128, "L"),      # 43.8 before, 49.9 then
    (5, 1280, (3088,) * 3, "bf16", "act", 64, 128, "B1 B2 B3 B4 B8"),      # 7.5 before, 8.4 then
    (14, 6272, (5320,), "f16", "f32", 64, 128, "B7"),      # 12.6 before, 14.2 then
    (34, 512, (13072,) * 3, "f16", "act", 72, 128, "B6"),      # 12.6 before, 14.1 then
    (7, 3456, (1976,) * 3, "f16", "act", 64, 128, "B7"),      # 8.8 before, 9.8 then
    (16, 256, (344,) * 2, "f16", "f32", 32, 64, "B0 B1 B2 B3 B4 B7 B8"),      # 7.3 before, 8.1 then
    (13, 1152, (4368,), "bf16", "act", 64, 128, "B1 B2 B3 B4 B7 B8"),      # 7.6 before, 8.4 then
    (1357, 14336, (1768,) * 3, "f16", "f32", 16, 128, "L"),      # 219.6 before, 241.9 then
    (10, 3712, (7616,), "bf16", "f32", 72, 64, "B0 B2 B7 B8"),      # 12.4 before, 13.6 then
    (9, 3584, (4696,), "f16", "act", 64, 128, "B7"),      # 7.7 before, 8.4 then
    (7, 1408, (568,) * 3, "bf16", "f32", 64, 64, "B0 B2 B7"),      # 7.4 before, 8.0 then
]


@pytest.mark.parametrize("T,d_in,d_outs,act,out,r,Gs,good", NOT_SLOWER)
def test_calls_keep_their_speed(T, d_in, d_outs, act, out, r, Gs, good):
    a = {"f16": G.GLOWQ_F16, "bf16": G.GLOWQ_BF16}[act]
    got = route(T, d_in, d_outs, r=r, Gs=Gs, act=a, out=a if out == "act" else G.GLOWQ_F32)
    name = "LH"[got.tile] if got.kernel == G.GLOWQ_ROUTE_TILED else f"B{got.tile}"
    assert name in good.split()


def tile_tokens(units):
    return set(G.glowq_debug_tile_tokens(units))


def decoder_layers(hidden, kv, inter, layers, T, r, act, Gs=128):
    shapes = [(hidden, (hidden, kv, kv)), (hidden, (hidden,)), (hidden, (inter, inter)), (inter, (hidden,))] * layers
    return [unit(T, d, outs, r=r, Gs=Gs, act=act, out=act) for d, outs in shapes]


# The projection's workgroups hold places of their own: calls whose wide tiles would fit one round (or a whole number)
# without them, and do not beside them (us on wide tiles, on tiles of 128 tokens)
@pytest.mark.parametrize("T,d_in,d_outs,act,out,r,Gs", [
    (2969, 4224, (4104,), "f16", "act", 128, 128),       # 137.4, 112.3: 204 tiles and 72 projection workgroups
    (1522, 3840, (3256,) * 3, "f16", "act", 16, 128),    # 127.8, 107.2
    (1678, 3456, (4288,) * 2, "f16", "f32", 128, 64),    # 128.0, 108.5
    (1066, 3968, (12328,), "f16", "f32", 128, 64),       # 137.3, 117.5
    (2989, 5376, (2184,) * 2, "f16", "f32", 64, 128),    # 162.2, 139.6
    (1821, 4480, (2120,) * 3, "f16", "f32", 64, 64),     # 136.7, 122.0
    (2145, 4352, (2936,) * 2, "f16", "f32", 128, 64)])   # 139.9, 129.2
def test_no_wide_tiles_where_the_projection_fills_the_round(T, d_in, d_outs, act, out, r, Gs):
    a = {"f16": G.GLOWQ_F16, "bf16": G.GLOWQ_BF16}[act]
    assert tile_tokens([unit(T, d_in, d_outs, r=r, Gs=Gs, act=a, out=a if out == "act" else G.GLOWQ_F32)]) == {128}


def test_no_wide_tiles_where_their_rounds_come_out_uneven():
    # tiles of several lengths, whose rounds are not those of one length (us on wide tiles, on tiles of 128 tokens)
    assert tile_tokens(decoder_layers(4352, 4352, 2944, 1, 761, 16, G.GLOWQ_BF16)) == {128}      # 183.9, 166.4
    assert tile_tokens(decoder_layers(3968, 3968, 12288, 2, 521, 128, G.GLOWQ_F16)) == {128}     # 529.4, 487.5


def test_wide_tiles_where_they_are_faster():
    assert tile_tokens([unit(2048, 4096, (11008,) * 2, r=64, act=G.GLOWQ_BF16, out=G.GLOWQ_BF16)]) == {256}
    assert tile_tokens(decoder_layers(4096, 1024, 14336, 1, 512, 128, G.GLOWQ_F16)) == {256}
    assert tile_tokens(decoder_layers(5120, 5120, 13824, 4, 1000, 64, G.GLOWQ_F16)) == {256}


def test_the_order_of_units_does_not_decide_the_tile():
    # units of several token counts in one launch: what most of its work belongs to decides, first or last
    for act in (G.GLOWQ_F16, G.GLOWQ_BF16):
        def of(T, rows):
            return unit(T, 4096, rows, r=64, act=act, out=act)

        for units, tokens in (([of(2048, (14336,) * 2), of(1024, (14336,) * 2), of(70, (1024,))], 256),
                              ([of(2048, (1024,)), of(70, (32768,) * 3)], 128)):
            for u in (units, units[::-1]):
                routes = G.glowq_debug_route(u)
                assert {r.launch for r in routes} == {0} and {r.kernel for r in routes} == {G.GLOWQ_ROUTE_TILED}
                assert tile_tokens(u) == {tokens}


# The batched kernel has to beat the tile that the call would take (us on wide tiles, on the batched kernel)
@pytest.mark.parametrize("T,d_in,d_outs,out,r,Gs", [
    (420, 3968, (8744,) * 2, "act", 128, 128),      # 78.3, 97.6
    (385, 6528, (5512,) * 3, "f32", 128, 64),       # 119.3, 144.3
    (394, 4224, (8712,) * 2, "f32", 128, 128),      # 87.1, 104.1
    (388, 3456, (5784,) * 3, "f32", 16, 64),        # 72.9, 82.5
    (407, 7296, (5760,) * 3, "f32", 16, 128),       # 134.7, 149.2
    (428, 5888, (8464,) * 2, "act", 64, 128)])      # 111.9, 121.4
def test_the_batched_kernel_is_compared_with_the_chosen_tile(T, d_in, d_outs, out, r, Gs):
    u = unit(T, d_in, d_outs, r=r, Gs=Gs, out=G.GLOWQ_F16 if out == "act" else G.GLOWQ_F32)
    assert tile_tokens([u]) == {256}


# calls of the microscaling variant that were slower on small tiles (us on tiles 0 .. 4)
@pytest.mark.parametrize("T,d_in,d_outs,act,out", [
    (1931, 896, (8680,) * 3, "f16", "f32"),          # 99.8 .. 128.1 on tile 4
    (1938, 512, (12712,) * 3, "bf16", "act"),        # 121.6, 323.3, 320.6, 171.8, 155.7
    (1018, 7424, (10352,), "bf16", "f32"),           # 86.2, 203.8, 147.1, 112.5, 95.6
    (1364, 12288, (4600,), "bf16", "act"),           # 113.8, 249.6, 232.0, 158.9, 126.7
    (1155, 3200, (5624,) * 3, "bf16", "act"),        # 114.3, 256.6, 216.1, 145.9, 126.0
    (522, 8320, (2752,) * 3, "bf16", "f32"),         # 75.0, 141.1, 106.8, 90.7, 86.2
    (1182, 9216, (2176, 2176), "bf16", "act")])      # 79.2, 153.7, 139.0, 96.1, 85.5
def test_microscaling_keeps_large_tiles_where_they_are_faster(T, d_in, d_outs, act, out):
    a = {"f16": G.GLOWQ_F16, "bf16": G.GLOWQ_BF16}[act]
    u = unit(T, d_in, d_outs, r=64, act=a, out=a if out == "act" else G.GLOWQ_F32)
    assert G.glowq_debug_mx_route(u).tile == 0


# Units that wait for projections are not cut where that took longer (us whole, cut)
@pytest.mark.parametrize("units,T,r,act", [
    ([(9088, (192,) * 3)] * 2, 10, 64, "f16"),          # 12.9, 14.6
    ([(9088, (192,) * 3)] * 4, 10, 64, "bf16"),         # 15.5, 17.9
    ([(13568, (1168,))] * 2, 11, 64, "f16"),            # 19.2, 21.3
    ([(13568, (1168,))] * 4, 11, 64, "bf16"),           # 23.2, 25.8
    ([(9088, (480,))] * 4, 13, 64, "bf16"),             # 15.7, 18.7
    ([(8320, (424,))] * 2, 10, 128, "f16"),             # 11.8, 14.6
    ([(11136, (256,) * 2)] * 2, 31, 128, "bf16"),       # 17.6, 22.2
    ([(13056, (3056,))] * 2, 11, 128, "bf16"),          # 24.0, 33.7
    ([(9472, (1392,)), (2816, (4504,))], 8, 64, "bf16"),           # 16.3, 17.6
    # one that would fill the chip with three slices
    ([(10624, (1768,) * 3)], 14, 128, "f16"),           # 18.9, 22.0
    ([(11520, (1712,) * 3)], 17, 128, "f16")])          # 22.0, 24.4
def test_corrected_units_run_whole_where_that_is_faster(units, T, r, act):
    a = {"f16": G.GLOWQ_F16, "bf16": G.GLOWQ_BF16}[act]
    assert all(x.k_slices == 1 for x in G.glowq_debug_route([unit(T, d, o, r=r, act=a, out=a) for d, o in units]))


def test_whole_layers_are_cut_where_that_is_faster():
    for hidden, kv, inter, layers, T, r, act in [(4096, 1024, 14336, 1, 24, 128, G.GLOWQ_F16), (4096, 1024, 14336, 1, 24, 128, G.GLOWQ_BF16),
                                                 (768, 768, 13056, 1, 31, 64, G.GLOWQ_F16), (512, 512, 7552, 4, 7, 64, G.GLOWQ_BF16)]:
        ks = [x.k_slices for x in G.glowq_debug_route(decoder_layers(hidden, kv, inter, layers, T, r, act))]
        assert min(ks[3::4]) > 1


def test_third_slices_for_all_units_of_a_launch_or_for_none():
    # (a third slice for the first of two down projections left the second one whole: us in two slices each, and so)
    for T, r, layers, want in [(100, 64, 1, 3), (100, 16, 2, 2),             # 2 x 3584 / 9984: 117.5, 156.3
                               (104, 64, 2, 2), (113, 16, 4, 2),             # 4 x 4736 / 11136: 295.6, 371.1
                               (100, 128, 1, 3), (129, 64, 1, 2)]:
        for hidden, inter in ((4096, 11008), (3584, 9984), (4736, 11136)):
            routes = G.glowq_debug_route(decoder_layers(hidden, hidden, inter, layers, T, r, G.GLOWQ_F16))
            assert {x.kernel for x in routes} == {G.GLOWQ_ROUTE_TILED} and [x.k_slices for x in routes[3::4]] == [want] * layers
    # (85.4 in two slices and on the batched kernel, 92.4 in three)
    assert {x.kernel for x in G.glowq_debug_route(decoder_layers(3072, 3072, 10752, 1, 111, 128, G.GLOWQ_F16))} == {G.GLOWQ_ROUTE_BATCHED}
    wide = [unit(108, d, o, r=16) for d, o in ((6528, (5928,)), (10368, (5944,) * 2), (3328, (1408,) * 2))]        # 77.1, 89.9
    assert [x.k_slices for x in G.glowq_debug_route(wide)] == [1, 2, 1]
    for T in (70, 107, 125):                   # a unit alone: 2 x 5560 rows x 11008 at 107 tokens 75.9 us, in three slices 93.9
        assert all(route(T, 11008, rows, r=128).k_slices <= 2 for rows in ((5560,) * 2, (4096,), (7848,) * 2))


# Short calls with a correction that fewer tokens a tile moved to half-size tiles (us on the batched kernel, on these)
@pytest.mark.parametrize("T,d_in,d_outs,r,Gs,act", [
    (172, 3200, (5384,) * 3, 128, 64, "f16"),       # 44.5, 58.9
    (151, 2048, (5536,) * 2, 128, 128, "f16"),      # 29.9, 43.3
    (65, 1280, (5576,) * 3, 64, 128, "f16"),        # 20.4, 24.8
    (94, 2048, (5904,) * 3, 64, 64, "f16"),         # 28.7, 36.7
    (179, 2048, (5728,) * 3, 64, 128, "f16"),       # 30.9, 39.4
    (66, 3968, (6040,) * 3, 128, 128, "bf16")])     # 44.7, 54.3
def test_short_corrected_calls_keep_the_batched_kernel(T, d_in, d_outs, r, Gs, act):
    a = {"f16": G.GLOWQ_F16, "bf16": G.GLOWQ_BF16}[act]
    assert route(T, d_in, d_outs, r=r, Gs=Gs, act=a, out=a).kernel == G.GLOWQ_ROUTE_BATCHED
    layer = decoder_layers(2944, 736, 3072, 1, 67, 128, G.GLOWQ_F16)           # 33.2, 47.0
    assert {x.kernel for x in G.glowq_debug_route(layer)} == {G.GLOWQ_ROUTE_BATCHED}


def test_tile_heights_are_those_of_the_launch():
    for T, height in [(65, 80), (80, 80), (81, 96), (97, 112), (113, 128), (129, 80), (300, 112), (521, 112), (1024, 128)]:
        u = unit(T, 768, (16008,) * 3, act=G.GLOWQ_BF16, out=G.GLOWQ_BF16)
        assert G.glowq_debug_tile_height([u]) == [height] and G.glowq_debug_tile_tokens([u]) == [128]
    assert G.glowq_debug_tile_height([unit(2048, 4096, (11008,) * 2, r=64, act=G.GLOWQ_BF16, out=G.GLOWQ_BF16)]) == [256]
    # batched: 48 of the 64 tokens that tiles 5 and 6 hold
    for T, d, rows, height in [(48, 2688, 12008, 48), (49, 2688, 10008, 64), (16, 1024, 4096, 16), (32, 2048, 14336, 32)]:
        assert G.glowq_debug_tile_height([unit(T, d, (rows,))]) == [height]
    assert G.glowq_debug_tile_height([unit(4, 1024, (4096,))]) == [0]


def test_argument_checks():
    for units, status in [([unit(0, 256, (64,))], G.GLOWQ_ERR_SHAPE), ([unit(4, 192, (64,))], G.GLOWQ_ERR_SHAPE),
                          ([unit(4, 320, (64,), Gs=64)], G.GLOWQ_ERR_UNSUPPORTED)]:
        with pytest.raises(G.GlowqError) as e:
            G.glowq_debug_route(units)
        assert e.value.status == status
    bare = unit(20, 256, (64,))
    bare.modules = None
    for call in (lambda: G.glowq_debug_route([bare]), lambda: G.glowq_debug_mx_route(bare)):
        with pytest.raises(G.GlowqError) as e:
            call()
        assert e.value.status == G.GLOWQ_ERR_NULL
