"""Pointwise layers on the long-reduction kernel (csrc/k_gemm_deep.hip) against the float64 oracle, in bfloat16 with bfloat16 storage:
CASES and CASES_F32 are layers on both sides of its limits, TILES runs every tile in either direction at its edges."""
import pytest

import synth
from harness import Pair, TOL, assert_close, routes
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (rows as h, w, batch; cin, cout): a last row tile of one row, columns off 32, reductions off 64, of a single step and of many; both sides of
# 8192 rows and of 2048
CASES = [(3, 683, 1, 64, 32), (3, 683, 1, 72, 480), (41, 50, 1, 96, 320), (41, 50, 1, 64, 576), (41, 100, 1, 64, 960), (41, 50, 1, 96, 1280),
         (50, 52, 1, 64, 1280), (37, 100, 1, 64, 1280), (64, 128, 1, 88, 136), (8193, 1, 1, 200, 88), (7, 7, 64, 960, 160), (45, 46, 1, 1280, 72),
         (2048, 1, 1, 200, 64), (2049, 1, 1, 56, 64)]
# short reductions, fewer rows than 2048, both sides of what widens them at 8192 and 16384 rows, and of 32768 rows
CASES += [(7, 10, 10, 960, 320), (2051, 1, 1, 24, 144), (8193, 1, 1, 32, 96), (8193, 1, 1, 32, 104), (16385, 1, 1, 40, 96), (32769, 1, 1, 64, 32)]


@pytest.mark.parametrize("h,w,batch,cin,cout", CASES)
def test_deep_tiles(h, w, batch, cin, cout):
    import paper_2110_02781_amd.binding as B
    print(f"deep tiles {h}x{w} batch {batch} {cin}->{cout}", flush=True)
    o = [OM.Unit('conv', cin, cin, act=L.ACT_RELU6), OM.Unit('conv', cin, cout, act=L.ACT_NONE)]
    unit = lambda co, act: dict(kind=B.UNIT_CONV, cin=cin, cout=co, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=act)
    hu = [unit(cin, B.ACT_RELU6), unit(cout, B.ACT_NONE)]
    # the second unit alone (its input as stored), and behind the first (through that one's BatchNorm and activation)
    for a in (1, 0):
        pair = Pair(o, hu, (h, w, cin), batch, a, 2, "bf16", seed=8, ties="off" if a else "bounded")
        try:
            x = synth.normal(51, "x", (batch, h, w, cin))
            y, yo = pair.forward(0, x)
            assert_close(y, yo, TOL["bf16"], "y")
            if a == 0:
                continue
            dx, dxo = pair.backward(0, synth.normal(51, "dy", yo.shape))
            assert_close(dx, dxo, TOL["bf16"], "dx")
            pair.compare_unit_vectors("grads", TOL["bf16"], floor=1e-6)
            pair.compare_unit_vectors("bn", TOL["bf16"])
        finally:
            pair.close()


# fp32: rows off 32, 64 and 128, reductions off 32 and of a single step, columns off 32, more and fewer than 256 blocks;
# both sides of the short kernel's limit of products (700 rows), of 4096 and 16384 rows for forward layers that widen, of 65536 rows
CASES_F32 = [(3, 683, 1, 64, 32), (3, 683, 1, 72, 480), (41, 100, 1, 64, 960), (41, 50, 1, 96, 1280), (37, 100, 1, 64, 1280), (64, 128, 1, 88, 136),
             (8193, 1, 1, 200, 88), (7, 10, 10, 960, 320), (7, 7, 64, 960, 160), (45, 46, 1, 1280, 72), (2049, 1, 1, 24, 40), (4097, 1, 1, 24, 56),
             (16385, 1, 1, 200, 96), (16384, 1, 1, 64, 72), (16385, 1, 1, 64, 72), (33001, 1, 1, 72, 40), (256, 257, 1, 32, 40)]


@pytest.mark.parametrize("h,w,batch,cin,cout", CASES_F32)
def test_deep_tiles_f32(h, w, batch, cin, cout):
    import paper_2110_02781_amd.binding as B
    print(f"deep tiles f32 {h}x{w} batch {batch} {cin}->{cout}", flush=True)
    o = [OM.Unit('conv', cin, cin, act=L.ACT_RELU6), OM.Unit('conv', cin, cout, act=L.ACT_NONE)]
    unit = lambda co, act: dict(kind=B.UNIT_CONV, cin=cin, cout=co, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=act)
    hu = [unit(cin, B.ACT_RELU6), unit(cout, B.ACT_NONE)]
    for a in (1, 0):
        pair = Pair(o, hu, (h, w, cin), batch, a, 2, "f32", seed=8, ties="off" if a else "bounded")
        try:
            x = synth.normal(51, "x", (batch, h, w, cin))
            y, yo = pair.forward(0, x)
            assert_close(y, yo, TOL["f32"], "y")
            dx, dxo = pair.backward(0, synth.normal(51, "dy", yo.shape))
            assert_close(dx, dxo, TOL["f32"], "dx")
            pair.compare_unit_vectors("grads", TOL["f32"], floor=1e-6)
            pair.compare_unit_vectors("bn", TOL["f32"])
        finally:
            pair.close()


# (type, data gradient, tile in units of 32 x 32, rows, reduction, columns): every tile in either direction and type, all three extents off the
# tile (last row tiles of one row and of dozens), a reduction of one step and of several
TILES = [("f32", False, "1x1", 2049, 16, 40), ("f32", False, "2x1", 3137, 16, 232), ("f32", False, "2x2", 2600, 16, 584), ("f32", False, "2x3", 3700, 16, 264),
         ("f32", False, "4x2", 3137, 16, 968), ("f32", False, "1x1", 2049, 104, 40), ("f32", False, "2x1", 12545, 104, 40), ("f32", False, "2x2", 25089, 104, 40),
         ("f32", False, "2x3", 12545, 104, 72), ("f32", False, "4x2", 25089, 104, 104),
         ("f32", True, "1x1", 2049, 16, 40), ("f32", True, "2x1", 12545, 16, 40), ("f32", True, "2x2", 25089, 16, 40), ("f32", True, "2x3", 12545, 16, 72),
         ("f32", True, "4x2", 25089, 16, 104), ("f32", True, "1x1", 2049, 104, 40), ("f32", True, "2x1", 12545, 104, 40), ("f32", True, "2x2", 25089, 104, 40),
         ("f32", True, "2x3", 12545, 104, 72), ("f32", True, "4x2", 25089, 104, 104),
         ("bf16", False, "1x1", 2049, 16, 40), ("bf16", False, "2x1", 4100, 16, 200), ("bf16", False, "2x2", 8193, 16, 40), ("bf16", False, "2x3", 4100, 16, 232),
         ("bf16", False, "4x2", 4100, 16, 904), ("bf16", False, "4x3", 16385, 24, 72), ("bf16", False, "4x4", 4100, 16, 680), ("bf16", False, "4x5", 5003, 16, 776),
         ("bf16", False, "1x1", 2049, 104, 40), ("bf16", False, "2x1", 8193, 104, 72), ("bf16", False, "2x2", 8193, 104, 40), ("bf16", False, "2x3", 12545, 104, 72),
         ("bf16", False, "4x2", 16385, 104, 136), ("bf16", False, "4x3", 16385, 104, 72), ("bf16", False, "4x4", 16385, 104, 104), ("bf16", False, "4x5", 25089, 104, 136),
         ("bf16", True, "1x1", 2049, 16, 40), ("bf16", True, "2x1", 8193, 16, 72), ("bf16", True, "2x2", 8193, 16, 40), ("bf16", True, "2x3", 12545, 16, 72),
         ("bf16", True, "4x2", 8193, 16, 392), ("bf16", True, "4x3", 8193, 16, 200), ("bf16", True, "4x4", 8193, 16, 296), ("bf16", True, "4x5", 8193, 16, 456),
         ("bf16", True, "1x1", 2049, 104, 40), ("bf16", True, "2x1", 8193, 104, 72), ("bf16", True, "2x2", 8193, 104, 40), ("bf16", True, "2x3", 12545, 104, 72),
         ("bf16", True, "4x2", 16385, 104, 136), ("bf16", True, "4x3", 16385, 104, 72), ("bf16", True, "4x4", 16385, 104, 104), ("bf16", True, "4x5", 25089, 104, 136)]


def layer(cin, cout):
    import paper_2110_02781_amd.binding as B
    return ([OM.Unit('conv', cin, cin, act=L.ACT_RELU6), OM.Unit('conv', cin, cout, act=L.ACT_NONE)],
            [dict(kind=B.UNIT_CONV, cin=cin, cout=c, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=a) for c, a in ((cin, B.ACT_RELU6), (cout, B.ACT_NONE))])


@pytest.mark.parametrize("dtype,dgrad,tile,rows,red,cols", TILES, ids=["-".join(map(str, c)) for c in TILES])
def test_every_tile_in_either_direction(dtype, dgrad, tile, rows, red, cols):
    print(f"deep tile {tile} {dtype} dgrad {dgrad} {rows} rows {red} -> {cols}", flush=True)
    cin, cout = (cols, red) if dgrad else (red, cols)
    o, hu = layer(cin, cout)
    got = []
    for a in (1,) if dgrad else (1, 0):              # the layer alone, and behind another (through that one's BatchNorm and activation)
        pair = Pair(o, hu, (rows, 1, cin), 1, a, 2, dtype, seed=9, ties="off" if a else "bounded")
        try:
            n = routes(lambda: got.append(pair.forward(0, synth.normal(52, "x", (1, rows, 1, cin)))))
            if not dgrad:
                assert n.get(f"deep {tile} pw_fwd {rows} {cin} {cout}") == (2 if a == 0 and cin == cout else 1), n
                assert_close(*got[-1], TOL[dtype], "y")
                continue
            n = routes(lambda: got.append(pair.backward(0, synth.normal(52, "dy", got[0][1].shape))))
            assert n.get(f"deep {tile} pw_dgrad {rows} {cin} {cout}") == 1, n
            assert_close(*got[-1], TOL[dtype], "dx")
        finally:
            pair.close()


# short reductions that widen the layer, and fp32 reductions of few steps above 32768 rows: both sides of where the streaming kernels take them
@pytest.mark.parametrize("dtype,dgrad,rows,red,cols,here", [("bf16", False, 13108, 160, 320, False), ("bf16", False, 13107, 160, 320, True), ("bf16", False, 14600, 96, 288, False),
                                                            ("bf16", False, 14600, 104, 288, True), ("bf16", True, 9000, 96, 576, False), ("bf16", True, 9000, 88, 576, True),
                                                            ("bf16", True, 9000, 96, 568, True), ("bf16", True, 9000, 128, 768, True), ("f32", False, 32769, 64, 64, False),
                                                            ("f32", False, 32768, 64, 64, True), ("f32", False, 32769, 64, 32, True), ("f32", True, 32769, 32, 40, False),
                                                            ("f32", True, 32769, 40, 48, True)])
def test_layers_that_stay_on_the_streaming_kernels(dtype, dgrad, rows, red, cols, here):
    print(f"deep or streaming {dtype} dgrad {dgrad} {rows} rows {red} -> {cols}", flush=True)
    cin, cout = (cols, red) if dgrad else (red, cols)
    o, hu = layer(cin, cout)
    pair = Pair(o, hu, (rows, 1, cin), 1, 1, 2, dtype, seed=10)
    got = []
    try:
        n = routes(lambda: got.append(pair.forward(0, synth.normal(53, "x", (1, rows, 1, cin)))))
        if dgrad:
            n = routes(lambda: got.append(pair.backward(0, synth.normal(53, "dy", got[0][1].shape))))
        assert any(k.endswith(f"{'pw_dgrad' if dgrad else 'pw_fwd'} {rows} {cin} {cout}") for k in n) == here, n
        assert_close(*got[-1], TOL[dtype], "dx" if dgrad else "y")
    finally:
        pair.close()


# the residual is added in the data gradient of the expand layer: rows off the tile by one and by many, channels off 32, one and several column tiles
@pytest.mark.parametrize("h,w,batch,c,dtype", [(7, 293, 1, 40, "f32"), (40, 65, 1, 72, "f32"), (11, 197, 1, 136, "f32"), (7, 293, 1, 56, "bf16"),
                                                (40, 65, 1, 72, "bf16"), (11, 197, 1, 136, "bf16")])
def test_data_gradients_that_add_a_residual(h, w, batch, c, dtype):
    import paper_2110_02781_amd.binding as B
    print(f"deep residual {dtype} {h}x{w} batch {batch} channels {c}", flush=True)
    o, hu = [OM.Unit('invres', c, c, stride=1, expand=6)], [dict(kind=B.UNIT_INVRES, cin=c, cout=c, stride=1, expand=6)]
    pair = Pair(o, hu, (h, w, c), batch, 0, 1, dtype, seed=11, ties="bounded")
    got = []
    try:
        y, yo = pair.forward(0, synth.normal(54, "x", (batch, h, w, c)))
        assert_close(y, yo, TOL[dtype], "y")
        n = routes(lambda: got.append(pair.backward(0, synth.normal(54, "dy", yo.shape))))
        assert any(k.startswith("deep ") and k.endswith(f" pw_dgrad {batch * h * w} {c} {6 * c}") for k in n), n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
    finally:
        pair.close()
