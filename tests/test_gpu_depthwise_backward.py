"""Depthwise layers backward in one pass (csrc/k_conv.hip, dw_bwd_k): data gradient, weight gradient and the BatchNorm sums of the layer in front, which has no
pass of its own for them, against the float64 oracle."""
import pytest

import synth
from harness import Pair, TOL, assert_close, launches, launches_by_shape
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (stride, cin, cout, expand, h, w, batch, copies in the batch).  Fewer tiles than partials, one more than as many, two and three to a block with a
# last block of fewer, more than go through one chain of additions; odd sizes, a tile of one row and of one column; slabs of 1, 3, 6 and 8 column groups, a last slab of fewer; images of 7, 14 and 28
# rows (tiles of 7 in bfloat16) and one row more; an output of up to 2048 rows (its BatchNorm backward is a launch of its own)
CASES = [(2, 8, 16, 3, 41, 51, 1, 1), (2, 16, 24, 6, 9, 17, 19, 1), (2, 8, 8, 3, 8, 16, 513, 27), (2, 24, 16, 6, 33, 35, 60, 6), (2, 16, 32, 4, 45, 50, 48, 4),
         (2, 8, 16, 6, 2, 1030, 8, 1), (2, 16, 16, 6, 7, 1, 700, 35), (2, 8, 8, 3, 8, 16, 13311, 459),
         (1, 8, 16, 3, 41, 51, 1, 1), (1, 16, 24, 6, 14, 14, 32, 4), (1, 16, 16, 5, 15, 14, 33, 3), (1, 24, 24, 6, 28, 30, 4, 1), (1, 8, 8, 3, 8, 16, 513, 27),
         (1, 24, 16, 6, 33, 35, 60, 6), (1, 88, 40, 6, 7, 7, 64, 8), (1, 8, 16, 6, 2, 1030, 3, 1), (1, 16, 8, 6, 2051, 1, 1, 1), (1, 8, 8, 3, 8, 16, 8721, 459)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,cin,cout,expand,h,w,batch,tile", CASES)
def test_depthwise_backward_in_one_pass(dtype, stride, cin, cout, expand, h, w, batch, tile):
    import paper_2110_02781_amd.binding as B
    print(f"depthwise backward {dtype} stride {stride} {cin}->{cout} x{expand} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=stride, expand=expand)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=expand)]
    pair = Pair(o, hu, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="bounded", tile=tile)
    try:
        y, yo = pair.forward(0, synth.normal(51, "x", (batch // tile, h, w, cin)))
        assert_close(y, yo, TOL[dtype], "y")
        got = []
        n = launches_by_shape(lambda: got.append(pair.backward(0, synth.normal(51, "dy", (batch // tile,) + tuple(pair.out_shape)))))
        # passes for sums: one for the block's last BatchNorm (long ones), one for the layer's own where the data gradient behind it leaves none (beyond the long-reduction
        # kernel's rows a rule's matter), none for the layer in front: at stride 1, where the two are of one shape, one at most
        rows, rows_out, c = h * w * batch, batch * pair.out_shape[0] * pair.out_shape[1], cin * expand
        passes = {k: v for k, v in n.items() if k.startswith("bn_bwd_reduce")}
        own = passes.pop(f"bn_bwd_reduce {rows_out} {c} 2", 0)
        assert own <= (1 if rows_out > 16384 else 0), n
        assert passes == ({f"bn_bwd_reduce {rows_out} {cout} 0": 1} if rows_out > 2048 else {}), n
        assert n.get(f"dw_bwd {rows} {c} {stride}", 0) == 1, n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stem,stride,cin,cout,h,w,batch", [(True, 1, 16, 24, 41, 51, 2), (True, 2, 24, 16, 30, 45, 4), (True, 1, 16, 16, 41, 51, 2), (False, 1, 24, 24, 37, 60, 3),
                                                            (False, 2, 16, 24, 61, 55, 3), (False, 1, 16, 8, 9, 9, 3)])
def test_depthwise_layer_without_expansion(dtype, stem, stride, cin, cout, h, w, batch):
    """Its input is the view of a convolution in front (whose BatchNorm gets its sums, unless a residual is added on the way) or as it is stored; a
    second backward without an input gradient adds to the first one's gradients."""
    import paper_2110_02781_amd.binding as B
    print(f"depthwise backward, no expansion {dtype} stem {stem} stride {stride} {cin}->{cout} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=stride, expand=1)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=1)]
    if stem:
        o.insert(0, OM.Unit('conv', 8, cin, act=L.ACT_RELU6))
        hu.insert(0, dict(kind=B.UNIT_CONV, cin=8, cout=cin, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=B.ACT_RELU6))
    c = 8 if stem else cin
    pair = Pair(o, hu, (h, w, c), batch, 0, len(o), dtype, n_slots=2, seed=8, ties="bounded")
    try:
        for slot in range(2):
            y, yo = pair.forward(slot, synth.normal(51, f"x{slot}", (batch, h, w, c)))
            assert_close(y, yo, TOL[dtype], "y")
        for slot in range(2):
            got = []
            n = launches(lambda: got.append(pair.backward(slot, synth.normal(51, f"dy{slot}", yo.shape), want_dx=slot == 0)))
            assert n.get("dw_bwd", 0) == 1, n
            if slot == 0:
                assert_close(*got[0], TOL[dtype], "dx")
            pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
    finally:
        pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("act", ["relu", "none"])
@pytest.mark.parametrize("stride,cin,cout,h,w,batch", [(1, 16, 24, 41, 51, 2), (2, 24, 16, 30, 45, 4)])
def test_depthwise_layer_behind_other_activations(dtype, act, stride, cin, cout, h, w, batch):
    """Without expansion the view in front is that of a convolution with an activation of its own, or none."""
    import paper_2110_02781_amd.binding as B
    print(f"depthwise backward behind {act} {dtype} stride {stride} {cin}->{cout} {h}x{w}", flush=True)
    oact, hact = (L.ACT_RELU, B.ACT_RELU) if act == "relu" else (L.ACT_NONE, B.ACT_NONE)
    o = [OM.Unit('conv', 8, cin, act=oact), OM.Unit('invres', cin, cout, stride=stride, expand=1)]
    hu = [dict(kind=B.UNIT_CONV, cin=8, cout=cin, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=hact), dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=1)]
    pair = Pair(o, hu, (h, w, 8), batch, 0, 2, dtype, seed=8, ties="bounded")
    try:
        y, yo = pair.forward(0, synth.normal(51, "x", (batch, h, w, 8)))
        assert_close(y, yo, TOL[dtype], "y")
        got = []
        n = launches_by_shape(lambda: got.append(pair.backward(0, synth.normal(51, "dy", yo.shape))))
        assert n.get(f"dw_bwd {h * w * batch} {cin} {stride}", 0) == 1 and f"bn_bwd_reduce {h * w * batch} {cin} {hact}" not in n, n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()


# input rows (h * w * batch) at each line of the split: up to 256 | 512 | 1024 | 2048, up to 512 channels and more, and one row or pixel beyond
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride,cin,cout,expand,h,w,batch", [(1, 8, 8, 4, 16, 16, 1), (1, 128, 24, 4, 257, 1, 1), (2, 24, 16, 4, 16, 16, 2), (1, 16, 16, 6, 19, 27, 1), (2, 16, 16, 6, 9, 19, 3),
                                                             (1, 32, 32, 6, 16, 16, 4), (2, 32, 24, 6, 41, 25, 1), (1, 32, 32, 6, 32, 32, 2), (1, 104, 24, 5, 257, 1, 1), (1, 104, 24, 5, 19, 27, 1),
                                                             (2, 104, 24, 5, 5, 41, 5), (1, 104, 104, 5, 16, 16, 8)])
def test_short_depthwise_backward(dtype, stride, cin, cout, expand, h, w, batch):
    """Up to 2048 rows: both BatchNorm backwards in the same launch (dw_bwd_small_k)."""
    import paper_2110_02781_amd.binding as B
    print(f"short depthwise backward {dtype} stride {stride} {cin}->{cout} x{expand} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=stride, expand=expand)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=expand)]
    pair = Pair(o, hu, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="bounded")
    try:
        y, yo = pair.forward(0, synth.normal(51, "x", (batch, h, w, cin)))
        assert_close(y, yo, TOL[dtype], "y")
        got = []
        n = launches(lambda: got.append(pair.backward(0, synth.normal(51, "dy", yo.shape))))
        assert n.get("dw_bwd_small", 0) == 1 and n.get("dw_bwd", 0) == 0, n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()


# (widths of the blocks in front, in the middle (residual) and behind, expansion, h, w, batch): rows off every tile, columns off 32 and 64; more rows than the
# long-reduction kernels take; up to 256 partial sums and more.  Last, by type, of the two blocks that have another behind them those whose last BatchNorm keeps a pass for
# its sums: behind the widest fused backward (bfloat16, more than 32 columns), and where a pass leaves few enough partial sums to be finished where they are
# applied and the data gradient does not (24 columns but for one fused backward); and of the three blocks those whose depthwise BatchNorm does (the last again).
CHAINS = [(24, 40, 48, 6, 37, 61, 1, (0, 2), (0, 0)), (16, 88, 96, 6, 41, 51, 2, (0, 0), (0, 0)), (40, 96, 160, 5, 33, 35, 8, (0, 0), (0, 0)), (16, 24, 32, 6, 64, 65, 16, (2, 0), (0, 0)),
          (16, 24, 32, 4, 128, 130, 5, (2, 2), (1, 0))]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c0,c1,c2,expand,h,w,batch,front,depthwise", CHAINS)
def test_sums_left_by_data_gradients(dtype, c0, c1, c2, expand, h, w, batch, front, depthwise):
    """Project layers leave the backward sums of the depthwise BatchNorm, expand layers (one of them adding a residual) those of the block in front."""
    import paper_2110_02781_amd.binding as B
    print(f"sums left by data gradients {dtype} {c0}->{c1}->{c1}->{c2} x{expand} {h}x{w} batch {batch}", flush=True)
    dims = [(c0, c1, 1), (c1, c1, 1), (c1, c2, 2)]
    o = [OM.Unit('invres', i, k, stride=s, expand=expand) for i, k, s in dims]
    hu = [dict(kind=B.UNIT_INVRES, cin=i, cout=k, stride=s, expand=expand) for i, k, s in dims]
    pair = Pair(o, hu, (h, w, c0), batch, 0, 3, dtype, seed=8, ties="bounded")
    try:
        y, yo = pair.forward(0, synth.normal(51, "x", (batch, h, w, c0)))
        assert_close(y, yo, TOL[dtype], "y")
        got = []
        n = launches_by_shape(lambda: got.append(pair.backward(0, synth.normal(51, "dy", yo.shape))))
        by, rows, rows_out = dtype == "bf16", h * w * batch, yo.shape[0] * yo.shape[1] * yo.shape[2]
        want = {f"bn_bwd_reduce {rows} {c1} 0": front[by], f"bn_bwd_reduce {rows_out} {c1 * expand} 2": depthwise[by],
                f"bn_bwd_reduce {rows_out} {c2} 0": 1 if rows_out > 2048 else 0}             # nothing is behind the last block
        assert {k: v for k, v in n.items() if k.startswith("bn_bwd_reduce")} == {k: v for k, v in want.items() if v}, n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()
