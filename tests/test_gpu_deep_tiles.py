"""Pointwise layers on the long-reduction kernel (csrc/k_gemm_deep.hip): every tile shape, at its edges, against the float64
oracle, in bfloat16 with bfloat16 storage."""
import pytest

import synth
from harness import Pair, TOL, assert_close
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (rows as h, w, batch; cin, cout): the tiles that forward (cin -> cout) and data gradient (cout -> cin) take, in units of 32 x 32: a last
# row tile of one row, columns off 32, reductions off 64, of a single step and of many; both sides of 8192 rows and of 2048
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


# fp32: every tile in either direction, rows off 32, 64 and 128, reductions off 32 and of a single step, columns off 32, more and fewer than 256 blocks;
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
