"""Stride-2 depthwise data gradient that leaves the backward sums of the BatchNorm in front (csrc/k_conv.hip, dw_dgrad_s2_k with SUMS) against the float64 oracle:
that BatchNorm has no pass of its own for them."""
import pytest

import synth
from harness import Pair, TOL, assert_close, launches
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (cin, cout, expand, h, w, batch, copies in the batch): fewer tiles than partials, one more than as many, two and three to a block with a last
# block of fewer; odd sizes, a tile of one row and of one column; slabs of 3, 6 and 8 column groups
CASES = [(8, 16, 3, 41, 51, 1, 1), (16, 24, 6, 9, 17, 19, 1), (8, 8, 3, 8, 16, 513, 27), (24, 16, 6, 33, 35, 60, 6), (16, 32, 4, 45, 50, 48, 4), (8, 16, 6, 2, 1030, 8, 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout,expand,h,w,batch,tile", CASES)
def test_sums_of_the_stride_2_data_gradient(dtype, cin, cout, expand, h, w, batch, tile):
    import paper_2110_02781_amd.binding as B
    print(f"stride 2 sums {dtype} {cin}->{cout} x{expand} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=2, expand=expand)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=2, expand=expand)]
    pair = Pair(o, hu, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="bounded", tile=tile)
    try:
        y, yo = pair.forward(0, synth.normal(51, "x", (batch // tile, h, w, cin)))
        assert_close(y, yo, TOL[dtype], "y")
        got = []
        n = launches(lambda: got.append(pair.backward(0, synth.normal(51, "dy", (batch // tile,) + tuple(pair.out_shape)))))
        rows = batch * ((h + 1) // 2) * ((w + 1) // 2)
        assert n.get("bn_bwd_reduce", 0) == (2 if rows > 2048 else 0), n
        assert_close(*got[0], TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()
