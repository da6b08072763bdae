"""The patch matrix of small dense convolutions (im2col_k, csrc/k_conv.hip), through the weight gradient that reads it."""
import pytest

import synth
from harness import Pair, TOL, assert_close
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# cin, cout, kh, kw, stride, ph, pw, h, w, batch.  One group of 8 columns; groups that do not divide 256 (threads left over); more
# than 256 groups (one pixel at a time); images of one pixel and one column (a block spans many); more pixels than 2048 blocks write
# at once; padding columns; taps that only ever see padding; windows too long for the kernels along one axis
CASES = [(1, 8, 1, 7, 1, 0, 3, 1, 40, 5), (3, 8, 3, 3, 2, 1, 1, 33, 29, 3), (7, 16, 3, 3, 1, 1, 1, 9, 5, 7), (8, 8, 3, 3, 1, 1, 1, 1, 1, 300),
         (5, 16, 5, 5, 2, 2, 2, 3, 300, 2), (232, 8, 3, 3, 1, 1, 1, 6, 5, 2), (3, 16, 3, 3, 2, 1, 1, 512, 515, 5), (9, 24, 1, 11, 1, 0, 5, 1, 61, 9)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_patches_at_their_edges(case, dtype):
    import paper_2110_02781_amd.binding as B
    cin, cout, kh, kw, stride, ph, pw, h, w, batch = case
    print(f"patches {case} {dtype}", flush=True)
    o = [OM.Unit('conv', cin, cout, kh, kw, stride, ph, pw, act=L.ACT_NONE)]
    d = [dict(kind=B.UNIT_CONV, cin=cin, cout=cout, kh=kh, kw=kw, stride=stride, pad_h=ph, pad_w=pw, act=L.ACT_NONE)]
    tol = TOL[dtype]
    pair = Pair(o, d, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="off")
    try:
        y, yo = pair.forward(0, synth.normal(31, "x", (batch, h, w, cin)))
        assert_close(y, yo, tol, "y")
        dx, dxo = pair.backward(0, synth.normal(31, "dy", yo.shape))
        assert_close(dx, dxo, tol, "dx")
        pair.compare_unit_vectors("grads", tol, floor=1e-6)
    finally:
        pair.close()
