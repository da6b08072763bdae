"""The BatchNorm in front of an average takes its backward sums from what the average's forward has counted (csrc/k_elem.hip, gap_fwd_k with open, gap_bwd_k
with sums; csrc/k_gemm.hip, fc_bwd_k with sums): no pass over the tensor for them, results against the float64 oracle."""
import pytest

import synth
from harness import Pair, TOL, assert_close, launches
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (windows or images as h, w, batch; channels; taps: 0 a pointwise layer; relu; a fully connected layer behind): one launch with the
# fully connected layer's (up to 1 M values) and one of its own, images off 16 and off a chunk of 8, more than 512 of them, channels off 256
CASES = [(1, 128, 8, 64, 5, "relu", True), (1, 33, 9, 24, 3, "relu6", True), (1, 200, 13, 32, 5, "relu", True), (1, 130, 70, 64, 5, "relu", False),
         (7, 7, 50, 264, 0, "relu6", True), (9, 11, 33, 520, 0, "none", True), (2, 2, 600, 40, 0, "relu6", True), (5, 5, 85, 72, 0, "relu", False)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,w,batch,c,taps,act,fc", CASES)
def test_sums_from_the_average(dtype, h, w, batch, c, taps, act, fc):
    import paper_2110_02781_amd.binding as B
    print(f"average sums {dtype} {h}x{w} batch {batch} {c} channels, {taps} taps, {act}, fc {fc}", flush=True)
    cin = 8
    oact = dict(relu=L.ACT_RELU, relu6=L.ACT_RELU6, none=L.ACT_NONE)[act]
    hact = dict(relu=B.ACT_RELU, relu6=B.ACT_RELU6, none=B.ACT_NONE)[act]
    k, p = (taps, taps // 2) if taps else (1, 0)
    o = [OM.Unit('conv', cin, c, 1, k, 1, 0, p, act=oact), OM.Unit('gap', c, c)]
    hu = [dict(kind=B.UNIT_CONV, cin=cin, cout=c, kh=1, kw=k, stride=1, pad_h=0, pad_w=p, act=hact), dict(kind=B.UNIT_GAP, cin=c, cout=c)]
    if fc:
        o.append(OM.Unit('fc', c, 10))
        hu.append(dict(kind=B.UNIT_FC, cin=c, cout=10))
    pair = Pair(o, hu, (h, w, cin), batch, 0, len(o), dtype, n_slots=2, seed=8, ties="bounded")
    try:
        for slot in range(2):
            y, yo = pair.forward(slot, synth.normal(41, f"x{slot}", (batch, h, w, cin)))
            assert_close(y, yo, TOL[dtype], "y")
        for slot in range(2):
            def back():
                dx, dxo = pair.backward(slot, synth.normal(41, f"dy{slot}", yo.shape))
                assert_close(dx, dxo, TOL[dtype], f"dx {slot}")
            n = launches(back)
            assert n.get("bn_bwd_reduce", 0) == 0 and n.get("bn_bwd_small", 0) == (1 if dtype == "bf16" and h * w * batch > 1536 and h * w * batch <= 2048 else 0), n
            pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
    finally:
        pair.close()
