"""The end of a network (average, fully connected layer) backward in one launch, against the float64 oracle at the edges of its tiles,
and short 1-D convolutions that finish each other's statistics."""
import pytest

import synth
from harness import Pair, TOL, assert_close
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu


def tail(k, classes, conv, gap):
    import paper_2110_02781_amd.binding as B
    o, h = [], []
    if conv:
        o.append(OM.Unit('conv', 8, k, 1, 1, 1, 0, 0, act=L.ACT_RELU6))
        h.append(dict(kind=B.UNIT_CONV, cin=8, cout=k, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=B.ACT_RELU6))
    if gap:
        o.append(OM.Unit('gap', k, k))
        h.append(dict(kind=B.UNIT_GAP, cin=k, cout=k))
    o.append(OM.Unit('fc', k, classes))
    h.append(dict(kind=B.UNIT_FC, cin=k, cout=classes))
    return o, h


# (features, classes, batch, H, W, a convolution in front, an average): classes of one, off 4 and off 16, more than a round of 64 per
# wavefront; batches of one, off 16, more than a round; average as the first unit (its own launch), behind a convolution (part of the
# data gradient), too large for that; features that are still a view (1 x 1 images); layers too large for the one launch
CASES = [(8, 1, 1, 2, 3, True, True), (24, 6, 5, 7, 1, True, True), (64, 17, 16, 4, 4, True, True), (40, 100, 33, 3, 5, True, True),
         (1280, 1000, 130, 1, 2, True, True), (72, 259, 512, 1, 1, True, False), (48, 10, 9, 5, 5, False, True), (56, 12, 20, 31, 32, True, True),
         (128, 7, 70, 11, 13, True, True), (16, 1030, 12, 2, 2, True, True), (32, 9, 600, 1, 1, False, False), (400, 1000, 512, 1, 1, False, False)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,classes,batch,h,w,conv,gap", CASES, ids=[f"{c[0]}x{c[1]}_b{c[2]}_{c[3]}x{c[4]}{'_conv' if c[5] else ''}{'_gap' if c[6] else ''}" for c in CASES])
def test_fully_connected_backward_edges(k, classes, batch, h, w, conv, gap, dtype):
    print(f"tail {k} -> {classes} batch {batch} {h}x{w} conv {conv} gap {gap} {dtype}", flush=True)
    o, hu = tail(k, classes, conv, gap)
    tol = TOL[dtype]
    cin = 8 if conv else k
    pair = Pair(o, hu, (h, w, cin), batch, 0, len(o), dtype, n_slots=2, seed=8, ties="bounded" if conv else "off")
    try:
        for slot in range(2):
            y, yo = pair.forward(slot, synth.normal(41, f"x{slot}", (batch, h, w, cin)))
            assert_close(y, yo, tol, "y")
        for slot in range(2):                             # the second adds to the first's gradients
            dx, dxo = pair.backward(slot, synth.normal(41, f"dy{slot}", yo.shape))
            assert_close(dx, dxo, tol, f"dx {slot}")
            pair.compare_unit_vectors("grads", tol, floor=1e-6)
    finally:
        pair.close()


# the average over a lane's one position, exactly a wavefront's 64, one more, four rounds and one more; behind a convolution (a view, whose
# statistics it finishes where the rows are few) and as a stage's first unit
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("conv", [True, False])
@pytest.mark.parametrize("h,w,batch", [(1, 1, 70), (1, 2, 40), (8, 8, 3), (8, 8, 40), (5, 13, 3), (5, 13, 40), (16, 16, 2), (16, 16, 9), (1, 257, 3), (1, 257, 9)])
def test_average_edges(h, w, batch, conv, dtype):
    print(f"average {h}x{w} batch {batch} conv {conv} {dtype}", flush=True)
    o, hu = tail(24, 10, conv, True)
    cin = 8 if conv else 24
    pair = Pair(o, hu, (h, w, cin), batch, 0, len(o), dtype, seed=8, ties="bounded" if conv else "off")
    try:
        y, yo = pair.forward(0, synth.normal(43, "x", (batch, h, w, cin)))
        assert_close(y, yo, TOL[dtype], "y")
        dx, dxo = pair.backward(0, synth.normal(43, "dy", yo.shape))
        assert_close(dx, dxo, TOL[dtype], "dx")
    finally:
        pair.close()


# fewer than 200 M products: one launch; more: a launch for each gradient, which were faster there (512 x 1792 -> 1000: 129 against 178 us)
@pytest.mark.parametrize("batch,k,classes,one", [(128, 1280, 1000, True), (512, 384, 1000, True), (512, 400, 1000, False), (256, 1280, 1000, False)])
def test_fully_connected_backward_takes_one_launch_where_it_is_faster(batch, k, classes, one):
    import torch
    import paper_2110_02781_amd as P
    print(f"fc route {batch} x {k} -> {classes}", flush=True)
    model = P.model_create(tail(k, classes, False, False)[1], 1, 1, k, P.F32)
    stage = P.stage_create(model, 0, 1, batch, 1)
    try:
        x, dy = torch.zeros(batch, k, device="cuda"), torch.zeros(batch, classes, device="cuda")
        sp = torch.cuda.current_stream().cuda_stream
        P.stage_forward(stage, 0, x, None, sp)
        torch.cuda.synchronize()
        P.ktrace_begin()
        P.stage_backward(stage, 0, dy, torch.empty_like(x), sp)
        torch.cuda.synchronize()
        assert any(r["name"] == "fc_bwd" for r in P.ktrace_end()) == one
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)
