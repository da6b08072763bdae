"""BatchNorm finished by the kernel that applies it (csrc/k_elem.hip: bn_finish_apply_k, bn_bwd_finish_apply_k) against the float64 oracle."""
import numpy as np
import pytest

import synth
from harness import Pair, TOL, assert_close, routes
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (cin, cout, expand, stride, h, w, batch): the fewest rows; slabs of 5, 6 and 7 column groups, a last slab of fewer (72, 88, 104 channels); 8 channels;
# a residual; more partials than one round of a thread's requests; the most values, and beyond them
CASES = [(24, 24, 3, 1, 3, 683, 1), (16, 104, 4, 1, 41, 50, 1), (8, 8, 11, 1, 45, 46, 1), (32, 88, 6, 2, 93, 95, 1), (16, 16, 6, 1, 50, 61, 2),
         (8, 24, 6, 1, 80, 100, 3), (24, 32, 6, 2, 112, 112, 8)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout,expand,stride,h,w,batch", CASES)
def test_finish_and_apply(dtype, cin, cout, expand, stride, h, w, batch):
    import paper_2110_02781_amd.binding as B
    print(f"finish {dtype} {cin}->{cout} x{expand} stride {stride} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=stride, expand=expand)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=expand)]
    pair = Pair(o, hu, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="bounded")
    try:
        x = synth.normal(51, "x", (batch, h, w, cin))

        def both():
            y, yo = pair.forward(0, x)
            assert_close(y, yo, TOL[dtype], "y")
            dx, dxo = pair.backward(0, synth.normal(51, "dy", yo.shape))
            assert_close(dx, dxo, TOL[dtype], "dx")
        took = routes(both)
        assert any("finish" in r for r in took), took
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,w,batch", [(7, 9, 4), (30, 41, 3), (129, 130, 2)])
def test_block_output_goes_where_the_caller_wants_it(dtype, h, w, batch):
    """A block at a stage's end writes the caller's tensor itself: aligned or not (then it is copied), and over the stage's own input.  Short, finished on
    the way and finished before."""
    import torch
    import paper_2110_02781_amd as P
    B = P.binding
    print(f"block output {dtype} {h}x{w} batch {batch}", flush=True)
    units = [dict(kind=B.UNIT_INVRES, cin=16, cout=16, stride=1, expand=6)] * 2
    model = P.model_create(units, h, w, 16, P.F32 if dtype == "f32" else P.BF16)
    stage = P.stage_create(model, 0, 2, batch, 3)
    try:
        for l, wts in enumerate(P.models.init_unit_params(units, 74)):
            P.stage_import_weights(stage, l, wts)
        tt = torch.float32 if dtype == "f32" else torch.bfloat16
        x = torch.from_numpy(synth.normal(74, "x", (batch, h, w, 16)).astype(np.float32)).cuda().to(tt)
        y = torch.zeros_like(x)
        odd = torch.zeros(x.numel() + 1, dtype=tt, device="cuda")[1:].view(x.shape)
        over = x.clone()
        sp = torch.cuda.current_stream().cuda_stream
        for slot, (a, b) in enumerate([(x, y), (x, odd), (over, over)]):
            P.stage_forward(stage, slot, a, b, sp)
        torch.cuda.synchronize()
        assert torch.isfinite(y.float()).all() and y.float().abs().max() > 0
        assert torch.equal(y, odd) and torch.equal(y, over)
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)
