"""Short inverted-residual blocks behind one another: the block output and the project layer's BatchNorm backward are formed by the
pointwise layer that reads them (csrc/k_gemm.hip), against the float64 oracle and against stages of one block each, which have
launches of their own for both."""
import numpy as np
import pytest

import synth
from harness import Pair, TOL, assert_close, launches
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (channels of the blocks, last one stride 2; cout of the pointwise convolution behind them, h, w, batch, copies in the batch, blocks whose
# output / whose project BatchNorm backward the next layer forms).  Rows off 16, the most (2048), one more; 64 channels in fp32
# and 96 in bfloat16 are the widest; 64 KB of partials and more; fewer than 16 channels; so few rows that both gradients of a layer are one launch
CASES = [("f32", [64, 64, 24], 40, 8, 8, 8, 1, 3, 3), ("f32", [32, 32, 32], 48, 8, 16, 16, 8, 3, 3), ("f32", [32, 64, 72], 40, 13, 53, 2, 1, 2, 2),
         ("f32", [8, 16, 8], 24, 13, 40, 3, 1, 3, 1), ("f32", [64, 64, 64], 24, 23, 89, 1, 1, 3, 3), ("f32", [64, 64, 16], 24, 2, 683, 3, 1, 1, 1),
         ("f32", [24, 32, 64], 24, 5, 11, 1, 1, 3, 0),
         ("bf16", [96, 96, 64], 40, 9, 15, 8, 1, 3, 3), ("bf16", [32, 96, 104], 24, 7, 9, 24, 1, 1, 1), ("bf16", [16, 32, 64], 24, 16, 16, 8, 1, 3, 3)]


def units(chans, cout):
    import paper_2110_02781_amd.binding as B
    o, h = [], []
    c = chans[0]
    for i, n in enumerate(chans):
        s = 2 if i + 1 == len(chans) else 1
        o.append(OM.Unit('invres', c, n, stride=s, expand=6))
        h.append(dict(kind=B.UNIT_INVRES, cin=c, cout=n, stride=s, expand=6))
        c = n
    o.append(OM.Unit('conv', c, cout, act=L.ACT_RELU6))
    h.append(dict(kind=B.UNIT_CONV, cin=c, cout=cout, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=B.ACT_RELU6))
    return o, h


def run(h, shape, batch, dtype, cuts, x, dy):
    """One forward and backward of stages [cuts[i], cuts[i + 1]): (y, dx, gradients, running statistics), launches by family."""
    import torch
    import paper_2110_02781_amd as P
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    model = P.model_create(h, shape[0], shape[1], shape[2], P.F32 if dtype == "f32" else P.BF16)
    vecs = P.models.init_unit_params(h, 31)
    stages = [(a, b, P.stage_create(model, a, b, batch, 1)) for a, b in zip(cuts, cuts[1:])]
    shapes = [(batch,) + P.model_unit_in_shape(model, u) for u in range(len(h) + 1)]
    sp = torch.cuda.current_stream().cuda_stream
    try:
        for a, b, s in stages:
            for u in range(a, b):
                P.stage_import_weights(s, u, vecs[u])
        t = torch.from_numpy(x.astype(np.float32)).cuda().to(tdt)
        d = torch.from_numpy(dy.astype(np.float32)).cuda().to(tdt)

        def both():
            nonlocal t, d
            for a, b, s in stages:
                y = torch.empty(shapes[b], dtype=tdt, device="cuda")
                P.stage_forward(s, 0, t, y, sp)
                t = y
            for a, b, s in stages[::-1]:
                dx = torch.empty(shapes[a], dtype=tdt, device="cuda")
                P.stage_backward(s, 0, d, dx, sp)
                d = dx
        n = launches(both)
        g = [P.stage_export_grads(s, u, vecs[u].size) for a, b, s in stages for u in range(a, b)]
        r = [P.stage_export_bn_stats(s, u, 2 * P.model_unit_bn_channels(model, u)) for a, b, s in stages for u in range(a, b)]
        return (t.float().cpu().numpy(), d.float().cpu().numpy(), g, r), n
    finally:
        for _, _, s in stages:
            P.stage_destroy(s)
        P.model_destroy(model)


@pytest.mark.parametrize("dtype,chans,cout,h,w,batch,tile,n_out,n_bn", CASES, ids=["-".join(map(str, c)).replace(" ", "") for c in CASES])
def test_blocks_that_the_next_layer_forms(dtype, chans, cout, h, w, batch, tile, n_out, n_bn):
    print(f"block chain {dtype} {chans} -> {cout}, {h}x{w} batch {batch}", flush=True)
    o, hu = units(chans, cout)
    shape = (h, w, chans[0])
    xs = synth.normal(41, "x", (batch // tile,) + shape)
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    dys = synth.normal(41, "dy", (batch // tile, ho, wo, cout)) / batch
    x, dy = np.concatenate([xs] * tile), np.concatenate([dys] * tile)
    one, n1 = run(hu, shape, batch, dtype, [0, len(hu)], x, dy)
    each, n2 = run(hu, shape, batch, dtype, list(range(len(hu) + 1)), x, dy)
    small = ("bn_fin_apply_small", "bn_bwd_small")
    assert [n2.get(k, 0) - n1.get(k, 0) for k in small] == [n_out, n_bn], (n1, n2)
    # the same sums in another order: float64 sums of fp32 partials over 16 rows against one or two rows a thread; an element of bfloat16
    # falls to the other side of a rounding now and then, one activation in all switches at most
    tol = 2e-5 if dtype == "f32" else 4e-3
    for a, b, name in zip(one[:2], each[:2], ("y", "dx")):
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b), name
    for name, i in (("gradients", 2), ("running statistics", 3)):
        for u, (a, b) in enumerate(zip(one[i], each[i])):
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b), f"{name} of unit {u}: {np.linalg.norm(a - b) / np.linalg.norm(b):.2e}"
    if dtype != "f32":
        return
    pair = Pair(o, hu, shape, batch, 0, len(o), dtype, seed=31, ties="bounded", tile=tile)
    try:
        y, yo = pair.forward(0, xs)
        assert_close(y, yo, TOL[dtype], "y")
        dx, dxo = pair.backward(0, dys)
        assert_close(dx, dxo, TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()
