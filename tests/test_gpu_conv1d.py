"""Convolutions along one axis (implicit GEMMs, csrc/k_conv1d.hip) against the float64 oracle, at the edges of their tiles."""
import pytest

import synth
from harness import Pair, TOL, assert_close
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu


def units(cins, cout, k, act):
    import paper_2110_02781_amd.binding as B
    o, h = [], []
    for a, b in zip(cins, cins[1:] + [cout]):
        o.append(OM.Unit('conv', a, b, 1, k, 1, 0, k // 2, act=act))
        h.append(dict(kind=B.UNIT_CONV, cin=a, cout=b, kh=1, kw=k, stride=1, pad_h=0, pad_w=k // 2, act=act))
    return o, h


# (channels of the chain's inputs, last cout, taps, window, batch).  Up to 2048 rows the 16 x 16 kernels, above them the row
# tiles (128 x 32 or 64 x 64, weight gradient in pieces of 32 x 80): windows shorter than a tile, longer, odd and the shortest;
# channels off 8 and off 4; columns off 16 and 32; a last tile of one row; more row tiles than partials; each tap count.
# A chain of two has the data gradient leave the backward sums of the BatchNorm in front (above 2048 rows).
CASES = [([16], 8, 5, 16, 1), ([3], 24, 3, 17, 7), ([9], 40, 9, 50, 40), ([16], 32, 5, 128, 16), ([64], 64, 5, 131, 15),
         ([16], 32, 5, 683, 3), ([9], 32, 5, 37, 56), ([13], 24, 3, 16, 200), ([64], 40, 9, 97, 27), ([12, 40], 64, 5, 47, 61),
         ([24, 64], 64, 5, 256, 17), ([64, 32], 8, 7, 19, 130), ([8, 16], 16, 3, 200, 400), ([64], 64, 3, 128, 300)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cins,cout,k,w,batch", CASES, ids=[f"{'-'.join(map(str, c[0]))}-{c[1]}_k{c[2]}_w{c[3]}_b{c[4]}" for c in CASES])
def test_conv1d_edges(cins, cout, k, w, batch, dtype):
    print(f"conv1d {cins} -> {cout} taps {k} window {w} batch {batch} {dtype}", flush=True)
    # no activation: nothing but sums, so two bfloat16 layers stay comparable too
    o, h = units(cins, cout, k, L.ACT_NONE if dtype == "bf16" else L.ACT_RELU)
    tol = TOL[dtype]
    pair = Pair(o, h, (1, w, cins[0]), batch, 0, len(o), dtype, seed=5, ties="off" if dtype == "bf16" else "bounded")
    try:
        x = synth.normal(21, "x", (batch, 1, w, cins[0]))
        y, yo = pair.forward(0, x)
        assert_close(y, yo, tol, "y")
        dx, dxo = pair.backward(0, synth.normal(21, "dy", yo.shape))
        assert_close(dx, dxo, tol, "dx")
        pair.compare_unit_vectors("grads", tol, floor=1e-6)
        pair.compare_unit_vectors("bn", tol)
    finally:
        pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_gradient_that_is_not_finite_stays_out_of_channels_that_are_off(dtype):
    """Two convolutions above 2048 rows: the second's data gradient leaves the first's BatchNorm-backward sums.  An infinite output gradient
    makes all of them NaN, but a channel whose ReLU is off everywhere passes none of it: its gradients are exactly zero."""
    import numpy as np
    import torch
    import paper_2110_02781_amd as P
    print(f"channel off, infinite gradient {dtype}", flush=True)
    _, h = units([16, 24], 32, 5, L.ACT_RELU)
    batch, w, off = 20, 128, 7
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    model = P.model_create(h, 1, w, 16, P.F32 if dtype == "f32" else P.BF16)
    stage = P.stage_create(model, 0, 2, batch, 1)
    try:
        vecs = P.models.init_unit_params(h, 3)
        vecs[0][24 * 5 * 16 + 24 + off] = -100.0                    # that channel's BatchNorm shift
        for i, v in enumerate(vecs):
            P.stage_import_weights(stage, i, v)
        x = torch.from_numpy(synth.normal(22, "x", (batch, 1, w, 16)).astype(np.float32)).cuda().to(tdt)
        dy = torch.from_numpy(synth.normal(22, "dy", (batch, 1, w, 32)).astype(np.float32)).cuda().to(tdt)
        dy[3, 0, 40] = float("inf")
        sp = torch.cuda.current_stream().cuda_stream
        P.stage_forward(stage, 0, x, None, sp)
        P.stage_backward(stage, 0, dy, None, sp)
        g = P.stage_export_grads(stage, 0, vecs[0].size)
        gw, gamma, beta = g[:24 * 80].reshape(24, 80), g[24 * 80:24 * 80 + 24], g[24 * 80 + 24:]
        assert np.all(gw[off] == 0) and gamma[off] == 0 and beta[off] == 0, (gamma[off], beta[off])
        assert not np.isfinite(gw[off - 1]).any()
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)
