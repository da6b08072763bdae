"""How far the weight gradients that a stage runs together at the end of its backward call are from the exact product of what their
kernels were given: the length of their fp32 chains of additions is what decides it.

A convolution's dz is not visible from outside, so it is made known: no activation, the convolution sees eight of its input channels
only (the other weights are zero), and rows come in pairs with equal values in those eight and opposite output gradients.  Then both
BatchNorm-backward sums vanish, and with gamma = 1 / invstd dz is the output gradient times a constant per channel (one to a rounding).
The gradients with respect to the other weights are ordinary sums, dy^T a, and are compared with those in float64."""
import numpy as np
import pytest

import synth
from harness import from_bf16_bits, to_bf16_bits

pytestmark = pytest.mark.gpu

# One fp32 addition rounds by 0.4 * 2^-24 of the sum (r.m.s.), so a chain of s random terms by 0.4 * 2^-24 * sqrt((s + 1) / 2) of
# its result, and each further rounding of the result (dz, partial, gradient) counts like two more terms.  float: s = 64 rows, what the
# kernel of a single layer takes: 1.42e-7 (a chain of 256 rows: 2.7e-7).  bfloat16 products have 16 bits, so the first additions of a
# chain round nothing: measured 6.3e-8 with the 128 rows of a single layer's kernel, 1.1e-7 with 256 (narrow layers) and 640 rows.
BAR = {"f32": 0.4 * 2.0 ** -24 * np.sqrt((64 + 1) / 2 + 3), "bf16": 6.5e-8}


def stored(a, dtype):
    return np.asarray(a, np.float32) if dtype == "f32" else from_bf16_bits(to_bf16_bits(a))


def last_layers_gradient_error(h, w, batch, K, N, layers, dtype):
    """(relative 2-norm of the error of the last weight gradient of a chain of pointwise layers, largest deviation of its scale from 1)"""
    import torch
    import paper_2110_02781_amd as P
    B = P.binding
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    M = batch * h * w
    half = M // 2
    x = synth.normal(71, "x", (M, K))
    x[half:2 * half, :8] = x[:half, :8]
    x = stored(x, dtype)
    dy = synth.normal(71, "dy", (M, N))
    dy[half:2 * half] = -dy[:half]
    dy[2 * half:] = 0.0
    dy = stored(dy, dtype)
    units = [dict(kind=B.UNIT_CONV, cin=K, cout=c, kh=1, kw=1, stride=1, act=B.ACT_NONE) for c in [K] * (layers - 1) + [N]]
    vecs = []
    for l, u in enumerate(units):
        n = u["cout"]
        wm = synth.normal(71, f"w{l}", (n, K), std=8 ** -0.5)
        if l + 1 < layers:              # the eight channels stay among themselves, and so does what repeats over the pairs
            wm[:8, 8:] = 0.0
            wm[8:, :8] = 0.0
        else:
            wm[:, 8:] = 0.0
        vecs.append(np.concatenate([wm.ravel(), np.ones(n), np.zeros(n)]).astype(np.float32))
    model = P.model_create(units, h, w, K, P.F32 if dtype == "f32" else P.BF16)
    stage = P.stage_create(model, 0, layers, batch, 1)
    try:
        sp = torch.cuda.current_stream().cuda_stream
        xd = torch.from_numpy(x).cuda().to(tdt)
        dyd = torch.from_numpy(dy).cuda().to(tdt)
        for l in range(layers):
            P.stage_import_weights(stage, l, vecs[l])
        P.stage_forward(stage, 0, xd, None, sp)
        inv = P.stage_export_bn_batch_stats(stage, 0, layers - 1, 0, 4 * N)[N:2 * N].astype(np.float64)
        P.stage_backward(stage, 0, dyd, None, sp)
        vecs[-1][N * K:N * K + N] = 1.0 / inv
        P.stage_import_weights(stage, layers - 1, vecs[-1])
        P.stage_update(stage, 0.0, 0.0, 0.0, sp)              # gradients back to zero
        P.stage_forward(stage, 0, xd, None, sp)
        a = x.astype(np.float64)
        if layers > 1:
            z = P.stage_export_conv_output(stage, 0, layers - 2, 0, M * K).reshape(M, K).astype(np.float64)
            st = P.stage_export_bn_batch_stats(stage, 0, layers - 2, 0, 4 * K).reshape(4, K).astype(np.float64)
            a = stored(z * st[2] + st[3], dtype).astype(np.float64)
        P.stage_backward(stage, 0, dyd, None, sp)
        g = P.stage_export_grads(stage, layers - 1, N * K + 2 * N)[:N * K].reshape(N, K)[:, 8:].astype(np.float64)
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)
    want = (dy.astype(np.float64).T @ a)[:, 8:]
    scale = (g * want).sum(1, keepdims=True) / (want * want).sum(1, keepdims=True)
    return np.linalg.norm(g - scale * want) / np.linalg.norm(want), np.abs(scale - 1).max()


# h, w, batch, K, N, layers, type: rows below and above 2048 (one or several partials), odd rows, narrow before wide and after it,
# several layers together, narrow bfloat16 layers (48 columns and more go through another kernel)
GROUPED = [(16, 16, 1, 40, 64, 1, "f32"), (14, 14, 8, 64, 384, 1, "f32"), (14, 14, 32, 64, 384, 1, "f32"), (28, 28, 16, 48, 48, 30, "f32"),
           (14, 14, 64, 96, 96, 12, "f32"), (28, 28, 64, 192, 32, 1, "f32"), (13, 11, 37, 72, 136, 2, "f32"), (56, 56, 32, 24, 24, 3, "f32"),
           (28, 28, 64, 192, 32, 1, "bf16"), (32, 32, 16, 96, 24, 1, "bf16"), (64, 64, 32, 32, 16, 1, "bf16"), (56, 56, 32, 24, 24, 3, "bf16"), (14, 14, 8, 64, 384, 1, "bf16")]


@pytest.mark.parametrize("h,w,batch,K,N,layers,dtype", GROUPED, ids=["-".join(map(str, c)) for c in GROUPED])
def test_grouped_weight_gradients_add_in_short_chains(h, w, batch, K, N, layers, dtype):
    print(f"weight gradient sums {h}x{w} batch {batch} {K}->{N} x{layers} {dtype}", flush=True)
    err, off = last_layers_gradient_error(h, w, batch, K, N, layers, dtype)
    print(f"  error {err:.3e} (bar {BAR[dtype]:.3e}), scale within {off:.1e}", flush=True)
    assert off <= 4e-7 and err <= BAR[dtype]


# bfloat16 layers of 48 columns and more above 2048 rows: alone, two and seven in a launch, twelve, and thirty (two launches); one
# column tile and several; with so many tiles that every block takes all rows; odd rows
TRANSPOSED = [(14, 14, 32, 64, 384, 1), (14, 14, 32, 96, 576, 7), (14, 14, 32, 96, 96, 12), (14, 14, 128, 96, 96, 12), (7, 7, 128, 320, 1280, 12),
              (28, 28, 16, 48, 48, 30), (13, 11, 37, 72, 136, 2), (47, 3, 15, 1280, 1536, 1)]


@pytest.mark.parametrize("h,w,batch,K,N,layers", TRANSPOSED, ids=["-".join(map(str, c)) for c in TRANSPOSED])
def test_transposing_weight_gradients_add_in_short_chains(h, w, batch, K, N, layers):
    print(f"transposing weight gradient sums {h}x{w} batch {batch} {K}->{N} x{layers}", flush=True)
    err, off = last_layers_gradient_error(h, w, batch, K, N, layers, "bf16")
    print(f"  error {err:.3e} (bar {BAR['bf16']:.3e}), scale within {off:.1e}", flush=True)
    assert off <= 4e-7 and err <= BAR["bf16"]


@pytest.mark.parametrize("channels,h,w,batch", [([96] * 13, 14, 14, 16), ([56, 48] * 15 + [56], 13, 17, 11), ([24, 64] * 6 + [24], 15, 15, 12)],
                         ids=["twelve", "thirty", "both_kernels"])
def test_many_layers_together_give_the_gradients_of_each_alone(channels, h, w, batch):
    """Every layer of a bfloat16 chain in one stage (weight gradients together at the end of the call) against a stage of its own on
    the same tensors: the same products, so the gradients differ by the order of additions only.  Both are within the bar above
    of the exact product, two independent errors of it apart at most."""
    import torch
    import paper_2110_02781_amd as P
    B = P.binding
    print(f"chain of {len(channels) - 1} layers {channels[:3]} {h}x{w} batch {batch}", flush=True)
    units = [dict(kind=B.UNIT_CONV, cin=a, cout=b, kh=1, kw=1, stride=1, act=B.ACT_RELU6) for a, b in zip(channels, channels[1:])]
    L = len(units)
    model = P.model_create(units, h, w, channels[0], P.BF16)
    params = P.models.init_unit_params(units, 72)
    stages = [P.stage_create(model, 0, L, batch, 1)] + [P.stage_create(model, l, l + 1, batch, 1) for l in range(L)]
    try:
        for l in range(L):
            P.stage_import_weights(stages[0], l, params[l])
            P.stage_import_weights(stages[1 + l], l, params[l])
        sp = torch.cuda.current_stream().cuda_stream
        t = [torch.from_numpy(synth.normal(72, "x", (batch, h, w, channels[0])).astype(np.float32)).cuda().to(torch.bfloat16)]
        for c in channels[1:]:
            t.append(torch.empty(batch, h, w, c, dtype=torch.bfloat16, device="cuda"))
        dy = torch.from_numpy(synth.normal(72, "dy", tuple(t[-1].shape)).astype(np.float32)).cuda().to(torch.bfloat16)
        y, dx = torch.empty_like(t[-1]), torch.empty_like(t[0])
        P.stage_forward(stages[0], 0, t[0], y, sp)
        P.stage_backward(stages[0], 0, dy, dx, sp)
        for l in range(L):
            P.stage_forward(stages[1 + l], 0, t[l], t[l + 1], sp)
        assert torch.equal(y, t[-1])
        d = dy
        for l in reversed(range(L)):
            dl = torch.empty_like(t[l])
            P.stage_backward(stages[1 + l], 0, d, dl, sp)
            d = dl
        assert torch.equal(dx, d)
        for l in range(L):
            n = P.model_unit_param_count(model, l)
            a, b = (P.stage_export_grads(s, l, n).astype(np.float64) for s in (stages[0], stages[1 + l]))
            err = np.linalg.norm(a - b) / np.linalg.norm(b)
            assert err <= 2 ** 0.5 * BAR["bf16"], f"layer {l}: {err:.3e}"
    finally:
        for s in stages:
            P.stage_destroy(s)
        P.model_destroy(model)
