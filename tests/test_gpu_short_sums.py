"""How far the fp32 matrix products of convolutions are from 64 bits: the length of their chains of additions decides it."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def errors(unit, h, w, batch):
    """Relative 2-norms of the errors of a stage of one fp32 convolution without activation: (convolution output, input gradient)."""
    import torch
    import paper_2110_02781_amd as P
    units = [unit]
    model = P.model_create(units, h, w, unit["cin"], P.F32)
    stage = P.stage_create(model, 0, 1, batch, 1)
    try:
        kh, kw, co, ci = unit["kh"], unit["kw"], unit["cout"], unit["cin"]
        vec = P.models.init_unit_params(units, 73)[0]
        P.stage_import_weights(stage, 0, vec)
        x = synth.normal(73, "x", (batch, h, w, ci)).astype(np.float32)
        dy = synth.normal(73, "dy", (batch, h, w, co)).astype(np.float32)
        xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
        dxd = torch.empty_like(xd)
        sp = torch.cuda.current_stream().cuda_stream
        P.stage_forward(stage, 0, xd, None, sp)
        z = P.stage_export_conv_output(stage, 0, 0, 0, dy.size).reshape(-1, co)
        P.stage_backward(stage, 0, dyd, dxd, sp)
        torch.cuda.synchronize()
        wt = torch.from_numpy(vec[:co * kh * kw * ci].astype(np.float64)).reshape(co, kh * kw * ci)
        xt = torch.from_numpy(x.astype(np.float64)).requires_grad_()
        padded = torch.nn.functional.pad(xt, (0, 0, kw // 2, kw // 2, kh // 2, kh // 2))
        patches = torch.cat([padded[:, i:i + h, j:j + w] for i in range(kh) for j in range(kw)], dim=3)
        zt = patches.reshape(-1, kh * kw * ci) @ wt.t()
        var, mean = torch.var_mean(zt, 0, correction=0)
        gx, = torch.autograd.grad((zt - mean) * torch.rsqrt(var + 1e-5), xt, torch.from_numpy(dy.astype(np.float64)).reshape(-1, co))
        rel = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))
        return rel(z, zt.detach().numpy()), rel(dxd.cpu().numpy(), gx.numpy())
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)


def unit(ci, co, kw=1):
    import paper_2110_02781_amd.binding as B
    return dict(kind=B.UNIT_CONV, cin=ci, cout=co, kh=1, kw=kw, stride=1, pad_h=0, pad_w=kw // 2, act=B.ACT_NONE)


def bar(chain, chains):
    """A fp32 addition rounds by 0.4 * 2^-24 of the sum (r.m.s.): chains of `chain` random terms, `chains` of them added one behind the
    other, and a fifth more for what a sample of this size scatters."""
    return 1.2 * 0.4 * 2.0 ** -24 * np.sqrt((chain + 1) / 2 + (chains + 1) / 2)


# up to 64 terms: four chains of 16 (one of 64: 1.4e-7); the input gradient carries the rounding of dz besides
@pytest.mark.parametrize("ci,co,hw,batch", [(64, 384, 4, 64), (48, 64, 8, 8), (64, 64, 5, 9), (40, 64, 3, 1)])
def test_short_pointwise_products_add_in_short_chains(ci, co, hw, batch):
    print(f"short product {ci}->{co} {hw}x{hw} batch {batch}", flush=True)
    z, dx = errors(unit(ci, co), hw, hw, batch)
    print(f"  output {z:.3e}, input gradient {dx:.3e}, bar {bar(16, 4):.3e}", flush=True)
    assert z <= bar(16, 4)
    # with few rows dz itself is far off: dy - mean(dy) - xhat mean(dy xhat) cancels, by about 1 / rows of its square
    if co <= 64 and batch * hw * hw >= 200:
        assert dx <= bar(16, 4) + 0.4 * 2.0 ** -24


# convolutions along one axis above 2048 rows: chains of 64 terms, up to nine of them (64 -> 64 channels, 9 taps); two halves of the
# reduction for 32 columns and fewer; channels off 8
@pytest.mark.parametrize("ci,co,taps,w,batch", [(64, 64, 9, 256, 64), (64, 64, 5, 128, 17), (64, 32, 9, 100, 30), (24, 64, 9, 97, 40), (13, 40, 9, 64, 50)])
def test_products_along_one_axis_add_in_short_chains(ci, co, taps, w, batch):
    print(f"1-D products {ci}->{co} taps {taps} window {w} batch {batch}", flush=True)
    z, dx = errors(unit(ci, co, taps), 1, w, batch)
    chains = [(taps * ((c + 7) // 8 * 8) + 63) // 64 for c in (ci, co)]
    print(f"  output {z:.3e} (bar {bar(64, chains[0]):.3e}), input gradient {dx:.3e} (bar {bar(64, chains[1]) + 0.4 * 2.0 ** -24:.3e})", flush=True)
    assert z <= bar(64, chains[0]) and dx <= bar(64, chains[1]) + 0.4 * 2.0 ** -24
