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


def lost_in_the_longest_chain(unit, h, w, batch):
    """How many terms of a product vanish next to a large one: all inputs are 1, the first weight of every channel is 2^24 and the others
    are 1/4, so what is added to the large term one by one rounds away, and what is added up elsewhere first does not (chains of a multiple
    of 8 terms: their sums are even).  The largest number over all rows that see every tap."""
    import torch
    import paper_2110_02781_amd as P
    model = P.model_create([unit], h, w, unit["cin"], P.F32)
    stage = P.stage_create(model, 0, 1, batch, 1)
    try:
        kw, co, ci = unit["kw"], unit["cout"], unit["cin"]
        wt = np.full((co, kw * ci), 0.25, np.float32)
        wt[:, 0] = 2.0 ** 24
        P.stage_import_weights(stage, 0, np.concatenate([wt.ravel(), np.ones(co), np.zeros(co)]).astype(np.float32))
        x = torch.ones(batch, h, w, ci, device="cuda")
        P.stage_forward(stage, 0, x, None, torch.cuda.current_stream().cuda_stream)
        z = P.stage_export_conv_output(stage, 0, 0, 0, batch * h * w * co).reshape(batch * h, w, co).astype(np.float64)
        z = z[:, kw // 2:w - kw // 2]
        return float(((kw * ci - 1) * 0.25 - (z - 2.0 ** 24)).max() * 4)
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)


# 64 columns: chains of 64 terms; 32 columns and fewer, where wavefronts share a tile's reduction: of 32.  Tiles of 32, 64 and 128 rows
@pytest.mark.parametrize("ci,co,taps,w,batch,chain", [(64, 64, 5, 128, 17, 64), (64, 64, 5, 128, 80, 64), (64, 64, 5, 128, 256, 64), (64, 64, 9, 128, 256, 64),
                                                      (32, 32, 5, 128, 256, 32), (64, 32, 9, 128, 256, 32), (64, 32, 9, 128, 80, 32), (32, 24, 9, 128, 600, 32)])
def test_no_longer_chains_along_one_axis(ci, co, taps, w, batch, chain):
    print(f"1-D chain {ci}->{co} taps {taps} window {w} batch {batch}", flush=True)
    lost = lost_in_the_longest_chain(unit(ci, co, taps), 1, w, batch)
    print(f"  {lost:.0f} terms lost", flush=True)
    assert 0 <= lost < chain


@pytest.mark.parametrize("w,batch", [(128, 8), (128, 16), (100, 20)])
def test_short_layers_along_one_axis_that_take_sums_lose_nothing_in_their_weight_gradients(w, batch):
    """Layers of one stage do their BatchNorm backward on the way into both gradients, layers of a stage each have a launch for it and more
    wavefronts to the weight gradient's rows: the first may be no further from 64 bits than the second, but for what a sample of
    this size scatters (5 %; a chain of twice the length: 8 - 20 %)."""
    import torch
    import paper_2110_02781_amd as P
    print(f"short 1-D weight gradients window {w} batch {batch}", flush=True)
    units = [unit(16, 32, 5), unit(32, 64, 5), unit(64, 64, 5)]
    vecs = P.models.init_unit_params(units, 74)
    x = torch.from_numpy(synth.normal(74, "x", (batch, 1, w, 16)).astype(np.float32)).cuda()
    dy = torch.from_numpy(synth.normal(74, "dy", (batch, 1, w, 64)).astype(np.float32)).cuda()

    def gradients(cuts):
        model = P.model_create(units, 1, w, 16, P.F32)
        stages = [(a, b, P.stage_create(model, a, b, batch, 1)) for a, b in zip(cuts, cuts[1:])]
        sp = torch.cuda.current_stream().cuda_stream
        try:
            t, d = x, dy
            for a, b, s in stages:
                for u in range(a, b):
                    P.stage_import_weights(s, u, vecs[u])
                y = torch.empty((batch,) + P.model_unit_in_shape(model, b), device="cuda")
                P.stage_forward(s, 0, t, y, sp)
                t = y
            for a, b, s in stages[::-1]:
                dx = torch.empty((batch,) + P.model_unit_in_shape(model, a), device="cuda")
                P.stage_backward(s, 0, d, dx, sp)
                d = dx
            return [P.stage_export_grads(s, u, vecs[u].size)[:-2 * units[u]["cout"]].astype(np.float64) for a, b, s in stages for u in range(a, b)]
        finally:
            for _, _, s in stages:
                P.stage_destroy(s)
            P.model_destroy(model)

    wt = [torch.from_numpy(v[:-2 * u["cout"]].astype(np.float64)).cuda().requires_grad_() for v, u in zip(vecs, units)]
    h = x.double()
    for u, p in zip(units, wt):
        padded = torch.nn.functional.pad(h, (0, 0, 2, 2))
        z = torch.cat([padded[:, :, i:i + w] for i in range(5)], dim=3) @ p.reshape(u["cout"], -1).t()
        var, mean = torch.var_mean(z, (0, 1, 2), correction=0)
        h = (z - mean) * torch.rsqrt(var + 1e-5)
    want = [g.cpu().numpy() for g in torch.autograd.grad(h, wt, dy.double())]
    one, each = gradients([0, 3]), gradients([0, 1, 2, 3])
    for u, (a, b, g) in enumerate(zip(one, each, want)):
        ea, eb = (np.linalg.norm(t - g) / np.linalg.norm(g) for t in (a, b))
        print(f"  layer {u}: {ea:.3e} in one stage, {eb:.3e} alone", flush=True)
        assert ea <= 1.05 * eb


# fp32 pointwise layers above 512 rows on the long-reduction kernel: chains of 32 terms in short and long reductions, as short as where four
# wavefronts share a reduction of 128 (192 -> 32, 8192 rows: 1.38e-7 off in that way, 1.48e-7 in chains of 64)
@pytest.mark.parametrize("ci,co,hw,batch", [(192, 32, 64, 2), (128, 64, 32, 3), (960, 160, 14, 16), (64, 64, 64, 4), (136, 88, 33, 5)])
def test_long_pointwise_products_add_in_short_chains(ci, co, hw, batch):
    print(f"long product {ci}->{co} {hw}x{hw} batch {batch}", flush=True)
    lost = lost_in_the_longest_chain(unit(ci, co), hw, hw, batch)
    print(f"  {lost:.0f} terms lost", flush=True)
    assert 0 <= lost < 32


# 1-D weight gradients above 2048 rows: a wavefront adds its share of a block's rows (half of them, a quarter or an eighth) in two chains, what meets
# behind them is four more roundings at most, and dz carries its own three
@pytest.mark.parametrize("ci,co,taps,w,batch,chain", [(16, 16, 3, 128, 256, 16), (12, 32, 5, 128, 256, 16), (32, 32, 5, 128, 256, 16), (64, 64, 9, 128, 40, 32),
                                                      (64, 64, 5, 128, 256, 64), (64, 64, 5, 256, 512, 256)])
def test_weight_gradients_along_one_axis_add_in_short_chains(ci, co, taps, w, batch, chain):
    import torch
    import paper_2110_02781_amd as P
    print(f"1-D weight gradient {ci}->{co} taps {taps} window {w} batch {batch}", flush=True)
    u = unit(ci, co, taps)
    model = P.model_create([u], 1, w, ci, P.F32)
    stage = P.stage_create(model, 0, 1, batch, 1)
    try:
        vec = P.models.init_unit_params([u], 75)[0]
        P.stage_import_weights(stage, 0, vec)
        x = torch.from_numpy(synth.normal(75, "x", (batch, 1, w, ci)).astype(np.float32)).cuda()
        dy = torch.from_numpy(synth.normal(75, "dy", (batch, 1, w, co)).astype(np.float32)).cuda()
        sp = torch.cuda.current_stream().cuda_stream
        P.stage_forward(stage, 0, x, None, sp)
        P.stage_backward(stage, 0, dy, torch.empty_like(x), sp)
        n = co * taps * ci
        g = P.stage_export_grads(stage, 0, vec.size)[:n].astype(np.float64)
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)
    wt = torch.from_numpy(vec[:n].astype(np.float64)).cuda().requires_grad_()
    padded = torch.nn.functional.pad(x.double(), (0, 0, taps // 2, taps // 2))
    z = torch.cat([padded[:, :, i:i + w] for i in range(taps)], dim=3).reshape(-1, taps * ci) @ wt.reshape(co, -1).t()
    var, mean = torch.var_mean(z, 0, correction=0)
    want, = torch.autograd.grad((z - mean) * torch.rsqrt(var + 1e-5), wt, dy.double().reshape(-1, co))
    want = want.cpu().numpy()
    err = np.linalg.norm(g - want) / np.linalg.norm(want)
    limit = 1.1 * 0.4 * 2.0 ** -24 * np.sqrt((chain + 1) / 2 + 6)
    print(f"  error {err:.3e} (bar {limit:.3e})", flush=True)
    assert err <= limit
