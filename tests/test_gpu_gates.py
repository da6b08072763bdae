"""Channels that an activation has switched off: whatever gradient reaches them, infinite too, is chosen away where BatchNorm backward sums are left on the way and where dz is formed,
not multiplied by zero.  A stage with such a channel's outgoing weight (or the gradient behind it) at the top of the type's range has the gradients, bit for bit, of one where it is zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
OFF, BIG = 5, 3e38


def gradients(units, in_shape, batch, dtype, vectors, scale=None):
    """Every unit's gradients and the input's.  scale: what the output's gradient in channel OFF is multiplied by."""
    import torch
    import paper_2110_02781_amd as P
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    m = P.model_create(units, *in_shape, P.F32 if dtype == "f32" else P.BF16)
    s = P.stage_create(m, 0, len(units), batch, 1, 0)
    try:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(11)
        for u, v in enumerate(vectors):
            if v.size:
                P.stage_import_weights(s, u, v)
        x = torch.randn((batch,) + tuple(in_shape), generator=gen, device="cuda").to(tdt)
        y, dx = torch.empty((batch,) + tuple(P.model_unit_in_shape(m, len(units))), dtype=tdt, device="cuda"), torch.empty_like(x)
        dy = torch.randn(y.shape, generator=gen, device="cuda").to(tdt)
        if scale is not None:
            dy[..., OFF] = dy[..., OFF].abs().clamp_(0.1) * scale
        P.stage_forward(s, 0, x, y, 0)
        P.stage_backward(s, 0, dy, dx, 0)
        torch.cuda.synchronize()
        return [P.stage_export_grads(s, u, v.size) for u, v in enumerate(vectors) if v.size] + [dx.float().cpu().numpy()]
    finally:
        P.stage_destroy(s)
        P.model_destroy(m)


def with_part(unit, vector, name, change):
    import paper_2110_02781_amd as P
    out, o = vector.copy(), 0
    for part, n, _ in P.models.unit_param_layout(unit):
        if part == name:
            change(out[o:o + n])
        o += n
    return out


# rows of the streaming kernels, of the long-reduction ones, of the short ones
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layer", ["expand", "depthwise"])
@pytest.mark.parametrize("stride,cin,cout,expand,h,w,batch", [(1, 24, 16, 6, 33, 35, 60), (2, 24, 16, 6, 33, 35, 60), (1, 16, 24, 6, 14, 14, 32), (1, 16, 16, 6, 12, 12, 8)])
def test_switched_off_channel_of_a_block(dtype, layer, stride, cin, cout, expand, h, w, batch):
    import paper_2110_02781_amd as P
    import paper_2110_02781_amd.binding as B
    print(f"switched off {layer} channel {dtype} stride {stride} {cin}->{cout} x{expand} {h}x{w} batch {batch}", flush=True)
    units = [dict(kind=B.UNIT_INVRES, cin=8, cout=cin, stride=1, expand=1), dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=expand)]
    v = P.models.init_unit_params(units, 3)
    c = cin * expand

    def off(p):
        p[OFF] = -100.0

    def outgoing(value):
        def change(p):
            if layer == "depthwise":
                p.reshape(cout, c)[:, OFF] = [value] + [0.0] * (cout - 1)
            else:
                p.reshape(c, 9)[OFF] = [0.0] * 4 + [value] + [0.0] * 4
        return change
    v[1] = with_part(units[1], v[1], "beta2" if layer == "depthwise" else "beta1", off)
    big, zero = (gradients(units, (h, w, 8), batch, dtype, [v[0], with_part(units[1], v[1], "w3" if layer == "depthwise" else "wd", outgoing(value))]) for value in (BIG, 0.0))
    for a, b in zip(big, zero):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,w,batch,taps", [(7, 7, 50, 0), (14, 14, 20, 0), (1, 128, 8, 5), (1, 130, 70, 5)])
def test_switched_off_channel_in_front_of_an_average(dtype, h, w, batch, taps):
    import paper_2110_02781_amd as P
    import paper_2110_02781_amd.binding as B
    print(f"switched off channel in front of an average {dtype} {h}x{w} batch {batch}", flush=True)
    k, pad = (taps, taps // 2) if taps else (1, 0)
    units = [dict(kind=B.UNIT_CONV, cin=8, cout=64, kh=1, kw=k, stride=1, pad_h=0, pad_w=pad, act=B.ACT_RELU6), dict(kind=B.UNIT_GAP, cin=64, cout=64)]
    v = P.models.init_unit_params(units, 3)
    v[0] = with_part(units[0], v[0], "beta", lambda p: p.__setitem__(OFF, -100.0))
    big, zero = (gradients(units, (h, w, 8), batch, dtype, v, scale) for scale in (float("inf"), 0.0))
    for a, b in zip(big, zero):
        assert np.isfinite(a).all() and np.array_equal(a, b)
