"""Convolutions along one axis (implicit GEMMs, csrc/k_conv1d.hip) against the float64 oracle, at the edges of their tiles."""
import pytest

import synth
from harness import Pair, TOL, assert_close, launches
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
# tiles (64 x 32 or 64 x 64, weight gradient in pieces of 32 x 80): windows shorter than a tile, longer, odd and the shortest;
# channels off 8 and off 4; columns off 16 and 32; a last tile of one row; more row tiles than partials; each tap count.
# In bfloat16 the wider of the first layers go through patch matrices: ROUTES has row tiles of that type.
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


# Row tiles: 32, 64 and 128 rows with a last one of 31, 1 and 63 rows; two and three tiles to a block; weights in two phases, with one tile
# and with two; windows of 16 (the weight gradient's counter wraps twice a step); whole tiles only; 4, 2 and 1 pieces to a wavefront group.
TILES = [([64], 64, 5, 8191, 1, "f32"), ([64], 64, 5, 2731, 3, "f32"), ([9], 32, 5, 2340, 7, "f32"), ([64], 64, 9, 21, 1563, "f32"), ([8], 8, 3, 16, 2050, "f32"),
         ([32], 32, 5, 128, 256, "f32"), ([40], 24, 7, 5471, 3, "f32"), ([64], 64, 9, 16, 3073, "f32"), ([12, 24], 32, 5, 16, 3073, "f32"),
         ([16], 32, 5, 16, 1040, "bf16"), ([24, 24], 32, 9, 49, 47, "bf16")]


@pytest.mark.parametrize("cins,cout,k,w,batch,dtype", TILES, ids=["-".join(map(str, c)).replace(" ", "") for c in TILES])
def test_conv1d_row_tiles(cins, cout, k, w, batch, dtype):
    test_conv1d_edges(cins, cout, k, w, batch, dtype)


# (cin, cout, taps, window, batch, copies in the batch, first unit of the model, type, by the kernels for these layers): both sides of the lines
# of conv1d_pays, single layers and (two couts) chains; 64-row tiles with a last one of one row, of 63, two column halves
ROUTES = [(32, 64, 9, 64, 64, 8, False, "bf16", False), (32, 64, 9, 65, 64, 1, False, "bf16", True), (24, 32, 9, 49, 47, 1, False, "bf16", True),
          (64, 64, 3, 127, 64, 8, False, "bf16", False), (64, 64, 9, 83, 99, 1, False, "bf16", False), (48, 40, 7, 64, 127, 1, False, "bf16", True),
          (48, 40, 7, 65, 127, 1, False, "bf16", False),
          (64, 48, 7, 128, 400, 40, False, "bf16", False), (64, 64, 3, 128, 312, 24, False, "bf16", True), (64, 64, 3, 128, 320, 32, False, "bf16", False), (40, 64, 3, 128, 800, 80, False, "bf16", False),
          (8, 8, 3, 128, 560, 56, False, "bf16", True), (8, 8, 3, 128, 768, 64, False, "bf16", False), (16, 48, 3, 128, 2400, 240, False, "bf16", True),
          (8, 8, 3, 128, 1600, 80, False, "f32", False), (8, 16, 3, 128, 1600, 80, False, "f32", True),
          (9, 32, 5, 127, 32, 1, True, "bf16", False), (9, 32, 3, 63, 65, 1, True, "bf16", True), (16, 64, 5, 63, 65, 1, True, "bf16", False),
          (3, 16, 3, 128, 191, 1, True, "bf16", True), (3, 16, 3, 128, 192, 24, True, "bf16", False), (64, 24, 5, 91, 99, 1, True, "bf16", True),
          (9, 32, 5, 128, 255, 15, True, "f32", True), (9, 32, 5, 128, 256, 32, True, "f32", False), (9, 64, 5, 128, 256, 32, True, "f32", True)]


@pytest.mark.parametrize("cin,cout,k,w,batch,tile,first,dtype,here", ROUTES, ids=["-".join(map(str, c)) for c in ROUTES])
def test_conv1d_routes(cin, cout, k, w, batch, tile, first, dtype, here):
    print(f"conv1d route {cin}->{cout} taps {k} window {w} batch {batch} first {first} {dtype}", flush=True)
    o, h = units([cin] if first else [cin, cin], cout, k, L.ACT_NONE)
    tol = TOL[dtype]
    pair = Pair(o, h, (1, w, cin), batch, len(o) - 1, len(o), dtype, seed=6, tile=tile)
    try:
        got = []
        n = launches(lambda: got.append(pair.forward(0, synth.normal(23, "x", (batch // tile, 1, w, cin)))))
        assert ("conv1d_fwd" in n) == here and ("im2col" in n or "conv_direct_fwd" in n) != here, n
        assert_close(*got[0], tol, "y")
        dy = synth.normal(23, "dy", (batch // tile,) + tuple(pair.out_shape))
        n = launches(lambda: got.append(pair.backward(0, dy, want_dx=not first)))
        assert ("conv1d_wgrad" in n) == here, n
        if not first:
            assert_close(*got[1], tol, "dx")
        pair.compare_unit_vectors("grads", tol, floor=1e-6)
        pair.compare_unit_vectors("bn", tol)
    finally:
        pair.close()


# Two, three and four pieces of the weight gradient on both sides of the lines at which a block takes more of them (so that fewer blocks read the
# same rows), a last tile of 62 rows and less; partials: what the launch leaves, one for every range of rows
PIECES = [(8, 64, 3, 252, "f32", 128), (8, 64, 3, 256, "f32", 194), (32, 32, 3, 256, "bf16", 194), (64, 8, 3, 168, "f32", 85), (64, 8, 3, 252, "f32", 128),
          (64, 8, 3, 256, "f32", 194), (64, 8, 3, 256, "bf16", 194), (32, 64, 3, 252, "f32", 128), (32, 64, 3, 256, "f32", 194), (64, 64, 3, 256, "f32", 78)]


@pytest.mark.parametrize("cin,cout,k,batch,dtype,partials", PIECES, ids=["-".join(map(str, c)) for c in PIECES])
def test_conv1d_weight_gradient_pieces(cin, cout, k, batch, dtype, partials):
    import torch
    import paper_2110_02781_amd as P
    print(f"conv1d weight gradient {cin}->{cout} taps {k} batch {batch} {dtype}", flush=True)
    o, h = units([cin, cin], cout, k, L.ACT_NONE)
    pair = Pair(o, h, (1, 97, cin), batch, 1, 2, dtype, seed=7, tile=4)
    try:
        pair.forward(0, synth.normal(24, "x", (batch // 4, 1, 97, cin)))
        torch.cuda.synchronize()
        P.ktrace_begin()
        dx, dxo = pair.backward(0, synth.normal(24, "dy", (batch // 4,) + tuple(pair.out_shape)))
        torch.cuda.synchronize()
        row = {r["name"]: r for r in P.ktrace_end()}["conv1d_wgrad"]
        moved = row["alg_bytes"] / row["launches"] - batch * 97 * (cin + cout) * (4 if dtype == "f32" else 2)
        assert moved == partials * cout * k * cin * 4
        assert_close(dx, dxo, TOL[dtype], "dx")
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
    finally:
        pair.close()


@pytest.mark.parametrize("cins,cout,k,w,batch,tile,dtype,n_here", [([9, 32, 64], 64, 5, 128, 240, 24, "bf16", 3), ([9, 32, 64], 64, 5, 128, 280, 28, "bf16", 2),
                                                                  ([16, 16, 16], 16, 3, 128, 800, 80, "bf16", 2), ([8, 8, 8], 8, 3, 128, 1600, 100, "bf16", 0),
                                                                  ([8, 8, 16], 64, 3, 128, 1600, 100, "f32", 2)])
def test_conv1d_chains_of_both_routes(cins, cout, k, w, batch, tile, dtype, n_here):
    """The first layer's patches wait for its weight gradient while layers of either kind run behind it; the BatchNorm-backward sums of a
    layer come from the data gradient behind it or from a pass of their own."""
    print(f"conv1d chain {cins} -> {cout} taps {k} window {w} batch {batch} {dtype}", flush=True)
    o, h = units(cins, cout, k, L.ACT_NONE if dtype == "bf16" else L.ACT_RELU)
    pair = Pair(o, h, (1, w, cins[0]), batch, 0, len(o), dtype, seed=7, tile=tile, ties="off" if dtype == "bf16" else "bounded")
    try:
        got = []
        for step in range(2):
            n = launches(lambda: got.append(pair.forward(0, synth.normal(24, f"x{step}", (batch // tile, 1, w, cins[0])))))
            assert n.get("conv1d_fwd", 0) == n_here, n
            assert_close(*got[-1], TOL[dtype], "y")
            pair.backward(0, synth.normal(24, f"dy{step}", (batch // tile,) + tuple(pair.out_shape)), want_dx=False)
            pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
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


# chains of up to 2048 rows: the BatchNorm backward of all but the last layer is done on the way into its gradients, from sums the layer
# behind has left (in alternating halves of a buffer, so three in a row); 2048 rows and one window more; rows off 16; few channels, which
# keep launches of their own; the widest, which keep them where there are more blocks than CUs, and above 1536 rows in bfloat16
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cins,cout,k,w,batch,n_bn", [([9, 32, 64, 64], 64, 5, 128, 8, 1), ([16, 16, 24, 40], 16, 3, 16, 1, 1), ([3, 64, 64], 64, 9, 32, 64, {"f32": 2, "bf16": 3}), ([3, 64, 64], 64, 5, 32, 48, {"f32": 2, "bf16": 2}), ([16, 32], 24, 3, 96, 16, 1), ([16, 32], 24, 3, 97, 16, {"f32": 1, "bf16": 2}),
                                                      ([12, 8, 32], 24, 7, 37, 11, 1), ([32, 48, 16], 32, 5, 128, 17, 0)])
def test_conv1d_short_chains(cins, cout, k, w, batch, n_bn, dtype):
    print(f"conv1d short chain {cins} -> {cout} taps {k} window {w} batch {batch} {dtype}", flush=True)
    o, h = units(cins, cout, k, L.ACT_NONE if dtype == "bf16" else L.ACT_RELU)
    pair = Pair(o, h, (1, w, cins[0]), batch, 0, len(o), dtype, seed=9, ties="off" if dtype == "bf16" else "bounded")
    try:
        got = []
        for step in range(2):
            y, yo = pair.forward(0, synth.normal(25, f"x{step}", (batch, 1, w, cins[0])))
            assert_close(y, yo, TOL[dtype], "y")
            n = launches(lambda: got.append(pair.backward(0, synth.normal(25, f"dy{step}", yo.shape))))
            assert n.get("bn_bwd_small", 0) == (n_bn[dtype] if isinstance(n_bn, dict) else n_bn), n
            assert_close(*got[-1], TOL[dtype], "dx")
            pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
            pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()
