"""Weight gradients that a small stage runs together at the end of its backward call, against the float64 oracle: the edges of
the tiles (128 along the wider of the channel counts, 16 to 64 along the narrower, 256 rows) and of the sums over partials."""
import pytest

import synth
from harness import Pair, TOL, assert_close, launches
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu


def chain(channels):
    import paper_2110_02781_amd.binding as B
    o = [OM.Unit('conv', a, b, 1, 1, 1, 0, 0, act=L.ACT_NONE) for a, b in zip(channels, channels[1:])]
    h = [dict(kind=B.UNIT_CONV, cin=a, cout=b, kh=1, kw=1, stride=1, pad_h=0, pad_w=0, act=B.ACT_NONE) for a, b in zip(channels, channels[1:])]
    return o, h


# (channels of a chain of pointwise layers, rows as H x W, batch): one row tile and less, exactly one, one row more, 16 and 17
# partials (the two forms of their sum), more than 128; wide before narrow and after it, equal, off 16 / 64 / 128; a chain of 40 layers
# is more than a launch takes; the second backward adds to what the first has left
CASES = [([8, 8], 3, 5, 1), ([16, 136, 24], 16, 16, 1), ([24, 144, 40], 257, 1, 1), ([64, 72, 264], 31, 33, 4), ([40, 48], 64, 64, 1),
         ([72, 80], 241, 17, 1), ([136, 128], 9, 113, 4), ([8, 16, 96, 24], 93, 127, 3), ([16] * 41, 5, 6, 11),
         ([16, 136, 24] * 3, 16, 16, 1), ([24, 144, 40] * 3, 257, 1, 1), ([8, 264] * 4, 13, 31, 1)]


# bfloat16 roundings chained over many layers have no bound to hold a run against
RUNS = [c + (dt,) for c in CASES for dt in ("f32", "bf16") if dt == "f32" or len(c[0]) <= 3]


@pytest.mark.parametrize("channels,h,w,batch,dtype", RUNS, ids=[f"{'-'.join(map(str, c[0][:4]))}x{len(c[0]) - 1}_{c[1]}x{c[2]}_b{c[3]}_{c[4]}" for c in RUNS])
def test_weight_gradients_at_the_end_of_the_call(channels, h, w, batch, dtype):
    print(f"pointwise chain {channels[:5]} ({len(channels) - 1} layers) {h}x{w} batch {batch} {dtype}", flush=True)
    o, hu = chain(channels)
    tol = TOL[dtype]
    pair = Pair(o, hu, (h, w, channels[0]), batch, 0, len(o), dtype, n_slots=2, seed=6)
    try:
        for slot in range(2):
            y, yo = pair.forward(slot, synth.normal(31, f"x{slot}", (batch, h, w, channels[0])))
            assert_close(y, yo, tol, "y")
        for slot in range(2):
            dx, dxo = pair.backward(slot, synth.normal(31, f"dy{slot}", yo.shape))
            assert_close(dx, dxo, tol, f"dx {slot}")
            pair.compare_unit_vectors("grads", tol, floor=1e-6)
    finally:
        pair.close()


# (channels of a chain, rows as H x W, batch, the types whose layers each run their weight gradient next to the data gradient: no partial
# sums are left then): both sides of the lines, one layer of up to 2048 rows, several of up to 1600 together, two of up to 2080 in
# bfloat16, two to four of up to 3200 in fp32 (150 M products), 300 M products
AT_ONCE = [([64, 72], 32, 64, 1, "f32 bf16"), ([64, 72], 3, 683, 1, ""), ([24, 40] * 3 + [24], 2, 133, 1, "f32 bf16"), ([24, 40] * 3 + [24], 3, 89, 1, ""),
           ([24, 40] * 2 + [24], 20, 20, 1, "f32 bf16"), ([24, 40] * 2 + [24], 401, 1, 1, "f32"), ([24, 40] * 2 + [24], 20, 40, 1, "f32"),
           ([24, 40] * 2 + [24], 9, 89, 1, ""), ([64, 72, 64], 26, 40, 1, "f32 bf16"), ([64, 72, 64], 3, 347, 1, "f32"), ([64, 72, 64], 40, 40, 1, "f32"),
           ([64, 72, 64], 1601, 1, 1, ""), ([320, 288, 320], 27, 30, 1, "f32 bf16"), ([320, 288, 320], 5, 163, 1, ""),
           ([320, 1280], 16, 45, 1, "f32 bf16"), ([320, 1280], 16, 46, 1, ""), ([16, 48, 8], 17, 1, 3, "f32 bf16")]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("channels,h,w,batch,at_once", AT_ONCE, ids=[f"{'-'.join(map(str, c[0]))}_{c[1]}x{c[2]}" for c in AT_ONCE])
def test_a_few_short_layers_run_both_gradients_at_once(channels, h, w, batch, at_once, dtype):
    print(f"pointwise chain {channels} {h}x{w} batch {batch} {dtype}", flush=True)
    o, hu = chain(channels)
    pair = Pair(o, hu, (h, w, channels[0]), batch, 0, len(o), dtype, seed=8)
    try:
        y, yo = pair.forward(0, synth.normal(32, "x", (batch, h, w, channels[0])))
        got = []
        n = launches(lambda: got.append(pair.backward(0, synth.normal(32, "dy", yo.shape))))
        assert ("reduce_partials" not in n) == (dtype in at_once.split()), n
        if dtype == "f32" or len(o) <= 2:
            assert_close(y, yo, TOL[dtype], "y")
            assert_close(*got[0], TOL[dtype], "dx")
            pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
    finally:
        pair.close()


def test_a_stage_with_a_longer_layer_runs_its_short_ones_with_it():
    """A stride-2 block: the expand layer has 2304 rows, the project layer 576."""
    import paper_2110_02781_amd.binding as B
    print("stride-2 block, 2304 and 576 rows f32", flush=True)
    o = [OM.Unit('invres', 16, 24, 3, 3, 2, 1, 1, expand=6, act=L.ACT_RELU6)]
    h = [dict(kind=B.UNIT_INVRES, cin=16, cout=24, kh=3, kw=3, stride=2, pad_h=1, pad_w=1, expand=6, act=B.ACT_RELU6)]
    pair = Pair(o, h, (16, 16, 16), 9, 0, 1, "f32", seed=9, ties="bounded")
    try:
        y, yo = pair.forward(0, synth.normal(33, "x", (9, 16, 16, 16)))
        assert_close(y, yo, TOL["f32"], "y")
        got = []
        n = launches(lambda: got.append(pair.backward(0, synth.normal(33, "dy", yo.shape))))
        assert "pw_bwd" not in n, n
        assert_close(*got[0], TOL["f32"], "dx")
        pair.compare_unit_vectors("grads", TOL["f32"], floor=1e-6)
    finally:
        pair.close()


# (channels, H x W, batch): a single bfloat16 layer of 16384 rows and more with up to 32 outputs runs by itself: a last chunk of one row
# and of a few, outputs off 16, several column tiles; fewer rows, more outputs and two layers do not
NARROW = [([24, 32], 113, 145, 1), ([96, 24], 128, 64, 2), ([40, 8], 131, 129, 1), ([200, 32], 64, 64, 9), ([24, 32], 127, 129, 1), ([24, 40], 113, 145, 1),
          ([24, 32, 16], 113, 145, 1)]


@pytest.mark.parametrize("want_dx", [True, False])
@pytest.mark.parametrize("channels,h,w,batch", NARROW, ids=[f"{'-'.join(map(str, c[0]))}_{c[1]}x{c[2]}_b{c[3]}" for c in NARROW])
def test_a_single_narrow_layer_runs_by_itself(channels, h, w, batch, want_dx):
    print(f"narrow pointwise {channels} {h}x{w} batch {batch} bf16 dx {want_dx}", flush=True)
    o, hu = chain(channels)
    pair = Pair(o, hu, (h, w, channels[0]), batch, 0, len(o), "bf16", seed=8)
    try:
        y, yo = pair.forward(0, synth.normal(34, "x", (batch, h, w, channels[0])))
        dx, dxo = pair.backward(0, synth.normal(34, "dy", yo.shape), want_dx=want_dx)
        if want_dx:
            assert_close(dx, dxo, TOL["bf16"], "dx")
        pair.compare_unit_vectors("grads", TOL["bf16"], floor=1e-6)
    finally:
        pair.close()
