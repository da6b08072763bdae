"""Weight gradients that a small stage runs together at the end of its backward call, against the float64 oracle: the edges of
the tiles (128 along the wider of the channel counts, 16 to 64 along the narrower, 256 rows) and of the sums over partials."""
import pytest

import synth
from harness import Pair, TOL, assert_close
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
         ([72, 80], 241, 17, 1), ([136, 128], 9, 113, 4), ([8, 16, 96, 24], 93, 127, 3), ([16] * 41, 5, 6, 11)]


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
