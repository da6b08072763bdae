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
