"""Stages that run their weight gradients on a second stream (20 M values per convolution output on average and more), whole steps against
the float64 oracle.  The batch is copies of a small one, see Pair(tile=...)."""
import pytest

import synth
from harness import Pair, TOL, assert_close, assert_two_streams
from oracle import layers as L
from oracle import models as OM

pytestmark = pytest.mark.gpu


def conv(cin, cout, kh=1, kw=1, stride=1, act=L.ACT_RELU6):
    import paper_2110_02781_amd.binding as B
    ph, pw = kh // 2, kw // 2
    return (OM.Unit('conv', cin, cout, kh, kw, stride, ph, pw, act=act),
            dict(kind=B.UNIT_CONV, cin=cin, cout=cout, kh=kh, kw=kw, stride=stride, pad_h=ph, pad_w=pw, act=act))


def block(cin, cout, stride):
    import paper_2110_02781_amd.binding as B
    return (OM.Unit('invres', cin, cout, 3, 3, stride, 1, 1, expand=6, act=L.ACT_RELU6),
            dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=6))


def two_steps(units, shape, batch, tile, dtype, layers):
    """Two forward-backward pairs in a row, the first with and the second without an input gradient: the second one's weight gradients add to the
    first one's, and its first buffers are those that the first one's side stream read last."""
    o, h = [u[0] for u in units], [u[1] for u in units]
    tol = TOL[dtype]
    pair = Pair(o, h, shape, batch, 0, len(o), dtype, seed=9, ties="bounded", tile=tile)
    try:
        for step in range(2):
            y, yo = pair.forward(0, synth.normal(51, f"x{step}", (batch // tile,) + shape))
            assert_close(y, yo, tol, "y")
            dy = synth.normal(51, f"dy{step}", (batch // tile,) + tuple(pair.out_shape))
            run = lambda: dx.append(pair.backward(0, dy, want_dx=step == 0))
            dx = []
            if step == 0:
                assert_two_streams(layers, run)
                assert_close(*dx[0], tol, "dx")
            else:
                run()
            pair.compare_unit_vectors("grads", tol, floor=1e-6)
    finally:
        pair.close()


def test_layers_too_short_to_fork_behind_forked_ones():
    """Two layers of 115 M values, a convolution through the patch matrix and a block's project layer of 0.4 M (too short to fork: they run on the
    caller's stream and wait for the side stream, whose workspace they share), blocks of up to 2.4 M that fork once."""
    print("two streams: long and short layers, fp32", flush=True)
    units = [conv(8, 144), conv(144, 144), conv(144, 32, 3, 3, 8), block(32, 32, 1), block(32, 32, 2)]
    two_steps(units, (112, 112, 8), 64, 16, "f32", 6)


# behind two long layers and one of 14x14: convolutions (3x3, by stride) and blocks (output channels, stride).  The depthwise layers' input rows: 12544 and
# 256, 1024 alone, 256 twice; every one's partial weight gradients wait for the end of the call
SHORT = {"behind a long one": [(32, 2), 4, (32, 1)], "alone": [4, (32, 1)], "two": [8, (24, 1), (32, 1)]}


@pytest.mark.parametrize("which", SHORT)
def test_short_blocks_on_two_streams(which):
    """Blocks that a stage of short layers would run in the short kernels.  Single precision: the places do not depend on the type, and through BatchNorms over
    16 different values a bfloat16 chain has no bound (activation decisions off by more than a tie)."""
    print(f"two streams: short blocks, {which}", flush=True)
    units, c = [conv(8, 144), conv(144, 144), conv(144, 32, 3, 3, 8)], 32
    for what in SHORT[which]:
        units.append(conv(c, c, 3, 3, what) if isinstance(what, int) else block(c, *what))
        c = c if isinstance(what, int) else what[0]
    two_steps(units, (112, 112, 8), 64, 16, "f32", 4)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_convolutions_along_one_axis_on_two_streams(dtype):
    """655360 rows of 64 channels: weight gradients on the side stream, that of the first layer on the caller's where there is no input gradient."""
    print(f"two streams: convolutions along one axis {dtype}", flush=True)
    two_steps([conv(64, 64, 1, 5, act=L.ACT_RELU), conv(64, 64, 1, 3, act=L.ACT_RELU), conv(64, 64, 1, 9, act=L.ACT_RELU)], (1, 256, 64), 2560, 64, dtype, 3)
