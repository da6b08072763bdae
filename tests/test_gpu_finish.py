"""BatchNorm finished by the kernel that applies it (csrc/k_elem.hip: bn_finish_apply_k, bn_bwd_finish_apply_k) against the float64 oracle."""
import pytest

import synth
from harness import Pair, TOL, assert_close, routes
from oracle import models as OM

pytestmark = pytest.mark.gpu

# (cin, cout, expand, stride, h, w, batch): the fewest rows; slabs of 5, 6 and 7 column groups, a last slab of fewer (72, 88, 104 channels); 8 channels;
# a residual; more partials than one round of a thread's requests; the most values, and beyond them
CASES = [(24, 24, 3, 1, 3, 683, 1), (16, 104, 4, 1, 41, 50, 1), (8, 8, 11, 1, 45, 46, 1), (32, 88, 6, 2, 93, 95, 1), (16, 16, 6, 1, 50, 61, 2),
         (8, 24, 6, 1, 80, 100, 3), (24, 32, 6, 2, 112, 112, 8)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout,expand,stride,h,w,batch", CASES)
def test_finish_and_apply(dtype, cin, cout, expand, stride, h, w, batch):
    import paper_2110_02781_amd.binding as B
    print(f"finish {dtype} {cin}->{cout} x{expand} stride {stride} {h}x{w} batch {batch}", flush=True)
    o = [OM.Unit('invres', cin, cout, stride=stride, expand=expand)]
    hu = [dict(kind=B.UNIT_INVRES, cin=cin, cout=cout, stride=stride, expand=expand)]
    pair = Pair(o, hu, (h, w, cin), batch, 0, 1, dtype, seed=8, ties="bounded")
    try:
        x = synth.normal(51, "x", (batch, h, w, cin))

        def both():
            y, yo = pair.forward(0, x)
            assert_close(y, yo, TOL[dtype], "y")
            dx, dxo = pair.backward(0, synth.normal(51, "dy", yo.shape))
            assert_close(dx, dxo, TOL[dtype], "dx")
        took = routes(both)
        assert any("finish" in r for r in took), took
        pair.compare_unit_vectors("grads", TOL[dtype], floor=1e-6)
        pair.compare_unit_vectors("bn", TOL[dtype])
    finally:
        pair.close()
