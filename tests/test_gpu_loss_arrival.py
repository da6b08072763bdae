"""The mean loss added by the last block to arrive (csrc/k_elem.hip, softmax_ce_wave_k): calls behind one another on the same counters, the forms
without them (a captured call, more streams than there are counters for), all bit for bit the same, against the oracle.  How exact and how small the probabilities are."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# one block and a few rows, 31, 32 and 33 blocks (the groups), a last block of one row, 513 and more blocks, more than 1024 (a captured call's mean takes them 1024 at a time); rows
# whose mean is a launch of its own on every stream: short ones beyond 8192 and 256 classes beyond 4096, four and eight rows a block
SIZES = [(17, 1000), (248, 300), (256, 1000), (257, 300), (600, 33), (1024, 40), (1025, 65), (4097, 250), (4096, 9), (8191, 200), (16390, 520),
         (4097, 264), (4099, 300), (16390, 9)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_last_block_adds_the_mean(dtype):
    import torch
    import paper_2110_02781_amd as P
    from oracle import layers as L
    tdt, code = (torch.float32, P.F32) if dtype == "f32" else (torch.bfloat16, P.BF16)
    first = {}
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def call(i, b, n, sp, logits, labels, d, loss):
        P.softmax_ce_static(logits, labels, b, n, code, d, loss, sp)

    for i, (b, n) in enumerate(SIZES):
        print(f"loss arrival {dtype} {b} x {n}", flush=True)
        logits = torch.from_numpy(synth.normal(95 + i, "logits", (b, n), std=3.0).astype(np.float32)).cuda().to(tdt)
        lab = synth.labels(95 + i, "labels", b, n).astype(np.int32)
        labels, d, loss = torch.from_numpy(lab).cuda(), torch.empty_like(logits), torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        for sp in (streams[0], streams[0], streams[1]):
            loss.fill_(-1.0)
            torch.cuda.synchronize()
            call(i, b, n, sp.cuda_stream, logits, labels, d, loss)
            torch.cuda.synchronize()
            first.setdefault(i, (loss.clone(), d.clone()))
            assert torch.equal(loss, first[i][0]) and torch.equal(d, first[i][1])
        lo, do = L.softmax_ce(logits.float().cpu().numpy().astype(np.float64), lab)
        # sums of 8 rows, then of partials in chains of up to 33, then a tree over 64 lanes: some 45 additions in 32 bits at most
        assert abs(float(loss) - lo) <= 45 * 2.0 ** -24 * max(1.0, abs(lo))
        assert np.abs(d.float().cpu().numpy() - do).max() <= (2e-6 if dtype == "f32" else 2.0 ** -8) * np.abs(do).max() + 2e-7 / b
        g = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        with torch.cuda.graph(g, stream=side):
            call(i, b, n, side.cuda_stream, logits, labels, d, loss)
        for _ in range(3):
            loss.fill_(-1.0)
            d.fill_(0.0)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(loss, first[i][0]) and torch.equal(d, first[i][1])


def test_more_streams_than_counters():
    """64 streams of a GPU have counters; on those that come later the mean is a launch of its own, with the same result."""
    import ctypes
    import torch
    import paper_2110_02781_amd as P
    import paper_2110_02781_amd.binding as B
    from harness import routes
    b, n, handles = 600, 33, []
    logits = torch.from_numpy(synth.normal(5, "logits", (b, n), std=3.0).astype(np.float32)).cuda()
    labels, d, loss = torch.from_numpy(synth.labels(5, "labels", b, n).astype(np.int32)).cuda(), torch.empty_like(logits), torch.zeros(1, device="cuda")
    first, how = None, []
    try:
        for _ in range(66):                                            # of this process's own: torch deals 32 out again and again
            h = ctypes.c_void_p()
            assert B.lib.hipStreamCreateWithFlags(ctypes.byref(h), 1) == 0
            handles.append(h)
        assert len({h.value for h in handles}) == 66
        for k in list(range(66)) + [0, 65]:
            loss.fill_(-1.0)
            torch.cuda.synchronize()
            how += routes(lambda: P.softmax_ce_static(logits, labels, b, n, P.F32, d, loss, handles[k].value))
            first = first or (loss.clone(), d.clone())
            assert torch.equal(loss, first[0]) and torch.equal(d, first[1])
        assert how[0].startswith("arrival") and sum(r.startswith("arrival") for r in how) <= 64 + 1 and how[65].startswith("two") and how[-1].startswith("two"), how
    finally:
        for h in handles:
            assert B.lib.hipStreamDestroy(h) == 0


@pytest.mark.parametrize("b,n,std", [(64, 1000, 2.0), (2048, 1000, 3.0), (4096, 10, 3.0), (256, 200, 3.0)])
def test_exponentials(b, n, std):
    """Logits on a grid of 2^-10: what is taken from the row's largest is exact.  Divided by a power of two of rows, a probability has the error of its exponential (a power of two that is right to about half
    a last place, r.m.s. 0.43 * 2^-24 as after a rounding) and of its product with the inverse sum (0.43): 0.60, and a tenth for the sample; the sum's own error, the same for
    a whole row, is taken out."""
    import torch
    import paper_2110_02781_amd as P
    print(f"loss, exponentials {b} x {n}", flush=True)
    x = torch.from_numpy((np.round(synth.normal(7, "logits", (b, n), std=std) * 1024) / 1024).astype(np.float32)).cuda()
    d, loss = torch.empty_like(x), torch.zeros(1, device="cuda")
    P.softmax_ce_static(x, torch.zeros(b, dtype=torch.int32, device="cuda"), b, n, P.F32, d, loss, 0)
    torch.cuda.synchronize()
    p = torch.softmax(x.double(), 1) / b
    e = ((d.double() - p) / p)[:, 1:]                                   # column 0 is the label's
    e = (e - e.median(1, keepdim=True).values) * 2.0 ** 24
    assert float(e.pow(2).mean().sqrt()) <= 0.66


def test_smallest_exponentials():
    """Probabilities below 2^-126 are kept as far as single precision holds them."""
    import torch
    import paper_2110_02781_amd as P
    x = torch.zeros(32, 300, device="cuda")
    x[:, 1:] = -torch.linspace(80, 104, 299, device="cuda")
    d, loss = torch.empty_like(x), torch.zeros(1, device="cuda")
    P.softmax_ce_static(x, torch.zeros(32, dtype=torch.int32, device="cuda"), 32, 300, P.F32, d, loss, 0)
    torch.cuda.synchronize()
    p = (torch.softmax(x.double(), 1) / 32)[:, 1:]
    # half a step of the smallest numbers in front of the division by 32 rows and behind it, and a few roundings
    assert bool(((d[:, 1:].double() - p).abs() <= 2.0 ** -149 + 4 * 2.0 ** -24 * p).all())
    assert float(d[0, 200]) > 0.0
