"""The loss entry point that allocates nothing (ftp_softmax_ce_static: its per-row losses live in a file-scope device
array) against ftp_stage_loss, through the C ABI: same loss and same logits gradient, bit for bit, on two calls in a
row, the second on a smaller input; sizes beyond the array are refused."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def stage_loss_reference(P, torch, dtype, batch, classes, logits, labels):
    """(loss, dlogits) of ftp_stage_loss + ftp_stage_backward on a stage that holds only the loss unit."""
    B = P.binding
    units = [dict(kind=B.UNIT_FC, cin=8, cout=classes), dict(kind=B.UNIT_LOSS, cin=classes, cout=classes)]
    model = P.model_create(units, 1, 1, 8, P.F32 if dtype == "f32" else P.BF16)
    stage = P.stage_create(model, 1, 2, batch, 1)
    try:
        sp = torch.cuda.current_stream().cuda_stream
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        d = torch.full_like(logits, float("nan"))
        P.stage_forward(stage, 0, logits, None, sp)
        P.stage_loss(stage, 0, labels, loss, sp)
        P.stage_backward(stage, 0, None, d, sp)
        torch.cuda.synchronize()
        return loss.clone(), d
    finally:
        P.stage_destroy(stage)
        P.model_destroy(model)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_static_loss_matches_stage_loss_on_two_calls_in_a_row(dtype):
    import torch
    import paper_2110_02781_amd as P
    from oracle import layers as L
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    sp = torch.cuda.current_stream().cuda_stream
    for call, (batch, classes) in enumerate([(48, 1000), (7, 10)]):      # the second call is the smaller one
        print(f"static loss {dtype} call {call}: batch {batch} classes {classes}", flush=True)
        logits = torch.from_numpy(synth.normal(90 + call, "logits", (batch, classes), std=3.0).astype(np.float32)).cuda().to(tdt)
        labels = torch.from_numpy(synth.labels(90 + call, "labels", batch, classes).astype(np.int32)).cuda()
        loss = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
        d = torch.full_like(logits, float("nan"))
        P.softmax_ce_static(logits, labels, batch, classes, P.F32 if dtype == "f32" else P.BF16, d, loss, sp)
        torch.cuda.synchronize()
        ref_loss, ref_d = stage_loss_reference(P, torch, dtype, batch, classes, logits, labels)
        assert torch.equal(loss, ref_loss), (float(loss), float(ref_loss))
        assert torch.equal(d, ref_d)
        # and both against the oracle's definition on the values the kernels saw
        lo, do = L.softmax_ce(logits.float().cpu().numpy().astype(np.float64), labels.cpu().numpy())
        tol = 1e-4 if dtype == "f32" else 2e-2
        assert abs(float(loss) - lo) <= tol * max(1.0, abs(lo))
        assert np.abs(d.float().cpu().numpy() - do).max() <= tol * np.abs(do).max()


def test_static_loss_refuses_what_the_array_cannot_hold():
    import torch
    import paper_2110_02781_amd as P
    t = torch.zeros(16, device="cuda")
    li = torch.zeros(16, dtype=torch.int32, device="cuda")
    with pytest.raises(P.FtpError) as ei:
        P.softmax_ce_static(t, li, P.STATIC_LOSS_MAX_BATCH + 1, 4, P.F32, t, t, None)
    assert ei.value.status == -1 and "beyond" in str(ei.value)
    for bad in (dict(batch=0), dict(classes=0), dict(dtype=7)):
        kw = dict(batch=4, classes=4, dtype=P.F32)
        kw.update(bad)
        with pytest.raises(P.FtpError):
            P.softmax_ce_static(t, li, kw["batch"], kw["classes"], kw["dtype"], t, t, None)
    with pytest.raises(P.FtpError):
        P.softmax_ce_static(None, li, 4, 4, P.F32, t, t, None)


# the edges of the one-block form (rounds and lane groups of each width), of the row widths a wavefront holds, and the
# general form; a column of the buffer in front makes the last two start off a 16-byte line
@pytest.mark.parametrize("batch,classes,offset", [(1, 1, 0), (256, 16, 0), (257, 16, 0), (128, 17, 0), (129, 64, 0), (64, 65, 0), (32, 256, 0),
                                                  (33, 256, 0), (16, 257, 0), (17, 257, 0), (16, 1024, 0), (17, 1024, 0), (130, 512, 0),
                                                  (2049, 3, 0), (8300, 9, 0), (5, 1025, 0), (40, 1000, 1), (40, 300, 3)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_static_loss_over_the_forms_it_takes(dtype, batch, classes, offset):
    import torch
    import paper_2110_02781_amd as P
    from oracle import layers as L
    print(f"static loss {dtype} batch {batch} classes {classes} offset {offset}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    n = batch * classes
    buf = torch.zeros(n + 8, dtype=tdt, device="cuda")
    logits = buf[offset:offset + n].view(batch, classes)
    logits.copy_(torch.from_numpy(synth.normal(93, "logits", (batch, classes), std=3.0).astype(np.float32)).cuda().to(tdt))
    lab = synth.labels(93, "labels", batch, classes).astype(np.int32)
    labels = torch.from_numpy(lab).cuda()
    out = torch.full((n + 8,), 7.0, dtype=tdt, device="cuda")
    d = out[offset:offset + n].view(batch, classes)
    loss = torch.full((1,), float("nan"), device="cuda")
    sp = torch.cuda.current_stream().cuda_stream
    args = (labels, batch, classes, P.F32 if dtype == "f32" else P.BF16)
    P.softmax_ce_static(logits, *args, d, loss, sp)
    lo, do = L.softmax_ce(logits.float().cpu().numpy().astype(np.float64), lab)
    # 32-bit arithmetic: up to 16 terms a lane, a tree over the lanes, exp and log within a few units of 2^-24; then one rounding
    assert abs(float(loss) - lo) <= 2e-6 * max(1.0, abs(lo))
    assert np.abs(d.float().cpu().numpy() - do).max() <= (2e-6 if dtype == "f32" else 2.0 ** -8) * max(np.abs(do).max(), 1e-30) + 2e-7 / batch
    assert bool((out[:offset] == 7).all()) and bool((out[offset + n:] == 7).all())
    # the same values from buffers that do lie on 16-byte lines: the same bits
    d2, loss2 = torch.empty_like(d), torch.empty_like(loss)
    P.softmax_ce_static(logits.clone(), *args, d2, loss2, sp)
    assert torch.equal(d2, d) and torch.equal(loss2, loss)
    # an invalid label: NaN loss
    labels[batch - 1] = classes
    P.softmax_ce_static(logits, *args, d, loss, sp)
    assert bool(torch.isnan(loss).all())
