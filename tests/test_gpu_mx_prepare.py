"""MX activations on both sides of the line between quantising in the union's launch and in one of its own: no union
(T <= 64), 320 and 321 quantising workgroups (two tokens of 4096 each) in a single pass of slots, and several passes;
and the timed entry point around those launches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_12696_amd as moe
import synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
# As in the parity tests: bf16 rounding of y, and MX codes that flip at a rounding boundary between fp32 and fp64.
YTOL = 1e-2


@pytest.mark.parametrize("T,k", [(1, 1), (64, 1), (65, 1), (640, 1), (641, 1), (643, 2), (1300, 1)])
def test_quantised_rows(T, k):
    d, d_ff, E = 4096, 96, 5
    print(f"MX prepare T={T} k={k}", flush=True)
    layer = dict(synth.layer_weights(synth.Shape("p", d, d_ff, E, k, synth.FMT_MXFP4, 0, False), seed=7, device=DEV),
                 act_fmt=moe.MOE_ACTQ_MXFP8)
    x = synth.activations(T, d, seed=T)
    lg = synth.logits_scattered(T, E, seed=T)
    dl = moe.pack_layer(layer)
    ws = torch.full((moe.moe_verify_workspace_size(dl, T, k),), 0xFF, dtype=torch.uint8, device=DEV)
    y, r = moe.moe_verify_step(x.to(DEV), lg.to(DEV), dl, k, 0, workspace=ws)
    idx, w = oracle.route(lg.numpy(), k, 0)
    u = oracle.union(idx, E)
    for name in ("counts", "union_ids", "offsets", "perm"):
        assert np.array_equal(getattr(r, name).cpu().numpy(), u[name]), name
    rows = sorted({0, 1 % T, T // 2, T - 1})
    host = {n: (v.cpu() if hasattr(v, "cpu") else v) for n, v in layer.items()}
    ref = oracle.verify_tokens(host, x, idx, w, tokens=rows, threads=8)
    got = y.float().cpu().numpy()[rows].astype(np.float64)
    assert np.abs(got - ref).max() <= YTOL * np.abs(ref).max()
    assert torch.isfinite(y.float()).all()


@pytest.mark.parametrize("T,mx", [(8, False), (8, True), (30, False), (30, True), (70, False), (70, True), (641, True)])
def test_timed_call_marks_and_result(T, mx):
    """The timed entry point's five marks lie in order around the same work, on each side of the launches before them."""
    d, d_ff, E, k = 4096, 96, 5, 1
    print(f"timed call T={T} mx={mx}", flush=True)
    layer = synth.layer_weights(synth.Shape("p", d, d_ff, E, k, synth.FMT_MXFP4, 0, False), seed=7, device=DEV)
    if mx:
        layer["act_fmt"] = moe.MOE_ACTQ_MXFP8
    x, dl = synth.activations(T, d, seed=T).to(DEV), moe.pack_layer(layer)
    idx, w = moe.moe_route_topk(synth.logits_scattered(T, E, seed=T).to(DEV), k, 0)
    r = moe.routing_for(idx, w, E)
    ws = torch.full((moe.moe_verify_workspace_size(dl, T, k),), 0xFF, dtype=torch.uint8, device=DEV)
    want = moe.moe_verify_layer(x, dl, r, workspace=ws)
    ws.fill_(0xFF)
    y, ev = torch.zeros_like(x), [torch.cuda.Event(enable_timing=True) for _ in range(7)]
    for e in ev:  # torch creates the HIP event on first record; the library records raw handles
        e.record()
    torch.cuda.synchronize()
    ev[0].record()
    moe.moe_verify_layer_timed(x, dl, r, y, ws, ev[1:6])
    ev[6].record()
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    spans = [ev[i].elapsed_time(ev[i + 1]) for i in range(6)]
    assert all(s >= 0 for s in spans) and min(spans[1], spans[3], spans[4]) > 0
