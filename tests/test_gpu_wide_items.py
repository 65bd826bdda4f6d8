"""Items spread over more than three workgroups in the general kernels (T = 17: one more than the small calls' kernels
take, which cut no item): the fix-up then walks the ranges, and so does the combine, with and without the shared expert's
group, against the CPU oracle.  The spread itself is checked on the device's own grid size."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_12696_amd as moe
import synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from test_gpu_parity import YTOL, note, y_err
from test_split_bookkeeping import brute_owner, kernel_costs

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("fmt,size,shared,mx", [(0, 2048, False, False), (1, 1024, True, False), (2, 2048, False, False),
                                                (2, 1024, True, False), (2, 2048, False, True), (2, 1024, True, True)])
def test_items_over_more_than_three_workgroups(fmt, size, shared, mx):
    T, E = 17, 3
    note(f"wide items fmt={fmt} size={size} shared={shared} mx={mx}")
    W = min(torch.cuda.get_device_properties(0).multi_processor_count, 512)
    steps = size // (256 if fmt == 2 else 128)
    for band in (128, 256):  # gate/up, down
        own = brute_owner(kernel_costs(("bf16", "fp8", "fp4")[fmt], [T] * (2 if shared else 1)), size // band * steps, W)
        assert max(len(set(r)) for r in own.reshape(-1, steps).tolist()) > 3
    layer = synth.layer_weights(synth.Shape("w", size, size, E, 1, fmt, 1, shared), seed=size + fmt, device=DEV)
    if mx:
        layer["act_fmt"] = moe.MOE_ACTQ_MXFP8
    x = synth.activations(T, size, seed=fmt)
    lg = torch.zeros(T, E)
    lg[:, 1] = 3.0  # every token on expert 1
    dl = moe.pack_layer(layer)
    ws = torch.full((moe.moe_verify_workspace_size(dl, T, 1),), 0xFF, dtype=torch.uint8, device=DEV)
    y, r = moe.moe_verify_step(x.to(DEV), lg.to(DEV), dl, 1, 1, workspace=ws)
    idx, w = oracle.route(lg.numpy(), 1, 1)
    assert int(r.n_unique.item()) == 1
    rows = [0, 15, 16]
    host = {n: (v.cpu() if hasattr(v, "cpu") else v) for n, v in layer.items()}
    ref = oracle.verify_tokens(host, x, idx, w, tokens=rows, threads=8)
    assert y_err(y.float().cpu().numpy()[rows], ref) <= YTOL
    assert torch.isfinite(y.float()).all()
    assert np.array_equal(r.counts.cpu().numpy(), [0, T, 0])
