"""Routing kernels at the edges of their lane layouts: 8, 9, 16 and 17 K slices of the router and one or several experts
per lane; 1 to 64 groups with 64 to 1 lanes each; more than 16 and 32 selected experts (the wider steps of the gate
sum); NaN, infinities and ties.  Against the CPU oracle, as the parity tests do."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_12696_amd as moe
import synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from test_gpu_parity import WTOL, _abs_bits, _grouped_margins_ok, check_grouped_selection

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("T,d,E,k", [(2, 4096, 256, 8), (3, 4608, 200, 7), (5, 8192, 64, 6), (3, 8224, 128, 8),
                                     (2, 8224, 300, 9), (2, 4640, 520, 4)])
def test_router_slices(T, d, E, k):
    x, w = synth.activations(T, d, seed=T), synth.router_weight(E, d, seed=E)
    lg = torch.empty(T, E, dtype=torch.float32, device=DEV)
    ws = torch.full((moe.moe_router_workspace_size(T, d, E),), 0x7F, dtype=torch.uint8, device=DEV)
    idx, _ = moe.moe_route_topk_hidden(x.to(DEV), w.to(DEV), k, 0, logits=lg, workspace=ws)
    # exact bf16 products summed in fp32 in any order: |err| <= (d - 1) * 2^-24 * sum |x w|
    tol = d * 2.0 ** -24 * oracle.router_logits(_abs_bits(x), _abs_bits(w))
    assert np.all(np.abs(lg.cpu().numpy().astype(np.float64) - oracle.router_logits(x, w)) <= tol)
    assert np.array_equal(idx.cpu().numpy(), oracle.route(lg.cpu().numpy(), k, 0)[0])


@pytest.mark.parametrize("E,k,score", [(64, 16, 0), (65, 17, 1), (256, 33, 0), (1000, 64, 1), (3, 3, 0)])
@pytest.mark.parametrize("kind", ["scattered", "ties", "special"])
def test_topk_wide(E, k, score, kind):
    T = 5
    lg = synth.logits_tie_grid(T, E, seed=E) if kind == "ties" else synth.logits_scattered(T, E, seed=E)
    if kind == "special":  # NaN ranks after -inf; the finite logits of the first token stay above k
        lg[1:, 0] = float("nan")
        lg[1:, E // 2] = -float("inf")
        lg[1:, E - 1] = -0.0
    idx, w = moe.moe_route_topk(lg.to(DEV), k, score)
    idx_o, w_o = oracle.route(lg.numpy(), k, score)
    assert np.array_equal(idx.cpu().numpy(), idx_o)
    fin = np.isfinite(np.take_along_axis(lg.numpy(), idx_o, 1)).all(1)
    assert fin.any() and np.abs(w.cpu().numpy().astype(np.float64) - w_o)[fin].max() <= WTOL


@pytest.mark.parametrize("T,E,G,TG,k", [(5, 64, 1, 1, 8), (9, 128, 64, 5, 7), (4, 96, 2, 1, 40), (3, 1024, 2, 1, 33), (6, 330, 33, 9, 17),
                                        (7, 256, 16, 16, 20), (2, 1000, 5, 2, 64)])
def test_grouped_lanes(T, E, G, TG, k):
    lg, b = synth.logits_scattered(T, E, seed=T + E), synth.router_bias(E, seed=E)
    idx, w = moe.moe_route_topk_grouped(lg.to(DEV), b.to(DEV), k, G, TG, 1.5)
    idx_o, w_o = oracle.route_grouped(lg.numpy(), b.numpy(), k, G, TG, 1.5)
    ig, wg = idx.cpu().numpy(), w.cpu().numpy().astype(np.float64)
    for t in range(T):
        if list(ig[t]) == list(idx_o[t]):
            assert np.abs(wg[t] - w_o[t]).max() <= 1.5 * WTOL
        else:  # a near-tie in fp64
            assert not _grouped_margins_ok(lg.numpy(), b.numpy(), k, G, TG, t)
            check_grouped_selection(ig[t], lg.numpy()[t], b.numpy(), k, G, TG)


def test_grouped_nan_only_counts_in_a_short_group():
    # Groups of two: group 0 holds a NaN, so its score is NaN and ranks after every number.
    lg = torch.tensor([[5.0, float("nan"), 0.0, 0.1, -1.0, -1.1, -3.0, -3.1]])
    idx, _ = moe.moe_route_topk_grouped(lg.to(DEV), None, 4, 4, 2, 1.0)
    assert idx.cpu().tolist() == [[3, 2, 4, 5]]
