"""Verification passes of at most 16 tokens (their own kernels) against the CPU oracle, at the sizes where the
kernels' K blocks per wavefront, their tails and their split change: 1 to 8 rounds of eight 128-wide blocks in both
projections, ragged last blocks, fewer items than workgroups, both packings, biases, a shared expert, and 17 tokens or more than 64 blocks, which the general kernels take."""
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
# bf16 rounding of the SwiGLU rows and of y, relative to max|y|: 2^-9 each, the first averaged over d_ff products.
YTOL = 1e-2

# (d, d_ff): the reduction lengths cover 1, 2, ... 8 rounds per projection; 8224 is beyond the small kernels.
RAGGED = [(96, 1056), (1120, 96), (2080, 3104), (3232, 2112), (4128, 5152), (5280, 4160), (6176, 7200), (7232, 6240),
          (8192, 160), (160, 8192), (8224, 64)]
BLOCKED = [(128, 1152), (2176, 3200), (3328, 2176), (4224, 5248), (5376, 4224), (6272, 7296), (8192, 128), (128, 8192)]


def check(fmt, d, d_ff, T, E=2, k=1, shared=False, oai=False, pair=True, rows=2):
    print(f"small call fmt={fmt} d={d} d_ff={d_ff} T={T} E={E} k={k} shared={shared} oai={oai} pair={pair}", flush=True)
    sh = synth.Shape("s", d, d_ff, E, k, fmt, 1, shared)
    layer = synth.layer_weights(sh, seed=d + d_ff, device=DEV)
    if oai:
        layer.update(act=moe.MOE_ACT_SWIGLU_OAI, alpha=1.702, limit=7.0, b_gate=synth.expert_biases(E, d_ff, 1, "bg", DEV),
                     b_up=synth.expert_biases(E, d_ff, 1, "bu", DEV), b_down=synth.expert_biases(E, d, 1, "bd", DEV))
    x = synth.activations(T, d, seed=T)
    lg = synth.logits_scattered(T, E, seed=T + 1)
    dl = moe.pack_layer(layer, pair=pair, down_pair=pair)
    ws = torch.full((moe.moe_verify_workspace_size(dl, T, k),), 0xFF, dtype=torch.uint8, device=DEV)
    y, r = moe.moe_verify_step(x.to(DEV), lg.to(DEV), dl, k, sh.score, workspace=ws)
    y2, _ = moe.moe_verify_step(x.to(DEV), lg.to(DEV), dl, k, sh.score, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    idx_o, w_o = oracle.route(lg.numpy(), k, sh.score)
    u = oracle.union(idx_o, E)
    assert int(r.n_unique.item()) == u["n_unique"]
    for name in ("counts", "union_ids", "offsets", "perm"):
        assert np.array_equal(getattr(r, name).cpu().numpy(), u[name]), name
    pick = sorted({0, T - 1}) if rows == 2 else list(range(T))
    host = {n: (v.cpu() if hasattr(v, "cpu") else v) for n, v in layer.items()}
    ref = oracle.verify_tokens(host, x, idx_o, w_o, tokens=pick, threads=8)
    got = y.float().cpu().numpy()[pick].astype(np.float64)
    assert np.abs(got - ref).max() <= YTOL * np.abs(ref).max()
    return y


@pytest.mark.parametrize("fmt", [synth.FMT_BF16, synth.FMT_MXFP4])
@pytest.mark.parametrize("d,d_ff", RAGGED)
def test_rounds_and_ragged_blocks(fmt, d, d_ff):
    check(fmt, d, d_ff, 3)


@pytest.mark.parametrize("d,d_ff", BLOCKED)
def test_rounds_fp8(d, d_ff):
    check(synth.FMT_FP8, d, d_ff, 3, shared=True)


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17])
@pytest.mark.parametrize("fmt,shared,oai", [(0, False, True), (1, True, False), (2, True, True)])
@pytest.mark.parametrize("pair", [True, False])
def test_tokens_options_and_packings(T, fmt, shared, oai, pair):
    check(fmt, 384, 640, T, E=7, k=3, shared=shared, oai=oai, pair=pair, rows=T)


# Few large items: fewer than workgroups (one expert of 96 or 10 items), or little more than a range each.
@pytest.mark.parametrize("fmt,d,d_ff,E,oai", [(0, 4096, 1536, 1, False), (0, 8192, 1024, 1, True), (0, 4096, 160, 2, False),
                                              (1, 7168, 512, 3, True), (2, 8192, 512, 1, True), (1, 128, 4224, 1, False)])
def test_few_large_items(fmt, d, d_ff, E, oai):
    check(fmt, d, d_ff, 16, E=E, k=1, shared=fmt == 1, oai=oai)


def test_many_slots_per_token():
    check(synth.FMT_BF16, 64, 64, 16, E=1024, k=64, rows=16)


# Reductions of 1 to 8 blocks, whose items 1, 2 or 4 wavefronts share: 8, 4 or 2 items side by side.  Experts of a
# single item (32 x 32) put several experts side by side; with 40 experts some workgroups get a last, partial turn.
@pytest.mark.parametrize("fmt,d,d_ff", [(0, 32, 32), (2, 32, 32), (0, 288, 544), (2, 288, 544), (0, 480, 800), (2, 480, 800),
                                        (0, 1024, 640), (2, 1024, 640), (0, 160, 1152), (2, 3072, 96), (1, 128, 128), (1, 384, 512),
                                        (1, 640, 256), (1, 768, 896), (1, 1024, 128), (1, 128, 3072)])
@pytest.mark.parametrize("T,E,k", [(1, 5, 1), (16, 40, 8)])
def test_short_reductions(fmt, d, d_ff, T, E, k):
    check(fmt, d, d_ff, T, E=E, k=k, shared=True, oai=fmt == 2, pair=d != d_ff)
