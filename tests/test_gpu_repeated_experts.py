"""Routings in which a token names an expert more than once (rows padded with zeros, ids drawn with replacement), or
none at all (ids outside [0, E)): an expert then serves more slots than the call has tokens.  Against the CPU oracle, on
a workspace of NaNs, so that a row of the expert outputs that no launch wrote shows in y."""
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


def routing(kind, T, k, E):
    """[T, k] expert ids."""
    rng = np.random.default_rng([T, k])
    if kind == "one":
        return np.full((T, k), 3, np.int32)
    if kind == "padded":  # the later half of the rows zero-filled
        idx = np.array([rng.permutation(E)[np.arange(k) % E] for _ in range(T)], np.int32)
        idx[(T + 1) // 2:] = 0
        return idx
    idx = np.asarray([1, 2, 5], np.int32)[rng.choice(3, (T, k), p=[0.1, 0.3, 0.6])]
    if kind == "outside":
        idx[rng.random((T, k)) < 0.3] = -1
        idx[rng.random((T, k)) < 0.2] = E + 40
    return idx


def check(kind, fmt, d, d_ff, T, k, shared=False, oai=False, mx=False, E=7):
    print(f"repeated experts {kind} fmt={fmt} d={d} d_ff={d_ff} T={T} k={k} E={E} shared={shared} oai={oai} mx={mx}", flush=True)
    layer = synth.layer_weights(synth.Shape("r", d, d_ff, E, k, fmt, 1, shared), seed=d + d_ff, device=DEV)
    if oai:
        layer.update(act=moe.MOE_ACT_SWIGLU_OAI, alpha=1.702, limit=7.0, b_gate=synth.expert_biases(E, d_ff, 1, "bg", DEV),
                     b_up=synth.expert_biases(E, d_ff, 1, "bu", DEV), b_down=synth.expert_biases(E, d, 1, "bd", DEV))
    if mx:
        layer["act_fmt"] = moe.MOE_ACTQ_MXFP8
    x = synth.activations(T, d, seed=T)
    idx = routing(kind, T, k, E)
    w = np.random.default_rng(T).uniform(0.1, 1.0, (T, k)).astype(np.float32)
    dl = moe.pack_layer(layer)
    ws = torch.full((moe.moe_verify_workspace_size(dl, T, k),), 0xFF, dtype=torch.uint8, device=DEV)
    r = moe.routing_for(torch.from_numpy(idx).to(DEV), torch.from_numpy(w).to(DEV), E)
    y = moe.moe_verify_layer(x.to(DEV), dl, r, workspace=ws)
    ok = (idx >= 0) & (idx < E)
    slots = np.flatnonzero(ok)
    order = slots[np.argsort(idx.reshape(-1)[slots], kind="stable")]
    counts = np.bincount(idx.reshape(-1)[slots], minlength=E)
    used = np.flatnonzero(counts)
    assert np.array_equal(r.counts.cpu().numpy(), counts)
    assert int(r.n_unique.item()) == len(used)
    assert np.array_equal(r.union_ids.cpu().numpy(), np.pad(used, (0, E - len(used)), constant_values=-1))
    first = np.concatenate([[0], np.cumsum(counts[used])])
    assert np.array_equal(r.offsets.cpu().numpy(), np.pad(first, (0, E + 1 - len(first)), constant_values=len(slots)))
    assert np.array_equal(r.perm.cpu().numpy()[:len(slots)], order)
    # The oracle takes no id outside [0, E): such a slot adds nothing, as does one of gate weight 0.
    host = {n: (v.cpu() if hasattr(v, "cpu") else v) for n, v in layer.items()}
    ref = oracle.verify_tokens(host, x, np.where(ok, idx, 0), np.where(ok, w, 0.0).astype(np.float64), threads=8)
    got = y.float().cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= YTOL * np.abs(ref).max()
    assert torch.equal(y, moe.moe_verify_layer(x.to(DEV), dl, r, workspace=ws))


KINDS = ["one", "padded", "mixed", "outside"]
LAYERS = [(0, 1120, 96, False, True), (1, 128, 256, True, False), (2, 160, 1056, False, True)]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("T,k", [(1, 7), (3, 6), (3, 7), (11, 3), (16, 1), (16, 5), (16, 7)])
@pytest.mark.parametrize("fmt,d,d_ff,shared,oai", LAYERS)
def test_small_calls(kind, T, k, fmt, d, d_ff, shared, oai):
    check(kind, fmt, d, d_ff, T, k, shared=shared, oai=oai)


@pytest.mark.parametrize("kind", KINDS)
def test_small_calls_of_1024_slots(kind):
    check(kind, 0, 64, 64, 16, 64, E=64)


# The general kernels: 17 to 64 tokens, where an expert's slots may need several token groups and nearly every item is
# cut between workgroups; MX activations and more than 64 K blocks at any T; and the token-group plan beyond 64.
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("T,k", [(17, 2), (17, 7), (32, 5), (33, 7), (48, 7), (49, 1), (64, 2), (64, 7), (70, 3)])
@pytest.mark.parametrize("fmt,d,d_ff,shared,oai", LAYERS)
def test_general_calls(kind, T, k, fmt, d, d_ff, shared, oai):
    check(kind, fmt, d, d_ff, T, k, shared=shared, oai=oai)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("T,k", [(1, 7), (3, 7), (16, 7), (33, 7), (64, 3), (70, 3)])
def test_mx_calls(kind, T, k):
    check(kind, 2, 160, 320, T, k, shared=True, mx=True)


@pytest.mark.parametrize("kind", KINDS)
def test_long_reductions(kind):
    check(kind, 0, 8224, 64, 3, 7)


@pytest.mark.parametrize("kind", KINDS)
def test_general_calls_of_4096_slots(kind):
    check(kind, 0, 64, 64, 64, 64, E=64)
