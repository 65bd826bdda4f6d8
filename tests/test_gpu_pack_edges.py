"""Weight packing at the edges of the kernel's runs along K (runs of 4 blocks, 32 blocks a turn of the workgroup) and of
the last block, and on both sides of its three splits (few tiles, small tiles, a workgroup a tile), for the three layouts, against the numpy statement of the format in the parity tests; a guard behind
every output stays untouched."""
import numpy as np
import pytest
import torch

import paper_2607_12696_amd as moe
import synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from test_gpu_parity import _expected_packed, _expected_pair

DEV = torch.device("cuda:0")


def weights(fmt, E, N, K, seed):
    if fmt == 0:
        return synth.weights_bf16(E, N, K, seed), None
    return (synth.weights_fp8_b128 if fmt == 1 else synth.weights_mxfp4)(E, N, K, seed)


@pytest.mark.parametrize("fmt,N,K", [(0, 16, 32), (0, 32, 4096), (0, 32, 4128), (0, 16, 8256), (1, 128, 4224), (1, 256, 640),
                                     (2, 32, 4096), (2, 16, 4640), (2, 32, 8224), (2, 16, 32)])
def test_layouts(fmt, N, K):
    E = 2
    w, s = weights(fmt, E, N, K, 3)
    w2, s2 = weights(fmt, E, N, K, 4)
    wd, sd = w.to(DEV), None if s is None else s.to(DEV)
    ew, es = _expected_packed(fmt, w, s)
    wb, sb = moe.moe_packed_size(fmt, E, N, K)
    guard = torch.full((wb + sb + 8192,), 0xA5, dtype=torch.uint8, device=DEV)
    sp = guard[wb + 4096:wb + 4096 + sb] if sb else None
    moe.lib().moe_pack_weights(fmt, E, N, K, wd.data_ptr(), 0 if sd is None else sd.data_ptr(), guard.data_ptr(),
                               0 if sp is None else sp.data_ptr(), torch.cuda.current_stream().cuda_stream)
    out = guard.cpu().numpy()
    assert np.array_equal(out[:wb], ew) and (out[wb:wb + 4096] == 0xA5).all() and (out[wb + 4096 + sb:] == 0xA5).all()
    if sb:
        assert np.array_equal(out[wb + 4096:wb + 4096 + sb], es)
    wp, sgp, sup = moe.moe_pack_gate_up(fmt, wd, w2.to(DEV), sd, None if s2 is None else s2.to(DEV))
    assert np.array_equal(wp.cpu().numpy(), _expected_pair(fmt, w, s, w2, s2))
    if sb:
        assert np.array_equal(sgp.cpu().numpy(), es)
        assert np.array_equal(sup.cpu().numpy(), _expected_packed(fmt, w2, s2)[1])
    if N % 32 == 0:
        B = {0: 4096, 1: 2048, 2: 1024}[fmt]
        tiles = ew.reshape(E, N // 32, 2, -1, B).transpose(0, 1, 3, 2, 4)
        dp, dsp = moe.moe_pack_down(fmt, wd, sd)
        assert np.array_equal(dp.cpu().numpy(), np.ascontiguousarray(tiles).reshape(-1))
        if sb:
            assert np.array_equal(dsp.cpu().numpy(), es)


# More than 256 row tiles: a wavefront a tile up to 4 KiB of source (also with tiles left over from the last workgroup's
# eight), beyond that a workgroup a tile, with one run, several, and more than a turn of them.
@pytest.mark.parametrize("fmt,N,K", [(0, 2064, 32), (0, 2080, 64), (0, 2064, 128), (0, 2080, 160), (0, 2064, 4224), (1, 2176, 128),
                                     (1, 2176, 256), (1, 2176, 384), (1, 2176, 4224), (2, 2080, 32), (2, 2064, 256), (2, 2080, 544),
                                     (2, 2080, 4640)])
def test_layouts_of_many_tiles(fmt, N, K):
    test_layouts(fmt, N, K)
