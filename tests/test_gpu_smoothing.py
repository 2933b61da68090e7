"""x / lambda of the tile kernels from the reciprocal, and where that is not exact by division: codes against the
per-token kernel, which divides."""
import numpy as np
import pytest
import torch

from helpers import cfg_of, dev
from paper_2510_06175_amd import binding as vb
from paper_2510_06175_amd import synth

pytestmark = pytest.mark.gpu


def _lambda(kind, g, Hkv, D):
    lam = np.exp(g.normal(size=(Hkv, D)) * 2).astype(np.float32)
    if kind == "all-ones":                 # mantissas next to and of all ones
        lam.view(np.uint32)[0, 5] |= 0x7fffff
        lam.view(np.uint32)[:, 9] = (lam.view(np.uint32)[:, 9] & 0xff800000) | 0x7ffffe
    elif kind == "tiny":
        lam[0, 3] = 1e-30
    elif kind == "huge":
        lam[:, 7] = 1e25
    elif kind == "powers":
        lam = np.exp2(np.round(g.normal(size=(Hkv, D)) * 20)).astype(np.float32)
    return lam


@pytest.mark.parametrize("kind", ["usual", "all-ones", "tiny", "huge", "powers"])
@pytest.mark.parametrize("D,d,bits", [(128, 2, 8), (128, 4, 8), (128, 8, 8), (64, 2, 8), (64, 4, 8), (64, 8, 8), (128, 8, 12),
                                      (128, 4, 10), (64, 8, 12)])
def test_smoothed_keys(D, d, bits, kind):
    T, shape = 200, synth.Shape(1, 4, 2, D, 200, d, d, bits, bits)
    cfg, g = cfg_of(shape), synth.rng(D + d + bits)
    lam = _lambda(kind, g, shape.Hkv, D)
    k = (g.normal(size=(1, shape.Hkv, T, D)) * np.exp(g.normal(size=(1, shape.Hkv, T, 1)))).astype(np.float16)
    k[0, 0, 3] = 0
    k[0, 1, 4, 11] = 6e-8                   # the smallest fp16
    k[0, 0, 5, 2] = np.inf
    k[0, 1, 6, 1] = np.nan
    k[0, 0, 7] = 65504
    cb = dev(g.normal(size=cfg.cb_shape(True)).astype(np.float16))
    kt, lt = dev(k), dev(lam)
    tile = torch.zeros((1, shape.Hkv, T, cfg.row_bytes(True)), dtype=torch.uint8, device="cuda")
    token = torch.zeros_like(tile)
    vb.vecinfer_encode_keys(cfg, kt, lt, cb, tile)
    for t in range(0, T, 8):
        vb.vecinfer_encode_keys(cfg, kt[:, :, t:t + 8].contiguous(), lt, cb, token, pos0=t)
    torch.cuda.synchronize()
    assert torch.equal(tile, token)
