"""The per-token encode kernel against the tile kernel on the same rows: ties, rows of the fp16 range's
edge and non-finite rows, every head dim and sub-vector dim, codes in rows and in tiles."""
import pytest
import torch

from paper_2510_06175_amd import binding as vb


@pytest.mark.gpu
@pytest.mark.parametrize("D,d,tiled", [(128, 2, 0), (128, 2, 1), (128, 4, 0), (128, 4, 1), (128, 8, 0), (128, 8, 1),
                                       (64, 2, 0), (64, 4, 1), (64, 8, 0)])
def test_token_kernel_writes_the_tile_kernel_s_codes(D, d, tiled):
    B, Hkv, T, cap = 2, 3, 64, 64
    cfg = vb.Config(D, 6, Hkv, d, d, 8, 8, tiled)
    g = torch.Generator(device="cuda").manual_seed(D + d)
    cb = torch.randn(cfg.cb_shape(True), generator=g, device="cuda").half()
    cb[:, :, 200:] = cb[:, :, 3:59]                        # duplicates: the lower index wins
    x = torch.randn((B, Hkv, T, D), generator=g, device="cuda").half()
    x[:, :, 5] = cb[:, :, 220].reshape(Hkv, D)             # exact hits of a duplicated centroid
    x[:, :, 9] = 60000.0
    x[:, :, 17] = float("nan")                             # (a row without any finite distance: code 0)
    lam = torch.exp(0.3 * torch.randn((Hkv, D), generator=g, device="cuda"))
    for keys in (True, False):
        rows = cfg.row_bytes(keys)
        tile, token, both = (torch.zeros((B, Hkv, cap, rows), dtype=torch.uint8, device="cuda") for _ in range(3))
        other = torch.zeros_like(both)
        if keys:
            vb.vecinfer_encode_keys(cfg, x, lam, cb, tile)
        else:
            vb.vecinfer_encode_values(cfg, x, cb, tile)
        for t0, n in ((0, 1), (1, 16), (17, 16), (33, 15), (48, 16)):
            part = x[:, :, t0:t0 + n].contiguous()
            if keys:
                vb.vecinfer_encode_keys(cfg, part, lam, cb, token, pos0=t0)
                vb.vecinfer_append_kv(cfg, part, part, lam, cb, cb, both, other, pos0=t0)
            else:
                vb.vecinfer_encode_values(cfg, part, cb, token, pos0=t0)
                vb.vecinfer_append_kv(cfg, part, part, lam, cb, cb, other, both, pos0=t0)
        assert torch.equal(tile, token)
        assert torch.equal(tile, both)
        if not keys and not tiled:
            want = torch.arange(20 + 3, 20 + 4, device="cuda", dtype=torch.uint8)   # 220 repeats 23
            assert torch.equal(tile[:, :, 5], want.expand(B, Hkv, rows))
