"""The automatic number of splits: fills the compute units once, grows with the sequence, and gives
way to a smaller workspace."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2510_06175_amd import binding as vb
from paper_2510_06175_amd import synth

CUS = 256


@pytest.mark.parametrize("heads,wide", itertools.product([(32, 8), (28, 4), (8, 8), (64, 16)], [0, 1]))
def test_auto_splits_rule(heads, wide):
    cfg = vb.Config(128, *heads, 8, 8, 12, 12) if wide else vb.Config(128, *heads, 4, 4)
    for B in (1, 2, 3, 5, 8, 16, 24, 31, 32, 48):
        last = 0
        for N in (1, 33, 64, 191, 300, 767, 768, 1000, 2000, 3071, 3072, 8000, 30001, 196608):
            s = vb.vecinfer_decode_auto_splits(cfg, B, N)
            assert s >= last, (B, N)                       # a workspace for N tokens serves every shorter call
            last = s
            assert s == 1 or B * heads[1] * s <= CUS, (B, N)
            assert s == 1 or (s - 1) * (32 if wide else 64) < N, (B, N)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [300, 1000, 3073, 5000])
def test_smaller_workspace_takes_fewer_splits(N):
    shape = synth.Shape(B=1, Hq=8, Hkv=2, D=128, N=N, d_k=4, d_v=4)
    cfg = vb.Config(shape.D, shape.Hq, shape.Hkv, shape.d_k, shape.d_v)
    case = synth.decode_inputs(shape, seed=N)
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in case.items() if isinstance(v, np.ndarray)}
    auto = vb.vecinfer_decode_auto_splits(cfg, 1, N)
    few = max(1, -(-N // 1024))
    assert few < auto
    outs = []
    for ws_splits in (auto, few):
        ws = vb.new_workspace(cfg, 1, N, ws_splits)
        out = torch.empty((1, shape.Hq, shape.D), dtype=torch.float16, device="cuda")
        lse = torch.empty((1, shape.Hq), dtype=torch.float32, device="cuda")
        vb.vecinfer_decode_attention(cfg, t["q"], t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"], ws, out, lse=lse, N=N)
        outs.append((out.float().cpu().numpy(), lse.cpu().numpy()))
    ref_o, ref_l = oracle.decode_attention(case["q"], case["lam"], case["cb_k"], case["cb_v"], case["k_idx"], case["v_idx"])
    for o, l in outs:
        # fp16 softmax weights and outputs: 2^-11 relative each
        assert np.abs(o - ref_o).max() <= 2e-3 * np.abs(ref_o).max()
        assert np.abs(l - ref_l).max() <= 1e-3
    with pytest.raises(vb.VecInferError):
        vb.vecinfer_decode_attention(cfg, t["q"], t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"], ws[:256], out, N=N)
