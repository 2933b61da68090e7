"""The merge of the splits inside the attention launch: numbers of splits at the edges of its batches and of a
wavefront, workspaces full of anything, replays of a captured launch."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_decode_close, cfg_of, dev, gpu_decode, oracle_view
from paper_2510_06175_amd import binding as vb
from paper_2510_06175_amd import synth

pytestmark = pytest.mark.gpu

# D, (Hq, Hkv), d: one and two output elements per thread, one query head, a spare head slot
SHAPES = [(128, (8, 2), 4), (128, (16, 2), 8), (128, (2, 2), 2), (64, (14, 2), 4)]


@pytest.mark.parametrize("splits", [2, 8, 9, 32, 33, 64, 65, 129, 256])
@pytest.mark.parametrize("D,heads,d", SHAPES)
def test_every_batch_of_splits(D, heads, d, splits):
    # (1000 tokens: at 33 splits and more the last ones are empty)
    shape = synth.Shape(2, *heads, D, 1000, d, d)
    x = synth.decode_inputs(shape, seed=splits + D)
    lens = np.array([1000, 77])
    junk = torch.randint(0, 256, (vb.vecinfer_decode_workspace_bytes(cfg_of(shape), 2, 1000, splits),),
                         dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(splits))
    y = oracle_view(shape, x)
    ref = oracle.decode_attention(y["q"], y["lam"], y["cb_k"], y["cb_v"], y["k_idx"], y["v_idx"], lens)
    first = gpu_decode(shape, x, seq_lens=lens, num_splits=splits, ws=junk)
    assert_decode_close(*first, *ref, what=f"{splits} splits")
    # the same numbers whichever workgroup came last, and whatever the workspace held
    for ws in (junk, torch.zeros_like(junk), torch.full_like(junk, 255)):
        again = gpu_decode(shape, x, seq_lens=lens, num_splits=splits, ws=ws)
        np.testing.assert_array_equal(again[0], first[0])
        np.testing.assert_array_equal(again[1], first[1])


def test_one_workspace_for_changing_inputs():
    """Partials of the call before must never be taken for this call's: new queries on the same workspace, with
    nothing between the calls, against calls on workspaces of their own."""
    shape = synth.Shape(3, 32, 8, 128, 3000, 4, 4)
    cfg = cfg_of(shape)
    x = synth.decode_inputs(shape, seed=5)
    t = {k: dev(v) for k, v in x.items()}
    g = torch.Generator("cuda").manual_seed(6)
    qs = torch.randn((40, shape.B, shape.Hq, shape.D), generator=g, device="cuda").half()

    def call(q, ws):
        out = torch.empty_like(q)
        vb.vecinfer_decode_attention(cfg, q, t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"], ws, out, num_splits=10)
        return out

    ws = vb.new_workspace(cfg, shape.B, shape.N, 10)
    shared = [call(q, ws) for q in qs]
    own = [call(q, vb.new_workspace(cfg, shape.B, shape.N, 10)) for q in qs]
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(shared, own))


def test_replays_without_anything_between():
    shape = synth.Shape(1, 32, 8, 128, 5000, 4, 4)
    cfg = cfg_of(shape)
    x = synth.decode_inputs(shape, seed=8)
    t = {k: dev(v) for k, v in x.items()}
    ws = vb.new_workspace(cfg, 1, shape.N)
    q, out = t["q"].clone(), torch.empty_like(t["q"])
    call = lambda: vb.vecinfer_decode_attention(cfg, q, t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"], ws, out)  # noqa: E731
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    g = torch.Generator("cuda").manual_seed(9)
    for _ in range(4):
        new = torch.randn(q.shape, generator=g, device="cuda").half()
        q.copy_(new)
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        out.zero_()
        call()
        torch.cuda.synchronize()
        assert torch.equal(got, out)


def test_every_split_is_weighed_against_the_same_maximum():
    """A new token whose score is the largest, at a size (about 2^18) where the order in which its shares are added
    shows: 32 splits of equal tokens, each with a value channel of its own, must come out with equal weights."""
    D, d, S = 128, 4, 32
    N = 64 * S + 1
    cfg, g = vb.Config(D, 1, 1, d, d), synth.rng(3)
    H = oracle.hadamard(D)                                                 # orthonormal
    row = g.uniform(15, 30, D).astype(np.float16)                          # the key of every token ..
    x = g.uniform(50, 120, D)
    x[0] = 1.0                                                             # .. but for channel 0, where the query is small
    cb_k = np.zeros((1, D // d, 256, d), np.float16)
    cb_k[0, :, 1] = cb_k[0, :, 2] = row.reshape(D // d, d)
    cb_k[0, 0, 2, 0] -= 1                                                  # the older tokens score one unit (log2) less
    cb_v = np.zeros((1, D // d, 256, d), np.float16)
    cb_v[0, :, 1:1 + d] = 8 * np.eye(d)
    q = (x * (D / np.log2(np.e)) @ H / np.sqrt(D)).astype(np.float16)      # (q H sqrt(D)) log2(e) / D = x
    k_new = (row.astype(np.float64) @ H).astype(np.float16)
    k_idx = np.ones((1, 1, N, D // d), np.uint8)
    k_idx[:, :, :, 0] = 2
    v_idx = np.zeros_like(k_idx)
    for s in range(S):
        v_idx[0, 0, 64 * s:64 * s + 64, s // d] = 1 + s % d
    t = {n: dev(a) for n, a in dict(q=q[None, None], k=k_new[None, None, None], v=np.zeros((1, 1, 1, D), np.float16),
                                    lam=np.ones((1, D), np.float32), cb_k=cb_k, cb_v=cb_v, k_idx=k_idx, v_idx=v_idx).items()}
    out, lse = torch.zeros((1, 1, D), dtype=torch.float16, device="cuda"), torch.zeros((1, 1), device="cuda")
    vb.vecinfer_decode_step(cfg, t["q"], t["k"], t["v"], t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"],
                            vb.new_workspace(cfg, 1, N, S), out, lse=lse, num_splits=S)
    torch.cuda.synchronize()
    assert (t["k_idx"][0, 0, -1] == 1).all()                               # the new token is what it was made to be
    assert lse.item() * np.log2(np.e) > 1 << 17
    got = out[0, 0, :S].cpu().numpy()
    assert 0.2 < got[0] < 0.26                                             # 8 / 32, less the new token's share
    np.testing.assert_array_equal(got, got[0])
