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


def _rounded_up(heads, B, N):
    """ceil(compute units / groups) splits of at least 1024 tokens each."""
    return min(-(-CUS // (B * heads[1])), -(-N // 1024))


@pytest.mark.parametrize("heads", [(32, 8), (28, 4), (8, 8), (64, 16), (4, 1)])
def test_a_workspace_has_room_for_smaller_batches(heads):
    """The automatic size never falls below that of the rounded-up count, which grows with the batch
    (to within a row of splits), and holds what a window call takes."""
    cfg = vb.Config(128, *heads, 4, 4)
    for B in (1, 2, 3, 5, 8, 12, 16, 17, 20, 24, 31, 32, 48):
        for N in (100, 1500, 8192, 32768, 196608):
            size = vb.vecinfer_decode_workspace_bytes(cfg, B, N, 0)
            assert size >= vb.vecinfer_decode_workspace_bytes(cfg, B, N, _rounded_up(heads, B, N)), (B, N)
            assert size >= vb.vecinfer_decode_workspace_bytes(cfg, B, N, vb.vecinfer_decode_auto_splits(cfg, B, N)), (B, N)
            # (and the fixed array of the static entry point holds whatever is taken)
            assert size <= vb.STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("N,splits", [(100, 4), (250, 8)])
def test_a_workspace_has_room_for_a_step_with_wide_codes(N, splits):
    """The step shares its search among splits of 32 tokens where attention and window calls take one."""
    cfg = vb.Config(128, 32, 8, 8, 8, 12, 12)
    assert vb.vecinfer_decode_auto_splits(cfg, 1, N) == splits
    assert vb.vecinfer_decode_workspace_bytes(cfg, 1, N, 0) >= vb.vecinfer_decode_workspace_bytes(cfg, 1, N, splits)


def _decode_state(cfg, B, N, seed, R=0):
    """Random codes, codebooks and query of one layer on the GPU (the values do not matter here, only
    that the calls run and agree)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    Hkv, D = cfg.num_kv_heads, cfg.head_dim

    def rn(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    def code(keys):
        return torch.randint(0, 256, (B, Hkv, N, cfg.row_bytes(keys)), generator=g, device="cuda", dtype=torch.uint8)
    return {"q": rn(B, cfg.num_q_heads, D).half(), "lam": torch.exp(0.5 * rn(Hkv, D)),
            "cb_k": rn(*cfg.cb_shape(True)).half(), "cb_v": rn(*cfg.cb_shape(False)).half(),
            "k_idx": code(True), "v_idx": code(False),
            "k": rn(B, Hkv, max(R, 1), D).half(), "v": rn(B, Hkv, max(R, 1), D).half()}


def _call(kind, cfg, s, B, N, ws, num_splits=0, seq_lens=None, variant=vb.VARIANT_AUTO):
    """(out, lse) of one decode call over the first B sequences of the state."""
    t = {k: (v if k in ("lam", "cb_k", "cb_v") else v[:B]) for k, v in s.items()}
    out = torch.empty((B, cfg.num_q_heads, cfg.head_dim), dtype=torch.float16, device="cuda")
    lse = torch.empty((B, cfg.num_q_heads), dtype=torch.float32, device="cuda")
    kw = dict(lse=lse, seq_lens=seq_lens, N=N, num_splits=num_splits, variant=variant)
    head = (cfg, t["q"], t["lam"], t["cb_k"], t["cb_v"], t["k_idx"], t["v_idx"])
    if kind == "attention":
        vb.vecinfer_decode_attention(*head, ws, out, **kw)
    elif kind == "window":
        vb.vecinfer_decode_attention_residual(*head, t["k"], t["v"], ws, out, **kw)
    else:
        new = (t[n][:, :, :1].contiguous() for n in ("k", "v"))
        vb.vecinfer_decode_step(cfg, t["q"], *new, *head[2:], ws, out, **kw)
    return out, lse


@pytest.mark.gpu
@pytest.mark.parametrize("most", [5, 17, 24])
def test_one_workspace_serves_every_smaller_batch(most):
    cfg, N = vb.Config(128, 32, 8, 4, 4), 8192
    s = _decode_state(cfg, most, N, most)
    ws = vb.new_workspace(cfg, most, N)
    for B in range(1, most + 1):
        out, lse = _call("attention", cfg, s, B, N, ws)
        own, own_lse = _call("attention", cfg, s, B, N, vb.new_workspace(cfg, B, N))
        # another number of splits at most: fp16 outputs and softmax weights, fp32 sums
        assert (out - own).abs().max() <= 2e-3 * own.abs().max(), B
        assert (lse - own_lse).abs().max() <= 1e-3, B


@pytest.mark.gpu
def test_window_call_in_a_workspace_of_the_reported_splits():
    cfg, B, N = vb.Config(128, 8, 8, 4, 4), 16, 1500
    s = _decode_state(cfg, B, N, 3, R=40)
    few = vb.new_workspace(cfg, B, N, vb.vecinfer_decode_auto_splits(cfg, B, N))
    out, lse = _call("window", cfg, s, B, N, few)
    own, own_lse = _call("window", cfg, s, B, N, vb.new_workspace(cfg, B, N))
    assert (out - own).abs().max() <= 2e-3 * own.abs().max()
    assert (lse - own_lse).abs().max() <= 1e-3
    with pytest.raises(vb.VecInferError):                  # not even one split
        _call("window", cfg, s, B, N, vb.new_workspace(cfg, B, N, 1)[:-256])


# (call, Config arguments, B, N, ragged, variant) -> the splits that num_splits = 0 takes, and another
# count whose result differs in some last bits (up to 512 tokens none does: a wavefront's tile each)
CHOICES = [
    # the lookup-table kernel: the larger of both rules
    ("attention", (64, 4, 2, 4, 4), 90, 4000, 0, vb.VARIANT_LUT, 2, 1),
    ("step", (128, 4, 2, 4, 4), 48, 2500, 0, vb.VARIANT_LUT, 3, 2),
    ("attention", (128, 4, 1, 4, 4), 3, 1000, 0, vb.VARIANT_LUT, 16, 1),
    # few KV heads: no more splits than the length pays for
    ("attention", (128, 4, 1, 4, 4), 1, 57343, 0, 0, 32, 64),
    ("attention", (128, 4, 1, 2, 2), 1, 49151, 0, 0, 32, 64),
    ("step", (128, 4, 1, 2, 2), 1, 49152, 0, 0, 64, 32),
    ("window", (128, 8, 1, 2, 2), 1, 57343, 0, 0, 32, 64),
    ("step", (128, 8, 1, 8, 8, 12, 12), 1, 57344, 0, 0, 64, 256),
    ("attention", (128, 1, 1, 4, 4), 1, 196607, 0, 0, 64, 256),
    ("attention", (128, 1, 1, 2, 2), 1, 131072, 0, 0, 128, 64),
    ("step", (128, 4, 2, 4, 4), 1, 196608, 0, 0, 128, 64),
    ("step", (128, 4, 1, 4, 4), 1, 524287, 0, 0, 128, 256),
    ("step", (128, 4, 1, 4, 4), 1, 524288, 0, 0, 256, 128),
    # attention alone: short sequences whole
    ("attention", (128, 4, 1, 4, 4), 8, 1000, 0, 0, 1, 16),
    ("attention", (64, 8, 1, 8, 8), 1, 1024, 0, 0, 1, 16),
    ("attention", (128, 8, 1, 8, 8, 12, 12), 2, 900, 0, 0, 1, 29),
    ("attention", (128, 4, 1, 4, 4), 8, 1025, 0, 0, 17, 1),
    ("attention", (128, 4, 1, 4, 4), 100, 2047, 0, 0, 1, 2),
    ("attention", (128, 4, 1, 4, 4), 100, 2048, 0, 0, 2, 1),
    ("attention", (128, 4, 1, 2, 2), 100, 1792, 0, 0, 2, 1),
    ("attention", (128, 4, 1, 2, 4), 8, 768, 0, 0, 1, 12),
    ("attention", (128, 4, 1, 2, 4), 8, 769, 0, 0, 13, 1),
    ("attention", (128, 4, 1, 2, 4), 80, 1024, 0, 0, 1, 3),
    # the step: whole where the search for the new token is not worth a merge
    ("step", (128, 4, 1, 4, 4), 8, 1000, 0, 0, 16, 1),
    ("step", (128, 8, 1, 4, 4), 8, 704, 0, 0, 1, 11),
    ("step", (128, 8, 1, 4, 4), 8, 705, 0, 0, 12, 1),
    ("step", (128, 8, 1, 2, 2), 8, 600, 0, 0, 10, 1),
    ("step", (128, 8, 1, 4, 4), 64, 1024, 0, 0, 1, 4),
    ("step", (128, 8, 1, 8, 8), 64, 705, 0, 0, 4, 1),
    ("step", (128, 4, 1, 4, 4), 85, 1024, 0, 0, 1, 3),
    ("step", (128, 4, 1, 2, 2), 85, 768, 0, 0, 3, 1),
    ("step", (128, 4, 1, 4, 4), 128, 2047, 0, 0, 1, 2),
    ("step", (128, 8, 1, 2, 4), 128, 2047, 0, 0, 1, 2),
    ("step", (128, 4, 1, 8, 8), 128, 1025, 0, 0, 2, 1),
    ("step", (128, 4, 1, 8, 8, 12, 12), 128, 700, 0, 0, 2, 1),
    ("step", (64, 4, 1, 4, 4), 8, 704, 0, 0, 1, 11),
    ("step", (64, 4, 1, 2, 2), 8, 600, 0, 0, 10, 1),
    ("step", (64, 4, 1, 2, 8), 8, 705, 0, 0, 12, 1),
    ("step", (64, 4, 1, 8, 8), 8, 1024, 0, 0, 1, 16),
    ("step", (64, 4, 1, 4, 8), 8, 1025, 0, 0, 17, 1),
    ("step", (64, 4, 1, 2, 2), 85, 1024, 0, 0, 1, 3),
    # sequences of different lengths: one more split where they are long
    ("step", (128, 4, 1, 4, 4), 136, 4096, 1, 0, 2, 1),
    ("attention", (128, 4, 1, 4, 4), 136, 4095, 1, 0, 1, 2),
    ("window", (128, 4, 1, 4, 4), 100, 8192, 1, 0, 3, 2),
    ("attention", (128, 16, 8, 8, 8), 5, 49152, 1, 0, 7, 6),
    ("attention", (128, 16, 8, 8, 8), 5, 49152, 0, 0, 6, 7),
    ("attention", (128, 16, 8, 8, 8), 5, 49151, 1, 0, 6, 7),
    ("attention", (128, 16, 8, 2, 2), 5, 24576, 1, 0, 7, 6),
    ("step", (128, 16, 8, 8, 8), 3, 50000, 1, 0, 10, 11),
    ("window", (128, 4, 1, 4, 4), 8, 1000, 0, 0, 16, 1),
]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,args,B,N,ragged,variant,want,other", CHOICES)
def test_automatic_choice(kind, args, B, N, ragged, variant, want, other):
    """The automatic call is bit for bit the call with the expected number of splits (and the number
    shows in the bits)."""
    cfg = vb.Config(*args)
    s = _decode_state(cfg, B, N, N + B, R=33)
    lens = torch.linspace(N // 8, N, B, device="cuda").to(torch.int32) if ragged else None
    run = lambda S: _call(kind, cfg, s, B, N, vb.new_workspace(cfg, B, N, S), S, lens, variant)  # noqa: E731
    (out, lse), (w_out, w_lse), (o_out, o_lse) = run(0), run(want), run(other)
    assert torch.equal(out, w_out) and torch.equal(lse, w_lse)
    assert not (torch.equal(out, o_out) and torch.equal(lse, o_lse))
