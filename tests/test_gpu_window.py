"""The residual window inside the attention launch: how its rows are dealt to workgroups and wavefronts, rows behind a
sequence's own window, sequences with nothing quantized."""
import numpy as np
import pytest

import oracle
from helpers import assert_decode_close, gpu_decode_residual, oracle_view, tile_value_codes
from paper_2510_06175_amd import synth

pytestmark = pytest.mark.gpu

# D, (Hq, Hkv), d_k, d_v: every form of the accumulators (d_v = 2, 4, 8, split sub-spaces), both numbers of head groups
SHAPES = [(128, (8, 2), 4, 4), (128, (2, 1), 4, 2), (128, (16, 2), 8, 8), (128, (7, 1), 2, 4), (64, (8, 2), 4, 4),
          (64, (16, 2), 2, 2), (64, (3, 1), 8, 8)]


@pytest.mark.parametrize("splits", [1, 2, 7, 8, 33])
@pytest.mark.parametrize("D,heads,dk,dv", SHAPES)
def test_window_rows(D, heads, dk, dv, splits):
    shape = synth.Shape(6, *heads, D, 700, dk, dv)
    x = synth.decode_inputs(shape, seed=splits + D + dv)
    x.update(synth.residual_window(shape, splits + 50, 128))
    # a full window, edges of a wavefront's 16 rows, none; with a full cache, one token, none
    seq_lens, res_lens = np.array([700, 1, 0, 700, 0, 333]), np.array([128, 127, 17, 0, 1, 16])
    ox = oracle_view(shape, x)
    ref = oracle.decode_attention_residual(ox["q"], ox["lam"], ox["cb_k"], ox["cb_v"], ox["k_idx"], ox["v_idx"],
                                           x["k_res"], x["v_res"], seq_lens, res_lens)
    # rows behind a sequence's own window may hold anything
    g = {k: v.copy() for k, v in x.items() if isinstance(v, np.ndarray)}
    for b, r in enumerate(res_lens):
        g["k_res"][b, :, r:] = np.nan
        g["v_res"][b, :, r:] = np.inf
    got = gpu_decode_residual(shape, g, seq_lens=seq_lens, res_lens=res_lens, num_splits=splits)
    assert_decode_close(*got, *ref, what=f"{splits} splits")


def _dominating(shape, ahead, rows, seed):
    """Inputs whose window outweighs all quantized tokens together by 2^ahead and has values of zero, so that the
    output is nothing but the quantized tokens' small weights times their (positive) values."""
    x = synth.decode_inputs(shape, seed=seed)
    x["q"] = np.repeat(x["q"][:, ::shape.G], shape.G, axis=1)              # one query per KV head: one window key fits all
    x["cb_v"] = np.abs(x["cb_v"]) * np.float16(8000)
    ox = oracle_view(shape, x)
    _, lse = oracle.decode_attention(ox["q"], ox["lam"], ox["cb_k"], ox["cb_v"], ox["k_idx"], ox["v_idx"])
    score = lse + ahead * np.log(2) - np.log(rows)                         # natural units, each window row
    q = x["q"].astype(np.float64)
    k = q * (score * np.sqrt(shape.D) / (q * q).sum(-1))[..., None]
    x["k_res"] = np.repeat(k[:, ::shape.G, None].astype(np.float16), rows, axis=2)
    x["v_res"] = np.zeros_like(x["k_res"])
    return x


@pytest.mark.parametrize("splits", [1, 2, 8, 33])
@pytest.mark.parametrize("D,heads,dk,dv,bits", [(128, (8, 2), 4, 4, 8), (128, (16, 2), 2, 2, 8), (128, (16, 2), 2, 8, 8),
                                                (64, (8, 2), 4, 4, 8), (64, (16, 2), 8, 8, 8), (128, (8, 2), 8, 8, 12)])
def test_a_dominating_window_leaves_the_tokens_their_weights(D, heads, dk, dv, bits, splits):
    """The quantized tokens' weights are fp16 numbers relative to a maximum.  That must be the tokens' own, not the
    window's: 4000 tokens behind a window ahead by 2^24 weigh about 2^-29 of one of its 128 rows each, which fp16
    rounds to zero.
    Tolerance: weights and outputs are fp16 roundings, 2^-11 each, of positive terms."""
    shape = synth.Shape(1, *heads, D, 4000, dk, dv, bits, bits)
    x = _dominating(shape, 24, 128, seed=D + dk + dv)
    ox = oracle_view(shape, x)
    ref, lse = oracle.decode_attention_residual(ox["q"], ox["lam"], ox["cb_k"], ox["cb_v"], ox["k_idx"], ox["v_idx"],
                                                x["k_res"], x["v_res"])
    assert np.abs(ref).min() > 2 ** -13                                    # well inside fp16's normal numbers
    out, got_lse = gpu_decode_residual(shape, x, num_splits=splits)
    assert np.abs(out / ref - 1).max() <= 2 ** -10
    assert np.abs(got_lse - lse).max() <= 1e-4


@pytest.mark.parametrize("splits", [1, 7])
@pytest.mark.parametrize("heads", [(8, 2), (14, 2)])
@pytest.mark.parametrize("D,dk,dv", [(D, dk, dv) for D in (128, 64) for dk in (2, 4, 8) for dv in (2, 4, 8) if D // dv >= 16])
def test_window_with_tiled_value_codes(D, dk, dv, heads, splits):
    """Tiles instead of rows of value codes: the same numbers, bit for bit."""
    shape = synth.Shape(3, *heads, D, 640, dk, dv)
    x = synth.decode_inputs(shape, seed=D + 8 * dk + dv)
    x.update(synth.residual_window(shape, 7, 128))
    lens = dict(seq_lens=np.array([640, 0, 577]), res_lens=np.array([100, 33, 128]), num_splits=splits)
    rows = gpu_decode_residual(shape, x, **lens)
    tiled = gpu_decode_residual(shape, {**x, "v_idx": tile_value_codes(x["v_idx"])}, v_tiled=1, **lens)
    for a, b in zip(rows, tiled):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("splits", [1, 7])
@pytest.mark.parametrize("heads", [(8, 2), (16, 2)])
@pytest.mark.parametrize("D,dk,bk,dv,bv", [
    (D, dk, bk, dv, bv) for D in (128, 64) for dk in (4, 8) for dv in (4, 8) for bk in (8, 10, 12) for bv in (8, 10, 12)
    if (bk, bv) != (8, 8) and (bk == 8 or D // dk * bk % 32 == 0) and (bv == 8 or D // dv * bv % 32 == 0)])
def test_window_with_wide_codes(D, dk, bk, dv, bv, heads, splits):
    shape = synth.Shape(2, *heads, D, 300, dk, dv, bk, bv)
    x = synth.decode_inputs(shape, seed=D + dk + dv + bk + bv)
    x.update(synth.residual_window(shape, 9, 128))
    seq_lens, res_lens = np.array([300, 65]), np.array([128, 19])
    ox = oracle_view(shape, x)
    ref = oracle.decode_attention_residual(ox["q"], ox["lam"], ox["cb_k"], ox["cb_v"], ox["k_idx"], ox["v_idx"],
                                           x["k_res"], x["v_res"], seq_lens, res_lens)
    got = gpu_decode_residual(shape, x, seq_lens=seq_lens, res_lens=res_lens, num_splits=splits)
    assert_decode_close(*got, *ref, what=f"{splits} splits")
