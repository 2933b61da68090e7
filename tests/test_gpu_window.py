"""The residual window inside the attention launch: how its rows are dealt to workgroups and wavefronts, rows behind a
sequence's own window, sequences with nothing quantized."""
import numpy as np
import pytest

import oracle
from helpers import assert_decode_close, gpu_decode_residual, oracle_view
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
