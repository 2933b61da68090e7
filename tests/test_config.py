"""What a Config keeps for its calls: worked out on first use, without a lock, each value by itself."""
import copy
import dataclasses
import functools
import pickle

import pytest

from paper_2510_06175_amd import binding as vb


def test_values_for_the_calls():
    cfg = vb.Config(128, 32, 8, 4, 8, 8, 12)
    assert not any(isinstance(v, functools.cached_property) for v in vars(vb.Config).values())
    assert set(vars(cfg)) == {f.name for f in dataclasses.fields(cfg)}
    want = {"_lam_shape": (8, 128), "_cb_k": cfg.cb_shape(True), "_cb_v": cfg.cb_shape(False),
            "_row_k": cfg.row_bytes(True), "_row_v": cfg.row_bytes(False)}
    for name, value in want.items():
        assert getattr(cfg, name) == value and vars(cfg)[name] is getattr(cfg, name)
    assert cfg._c is cfg._c and (cfg._c.head_dim, cfg._c.v_bits, cfg._c.v_tiled) == (128, 12, 0)
    for other in (pickle.loads(pickle.dumps(cfg)), copy.deepcopy(cfg), dataclasses.replace(cfg)):
        assert other == cfg and hash(other) == hash(cfg) and "_c" not in vars(other)
    assert dataclasses.replace(cfg, v_bits=8, v_tiled=1)._c.v_tiled == 1


def test_a_side_that_no_call_asks_for_is_not_worked_out():
    cfg = vb.Config(128, 32, 8, 4, 0)
    assert cfg._cb_k == (8, 32, 256, 4) and cfg._row_k == 32
    assert vb.vecinfer_decode_workspace_bytes(cfg, 1, 64) == 0
    with pytest.raises(ZeroDivisionError):
        cfg._cb_v
