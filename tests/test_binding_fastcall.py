"""The native argument checks leave every call they do not know to the interpreter's, which say what is wrong."""
import ctypes

import pytest
import torch

from paper_2510_06175_amd import binding as vb

CFG = vb.Config(128, 8, 2, 4, 4)
HALF = dict(dtype=torch.float16)


def step_args(**change):
    a = dict(q_f16=torch.zeros(1, 8, 128, **HALF), k_new=torch.zeros(1, 2, 1, 128, **HALF), v_new=torch.zeros(1, 2, 1, 128, **HALF),
             lam=torch.ones(2, 128), cb_k=torch.zeros(2, 32, 256, 4, **HALF), cb_v=torch.zeros(2, 32, 256, 4, **HALF),
             k_idx=torch.zeros(1, 2, 64, 32, dtype=torch.uint8), v_idx=torch.zeros(1, 2, 64, 32, dtype=torch.uint8),
             workspace=torch.zeros(1 << 16, dtype=torch.uint8), out_f16=torch.zeros(1, 8, 128, **HALF))
    return {**a, **change}


def outcome(call):
    try:
        return call()
    except Exception as e:
        return type(e), str(e)


@pytest.mark.parametrize("change", [{}, {"lam": None}, {"cb_k": 7}, {"N": "x"}, {"N": 1.5}, {"num_splits": 1 << 40}, {"stream": "x"},
                                    {"q_f16": torch.zeros(8, 128, **HALF)}, {"k_idx": torch.zeros(2, 64)}],
                         ids=lambda c: "-".join(c) or "host-tensors")
def test_refusals_are_the_interpreters(change, monkeypatch):
    vb.lib()
    if vb._fast is None:
        pytest.skip("the native module is not built: nothing to compare")
    with_native = outcome(lambda: vb.vecinfer_decode_step(CFG, **step_args(**change)))
    monkeypatch.setattr(vb, "_fast", None)
    assert with_native == outcome(lambda: vb.vecinfer_decode_step(CFG, **step_args(**change)))
    assert issubclass(with_native[0], Exception)


@pytest.mark.gpu
@pytest.mark.parametrize("change", [{}, {"N": 0}, {"N": 65}, {"num_splits": 257}, {"num_splits": 1 << 32}, {"variant": 9}, {"workspace": 16},
                                    {"lam": "f16"}, {"v_new": "strided"}, {"out_f16": "cpu"}, {"k_idx": "short"}],
                         ids=lambda c: "-".join(map(str, [*c, *c.values()])) or "accepted")
def test_same_outcome_and_result_on_the_gpu(change, monkeypatch):
    """Each of these either runs or is an error of the host's own checks, the same one with and without the module."""
    def run():
        g = torch.Generator().manual_seed(1)
        t = {n: x.normal_(generator=g) if x.dtype == torch.float16 and n != "out_f16" else x for n, x in step_args().items()}
        t["lam"].fill_(1)
        t = {n: x.cuda() for n, x in t.items()}
        for n, v in change.items():
            t[n] = {"f16": lambda: t[n].half(), "strided": lambda: torch.zeros(1, 2, 1, 256, device="cuda", **HALF)[..., ::2],
                    "cpu": lambda: t[n].cpu(), "short": lambda: t[n][..., :16].contiguous(),
                    16: lambda: t[n][:16].clone()}.get(v if n not in ("N", "num_splits", "variant") else None, lambda: v)()
        r = outcome(lambda: vb.vecinfer_decode_step(CFG, **t))
        torch.cuda.synchronize()
        return r, t["out_f16"].cpu(), t["k_idx"].cpu(), t["v_idx"].cpu()

    vb.lib()
    assert vb._fast is not None
    native = run()
    monkeypatch.setattr(vb, "_fast", None)
    plain = run()
    assert native[0] == plain[0]
    assert all(torch.equal(a, b) for a, b in zip(native[1:], plain[1:]))


@pytest.mark.gpu
def test_an_interrupt_while_the_stream_is_asked_for_is_raised():
    """Ctrl-C may arrive in the Python function that finds the stream: it must end the call, not vanish in it."""
    L = vb.lib()
    names = ("encode_keys", "encode_values", "append_kv", "decode_attention", "decode_attention_residual", "decode_step")
    at = [ctypes.cast(getattr(L, "vecinfer_" + n), ctypes.c_void_p).value for n in names]

    def interrupted(stream):
        raise KeyboardInterrupt

    t = {n: x.cuda() for n, x in step_args().items()}
    vb._fast.bind(*at, interrupted)
    try:
        with pytest.raises(KeyboardInterrupt):
            vb.vecinfer_decode_step(CFG, **t)
    finally:
        vb._fast.bind(*at, vb._stream)
    vb.vecinfer_decode_step(CFG, **t)
    torch.cuda.synchronize()
