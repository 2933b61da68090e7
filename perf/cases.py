"""The work a user of this library has it do, as timed cases: decode steps over a quantized cache, the
decode-time append, the cache fill of a prefill, and the training of the codebooks.

    listed()            named cases over the range of sizes, code widths and layouts in use
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call, on the GPU
    run(state)          one pass through the public entry points, and its outputs
    work(case)          bytes and operations of one pass that nothing can save
    tolerance(case)     how far two correct implementations may lie apart

Kinds of case (`kind`):
    step    vecinfer_decode_step: append the new token, attend to the cache (one layer, one token)
    window  vecinfer_decode_attention_residual: attend to the cache and a full-precision window
    append  vecinfer_append_kv: T tokens per sequence into the cache, no attention
    fill    vecinfer_encode_keys + vecinfer_encode_values: T tokens per sequence from row pos0
    train   vecinfer_calibrate_lambda + vecinfer_kmeans_train: smoothing factors and key codebooks
"""
from __future__ import annotations

import math

import torch

from paper_2510_06175_amd import binding as vb

# (d_k, d_v, b_k, b_v) by name; "b2d4" is two bits per element, d = 4 with 8-bit codes
CODES = {
    "b2d4": (4, 4, 8, 8),
    "b4d2": (2, 2, 8, 8),
    "k4v2": (2, 4, 8, 8),           # more bits for the keys
    "d8b8": (8, 8, 8, 8),           # one bit per element
    "d8b12": (8, 8, 12, 12),        # one table of 4096 centroids per KV head
    "d4b12": (4, 4, 12, 12),
    "kd4b10-vd8b12": (4, 8, 10, 12),
    "kd8b12-vd8b8": (8, 8, 12, 8),
}


def _case(kind, code, B, Hq, Hkv, D, N, **more):
    return dict({"kind": kind, "code": code, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "N": N}, **more)


def listed():
    c = lambda name, *a, **k: dict(_case(*a, **k), name=name)  # noqa: E731
    return [
        # a chat turn's first tokens: one sequence, a short cache; latency and launches are what it costs
        c("step-1000", "step", "b2d4", 1, 32, 8, 128, 1000, tiled=1),
        # one long document
        c("step-32k", "step", "b2d4", 1, 32, 8, 128, 32768, tiled=1),
        # the longest context the layer is benchmarked on, two and four bits per element
        c("step-196k", "step", "b2d4", 1, 32, 8, 128, 196608, tiled=1),
        c("step-196k-b4d2", "step", "b4d2", 1, 32, 8, 128, 196608, tiled=1),
        # a serving batch: 32 sequences of different lengths, up to 8192 tokens
        c("step-batch32", "step", "b2d4", 32, 32, 8, 128, 8192, tiled=1, ragged=1),
        # 1.5 bits per element, 12-bit codes with a shared codebook
        c("step-100k-d8b12", "step", "d8b12", 1, 32, 8, 128, 100003),
        # head dim 64, a few sequences, recent tokens kept in full precision, codes in rows
        c("window-d64", "window", "b2d4", 4, 32, 8, 64, 30001, R=128),
        # decode-time append of a batch whose attention runs elsewhere
        c("append-32", "append", "b2d4", 32, 32, 8, 128, 1, pos0=4095),
        # the full-precision windows of a batch flushed into the cache
        c("fill-128", "fill", "b2d4", 8, 32, 8, 128, 128, pos0=3968, tiled=1),
        # prefill of a long prompt
        c("fill-64k", "fill", "b2d4", 1, 32, 8, 128, 65536, pos0=0, tiled=1),
        # prefill with 12-bit codes, a prompt of no particular length
        c("fill-10k-d8b12", "fill", "d8b12", 1, 32, 8, 128, 10007, pos0=0),
        # codebooks of one layer's keys from calibration text
        c("train-32k", "train", "b2d4", 1, 32, 8, 128, 32768, iters=8),
    ]


def _log(rng, lo, hi):
    """An integer from lo to hi, spread over its logarithm, mostly odd sizes."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _row_bytes(case, keys):
    d, b = CODES[case["code"]][0 if keys else 1], CODES[case["code"]][2 if keys else 3]
    return case["D"] // d * b // 8


def draw(rng):
    kind = rng.choices(["step", "window", "append", "fill", "train"], [9, 3, 2, 4, 2])[0]
    D = rng.choices([128, 64], [3, 1])[0]
    code = rng.choices(list(CODES), [6, 3, 2, 2, 2, 1, 1, 1])[0]
    dk, dv, bk, bv = CODES[code]
    Hq, Hkv = rng.choices([(32, 8), (28, 4), (64, 8), (16, 8), (8, 8), (40, 8)], [5, 1, 1, 1, 1, 1])[0]
    wide = bk != 8 or bv != 8
    can_tile = not wide and D // dv >= 16
    more = {"tiled": 1} if can_tile and rng.random() < 0.7 else {}
    if kind in ("step", "window"):
        B = rng.choice([1, 1, 1, 2, 3, 4, 8, 16, 24, 32])
        c = _case(kind, code, B, Hq, Hkv, D, 1, **more)
        per_token = B * Hkv * (_row_bytes(c, True) + _row_bytes(c, False))
        c["N"] = _log(rng, 300, min(196608, int(2.0e8 / per_token)))     # no more codes than the largest listed cache
        if B > 1 and rng.random() < 0.6:
            c["ragged"] = 1
        if kind == "window":
            c["R"] = rng.choice([128, 128, 96, 33, 1])
        return c
    if kind == "append":
        return _case(kind, code, rng.randint(1, 48), Hq, Hkv, D, rng.choice([1, 1, 2, 3, 7, 16]),
                     pos0=rng.randint(0, 8192), **more)
    if kind == "fill":
        B = rng.choice([1, 1, 1, 2, 4, 8])
        return _case(kind, code, B, Hq, Hkv, D, _log(rng, 20, (10000 if wide else 65536) * 8 // (B * Hkv)),
                     pos0=rng.choice([0, 0, rng.randint(1, 5000)]), **more)
    B = rng.choice([1, 1, 2, 4])
    return _case(kind, code, B, Hq, Hkv, D, _log(rng, 1000, (4096 if wide else 32768) * 8 // (B * Hkv)),
                 iters=rng.randint(2, 8))


def _cfg(case):
    dk, dv, bk, bv = CODES[case["code"]]
    return vb.Config(case["D"], case["Hq"], case["Hkv"], dk, dv, bk, bv, case.get("tiled", 0))


def _capacity(case):
    """Rows of the code caches: whole blocks of 64 tokens."""
    n = case["N"] + case.get("pos0", 0)
    return (n + 63) // 64 * 64


def _lengths(case):
    """Lengths of a ragged batch: spread evenly from an eighth of N to N."""
    B, N = case["B"], case["N"]
    return [max(1, N // 8 + (N - N // 8) * (i + 1) // B) for i in range(B)]


class _Draws:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def codes(self, *shape):
        return torch.randint(0, 256, shape, generator=self.g, device="cuda", dtype=torch.uint8)

    def keys(self, B, Hkv, T, D):
        """Raw keys: a few channels of each head are twenty times the others."""
        k = self.normal(B, Hkv, T, D)
        ch = torch.randint(0, D, (Hkv, 4), generator=self.g, device="cuda")
        scale = torch.ones(Hkv, D, device="cuda").scatter_(1, ch, 20.0)
        return (k * scale[None, :, None, :]).half(), scale


def _hadamard(D):
    h = torch.ones(1, 1, device="cuda")
    while h.shape[0] < D:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h / math.sqrt(D)


def _codebook(cfg, keys, vectors):
    """Centroids as an initial codebook has them: sub-vectors of other tokens, `vectors` [Hkv, n, D]."""
    d, bits = (cfg.k_sub_dim, cfg.k_bits) if keys else (cfg.v_sub_dim, cfg.v_bits)
    Hkv, n, D = vectors.shape
    if bits == 8:
        cb = vectors[:, :256].reshape(Hkv, 256, D // d, d).transpose(1, 2)
    else:
        cb = vectors.reshape(Hkv, n * D // d, d)[:, : 1 << bits]
    return cb.half().contiguous()


def prepare(case, seed):
    r, cfg, kind = _Draws(seed), _cfg(case), case["kind"]
    B, Hq, Hkv, D, N = (case[k] for k in ("B", "Hq", "Hkv", "D", "N"))
    s = {"kind": kind, "cfg": cfg, "N": N, "pos0": case.get("pos0", 0), "iters": case.get("iters", 0)}
    cap = _capacity(case)
    if kind in ("step", "window"):
        # codes, codebooks, smoothing factors and query of one layer
        s["q"] = r.normal(B, Hq, D).half()
        s["lam"] = torch.exp(0.5 * r.normal(Hkv, D))
        s["cb_k"], s["cb_v"] = r.normal(*cfg.cb_shape(True)).half(), r.normal(*cfg.cb_shape(False)).half()
        s["k_idx"] = r.codes(B, Hkv, cap, cfg.row_bytes(True))
        s["v_idx"] = r.codes(B, Hkv, cap, cfg.row_bytes(False))
        s["seq_lens"] = None
        if case.get("ragged"):
            order = torch.randperm(B, generator=r.g, device="cuda")
            s["seq_lens"] = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")[order].contiguous()
        if kind == "step":
            s["k"], s["v"] = r.keys(B, Hkv, 1, D)[0], r.normal(B, Hkv, 1, D).half()
        else:
            s["k"], s["v"] = r.keys(B, Hkv, case["R"], D)[0], r.normal(B, Hkv, case["R"], D).half()
        s["ws"] = vb.new_workspace(cfg, B, N)
        s["out"] = torch.empty(B, Hq, D, dtype=torch.float16, device="cuda")
        s["lse"] = torch.empty(B, Hq, dtype=torch.float32, device="cuda")
        return s
    s["k"], scale = r.keys(B, Hkv, N, D)
    s["v"] = r.normal(B, Hkv, N, D).half()
    # smoothing factors and codebooks come from other tokens of the same heads; as many of them as
    # the largest shared table needs (4096 sub-vectors of 8 channels)
    n = 4096 * 8 // D
    other = r.normal(Hkv, max(n, 256), D) * scale[:, None, :]
    s["lam"] = other.abs().amax(1).sqrt()
    s["cb_k"] = _codebook(cfg, True, (other / s["lam"][:, None, :]) @ _hadamard(D))
    if kind == "train":
        s["cb"], s["codes"] = torch.empty_like(s["cb_k"]), torch.zeros(B, Hkv, N, cfg.row_bytes(True), dtype=torch.uint8, device="cuda")
        s["ws"] = vb.new_kmeans_workspace(cfg, True)
        s["iters_run"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        s["errors"] = torch.zeros(s["iters"], dtype=torch.float64, device="cuda")
        return s
    s["cb_v"] = _codebook(cfg, False, r.normal(Hkv, max(n, 256), D))
    s["k_idx"] = torch.zeros(B, Hkv, cap, cfg.row_bytes(True), dtype=torch.uint8, device="cuda")
    s["v_idx"] = torch.zeros(B, Hkv, cap, cfg.row_bytes(False), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    kind, cfg = s["kind"], s["cfg"]
    if kind == "step":
        vb.vecinfer_decode_step(cfg, s["q"], s["k"], s["v"], s["lam"], s["cb_k"], s["cb_v"], s["k_idx"], s["v_idx"],
                                s["ws"], s["out"], lse=s["lse"], seq_lens=s["seq_lens"], N=s["N"])
        return {"out": s["out"], "lse": s["lse"], "k_idx": s["k_idx"], "v_idx": s["v_idx"]}
    if kind == "window":
        vb.vecinfer_decode_attention_residual(cfg, s["q"], s["lam"], s["cb_k"], s["cb_v"], s["k_idx"], s["v_idx"],
                                              s["k"], s["v"], s["ws"], s["out"], lse=s["lse"], seq_lens=s["seq_lens"],
                                              N=s["N"])
        return {"out": s["out"], "lse": s["lse"]}
    if kind == "append":
        vb.vecinfer_append_kv(cfg, s["k"], s["v"], s["lam"], s["cb_k"], s["cb_v"], s["k_idx"], s["v_idx"], pos0=s["pos0"])
        return {"k_idx": s["k_idx"], "v_idx": s["v_idx"]}
    if kind == "fill":
        vb.vecinfer_encode_keys(cfg, s["k"], s["lam"], s["cb_k"], s["k_idx"], pos0=s["pos0"])
        vb.vecinfer_encode_values(cfg, s["v"], s["cb_v"], s["v_idx"], pos0=s["pos0"])
        return {"k_idx": s["k_idx"], "v_idx": s["v_idx"]}
    # the smoothing factors of the calibration tokens, then the codebooks of the keys they transform,
    # from the same initial centroids every time
    vb.vecinfer_calibrate_lambda(cfg, s["k"], s["lam"])
    s["cb"].copy_(s["cb_k"])
    vb.vecinfer_kmeans_train(cfg, s["k"], s["lam"], s["cb"], s["codes"], s["ws"], max_iters=s["iters"],
                             iters_run=s["iters_run"], errors=s["errors"])
    return {"lam": s["lam"], "cb": s["cb"], "codes": s["codes"], "iters_run": s["iters_run"], "errors": s["errors"]}


def work(case):
    kind, cfg = case["kind"], _cfg(case)
    B, Hq, Hkv, D, N = (case[k] for k in ("B", "Hq", "Hkv", "D", "N"))
    rows = cfg.row_bytes(True) + cfg.row_bytes(False)
    tables = 2 * (math.prod(cfg.cb_shape(True)) + math.prod(cfg.cb_shape(False)))
    if kind in ("step", "window"):
        tokens = sum(_lengths(case)) if case.get("ragged") else B * N
        extra = B * (case.get("R", 0) if kind == "window" else 1)         # full-precision tokens: key and value
        return {"bytes": Hkv * (tokens * rows + extra * 4 * D) + tables + 4 * Hkv * D + B * Hq * (4 * D + 4),
                "flops": 4 * Hq * D * (tokens + extra)}
    if kind in ("append", "fill"):
        # distances of every sub-vector to every centroid of its table: one product, 2 C D per token
        return {"bytes": B * Hkv * N * (4 * D + rows) + tables + 4 * Hkv * D,
                "flops": 2 * B * Hkv * N * D * ((1 << cfg.k_bits) + (1 << cfg.v_bits))}
    cb = 2 * math.prod(cfg.cb_shape(True))
    return {"bytes": B * Hkv * N * (2 * D + cfg.row_bytes(True)) + 2 * cb + 4 * Hkv * D,
            "flops": 2 * B * Hkv * N * D * (1 << cfg.k_bits) * case["iters"]}


def tolerance(case):
    if case["kind"] in ("append", "fill"):
        return "exact"              # codes: the nearest centroid in fp32, lowest index among equals
    if case["kind"] == "train":
        # Sums in another order round a few centroids to the neighbouring fp16 value, and a few
        # sub-vectors on the border of two cells then change sides, which moves a small cluster's mean
        # (two trainings on the same inputs: 7e-4, 0.07 and 6e-5).
        return {"rel": 3e-3, "max": 0.3, "differ": 3e-4}
    # fp16 outputs and fp16 softmax weights, fp32 scores and sums (against fp64: 2.4e-4 and 7e-4)
    return {"rel": 1e-3, "max": 3e-3}
