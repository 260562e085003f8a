"""Performance cases of the fused VQ kernels: the calls a serving program makes, over the range it makes them.

A weight case is one linear layer (or a list of layers) of a decoder whose weight is stored as vector-quantization
codes; shapes are those of the benchmark configurations (Llama-7B layers: 4096 x 4096, 11008 x 4096, 4096 x 11008) and
sizes below them, odd row counts among them.  A cache case is decode attention over, or quantization into, a
VQ-compressed KV cache.  Codes are uniform over the codebook, codebooks and activations normal, scales uniform in
[0.5, 1.5): the distributions of ``paper_2503_02236_amd.workloads``.
"""
import math

import numpy as np
import torch

import paper_2503_02236_amd as vq
from paper_2503_02236_amd import workloads as wl

DEV = "cuda:0"

#: weight formats: v, code bits, additive codebooks R, entries E, sigma of the codebooks, tile of the codebook scope
FORMATS = {
    "u8x1": (8, 8, 1, 256, 0.02, None),           # one 256-entry codebook (1 bit per weight)
    "u8x2": (8, 8, 2, 256, 0.01, None),           # two additive 256-entry codebooks (2 bit)
    "u12x2": (8, 12, 2, 4096, 0.01, None),        # two additive 4096-entry codebooks, packed 12-bit codes (3 bit)
    "u16": (8, 16, 1, 65536, 0.02, None),         # one 2^16-entry codebook (2 bit), canonical codes
    "u16v4": (4, 16, 1, 65536, 0.02, None),       # one 2^16-entry codebook of 4-vectors (4 bit)
    "u16pack": (8, 16, 1, 65536, 0.02, None),     # "u16" with the offline re-tiled codes of the bs = 1 path
    "tile": (4, 8, 1, 256, 0.02, (256, 256)),     # one 256-entry codebook per 256 x 256 tile (2 bit)
}


def listed():
    return [
        # the smallest call: a 256 x 256 layer, one token; latency only
        {"name": "gemv_256", "kind": "gemv", "fmt": "u8x1", "N": 256, "K": 256, "bs": 1, "scale": False},
        # one attention projection of a single decoding sequence, large codebook, re-tiled codes
        {"name": "gemv_64k_bs1", "kind": "gemv", "fmt": "u16pack", "N": 4096, "K": 4096, "bs": 1, "scale": True},
        # the up projection of eight decoding sequences, large codebook
        {"name": "gemv_64k_bs8", "kind": "gemv", "fmt": "u16", "N": 11008, "K": 4096, "bs": 8, "scale": True},
        # the down projection of sixteen decoding sequences, additive codebooks
        {"name": "gemv_additive_bs16", "kind": "gemv", "fmt": "u8x2", "N": 4096, "K": 11008, "bs": 16, "scale": True},
        # a ragged output dimension (a vocabulary shard, say), three sequences, 12-bit codes
        {"name": "gemv_12bit_bs3", "kind": "gemv", "fmt": "u12x2", "N": 4001, "K": 4096, "bs": 3, "scale": True},
        # all projections of two decoder blocks for one token, large codebooks, one pipelined call
        {"name": "stack_64k", "kind": "stack", "fmt": "u16pack", "d": 4096, "f": 11008, "blocks": 2},
        # all projections of a whole 32-block decoder for one token, additive codebooks, one pipelined call
        {"name": "stack_additive", "kind": "stack", "fmt": "u8x2", "d": 4096, "f": 11008, "blocks": 32},
        # prefill of a 2048-token prompt through an up projection
        {"name": "gemm_prefill", "kind": "gemm", "fmt": "u16", "N": 11008, "K": 4096, "M": 2048, "scale": False},
        # prefill of a short prompt, additive codebooks
        {"name": "gemm_short", "kind": "gemm", "fmt": "u8x2", "N": 4096, "K": 4096, "M": 77, "scale": True},
        # decode attention of sixteen sequences over 4096 cached tokens, one codebook per head and side
        {"name": "attn_b16", "kind": "attn", "B": 16, "H": 32, "T": 4096, "v": 4, "G": 1, "ragged": False, "append": False},
        # a decode step of a few sequences on a coupled-quantization cache: quantize the new token, then attend
        {"name": "attn_cq_append", "kind": "attn", "B": 3, "H": 32, "T": 3001, "v": 4, "G": 32, "ragged": False, "append": True},
        # quantization of a prompt's keys and values into the cache
        {"name": "kv_prefill", "kind": "kvq", "B": 2, "H": 32, "T": 2560, "v": 4, "G": 1, "n_new": 2048, "pos": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "batch", "stack", "gemm", "gemm", "attn", "attn", "kvq"])
    if kind in ("gemv", "batch", "gemm"):
        c = {"kind": kind, "fmt": rng.choice(sorted(FORMATS)), "N": _log(rng, 64, 11008), "scale": rng.random() < 0.7}
        c["K"] = 256 * max(1, min(43, _log(rng, 256, 11008) // 256)) if c["fmt"] == "tile" else 64 * max(4, _log(rng, 256, 11008) // 64)
        if kind == "gemv":
            c["bs"] = 1 if c["fmt"] == "u16pack" else rng.randint(1, 16)
        elif kind == "batch":
            c["count"] = rng.randint(2, 4)      # projections that share their input
        else:
            if c["fmt"] == "u16pack":
                c["fmt"] = "u16"                # re-tiled codes are for one token
            c["M"] = _log(rng, 17, 2048)
        return c
    if kind == "stack":
        fmt = rng.choice(["u8x1", "u8x2", "u16pack"])
        d = 64 * (_log(rng, 512, 4096) // 64)
        return {"kind": kind, "fmt": fmt, "d": d, "f": 64 * (d * 43 // 1024), "blocks": rng.randint(1, 2) if fmt == "u16pack" else _log(rng, 1, 32)}
    B, H, T = _log(rng, 1, 16), rng.choice([8, 32]), _log(rng, 64, 4096)
    v, G = rng.choice([(4, 1), (4, 1), (4, 32), (2, 64), (8, 1)])
    if kind == "attn":
        ragged = rng.random() < 0.4
        return {"kind": kind, "B": B, "H": H, "T": T, "v": v, "G": G, "ragged": ragged, "append": not ragged and rng.random() < 0.6}
    B = min(B, 4)
    n_new = min(_log(rng, 1, min(T, 2048)), 4096 * v // 4 // B)
    return {"kind": kind, "B": B, "H": H, "T": T, "v": v, "G": G, "n_new": n_new, "pos": rng.randint(0, T - n_new)}


# ------------------------------------------------------------------------------------------------ inputs

def _normal(g, shape, sigma=1.0):
    return (torch.randn(shape, generator=g, device=DEV) * sigma).to(torch.float16)


def _weight(g, seed, fmt, N, K, scale):
    """A weight on the GPU, as the loader of a checkpoint leaves it."""
    v, bits, R, E, sigma, tile = FORMATS[fmt]
    if fmt == "u16pack":   # codes are re-tiled on the host
        return vq.weight_to_device(wl.make_weight(N, K, v, bits, R, E, sigma, seed, with_scale=scale), DEV, prepack=True, keep_codes=False)
    codes = torch.randint(0, 256 if bits == 12 else E, (N, K // v * R * 3 // 2) if bits == 12 else (N, K // v, R), generator=g,
                          device=DEV, dtype=torch.int32)   # (a random 12-bit string is random bytes)
    codes = codes.to(torch.uint16 if bits == 16 else torch.uint8)
    cb_shape = (R, E, v) if tile is None else (-(-N // tile[0]), K // tile[1], R, E, v)
    sc = (torch.rand(N, generator=g, device=DEV) + 0.5).to(torch.float16) if scale else None
    return vq.VQWeightDev(N, K, v, bits, codes, _normal(g, cb_shape, sigma), sc, cb_tile=tile)


def _stack_shapes(case):
    d, f = case["d"], case["f"]
    return [[(d, d)] * 3, [(d, d)], [(f, d)] * 2, [(d, f)]]   # q/k/v, o, gate/up, down


def _lens(case):
    """Valid tokens per sequence of a ragged batch: from T downwards."""
    return [case["T"] - b * case["T"] // case["B"] if case.get("ragged") else case["T"] for b in range(case["B"])]


def _cache(g, case, D=128):
    B, H, T, v, G = (case[k] for k in ("B", "H", "T", "v", "G"))
    codes = lambda: torch.randint(0, 256, (B, H, T, D // v), generator=g, device=DEV, dtype=torch.uint8)  # noqa: E731
    kv = vq.VQKVDev(B, H, D, T, v, codes(), codes(), _normal(g, (H, G, 256, v)), _normal(g, (H, G, 256, v)))
    if case.get("ragged"):
        kv.seq_lens = torch.tensor(_lens(case), dtype=torch.int32, device=DEV)
    return kv


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "gemv":
        w = _weight(g, seed, case["fmt"], case["N"], case["K"], case["scale"])
        need = vq.vq_gemv_workspace(w, case["bs"])
        return {"kind": kind, "w": w, "x": _normal(g, (case["bs"], case["K"])), "ws": vq.new_workspace(need, DEV) if need else None}
    if kind == "batch":
        w = [_weight(g, seed + 7919 * i, case["fmt"], case["N"], case["K"], case["scale"]) for i in range(case["count"])]
        x = _normal(g, (1, case["K"]))
        need = sum(vq.vq_gemv_workspace(t, 1) + 256 for t in w)
        return {"kind": kind, "w": w, "x": [x] * len(w), "ws": vq.new_workspace(need, DEV)}
    if kind == "gemm":
        w = _weight(g, seed, case["fmt"], case["N"], case["K"], case["scale"])
        need = vq.vq_gemm_workspace(w, case["M"])
        return {"kind": kind, "w": w, "x": _normal(g, (case["M"], case["K"])), "ws": vq.new_workspace(need, DEV) if need else None}
    if kind == "stack":
        calls, n = [], 0
        y = torch.empty(case["blocks"] * sum(N for c in _stack_shapes(case) for N, _ in c), dtype=torch.float16, device=DEV)
        for blk in range(case["blocks"]):
            for c in _stack_shapes(case):
                x = _normal(g, (1, c[0][1]))
                call = []
                for N, K in c:
                    w = _weight(g, seed + 7919 * (n + 1), case["fmt"], N, K, True)
                    call.append((w, x, y[n:n + N].view(1, N)))
                    n += N
                calls.append(call)
        return {"kind": kind, "pipe": vq.GemvPipeline(calls), "y": y, "calls": calls}
    kv = _cache(g, case)
    n_new = case.get("n_new", 1)
    state = {"kind": kind, "kv": kv, "pos": case.get("pos", case["T"] - 1)}
    if kind == "kvq" or case["append"]:
        state["k_new"] = _normal(g, (case["B"], case["H"], n_new, 128))
        state["v_new"] = _normal(g, (case["B"], case["H"], n_new, 128))
    if kind == "attn":
        need = vq.vq_attn_decode_workspace(kv)
        state["q"] = _normal(g, (case["B"], case["H"], 128))
        state["ws"] = vq.new_workspace(need, DEV) if need else None
    return state


# ------------------------------------------------------------------------------------------------ one pass

def run(s):
    kind = s["kind"]
    if kind == "gemv":
        return vq.vq_gemv(s["w"], s["x"], ws=s["ws"])
    if kind == "batch":
        return vq.vq_gemv_batch(s["w"], s["x"], ws=s["ws"])
    if kind == "gemm":
        return vq.vq_gemm(s["w"], s["x"], ws=s["ws"])
    if kind == "stack":
        status = s["pipe"].run()
        if status != 0:
            raise vq.VQError(status, "vq_gemv_pipeline_run")
        return s["y"]
    if "k_new" in s:
        vq.vq_kv_quantize(s["kv"], s["k_new"], s["v_new"], s["pos"])
    codes = [s["kv"].k_codes, s["kv"].v_codes] if "k_new" in s else []
    if kind == "kvq":
        return codes
    return [vq.vq_attn_decode(s["kv"], s["q"], 128.0 ** -0.5, ws=s["ws"])] + codes


# ------------------------------------------------------------------------------------------------ what it costs, how exact it is

def _gemv_bytes(fmt, N, K, tokens, scale, with_x=True):
    v, bits, R, E, _, tile = FORMATS[fmt]
    sets = 1 if tile is None else -(-N // tile[0]) * (K // tile[1])
    entries = min(sets * E, N * (K // v))     # no more than there are codes
    return N * (K // v) * R * bits // 8 + R * entries * v * 2 + (tokens * K * 2 if with_x else 0) + tokens * N * 2 + (N * 2 if scale else 0)


def work(case):
    kind = case["kind"]
    if kind in ("gemv", "gemm"):
        tokens = case["bs"] if kind == "gemv" else case["M"]
        return {"bytes": _gemv_bytes(case["fmt"], case["N"], case["K"], tokens, case["scale"]), "flops": 2.0 * tokens * case["N"] * case["K"]}
    if kind == "batch":
        return {"bytes": case["count"] * _gemv_bytes(case["fmt"], case["N"], case["K"], 1, case["scale"], with_x=False) + 2 * case["K"],
                "flops": 2.0 * case["count"] * case["N"] * case["K"]}
    if kind == "stack":
        calls = _stack_shapes(case)
        b = sum(_gemv_bytes(case["fmt"], N, K, 1, True, with_x=False) for c in calls for N, K in c) + sum(2 * c[0][1] for c in calls)
        return {"bytes": case["blocks"] * b, "flops": case["blocks"] * sum(2.0 * N * K for c in calls for N, K in c)}
    H, v, P = case["H"], case["v"], 128 // case["v"]
    books = 2 * H * case["G"] * 256 * v * 2
    heads = case["B"] * H
    b, f = float(books), 0.0
    if kind == "attn":
        tokens = sum(_lens(case)) * H
        b += 2 * tokens * P + 2 * heads * 128 * 2
        f += 4.0 * tokens * 128
    if kind == "kvq" or case["append"]:
        n = case.get("n_new", 1) * heads
        b += 2 * n * (128 * 2 + P)
        f += 2 * n * P * 256 * 2.0 * v    # every distance: at least the inner product with every entry
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "kvq":
        return "exact"   # codes
    # Against the same products in 64 bits: fp16 outputs of fp32 sums are off by 2.1e-4 (largest 4.9e-4, half an ulp);
    # where additive codebooks are summed into an fp16 operand, by 3.1e-4 (largest 1.45e-3).  Four times that.
    if case.get("fmt") in ("u8x2", "u12x2"):
        return {"rel": 1.2e-3, "max": 6e-3}
    return {"rel": 9e-4, "max": 2e-3}
