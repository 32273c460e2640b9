"""Workloads of the framework's public entry points, for timing one build of it against another.

Every case compresses seeded synthetic bf16 weights in prepare() and takes one call through the library in run():
the decode of the experts a gate selected (the main path, in its three forms), the split path's recovery kernel, a
fetch from the expert cache, and the offline compression.  All outputs are whole numbers (bf16 bit patterns, bytes)
and have to come out bit for bit: the codec is lossless and its encoder is a function of its input alone.
"""
import ctypes
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2601_21198_amd import zipmoe as zm

DEVICE = "cuda:0"
WORKERS = 16

# Bytes per value of a compressed Gaussian tensor: one sign-mantissa byte and about 2.7 bits of code and framing.
SM_BYTES, E_BYTES, BF16_BYTES = 1.0, 0.345, 2.0


def decode_case(name, api, rows, cols, matrices, resident, selected, chunk, stream, max_len=8, stores="auto",
                values="gauss", ragged=0):
    """api: "call" (ExpertLayer.make_call, a pre-marshalled call repeated as it is), "decode" (ExpertLayer.decode, ids
    named anew on every pass), "handle" (Layer, the library's own handle).  An expert has `matrices` matrices of
    rows x cols values; ragged > 0: expert e's matrices are cut to lengths that fall off towards rows*cols / ragged."""
    return {"name": name, "kind": "decode", "api": api, "rows": rows, "cols": cols, "matrices": matrices,
            "resident": resident, "selected": selected, "chunk": chunk, "stream": stream, "max_len": max_len,
            "stores": stores, "values": values, "ragged": ragged}


def listed():
    return [
        # one small matrix: the smallest call there is, all latency
        decode_case("matrix", "call", 256, 512, 1, 1, 1, 4096, 4096),
        # one expert of a 2048 x 1408 SwiGLU layer with outlier weights (a single token that activates one expert, or
        # a shared expert)
        decode_case("expert-outliers", "decode", 1408, 2048, 3, 1, 1, 16384, 4096, values="outliers"),
        # one token's gate: top-4 of a layer's resident experts; the program's output buffers are not cache-resident
        # and it says so.  This is the call that bench.py times.
        decode_case("layer-top4", "decode", 1408, 2048, 3, 8, 4, 16384, 4096, stores="streaming"),
        # top-8 of a layer whose experts were compressed with the longest codes the format admits (the densest blobs),
        # through the library's layer handle
        decode_case("layer-top8-long-codes", "handle", 1024, 2048, 3, 12, 8, 16384, 4096, max_len=12),
        # the largest call of the benchmark's configurations (two experts of 4096 x 14336, rows of different scale): bound
        # by bandwidth
        decode_case("layer-large", "decode", 14336, 4096, 3, 2, 2, 16384, 4096, values="row-scaled"),
        # a finer compression geometry (small chunks can be replaced or cached in small units), small codes
        decode_case("short-streams", "decode", 1024, 2048, 3, 4, 2, 4096, 1024),
        # a coarse geometry: one long stream per chunk, the least framing
        decode_case("long-streams", "decode", 1408, 2048, 3, 4, 2, 16384, 16384),
        # a prompt: many tokens activate every expert of a fine-grained layer at once (192 tensors in a call)
        decode_case("prefill-all-experts", "handle", 512, 1024, 3, 64, 64, 16384, 4096),
        # tensors of very different, odd lengths in one call (pruned experts, a shared expert beside routed ones)
        decode_case("ragged-lengths", "decode", 1024, 2049, 3, 8, 8, 16384, 4096, ragged=300),
        # the split path: exponent bytes decompressed elsewhere, the recovery kernel merges one large matrix
        {"name": "recover-large", "kind": "recover", "values": 14336 * 4096},
        # a serving loop over a layer that does not fit: four pools, the missing parts come over the host link
        {"name": "cache-fetch", "kind": "cache", "rows": 1024, "cols": 2048, "matrices": 3, "resident": 24, "selected": 4,
         "full": 2, "compressed": 6, "sm": 6, "e": 4, "chunk": 16384, "stream": 4096, "max_len": 8},
        # offline: one matrix from bf16 words to its serialised object, on the host
        {"name": "compress", "kind": "compress", "n": 1408 * 2048, "chunk": 16384, "stream": 4096, "max_len": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 7 + ["recover", "cache", "compress"])
    stream = rng.choice([512, 1024, 2048, 4096, 4096, 4096, 8192, 16384])
    chunk = stream * rng.choice([c for c in (1, 2, 4, 8) if stream * c <= 32768])
    max_len = rng.choice([8, 8, 8, 10, 12])
    if kind == "recover":
        return {"kind": kind, "values": _log_int(rng, 1 << 17, 14336 * 4096)}
    if kind == "compress":
        return {"kind": kind, "n": _log_int(rng, 1 << 15, 1408 * 2048), "chunk": chunk, "stream": stream, "max_len": max_len}
    if kind == "cache":
        resident = rng.randint(12, 24)
        return {"kind": kind, "rows": _log_int(rng, 128, 1024), "cols": _log_int(rng, 512, 2048), "matrices": 3,
                "resident": resident, "selected": rng.randint(1, 4), "full": rng.randint(0, 3), "compressed": rng.randint(0, 6),
                "sm": rng.randint(0, 6), "e": rng.randint(0, 4), "chunk": chunk, "stream": stream, "max_len": max_len}
    rows, cols = _log_int(rng, 64, 4096), _log_int(rng, 256, 8192)
    matrices = rng.choice([1, 3, 3])
    # the resident experts of a drawn case hold at most a sixth of the largest listed case's values
    most = max(1, min(64, 14336 * 4096 // (rows * cols * matrices)))
    resident = _log_int(rng, 1, most)
    ragged = rng.choice([0, 0, 0, 30, 300])
    selected = resident if ragged else _log_int(rng, 1, resident)
    case = decode_case("", rng.choice(["call", "decode", "handle"]), rows, cols, matrices, resident, selected, chunk, stream,
                       max_len, rng.choice(["auto", "auto", "streaming", "cached"]),
                       rng.choice(["gauss", "gauss", "outliers", "row-scaled"]), ragged)
    del case["name"]
    return case


# ---- inputs ----------------------------------------------------------------------------------------------------

def _weights(gen, rows, cols, values, std):
    """bf16 patterns of one matrix, made on the GPU: N(0, std^2) entries, with 1 % of them replaced by draws from a ten
    times wider distribution ("outliers") or with a log-normal scale per row ("row-scaled")."""
    x = torch.randn(rows, cols, generator=gen, device=DEVICE) * std
    if values == "outliers":
        mask = torch.rand(rows, cols, generator=gen, device=DEVICE) < 0.01
        x = torch.where(mask, torch.randn(rows, cols, generator=gen, device=DEVICE) * (10 * std), x)
    elif values == "row-scaled":
        x = x * torch.exp(0.3 * torch.randn(rows, 1, generator=gen, device=DEVICE))
    return x.to(torch.bfloat16).view(torch.int16).reshape(-1)


def _lengths(case):
    """values of every matrix, expert by expert"""
    n, ragged = case["rows"] * case["cols"], case.get("ragged", 0)
    if not ragged:
        return [[n] * case["matrices"] for _ in range(case["resident"])]
    top = max(1, case["resident"] * case["matrices"] - 1)
    return [[max(1, int(n / ragged ** ((e * case["matrices"] + m) / top))) for m in range(case["matrices"])]
            for e in range(case["resident"])]


def _blobs(case, seed):
    """the serialised objects of a layer's experts"""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    flat = []
    for lengths in _lengths(case):
        std = 0.01 + 0.04 * float(torch.rand(1, generator=gen, device=DEVICE))
        for n in lengths:
            w = _weights(gen, case["rows"], case["cols"], case.get("values", "gauss"), std)[:n]
            flat.append(w.cpu().numpy().view(np.uint16))
    with ThreadPoolExecutor(WORKERS) as pool:
        blobs = list(pool.map(lambda w: zm.compress(w, case["chunk"], case["stream"], case["max_len"])[0], flat))
    m = case["matrices"]
    return [blobs[i: i + m] for i in range(0, len(blobs), m)]


def _selected(case, seed):
    return [int(e) for e in np.random.default_rng(seed).permutation(case["resident"])[: case["selected"]]]


STORES = {"auto": zm.STORES_AUTO, "cached": zm.STORES_CACHED, "streaming": zm.STORES_STREAMING}


def _prepare_decode(case, seed):
    blobs = _blobs(case, seed)
    ids = _selected(case, seed)
    stores = STORES[case["stores"]]
    lengths = _lengths(case)
    widest = max(range(case["resident"]), key=lambda e: sum(lengths[e]))
    if case["api"] == "handle":
        layer = zm.Layer(blobs, DEVICE)
        starts = [sum(-(-n // 8) * 8 for n in lengths[widest][:m]) for m in range(case["matrices"] + 1)]
        bufs = [torch.zeros(starts[-1], dtype=torch.int16, device=DEVICE) for _ in ids]
        ptrs = [b.data_ptr() + 2 * s for b in bufs for s in starts[:-1]]
        return {"layer": layer, "ids": ids, "ptrs": ptrs, "stores": stores, "bufs": bufs, "run": _run_handle}
    layer = zm.ExpertLayer(blobs, DEVICE)
    bufs, starts, _ = layer.alloc_outputs(len(ids), expert=widest)
    for b in bufs:
        b.zero_()                                # the few values between tensors that nothing writes
    state = {"layer": layer, "ids": ids, "bufs": bufs, "starts": starts, "stores": stores, "run": _run_decode}
    if case["api"] == "call":
        state["call"] = layer.make_call(ids, bufs, starts, stores)
        state["run"] = _run_call
    return state


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _run_call(s):
    s["call"](_stream())
    return s["bufs"]


def _run_decode(s):
    s["layer"].decode(s["ids"], s["bufs"], s["starts"], _stream(), s["stores"])
    return s["bufs"]


def _run_handle(s):
    s["layer"].decode(s["ids"], s["ptrs"], _stream(), s["stores"])
    return s["bufs"]


def _prepare_recover(case, seed):
    n = case["values"]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    w = _weights(gen, 1, n, "gauss", 0.02).to(torch.int32) & 0xFFFF
    e = ((w >> 7) & 0xFF).to(torch.uint8)
    sm = (((w >> 8) & 0x80) | (w & 0x7F)).to(torch.uint8)
    return {"e": e, "sm": sm, "n": n, "out": torch.empty(n, dtype=torch.int16, device=DEVICE), "run": _run_recover}


def _run_recover(s):
    zm.recover(s["e"].data_ptr(), s["sm"].data_ptr(), s["n"], s["out"].data_ptr(), _stream())
    return s["out"]


def _prepare_cache(case, seed):
    blobs = _blobs(case, seed)
    cache = zm.ExpertCache(blobs, (case["full"], case["compressed"], case["sm"], case["e"]), 1, case["selected"], DEVICE)
    # a skewed popularity (rank r has weight 1/(r+1)); every pass asks for the next token's experts
    rng = np.random.default_rng(seed)
    p = 1.0 / np.arange(1, case["resident"] + 1)
    perm = rng.permutation(case["resident"])
    routes = [[int(perm[r]) for r in rng.choice(case["resident"], case["selected"], replace=False, p=p / p.sum())] for _ in range(256)]
    for ids in routes[:32]:                      # a server that has been running for a while
        cache.fetch(ids, _stream())
    return {"cache": cache, "routes": routes, "at": 32, "n": case["rows"] * case["cols"], "words": cache.arena.view(torch.int16),
            "run": _run_cache}


def _run_cache(s):
    ids = s["routes"][s["at"] % len(s["routes"])]
    s["at"] += 1
    ptrs, _ = s["cache"].fetch(ids, _stream())
    base = s["words"].data_ptr()
    return [[s["words"][(p - base) // 2: (p - base) // 2 + s["n"]] for p in row] for row in ptrs]


def _prepare_compress(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    w = _weights(gen, 1, case["n"], "gauss", 0.02)
    # the program's own buffer, from which it writes the object to its store
    out = np.zeros(zm.encode_bound(case["n"], case["chunk"], case["stream"]), np.uint8)
    return {"w": w.cpu().numpy().view(np.uint16), "case": case, "out": out, "run": _run_compress}


def _run_compress(s):
    c = s["case"]
    blob, table = zm.compress(s["w"], c["chunk"], c["stream"], c["max_len"])
    s["out"][: blob.size] = blob
    return [s["out"], table.view(np.int64)]


PREPARE = {"decode": _prepare_decode, "recover": _prepare_recover, "cache": _prepare_cache, "compress": _prepare_compress}


def prepare(case, seed):
    return PREPARE[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def work(case):
    """every compressed byte read once, every output byte written once; no floating-point work anywhere"""
    kind = case["kind"]
    if kind == "recover":
        return {"bytes": 4.0 * case["values"], "flops": 0}
    if kind == "compress":
        return {"bytes": (BF16_BYTES + SM_BYTES + E_BYTES) * case["n"], "flops": 0}
    lengths = [sum(row) for row in _lengths(case)]
    per_expert = sum(lengths) / len(lengths)
    return {"bytes": (SM_BYTES + E_BYTES + BF16_BYTES) * per_expert * case["selected"], "flops": 0}


def tolerance(case):
    return "exact"
