"""Workloads by which the library is timed: the calls a serving program makes around a prefill and while decoding.

A case is a dict of plain values.  ``path`` names what the program does:

  compress   the whole path after a prefill: score, refine, search + select, compact, all layers in the case in one
             call sequence.  ``lse`` says where the rows' softmax denominators come from: "own" (the scoring step
             computes them, K is read twice) or "window" (the attention of the window queries runs first and hands
             them over, as in a prefill that calls it)
  shared     the variant with one retained set per layer (head mean over all heads)
  decode     attention of one new token over a cache, the full one or the compacted one
  segment    token ids of a batch of prompts to segment offsets, which the other calls take

Inputs are normal variates (plus, where ``heavy`` is set, that many key rows per head scaled by four: the peaked
attention of real prompts); a region of T tokens is cut into T / mean segments at random places, which gives nearly
geometric lengths.  Everything comes from the seed alone.
"""

import math

import numpy as np
import torch

from paper_2510_22556_amd import binding as B
from paper_2510_22556_amd import synth

DEV = "cuda:0"
POW2 = "1,2,4,8,16,32,64"                      # candidate block sizes: powers of two, or the paper's own list
PAPER = "1,2,3,5,7,9,11,13"


def _compress(name, **kw):
    c = {"name": name, "path": "compress", "lse": "own", "dtype": "bf16", "n_seq": 1, "layers": 1, "q_heads": 32,
         "kv_heads": 8, "dim": 128, "length": 8192, "window": 32, "cache": 1024, "cand": POW2, "mean": 64, "heavy": 0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one small fp32 layer, all launches and latency (a unit test of a user's model, a toy model)
        _compress("tiny_f32", dtype="f32", q_heads=4, kv_heads=2, dim=64, length=2048, window=16, cache=128,
                  cand="1,2,4,8", mean=24),
        # one layer of an 8B model with a short prompt: a prefill loop that compresses layer by layer
        _compress("layer_8k", mean=32, cand="1,2,4,8,16,32"),
        # the same loop with a long prompt
        _compress("layer_128k", length=131072),
        # all layers at once behind a prefill that hands the softmax denominators over; peaked attention
        _compress("model_32k_window", lse="window", layers=32, length=32768, cand="1,2,4,8,16,32", mean=48, heavy=64),
        # all layers at once, long prompt, the path alone: the library's headline workload
        _compress("model_128k", layers=32, length=131072),
        # a batch of long prompts with a window of 64: the largest call
        _compress("batch_4x64k", n_seq=4, layers=32, length=65536, window=64, cache=2048, mean=48),
        # the paper's own settings: window of 8, candidate sizes up to 13, a small cache
        _compress("paper_32k", layers=32, length=32768, window=8, cache=128, cand=PAPER, mean=28),
        # a group size that is no power of two and a prompt of odd length
        _compress("gqa7_ragged", layers=28, q_heads=28, kv_heads=4, length=30011, window=16, cand="1,2,4,8,16,32", mean=32),
        # one retained set per layer
        _compress("shared_32k", path="shared", layers=32, length=32768, mean=48),
        # one decode step over the cache as it was before compression ...
        {"name": "decode_full_128k", "path": "decode", "dtype": "bf16", "n_seq": 1, "layers": 32, "q_heads": 32,
         "kv_heads": 8, "dim": 128, "rows": 131072, "budget": 0},
        # ... and over the compacted one: what every later token costs
        {"name": "decode_compacted", "path": "decode", "dtype": "bf16", "n_seq": 1, "layers": 32, "q_heads": 32,
         "kv_heads": 8, "dim": 128, "rows": 1024, "budget": 992},
        # the segmentation of a batch of prompts, offsets in the program's hands
        {"name": "segment_4x64k", "path": "segment", "n_seq": 4, "length": 65472, "mean": 48},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_KEYS = 1024 * 65536                        # keys x KV heads x layers of the largest listed case ...
MAX_ROW_KEYS = MAX_KEYS * 256                  # ... times its window-query rows per KV head


def draw(rng):
    path = rng.choice(["compress"] * 6 + ["shared", "decode", "decode", "segment"])
    if path == "segment":
        return {"path": "segment", "n_seq": rng.randint(1, 8), "length": _log_int(rng, 1000, 131000), "mean": rng.choice([16, 28, 48, 64, 128])}
    c = {"path": path, "dtype": "f32" if path != "shared" and rng.random() < 0.2 else "bf16"}
    c["n_seq"] = rng.choice([1, 1, 1, 2, 4])
    c["layers"] = _log_int(rng, 1, 32)
    c["kv_heads"] = rng.choice([2, 4, 8, 8])
    group = rng.choice([1, 2, 4, 4, 4, 5, 7, 8])
    c["q_heads"] = group * c["kv_heads"]
    c["dim"] = 128 if path == "shared" else rng.choice([64, 128, 128, 128, 256 if path == "compress" else 64])
    problems = c["n_seq"] * c["layers"] * c["kv_heads"]
    if path == "decode":
        c["rows"] = min(_log_int(rng, 128, 131072), 2 ** 25 // problems)
        c["budget"] = 0 if c["rows"] > 4500 else max(c["rows"] - rng.choice([8, 16, 32, 64]), 0)
        return c
    windows = [8, 16, 32] if path == "shared" else [8, 16, 32, 32, 64]
    most = 96 if c["dim"] == 256 else 256 if c["dim"] == 128 and path == "compress" and c["dtype"] == "bf16" else 128
    c["window"] = rng.choice([w for w in windows if group * w <= min(most, 128) or (w >= 32 and group * w <= most)])
    rows = group * c["window"]
    # fp32 runs on the vector pipe: contexts of the size that such a model is given, and few layers
    longest = 16384 if c["dtype"] == "f32" else 131072
    room = min(MAX_KEYS, MAX_ROW_KEYS // max(rows, 64)) * 128 // max(c["dim"], 128)
    if c["dtype"] == "f32":
        room = 2 ** 34 // (rows * c["dim"])
    c["length"] = max(1024, min(_log_int(rng, 1024, longest), room // problems))
    while c["length"] * problems > room and c["layers"] > 1:
        c["layers"] = max(1, c["layers"] // 2)
        problems = c["n_seq"] * c["layers"] * c["kv_heads"]
    c["lse"] = "window" if path == "compress" and c["dtype"] == "bf16" and c["dim"] == 128 and rng.random() < 0.3 else "own"
    c["cache"] = max(c["window"] + 32, min(_log_int(rng, 96, 4096), c["length"] // 2))
    c["cand"] = rng.choice([POW2, PAPER, "1,2,4,8"])
    c["mean"] = rng.choice([16, 28, 48, 64, 128])
    c["heavy"] = rng.choice([0, 0, 64])
    return c


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, dtype=dtype, device=DEV)


def _cuts(seed, T, mean):
    """Ascending places, each in [1, T), at which a region of T tokens is cut into T / mean segments."""
    rng = np.random.default_rng(seed)
    return np.sort(rng.choice(T - 1, max(T // mean, 1) - 1, replace=False)) + 1


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if case["path"] == "segment":
        first = max(synth.DELIMS) + 1                          # ordinary token ids lie above the delimiters
        tok = torch.randint(first, 128256, (case["n_seq"], case["length"]), generator=gen, dtype=torch.int32, device=DEV)
        for s in range(case["n_seq"]):                         # a delimiter in front of every cut
            at = _cuts(seed + 7919 * s, case["length"], case["mean"]) - 1
            tok[s, torch.as_tensor(at).to(DEV)] = torch.as_tensor(np.resize(synth.DELIMS, len(at)).astype(np.int32)).to(DEV)
        return {"case": case, "tok": tok}
    n, nl, hq, hkv, D, dt = case["n_seq"], case["layers"], case["q_heads"], case["kv_heads"], case["dim"], _dtype(case)
    if case["path"] == "decode":
        q = _normal(gen, (n, nl, hq, D), dt)
        k, v = (_normal(gen, (n, nl, hkv, case["rows"], D), dt) for _ in range(2))
        shape = B.make_cache_shape(q, k, v)
        st = {"case": case, "q": q, "k": k, "v": v, "shape": shape, "n_sel": None,
              "out": torch.empty(q.shape, dtype=torch.float32, device=DEV),
              "ws": torch.empty((B.sablock_decode_workspace_bytes(shape),), dtype=torch.uint8, device=DEV)}
        if case["budget"] > 0:
            st["n_sel"] = torch.full((n * nl * hkv,), case["budget"], dtype=torch.int32, device=DEV)
        return st
    L, W = case["length"], case["window"]
    q = _normal(gen, (n, nl, hq, W, D), dt)
    k, v = (_normal(gen, (n, nl, hkv, L, D), dt) for _ in range(2))
    if case["heavy"]:
        at = torch.randperm(L - W, generator=gen, device=DEV)[: case["heavy"]]
        k[:, :, :, at] *= 4.0
    offs = [np.concatenate([[0], _cuts(seed + 7919 * s, L - W, case["mean"]), [L - W]]) for s in range(n)]
    ptr = np.cumsum([0] + [len(o) for o in offs])
    seg = B.make_segments(np.concatenate(offs), ptr, DEV)
    shape = B.make_shape(q, k, v)
    budget = case["cache"] - W
    st = {"case": case, "q": q, "k": k, "v": v, "seg": seg, "shape": shape, "budget": budget,
          "cand": [int(g) for g in case["cand"].split(",")], "lse": None}
    if case["path"] == "shared":
        per_layer = B.layer_shape(shape)
        st["layer"] = per_layer
        st["buf"] = B.Buffers(per_layer, seg, budget, DEV, append_window=True, dtype=dt)
        st["ws"] = torch.empty((B.sablock_score_all_heads_workspace_bytes(shape),), dtype=torch.uint8, device=DEV)
        rows = (n * nl * hkv, budget + W, D)
        st["k_out"], st["v_out"] = (torch.empty(rows, dtype=dt, device=DEV) for _ in range(2))
        return st
    st["buf"] = B.Buffers(shape, seg, budget, DEV, append_window=True)
    if case["lse"] == "window":
        st["lse"] = torch.empty((n, nl, hq, W), dtype=torch.float32, device=DEV)
        st["att"] = torch.empty((n, nl, hq, W, D), dtype=torch.float32, device=DEV)
        st["att_ws"] = torch.empty((B.sablock_window_attention_workspace_bytes(shape),), dtype=torch.uint8, device=DEV)
    return st


def _bits(t):
    """Rows of the compacted cache are bit copies of K and V rows: whole numbers of the element's width."""
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def run(state):
    c = state["case"]
    if c["path"] == "segment":
        seg = B.segment(state["tok"], synth.DELIMS)
        return {"offsets": seg.seg_off, "ptr": list(seg.seg_ptr), "max": seg.max_segments}
    if c["path"] == "decode":
        B.sablock_decode_attention(state["shape"], state["q"], state["k"], state["v"], state["out"], state["ws"],
                                   n_sel=state["n_sel"], budget=c["budget"])
        return {"out": state["out"]}
    q, k, v, seg, shape, budget, buf = (state[x] for x in ("q", "k", "v", "seg", "shape", "budget", "buf"))
    out = {}
    if c["path"] == "shared":
        per_layer = state["layer"]
        B.sablock_score_all_heads(shape, q, k, buf.s, buf.ent, state["ws"])
        B.sablock_refine(per_layer, buf.s, buf.ent, seg, buf.s_tilde, buf.ws, omega_out=buf.omega)
        B.sablock_search_select(per_layer, buf.s_tilde, seg, state["cand"], budget, 0.85, buf.seg_budget, buf.block_size,
                                buf.idx, buf.n_sel, buf.ws, topb_out=buf.topb)
        B.sablock_compact_shared(shape, k, v, buf.idx, buf.n_sel, budget, True, state["k_out"], state["v_out"])
        k_out, v_out = state["k_out"], state["v_out"]
    else:
        if c["lse"] == "window":
            B.sablock_window_attention(shape, q, k, v, state["att"], state["lse"], state["att_ws"])
            out.update(att=state["att"], lse=state["lse"])
        B.compress(shape, q, k, v, seg, state["cand"], budget, buf, row_lse=state["lse"])
        k_out, v_out = buf.k_out, buf.v_out
    out.update(s=buf.s, ent=buf.ent, s_tilde=buf.s_tilde, omega=buf.omega, seg_budget=buf.seg_budget,
               block_size=buf.block_size, idx=buf.idx, n_sel=buf.n_sel, k_out=_bits(k_out), v_out=_bits(v_out))
    return out


def work(case):
    if case["path"] == "segment":
        tokens = case["n_seq"] * case["length"]
        return {"bytes": 4 * tokens + 4 * tokens / case["mean"], "flops": 0}
    elt = 4 if case["dtype"] == "f32" else 2
    n, nl, hq, hkv, D = (case[x] for x in ("n_seq", "layers", "q_heads", "kv_heads", "dim"))
    P = n * nl * hkv
    if case["path"] == "decode":
        q = n * nl * hq * D
        return {"bytes": 2 * P * case["rows"] * D * elt + q * (elt + 4), "flops": 4.0 * q * case["rows"]}
    L, W, budget = case["length"], case["window"], case["cache"] - case["window"]
    rows = n * nl * hq * W                                     # window-query rows
    R = n * nl if case["path"] == "shared" else P              # score rows
    # K and the window queries in, s, its entropy term and s~ out (each once), the retained rows of K and V in and out
    nbytes = P * L * D * elt + rows * D * elt + R * (8 * L + 4 * (L - W)) + 4 * P * (budget + W) * D * elt + 4 * R * budget
    # products with K: once for the rows' denominators, once for the columns (the entropy term is not linear)
    flops = 2 * 2.0 * rows * L * D
    if case["lse"] == "window":
        nbytes += P * L * D * elt + rows * (D + 1) * 4         # V in, the attention's rows out
        flops += 2.0 * rows * L * D                            # probabilities times V
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the path differs from the same arithmetic in 64 bits."""
    if case["path"] == "segment":
        return "exact"
    if case["path"] == "decode":
        return {"rel": 2e-6, "max": 6e-6}                      # fp32 sums (4e-7, 1.3e-6 over 131 072 rows)
    if case["lse"] == "window":
        return {"rel": 6e-3, "max": 2e-2, "differ": 0.01}      # probabilities enter the product with V in bf16 (1.6e-3, 5e-3)
    # fp32 logits and sums (1.0e-6, 2.6e-6); whole values differ where the scores of two tokens tie to that
    return {"rel": 5e-6, "max": 2e-5, "differ": 0.01}
