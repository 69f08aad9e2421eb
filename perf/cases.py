"""The work whose speed is measured: what a program that serves long prompts has this library do on one GPU.

Eight kinds of work, each through the public entry points of ``paper_2409_15104_amd.binding``:

* ``member``   -- one ring member's prefill, one launch (``pec_sp_prefill``);
* ``sweep``    -- the same as a launch that a scheduler can stop (``pec_sp_prefill_resumable``, never stopped here);
* ``steps``    -- the same as one call per ring step (``pec_sp_prefill_step``), the caller keeping the running state;
* ``partials`` -- two ring steps as separate fp32 partials, their merge and the rounding to bf16 (``pec_attn_chunk``,
  ``pec_attn_merge``, ``pec_finalize``);
* ``packed``   -- a packed batch of prompts (``pec_attn_varlen``);
* ``mixed``    -- short prompts batched with the decode steps of long requests (``pec_attn_colocated``);
* ``decode``   -- one new token of a request against its KV cache (``pec_decode_splitkv``);
* ``exchange`` -- the head <-> sequence layout exchange, both directions (``pec_ulysses_layout``).

Q, K and V are N(0,1) rounded to bf16 as everywhere in this repository; prompt lengths are the log-normal mix of
``synth.lognormal_lengths``.  Outputs, workspaces and stop words are laid out once, as a serving program keeps them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2409_15104_amd import binding as pec
from paper_2409_15104_amd import synth

DEV = "cuda:0"
FLOP_PER_PAIR = 512.0      # per visible (query, key, head): 2 * 128 for q.k and 2 * 128 for p.v
ROW = 128


def listed():
    return [
        # the shortest ring: the last of four members of a 2K-token prompt, all query heads with their own KV head.
        # A handful of query tiles: launch and latency, a chip that is hard to fill.
        {"name": "member_2k", "kind": "member", "hq": 8, "hkv": 8, "s_q": 512, "q_off": 1536, "s_kv": 2048, "chunk": 512,
         "causal": True, "f32": False},
        # the last of eight members of a 32K-token prompt, grouped heads: an ordinary long prompt
        {"name": "member_32k", "kind": "member", "hq": 32, "hkv": 8, "s_q": 4096, "q_off": 28672, "s_kv": 32768,
         "chunk": 4096, "causal": True, "f32": False},
        # the last of sixteen members of a 128K-token prompt, as a launch that can be preempted: the headline workload
        {"name": "sweep_128k", "kind": "sweep", "hq": 32, "hkv": 8, "s_q": 8192, "q_off": 122880, "s_kv": 131072,
         "chunk": 8192, "causal": True, "f32": False},
        # the last of thirty-two members of a 512K-token prompt, 64 query heads: the largest share of one GPU
        {"name": "sweep_512k", "kind": "sweep", "hq": 64, "hkv": 8, "s_q": 16384, "q_off": 507904, "s_kv": 524288,
         "chunk": 16384, "causal": True, "f32": False},
        # the fourth member of a 32K-token prompt called one ring step at a time, the running fp32 state in memory
        {"name": "steps_32k", "kind": "steps", "hq": 32, "hkv": 8, "s_q": 4096, "q_off": 12288, "s_kv": 32768,
         "chunk": 4096, "causal": True, "f32": False},
        # two partial results over odd-sized key segments without a mask, merged and rounded: what members exchange
        # when partial results travel instead of keys
        {"name": "partials_ragged", "kind": "partials", "hq": 32, "hkv": 8, "s_q": 1999, "q_off": 6001, "s_a": 3001,
         "s_b": 2999, "causal": False},
        # a handful of short prompts that arrived together: the ordinary prefill of a lightly loaded server
        {"name": "packed_8", "kind": "packed", "hq": 32, "hkv": 8, "n": 8, "len_seed": 11, "long": 0, "f32": False},
        # the colocated batch of the benchmark: 256 short prompts and one of 65,536 tokens
        {"name": "packed_256_long", "kind": "packed", "hq": 32, "hkv": 8, "n": 256, "len_seed": synth.VARLEN_SEED,
         "long": synth.VARLEN_LONG, "f32": False},
        # 256 short prompts batched with the decode step of a request that has 524,288 cached tokens
        {"name": "mixed_256_512k", "kind": "mixed", "hq": 32, "hkv": 8, "n": 256, "len_seed": synth.VARLEN_SEED,
         "n_dec": 1, "cache": 524288, "f32": False},
        # one token of a request with a short cache: launches and latency
        {"name": "decode_4k", "kind": "decode", "hq": 32, "hkv": 8, "sk": 4096, "f32": False},
        # one token of a request with 524,288 cached tokens, fp32 partial for the merge over GPUs: memory bandwidth
        {"name": "decode_512k", "kind": "decode", "hq": 64, "hkv": 8, "sk": 524288, "f32": True},
        # a segment of 16,384 tokens and 64 heads packed for eight GPUs and unpacked again
        {"name": "exchange_16k", "kind": "exchange", "h": 64, "gpus": 8, "s": 16384},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads, KV heads): the configurations of the benchmark and what tensor parallelism leaves of them on one GPU
_HEADS = ((8, 8), (32, 8), (64, 8), (16, 4), (8, 2), (8, 1), (4, 1))


def draw(rng):
    kind = rng.choice(("member", "sweep", "steps", "partials", "packed", "mixed", "decode", "exchange"))
    hq, hkv = rng.choice(_HEADS)
    f32 = rng.random() < 0.25
    if kind in ("member", "sweep", "steps"):
        chunk = max(64, _log(rng, 256, 8192) // 64 * 64)
        parts = rng.randint(1, 16)
        r = rng.randrange(parts)
        s_kv = parts * chunk - rng.choice((0, 0, rng.randrange(chunk // 2)))      # the last segment may be short
        q_off = r * chunk
        s_q = min(chunk, s_kv - q_off)
        return {"kind": kind, "hq": hq, "hkv": hkv, "s_q": s_q, "q_off": q_off, "s_kv": s_kv, "chunk": chunk,
                "causal": rng.random() < 0.9, "f32": f32}
    if kind == "partials":
        s_a, s_b = _log(rng, 256, 8192), _log(rng, 256, 8192)
        s_q = min(_log(rng, 256, 8192), s_b)
        return {"kind": kind, "hq": hq, "hkv": hkv, "s_q": s_q, "q_off": s_a + s_b - s_q, "s_a": s_a, "s_b": s_b,
                "causal": rng.random() < 0.5}
    if kind == "packed":
        return {"kind": kind, "hq": hq, "hkv": hkv, "n": _log(rng, 1, 256), "len_seed": rng.randrange(1 << 20),
                "long": rng.choice((0, 0, _log(rng, 8192, 65536))), "f32": f32}
    if kind == "mixed":
        return {"kind": kind, "hq": hq, "hkv": hkv, "n": _log(rng, 1, 256), "len_seed": rng.randrange(1 << 20),
                "n_dec": rng.randint(1, 4), "cache": _log(rng, 2048, 524288), "f32": f32}
    if kind == "decode":
        return {"kind": kind, "hq": hq, "hkv": hkv, "sk": _log(rng, 1024, 524288), "f32": f32}
    gpus = rng.choice((2, 4, 8))
    return {"kind": kind, "h": rng.choice((8, 16, 32, 64)), "gpus": gpus, "s": _log(rng, 256, 32768)}


def _lengths(case):
    """Query and key lengths of the sequences of a packed or mixed batch."""
    n = synth.lognormal_lengths(case["len_seed"], case["n"])
    if case["kind"] == "packed":
        if case["long"]:
            n = np.concatenate([n, [case["long"]]])
        return n, n
    caches = [case["cache"] // (i + 1) for i in range(case["n_dec"])]
    return np.concatenate([n, [1] * len(caches)]), np.concatenate([n, caches])


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": dict(case)}
    if kind == "exchange":
        h, g, s = case["h"], case["gpus"], case["s"]
        st["x"] = synth.randn_bf16((s, h, ROW), seed, DEV)
        st["y"] = torch.empty((g, s, h // g, ROW), dtype=torch.bfloat16, device=DEV)
        st["z"] = torch.empty_like(st["x"])
        return st
    hq, hkv = case["hq"], case["hkv"]
    if kind == "decode":
        n_q, n_k = 1, case["sk"]
    elif kind == "partials":
        n_q, n_k = case["s_q"], case["s_a"] + case["s_b"]
    elif kind in ("packed", "mixed"):
        len_q, len_k = _lengths(case)
        cu_q, cu_k = synth.cu_seqlens_of(len_q), synth.cu_seqlens_of(len_k)
        n_q, n_k = int(cu_q[-1]), int(cu_k[-1])
        st["cu_q"], st["cu_k"] = torch.from_numpy(cu_q).to(DEV), torch.from_numpy(cu_k).to(DEV)
        st["max_len"] = int(len_q.max())
    else:
        n_q, n_k = case["s_q"], case["s_kv"]
    q, k, v = synth.qkv(seed, n_q, n_k, hq, hkv, device=DEV)
    st.update(q=q, k=k, v=v)
    st["dtype"] = torch.float32 if case.get("f32") else torch.bfloat16
    st["out"] = torch.empty((n_q, hq, ROW), dtype=st["dtype"], device=DEV)
    st["lse"] = torch.empty((hq, n_q) if kind != "decode" else (hq,), dtype=torch.float32, device=DEV)
    if kind == "member":
        st["ws"] = torch.empty(max(16, pec.pec_sp_workspace_bytes(hq, hkv, n_q)), dtype=torch.uint8, device=DEV)
    elif kind == "sweep":
        st["ws"] = torch.empty(pec.pec_sp_resumable_workspace_bytes(q, k), dtype=torch.uint8, device=DEV)
        st["stop"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        st["pending"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    elif kind == "steps":
        st["o_acc"] = torch.empty((n_q, hq, ROW), dtype=torch.float32, device=DEV)
        st["n_steps"] = pec.pec_sp_prefill_num_steps(q, k, case["q_off"], case["chunk"], case["causal"])
    elif kind == "partials":
        st["o"] = [torch.empty((n_q, hq, ROW), dtype=torch.float32, device=DEV) for _ in range(2)]
        st["l"] = [torch.empty((hq, n_q), dtype=torch.float32, device=DEV) for _ in range(2)]
        s_a = case["s_a"]
        st["kv"] = [(k[:s_a], v[:s_a], 0), (k[s_a:], v[s_a:], s_a)]
    elif kind == "packed":
        st["ws"] = torch.empty(pec.pec_varlen_workspace_bytes(len(len_q), n_q), dtype=torch.uint8, device=DEV)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "exchange":
        pec.pec_ulysses_layout(state["x"], case["gpus"], True, out=state["y"])
        pec.pec_ulysses_layout(state["y"], case["gpus"], False, out=state["z"])
        return state["y"], state["z"]
    q, k, v, out, lse = state["q"], state["k"], state["v"], state["out"], state["lse"]
    if kind == "member":
        pec.pec_sp_prefill(q, k, v, case["q_off"], case["chunk"], case["causal"], out_dtype=state["dtype"], out=out,
                           lse=lse, workspace=state["ws"])
    elif kind == "sweep":
        pec.pec_sp_prefill_resumable(q, k, v, case["q_off"], case["chunk"], out, lse, state["ws"], state["pending"],
                                     stop=state["stop"], causal=case["causal"])
        return out, lse, state["pending"]
    elif kind == "steps":
        last = state["n_steps"] - 1
        for t in range(last + 1):
            pec.pec_sp_prefill_step(q, k, v, case["q_off"], case["chunk"], t, state["o_acc"], lse, case["causal"],
                                    out_final=out if t == last else None)
    elif kind == "partials":
        for (ks, vs, off), o, l in zip(state["kv"], state["o"], state["l"]):
            pec.pec_attn_chunk(q, ks, vs, case["q_off"], off, case["causal"], out_dtype=torch.float32, out=o, lse=l)
        pec.pec_attn_merge(state["o"][0], state["l"][0], state["o"][1], state["l"][1])
        pec.pec_finalize(state["o"][0], out)
        return out, state["o"][0], state["l"][0], state["o"][1], state["l"][1]
    elif kind == "packed":
        pec.pec_attn_varlen(q, k, v, state["cu_q"], state["max_len"], True, out_dtype=state["dtype"], out=out, lse=lse,
                            workspace=state["ws"])
    elif kind == "mixed":
        pec.pec_attn_colocated(q, k, v, state["cu_q"], state["cu_k"], True, out_dtype=state["dtype"], out=out, lse=lse)
    else:
        pec.pec_decode_splitkv(q, k, v, out_dtype=state["dtype"], out=out, lse=lse)
    return out, lse


def work(case):
    kind = case["kind"]
    if kind == "exchange":
        return {"bytes": 2 * 2.0 * 2 * case["s"] * case["h"] * ROW, "flops": 0.0}
    hq, hkv = case["hq"], case["hkv"]
    kv_row, q_row = 2.0 * 2 * hkv * ROW, hq * ROW
    out_b = 4.0 if case.get("f32") else 2.0
    if kind == "decode":
        n_q, n_k, pairs = 1, case["sk"], case["sk"]
    elif kind == "partials":
        n_q, n_k = case["s_q"], case["s_a"] + case["s_b"]
        pairs = sum(synth.visible_pairs(n_q, n, case["q_off"], off, case["causal"])
                    for n, off in ((case["s_a"], 0), (case["s_b"], case["s_a"])))
        out_b = 2.0 + 4.0 + 4.0       # bf16 result, merged fp32 result, second fp32 partial
    elif kind in ("packed", "mixed"):
        len_q, len_k = _lengths(case)
        n_q, n_k = int(len_q.sum()), int(len_k.sum())
        pairs = sum(synth.visible_pairs(int(a), int(b), int(b - a), 0, True) for a, b in zip(len_q, len_k))
    else:
        n_q = case["s_q"]
        n_k = min(case["s_kv"], case["q_off"] + n_q) if case["causal"] else case["s_kv"]
        pairs = synth.visible_pairs(n_q, case["s_kv"], case["q_off"], 0, case["causal"])
    return {"bytes": n_k * kv_row + n_q * (q_row * (2.0 + out_b) + 4.0 * hq), "flops": FLOP_PER_PAIR * hq * pairs}


def tolerance(case):
    if case["kind"] == "exchange":
        return "exact"
    # The weights are rounded to bf16 before the second product and most results to bf16 once more.  Measured: the default
    # and the plain kernel differ by 1.6e-3 ... 3.1e-3 (largest single difference 3e-2), each from fp64 by as much.
    return {"rel": 1e-2, "max": 0.12}
