"""Workloads by which the speed of the attention-layer path is measured.

`listed()` names twelve of them and `draw()` picks more from the same ranges; `prepare()` makes what a serving program
holds before the call (activations, paged cache, weights, workspace), `run()` is one pass through the public entry points
of `paper_2509_16495_amd.binding`.  A case is a dict of plain values; its `kind` says which path it takes:

  step_f32   fp32 shard: pack, causal prefill with K/V append, unpack
  decode     one new token per sequence with K/V append, bf16 or FP8 cache
  prefill    prompts, or chunks behind cached tokens, with K/V append, bf16 or FP8 cache
  mixed      a chunked-prefill engine's step: pack, unified batch (chunks + decode rows) with K/V append, unpack
  exchange   both local layout transforms of the sequence <-> head exchange
  proj       q|k|v projection into the send buffers and output projection out of the receive buffers, bf16 or FP8 operands
             (with FP8 operands the activations are quantised in the pass)

Head geometries are those of the models the repository serves (64q/8kv, 40q/8kv, 32q/8kv, 32q/4kv, head_dim 128) split
over P GPUs.  Sequence lengths come from the case's own `lens_seed`, so every preparation of a case has the same amount
of work; values and block tables come from the preparation's seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2509_16495_amd import binding as B

BLOCK = B.BLOCK_SIZE
DEVICE = "cuda:0"
KV_SCALE = 5.0 / 448.0  # FP8 cache: the largest of some million N(0, 1) values lands on the largest code

# (query heads, KV heads, d_model) of the served models
MODELS = ((64, 8, 8192), (64, 8, 5120), (40, 8, 5120), (32, 8, 4096), (32, 4, 2048))


def listed():
    return [
        # the smallest call of the repository's configurations: launches and host path are all there is to it
        dict(name="fp32_shard_256", kind="step_f32", seqs=1, len_lo=256, len_hi=256, hq=4, hkv=1, D=64, P=2, lens_seed=1),
        # interactive decoding (the shift configuration's side of the switch): a handful of sequences, latency counts
        dict(name="decode_4_seqs", kind="decode", seqs=4, ctx_lo=1900, ctx_hi=6300, hq=8, hkv=1, kv="bf16", lens_seed=2),
        # throughput decoding of a 70B shard
        dict(name="decode_256_seqs", kind="decode", seqs=256, ctx_lo=512, ctx_hi=8192, hq=8, hkv=1, kv="bf16", lens_seed=4),
        # conversation serving over an FP8 cache: one chunk continues a prompt while other sequences decode
        dict(name="fp8_kv_step", kind="mixed", chunks=1, chunk=1000, cached=20000, decs=97, ctx_lo=1000, ctx_hi=16000,
             P=8, h=64, h_kv=8, kv="fp8", lens_seed=5),
        # a batch of equal prompts on an 8B shard
        dict(name="prefill_8b_4x4096", kind="prefill", seqs=4, len_lo=4096, len_hi=4096, cached=0, hq=4, hkv=1, kv="bf16", lens_seed=6),
        # one long prompt on a 70B shard
        dict(name="prefill_70b_16384", kind="prefill", seqs=1, len_lo=16384, len_hi=16384, cached=0, hq=8, hkv=1, kv="bf16", lens_seed=7),
        # ordinary traffic: short prompts of all lengths, five query heads per KV head
        dict(name="prefill_short_prompts", kind="prefill", seqs=11, len_lo=60, len_hi=1500, cached=0, hq=5, hkv=1, kv="bf16", lens_seed=8),
        # long context: a 2048-token chunk on 131072 cached tokens next to 64 decodes
        dict(name="long_context_step", kind="mixed", chunks=1, chunk=2048, cached=131072, decs=64, ctx_lo=1024, ctx_hi=32768,
             P=8, h=64, h_kv=8, kv="bf16", lens_seed=9),
        # the exchange's layouts at the size of a large prefill
        dict(name="exchange_16384", kind="exchange", P=8, h=64, h_kv=0, D=128, dtype="bf16", T=16384, pad=0),
        # projections of a large prefill
        dict(name="proj_16384_bf16", kind="proj", T=16384, pad=0, P=8, h=64, h_kv=8, d_model=8192, dtype="bf16"),
        # projections of a decode step
        dict(name="proj_19_rows_bf16", kind="proj", T=19, pad=0, P=8, h=64, h_kv=8, d_model=8192, dtype="bf16"),
        # projections of a chunked-prefill step with FP8 weights, ragged
        dict(name="proj_701_rows_fp8", kind="proj", T=701, pad=1, P=8, h=64, h_kv=8, d_model=5120, dtype="fp8"),
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step_f32", "decode", "decode", "prefill", "prefill", "prefill", "mixed", "mixed", "exchange", "proj", "proj", "proj"])
    seed = rng.randrange(1 << 30)
    hq, hkv = rng.choice([(8, 1), (8, 1), (4, 1), (5, 1), (16, 2), (10, 2)])  # heads per GPU of the served models
    kv = rng.choice(["bf16", "bf16", "fp8"])
    if kind == "step_f32":
        P = rng.choice([1, 2, 4])
        n = _log_int(rng, 48, 700)
        return dict(kind=kind, seqs=rng.randint(1, 3), len_lo=n - n // 4, len_hi=n, hq=4, hkv=1, D=rng.choice([64, 64, 128]), P=P, lens_seed=seed)
    if kind == "decode":
        seqs = _log_int(rng, 1, 400)
        hi = min(_log_int(rng, 300, 33000), 2_200_000 // (seqs * hkv))  # at most about 1.1 GB of bf16 K and V
        return dict(kind=kind, seqs=seqs, ctx_lo=max(1, hi // rng.choice([2, 4, 16])), ctx_hi=hi, hq=hq, hkv=hkv, kv=kv, lens_seed=seed)
    if kind == "prefill":
        hi = _log_int(rng, 40, 14000)
        seqs = rng.randint(1, max(1, min(12, 24000 // hi)))
        cached = rng.choice([0, 0, 0, _log_int(rng, 100, 30000)])
        if cached:
            hi = min(hi, 3000)
            seqs = min(seqs, 4)
        return dict(kind=kind, seqs=seqs, len_lo=max(1, hi // rng.choice([1, 2, 8])), len_hi=hi, cached=cached, hq=hq, hkv=hkv, kv=kv, lens_seed=seed)
    if kind == "mixed":
        h, h_kv, _ = rng.choice(MODELS)
        chunk = _log_int(rng, 100, 2048)
        decs = _log_int(rng, 2, 128)
        hi = min(_log_int(rng, 500, 30000), 2_000_000 // decs)
        return dict(kind=kind, chunks=rng.choice([1, 1, 2]), chunk=chunk, cached=_log_int(rng, 1000, 60000), decs=decs,
                    ctx_lo=max(1, hi // 8), ctx_hi=hi, P=8, h=h, h_kv=h_kv, kv=kv, lens_seed=seed)
    if kind == "exchange":
        h, h_kv, _ = rng.choice(MODELS)
        P = rng.choice([2, 4, 8])
        return dict(kind=kind, P=P, h=h, h_kv=rng.choice([0, h_kv]), D=128, dtype=rng.choice(["bf16", "bf16", "f32"]),
                    T=_log_int(rng, 2, 6000), pad=rng.choice([0, 1]))
    h, h_kv, d_model = rng.choice(MODELS)
    if rng.random() < 0.25 and h != 40:  # the shift configuration: this GPU's head shard of the weights, nothing to exchange
        h, h_kv, P = h // 8, 1, 1
    else:
        P = rng.choice([4, 8, 8])
    return dict(kind="proj", T=_log_int(rng, 1, 8192), pad=0 if P == 1 else rng.choice([0, 1]), P=P, h=h, h_kv=h_kv, d_model=d_model,
                dtype=rng.choice(["bf16", "fp8"]))


# ---- sizes of a case ---------------------------------------------------------------------------------------------------
def _lengths(case):
    """(query tokens, context tokens) per sequence; chunks and prompts first, then decode rows."""
    r = random.Random(case["lens_seed"])
    kind = case["kind"]
    if kind == "decode":
        return [(1, r.randint(case["ctx_lo"], case["ctx_hi"])) for _ in range(case["seqs"])]
    if kind == "mixed":
        return ([(case["chunk"], case["chunk"] + case["cached"]) for _ in range(case["chunks"])] +
                [(1, r.randint(case["ctx_lo"], case["ctx_hi"])) for _ in range(case["decs"])])
    lens = [r.randint(case["len_lo"], case["len_hi"]) for _ in range(case["seqs"])]
    return [(n, n + case.get("cached", 0)) for n in lens]


def _heads(case):
    if case["kind"] == "mixed":
        return case["h"] // case["P"], B.local_kv_heads(case["P"], case["h_kv"])
    return case["hq"], case["hkv"]


def _attention_work(case):
    hq, hkv = _heads(case)
    D = case.get("D", 128)
    e = 4 if case["kind"] == "step_f32" else 2
    ekv = 1 if case.get("kv") == "fp8" else e
    by = fl = 0
    for n, ctx in _lengths(case):
        fl += 4 * D * hq * (n * (ctx - n) + n * (n + 1) // 2)
        by += n * (2 * hq + 2 * hkv) * D * e            # q, new K/V read, output written
        by += (ctx - n) * 2 * hkv * D * ekv + n * 2 * hkv * D * ekv  # cached K/V read, new K/V written to the cache
    return by, fl


def _exchange_bytes(P, h, h_kv, D, e, T, T_pad):
    hq_l, hkv_l = h // P, B.local_kv_heads(P, h_kv)
    pack = T * (h + 2 * h_kv) * D * e + P * T_pad * (hq_l + 2 * hkv_l) * D * e
    return pack + 2 * T * h * D * e


def work(case):
    kind = case["kind"]
    if kind == "proj":
        T, d, N, K = case["T"], case["d_model"], (case["h"] + 2 * case["h_kv"]) * 128, case["h"] * 128
        Tp = T + case["pad"]
        send = case["P"] * Tp * (case["h"] // case["P"] + 2 * B.local_kv_heads(case["P"], case["h_kv"])) * 128
        ew = 1 if case["dtype"] == "fp8" else 2
        by = (N * d + d * K) * ew + (T * d + T * K) * 2 + send * 2 + T * d * 2
        if ew == 1:
            by += T * d + T * K + 8 * T + (N + d) * 4  # codes and scales are results too
        return {"bytes": by, "flops": 2 * T * d * (N + K)}
    if kind == "exchange":
        e = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": _exchange_bytes(case["P"], case["h"], case["h_kv"], case["D"], e, case["T"], case["T"] + case["pad"]), "flops": 0}
    by, fl = _attention_work(case)
    if kind == "mixed":
        T = _rank_rows(case)
        by += _exchange_bytes(case["P"], case["h"], case["h_kv"], 128, 2, T, T)
    if kind == "step_f32":
        T = _total_rows(case)
        by += _exchange_bytes(case["P"], case["hq"] * case["P"], 0, case["D"], 4, T, T)
    return {"bytes": by, "flops": fl}


def _total_rows(case):
    return sum(n for n, _ in _lengths(case))


def _rank_rows(case):
    """Rows this rank holds of the step's (padded) batch before the exchange."""
    return B.padded_tokens(_total_rows(case), case["P"]) // case["P"]


# Errors measured against float64 on the same inputs, times about four.  Measured (relative 2-norm / largest): fp32 attention
# 2.5e-7 / 2.7e-6; projections 1.7e-3 / 3.9e-3 (one rounding to bf16); bf16 attention 2.0e-3 .. 2.3e-3 / 6e-3 .. 4e-2 (the
# same rounding, and P rounded to bf16 in front of P.V).  Integer outputs (FP8 caches, codes) are exact.
def tolerance(case):
    if case["kind"] == "exchange":
        return "exact"
    if case["kind"] == "step_f32":
        return {"rel": 2e-6, "max": 2.5e-5}
    if case["kind"] == "proj":
        return {"rel": 7e-3, "max": 0.02}
    return {"rel": 9e-3, "max": 0.16}


# ---- preparation -------------------------------------------------------------------------------------------------------
def _normal(shape, dtype, gen, std=1.0):
    return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=gen)


def _fp8_codes(shape, scale, gen):
    n = int(np.prod(shape))
    out = torch.empty(n, dtype=torch.uint8, device=DEVICE)
    step = 1 << 26
    for i in range(0, n, step):
        x = _normal((min(step, n - i),), torch.float32, gen).div_(scale).clamp_(-448.0, 448.0)
        out[i:i + step] = x.to(torch.float8_e4m3fn).view(torch.uint8)
    return out.view(shape)


def _prepare_attention(case, seed, gen):
    lens = _lengths(case)
    hq, hkv = _heads(case)
    D = case.get("D", 128)
    dtype = torch.float32 if case["kind"] == "step_f32" else torch.bfloat16
    fp8 = case.get("kv") == "fp8"
    pool = np.random.RandomState(seed & 0x7FFFFFFF)
    blocks = [(c + BLOCK - 1) // BLOCK for _, c in lens]
    num_blocks = max(sum(blocks) + sum(blocks) // 8, 1)
    ids = pool.permutation(num_blocks).astype(np.int32)
    table = np.full((len(lens), max(blocks)), -1, dtype=np.int32)
    slots, at = [], 0
    for s, (n, c) in enumerate(lens):
        table[s, :blocks[s]] = ids[at:at + blocks[s]]
        at += blocks[s]
        t = np.arange(c - n, c, dtype=np.int64)
        slots.append(table[s, t // BLOCK].astype(np.int64) * BLOCK + t % BLOCK)
    cache_shape = (num_blocks, hkv, 2, BLOCK * D)
    st = {"kind": case["kind"], "scale": 1.0 / math.sqrt(D), "kv_scale": KV_SCALE if fp8 else 1.0}
    st["cache"] = _fp8_codes(cache_shape, KV_SCALE, gen) if fp8 else _normal(cache_shape, dtype, gen)
    total = sum(n for n, _ in lens)
    rows = _normal((total, hq + 2 * hkv, D), dtype, gen)  # the fused rows the exchange delivers
    st["q"], st["k"], st["v"] = rows[:, :hq], rows[:, hq:hq + hkv], rows[:, hq + hkv:]
    st["table"] = torch.from_numpy(table).to(DEVICE)
    st["slots"] = torch.from_numpy(np.concatenate(slots)).to(DEVICE)
    st["seq_lens"] = torch.tensor([c for _, c in lens], dtype=torch.int32, device=DEVICE)
    st["out"] = torch.empty((total, hq, D), dtype=dtype, device=DEVICE)
    desc = B.attn_desc(st["q"], st["cache"], st["table"], st["scale"], st["k"], st["out"], st["kv_scale"], st["kv_scale"])
    if case["kind"] == "decode":
        st["max_ctx"] = max(c for _, c in lens)
        need = B.decode_workspace_bytes(len(lens), st["max_ctx"], desc)
    else:
        n_pre = case["chunks"] if case["kind"] == "mixed" else len(lens)
        pre, dec = lens[:n_pre], lens[n_pre:]
        st["n_pre"] = n_pre
        st["cu"] = torch.tensor(np.concatenate([[0], np.cumsum([n for n, _ in pre])]), dtype=torch.int32, device=DEVICE)
        st["max_q"], st["max_pre"] = max(n for n, _ in pre), max(c for _, c in pre)
        if case["kind"] == "mixed":
            st["max_ctx"] = max(c for _, c in dec)
            need = B.mixed_workspace_bytes(n_pre, sum(n for n, _ in pre), st["max_q"], st["max_pre"], len(dec), st["max_ctx"], desc)
        else:
            need = B.prefill_workspace_bytes(len(pre), total, st["max_q"], st["max_pre"], desc)
    st["ws"] = torch.empty(need, dtype=torch.uint8, device=DEVICE) if need else None
    return st


def _prepare_exchange(P, h, h_kv, D, dtype, T, T_pad, gen):
    return {"P": P, "h": h, "h_kv": h_kv,
            "rows": _normal((T, h + 2 * h_kv, D), dtype, gen),
            "send": torch.empty((P, T_pad, h // P + 2 * B.local_kv_heads(P, h_kv), D), dtype=dtype, device=DEVICE),
            "recv": _normal((P, T_pad, h // P, D), dtype, gen),
            "seq": torch.empty((T, h, D), dtype=dtype, device=DEVICE)}


def _prepare_proj(case, gen):
    P, h, h_kv, d, T = case["P"], case["h"], case["h_kv"], case["d_model"], case["T"]
    Tp, N, K = T + case["pad"], (h + 2 * h_kv) * 128, h * 128
    fp8 = case["dtype"] == "fp8"
    st = {"kind": "proj", "fp8": fp8, "P": P, "h": h, "h_kv": h_kv}
    st["x"] = _normal((T, d), torch.bfloat16, gen)
    st["recv"] = _normal((P, Tp, h // P, 128), torch.bfloat16, gen)
    w_qkv, w_o = _normal((N, d), torch.bfloat16, gen, 0.02), _normal((d, K), torch.bfloat16, gen, 0.02)
    st["send"] = torch.empty((P, Tp, h // P + 2 * B.local_kv_heads(P, h_kv), 128), dtype=torch.bfloat16, device=DEVICE)
    st["out"] = torch.empty((T, d), dtype=torch.bfloat16, device=DEVICE)
    if fp8:  # a checkpoint's weights are quantised once, when they are loaded
        for name, w in (("qkv", w_qkv), ("o", w_o)):
            st["w_" + name] = torch.empty(w.shape, dtype=torch.uint8, device=DEVICE)
            st["ws_" + name] = torch.empty(w.shape[0], dtype=torch.float32, device=DEVICE)
            B.quantize_rows_fp8(w, st["w_" + name], st["ws_" + name])
        st["xc"] = torch.empty((T, d), dtype=torch.uint8, device=DEVICE)
        st["xs"] = torch.empty(T, dtype=torch.float32, device=DEVICE)
        st["rc"] = torch.zeros(st["recv"].shape, dtype=torch.uint8, device=DEVICE)
        st["rs"] = torch.empty(T, dtype=torch.float32, device=DEVICE)
    else:
        st["w_qkv"], st["w_o"] = w_qkv, w_o
    need = max(B.proj_workspace_bytes(Tp, N, d, fp8), B.proj_workspace_bytes(T, d, K, fp8))
    st["ws"] = torch.empty(need, dtype=torch.uint8, device=DEVICE) if need else None
    return st


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "proj":
        return _prepare_proj(case, gen)
    if kind == "exchange":
        st = _prepare_exchange(case["P"], case["h"], case["h_kv"], case["D"], torch.bfloat16 if case["dtype"] == "bf16" else torch.float32,
                               case["T"], case["T"] + case["pad"], gen)
        st["kind"] = kind
        return st
    st = _prepare_attention(case, seed, gen)
    if kind == "mixed":
        T = _rank_rows(case)
        st["xchg"] = _prepare_exchange(case["P"], case["h"], case["h_kv"], 128, torch.bfloat16, T, T, gen)
    if kind == "step_f32":
        T = _total_rows(case)
        st["xchg"] = _prepare_exchange(case["P"], case["hq"] * case["P"], 0, case["D"], torch.float32, T, T, gen)
    return st


# ---- one pass ----------------------------------------------------------------------------------------------------------
def _run_proj(st):
    if st["fp8"]:
        B.quantize_rows_fp8(st["x"], st["xc"], st["xs"])
        B.qkv_proj_pack_fp8(st["xc"], st["xs"], st["w_qkv"], st["ws_qkv"], st["send"], st["P"], st["h"], st["h_kv"], st["ws"])
        B.quantize_recv_fp8(st["recv"], st["rc"], st["rs"])
        B.unpack_o_proj_fp8(st["rc"], st["rs"], st["w_o"], st["ws_o"], st["out"], st["ws"])
        return {"send": st["send"], "out": st["out"], "x_codes": st["xc"], "x_scales": st["xs"], "recv_codes": st["rc"], "recv_scales": st["rs"]}
    B.qkv_proj_pack(st["x"], st["w_qkv"], st["send"], st["P"], st["h"], st["h_kv"], st["ws"])
    B.unpack_o_proj(st["recv"], st["w_o"], st["out"], st["ws"])
    return {"send": st["send"], "out": st["out"]}


def run(state):
    st = state
    kind = st["kind"]
    if kind == "proj":
        return _run_proj(st)
    if kind == "exchange":
        B.pack_seq2head(st["rows"], st["send"], st["P"], st["h"], st["h_kv"])
        B.unpack_head2seq(st["recv"], st["seq"])
        return {"send": st["send"], "seq": st["seq"]}
    x = st.get("xchg")
    if x is not None:
        B.pack_seq2head(x["rows"], x["send"], x["P"], x["h"], x["h_kv"])
    new = dict(k_new=st["k"], v_new=st["v"], slot_mapping=st["slots"], workspace=st["ws"], k_scale=st["kv_scale"], v_scale=st["kv_scale"])
    if kind == "decode":
        B.decode(st["q"], st["cache"], st["table"], st["seq_lens"], st["max_ctx"], st["out"], st["scale"], **new)
    elif kind == "mixed":
        B.mixed(st["q"], st["cache"], st["table"], st["cu"], st["seq_lens"], st["n_pre"], st["max_q"], st["max_pre"], st["max_ctx"],
                st["out"], st["scale"], **new)
    else:
        B.prefill(st["q"], st["cache"], st["table"], st["cu"], st["seq_lens"], st["max_q"], st["max_pre"], st["out"], st["scale"], **new)
    res = {"out": st["out"], "cache": st["cache"]}
    if x is not None:
        B.unpack_head2seq(x["recv"], x["seq"])
        res["send"], res["seq"] = x["send"], x["seq"]
    return res
