"""Measured cases: the calls a program that serves from an L2-norm compressed KV cache makes, at
the shapes of this repository's workloads (``paper_2406_11430_amd/synth.py``) and over the range
around them.

Six kinds of pass, each through the public binding:

``path``      one small layer from prompt to output: compress, then attend to what was kept
``compress``  the step after a prefill: norms, selection and compaction of K and V
``decode``    one layer of one decode step over the compacted cache
``prompt``    the step after the prefill of a ragged batch: norms, selection, compaction into slots
``stream``    one decode step of a ragged batch at its budget: append, attend in every layer, evict
``loss``      the attention-loss analysis of one layer: discard order, then losses of every query head

All caches follow the recipe of ``synth.py``: rows ``s*g`` with ``g ~ N(0,1)``, ``s = exp(z/2)``, a
few low-norm tokens at the start of every sequence; values and queries ``N(0,1)``.
"""
from __future__ import annotations

import math

import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding as api

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
# rows the library supports, and the largest query group each one takes
ROWS = [("bf16", 128, 8), ("bf16", 64, 8), ("bf16", 256, 4), ("f32", 128, 8), ("f32", 64, 8)]
SINK_TOKENS, SINK_SCALE = 4, 0.1
STREAM_STEPS = 8            # prepared decode steps a streaming pass cycles through


# ---------------------------------------------------------------------------- the cases
def listed():
    return [
        # smallest call of the framework: the fp32 toy layer, where launches are all there is
        {"name": "path_tiny_f32", "kind": "path", "dtype": "f32", "B": 1, "Hkv": 4, "Hq": 4, "D": 64,
         "T": 512, "keep": 0.5},
        # one multi-head layer of a 7B model after a 4k prompt
        {"name": "compress_layer_4k", "kind": "compress", "dtype": "bf16", "L": 1, "B": 1, "Hkv": 32,
         "D": 128, "T": 4096, "keep": 0.5, "strategy": "lowest"},
        # one layer after a 131k prompt, nine tenths dropped: few heads, very long
        {"name": "compress_layer_131k", "kind": "compress", "dtype": "bf16", "L": 1, "B": 1, "Hkv": 8,
         "D": 128, "T": 131072, "keep": 0.1, "strategy": "lowest"},
        # eight layers of an 8B model, batch of four 32k prompts, compressed together
        {"name": "compress_stack_32k", "kind": "compress", "dtype": "bf16", "L": 8, "B": 4, "Hkv": 8,
         "D": 128, "T": 32768, "keep": 0.5, "strategy": "lowest"},
        # one decode layer of the 7B model after the 4k prompt: short rows, latency counts
        {"name": "decode_2k_mha", "kind": "decode", "dtype": "bf16", "B": 1, "Hkv": 32, "Hq": 32, "D": 128,
         "n": 2048, "out": "f32"},
        # one decode layer after the 131k prompt: a single sequence, few KV heads
        {"name": "decode_13k_single", "kind": "decode", "dtype": "bf16", "B": 1, "Hkv": 8, "Hq": 32, "D": 128,
         "n": 13108, "out": "f32"},
        # one decode layer of the 8B model's batch at 32k context: the headline launch
        {"name": "decode_16k_batch", "kind": "decode", "dtype": "bf16", "B": 4, "Hkv": 8, "Hq": 32, "D": 128,
         "n": 16384, "out": "f32"},
        # multi-head layer with 256-element heads, odd length, output in the model's own type
        {"name": "decode_4k_wide_heads", "kind": "decode", "dtype": "bf16", "B": 4, "Hkv": 16, "Hq": 16,
         "D": 256, "n": 4001, "out": "bf16"},
        # an fp32 cache of odd length
        {"name": "decode_5k_f32", "kind": "decode", "dtype": "f32", "B": 2, "Hkv": 8, "Hq": 32, "D": 128,
         "n": 5003, "out": "f32"},
        # one layer of the streaming batch after its prompts: 64 sequences of 1k to 8k tokens
        {"name": "prompt_ragged_64", "kind": "prompt", "dtype": "bf16", "n_seq": 64, "lo": 1024, "hi": 8192,
         "Hkv": 8, "D": 128, "keep": 0.5},
        # a decode step of that batch, two layers, every sequence at its budget
        {"name": "stream_step_64", "kind": "stream", "dtype": "bf16", "L": 2, "n_seq": 64, "lo": 1024,
         "hi": 8192, "Hkv": 8, "Hq": 32, "D": 128, "keep": 0.5, "ordered": True},
        # analysis of one layer of the 32k batch, one query per head
        {"name": "loss_layer_32k", "kind": "loss", "dtype": "bf16", "B": 4, "Hkv": 8, "Hq": 32, "D": 128,
         "T": 32768, "keep": 0.5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["path", "compress", "compress", "decode", "decode", "decode", "prompt", "stream", "loss"])
    dtype, D, max_group = rng.choice([ROWS[0], ROWS[0], ROWS[0]] + ROWS)     # mostly the common row
    row = D * DTYPES[dtype].itemsize
    Hkv = rng.choice([1, 2, 4, 8, 8, 16, 32])
    group = rng.choice([g for g in (1, 2, 3, 4, 4, 5, 6, 7, 8) if g <= max_group])
    keep = rng.choice([0.1, 0.3, 0.5, 0.5, round(rng.uniform(0.05, 1.0), 3)])
    if kind == "path":
        return {"kind": kind, "dtype": dtype, "B": rng.choice([1, 1, 2, 4]), "Hkv": Hkv, "Hq": Hkv * group, "D": D,
                "T": _log_int(rng, 100, 5000), "keep": keep}
    if kind == "compress":
        T = _log_int(rng, 500, 140000)
        planes = max(1, min(256, int((5 << 30) / (T * (row * (1 + 3 * keep) + 8)))))    # L*B*Hkv: cost in range
        Hkv = min(Hkv, planes)
        B = min(_log_int(rng, 1, 8), planes // Hkv)
        return {"kind": kind, "dtype": dtype, "L": min(rng.choice([1, 1, 2, 8]), max(1, planes // (Hkv * B))), "B": B,
                "Hkv": Hkv, "D": D, "T": T, "keep": keep, "strategy": rng.choice(["lowest"] * 4 + ["highest"])}
    if kind == "decode":
        B = _log_int(rng, 1, 32)
        n = min(_log_int(rng, 200, 66000), (1 << 30) // (2 * B * Hkv * row))
        return {"kind": kind, "dtype": dtype, "B": B, "Hkv": Hkv, "Hq": Hkv * group, "D": D, "n": n,
                "out": rng.choice(["f32", "f32", "bf16"])}
    if kind in ("prompt", "stream"):
        Hkv = min(Hkv, 8)
        n_seq = _log_int(rng, 2, 96)
        hi = _log_int(rng, 300, 9000)
        case = {"kind": kind, "dtype": dtype, "n_seq": n_seq, "lo": max(8, hi // 8), "hi": hi, "Hkv": Hkv, "D": D,
                "keep": keep}
        if kind == "stream":
            case.update(L=rng.choice([1, 2]), Hq=Hkv * group, ordered=rng.random() < 0.7)
        return case
    B = rng.choice([1, 2, 4])
    Hkv = min(Hkv, 8)
    return {"kind": kind, "dtype": dtype, "B": B, "Hkv": Hkv, "Hq": Hkv * group, "D": D, "T": _log_int(rng, 500, 33000),
            "keep": keep}


# ---------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rows(g, shape, dtype, sinks=None):
    """Keys ``[..., T, D]``: a log-normal scale per row, low-norm tokens at the positions `sinks`."""
    x = torch.randn(shape, generator=g, device="cuda")
    s = torch.exp(0.5 * torch.randn(shape[:-1] + (1,), generator=g, device="cuda"))
    if sinks is not None:
        s[..., sinks, :] *= SINK_SCALE
    return (x * s).to(dtype)


def _values(g, shape, dtype):
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


def _cache(g, planes, T, D, dtype):
    """K, V ``[planes, T, D]``, drawn in pieces so that the fp32 draws stay small."""
    K = torch.empty((planes, T, D), dtype=dtype, device="cuda")
    V = torch.empty_like(K)
    step = max(1, (1 << 27) // (T * D))
    sinks = torch.arange(min(SINK_TOKENS, T), device="cuda")
    for p in range(0, planes, step):
        n = min(step, planes - p)
        K[p:p + n] = _rows(g, (n, T, D), dtype, sinks)
        V[p:p + n] = _values(g, (n, T, D), dtype)
    return K, V


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _decode_workspace(B, Hq, n, D):
    ws = _empty(api.l2kv_decode_workspace_bytes(B, Hq, n, D), torch.uint8)
    api.l2kv_decode_workspace_init(ws)
    return ws


def _ragged(case):
    """Prompt lengths of a ragged batch (one set per case), the kept counts, and the offset arrays."""
    g = torch.Generator(device="cpu")
    g.manual_seed(case["n_seq"] * 7919 + case["hi"])
    lens = torch.randint(case["lo"], case["hi"] + 1, (case["n_seq"],), generator=g, dtype=torch.int64)
    kept = torch.tensor([api.l2kv_keep_count(int(t), case["keep"]) for t in lens], dtype=torch.int64)

    def offsets(x):
        return torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(x, 0)])
    return lens, kept, offsets(lens), offsets(kept)


def _prompt(g, case, lens, offsets):
    """K, V ``[Hkv, total_tokens, D]`` of one layer of a ragged batch."""
    dtype = DTYPES[case["dtype"]]
    total = int(lens.sum())
    sinks = (offsets[:-1, None] + torch.arange(SINK_TOKENS)[None, :]).clamp(max=total - 1).flatten().cuda()
    shape = (case["Hkv"], total, case["D"])
    return _rows(g, shape, dtype, sinks), _values(g, shape, dtype)


def prepare(case, seed):
    kind, dtype, D = case["kind"], DTYPES[case["dtype"]], case["D"]
    g = _gen(seed)
    st = {"case": case}
    if kind in ("path", "compress"):
        lead = (case["B"], case["Hkv"]) if kind == "path" else (case["L"], case["B"], case["Hkv"])
        T, planes = case["T"], math.prod(lead)
        k = api.l2kv_keep_count(T, case["keep"])
        K, V = _cache(g, planes, T, D, dtype)
        st.update(K=K.view(*lead, T, D), V=V.view(*lead, T, D), norms=_empty((*lead, T), torch.float32),
                  kept=_empty((*lead, k), torch.int32), Kc=_empty((*lead, k, D), dtype), Vc=_empty((*lead, k, D), dtype),
                  k=k, select_ws=_empty(api.l2kv_select_workspace_bytes(planes, T), torch.uint8))
        if kind == "path":
            B, Hq = case["B"], case["Hq"]
            st.update(Q=_values(g, (B, Hq, D), dtype), O=_empty((B, Hq, D), torch.float32),
                      decode_ws=_decode_workspace(B, Hq, k, D))
    elif kind == "decode":
        B, Hkv, Hq, n = case["B"], case["Hkv"], case["Hq"], case["n"]
        K, V = _cache(g, B * Hkv, n, D, dtype)
        st.update(Kc=K.view(B, Hkv, n, D), Vc=V.view(B, Hkv, n, D), Q=_values(g, (B, Hq, D), dtype),
                  O=_empty((B, Hq, D), DTYPES[case["out"]]), decode_ws=_decode_workspace(B, Hq, n, D))
    elif kind == "prompt":
        lens, kept, off, out = _ragged(case)
        Hkv, slots = case["Hkv"], int(kept.sum())
        K, V = _prompt(g, case, lens, off)
        st.update(K=K, V=V, norms=_empty(K.shape[:2], torch.float32), kept=_empty((Hkv, slots), torch.int32),
                  in_off=off.cuda(), out_off=out.cuda(), max_len=int(lens.max()), max_kept=int(kept.max()),
                  Kc=_empty((Hkv, slots, D), dtype), Vc=_empty((Hkv, slots, D), dtype),
                  norms_c=_empty((Hkv, slots), torch.float32), pos_c=_empty((Hkv, slots), torch.int32))
    elif kind == "stream":
        lens, kept, off, out = _ragged(case)
        L, Hkv, Hq, n_seq = case["L"], case["Hkv"], case["Hq"], case["n_seq"]
        slot = out + torch.arange(n_seq + 1)                     # room for the token of the running step
        slots = int(slot[-1])
        st.update(Kc=torch.zeros((L * Hkv, slots, D), dtype=dtype, device="cuda"),
                  Vc=torch.zeros((L * Hkv, slots, D), dtype=dtype, device="cuda"),
                  norms_c=torch.zeros((L * Hkv, slots), device="cuda"),
                  pos_c=torch.zeros((L * Hkv, slots), dtype=torch.int32, device="cuda"))
        off_d, out_d, slot_d = off.cuda(), out.cuda(), slot.cuda()
        for l in range(L):
            K, V = _prompt(g, case, lens, off)
            norms = _empty(K.shape[:2], torch.float32)
            idx = _empty((Hkv, int(kept.sum())), torch.int32)
            part = slice(l * Hkv, (l + 1) * Hkv)
            api.l2kv_norms(K, norms)
            api.l2kv_select_ragged(norms, off_d, out_d, int(lens.max()), idx)
            api.l2kv_compact_ragged(K, V, norms, idx, off_d, out_d, int(kept.max()), slot_d, st["Kc"][part],
                                    st["Vc"][part], st["norms_c"][part], st["pos_c"][part])
        budgets = kept.to(torch.int32).cuda()
        order = None
        if case["ordered"]:
            order = _empty((n_seq,), torch.int32)
            api.l2kv_length_order(budgets, order)
        max_len = int(kept.max()) + 1
        ws = _empty(api.l2kv_decode_ragged_workspace_bytes(n_seq, Hq, max_len, D), torch.uint8)
        api.l2kv_decode_workspace_init(ws)
        st.update(slot_off=slot_d, budgets=budgets, order=order, max_len=max_len, decode_ws=ws,
                  lens=[budgets.clone(), budgets.clone()], ids=lens.to(torch.int32).cuda(), step=0,
                  Knew=_rows(g, (STREAM_STEPS, L, n_seq, Hkv, D), dtype),
                  Vnew=_values(g, (STREAM_STEPS, L, n_seq, Hkv, D), dtype),
                  Q=_values(g, (STREAM_STEPS, L, n_seq, Hq, D), dtype), O=_empty((L, n_seq, Hq, D), torch.float32))
    elif kind == "loss":
        B, Hkv, Hq, T = case["B"], case["Hkv"], case["Hq"], case["T"]
        K, _ = _cache(g, B * Hkv, T, D, dtype)
        norms = _empty((B, Hkv, T), torch.float32)
        api.l2kv_norms(K, norms.view(B * Hkv, T))
        st.update(K=K.view(B, Hkv, T, D), norms=norms, Q=_values(g, (B, Hq, D), dtype),
                  m=T - api.l2kv_keep_count(T, case["keep"]), drop_rank=_empty((B, Hkv, T), torch.int32),
                  rank_ws=_empty(api.l2kv_norm_ranks_workspace_bytes(B * Hkv, T), torch.uint8),
                  alr_ws=_empty(api.l2kv_alr_workspace_bytes(B, Hq, T), torch.uint8),
                  **{name: _empty((B, Hq), torch.float64) for name in ("alr", "loss", "loss_ref")})
    else:
        raise ValueError(kind)
    return st


# ---------------------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind in ("path", "compress"):
        if case.get("strategy") == "highest":       # the keep-highest control takes the three calls
            l2kv.l2kv_norms(st["K"], st["norms"])
            l2kv.l2kv_select_k(st["norms"], st["k"], l2kv.L2KV_KEEP_HIGHEST, st["kept"], None, st["select_ws"])
            l2kv.l2kv_compact(st["K"], st["V"], st["kept"], st["Kc"], st["Vc"])
        else:
            l2kv.l2kv_compress(st["K"], st["V"], case["keep"], st["norms"], st["kept"], st["Kc"], st["Vc"],
                               st["select_ws"])
        out = {name: st[name] for name in ("norms", "kept", "Kc", "Vc")}
        if kind == "path":
            l2kv.l2kv_decode_attn(st["Q"], st["Kc"], st["Vc"], st["O"], st["decode_ws"])
            out["O"] = st["O"]
        return out
    if kind == "decode":
        if case["out"] == "bf16":
            l2kv.l2kv_decode_attn_out(st["Q"], st["Kc"], st["Vc"], st["O"], st["decode_ws"])
        else:
            l2kv.l2kv_decode_attn(st["Q"], st["Kc"], st["Vc"], st["O"], st["decode_ws"])
        return {"O": st["O"]}
    if kind == "prompt":
        l2kv.l2kv_norms(st["K"], st["norms"])
        l2kv.l2kv_select_ragged(st["norms"], st["in_off"], st["out_off"], st["max_len"], st["kept"])
        l2kv.l2kv_compact_ragged(st["K"], st["V"], st["norms"], st["kept"], st["in_off"], st["out_off"], st["max_kept"],
                                 st["out_off"], st["Kc"], st["Vc"], st["norms_c"], st["pos_c"])
        return {name: st[name] for name in ("norms", "kept", "Kc", "Vc", "norms_c", "pos_c")}
    if kind == "stream":
        i = st["step"] % STREAM_STEPS
        st["step"] += 1
        cur, grown = st["lens"]
        cache = (st["Kc"], st["Vc"], st["norms_c"], st["pos_c"])
        l2kv.l2kv_stream_append(st["Knew"][i], st["Vnew"][i], st["ids"], st["slot_off"], cur, grown, *cache)
        Hkv = case["Hkv"]
        for l in range(case["L"]):
            part = slice(l * Hkv, (l + 1) * Hkv)
            l2kv.l2kv_decode_attn_ragged(st["Q"][i, l], st["Kc"][part], st["Vc"][part], grown, st["slot_off"],
                                         st["max_len"], st["O"][l], st["decode_ws"], seq_order=st["order"])
        l2kv.l2kv_stream_evict(st["slot_off"], grown, st["budgets"], cur, *cache)
        st["ids"] += 1
        return {"O": st["O"], "lens": cur, "Kc": st["Kc"], "Vc": st["Vc"], "norms_c": st["norms_c"], "pos_c": st["pos_c"]}
    l2kv.l2kv_norm_ranks(st["norms"], st["drop_rank"], st["rank_ws"])
    l2kv.l2kv_alr(st["Q"], st["K"], st["drop_rank"], st["m"], st["alr"], st["loss"], st["loss_ref"], st["alr_ws"])
    return {name: st[name] for name in ("drop_rank", "alr", "loss", "loss_ref")}


# ---------------------------------------------------------------------------- what a pass cannot do without
def _mean_total(case):
    return case["n_seq"] * (case["lo"] + case["hi"]) / 2


def work(case):
    row = case["D"] * DTYPES[case["dtype"]].itemsize
    kind, D = case["kind"], case["D"]
    if kind in ("path", "compress"):
        planes = case.get("L", 1) * case["B"] * case["Hkv"]
        T = case["T"]
        k = max(1, math.ceil(case["keep"] * T - 1e-6))
        # K once, the kept rows of V, both dense caches, norms and indices
        b = planes * ((T + 3 * k) * row + 4 * T + 4 * k)
        f = 2 * planes * T * D
        if kind == "path":
            b += planes * 2 * k * row + case["B"] * case["Hq"] * (row + 4 * D)
            f += 4 * case["B"] * case["Hq"] * k * D
        return {"bytes": b, "flops": f}
    if kind == "decode":
        heads = case["B"] * case["Hq"]
        out = D * DTYPES[case["out"]].itemsize
        return {"bytes": 2 * case["B"] * case["Hkv"] * case["n"] * row + heads * (row + out),
                "flops": 4 * heads * case["n"] * D}
    if kind == "prompt":
        total = _mean_total(case)
        k = case["keep"] * total
        return {"bytes": int(case["Hkv"] * ((total + 3 * k) * row + 4 * total + 12 * k)),
                "flops": int(2 * case["Hkv"] * total * D)}
    if kind == "stream":
        planes = case["L"] * case["Hkv"]
        slots = case["keep"] * _mean_total(case) + case["n_seq"]
        # every cached row and norm once, the new rows in and out, queries and outputs
        b = planes * (slots * (2 * row + 4) + case["n_seq"] * 4 * row) + case["L"] * case["n_seq"] * case["Hq"] * (row + 4 * D)
        return {"bytes": int(b), "flops": int(4 * case["L"] * case["Hq"] * slots * D)}
    planes, heads, T = case["B"] * case["Hkv"], case["B"] * case["Hq"], case["T"]
    return {"bytes": planes * (T * row + 8 * T) + heads * (row + 24), "flops": 2 * heads * T * D}


# ---------------------------------------------------------------------------- what is right
def tolerance(case):
    if case["kind"] in ("compress", "prompt"):
        return "exact"                    # norms in a fixed summation order, indices, copied bytes
    if case["kind"] == "decode" and case["out"] == "bf16":
        return {"rel": 8e-3}              # one rounding to bf16 at the end
    if case["kind"] == "loss":
        return {"rel": 1e-6}              # fp32 scores (2e-7 measured), fp64 sums; ranks are whole numbers
    return {"rel": 3e-5}                  # fp32 sums over up to 66k rows (7e-6 measured against 64 bits)


def _attend(Q, K, V):
    """Q ``[Hq, D]``, K, V ``[Hkv, n, D]`` -> ``[Hq, D]`` in 64 bits."""
    Hq, D = Q.shape
    Hkv = K.shape[0]
    out = []
    for h in range(Hkv):
        q = Q[h * (Hq // Hkv):(h + 1) * (Hq // Hkv)].double()
        p = torch.softmax((q @ K[h].double().t()) / math.sqrt(D), dim=-1)
        out.append(p @ V[h].double())
    return torch.cat(out)


def _norms64(K):
    flat = K.reshape(-1, K.shape[-2], K.shape[-1])
    return torch.stack([x.double().square().sum(-1) for x in flat]).view(K.shape[:-1])


def _keep64(K, k):
    """Positions of the k lowest norms per head, ascending (norms in 64 bits)."""
    return torch.sort(torch.sort(_norms64(K), dim=-1, stable=True).indices[..., :k], dim=-1).values


def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    if kind == "compress":
        return {"norms": _norms64(st["K"]), "kept": None, "Kc": None, "Vc": None}
    if kind == "prompt":
        return {"norms": _norms64(st["K"]), "kept": None, "Kc": None, "Vc": None, "norms_c": None, "pos_c": None}
    if kind == "path":
        idx = _keep64(st["K"], st["k"])
        rows = idx[..., None].expand(*idx.shape, case["D"])
        Kc, Vc = (torch.gather(x, 2, rows) for x in (st["K"], st["V"]))
        return {"norms": _norms64(st["K"]), "kept": None, "Kc": None, "Vc": None,
                "O": torch.stack([_attend(q, k, v) for q, k, v in zip(st["Q"], Kc, Vc)])}
    if kind == "decode":
        return {"O": torch.stack([_attend(q, k, v) for q, k, v in zip(st["Q"], st["Kc"], st["Vc"])])}
    if kind == "stream":
        Hkv, L, n_seq = case["Hkv"], case["L"], case["n_seq"]
        slot = st["slot_off"].tolist()
        O = []
        for l in range(L):
            part = slice(l * Hkv, (l + 1) * Hkv)
            for s in range(n_seq):
                a, b = slot[s], slot[s + 1] - 1                   # the last slot takes the new token
                K = torch.cat([st["Kc"][part, a:b], st["Knew"][0, l, s][:, None]], dim=1)
                V = torch.cat([st["Vc"][part, a:b], st["Vnew"][0, l, s][:, None]], dim=1)
                O.append(_attend(st["Q"][0, l, s], K, V))
        return {"O": torch.stack(O).view(L, n_seq, case["Hq"], case["D"]), "lens": None, "Kc": None, "Vc": None,
                "norms_c": None, "pos_c": None}
    B, Hkv, Hq, T, D, m = case["B"], case["Hkv"], case["Hq"], case["T"], case["D"], st["m"]
    # discard order: highest norm bits first, among equals the later token first
    keep = torch.sort(st["norms"].view(torch.int32), dim=-1, stable=True).indices
    rank = torch.empty_like(keep)
    rank.scatter_(-1, keep, torch.arange(T - 1, -1, -1, device="cuda").expand_as(keep))
    group = Hq // Hkv
    count = torch.arange(T, device="cuda", dtype=torch.float64)
    out = {"drop_rank": None, "alr": [], "loss": [], "loss_ref": []}
    for b in range(B):
        for h in range(Hq):
            a = torch.softmax((st["K"][b, h // group].double() @ st["Q"][b, h].double()) / math.sqrt(D), dim=-1)
            low = torch.sort(a).values
            r = rank[b, h // group]
            out["alr"].append((low * count).sum() - (a * r.double()).sum())
            out["loss"].append(a[r < m].sum())
            out["loss_ref"].append(low[:m].sum())
    for name in ("alr", "loss", "loss_ref"):
        out[name] = torch.stack(out[name]).view(B, Hq)
    return out
