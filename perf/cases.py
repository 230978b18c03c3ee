"""Performance cases of the engine step: what an engine built on this library has it do, through the public binding.

A case is one of
  * an engine step or forward pass (``kind`` "step"): a batch of decode requests and prefill chunks over a paged cache,
    ps_step on the first layer and ps_step_next_layer on the others, with the block copies an engine issues next to it:
    ``swap_out`` / ``swap_in`` move blocks no request of this batch uses (offload, reload ahead of a later step),
    ``reload`` brings blocks of this batch's own requests back, layer by layer, each layer waiting for its own ticket;
  * a list of block copies alone (``kind`` "swap");
  * a serving run of the batch former on its virtual clock (``kind`` "former", host only).

Context lengths and the output lengths of a trace belong to the case (drawn from its own ``lengths`` number), tensors,
block tables, copy lists, arrivals and prompts to the seed given to prepare().
"""
from __future__ import annotations

import math
import weakref

import numpy as np
import torch

from paper_2512_12928_amd import binding as B
from paper_2512_12928_amd import tdg_sim
from paper_2512_12928_amd import workloads as W

DEV = "cuda:0"
D, BLK = 128, 16


def _step(name, hq, hkv, n_decode=0, mean=0, sigma=0.8, lo=1, hi=1, chunks="", layers=1, out="bf16", entry="step", append=True,
          swap_out=0, swap_in=0, reload=0, pool=0, lengths=1):
    """n_decode contexts: lognormal (mean, sigma) clipped to [lo, hi], or uniform in [lo, hi] if sigma is 0.
    chunks: "l_q+prefix" of every prefill chunk, comma separated."""
    c = dict(kind="step", hq=hq, hkv=hkv, n_decode=n_decode, mean=mean, sigma=sigma, lo=lo, hi=hi, chunks=chunks, layers=layers,
             out=out, entry=entry, append=append, swap_out=swap_out, swap_in=swap_in, reload=reload, pool=pool, lengths=lengths)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest engine step: a handful of short requests and one short prompt; launches and latency are all of it
        _step("tiny_mixed", 8, 2, 4, sigma=0, lo=17, hi=200, chunks="64+0"),
        # a lightly loaded server generating: few requests, every layer of a 36-layer model, the batch planned once
        _step("decode_pass_16", 32, 8, 16, sigma=0, lo=600, hi=1400, layers=36),
        # a well loaded server between prompts: decode tokens only, one layer
        _step("decode_256", 32, 8, 256, mean=1500, lo=16, hi=8192),
        # very few requests with very long contexts
        _step("decode_3_long", 64, 8, 3, sigma=0, lo=16385, hi=32767),
        # the first chunk of one prompt on an idle server: time to first token
        _step("prefill_first_512", 32, 8, chunks="512+0"),
        # prompts of odd lengths, some of them continued, float32 output
        _step("prefill_ragged", 64, 8, chunks="1999+0,777+1234,33+4097,1301+2803", out="f32"),
        # an ordinary mixed batch of an 8-KV-head, 32-head layer: many decode tokens and a prefill budget of 2048
        _step("mixed_2k_prefill", 32, 8, 256, mean=1500, lo=16, hi=8192, chunks="512+0,512+512,512+1536,512+3584"),
        # long contexts next to the last chunk of a long prompt
        _step("mixed_long_context", 32, 8, 32, sigma=0, lo=16384, hi=32768, chunks="4096+16384"),
        # the largest configuration: a 64-head layer, 512 decode tokens and a prefill budget of 8192
        _step("mixed_8k_prefill", 64, 8, 512, mean=2000, lo=16, hi=16384, chunks="2048+0,2048+2048,2048+4096,2048+8192"),
        # preemption: the ordinary mixed batch while 512 blocks leave for the host and 512 others come back
        _step("preempting_step", 32, 8, 256, mean=1500, lo=16, hi=8192, chunks="512+0,512+512,512+1536,512+3584", swap_out=512,
              swap_in=512, pool=40000),
        # evicted requests come back: four layers, each waiting only for its own part of the reload
        _step("reload_pass", 32, 8, 96, mean=1100, lo=16, hi=4096, chunks="384+640", layers=4, reload=120),
        # the batch former over a whole arrival trace, host only
        dict(name="former_trace", kind="former", requests=1000, rate=250.0, out_mean=256, gamma=0.9, lengths=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 150)


_BUDGET = None


def draw(rng):
    global _BUDGET
    if _BUDGET is None:
        _BUDGET = max(_cost(c) for c in listed() if c["kind"] == "step")
    while True:
        kind = rng.choice(["decode", "decode", "pass", "prefill", "prefill", "mixed", "mixed", "mixed", "swap", "former"])
        if kind == "former":
            return dict(kind="former", requests=_log(rng, 40, 1000), rate=float(_log(rng, 50, 400)), out_mean=_log(rng, 32, 256),
                        gamma=rng.choice([0.0, 0.9, 0.9, 1000.0]), lengths=rng.randrange(1 << 20))
        if kind == "swap":
            n, way = _log(rng, 1, 512), rng.choice(["out", "in", "both"])
            return dict(kind="swap", hkv=8, swap_out=n if way != "in" else 0, swap_in=n if way != "out" else 0, pool=4096)
        hq, hkv = rng.choice([(32, 8), (32, 8), (32, 8), (64, 8), (64, 8), (8, 2), (16, 2), (12, 4), (16, 1)])
        c = dict(hq=hq, hkv=hkv, out=rng.choice(["bf16", "bf16", "bf16", "f32"]), append=rng.random() < 0.85, lengths=rng.randrange(1 << 20))
        if kind != "prefill":
            c.update(n_decode=_log(rng, 1, 512), mean=_log(rng, 32, 16384), lo=1)
            c["hi"] = min(32768, 6 * c["mean"])
        if kind == "pass":
            c.update(n_decode=_log(rng, 1, 64), layers=rng.randint(4, 36))
        if kind in ("prefill", "mixed"):
            parts = []
            for _ in range(rng.randint(1, 4)):
                lq = _log(rng, 2, 4096)
                parts.append("%d+%d" % (lq, 0 if rng.random() < 0.4 else _log(rng, 1, 16384)))
            c["chunks"] = ",".join(parts)
        if kind == "mixed" and rng.random() < 0.25:
            c.update(swap_out=_log(rng, 8, 256), swap_in=_log(rng, 8, 256))
        if kind == "pass" and rng.random() < 0.4:
            c["reload"] = _log(rng, 4, 120)
        case = _step("", **c)
        if case["layers"] == 1 and _tokens(case)[0].size <= 32 and sum(q for q, _ in _chunks(case)) <= 256 and rng.random() < 0.4:
            case["entry"] = "static"
        if _cost(case) <= _BUDGET and sum(q for q, _ in _chunks(case)) <= 8192:
            return case


# ------------------------------------------------------------------------------------------------ sizes of a case
def _chunks(case):
    return [tuple(int(x) for x in part.split("+")) for part in case["chunks"].split(",") if part]


def _tokens(case):
    """(context lengths of the decode requests, including the new token; [(l_q, prefix)] of the chunks)."""
    rng = np.random.default_rng(case["lengths"])
    n = case["n_decode"]
    if case["sigma"]:
        mu = math.log(max(case["mean"], 1)) - 0.5 * case["sigma"] ** 2
        kv = np.clip(np.rint(rng.lognormal(mu, case["sigma"], size=n)), case["lo"], case["hi"]).astype(np.int64)
    else:
        kv = rng.integers(case["lo"], case["hi"] + 1, size=n)
    return kv, _chunks(case)


def _trace(case, seed):
    return W.make_trace(2, case["requests"], rate_per_s=case["rate"], seed=seed, out_mean=float(case["out_mean"]))


def work(case):
    if case["kind"] == "former":   # the trace in, the delivery times out
        return {"bytes": case["requests"] * (32 + 4) + 8 * sum(r.out_len for r in _trace(case, case["lengths"])), "flops": 0}
    block = 2 * case["hkv"] * BLK * D * 2
    moved = 2 * block * (case["swap_out"] + case["swap_in"])      # each block read once and written once
    if case["kind"] == "swap":
        return {"bytes": moved, "flops": 0}
    kv, chunks = _tokens(case)
    hq, hkv = case["hq"], case["hkv"]
    rows = len(kv) + sum(q for q, _ in chunks)
    ctx = int(kv.sum()) + sum(q + p for q, p in chunks)
    pairs = int(kv.sum()) + sum(q * p + q * (q + 1) // 2 for q, p in chunks)
    row = hkv * D * 2 * 2                                          # K and V of one token
    layer = ctx * row + rows * hq * D * (2 + (4 if case["out"] == "f32" else 2)) + (rows * row * 2 if case["append"] else 0)
    tables = 4 * (sum(-(-int(x) // BLK) for x in kv) + sum(-(-(q + p) // BLK) for q, p in chunks))
    back = min(case["reload"], sum((int(x) - 1) // BLK for x in kv) + sum(p // BLK for _, p in chunks))
    return {"bytes": case["layers"] * (layer + 2 * block * back) + moved + tables, "flops": case["layers"] * 4 * D * hq * pairs}


def tolerance(case):
    # attention: bf16 inputs, bf16 probabilities and (mostly) bf16 results; copies and the batch former are exact
    return {"rel": 1e-2} if case["kind"] == "step" else "exact"


# ------------------------------------------------------------------------------------------------ state and pass
_side = []


def _streams():
    """The engine's compute stream and its two copy streams."""
    if not _side:
        _side.extend(torch.cuda.Stream() for _ in range(3))
    return _side


class _State:
    pass


def _pinned(n, block, seed):
    h = torch.empty((n, block), dtype=torch.uint8, pin_memory=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    # bf16 N(0,1) blocks, as an earlier offload would have left them
    h.copy_(torch.randn((n, block // 2), generator=g, device=DEV).to(torch.bfloat16).view(torch.uint8))
    return h


def prepare(case, seed):
    st = _State()
    st.case = case
    rng = np.random.default_rng(seed)
    if case["kind"] == "former":
        st.cfg = tdg_sim.default_cfg(gamma_num=int(round(case["gamma"] * 10)), gamma_den=10)
        st.trace = _trace(case, seed)
        for r, own in zip(st.trace, _trace(case, case["lengths"])):
            r.out_len = own.out_len
        st.times = np.zeros(sum(r.out_len for r in st.trace), dtype=np.int64)
        st.dev_order, st.host_order = rng.permutation(40_000).astype(np.int32), rng.permutation(80_000).astype(np.int32)
        return st
    hkv, block = case["hkv"], 2 * case["hkv"] * BLK * D * 2
    n_out, n_in = case["swap_out"], case["swap_in"]
    st.streams = _streams()
    if case["kind"] == "swap":
        M, used, hq = case["pool"], np.zeros(0, np.int32), hkv
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        st.pool = torch.randn((M, block // 2), generator=g, device=DEV).to(torch.bfloat16)
        st.reload = 0
    else:
        hq = case["hq"]
        kv, chunks = _tokens(case)
        items = [(1, int(x)) for x in kv] + [(q, q + p) for q, p in chunks]
        need = sum(-(-n // BLK) for _, n in items)
        M = case["pool"] or max(need + 1, math.ceil(1.25 * need)) + n_out + n_in
        st.batch = W.build_batch(W.LayerShape(hq, hkv), items, [1] * len(items), rng, n_device_blocks=M, seed=seed)
        used = st.batch.block_ids
        L, T = case["layers"], st.batch.n_tokens
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        st.pool = torch.empty((L, M, block // 2), dtype=torch.bfloat16, device=DEV)
        flat, slab = st.pool.view(-1), 1 << 28
        for a in range(0, flat.numel(), slab):
            n = min(slab, flat.numel() - a)
            flat[a:a + n] = torch.randn(n, generator=g, device=DEV)

        def rows(heads):
            return torch.randn((L, T, heads, D), generator=g, device=DEV).to(torch.bfloat16)
        q, k, v = rows(hq), rows(hkv), rows(hkv)
        st.out = torch.zeros((L, T, hq, D), dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device=DEV)
        st.layer = [(q[i], k[i] if case["append"] else None, v[i] if case["append"] else None, st.pool[i], st.out[i]) for i in range(L)]
        st.reload = case["reload"]
    if n_out or n_in or st.reload:
        slots = n_out + n_in + L * st.reload if case["kind"] == "step" else n_out + n_in
        st.host = _pinned(slots, block, seed + 1)
        order = rng.permutation(n_out + n_in).astype(np.int32)
        st.out_slots, st.in_slots = order[:n_out], order[n_out:]
        free = rng.permutation(np.setdiff1d(np.arange(M, dtype=np.int32), used)).astype(np.int32)
        st.out_ids, st.in_ids = free[:n_out].copy(), free[n_out:n_out + n_in].copy()
        if st.reload:   # full blocks of the batch's own requests, none of which takes a new token
            b = st.batch
            full = [b.table(r)[:(int(b.kv_len[r]) - b.l_q(r)) // BLK] for r in range(b.n_req)]
            st.re_ids = np.ascontiguousarray(np.concatenate(full)[:st.reload])
            st.re_slots = [n_out + n_in + i * st.reload + rng.permutation(len(st.re_ids)).astype(np.int32) for i in range(L)]
    else:
        slots, st.host = 0, None
    st.ctx = B.ps_create(hq, hkv, M, slots, out_dtype=B.PS_F32 if case.get("out") == "f32" else B.PS_BF16)
    weakref.finalize(st, B.ps_destroy, st.ctx)
    if case["kind"] == "step":
        st.ws_bytes = B.ps_workspace_bytes(st.ctx, st.batch.n_req, T, len(st.batch.block_ids))
        st.ws = torch.empty(st.ws_bytes, dtype=torch.uint8, device=DEV)
        # an engine that copies blocks computes on a stream of its own next to its copy streams
        st.compute = st.streams[0] if st.host is not None else torch.cuda.current_stream()
    torch.cuda.synchronize()
    return st


def run(st):
    case = st.case
    if case["kind"] == "former":
        r = B.ps_sched_simulate(st.cfg, st.dev_order, st.host_order, st.trace, 6_000)
        counts = np.array([len(t) for t in r["token_times"]])
        done = np.concatenate(r["token_times"])
        st.times[:len(done)] = done
        return [st.times, counts,
                np.array([r["gain"], r["ideal_gain"], r["slo_attained"], r["finished"], r["steps"], r["end_ps"]])]
    _, side_out, side_in = st.streams
    if case["swap_out"]:
        B.ps_swap_out(st.ctx, st.out_ids, st.out_slots, -1, st.pool, st.host, side_out)
    if case["swap_in"]:
        B.ps_swap_in(st.ctx, st.in_slots, st.in_ids, -1, st.host, st.pool, side_in)
    if case["kind"] == "swap":
        return [st.pool, st.host]

    def reload(i):
        if not st.reload or i >= len(st.layer):
            return 0
        return B.ps_swap_in(st.ctx, st.re_slots[i], st.re_ids, -1, st.host, st.layer[i][3], side_in)[1]

    ticket = reload(0)
    for i, (q, k, v, cache, out) in enumerate(st.layer):
        ahead = reload(i + 1)
        if i:
            B.ps_step_next_layer(st.ctx, q, k, v, cache, out, st.ws, st.ws_bytes, st.compute, ticket)
        elif case["entry"] == "static":
            B.ps_step_static(st.ctx, st.batch, q, k, v, cache, out, st.compute, ticket)
        else:
            B.ps_step(st.ctx, st.batch, q, k, v, cache, out, st.ws, st.ws_bytes, st.compute, ticket)
        ticket = ahead
    return [st.out, st.pool] + ([st.host] if st.host is not None else [])
