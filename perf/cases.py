"""The calls whose speed counts: what an engine loop over this library does, through its public entry points.

A case is a prefix forest (tokens per level, children per node), a pool type, a head shape and what is done with it:
  decode   one decode step: optionally the store of each request's new token, then attention over the forest
  verify   one verification step: several drafted tokens per request are queried together
  prefill  the new tokens of each request against its cached prefix and themselves, optionally after their store
  mixed    a step with chunked prefill: decode rows next to chunks of prompts, two plans over one q / out
  write    prompts' K/V into the pool
Token counts of the last level are `tokens` or, with `ragged` = f < 1, drawn between f * tokens and tokens.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2603_16104_amd import binding as hkv
from paper_2603_16104_amd import runtime
from paper_2603_16104_amd import workloads as wl

D = hkv.HEAD_DIM
SCALE = float(np.float32(1.0 / np.sqrt(np.float32(D))))
DTYPES = {"bf16": hkv.BF16, "fp8": hkv.FP8_E4M3, "fp32": hkv.FP32}
ELEM = {"bf16": 2, "fp8": 1, "fp32": 4}


def _case(name, op, dtype, heads, tokens, fan, *, ragged=1.0, page=16, append=False, store=False, draft="", chunks=0, chunk=0):
    c = {"op": op, "dtype": dtype, "q_heads": heads[0], "kv_heads": heads[1], "tokens": ",".join(map(str, tokens)),
         "fan": ",".join(map(str, fan)), "ragged": float(ragged), "page": page}
    if append:
        c["append"] = True
    if store:
        c["store"] = True
    if draft:
        c["draft"] = draft
    if chunks:
        c.update(chunks=chunks, chunk=chunk)
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest step: four calls of one small workflow, a few hundred tokens each (two launches and their latency)
        _case("decode_tiny_bf16", "decode", "bf16", (8, 2), (256, 32, 17), (1, 4, 1)),
        # the ordinary generation step of a chat-like batch: 64 calls under one system prompt, each step stores a token
        # per call and attends (Llama-8B-shaped layer)
        _case("decode_chat_bf16", "decode", "bf16", (32, 8), (2048, 512), (1, 64), append=True),
        # a workflow that fans out twice (system prompt, context, one question each), answers of different lengths
        _case("decode_fanout_bf16", "decode", "bf16", (32, 8), (4096, 1024, 256), (1, 8, 16), ragged=0.3),
        # the large batch: 512 calls under 16 long prompts on a 70B-shaped layer, 2.4 GB of fp8 KV
        _case("decode_forest_fp8", "decode", "fp8", (64, 8), (8192, 2048), (16, 32)),
        # 100 questions over ten long contexts behind one system prompt (Qwen3-14B heads), fp8 pool with 64-token pages
        _case("decode_questions_fp8", "decode", "fp8", (40, 8), (1024, 8192, 192), (1, 10, 10), ragged=0.4, page=64),
        # speculative decoding: every call verifies a tree of 21 drafted tokens (branching 3, 2, 2)
        _case("verify_tree_bf16", "verify", "bf16", (32, 8), (2048, 512), (1, 64), ragged=0.8, draft="3-2-2"),
        # a batch of prompts that hit a long cached prefix, 768 to 1024 new tokens each
        _case("prefill_prefix_hit_bf16", "prefill", "bf16", (32, 8), (8192, 1024), (1, 32), ragged=0.75),
        # one call at a time, as a worker that follows a schedule runs them: store the new tokens, attend to the path
        _case("prefill_one_call_bf16", "prefill", "bf16", (32, 8), (4096, 700), (1, 1), store=True),
        # a few prompts at once over an fp8 pool (Qwen3-14B heads), cached prefix of 2048 tokens
        _case("prefill_batch_fp8", "prefill", "fp8", (40, 8), (2048, 512), (1, 6), ragged=0.5, store=True),
        # a chunked-prefill step: 64 decode rows next to 8 prompts that prefill 512 tokens behind the same prefix
        _case("mixed_step_bf16", "mixed", "bf16", (32, 8), (2048, 512), (1, 64), ragged=0.7, chunks=8, chunk=512),
        # the full-precision path, as checks and callers with fp32 weights run it
        _case("decode_checked_fp32", "decode", "fp32", (32, 8), (1024, 256), (1, 16), ragged=0.6),
        # prompts going into an fp8 pool: four calls' worth of tokens, quantised block by block
        _case("write_prompts_fp8", "write", "fp8", (32, 8), (2560,), (4,), ragged=0.6),
    ]


HEADS = [(32, 8), (32, 8), (40, 8), (64, 8), (8, 2)]  # Llama-8B / Qwen3-8B, Qwen3-14B, Qwen3-32B or 70B, a small layer


def draw(rng: random.Random):
    """A case of the same ranges: sizes spread over their logarithm, odd ones among them."""

    def size(lo, hi, multiple=1):
        return max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / multiple))) * multiple

    while True:
        op = rng.choice(["decode", "decode", "decode", "verify", "prefill", "prefill", "mixed", "write"])
        heads = rng.choice(HEADS)
        page = rng.choice([16, 16, 16, 32, 64])
        ragged = rng.choice([1.0, 0.75, 0.5, 0.3])
        if op == "decode":
            dtype = rng.choice(["bf16", "bf16", "fp8", "fp8", "fp32"])
            whole = page if dtype == "fp32" else 1  # the full-precision path takes only whole pages above a leaf
            if rng.random() < 0.5:
                tokens, fan = (size(256, 8192, whole), size(1, 2048)), (rng.choice([1, 1, 2, 4, 16]), size(1, 64))
            else:
                tokens = (size(64, 4096, whole), size(32, 8192, whole), size(1, 512))
                fan = (1, size(1, 16), size(1, 16))
            c = _case("", op, dtype, heads, tokens, fan, ragged=ragged, page=page, append=dtype == "bf16" and rng.random() < 0.4)
        elif op == "verify":
            c = _case("", op, rng.choice(["bf16", "bf16", "fp8"]), heads, (size(256, 4096), size(64, 1024)), (1, size(1, 64)),
                      ragged=max(ragged, 0.5), page=page, draft=rng.choice(["chain2", "chain4", "chain8", "2-2", "3-2-2"]))
        elif op == "prefill":
            c = _case("", op, rng.choice(["bf16", "bf16", "fp8"]), heads, (size(16, 8192, page), size(16, 1024)), (1, size(1, 32)),
                      ragged=ragged, page=page, store=rng.random() < 0.6)
        elif op == "mixed":
            c = _case("", op, rng.choice(["bf16", "bf16", "fp8"]), heads, (size(256, 4096, page), size(16, 1024)), (1, size(4, 128)),
                      ragged=ragged, page=page, chunks=size(1, 8), chunk=size(32, 512))
        else:
            c = _case("", op, rng.choice(["bf16", "fp8"]), heads, (size(16, 8192),), (size(1, 8),), ragged=ragged, page=page)
        w = work(c)
        most = {"bytes": 2.4e9, "flops": 4e12}
        if c["dtype"] == "fp32":
            most = {"bytes": 2e8, "flops": 4e9}
        elif op != "prefill":
            most["flops"] = 2.5e11
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


# ------------------------------------------------------------------------------------------------- shapes
def _numbers(text):
    return [int(x) for x in str(text).split(",")]


def _draft_masks(draft):
    """(drafted tokens per request, visibility masks or None for a causal run)."""
    if draft.startswith("chain"):
        return int(draft[5:]), None
    parents, level = [], [-1]
    for width in map(int, draft.split("-")):
        nxt = []
        for p in level:
            for _ in range(width):
                nxt.append(len(parents))
                parents.append(p)
        level = nxt
    masks = []
    for t, p in enumerate(parents):
        masks.append((1 << t) | (masks[p] if p >= 0 else 0))
    return len(parents), masks


def _shape(case):
    """The forest of a case, fixed by the case alone: parent, tokens per node, the requests' leaves, new tokens per request."""
    tokens, fan = _numbers(case["tokens"]), _numbers(case["fan"])
    rng = np.random.default_rng([len(tokens), *tokens, *fan])
    parent, ntok, level = [], [], [-1]
    for depth, (n, f) in enumerate(zip(tokens, fan)):
        last = depth == len(tokens) - 1
        nxt = []
        for p in level:
            for _ in range(f):
                nxt.append(len(parent))
                parent.append(p)
                least = max(1, int(case["ragged"] * n)) if last else n
                ntok.append(int(rng.integers(least, n + 1)))
        level = nxt
    q_len = [1] * len(level)
    if case["op"] == "verify":
        t, _ = _draft_masks(case["draft"])
        q_len = [t] * len(level)
        for v in level:
            ntok[v] = max(ntok[v], t)
    elif case["op"] == "prefill":
        q_len = [ntok[v] for v in level]
    elif case["op"] == "mixed":
        for _ in range(case["chunks"]):
            level.append(len(parent))
            q_len.append(max(2, case["chunk"]))
            parent.append(0)
            ntok.append(max(2, case["chunk"]))
    return parent, ntok, level, q_len


def _path(parent, v):
    out = []
    while v >= 0:
        out.append(v)
        v = parent[v]
    return out[::-1]


def work(case):
    """Every K/V token of the forest, the queries and the results once; 4 * 128 operations per visible pair and head."""
    parent, ntok, leaves, q_len = _shape(case)
    hq, hk = case["q_heads"], case["kv_heads"]
    per_token = 2 * hk * D * ELEM[case["dtype"]] + (2 * hk * 4 / 16 if case["dtype"] == "fp8" else 0)
    source = 2 * hk * D * (4 if case["dtype"] == "fp32" else 2)
    if case["op"] == "write":
        return {"bytes": sum(ntok) * (per_token + source), "flops": 0}
    rows, io = sum(q_len), 4 if case["dtype"] == "fp32" else 2
    total = sum(ntok) * per_token + rows * hq * (2 * D * io + 4)
    if case.get("append"):
        total += len(leaves) * source
    if case.get("store"):
        total += sum(q_len) * source
    pairs = 0
    masks = _draft_masks(case["draft"])[1] if case["op"] == "verify" else None
    for v, s in zip(leaves, q_len):
        before = sum(ntok[u] for u in _path(parent, v)) - s
        seen = s * (s + 1) // 2 if masks is None else sum(bin(m).count("1") for m in masks)
        pairs += s * before + seen
    return {"bytes": total, "flops": 4 * D * hq * pairs}


def tolerance(case):
    if case["op"] == "write":
        return "exact"  # bytes, and scales that are one division
    # about four times what the results are off the same in 64 bits (relative error of the whole, largest single difference)
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 5e-5}  # up to 1.6e-6 and 9e-6: 32-bit sums over up to 8 000 keys
    if case["dtype"] == "fp8" and case["op"] in ("prefill", "mixed"):
        return {"rel": 1.4e-2, "max": 0.12}  # 3.5e-3 and 3e-2: K and V of an fp8 pool are rounded to bf16 on the way
    return {"rel": 1e-2, "max": 5e-2}  # 2.1e-3 to 2.4e-3 and 1.4e-2: bf16 probabilities, bf16 results


# ------------------------------------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Page order, queries and the nodes' K/V (drawn one node at a time), on the GPU, from the seed alone."""
    _, ntok, _, q_len = _shape(case)
    dt = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)

    def normal(*shape):
        return torch.randn(shape, dtype=dt, device="cuda", generator=gen)

    q = normal(sum(q_len), case["q_heads"], D)

    def nodes():
        for n in ntok:
            yield normal(n, case["kv_heads"], D), normal(n, case["kv_heads"], D)

    return q, nodes()


class _State:
    """What a program keeps between calls: pool, plans, workspaces, queries and results."""

    def __init__(self):
        self.pool = self.decode = self.prefill = None
        self.stores, self.append = [], None

    def __del__(self):
        try:
            if self.decode is not None:
                hkv.hkv_decode_plan_destroy(self.decode)
            if self.prefill is not None:
                hkv.hkv_prefill_plan_destroy(self.prefill)
            if self.pool is not None:
                self.pool.close()
        except Exception:
            pass


def prepare(case, seed):
    parent, ntok, leaves, q_len = _shape(case)
    op, hq, hk, page, dtype = case["op"], case["q_heads"], case["kv_heads"], case["page"], DTYPES[case["dtype"]]
    n_pages = sum(-(-n // page) for n in ntok)
    total_pages = n_pages + n_pages // 4 + 1
    order = np.random.default_rng([int(seed), 5]).permutation(total_pages).astype(np.int32)
    st = _State()
    st.op = op
    st.pool = runtime.DevicePool(total_pages, hk, dtype, free_order=order, poison=False, page_size=page)
    handle = st.pool.handle
    forest = wl.make_forest(parent, ntok, leaves, hkv.kv_pool_alloc(handle, n_pages), page)
    st.stream = torch.cuda.current_stream().cuda_stream
    st.q, nodes = _inputs(case, seed)

    is_leaf = dict(zip(leaves, q_len))
    late = op == "write" or case.get("store")  # these tokens are stored by run() itself
    new_k, new_v = [], []
    for v, (k, val) in enumerate(nodes):
        pages = forest.node_pages[forest.page_begin[v]: forest.page_begin[v] + forest.n_pages[v]]
        if late and v in is_leaf:
            st.stores.append((pages, k, val))
            continue
        if case.get("append") and v in is_leaf:
            new_k.append(k[-1:].clone())
            new_v.append(val[-1:].clone())
            k, val = k[:-1], val[:-1]
        for t in range(0, k.shape[0], 1 << 16):
            st.pool.write(pages[t // page:], 0, k[t: t + (1 << 16)], val[t: t + (1 << 16)], st.stream)
    if op == "write":
        return st
    if new_k:
        last = [forest.node_pages[forest.page_begin[v] + forest.n_pages[v] - 1] for v in leaves]
        st.append = (np.asarray(last, dtype=np.int32), np.asarray([(ntok[v] - 1) % page for v in leaves], dtype=np.int32),
                     torch.cat(new_k), torch.cat(new_v))

    st.out = torch.empty_like(st.q)
    st.lse = torch.empty(st.q.shape[:2], dtype=torch.float32, device="cuda")
    cu = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    dec = [i for i, s in enumerate(q_len) if s == 1] if op == "mixed" else list(range(len(leaves)))
    pre = [i for i, s in enumerate(q_len) if s > 1] if op == "mixed" else list(range(len(leaves)))
    req_leaf = np.asarray(leaves, dtype=np.int32)
    if op in ("decode", "verify", "mixed"):
        if op == "verify":
            t, masks = _draft_masks(case["draft"])
            if masks is None:
                st.decode = hkv.hkv_decode_plan_create_multi(handle, forest.nodes, forest.node_pages, req_leaf, t, hq)
            else:
                st.decode = hkv.hkv_decode_plan_create_tree(handle, forest.nodes, forest.node_pages, req_leaf, t,
                                                            np.tile(np.asarray(masks, dtype=np.uint64), len(leaves)), hq)
        elif op == "mixed":
            st.decode = hkv.hkv_decode_plan_create_ex(handle, forest.nodes, forest.node_pages, req_leaf[dec], hq, q_rows=cu[dec])
        else:
            st.decode = hkv.hkv_decode_plan_create(handle, forest.nodes, forest.node_pages, req_leaf, hq)
        st.ws_bytes = hkv.hkv_decode_plan_workspace_bytes(st.decode)
        st.ws = torch.empty(max(st.ws_bytes, 256), dtype=torch.uint8, device="cuda")
    if op in ("prefill", "mixed"):
        table, kv_len, *_ = hkv.prefix_tree_flatten(forest.nodes, forest.node_pages, req_leaf[pre], max(1, forest.max_pages_per_req()), page)
        if op == "mixed":
            st.prefill = hkv.hkv_prefill_plan_create_rows(handle, cu[pre], np.asarray(q_len)[pre], table, kv_len, hq)
        else:
            st.prefill = hkv.hkv_prefill_plan_create(handle, cu, table, kv_len, hq)
        st.pws_bytes = hkv.hkv_prefill_plan_workspace_bytes(st.prefill)
        st.pws = torch.empty(st.pws_bytes, dtype=torch.uint8, device="cuda") if st.pws_bytes else None
    return st


def run(st):
    for pages, k, v in st.stores:
        hkv.kv_pool_write(st.pool.handle, pages, 0, k.shape[0], k, v, st.stream)
    if st.op == "write":
        p = st.pool
        return {"k": p.k, "v": p.v, "k_scale": p.k_scale, "v_scale": p.v_scale}
    if st.append is not None:
        pages, slots, k, v = st.append
        hkv.kv_pool_append(st.pool.handle, pages, slots, k, v, st.stream)
    if st.decode is not None:
        hkv.attn_decode_plan_run(st.decode, st.q, SCALE, st.out, st.lse, st.ws, st.ws_bytes, st.stream)
    if st.prefill is not None:
        hkv.attn_prefill_plan_run(st.prefill, st.q, SCALE, st.out, st.lse, st.stream, st.pws, st.pws_bytes)
    return {"out": st.out, "lse": st.lse}


# ------------------------------------------------------------------------------------------------- the same in 64 bits
def _amax_scale(x):
    """fp8 pools: one scale per 16 tokens and head, the largest magnitude over 448 (1 for a block of zeros)."""
    n = x.shape[0]
    pad = torch.zeros((-n % 16, *x.shape[1:]), dtype=torch.float32, device=x.device)
    blocks = torch.cat([x.float(), pad]).view(-1, 16, *x.shape[1:])
    amax = blocks.abs().amax(dim=(1, 3))
    # (a tensor divisor: a division by a number would multiply with its reciprocal, one unit off now and then)
    return blocks, torch.where(amax > 0, amax / torch.full_like(amax, 448.0), torch.ones_like(amax))


def _stored(x, dtype):
    """The values a pool of this type holds for x, as float64."""
    if dtype != "fp8":
        return x.double()
    blocks, scale = _amax_scale(x)
    s = scale[:, None, :, None]
    codes = (blocks / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return (codes.double() * s.double()).flatten(0, 1)[: x.shape[0]]


def exact(case, seed):
    parent, ntok, leaves, q_len = _shape(case)
    q, nodes = _inputs(case, seed)
    if case["op"] == "write":
        if case["dtype"] != "fp8":
            return None  # bytes moved, nothing computed
        S = case["page"] // 16
        n_pages = sum(-(-n // case["page"]) for n in ntok)
        total_pages = n_pages + n_pages // 4 + 1
        order = np.random.default_rng([int(seed), 5]).permutation(total_pages)
        scales = [torch.ones((total_pages * S, case["kv_heads"]), dtype=torch.float64, device="cuda") for _ in range(2)]
        begin = 0
        for k, v in nodes:
            for x, to in zip((k, v), scales):
                n = x.shape[0]
                pad = torch.zeros((-n % 16, *x.shape[1:]), dtype=torch.float64, device="cuda")
                amax = torch.cat([x.double(), pad]).view(-1, 16, *x.shape[1:]).abs().amax(dim=(1, 3)) / 448.0
                blocks = [int(order[begin + b // S]) * S + b % S for b in range(amax.shape[0])]
                to[torch.tensor(blocks, device="cuda")] = torch.where(amax > 0, amax, torch.ones_like(amax))
            begin += -(-k.shape[0] // case["page"])
        return {"k": None, "v": None, "k_scale": scales[0].flatten(), "v_scale": scales[1].flatten()}
    kv = [(_stored(k, case["dtype"]), _stored(v, case["dtype"])) for k, v in nodes]
    hk, G = case["kv_heads"], case["q_heads"] // case["kv_heads"]
    masks = _draft_masks(case["draft"])[1] if case["op"] == "verify" else None
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
    row = 0
    for leaf, s in zip(leaves, q_len):
        path = _path(parent, leaf)
        keys, vals = torch.cat([kv[u][0] for u in path]), torch.cat([kv[u][1] for u in path])
        n = keys.shape[0]
        seen = torch.ones((s, n), dtype=torch.bool, device="cuda")
        if masks is None:
            seen = torch.arange(n, device="cuda")[None, :] <= (n - s + torch.arange(s, device="cuda"))[:, None]
        else:
            seen[:, n - s:] = torch.tensor([[bool(m >> j & 1) for j in range(s)] for m in masks], device="cuda")
        for h in range(hk):
            qh = q[row: row + s, h * G: (h + 1) * G].double().reshape(s * G, D)
            sc = torch.matmul(qh, keys[:, h].T.contiguous()) * SCALE
            sc = sc.masked_fill(~seen.repeat_interleave(G, dim=0), -math.inf)
            l = torch.logsumexp(sc, dim=1)
            o = torch.matmul(torch.exp(sc - l[:, None]), vals[:, h].contiguous())
            out[row: row + s, h * G: (h + 1) * G] = o.view(s, G, D)
            lse[row: row + s, h * G: (h + 1) * G] = l.view(s, G)
        row += s
    return {"out": out, "lse": lse}
