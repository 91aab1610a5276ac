"""Performance cases of the library: what a serving program has it do, through the Python binding.

Four kinds of pass:

  prefill    the suffix tokens of a batch of agent requests attend to their cached prefix pages and
             causally to themselves (``prefix_prefill``), and their K/V go to the pool (``append_kv``)
  decode     one token per request: its K/V go to the pool (``append_kv``), then its query row attends
             to the whole context (``paged_decode``, or ``paged_decode_static``, the form for programs that
             may not allocate)
  swap       evicted pages go to the host tier (``swap_out_pages``), pages of a hit come back (``swap_in_pages``)
  predictor  one forward pass of the workflow predictor over a batch of workflow states

The lengths of a case follow from its own fields (``lens_seed`` among them); values, page placement and
the workflow states follow from the seed that ``prepare`` is given.  K, V and Q are N(0, 1/2) as the synthetic
workloads of this repository draw them (N(0, 1) in fp32).
"""
import math
import random

import numpy as np
import torch

from paper_2605_06472_amd import binding, predictor

PAGE = 16
BENCH_HEADS = (32, 8, 128)
# (query heads, KV heads, head width): every head ratio and both widths the bf16 kernels take
BF16_HEADS = (BENCH_HEADS, (8, 2, 128), (8, 2, 64), (4, 2, 128), (16, 2, 128), (16, 2, 64), (16, 1, 64), (32, 2, 128),
              (4, 4, 64), (8, 8, 128))
F32_HEADS = ((2, 1, 64), (4, 2, 64), (6, 2, 128), (8, 2, 128))
MAX_FLOPS = 5.6e12      # a drawn prefill does no more arithmetic than the largest listed one
MAX_BYTES = 2.6e9       # ... and a drawn decode reads no more than the largest listed one
MAX_SWAP_PAGES = 2048


def _prefill(name, batch, prefix, new, heads=BENCH_HEADS, dtype="bf16", root=0, branches=0, branch=(0, 0), lens_seed=1):
    return {"name": name, "kind": "prefill", "dtype": dtype, "batch": batch, "hq": heads[0], "hkv": heads[1], "d": heads[2],
            "root": root, "branches": branches, "branch_min": branch[0], "branch_max": branch[1],
            "prefix_min": prefix[0], "prefix_max": prefix[1], "new_min": new[0], "new_max": new[1], "lens_seed": lens_seed}


def _decode(name, batch, ctx, heads=BENCH_HEADS, static=False, lens_seed=1):
    return {"name": name, "kind": "decode", "dtype": "bf16", "batch": batch, "hq": heads[0], "hkv": heads[1], "d": heads[2],
            "ctx_min": ctx[0], "ctx_max": ctx[1], "static": static, "lens_seed": lens_seed}


def listed():
    return [
        # one user, one short conversation: the smallest call a server makes, once per layer and token
        _decode("decode_one", 1, (1003, 1003)),
        # the decode batch prefetch transfers hide behind: 64 requests, contexts U{1024..16384}
        _decode("decode_batch", 64, (1024, 16384)),
        # a narrow-head model in a serving loop that may not allocate, ragged short contexts
        _decode("decode_static_d64", 24, (17, 4097), heads=(16, 2, 64), static=True),
        # an agent's next turn: a tool result of a few dozen tokens on a long private history
        _prefill("prefill_turn", 1, (12001, 12001), (37, 37)),
        # four requests behind one shared 2048-token system prompt, 512 new tokens each
        _prefill("prefill_shared_prompt", 4, (0, 0), (512, 512), root=2048),
        # 16 requests over a radix tree: shared root, three branch histories, private tails
        _prefill("prefill_workflow", 16, (0, 2048), (128, 1024), root=1024, branches=3, branch=(512, 4096)),
        # four long accumulated histories, 2048 new tokens each
        _prefill("prefill_long_history", 4, (32768, 32768), (2048, 2048)),
        # 32 requests of mixed lengths, unaligned prefixes: the benchmark batch's shape
        _prefill("prefill_mixed", 32, (0, 16384), (64, 2048)),
        # cold requests of a narrow-head model: nothing cached, causal attention only
        _prefill("prefill_cold_d64", 6, (0, 0), (100, 2000), heads=(16, 2, 64)),
        # fp32 at the repository's smallest configuration
        _prefill("prefill_fp32", 1, (256, 256), (64, 64), heads=(2, 1, 64), dtype="f32"),
        # what one decode step can hide of the host tier: 347 pages out, 347 pages in
        {"name": "swap_pages", "kind": "swap", "hkv": 8, "d": 128, "pages": 347},
        # the predictor over a batch of 1024 workflow states
        {"name": "predictor_batch", "kind": "predictor", "batch": 1024, "agents": 8, "d": 64, "d_x": 5120, "hidden": 64,
         "horizon": 3, "max_prefix": 16},
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], even over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        case = _draw(rng)
        del case["name"]
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def _draw(rng):
    u = rng.random()
    heads = BENCH_HEADS if rng.random() < 0.5 else rng.choice(BF16_HEADS)
    if u < 0.30:
        hi, batch = _log_int(rng, 40, 32768), _log_int(rng, 1, 128)
        static = rng.random() < 0.4 and batch <= 64 and batch * hi <= 100000      # inside that entry point's limits
        return _decode("", batch, (max(1, hi // rng.choice((1, 2, 16))), hi), heads, static, rng.randrange(1 << 20))
    if u < 0.72:
        hi, new = _log_int(rng, 16, 32768), _log_int(rng, 1, 2048)
        lo = rng.choice((0, hi // 4, hi))
        root = PAGE * _log_int(rng, 1, 128) if rng.random() < 0.3 else 0
        if rng.random() < 0.1:
            hi = lo = 0
        return _prefill("", _log_int(rng, 1, 32), (lo, hi), (max(1, new // rng.choice((1, 1, 8))), new), heads, root=root,
                        lens_seed=rng.randrange(1 << 20))
    if u < 0.80:
        hi, new = _log_int(rng, 16, 2048), _log_int(rng, 1, 256)
        return _prefill("", _log_int(rng, 1, 4), (hi // rng.choice((1, 4)), hi), (max(1, new // 2), new), rng.choice(F32_HEADS), "f32",
                        lens_seed=rng.randrange(1 << 20))
    if u < 0.88:
        return {"name": "", "kind": "swap", "hkv": heads[1], "d": heads[2], "pages": _log_int(rng, 4, MAX_SWAP_PAGES)}
    return {"name": "", "kind": "predictor", "batch": _log_int(rng, 1, 4096), "agents": rng.randint(3, 32),
            "d": rng.choice((32, 64, 64, 128)), "d_x": 16 * _log_int(rng, 16, 320), "hidden": rng.choice((32, 64, 64, 100, 256)),
            "horizon": rng.randint(1, 4), "max_prefix": rng.randint(1, 32)}


# ---- lengths and sharing, from the case alone -------------------------------------------------------
def _segments(case):
    """Per request, its prefix as a list of (segment number, tokens), and the number of new tokens."""
    rng = random.Random(case["lens_seed"])
    tree = []
    if case["root"]:
        tree.append(case["root"])
    lo, hi = case["branch_min"] // PAGE, case["branch_max"] // PAGE
    branches = [PAGE * rng.randint(lo, hi) for _ in range(case["branches"])]
    n_shared = len(tree) + len(branches)
    out = []
    for r in range(case["batch"]):
        segs = [(0, case["root"])] if case["root"] else []
        if branches:
            b = r if r < len(branches) else rng.randrange(len(branches))
            segs.append((len(tree) + b, branches[b]))
        tail = rng.randint(case["prefix_min"], case["prefix_max"])
        if tail:
            segs.append((n_shared + r, tail))
        out.append((segs, rng.randint(case["new_min"], case["new_max"])))
    return out


def _contexts(case):
    rng = random.Random(case["lens_seed"])
    return [rng.randint(case["ctx_min"], case["ctx_max"]) for _ in range(case["batch"])]


def _pages(tokens):
    return -(-tokens // PAGE)


# ---- what one pass cannot do without ------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "swap":
        return {"bytes": 2.0 * 2 * case["pages"] * 2 * case["hkv"] * PAGE * case["d"] * 2, "flops": 0.0}
    if kind == "predictor":
        b, v, d, hid, k = case["batch"], case["agents"], case["d"], case["hidden"], case["horizon"]
        outs = k * (v + 1)
        weights = 4 * (d * case["d_x"] + 3 * d * hid + hid * outs + v * d)
        return {"bytes": float(b * (2 * case["d_x"] + 4 * (case["max_prefix"] + 2) + 4 * outs) + weights),
                "flops": 2.0 * b * (d * case["d_x"] + 3 * d * hid + hid * outs)}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    elt = 4 if case["dtype"] == "f32" else 2
    kv_token = 2 * hkv * d * elt
    if kind == "decode":
        tokens = sum(_contexts(case))
        return {"bytes": float(tokens * kv_token + case["batch"] * (kv_token + 2 * hq * d * elt)), "flops": 4.0 * d * hq * tokens}
    shared, flops, new_tokens = {}, 0, 0
    for segs, n in _segments(case):
        shared.update(segs)
        p = sum(t for _, t in segs)
        flops += 4 * d * hq * (n * p + n * (n + 1) // 2)
        new_tokens += n
    # the prefix K/V, the suffix K/V in and out, Q in and the result out
    return {"bytes": float((sum(shared.values()) + 2 * new_tokens) * kv_token + 2 * new_tokens * hq * d * elt), "flops": float(flops)}


# About four times the distance from the same path in 64-bit arithmetic: measured 2.5e-3 (bf16 prefill),
# 1.7e-3 (decode), 4.2e-7 (fp32 prefill), 7.5e-7 (predictor).
def tolerance(case):
    kind = case["kind"]
    if kind == "swap":
        return "exact"
    if kind == "predictor":
        return {"rel": 3e-6}
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    # bf16 results: probabilities and output rounded once each (prefill), output rounded once (decode)
    return {"rel": 1e-2 if kind == "prefill" else 7e-3}


# ---- what a program has in hand before the call --------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, sigma):
    t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32 if math.prod(shape) < 1 << 24 else dtype)
    return t.mul_(sigma).to(dtype)


def prepare(case, seed):
    g = _generator(seed)
    host = np.random.default_rng(seed)
    if case["kind"] == "predictor":
        return _prepare_predictor(case, g, host)
    if case["kind"] == "swap":
        n = case["pages"]
        pool_pages = 3 * n + 5
        ids = host.permutation(pool_pages).astype(np.int32)
        pool = _normal(g, (pool_pages, 2, case["hkv"], PAGE, case["d"]), torch.bfloat16, 2 ** -0.5)
        host_in = torch.empty((n,) + tuple(pool.shape[1:]), dtype=torch.bfloat16, pin_memory=True)
        host_in.copy_(_normal(g, tuple(host_in.shape), torch.bfloat16, 2 ** -0.5))
        return {"kind": "swap", "shape": binding.make_shape(1, case["hkv"], case["hkv"], case["d"], PAGE, pool_pages, 1, "bf16"),
                "pool": pool, "host_in": host_in, "host_out": torch.zeros_like(host_in, pin_memory=True),
                "ids_out": ids[:n].copy(), "ids_in": ids[n:2 * n].copy()}
    # attention: place the segments on scattered pages of a pool that holds a third more than is used
    if case["kind"] == "decode":
        ctx = _contexts(case)
        requests = [([(r, c - 1)] if c > 1 else [], 1) for r, c in enumerate(ctx)]
    else:
        requests = _segments(case)
    first_page, used = {}, 0
    rows = []
    for segs, n in requests:
        row = []
        for number, tokens in segs:
            if number not in first_page:
                first_page[number] = used
                used += _pages(tokens)
            row.extend(range(first_page[number], first_page[number] + _pages(tokens)))
        fresh = _pages(sum(t for _, t in segs) + n) - len(row)      # pages that only the new tokens fill
        row.extend(range(used, used + fresh))
        used += fresh
        rows.append(row)
    pool_pages = used + used // 3 + 3
    place = host.permutation(pool_pages).astype(np.int32)
    width = max(len(row) for row in rows)
    table = np.zeros((len(rows), width), np.int32)
    for r, row in enumerate(rows):
        table[r, :len(row)] = place[np.asarray(row, np.int64)]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    sigma = 1.0 if case["dtype"] == "f32" else 2 ** -0.5
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    new = np.array([n for _, n in requests], np.int32)
    prefix = np.array([sum(t for _, t in segs) for segs, _ in requests], np.int32)
    total = int(new.sum())
    state = {"kind": case["kind"], "static": bool(case.get("static")),
             "shape": binding.make_shape(len(rows), hq, hkv, d, PAGE, pool_pages, width, case["dtype"]),
             "q": _normal(g, (total, hq, d), dtype, sigma), "k_new": _normal(g, (total, hkv, d), dtype, sigma),
             "v_new": _normal(g, (total, hkv, d), dtype, sigma), "pool": _normal(g, (pool_pages, 2, hkv, PAGE, d), dtype, sigma),
             "table": torch.from_numpy(table).cuda(), "prefix_lens": prefix, "new_lens": new, "context_lens": prefix + new}
    state["out"] = torch.zeros_like(state["q"])
    return state


def _prepare_predictor(case, g, host):
    v, d, d_x, hid, k, slots, b = (case[n] for n in ("agents", "d", "d_x", "hidden", "horizon", "max_prefix", "batch"))
    trans = np.zeros((v, v), np.float32)
    for a in range(v):      # a looped call graph: one to three successors per agent
        nxt = host.choice(v, size=int(host.integers(1, min(3, v) + 1)), replace=False)
        trans[a, nxt] = host.integers(1, 20, size=len(nxt))
    trans /= trans.sum(1, keepdims=True)

    def normal(shape, fan_in):
        return _normal(g, shape, torch.float32, fan_in ** -0.5)

    weights = {"emb": normal((v, d), 1), "trans": torch.from_numpy(trans).cuda(), "w1": normal((d, 2 * d), 2 * d),
               "w2": normal((d, 2 * d), 2 * d), "wq": normal((d, d), d), "wt": normal((d, d_x), d_x),
               "wa": normal((hid, 3 * d), 3 * d), "ba": normal((hid,), 100), "wb": normal((k * (v + 1), hid), hid),
               "bb": normal((k * (v + 1),), 100)}
    shape = predictor.make_shape(v, d, d_x, hid, k, slots)
    nbytes = predictor.predictor_workspace_bytes(shape, b)
    workspace = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    predictor.predictor_prepare(shape, weights, workspace, nbytes, b)
    plen = host.integers(0, slots + 1, b).astype(np.int32)
    prefix = host.integers(0, v, (b, slots)).astype(np.int32)
    prefix[np.arange(slots)[None, :] >= plen[:, None]] = -1
    return {"kind": "predictor", "shape": shape, "workspace": workspace, "nbytes": nbytes, "batch": b, "weights": weights,
            "x": _normal(g, (b, d_x), torch.bfloat16, 1.0), "cur": torch.from_numpy(host.integers(0, v, b).astype(np.int32)).cuda(),
            "prefix": torch.from_numpy(prefix).cuda(), "prefix_len": torch.from_numpy(plen).cuda(),
            "probs": torch.zeros((b, k, v + 1), dtype=torch.float32, device="cuda")}


# ---- one pass ------------------------------------------------------------------------------------------
def run(state):
    s, kind = state, state["kind"]
    if kind == "predictor":
        predictor.predictor_forward(s["shape"], s["workspace"], s["nbytes"], s["batch"], s["x"], s["cur"], s["prefix"],
                                    s["prefix_len"], s["batch"], s["probs"])
        return s["probs"]
    if kind == "swap":
        binding.swap_out_pages(s["shape"], s["pool"], s["ids_out"], s["host_out"])
        binding.swap_in_pages(s["shape"], s["host_in"], s["ids_in"], s["pool"])
        return {"host": s["host_out"], "pool": s["pool"]}
    if kind == "decode":
        binding.append_kv(s["shape"], s["k_new"], s["v_new"], s["pool"], s["table"], s["prefix_lens"], s["new_lens"])
        decode = binding.paged_decode_static if s["static"] else binding.paged_decode
        decode(s["shape"], s["q"], s["pool"], s["table"], s["context_lens"], s["out"])
        return {"out": s["out"], "pool": s["pool"]}
    binding.prefix_prefill(s["shape"], s["q"], s["k_new"], s["v_new"], s["pool"], s["table"], s["prefix_lens"], s["new_lens"],
                           s["out"])
    binding.append_kv(s["shape"], s["k_new"], s["v_new"], s["pool"], s["table"], s["prefix_lens"], s["new_lens"])
    return {"out": s["out"], "pool": s["pool"]}
