"""What the speed of this library is judged on: the calls a serving loop makes.

A case is a dict of plain values. ``listed()`` holds the named ones,
``draw(rng)`` makes another one of the same ranges, and for a case

  prepare(case, seed)  the pools, queries, page lists and plan that a program
                       holds before the call (values and page placement from
                       the seed; the forest's lengths from the case);
  run(state)           one pass through the public entry points;
  work(case)           the bytes and flops one pass cannot do without;
  tolerance(case)      how far two correct implementations may be apart;
  exact(case, seed)    the same outputs in 64 bits with plain torch.

Kinds: "decode" (one query per request over a prefix forest), "prefill" (a
chunk of queries per request over cached segments), "loop" (decode steps with
the cache append and the plan update between them), "write" (copy-on-write
page copies, then new tokens into their pages) and "gather" (paged tokens
read back into dense buffers).
"""

import math
import random

import numpy as np
import torch

from paper_2509_02121_amd import halo

PAGE = 16
LOOP_STEPS = 4
# Slot of token t inside a dim row of a V page.
V_SLOT = [0, 1, 2, 3, 8, 9, 10, 11, 4, 5, 6, 7, 12, 13, 14, 15]
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _attention(kind, name=None, *, heads=(32, 8), dim=128, dtype="bf16", out=None, requests, groups=1, root=0,
               prefix=0, private=(0, 0), chunk=(0, 0)):
    """A forest: an optional root shared by all, `groups` prefixes shared by
    runs of requests, a private segment each and, for a prefill, a chunk."""
    case = {"kind": kind, "q_heads": heads[0], "kv_heads": heads[1], "head_dim": dim, "dtype": dtype,
            "out": out or dtype, "requests": requests, "groups": groups, "root": root, "prefix": prefix,
            "private_lo": private[0], "private_hi": private[1], "chunk_lo": chunk[0], "chunk_hi": chunk[1]}
    if name:
        case["name"] = name
    return case


def _tokens(kind, name=None, *, heads=8, dim=128, dtype="bf16", sequences, length=(0, 0), chunks=0, chunk=(1, 1),
            forks=0):
    """Sequences of cached tokens; for a write, `chunks` of them take a
    prefill chunk and the others one new token, `forks` of them on a page
    just copied from a shared one."""
    case = {"kind": kind, "kv_heads": heads, "head_dim": dim, "dtype": dtype, "sequences": sequences,
            "length_lo": length[0], "length_hi": length[1], "chunks": chunks, "chunk_lo": chunk[0],
            "chunk_hi": chunk[1], "forks": forks}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # The smallest call: a handful of agents on one short system prompt,
        # fp32. Launches and dependent loads are all there is.
        _attention("decode", "decode_tiny_fp32", heads=(4, 4), dim=64, dtype="fp32", requests=8, prefix=256,
                   private=(16, 64)),
        # One layer's decode step of an 8B-shaped model: 64 replicated
        # workflows on a 2048-token prompt, short private suffixes.
        _attention("decode", "decode_8b", requests=64, prefix=2048, private=(64, 512)),
        # Two levels of sharing (a system prompt and 16 templates), 64-dim
        # heads, fp32 output for a caller that accumulates in fp32.
        _attention("decode", "decode_tree_d64", dim=64, out="fp32", requests=256, groups=16, root=1024, prefix=1536,
                   private=(128, 1024)),
        # A 70B-shaped layer at full batch: 8 groups of 128 requests on
        # 8192-token prefixes. The largest call; most of it is the suffixes.
        _attention("decode", "decode_70b", heads=(64, 8), requests=1024, groups=8, prefix=8192, private=(256, 2048)),
        # A few long conversations with nothing in common: all keys private.
        _attention("decode", "decode_long", requests=4, private=(12000, 24000)),
        # Chunked prefill at full batch: 512 new tokens per request over a
        # cached 4096-token prompt.
        _attention("prefill", "prefill_chunked", requests=32, prefix=4096, chunk=(512, 512)),
        # One user's long prompt on an idle server: a ragged chunk over that
        # request's own cached tokens.
        _attention("prefill", "prefill_single", requests=1, private=(4999, 4999), chunk=(901, 901)),
        # Agents continuing with a tool's answer: short ragged chunks over a
        # shared prompt and a private history.
        _attention("prefill", "prefill_short", requests=16, prefix=2048, private=(100, 1000), chunk=(16, 128)),
        # The fp32 prefill, as a reference run of a small batch uses it.
        _attention("prefill", "prefill_fp32", dtype="fp32", requests=4, prefix=1000, chunk=(64, 256)),
        # Decode steps as a serving loop makes them: append the new token's
        # K and V, bring the plan up to date, attend; host work included.
        _attention("loop", "decode_loop", requests=64, prefix=2048, private=(64, 512)),
        # The cache writes of one mixed step: most sequences append a token
        # (some on a page just forked), some write a prefill chunk.
        _tokens("write", "kv_write_mixed", sequences=256, length=(16, 256), chunks=16, chunk=(64, 512), forks=64),
        # Read-back of a batch's cache (to move or to offload it), K and V.
        _tokens("gather", "kv_gather", sequences=64, length=(256, 2048)),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _range(rng, lo, hi):
    a, b = sorted((_log_int(rng, lo, hi), _log_int(rng, lo, hi)))
    return a, b


def _draw_once(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "loop", "write", "gather"])
    dim = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    if kind == "write":
        n = _log_int(rng, 1, 1024)
        return _tokens(kind, heads=rng.choice([4, 8]), dim=dim, dtype=dtype, sequences=n, length=_range(rng, 1, 300),
                       chunks=min(n, rng.choice([0, rng.randint(0, 32)])), chunk=_range(rng, 2, 512),
                       forks=rng.randint(0, n))
    if kind == "gather":
        return _tokens(kind, heads=rng.choice([4, 8]), dim=dim, dtype=dtype, sequences=_log_int(rng, 1, 300),
                       length=_range(rng, 16, 3000))
    heads = rng.choice([(4, 4), (16, 16), (32, 8), (32, 8), (64, 8), (16, 1)])
    out = "fp32" if dtype == "fp32" or rng.random() < 0.25 else dtype
    requests = _log_int(rng, 1, {"decode": 1024, "prefill": 32, "loop": 256}[kind])
    groups = _log_int(rng, 1, max(1, requests // 2))
    prefix = rng.choice([0, _log_int(rng, 16, 8192)])
    root = rng.choice([0, 0, _log_int(rng, 16, 2048)])
    if kind == "prefill":
        return _attention(kind, heads=heads, dim=dim, dtype=dtype, out=out, requests=requests, groups=groups,
                          root=root, prefix=prefix, private=rng.choice([(0, 0), _range(rng, 1, 5000)]),
                          chunk=_range(rng, 1, 1024))
    # a loop's private segments have to hold a token at every step
    return _attention(kind, heads=heads, dim=dim, dtype=dtype, out=out, requests=requests, groups=groups, root=root,
                      prefix=prefix, private=_range(rng, 1, 24000 if kind == "decode" else 2048))


def draw(rng):
    """One more case: sizes spread over the logarithm of their ranges, no
    more costly than the largest listed ones (fp32 products run at about a
    sixteenth of the bf16 rate)."""
    top = {c["name"]: work(c) for c in listed()}
    max_bytes = top["decode_70b"]["bytes"]
    max_flops = top["prefill_chunked"]["flops"]
    while True:
        case = _draw_once(rng)
        w = work(case)
        share = 16 if case["dtype"] == "fp32" else 1
        small = {"loop": 4, "write": 8, "gather": 4}.get(case["kind"], 1)
        if w["bytes"] * small <= max_bytes and w["flops"] * share <= max_flops:
            return case


# ------------------------------------------------------------------- forests

def _lengths(case, lo, hi, n, what):
    """n lengths in [lo, hi], the same for every seed of one case."""
    rng = random.Random(what + repr(sorted((k, v) for k, v in case.items() if k != "name")))
    return [rng.randint(lo, hi) for _ in range(n)]


def _forest(case):
    """(segment lengths, paths, query lengths or None, private segment ids)."""
    R = case["requests"]
    seg, paths, own = [], [[] for _ in range(R)], []
    if case["root"]:
        seg.append(case["root"])
        for p in paths:
            p.append(0)
    if case["prefix"]:
        first = len(seg)
        seg += [case["prefix"]] * case["groups"]
        for r, p in enumerate(paths):
            p.append(first + r * case["groups"] // R)
    if case["private_hi"]:
        for p, n in zip(paths, _lengths(case, case["private_lo"], case["private_hi"], R, "private")):
            own.append(len(seg))
            p.append(len(seg))
            seg.append(n)
    q_len = None
    if case["kind"] == "prefill":
        q_len = _lengths(case, case["chunk_lo"], case["chunk_hi"], R, "chunk")
        for p, n in zip(paths, q_len):
            p.append(len(seg))
            seg.append(n)
    return seg, paths, q_len, own


def _pages(n):
    return (n + PAGE - 1) // PAGE


def _csr(lists):
    indptr = np.zeros(len(lists) + 1, dtype=np.int32)
    indptr[1:] = np.cumsum([len(x) for x in lists])
    flat = np.concatenate([np.asarray(x, dtype=np.int32) for x in lists]) if lists else np.zeros(0, np.int32)
    return indptr, flat.astype(np.int32)


def _place(page_counts, seed, spare=1.25):
    """Page ids of each segment, at random in a pool a quarter larger."""
    need = sum(page_counts)
    size = max(1, math.ceil(need * spare))
    ids = np.random.default_rng(seed).permutation(size)[:need].astype(np.int32)
    cuts = np.cumsum([0] + list(page_counts))
    return [ids[a:b] for a, b in zip(cuts[:-1], cuts[1:])], size


def _pools(case, size, gen):
    dt = DTYPES[case["dtype"]]
    unit = 16 // torch.empty(0, dtype=dt).element_size()
    h, d = case["kv_heads"], case["head_dim"]
    k = torch.randn((size, h, d // unit, PAGE, unit), generator=gen, device="cuda", dtype=dt)
    v = torch.randn((size, h, d, PAGE), generator=gen, device="cuda", dtype=dt)
    return k, v


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _queries(case, rows, gen):
    # scores of standard deviation 2: a few keys carry most of a row's weight,
    # as they do in a trained model
    q = torch.randn((rows, case["q_heads"], case["head_dim"]), generator=gen, device="cuda") * 2
    return q.to(DTYPES[case["dtype"]])


def _cuda(values, dtype=torch.int32):
    return torch.tensor(np.asarray(values), dtype=dtype, device="cuda")


def _attention_inputs(case, seed):
    """Everything but the library's own objects."""
    seg, paths, q_len, own = _forest(case)
    grow = LOOP_STEPS if case["kind"] == "loop" else 0
    full = list(seg)   # lengths once the loop has run
    for s in own:
        full[s] += grow
    pages, size = _place([_pages(n) for n in full], seed)
    gen = _generator(seed)
    k, v = _pools(case, size, gen)
    rows = sum(q_len) if q_len else case["requests"]
    q = [_queries(case, rows, gen) for _ in range(grow or 1)]
    new = []
    for _ in range(grow):
        shape = (case["requests"], case["kv_heads"], case["head_dim"])
        new.append([torch.randn(shape, generator=gen, device="cuda", dtype=DTYPES[case["dtype"]]) for _ in range(2)])
    return {"seg": seg, "paths": paths, "q_len": q_len, "own": own, "pages": pages, "size": size, "k": k, "v": v,
            "q": q, "new": new}


def _forest_csr(x, grown=0):
    """The library's view of the forest after `grown` tokens per request."""
    seg = list(x["seg"])
    for s in x["own"] if grown else []:
        seg[s] += grown
    page_indptr, page_ids = _csr([p[:_pages(n)] for p, n in zip(x["pages"], seg)])
    req_indptr, req_ids = _csr(x["paths"])
    return {"seg_len": np.asarray(seg, dtype=np.int32), "seg_page_indptr": page_indptr, "seg_page_ids": page_ids,
            "req_seg_indptr": req_indptr, "req_seg_ids": req_ids,
            "q_len": None if x["q_len"] is None else np.asarray(x["q_len"], dtype=np.int32)}


def _params(case, size):
    out = case.get("out", case["dtype"])
    q_heads = case.get("q_heads", case["kv_heads"])
    return halo.make_params(q_heads, case["kv_heads"], case["head_dim"], DTYPES[case["dtype"]], size,
                            case["head_dim"] ** -0.5, DTYPES[out])


# ------------------------------------------------------------------- prepare and run

def prepare(case, seed):
    if case["kind"] in ("write", "gather"):
        return _prepare_tokens(case, seed)
    halo.load_library(require_gpu=True)
    x = _attention_inputs(case, seed)
    att = halo.PrefixAttention(_params(case, x["size"]), _forest_csr(x), "cuda")
    outs = [att.alloc_outputs(q) for q in x["q"]]
    if case["kind"] != "loop":
        # a layer's call is bound once to its buffers and made every step
        call = att.bind(x["q"][0], x["k"], x["v"], *outs[0])
        return {"kind": case["kind"], "call": call, "att": att, "inputs": x, "out": outs[0]}
    steps = []
    lists = [x["pages"][s] for s in x["own"]]
    indptr, ids = _csr(lists)
    for t in range(LOOP_STEPS):
        start = [x["seg"][s] + t for s in x["own"]]
        steps.append({"csr": _forest_csr(x, t + 1), "start": _cuda(start), "q": x["q"][t], "new": x["new"][t],
                      "out": outs[t]})
    return {"kind": "loop", "att": att, "inputs": x, "steps": steps, "params": _params(case, x["size"]),
            "indptr": _cuda(indptr), "ids": _cuda(ids), "count": _cuda([1] * case["requests"]),
            "offset": _cuda(range(case["requests"]), torch.int64)}


def _prepare_tokens(case, seed):
    halo.load_library(require_gpu=True)
    n = case["sequences"]
    length = _lengths(case, case["length_lo"], case["length_hi"], n, "length")
    count = [0] * n
    if case["kind"] == "write":
        count = [1] * n
        for i, c in enumerate(_lengths(case, case["chunk_lo"], case["chunk_hi"], case["chunks"], "chunk")):
            count[i * n // case["chunks"]] = c
    pages, size = _place([_pages(a + b) for a, b in zip(length, count)] + [case["forks"]], seed)
    gen = _generator(seed)
    k, v = _pools(case, size, gen)
    params = _params(case, size)
    indptr, ids = _csr(pages[:n])
    indptr, ids = _cuda(indptr), _cuda(ids)
    h, d, dt = case["kv_heads"], case["head_dim"], DTYPES[case["dtype"]]
    state = {"kind": case["kind"], "k": k, "v": v, "keep": [params, indptr, ids]}
    if case["kind"] == "gather":
        offset = _cuda(np.cumsum([0] + length[:-1]), torch.int64)
        seq_len = _cuda(length)
        out = [torch.zeros((sum(length), h, d), dtype=dt, device="cuda") for _ in range(2)]
        state["calls"] = [halo.bind_kv_page_gather(pool, params, which, ids, indptr, seq_len, offset, o)
                          for pool, which, o in ((k, halo.HALO_POOL_K, out[0]), (v, halo.HALO_POOL_V, out[1]))]
        state["keep"] += [seq_len, offset]
        state["out"] = tuple(out)
        return state
    new = [torch.randn((sum(count), h, d), generator=gen, device="cuda", dtype=dt) for _ in range(2)]
    start, cnt = _cuda(length), _cuda(count)
    offset = _cuda(np.cumsum([0] + count[:-1]), torch.int64)
    calls = []
    if case["forks"]:
        # the page that a forked sequence's next token goes to
        src, dst = _cuda(pages[n]), _cuda([pages[i][length[i] // PAGE] for i in range(case["forks"])])
        calls = [halo.bind_kv_page_copy(pool, params, src, dst) for pool in (k, v)]
        state["keep"] += [src, dst]
    calls.append(halo.bind_kv_page_scatter_kv(k, v, params, ids, indptr, start, cnt, offset, *new))
    state["keep"] += [start, cnt, offset, new]
    state["calls"] = calls
    state["out"] = (k, v)
    return state


def run(state):
    if state["kind"] in ("decode", "prefill"):
        state["call"]()
        return state["out"]
    if state["kind"] in ("write", "gather"):
        for call in state["calls"]:
            call()
        return state["out"]
    x, att = state["inputs"], state["att"]
    outs = []
    for s in state["steps"]:
        halo.kv_page_scatter_kv(x["k"], x["v"], state["params"], state["ids"], state["indptr"], s["start"],
                                state["count"], state["offset"], *s["new"])
        att.update(s["csr"])
        outs.append(att.run(s["q"], x["k"], x["v"], *s["out"]))
    return outs, x["k"], x["v"]


# ------------------------------------------------------------------- work, tolerance, exact

def _bytes_of(dtype):
    return 2 if dtype == "bf16" else 4


def work(case):
    elt, d, h = _bytes_of(case["dtype"]), case["head_dim"], case["kv_heads"]
    token = h * d * elt
    if case["kind"] == "gather":
        total = sum(_lengths(case, case["length_lo"], case["length_hi"], case["sequences"], "length"))
        return {"bytes": 4 * total * token, "flops": 0}
    if case["kind"] == "write":
        chunks = _lengths(case, case["chunk_lo"], case["chunk_hi"], case["chunks"], "chunk")
        total = sum(chunks) + case["sequences"] - len(chunks)
        return {"bytes": 4 * total * token + 4 * case["forks"] * PAGE * token, "flops": 0}
    seg, paths, q_len, _ = _forest(case)
    Hq = case["q_heads"]
    rows = sum(q_len) if q_len else case["requests"]
    steps = LOOP_STEPS if case["kind"] == "loop" else 1
    out = {"bytes": 0, "flops": 0}
    for t in range(1, steps + 1):
        grown = t if case["kind"] == "loop" else 0
        keys = sum(seg) + grown * case["requests"]
        pairs = 0
        for r, p in enumerate(paths):
            n = sum(seg[s] for s in p) + grown
            # a chunk's query i sees the cached keys and chunk keys 0..i
            pairs += q_len[r] * (n - q_len[r]) + q_len[r] * (q_len[r] + 1) // 2 if q_len else n
        out["bytes"] += 2 * keys * token + rows * Hq * (d * (elt + _bytes_of(case["out"])) + 4)
        out["bytes"] += 2 * case["requests"] * token if grown else 0   # the appended tokens' inputs
        out["flops"] += 4 * d * Hq * pairs
    return out


def tolerance(case):
    if case["kind"] in ("write", "gather"):
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4}
    # probabilities, partial results and outputs are rounded to bf16
    return {"rel": 1e-2, "max": 1e-1}


def exact(case, seed):
    if case["kind"] in ("write", "gather"):
        return None   # bytes are moved, nothing is computed
    x = _attention_inputs(case, seed)
    slot = torch.tensor(V_SLOT, device="cuda")
    if case["kind"] != "loop":
        return _exact_attention(case, x, x["seg"], x["q"][0], slot)
    outs = []
    for t in range(LOOP_STEPS):
        seg = list(x["seg"])
        for r, s in enumerate(x["own"]):
            page, at = int(x["pages"][s][(seg[s] + t) // PAGE]), (seg[s] + t) % PAGE
            k_new, v_new = x["new"][t][0][r], x["new"][t][1][r]
            x["k"][page, :, :, at, :] = k_new.view(case["kv_heads"], -1, x["k"].shape[-1])
            x["v"][page, :, :, V_SLOT[at]] = v_new
            seg[s] += t + 1   # x["seg"][s] + t + 1 keys at this step
        outs.append(_exact_attention(case, x, seg, x["q"][t], slot))
    return outs, x["k"].double(), x["v"].double()


def _exact_attention(case, x, seg, q_all, slot):
    """Softmax attention of every request over its path's keys, in float64."""
    h, d, Hq = case["kv_heads"], case["head_dim"], case["q_heads"]
    uses = [0] * len(seg)
    for p in x["paths"]:
        for s in p:
            uses[s] += 1
    kept = {}

    def keys_of(s):
        if s in kept:
            return kept[s]
        ids = torch.as_tensor(x["pages"][s][:_pages(seg[s])].astype(np.int64), device="cuda")
        k = x["k"][ids].permute(1, 0, 3, 2, 4).reshape(h, -1, d)[:, :seg[s]].double()   # [h, T, d]
        v = x["v"][ids][..., slot].permute(1, 0, 3, 2).reshape(h, -1, d)[:, :seg[s]].double()
        kv = k.transpose(1, 2).contiguous(), v.contiguous()
        if uses[s] > 1:
            kept[s] = kv
        return kv

    o = torch.empty(q_all.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q_all.shape[:2], dtype=torch.float64, device="cuda")
    row = 0
    for r, p in enumerate(x["paths"]):
        n = x["q_len"][r] if x["q_len"] else 1
        q = q_all[row:row + n].double().view(n, h, Hq // h, d).permute(1, 0, 2, 3).reshape(h, -1, d)
        kv = [keys_of(s) for s in p]
        score = torch.cat([torch.matmul(q, k) for k, _ in kv], dim=2) * (d ** -0.5)
        if x["q_len"]:
            pos = torch.arange(n, device="cuda").repeat_interleave(Hq // h)
            hidden = torch.arange(n, device="cuda")[None, :] > pos[:, None]
            score[:, :, -n:].masked_fill_(hidden, -math.inf)
        l = torch.logsumexp(score, dim=2)
        weight = torch.exp(score - l[..., None])
        out, at = 0, 0
        for _, v in kv:
            out = out + torch.matmul(weight[:, :, at:at + v.shape[1]].contiguous(), v)
            at += v.shape[1]
        o[row:row + n] = out.view(h, n, Hq // h, d).permute(1, 0, 2, 3).reshape(n, Hq, d)
        lse[row:row + n] = l.view(h, n, Hq // h).permute(1, 0, 2).reshape(n, Hq)
        row += n
    return o, lse
