"""The work a user of this library has it do, as cases that can be timed and checked.

Transfers move requests between two pools on one GPU (a prefill side and a
decode side); attention cases are the decode step that reads the pool
afterwards.  Pools are the caller's torch tensors, block tables come as the
allocator policies give them: "contiguous" (the segment allocator on a free
stretch), "freelist" (the lowest free IDs of a pool with 30% of its blocks held
at random) and "shuffled" (a shuffled free list, every block its own run).

Inputs come from the seed alone, with numpy and torch; ``exact`` computes the
expected outputs from the same inputs in plain torch (transfers: the indexed
copy; attention: the softmax in 64 bits).
"""

import math

import numpy as np
import torch

from paper_2504_03775_amd import flowkv as fk

LM, BM = "layer", "block"
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}

# KV geometries: the library's named ones, and one of small heads and odd blocks
GEOMS = {
    "8b": dict(layers=32, kv_heads=8, head_dim=128, block=16, dtype="bf16"),
    "70b-tp8": dict(layers=80, kv_heads=1, head_dim=128, block=16, dtype="bf16"),
    "tiny": dict(layers=2, kv_heads=2, head_dim=64, block=16, dtype="fp16"),
    "d64": dict(layers=8, kv_heads=4, head_dim=64, block=7, dtype="bf16"),
}


def _transfer(name, how, geom, src, dst, n_req, lo, hi, src_ids, dst_ids):
    return dict(name=name, kind="transfer", how=how, geom=geom, src=src, dst=dst, n_req=n_req,
                lo=lo, hi=hi, src_ids=src_ids, dst_ids=dst_ids)


def _attention(name, how, geom, layout, group, n_req, lo, hi, lens):
    return dict(name=name, kind="attention", how=how, geom=geom, layout=layout, group=group,
                n_req=n_req, lo=lo, hi=hi, lens=lens)


def listed():
    return [
        # a request of the two-layer shape the tests and the smoke check use:
        # 256 KiB, only latency and launches
        _transfer("move-tiny", "request", "tiny", LM, BM, 1, 256, 256, "shuffled", "shuffled"),
        # the shortest prompt of the length sweep, Llama-3-8B shape, placed by
        # the segment allocator on both sides
        _transfer("move-500", "request", "8b", BM, BM, 1, 500, 500, "contiguous", "contiguous"),
        # a middling prompt from a layer-major prefill pool into the
        # restructured block-major pool
        _transfer("move-4k-relayout", "request", "8b", LM, BM, 1, 4000, 4000, "contiguous",
                  "freelist"),
        # the headline request: receiver's blocks allocated, planned, moved, freed
        _transfer("move-13k", "admit", "8b", BM, BM, 1, 13000, 13000, "contiguous", "freelist"),
        # a prompt sent layer by layer as a prefill finishes them
        _transfer("move-layerwise", "layers", "8b", BM, BM, 1, 2000, 2000, "contiguous",
                  "freelist"),
        # several requests at once on one tensor-parallel share: 4 KiB chunks,
        # more runs than the kernel arguments carry
        _transfer("move-tp8-batch", "batch", "70b-tp8", LM, LM, 8, 1000, 8000, "shuffled",
                  "shuffled"),
        # decode attention, one layer: the 32-request batch
        _attention("attn-batch32", "workspace", "8b", BM, 4, 32, 2000, 20000, "host"),
        # one long request alone
        _attention("attn-13k", "noalloc", "8b", BM, 4, 1, 13000, 13000, "host"),
        # the tensor-parallel share: 8 query heads on 1 KV head, long contexts
        _attention("attn-tp8", "workspace", "70b-tp8", LM, 8, 16, 32000, 32000, "host"),
        # small heads, odd block size, lengths on the device
        _attention("attn-d64", "workspace", "d64", BM, 2, 24, 300, 6000, "device"),
        # the smallest call: one short context
        _attention("attn-one-short", "noalloc", "tiny-bf16", BM, 2, 1, 200, 200, "device"),
        # a chat batch's whole decode step: every layer's attention, captured
        # once in a HIP graph and replayed step by step as a serving loop does
        _attention("attn-step-graph", "graph", "8b", BM, 4, 48, 30, 1500, "device"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.5:
        how = rng.choice(["request", "request", "admit", "layers", "batch"])
        geom = rng.choice(["8b", "8b", "70b-tp8", "tiny", "d64"])
        top = {"8b": 13000, "70b-tp8": 40000, "tiny": 100000, "d64": 40000}[geom]
        n = _log(rng, 2, 16) if how == "batch" else 1
        hi = _log(rng, 16, top // n)
        lo = hi if n == 1 else max(1, hi // rng.choice([1, 3, 10]))
        src = rng.choice(["contiguous", "contiguous", "shuffled"])
        dst = "freelist" if how == "admit" else rng.choice(["contiguous", "freelist", "shuffled"])
        if how in ("request", "admit"):
            # what the kernel arguments carry whatever the lists
            hi = lo = min(hi, 900 if "shuffled" in (src, dst) or geom in ("70b-tp8", "tiny", "d64")
                          else top)
        c = _transfer("", how, geom, rng.choice([BM, LM]), rng.choice([BM, LM]), n, lo, hi, src, dst)
    else:
        geom = rng.choice(["8b", "8b", "70b-tp8", "d64", "tiny-bf16"])
        how = rng.choice(["workspace", "workspace", "noalloc", "graph"])
        n = _log(rng, 1, 64)
        hi = _log(rng, 16, min(32000, (32000 if how == "graph" else 400000) // n))
        if how == "noalloc":
            n = min(n, 8)
        lo = max(1, hi // rng.choice([1, 4, 20]))
        c = _attention("", how, geom, rng.choice([BM, LM]), rng.choice([1, 2, 4, 4, 8]), n, lo, hi,
                       "device" if how == "graph" else rng.choice(["host", "device"]))
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------

def _geom(case):
    if case["geom"] == "tiny-bf16":
        return dict(GEOMS["tiny"], dtype="bf16")
    return GEOMS[case["geom"]]


def _lengths(case):
    """The requests' tokens: a property of the case, whatever the seed."""
    n, lo, hi = case["n_req"], case["lo"], case["hi"]
    r = np.random.default_rng(n * 1_000_003 + lo * 1009 + hi)
    x = r.integers(lo, hi + 1, size=n).astype(np.int64)
    x[0] = hi
    return x


def _blocks(case):
    bs = _geom(case)["block"]
    return [-(-int(t) // bs) for t in _lengths(case)]


def _pool_blocks(case):
    # a receiver with 30% of its blocks held has room; attention pools are fuller
    return int((1.5 if case["kind"] == "transfer" else 1.1) * sum(_blocks(case))) + 16


def _held(case, seed):
    """Blocks of the receiver's pool that others hold (policy "freelist")."""
    B = _pool_blocks(case)
    return np.sort(np.random.default_rng(seed + 77).choice(B, size=int(0.3 * B), replace=False)
                   ).astype(np.int32)


def _tables(case, policy, seed):
    """One block list per request."""
    B, need = _pool_blocks(case), _blocks(case)
    r = np.random.default_rng(seed)
    if policy == "contiguous":
        start = int(r.integers(0, B - sum(need) + 1))
        ids = np.arange(start, start + sum(need))
    elif policy == "freelist":
        ids = np.setdiff1d(np.arange(B), _held(case, seed))
    else:
        ids = r.permutation(B)
    out, at = [], 0
    for k in need:
        out.append(ids[at:at + k].astype(np.int32))
        at += k
    return out


def _pool_tensor(g, layout, blocks, seed):
    """One allocation per pool: (B, L, 2, bs, Hkv, Dh), or (L, 2, B, bs, Hkv,
    Dh) whose L slices are the layer tensors; N(0, 1) values."""
    slot = (g["block"], g["kv_heads"], g["head_dim"])
    shape = ((blocks, g["layers"], 2) if layout == BM else (g["layers"], 2, blocks)) + slot
    t = torch.empty(shape, dtype=DTYPES[g["dtype"]], device="cuda")
    t.normal_(generator=torch.Generator("cuda").manual_seed(seed))
    return t


def _pool(layout, t):
    if layout == BM:
        return fk.KVPool(fk.LAYOUT_BLOCK_MAJOR, t)
    return fk.KVPool(fk.LAYOUT_LAYER_MAJOR, list(t.unbind(0)))


def _transfer_inputs(case, seed):
    g, B = _geom(case), _pool_blocks(case)
    return (_pool_tensor(g, case["src"], B, seed), _pool_tensor(g, case["dst"], B, seed + 1),
            _tables(case, case["src_ids"], seed + 2), _tables(case, case["dst_ids"], seed + 3))


def _attention_inputs(case, seed):
    g, B, n = _geom(case), _pool_blocks(case), case["n_req"]
    t = _pool_tensor(g, case["layout"], B, seed)
    lists = _tables(case, "shuffled", seed + 2)
    tab = np.full((n, max(len(x) for x in lists)), -1, dtype=np.int32)
    for r, x in enumerate(lists):
        tab[r, :len(x)] = x
    steps = g["layers"] if case["how"] == "graph" else 1
    q = torch.empty((steps, n, g["kv_heads"] * case["group"], g["head_dim"]),
                    dtype=torch.bfloat16, device="cuda")
    q.normal_(generator=torch.Generator("cuda").manual_seed(seed + 3))
    return t, tab, q


def _layer(case):
    return _geom(case)["layers"] // 2


# ---- one pass -----------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "transfer":
        s, d, S, D = _transfer_inputs(case, seed)
        st = dict(case=case, out=d, src=_pool(case["src"], s), dst=_pool(case["dst"], d))
        B = _pool_blocks(case)
        st["blocks"] = B
        if case["how"] == "batch":
            st["offsets"] = np.concatenate(([0], np.cumsum([len(x) for x in S]))).astype(np.int64)
            st["stager"] = fk.PlanStager("cuda")
        if case["how"] == "admit":
            st["alloc"] = fk.Allocator(B, fk.POLICY_FIFO_SORTED, 0)
            st["alloc"].mark_used(_held(case, seed + 3))
        st["S"], st["D"] = np.concatenate(S), np.concatenate(D)
        return st
    g = _geom(case)
    t, tab, q = _attention_inputs(case, seed)
    lens = _lengths(case).astype(np.int32)
    n, hq = case["n_req"], g["kv_heads"] * case["group"]
    st = dict(case=case, pool=_pool(case["layout"], t), q=q,
              tables=torch.as_tensor(tab, device="cuda"),
              lens=torch.as_tensor(lens, device="cuda"),
              host=lens if case["lens"] == "host" else None,
              out=torch.zeros((len(q), n, hq, g["head_dim"]), dtype=torch.float32, device="cuda"),
              max=int(lens.max()), scale=1.0 / math.sqrt(g["head_dim"]), layer=_layer(case))
    if case["how"] != "noalloc":
        st["ws"] = torch.empty(fk.flowkv_decode_attention_workspace(n, hq, g["head_dim"], st["max"]),
                               dtype=torch.uint8, device="cuda")
    if case["how"] == "graph":
        _all_layers(st)     # once outside the capture, as torch asks
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _all_layers(st)
    return st


def _all_layers(st):
    for layer in range(st["pool"].num_layers):
        fk.flowkv_decode_attention(st["pool"], layer, st["q"][layer], st["tables"], st["lens"],
                                   st["max"], st["scale"], st["out"][layer], st["ws"])


def run(st):
    how = st["case"]["how"]
    if how == "request":
        fk.flowkv_transfer_request(st["src"], st["dst"], st["S"], st["D"])
    elif how == "admit":
        ids = st["alloc"].alloc(len(st["S"]))
        fk.flowkv_transfer_request(st["src"], st["dst"], st["S"], ids)
        st["alloc"].free(ids)
    elif how == "layers":
        segs = fk.flowkv_plan(st["S"], st["D"], st["blocks"], st["blocks"])
        dev = fk.segments_to_device(segs, "cuda:0")
        total = fk.plan_total_blocks(segs)
        for layer in range(st["src"].num_layers):
            fk.flowkv_transfer_layers(st["src"], st["dst"], dev, len(segs), total, layer, 1)
    elif how == "batch":
        segs = fk.flowkv_plan_batch(st["offsets"], st["S"], st["D"], st["blocks"], st["blocks"])
        dev = st["stager"].stage(segs)
        fk.flowkv_transfer(st["src"], st["dst"], dev, len(segs), fk.plan_total_blocks(segs))
        st["stager"].release()
    elif how == "graph":
        st["graph"].replay()
    elif how == "noalloc":
        fk.flowkv_decode_attention_noalloc(st["pool"], st["layer"], st["q"][0], st["tables"],
                                           st["lens"], st["max"], st["scale"], st["out"][0],
                                           seq_lens_host=st["host"])
    else:
        fk.flowkv_decode_attention(st["pool"], st["layer"], st["q"][0], st["tables"], st["lens"],
                                   st["max"], st["scale"], st["out"][0], st["ws"],
                                   seq_lens_host=st["host"])
    return st["out"]


# ---- what it costs and what it gives -------------------------------------------

def work(case):
    g = _geom(case)
    slot = g["kv_heads"] * g["head_dim"] * 2
    if case["kind"] == "transfer":
        return {"bytes": 2 * sum(_blocks(case)) * 2 * g["layers"] * g["block"] * slot, "flops": 0}
    steps = g["layers"] if case["how"] == "graph" else 1
    tokens, n, hq = int(_lengths(case).sum()), case["n_req"], g["kv_heads"] * case["group"]
    heads = n * hq * g["head_dim"]
    return {"bytes": steps * (tokens * 2 * slot + heads * (2 + 4) + 4 * sum(_blocks(case))),
            "flops": steps * 4 * tokens * hq * g["head_dim"]}


def tolerance(case):
    if case["kind"] == "transfer":
        return "exact"
    # float32 sums of exact bf16 products; matrix-core weights carry 16 bits
    return {"rel": 1e-5, "max": 1e-4}


def exact(case, seed):
    if case["kind"] == "transfer":
        s, d, S, D = _transfer_inputs(case, seed)
        S = torch.as_tensor(np.concatenate(S).astype(np.int64), device="cuda")
        D = torch.as_tensor(np.concatenate(D).astype(np.int64), device="cuda")
        by_block = [t if lay == BM else t.movedim(2, 0)
                    for t, lay in ((s, case["src"]), (d, case["dst"]))]
        by_block[1][D] = by_block[0][S]
        return d
    g = _geom(case)
    t, tab, q = _attention_inputs(case, seed)
    lens = _lengths(case)
    layers = range(g["layers"]) if case["how"] == "graph" else [_layer(case)]
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    for i, layer in enumerate(layers):
        for r in range(case["n_req"]):
            T = int(lens[r])
            ids = torch.as_tensor(tab[r, :-(-T // g["block"])].astype(np.int64), device="cuda")
            for h in range(g["kv_heads"]):
                if case["layout"] == BM:
                    kv = t[:, layer, :, :, h][ids].movedim(1, 0)
                else:
                    kv = t[layer, :, :, :, h][:, ids]
                k, v = kv.reshape(2, -1, g["head_dim"])[:, :T].double()
                qs = q[i, r, h * case["group"]:(h + 1) * case["group"]].double()
                p = torch.softmax((qs @ k.T.contiguous()) / math.sqrt(g["head_dim"]), -1)
                out[i, r, h * case["group"]:(h + 1) * case["group"]] = p @ v
    return out
