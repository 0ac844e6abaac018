"""Performance cases of the layer-wise prefix-KV reload and prefill attention path.

Each case is one pass through the public entry points of
``paper_2606_16135_amd.swiftcache`` as a serving program calls them.  The
listed cases are the sizes this repository's configurations, benchmark and
tests use, from one launch-bound call to the long-context layer stack;
``draw`` gives more of the same ranges.

A case's ``kind`` names the calls of a pass:

``attn``
    ``sc_prefill_attn`` / ``sc_prefill_attn_f16`` (``noalloc``:
    ``sc_prefill_attn_noalloc``): one conversation's new turn over its active
    K/V; returns the output and the log-sum-exp.
``layer``
    one layer of a batch of conversations, call by call on one stream:
    ``sc_fetch_layer_kv``, ``sc_append_new_kv``, ``sc_prefill_attn_varlen``,
    ``sc_store_layer_kv``; optionally with part of each prefix in the regular
    cache.  Returns the attention output, the active K/V and the pool.
``fetch``
    ``sc_fetch_layer_kv`` alone; returns the active K/V.
``stack``
    ``sc_prefill_stack`` (``chunk`` > 0: ``sc_prefill_stack_chunked``), the
    overlapped layer pipeline; returns every layer's output, both active
    slots and the pool.
"""

import math

import numpy as np
import torch

from paper_2606_16135_amd import swiftcache as sc

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16}
BLOCK = 16   # tokens per pool block, as in every benchmark workload


def _attn(name, hq, hkv, d, p, n, dtype="bf16", noalloc=False):
    return {"name": name, "kind": "attn", "hq": hq, "hkv": hkv, "d": d, "p": p, "n": n, "dtype": dtype,
            "noalloc": noalloc}


def _pooled(name, kind, hq, hkv, d, batch, p, n, layers=1, dtype="bf16", rc=0.0, host=0.0, chunk=0, spread=0.0,
            lens=0):
    """``spread`` > 0: batch lengths drawn around p and n (see _lengths) with seed ``lens``."""
    return {"name": name, "kind": kind, "hq": hq, "hkv": hkv, "d": d, "batch": batch, "p": p, "n": n,
            "layers": layers, "dtype": dtype, "rc": rc, "host": host, "chunk": chunk, "spread": spread,
            "lens": lens}


def listed():
    return [
        # The smallest call: a short turn on a short history with 64-dim
        # heads, where launches and latency are all there is.
        _attn("attn-tiny-d64", 8, 8, 64, 256, 64),
        # A follow-up question of a few words over an ordinary chat history,
        # through the entry point for callers that may not allocate (graph
        # capture, tight serving loops).
        _attn("attn-turn-noalloc", 32, 8, 128, 2048, 24, noalloc=True),
        # A short question about a long document, fp16 as the paper serves.
        _attn("attn-document-f16", 40, 8, 128, 32768, 48, dtype="f16"),
        # A long turn over a long history: one layer of the 40/8-head shape.
        _attn("attn-14b-shape", 40, 8, 128, 32768, 1024),
        # The same path with 64-dim heads at an ordinary size.
        _attn("attn-d64", 32, 8, 64, 8192, 512),
        # One layer of 16 conversations of ragged lengths (the batch a
        # scheduler forms), call by call: fetch, append, attention, store.
        _pooled("layer-varlen", "layer", 32, 8, 128, 16, 4096, 1024, layers=2, spread=0.8, lens=3),
        # The same with half of each prefix in the regular cache (read in
        # place through the block table), fp16, fewer conversations.
        _pooled("layer-regular-cache-f16", "layer", 32, 8, 128, 8, 4096, 512, layers=2, dtype="f16", rc=0.5, spread=0.8,
                lens=8),
        # The KV load alone: one layer of a 32768-token prefix.
        _pooled("fetch-14b-shape", "fetch", 40, 8, 128, 1, 32768, 1024, layers=4),
        # The benchmark's 32-layer stack of one conversation.
        _pooled("stack-8b-shape", "stack", 32, 8, 128, 1, 8192, 512, layers=32),
        # A short turn through all 32 layers: many small launches.
        _pooled("stack-short-turn", "stack", 32, 8, 128, 1, 1024, 64, layers=32),
        # A long turn processed in chunks (bounded workspace and launches).
        _pooled("stack-chunked", "stack", 40, 8, 128, 1, 16384, 1024, layers=4, chunk=256),
        # The long-context stack with half of its blocks in pinned host
        # memory, two layers of it (each layer is the same work).
        _pooled("stack-host-tier", "stack", 32, 8, 128, 1, 131072, 2048, layers=2, host=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


HEADS = [(8, 8, 64), (32, 8, 64), (32, 8, 128), (40, 8, 128), (28, 4, 128), (16, 8, 128), (48, 8, 128)]
MOST_FLOPS = 4e12   # below the listed long-context stack


def draw(rng):
    while True:
        kind = rng.choice(["attn"] * 4 + ["layer"] * 2 + ["stack"] * 2 + ["fetch"])
        hq, hkv, d = rng.choice(HEADS)
        dtype = rng.choice(["bf16", "bf16", "f16"])
        if kind == "attn":
            c = _attn("", hq, hkv, d, _log_int(rng, 64, 32768), _log_int(rng, 1, 1024), dtype)
            c["noalloc"] = dtype == "bf16" and c["n"] <= 256 and rng.random() < 0.4
        else:
            batch = 1 if kind == "stack" and rng.random() < 0.6 else rng.randint(1, 16)
            layers = rng.choice([2, 4, 8, 16, 32]) if kind == "stack" else rng.choice([1, 2, 4])
            p, n = _log_int(rng, 256, 32768 if batch == 1 else 6000), _log_int(rng, 8, 1024)
            if rng.random() < 0.4:
                n = max(1, n // 4)
            c = _pooled("", kind, hq, hkv, d, batch, p, n, layers, dtype,
                        rc=rng.choice([0.0, 0.0, 0.25, 0.5]) if kind != "fetch" else 0.0,
                        host=rng.choice([0.0, 0.0, 0.0, 0.25]) if kind != "layer" else 0.0,
                        spread=rng.choice([0.3, 0.8]) if batch > 1 else 0.0, lens=rng.randint(0, 10**6))
            if kind == "stack" and n >= 64 and rng.random() < 0.3:
                c["chunk"] = max(16, n // rng.choice([2, 3, 4]))
        # At most a few GB of pool and the work of the largest listed case.
        tokens = c["p"] + c["n"] if kind == "attn" else sum(map(sum, zip(*_lengths(c))))
        pool = tokens * 4 * hkv * d * c.get("layers", 1)
        if work(c)["flops"] > MOST_FLOPS or pool > 3e9 or (c.get("host") and pool > 4e8):
            continue
        del c["name"]
        return c


def _lengths(c):
    """Prefix and new-turn lengths of the batch: one conversation's are p and
    n; a batch's prefixes are lognormal around p and its turns uniform up to
    n, as the benchmark's ragged batch is drawn."""
    b = c["batch"]
    if not c["spread"]:
        return [c["p"]] * b, [c["n"]] * b
    rng = np.random.default_rng(c["lens"])
    p = np.floor(np.clip(rng.lognormal(math.log(c["p"]), c["spread"], size=b), c["p"] / 8, c["p"] * 8))
    n = rng.integers(max(1, c["n"] // 16), c["n"], size=b, endpoint=True)
    return [int(x) for x in p], [int(x) for x in n]


def _randn(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(DTYPES[dtype])


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


class _Pool:
    """A donor pool in caller-owned memory and the block table of one batch,
    kept for as long as a program's conversations live."""

    def __init__(self, c, seed, gen):
        p, n = _lengths(c)
        per_seq = [-(-(a + b) // BLOCK) for a, b in zip(p, n)]
        in_rc = [int(c["rc"] * (a // BLOCK)) for a in p]
        rng = np.random.default_rng(int(seed))
        n_rc, donor = sum(in_rc), sum(per_seq) - sum(in_rc)
        total = donor + donor // 4 + 1
        n_host = int(c["host"] * total)
        n_dev = total - n_host
        place = rng.permutation(total)[:donor]
        place_rc = rng.permutation(n_rc) + total
        ids, cu, i, j = [], [0], 0, 0
        for m, r in zip(per_seq, in_rc):
            ids += [int(x) for x in place_rc[j:j + r]] + [int(x) for x in place[i:i + m - r]]
            i, j = i + m - r, j + r
            cu.append(len(ids))
        shape = (c["layers"], 2, BLOCK, c["hkv"], c["d"])
        self.ids, self.cu, self.p, self.n, self.n_dev, self.n_host = ids, cu, p, n, n_dev, n_host
        self.in_rc = in_rc
        td = DTYPES[c["dtype"]]

        def tier(blocks):
            t = torch.empty((blocks,) + shape, dtype=td, device="cuda")
            step = max(1, (1 << 27) // t[0].numel())
            for k in range(0, blocks, step):
                m = min(step, blocks - k)
                t[k:k + m] = _randn(gen, (m,) + shape, c["dtype"])
            return t

        self.dev = tier(n_dev)
        self.host = None
        if n_host:
            self.host = torch.empty((n_host,) + shape, dtype=td, pin_memory=True)
            self.host.copy_(tier(n_host))
        self.rc = tier(n_rc) if n_rc else None
        torch.cuda.synchronize()
        self.handle = self.table = None
        self.handle = sc.sc_pool_create(
            c["layers"], c["hkv"], c["d"], BLOCK, n_dev, n_host, torch.cuda.current_device(), self.dev.data_ptr(),
            self.host.data_ptr() if n_host else 0, n_rc, self.rc.data_ptr() if n_rc else 0,
            sc.DTYPE_CODES[c["dtype"]])
        self.table = sc.sc_table_create(self.handle, ids, cu, p, n, torch.cuda.current_stream().cuda_stream)

    def __del__(self):
        torch.cuda.synchronize()
        if self.table:
            sc.sc_table_destroy(self.table)
        if self.handle:
            sc.sc_pool_destroy(self.handle)

    def tensors(self):
        return [t for t in (self.dev, self.host, self.rc) if t is not None]


def prepare(case, seed):
    c = dict(case)
    gen = _generator(seed)
    hq, hkv, d, dtype = c["hq"], c["hkv"], c["d"], c["dtype"]
    st = {"case": c, "stream": torch.cuda.current_stream().cuda_stream}
    if c["kind"] == "attn":
        t = c["p"] + c["n"]
        st["q"] = _randn(gen, (c["n"], hq, d), dtype)
        st["k"] = _randn(gen, (t, hkv, d), dtype)
        st["v"] = _randn(gen, (t, hkv, d), dtype)
        st["out"] = torch.empty_like(st["q"])
        st["lse"] = torch.empty((hq, c["n"]), dtype=torch.float32, device="cuda")
        return st
    pool = st["pool"] = _Pool(c, seed, gen)
    total_q, total_kv = sum(pool.n), sum(pool.n) + sum(pool.p)

    def slot():
        k = torch.zeros((total_kv, hkv, d), dtype=DTYPES[dtype], device="cuda")
        v = torch.zeros_like(k)
        return k, v, sc.active(k.data_ptr(), v.data_ptr(), total_kv)

    layers = c["layers"] if c["kind"] == "stack" else 1
    st["slots"] = [slot() for _ in range(2 if c["kind"] == "stack" else 1)]
    if c["kind"] == "fetch":
        return st
    st["q"] = _randn(gen, (layers, total_q, hq, d), dtype)
    st["kn"] = _randn(gen, (layers, total_q, hkv, d), dtype)
    st["vn"] = _randn(gen, (layers, total_q, hkv, d), dtype)
    st["out"] = torch.empty_like(st["q"])
    if c["kind"] == "stack":
        st["ptrs"] = [[t[l].data_ptr() for l in range(layers)] for t in (st["q"], st["kn"], st["vn"], st["out"])]
        st["copy"] = torch.cuda.Stream()
    return st


def run(st):
    c = st["case"]
    s = st["stream"]
    if c["kind"] == "attn":
        f = (sc.sc_prefill_attn_f16 if c["dtype"] == "f16"
             else sc.sc_prefill_attn_noalloc if c["noalloc"] else sc.sc_prefill_attn)
        f(st["q"].data_ptr(), st["k"].data_ptr(), st["v"].data_ptr(), c["p"], c["n"], c["hq"], c["hkv"], c["d"],
          st["out"].data_ptr(), st["lse"].data_ptr(), stream=s)
        return {"out": st["out"], "lse": st["lse"]}
    pool = st["pool"]
    if c["kind"] == "stack":
        slots = [x[2] for x in st["slots"]]
        if c["chunk"]:
            sc.sc_prefill_stack_chunked(pool.handle, pool.table, *st["ptrs"], slots, c["hq"], c["chunk"],
                                        compute_stream=s, copy_stream=st["copy"].cuda_stream)
        else:
            sc.sc_prefill_stack(pool.handle, pool.table, *st["ptrs"], slots, c["hq"], compute_stream=s,
                                copy_stream=st["copy"].cuda_stream)
        return {"out": st["out"], "active": [t for x in st["slots"] for t in x[:2]], "pool": pool.tensors()}
    k, v, active = st["slots"][0]
    layer = c["layers"] - 1
    sc.sc_fetch_layer_kv(pool.handle, pool.table, layer, active, s)
    if c["kind"] == "fetch":
        return {"active": [k, v]}
    kn, vn = st["kn"].data_ptr(), st["vn"].data_ptr()
    sc.sc_append_new_kv(pool.handle, pool.table, kn, vn, active, s)
    sc.sc_prefill_attn_varlen(pool.handle, pool.table, layer, st["q"].data_ptr(), active, c["hq"],
                              st["out"].data_ptr(), stream=s)
    sc.sc_store_layer_kv(pool.handle, pool.table, layer, kn, vn, s)
    return {"out": st["out"], "active": [k, v], "pool": pool.tensors()}


def work(case):
    c = case
    row = 2 * c["hkv"] * c["d"]           # bytes of one token's K (or V)
    if c["kind"] == "attn":
        p, n, layers = [c["p"]], [c["n"]], 1
    else:
        p, n = _lengths(c)
        layers = c["layers"] if c["kind"] == "stack" else 1
    if c["kind"] == "fetch":
        return {"bytes": 2 * 2 * row * sum(p), "flops": 0}
    pairs = sum(b * a + b * (b + 1) // 2 for a, b in zip(p, n))
    q = 2 * c["hq"] * c["d"] * sum(n)
    # Prefix K/V read, q read, out written, the new turn's K/V read (and, for
    # the pooled paths, stored to the pool).
    new = 2 * row * sum(n) * (1 if c["kind"] == "attn" else 2)
    if c["kind"] == "layer":              # the active buffer is an output too
        new += 2 * row * (sum(p) - sum(BLOCK * int(c["rc"] * (a // BLOCK)) for a in p) + sum(n))
    return {"bytes": layers * (2 * row * sum(p) + 2 * q + new), "flops": layers * 4 * c["d"] * c["hq"] * pairs}


def tolerance(case):
    if case["kind"] == "fetch":
        return "exact"
    # Rounding of the probabilities, the split partials and the output to 16
    # bits: 2.9e-3 (bf16) and 3.6e-4 (fp16) measured against exact(), times
    # four.
    return {"rel": 1.2e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-3}


def _attention64(q, k, v, p):
    """Causal GQA attention of one sequence in float64: q [n][hq][d] over
    k, v [p + n][hkv][d]; returns out and the natural-log log-sum-exp."""
    n, hq, d = q.shape
    t, hkv = k.shape[0], k.shape[1]
    g = hq // hkv
    out = torch.empty((n, hq, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((hq, n), dtype=torch.float64, device=q.device)
    pos = torch.arange(t, device=q.device)
    step = max(1, (1 << 27) // (g * t))
    for h in range(hkv):
        kt = k[:, h].double().t().contiguous()
        vh = v[:, h].double().contiguous()
        for i in range(0, n, step):
            m = min(step, n - i)
            qs = q[i:i + m, h * g:(h + 1) * g].double().reshape(m * g, d).contiguous()
            s = (qs @ kt).mul_(1.0 / math.sqrt(d)).view(m, g, t)
            limit = p + i + torch.arange(m, device=q.device)
            s.masked_fill_((pos[None, :] > limit[:, None])[:, None, :], -math.inf)
            top = s.amax(dim=-1, keepdim=True)
            s.sub_(top).exp_()
            den = s.sum(dim=-1, keepdim=True)
            o = (s.view(m * g, t) @ vh).view(m, g, d) / den
            out[i:i + m, h * g:(h + 1) * g] = o
            lse[h * g:(h + 1) * g, i:i + m] = (top + den.log())[..., 0].t()
    return out, lse


def exact(case, seed):
    st = prepare(case, seed)
    c = st["case"]
    if c["kind"] == "attn":
        out, lse = _attention64(st["q"], st["k"], st["v"], c["p"])
        return {"out": out, "lse": lse}
    pool = st["pool"]

    def rows(layer, b):
        """K and V rows of every position of sequence b's block table."""
        parts = []
        for i in pool.ids[pool.cu[b]:pool.cu[b + 1]]:
            t, k = ((pool.dev, i) if i < pool.n_dev else (pool.host, i - pool.n_dev)
                    if i < pool.n_dev + pool.n_host else (pool.rc, i - pool.n_dev - pool.n_host))
            parts.append((t, k))
        out = torch.empty((len(parts), 2, BLOCK, c["hkv"], c["d"]), dtype=pool.dev.dtype, device="cuda")
        for t in pool.tensors():
            sel = [j for j, x in enumerate(parts) if x[0] is t]
            if sel:
                src = torch.tensor([parts[j][1] for j in sel], device=t.device)
                out[torch.tensor(sel, device="cuda")] = t[:, layer][src].to("cuda")
        return [out[:, h].reshape(-1, c["hkv"], c["d"]) for h in (0, 1)]

    if c["kind"] == "fetch":
        k, v = st["slots"][0][:2]
        at = 0
        for b, (p, n) in enumerate(zip(pool.p, pool.n)):
            kr, vr = rows(c["layers"] - 1, b)
            k[at:at + p], v[at:at + p] = kr[:p], vr[:p]
            at += p + n
        return {"active": [k.double(), v.double()]}
    out = torch.empty(st["q"].shape, dtype=torch.float64, device="cuda")
    for l in range(st["q"].shape[0]):
        at = 0
        for b, (p, n) in enumerate(zip(pool.p, pool.n)):
            kr, vr = rows(l if c["kind"] == "stack" else c["layers"] - 1, b)
            kf = torch.cat([kr[:p], st["kn"][l, at:at + n]])
            vf = torch.cat([vr[:p], st["vn"][l, at:at + n]])
            out[l, at:at + n] = _attention64(st["q"][l, at:at + n], kf, vf, p)[0]
            at += n
    return {"out": out, "active": None, "pool": None}
