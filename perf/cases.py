"""Performance cases of the ReSA decode path: what a serving program does with
one attention layer on one GPU, through the package's public entry points.

A case names a kind of call and its sizes:

* ``step``       one decode token: ``append_select`` then ``sparse_decode``;
* ``fused``      the same token through ``decode_step``;
* ``period``     one rectification period, f decode tokens and the
                 rectification that ends it, recorded in a HIP graph and replayed;
* ``rectify``    ``dense_rectify`` of the last f rows of a filled cache;
* ``prefill``    ``dense_rectify`` of a prompt or of a prompt chunk of f rows;
* ``summarize``  ``block_summarize`` of a filled cache.

``len`` is the longest sequence; with ``ragged`` the others are shorter. Inputs
are drawn on the GPU from the seed: N(0, 1) rounded to bf16, keys scaled per
(kv head, channel) by LogNormal(0, 0.5) as in caches with outlier channels, and
one block in a hundred shifted along a direction that the group's queries carry
(heavy hitters).
"""
import math

import torch

import paper_2506_04108_amd as R

D = 128
# Tokens a cache of a decode case has room for before the loop starts over.
ROOM = 64


def listed():
    return [
        # The smallest call in use: one token of one short sequence, where
        # launches and host work count most (32 query / 8 kv heads).
        dict(name="decode_4k", kind="step", batch=1, hq=32, hkv=8, len=4096, block=16, sparsity=0.9,
             min_tokens=1024, ragged=False, paged=False),
        # A short sequence as a serving loop runs it: 16 tokens and their
        # rectification, replayed from a graph.
        dict(name="period_4k", kind="period", batch=1, hq=32, hkv=8, len=4096, block=16, sparsity=0.9,
             min_tokens=1024, f=16, ragged=False, paged=False),
        # The one-call decode step on a 7B-class layer (28 query / 4 kv heads).
        dict(name="step_32k_g7", kind="fused", batch=4, hq=28, hkv=4, len=32768, block=16, sparsity=0.9,
             min_tokens=2048, ragged=False, paged=False),
        # The benchmark's token: 8 sequences of 64K.
        dict(name="decode_64k_b8", kind="step", batch=8, hq=32, hkv=8, len=65536, block=16, sparsity=0.9,
             min_tokens=2048, ragged=False, paged=False),
        # One very long sequence: few groups, long selections.
        dict(name="decode_256k", kind="step", batch=1, hq=32, hkv=8, len=262144, block=16, sparsity=0.95,
             min_tokens=4096, ragged=False, paged=False),
        # A continuous batch: odd ragged lengths on a shuffled page pool,
        # 32-token blocks, 8 query heads to a kv head.
        dict(name="decode_paged", kind="step", batch=6, hq=64, hkv=8, len=50001, block=32, sparsity=0.9,
             min_tokens=2048, ragged=True, paged=True),
        # The rectification of a 7B-class layer.
        dict(name="rectify_32k_g7", kind="rectify", batch=4, hq=28, hkv=4, len=32768, block=16, f=32,
             ragged=False, paged=False, masked=0),
        # The benchmark's rectification.
        dict(name="rectify_64k_b8", kind="rectify", batch=8, hq=32, hkv=8, len=65536, block=16, f=32,
             ragged=False, paged=False, masked=0),
        # Whole prompts: a batch of 8K ones, and one of 32K.
        dict(name="prefill_8k_b8", kind="prefill", batch=8, hq=32, hkv=8, len=8192, block=16, f=8192,
             ragged=False, paged=False, masked=0),
        dict(name="prefill_32k", kind="prefill", batch=1, hq=32, hkv=8, len=32768, block=16, f=32768,
             ragged=False, paged=False, masked=0),
        # Chunked prefill in a continuous batch: an odd chunk behind ragged
        # contexts, paged.
        dict(name="prefill_chunk_paged", kind="prefill", batch=2, hq=28, hkv=4, len=33001, block=16, f=2033,
             ragged=True, paged=True, masked=0),
        # Block summaries of a filled cache (after a prefill elsewhere).
        dict(name="summarize_64k_b8", kind="summarize", batch=8, hq=32, hkv=8, len=65536, block=16,
             ragged=False, paged=False),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    largest = max(max(work(c)["bytes"], work(c)["flops"] / 300) for c in listed())
    while True:
        kind = rng.choice(["step", "step", "fused", "period", "rectify", "rectify", "prefill", "prefill",
                           "prefill", "summarize"])
        hkv = rng.choice([2, 4, 8])
        group = rng.choice([1, 2, 3, 4, 4, 5, 6, 7, 8])
        c = dict(kind=kind, batch=rng.randint(1, 8), hq=hkv * group, hkv=hkv,
                 block=rng.choice([16, 16, 32, 64]), ragged=rng.random() < 0.5, paged=rng.random() < 0.35)
        c["len"] = _spread(rng, 1500, 262144)
        if rng.random() < 0.4:
            c["len"] = max(1024, c["len"] // 1024 * 1024)
        if kind in ("step", "fused", "period"):
            c["sparsity"] = rng.choice([0.8, 0.9, 0.9, 0.95])
            c["min_tokens"] = rng.choice([1024, 2048, 4096])
        if kind == "period":
            c["len"] = min(c["len"], 32768)
            c["f"] = rng.choice([16, 32])
        if kind == "rectify":
            c["f"] = rng.choice([1, 8, 16, 32, 32, 64])
            c["masked"] = rng.choice([0, 0, 1]) if c["batch"] > 1 else 0
        if kind == "prefill":
            whole = rng.random() < 0.4 and c["len"] <= 65536  # the longest chunk the call takes
            c["f"] = c["len"] if whole else _spread(rng, 100, min(c["len"], 16384))
            c["masked"] = 0
        # At most 4 Gi elements of cache (three states fit the card many times over).
        if c["batch"] * c["hkv"] * c["len"] * D * 2 > 1 << 32:
            continue
        w = work(c)
        if max(w["bytes"], w["flops"] / 300) <= largest:
            return c


# ------------------------------------------------------------------- inputs

def _lens(case):
    """Length of each sequence before the pass."""
    L, B = case["len"], case["batch"]
    if not case["ragged"]:
        return [L] * B
    least = max(case.get("f", 1), 64)
    return [max(L - (i * 3 * L) // (5 * B) - 5 * i, min(least, L)) for i in range(B)]


def _capacity(case):
    b = case["block"]
    room = ROOM if case["kind"] in ("step", "fused", "period") else 0
    return -(-(case["len"] + room) // b) * b


def _seen_blocks(case):
    """Blocks of the longest sequence a decode case can reach."""
    return -(-(case["len"] + ROOM) // case["block"])


def _n_min(case):
    return -(-case["min_tokens"] // case["block"])


def _count(m, case):
    """Blocks selected of m (the share kept, at least the minimum)."""
    keep = 1000000 - round(case["sparsity"] * 1e6)
    return min(m, max(_n_min(case), 1, -(-m * keep // 1000000)))


def _logical(case, seed):
    """Everything a case's pass reads, in the contiguous layout."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 7919 + 11)
    B, H, hq, b, cap = case["batch"], case["hkv"], case["hq"], case["block"], _capacity(case)
    group, mb = hq // H, _capacity(case) // case["block"]
    lens = _lens(case)
    rnd = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    bf = torch.bfloat16
    x = {"lens": lens}
    scale = torch.empty((H, 1, D), device=dev).log_normal_(0.0, 0.5, generator=g)
    u = rnd(B, H, D)
    u = u / u.norm(dim=-1, keepdim=True)
    K = torch.zeros((B, H, cap, D), dtype=bf, device=dev)
    V = torch.zeros_like(K)
    f = case.get("f", 0)
    for i in range(B):
        have = lens[i] - f if case["kind"] == "prefill" else lens[i]
        if have > 0:
            k = rnd(H, cap, D) * scale
            hot = torch.rand((H, mb), generator=g, device=dev) < 0.01
            k += 2.0 * hot.repeat_interleave(b, dim=1)[..., None] * u[i][:, None]
            K[i, :, :have] = k[:, :have].to(bf)
            V[i, :, :have] = rnd(H, have, D).to(bf)
    x["K"], x["V"] = K, V
    qu = u.repeat_interleave(group, dim=1)
    if case["kind"] in ("step", "fused", "period"):
        n = case["f"] if case["kind"] == "period" else ROOM
        x["q"] = (rnd(n, B, hq, D) + qu).to(bf)
        x["k_new"] = (rnd(n, B, H, D) * scale.view(1, 1, H, D)).to(bf)
        x["v_new"] = rnd(n, B, H, D).to(bf)
    if f:
        x["q_f"] = (rnd(B, hq, f, D) + qu[:, :, None]).to(bf)
        x["k_f"], x["v_f"] = (rnd(B, H, f, D) * scale).to(bf), rnd(B, H, f, D).to(bf)
        if case["kind"] == "rectify":  # re-encoded rows: close to the cached ones
            for i in range(B):
                rows = slice(lens[i] - f, lens[i])
                x["k_f"][i] = (K[i, :, rows].float() + 0.05 * x["k_f"][i].float()).to(bf)
                x["v_f"][i] = (V[i, :, rows].float() + 0.05 * x["v_f"][i].float()).to(bf)
    x["table"] = torch.randperm(B * mb, generator=g, device=dev).view(B, mb).to(torch.int32)
    x["mask"] = torch.tensor([int(i >= case.get("masked", 0)) for i in range(B)], dtype=torch.int32, device=dev)
    return x


def _pages(X, table, b):
    """Contiguous [B, Hkv, capacity, D] as a page pool [pages, Hkv, b, D]."""
    B, H, cap, _ = X.shape
    pool = torch.empty((table.numel(), H, b, D), dtype=X.dtype, device=X.device)
    pool[table.reshape(-1).long()] = X.view(B, H, cap // b, b, D).transpose(1, 2).reshape(-1, H, b, D)
    return pool


class _State:
    pass


def prepare(case, seed):
    x = _logical(case, seed)
    s = _State()
    s.case = case
    dev = x["K"].device
    B, H, hq, b = case["batch"], case["hkv"], case["hq"], case["block"]
    mb = _capacity(case) // b
    K, V, table = x.pop("K"), x.pop("V"), None
    if case["paged"]:
        table = x["table"]
        K, V = _pages(K, table, b), _pages(V, table, b)
    summary = lambda: torch.zeros((B, H, mb, D), dtype=torch.bfloat16, device=dev)  # noqa: E731
    s.cache = R.KVCache(K, V, summary(), summary(), b, table)
    s.lens0 = torch.tensor(x["lens"], dtype=torch.int32, device=dev)
    s.lens = s.lens0.clone()
    s.bound = case["len"]
    if case["kind"] != "summarize":
        R.block_summarize(s.cache, s.lens)
    s.at = 0
    if case["kind"] in ("step", "fused", "period"):
        s.q, s.k_new, s.v_new = x["q"], x["k_new"], x["v_new"]
        s.n_min = _n_min(case)
        s.n_cap = _count(_seen_blocks(case), case)
        n = s.q.shape[0] if case["kind"] == "period" else 1
        s.idx = torch.full((n, B, H, s.n_cap), -1, dtype=torch.int32, device=dev)
        s.nsel = torch.zeros((n, B, H), dtype=torch.int32, device=dev)
        s.out = torch.zeros((n, B, hq, D), device=dev)
        s.lse = torch.zeros((n, B, hq), device=dev)
        s.ws_select, s.ws_decode = R.Workspace(), R.Workspace()
    if "f" in case:
        s.q_f, s.k_f, s.v_f = x["q_f"], x["k_f"], x["v_f"]
        s.mask = x["mask"] if case.get("masked") else None
        s.ws_rectify = R.Workspace()
    if case["kind"] == "rectify" or case["kind"] == "period":
        s.out_f = torch.zeros((B, hq, case["f"], D), device=dev)
        s.lse_f = torch.zeros((B, hq, case["f"]), device=dev)
    if case["kind"] == "period":
        _record(s)
    return s


def _period(s):
    """f decode tokens and the rectification of their rows."""
    c = s.case
    for i in range(c["f"]):
        R.append_select(s.cache, s.k_new[i], s.v_new[i], s.q[i], s.lens, s.bound + i, c["sparsity"], s.n_min, 1,
                        n_cap=s.n_cap, block_idx=s.idx[i], num_sel=s.nsel[i], workspace=s.ws_select)
        R.sparse_decode(s.cache, s.q[i], s.lens, s.idx[i], s.nsel[i], out=s.out[i], lse=s.lse[i],
                        workspace=s.ws_decode)
    R.dense_rectify(s.cache, s.q_f, s.k_f, s.v_f, s.lens, s.bound + c["f"], out=s.out_f, lse=s.lse_f,
                    workspace=s.ws_rectify)


def _record(s):
    """Sizes the workspaces with one eager period, then records one."""
    kept = [t.clone() for t in (s.cache.k, s.cache.v, s.cache.kmin, s.cache.kmax)]
    _period(s)
    for t, old in zip((s.cache.k, s.cache.v, s.cache.kmin, s.cache.kmax), kept):
        t.copy_(old)
    s.lens.copy_(s.lens0)
    torch.cuda.synchronize()
    s.graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(s.graph, stream=side):
        _period(s)
    torch.cuda.current_stream().wait_stream(side)


# --------------------------------------------------------------------- a pass

def _cache_state(s):
    return {"k": s.cache.k, "v": s.cache.v, "kmin": s.cache.kmin, "kmax": s.cache.kmax}


def run(s):
    c = s.case
    if c["kind"] == "summarize":
        R.block_summarize(s.cache, s.lens)
        return {"kmin": s.cache.kmin, "kmax": s.cache.kmax}
    if c["kind"] == "prefill":
        out, lse = R.dense_rectify(s.cache, s.q_f, s.k_f, s.v_f, s.lens, s.bound, workspace=s.ws_rectify)
        return {"out": out, "lse": lse, "cache": _cache_state(s)}
    if c["kind"] == "rectify":
        out, lse = R.dense_rectify(s.cache, s.q_f, s.k_f, s.v_f, s.lens, s.bound, out=s.out_f, lse=s.lse_f,
                                   workspace=s.ws_rectify, seq_mask=s.mask)
        return {"out": out, "lse": lse, "cache": _cache_state(s)}
    if c["kind"] == "period":
        s.lens.copy_(s.lens0)
        s.graph.replay()
        return {"idx": s.idx, "nsel": s.nsel, "out": s.out, "lse": s.lse, "out_f": s.out_f, "lse_f": s.lse_f,
                "lens": s.lens, "cache": _cache_state(s)}
    # One token; once the room is used up the loop starts over.
    if s.at == ROOM:
        s.at = 0
        s.lens.copy_(s.lens0)
    i = s.at
    s.at += 1
    if c["kind"] == "step":
        idx, nsel = R.append_select(s.cache, s.k_new[i], s.v_new[i], s.q[i], s.lens, s.bound + i, c["sparsity"],
                                    s.n_min, 1, n_cap=s.n_cap, block_idx=s.idx[0], num_sel=s.nsel[0],
                                    workspace=s.ws_select)
        out, lse = R.sparse_decode(s.cache, s.q[i], s.lens, idx, nsel, out=s.out[0], lse=s.lse[0],
                                   workspace=s.ws_decode)
    else:
        idx, nsel, out, lse = R.decode_step(s.cache, s.k_new[i], s.v_new[i], s.q[i], s.lens, s.bound + i,
                                            c["sparsity"], s.n_min, 1, n_cap=s.n_cap, block_idx=s.idx[0],
                                            num_sel=s.nsel[0], out=s.out[0], lse=s.lse[0], workspace=s.ws_select)
    return {"idx": idx, "nsel": nsel, "out": out, "lse": lse, "lens": s.lens, "cache": _cache_state(s)}


# ----------------------------------------------------------------------- work

def work(case):
    H, g, b = case["hkv"], case["hq"] // case["hkv"], case["block"]
    nbytes = flops = 0
    f = case.get("f", 0)
    for i, L in enumerate(_lens(case)):
        if case["kind"] in ("step", "fused", "period"):
            for t in range(f if case["kind"] == "period" else 1):
                m = -(-(L + t + 1) // b)
                n = _count(m, case)
                # Summaries, selected rows, queries and new rows in; rows, output and ids out.
                nbytes += H * (512 * m + 512 * n * b + 256 * g + 1024 + 512 * g + 4 * n)
                flops += H * (2 * D * m + 4 * D * g * n * b)
            L += f if case["kind"] == "period" else 0
        if case["kind"] in ("rectify", "prefill", "period") and i >= case.get("masked", 0):
            rows_seen = f * (L - f) + f * (f + 1) // 2
            nbytes += H * (512 * (L - f) + f * (1024 + 256 * g + 512 * g) + 512 * (f // b))
            flops += H * 4 * D * g * rows_seen
        if case["kind"] == "summarize":
            nbytes += H * (256 * L + 512 * (-(-L // b)))
            flops += H * 2 * D * L
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "summarize":
        return "exact"
    if case["kind"] in ("rectify", "prefill"):
        # Weights are rounded to 11 significant bits before the product with
        # V (2.1e-4 off the 64-bit result).
        return {"rel": 1e-3, "max": 2e-2}
    if case["kind"] == "period":
        return {"rel": 1e-3, "max": 2e-2, "differ": 1e-3}
    # fp32 sums in another order (4e-7 off the 64-bit result); ids of near
    # ties may differ.
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}


# ---------------------------------------------------------------------- exact

def _attend64(q, K, V, first, out, lse):
    """Causal attention in 64 bits of rows q [rows, f, D] at positions first + r
    over K, V [L, D], written to out and lse."""
    rows, f, _ = q.shape
    L = K.shape[0]
    step = max(1, (1 << 28) // max(1, rows * L))
    pos = torch.arange(L, device=q.device)
    for r0 in range(0, f, step):
        r1 = min(f, r0 + step)
        end = first + r1
        s = (q[:, r0:r1].reshape(-1, D).double() @ K[:end].t().contiguous()) / math.sqrt(D)
        s = s.view(rows, r1 - r0, end)
        at = torch.arange(r0, r1, device=q.device)[:, None] + first
        s.masked_fill_(pos[:end][None] > at, -math.inf)
        z = torch.logsumexp(s, dim=-1)
        s.sub_(z[..., None]).exp_()
        out[:, r0:r1] = (s.view(-1, end) @ V[:end]).view(rows, r1 - r0, D)
        lse[:, r0:r1] = z


def _rectify64(case, x, lens):
    B, H, hq, f = case["batch"], case["hkv"], case["hq"], case["f"]
    g = hq // H
    out = torch.zeros((B, hq, f, D), dtype=torch.float64, device=x["K"].device)
    lse = torch.zeros((B, hq, f), dtype=torch.float64, device=x["K"].device)
    for i in range(case.get("masked", 0), B):
        for h in range(H):
            K, V = x["K"][i, h, :lens[i]], x["V"][i, h, :lens[i]]
            K[lens[i] - f:], V[lens[i] - f:] = x["k_f"][i, h], x["v_f"][i, h]
            hs = slice(h * g, (h + 1) * g)
            _attend64(x["q_f"][i, hs], K.double(), V.double(), lens[i] - f, out[i, hs], lse[i, hs])
    return out, lse


def _token64(case, x, lens, t):
    """Appends token t to the caches and decodes it in 64 bits."""
    B, H, hq, b = case["batch"], case["hkv"], case["hq"], case["block"]
    g = hq // H
    dev = x["K"].device
    out = torch.zeros((B, hq, D), dtype=torch.float64, device=dev)
    lse = torch.zeros((B, hq), dtype=torch.float64, device=dev)
    for i in range(B):
        L = lens[i] + 1
        m = -(-L // b)
        n = _count(m, case)
        x["K"][i, :, L - 1], x["V"][i, :, L - 1] = x["k_new"][t, i], x["v_new"][t, i]
        inside = torch.arange(m * b, device=dev) < L
        for h in range(H):
            K, V = x["K"][i, h, :m * b].double(), x["V"][i, h, :m * b].double()
            q = x["q"][t, i, h * g:(h + 1) * g].double()
            lo = K.masked_fill(~inside[:, None], math.inf).view(m, b, D).amin(1)
            hi = K.masked_fill(~inside[:, None], -math.inf).view(m, b, D).amax(1)
            mean = q.mean(0)
            score = torch.maximum(lo * mean, hi * mean).sum(-1)
            score[-1] = math.inf
            chosen = torch.zeros(m, dtype=torch.bool, device=dev)
            chosen[torch.sort(score, descending=True, stable=True).indices[:n]] = True
            keep = chosen.repeat_interleave(b) & inside
            s = (q @ K[keep].t().contiguous()) / math.sqrt(D)
            z = torch.logsumexp(s, dim=-1)
            out[i, h * g:(h + 1) * g] = torch.exp(s - z[:, None]) @ V[keep]
            lse[i, h * g:(h + 1) * g] = z
    return out, lse


def exact(case, seed):
    x = _logical(case, seed)
    lens = x["lens"]
    none = {"k": None, "v": None, "kmin": None, "kmax": None}
    if case["kind"] == "summarize":
        B, H, b = case["batch"], case["hkv"], case["block"]
        mb = _capacity(case) // b
        lo = torch.zeros((B, H, mb, D), dtype=torch.float64, device=x["K"].device)
        hi = torch.zeros_like(lo)
        for i in range(B):
            m = -(-lens[i] // b)
            inside = (torch.arange(m * b, device=lo.device) < lens[i])[None, :, None]
            K = x["K"][i, :, :m * b].double()
            lo[i, :, :m] = K.masked_fill(~inside, math.inf).view(H, m, b, D).amin(2)
            hi[i, :, :m] = K.masked_fill(~inside, -math.inf).view(H, m, b, D).amax(2)
        return {"kmin": lo, "kmax": hi}
    if case["kind"] in ("rectify", "prefill"):
        out, lse = _rectify64(case, x, lens)
        return {"out": out, "lse": lse, "cache": none}
    n = case["f"] if case["kind"] == "period" else 1
    outs, lses = [], []
    for t in range(n):
        out, lse = _token64(case, x, lens, t)
        lens = [L + 1 for L in lens]
        outs.append(out)
        lses.append(lse)
    y = {"idx": None, "nsel": None, "out": outs[0], "lse": lses[0], "lens": None, "cache": none}
    if case["kind"] == "period":
        out_f, lse_f = _rectify64(case, x, lens)
        y.update(out=torch.stack(outs), lse=torch.stack(lses), out_f=out_f, lse_f=lse_f)
    return y
