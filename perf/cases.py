"""What a serving program has this library do, as cases to be timed.

A program that serves long contexts encodes a layer's keys at prefill, appends the keys that leave the
update buffer, and at every decode step retrieves and attends: over all rows in HBM, over the four
regions (Sink, Retrieval, Local, Update Buffer), or with the Retrieval rows in pinned host memory.
The sizes are those of the repository's workloads (tiny, layer32k, batch8_128k, drift, host1m), ragged
neighbours of them, and a wide batch over short contexts with a head count that is no multiple of 4.

Keys follow the workloads' law: a mean offset per channel, unit scale except 4 outlier channels at 8,
values N(0, 1); a query is a planted key plus noise ("needle") or a draw from the key law ("law").
"""

import math

import numpy as np
import torch

import paper_2602_07721_amd as pk

D, B, M, CENTROIDS = 128, 16, 8, 256
SINK, LOCAL, UPDATE = 128, 512, 256  # region sizes of the decode loop
SCALE = D ** -0.5


def _decode(name, batch, hkv, g, n, cand, k, kind="decode", query="needle", **more):
    c = dict(kind=kind, batch=batch, hkv=hkv, g=g, n=n, cand=cand, k=k, query=query, host=False, group=False,
             flags=0, buffered=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def _encode(name, batch, hkv, n, **more):
    c = dict(kind="encode", batch=batch, hkv=hkv, g=4, n=n, flags=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def _append(name, batch, hkv, n, t, rows):
    c = dict(kind="append", batch=batch, hkv=hkv, g=4, n=n, t=t, rows=rows, flags=0)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # Prefill of one layer at 128K tokens: every key is encoded once.
        _encode("encode_128k", 1, 8, 131072),
        # Prefill of a few short prompts of no round length.
        _encode("encode_ragged", 3, 8, 10007),
        # One decode step's new key of every (sequence, KV head), without an update buffer.
        _append("append_step", 4, 8, 33000, 1, False),
        # A buffer update: the 256 oldest Local rows, read from the key cache, join the index.
        _append("append_update", 4, 8, 33000, UPDATE, True),
        # The smallest decode call: one KV head, 8 query heads, 4096 keys.
        _decode("decode_tiny", 1, 1, 8, 4096, 512, 64),
        # One sequence at 32K tokens: the interactive case, latency counts.
        _decode("decode_32k", 1, 8, 4, 32768, 2048, 256),
        # A decode step in a long generation: 4 sequences, any length, queries that ask for many keys.
        _decode("decode_ragged", 4, 8, 4, 45679, 2855, 256, query="law"),
        # Throughput: 8 sequences at 128K tokens.
        _decode("decode_8x128k", 8, 8, 4, 131072, 8192, 512),
        # A wide batch of short contexts, 7 query heads a KV head, the paper's top-100.
        _decode("decode_wide", 16, 4, 7, 7001, 876, 100),
        # Retrieval alone over a million keys, its winners and their estimates handed on.
        _decode("retrieve_1m", 1, 8, 4, 1 << 20, 32768, 1024, kind="retrieve"),
        # A decode step with the four regions resident in HBM, a partly filled update buffer.
        _decode("decode_window", 4, 8, 4, 36500, 2282, 256, kind="window", query="law", buffered=131),
        # The same step with the Retrieval rows in pinned host memory, one sequence at 128K.
        _decode("decode_offload", 1, 8, 4, 131072, 8192, 512, kind="tiered", host=True, buffered=200),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["encode", "append", "decode", "decode", "decode", "retrieve", "window", "tiered", "attend"])
    hkv = rng.choice([1, 2, 4, 8])
    batch = _log_int(rng, 1, 16)
    if kind == "encode":
        n = _log_int(rng, 64, min(131072, (1 << 20) // (batch * hkv)))
        return _encode(None, batch, hkv, n, flags=rng.choice([0, 0, 0, pk.NO_ROTATION, pk.NO_ALPHA_CORRECTION]))
    if kind == "append":
        return _append(None, batch, hkv, _log_int(rng, 256, 65536), _log_int(rng, 1, 2000), rng.random() < 0.5)
    g = rng.choice([1, 2, 3, 4, 4, 5, 7, 8])
    host = kind == "tiered" or (kind == "decode" and rng.random() < 0.2)
    most = (1 << 20) // (1 if kind in ("retrieve", "decode") and not host else 8)
    n = _log_int(rng, 512, max(512, min(most, (1 << 23) // (batch * hkv * ((g + 3) // 4)))))
    k = min(n, rng.choice([32, 64, 100, 256, 512, 1024]))
    if host:  # the rows cross the host link: no more of them than the listed offload step fetches
        k = max(1, min(k, 16384 // (batch * hkv * g)))
    k = max(1, min(k, (1 << 17) // (batch * hkv * g)))
    beta = rng.choice([1 / 32, 1 / 16, 1 / 16, 3 / 32, 1 / 8])
    cand = max(k, min(32768, math.ceil(beta * n), (1 << 21) // (batch * hkv * g)))
    group = host and min(g, 4) * k <= pk.MAX_ATTEND_ROWS and rng.random() < 0.5
    if kind == "attend" and rng.random() < 0.3:
        group = min(g, 4) * k <= pk.MAX_ATTEND_ROWS
    buffered = rng.randrange(UPDATE) if kind in ("window", "tiered") else 0
    flags = rng.choice([0, 0, 0, pk.BINARY_COLLISIONS]) if kind in ("decode", "retrieve") else 0
    return _decode(None, batch, hkv, g, n, cand, k, kind=kind, query=rng.choice(["needle", "law"]), host=host,
                   group=group, flags=flags, buffered=buffered)


# ---------------------------------------------------------------- inputs


def _regions(case):
    """Rows of the decode regions: index row i is cache row SINK + i, then the dense Local + buffer rows."""
    begin = SINK + case["n"]
    return begin, begin + LOCAL + case["buffered"]


def _cache_rows(case):
    if case["kind"] in ("window", "tiered"):
        return _regions(case)[1]
    if case["kind"] == "append":
        return case["n"] + case["t"]
    return case["n"]


def _seed(case, seed):
    text = ",".join(f"{k}={case[k]}" for k in sorted(case) if k != "name") + f",{seed}"
    h = 1469598103934665603
    for ch in text.encode():
        h = ((h ^ ch) * 1099511628211) % (1 << 63)
    return h


def _signs(seed):
    return np.where(np.random.default_rng(seed % (1 << 32)).integers(0, 2, size=D) == 1, -1, 1).astype(np.int8)


def _inputs(case, seed):
    """(K, V or None, q or None, signs) on the GPU."""
    s = _seed(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(s)
    rows, b, h = _cache_rows(case), case["batch"], case["hkv"]

    def randn(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")

    mu = 0.5 * randn(b, h, 1, D)
    scale = torch.ones(b, h, 1, D, device="cuda")
    scale.scatter_(3, torch.rand(b, h, 1, D, generator=gen, device="cuda").argsort(dim=3)[..., :4], 8.0)
    K = randn(b, h, rows, D).mul_(scale).add_(mu).half()
    V = q = None
    if case["kind"] not in ("encode", "append"):
        g = case["g"]
        if case["kind"] != "retrieve":
            V = randn(b, h, rows, D).half()
        if case["query"] == "needle":
            at = torch.randint(0, rows, (b, h, g), generator=gen, device="cuda")
            key = torch.gather(K, 2, at[..., None].expand(b, h, g, D))
            q = (key.float() + 0.1 * randn(b, h, g, D)).half()
        else:
            q = (mu + scale * randn(b, h, g, D)).half()
        q = q.reshape(b, h * g, D).contiguous()
    return K, V, q, _signs(s)


def _pinned(t):
    return torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t)


def _some_rows(case, seed):
    """Ascending distinct key lists, as a retrieval leaves them (for the attention alone)."""
    gen = torch.Generator(device="cuda").manual_seed(_seed(case, seed) ^ 0x5bd1e995)
    b, hq, n, k = case["batch"], case["hkv"] * case["g"], case["n"], case["k"]
    out = torch.empty(b, hq, k, dtype=torch.int32, device="cuda")
    for i in range(b):
        for j in range(hq):
            out[i, j] = torch.randperm(n, generator=gen, device="cuda")[:k].sort().values.int()
    return out


def prepare(case, seed):
    K, V, q, signs = _inputs(case, seed)
    kind, b, h, n = case["kind"], case["batch"], case["hkv"], case["n"]
    capacity = _cache_rows(case) if kind == "append" else n
    cfg = pk.Config(h, case["g"], capacity, signs, flags=case["flags"] if kind == "encode" else 0)
    st = dict(case=case, cfg=cfg)
    if kind != "attend":
        index = pk.Index.empty(cfg, b)
        index.ids.zero_()
        index.rec.zero_()
        st["index"] = index
    if kind == "encode":
        st["keys"] = K
    elif kind == "append":
        pk.encode(cfg, index, K[:, :, :n].contiguous())
        st["counts"] = index.counts.clone()
        st["keys"] = K if case["rows"] else K[:, :, n:].contiguous()
    else:
        st["q"] = q
        st["out"] = torch.empty(b, h * case["g"], D, dtype=torch.float32, device="cuda")
        if kind == "attend":
            st["idx"] = _some_rows(case, seed)
        else:
            keys = K[:, :, SINK:SINK + n].contiguous() if kind in ("window", "tiered") else K
            pk.encode(cfg, index, keys)
            flags = case["flags"] | (pk.GROUP_FETCH if case["group"] else 0)
            budget = pk.Budget(case["cand"], 2 * case["cand"], case["k"], flags)
            st["budget"] = budget
            st["idx"] = torch.empty(b, h * case["g"], case["k"], dtype=torch.int32, device="cuda")
            st["ws"] = torch.empty(pk.retrieve_workspace_size(cfg, b, n, budget), dtype=torch.uint8, device="cuda")
        if kind == "retrieve":
            st["score"] = torch.empty(b, h * case["g"], case["k"], dtype=torch.float32, device="cuda")
        if kind in ("window", "tiered"):
            begin, end = _regions(case)
            st["win"] = pk.Window(SINK, SINK, begin, end)
        if kind == "tiered":
            # Sink at slots [0, SINK), Local and the update buffer in a ring behind them.
            ring = LOCAL + UPDATE
            slots = SINK + (torch.arange(begin, end, device="cuda") - SINK) % ring
            st["K_win"], st["V_win"] = (torch.zeros(b, h, SINK + ring, D, dtype=torch.float16, device="cuda")
                                        for _ in range(2))
            for dst, src in ((st["K_win"], K), (st["V_win"], V)):
                dst[:, :, :SINK] = src[:, :, :SINK]
                dst[:, :, slots] = src[:, :, begin:end]
            K, V = K[:, :, :begin].contiguous(), V[:, :, :begin].contiguous()
        if kind != "retrieve":
            st["K"], st["V"] = (_pinned(K), _pinned(V)) if case["host"] else (K, V)
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- one pass


def run(st):
    case, cfg = st["case"], st["cfg"]
    kind, n = case["kind"], case["n"]
    if kind == "encode":
        ix = st["index"]
        pk.encode(cfg, ix, st["keys"])
        return {"ids": ix.ids, "rec": ix.rec, "counts": ix.counts}
    if kind == "append":
        ix = st["index"]
        ix.counts.copy_(st["counts"])  # the sequence goes on from its saved prefix
        if case["rows"]:
            pk.append_rows(cfg, ix, st["keys"], n, case["t"], n)
        else:
            pk.append(cfg, ix, st["keys"], n)
        return {"ids": ix.ids, "rec": ix.rec, "counts": ix.counts}
    if kind == "attend":
        attend = pk.group_attend if case["group"] else pk.sparse_attend
        attend(cfg, st["q"], st["K"], st["V"], st["idx"], SCALE, out=st["out"])
        return {"out": st["out"]}
    keep = dict(out_idx=st["idx"], workspace=st["ws"])
    if kind == "retrieve":
        pk.retrieve(cfg, st["index"], st["q"], n, st["budget"], out_score=st["score"], **keep)
        return {"idx": st["idx"], "score": st["score"]}
    if kind == "decode":
        pk.retrieve_attend(cfg, st["index"], st["q"], n, st["budget"], st["K"], st["V"], SCALE, out=st["out"],
                           kv_host_mapped=case["host"], **keep)
    elif kind == "window":
        pk.retrieve_window_attend(cfg, st["index"], st["q"], n, st["budget"], st["K"], st["V"], st["win"], SCALE,
                                  out=st["out"], **keep)
    else:
        pk.retrieve_tiered_attend(cfg, st["index"], st["q"], n, st["budget"], st["K_win"], st["V_win"], st["K"],
                                  st["V"], st["win"], SCALE, out=st["out"], kv_host_mapped=case["host"], **keep)
    return {"idx": st["idx"], "out": st["out"]}


# ---------------------------------------------------------------- what a pass cannot do without


def work(case):
    b, h, g, n, kind = case["batch"], case["hkv"], case["g"], case["n"], case["kind"]
    counts = b * h * B * CENTROIDS * 4
    # The transform's additions and, per coordinate, a square, two sums, a product and the binary search of its bin.
    per_key = 7 * D + 7 * D
    if kind in ("encode", "append"):
        t = n if kind == "encode" else case["t"]
        return {"bytes": b * h * t * (2 * D + B + D) + counts * (1 if kind == "encode" else 2),
                "flops": b * h * t * per_key}
    rows, k = b * h * g, case["k"]
    attended = k
    if kind in ("window", "tiered"):
        attended += SINK + LOCAL + case["buffered"]
    moved = rows * D * 2  # queries
    flops = 0
    if kind != "retrieve":
        # Each row once: the dense rows once a KV head, the winners at most once a query head.
        dense = attended - k
        moved += b * h * (dense + min(g * k, n)) * 2 * 2 * D + rows * D * 4
        flops += rows * attended * 4 * D
    if kind != "attend":
        cand = min(case["cand"], n)
        moved += b * h * n * B + counts + b * h * min(g * cand, n) * D + rows * k * 4
        flops += rows * (n * B + cand * 2 * D)
        if kind == "retrieve":
            moved += rows * k * 4
    else:
        moved += rows * k * 4
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] in ("encode", "append"):
        return "exact"  # ids, codes, weights and counts are defined bit for bit
    # Estimates and attention are 32-bit sums of 16-bit inputs.  Two estimates that agree to a few of their last bits
    # may change places at the k-th place, which moves every later entry of that list by one.
    return {"rel": 1e-5, "differ": 0.02}


# ---------------------------------------------------------------- the same in 64 bits


def _levels():
    """Lloyd-Max magnitude quantizer of a coordinate of a uniform direction in 8 dimensions: density (1 - u^2)^2.5."""
    a = (np.arange(8) + 0.5) / 8

    def mass(x):
        t = np.arcsin(x)
        return (20 * t + 15 * np.sin(2 * t) + 3 * np.sin(4 * t) + np.sin(6 * t) / 3) / 64

    def moment(x):
        return -((1 - x * x) ** 3.5) / 7

    for _ in range(20000):
        edge = np.concatenate(([0.0], (a[1:] + a[:-1]) / 2, [1.0]))
        a = np.diff(moment(edge)) / np.diff(mass(edge))
    return (a[1:] + a[:-1]) / 2, a


def _hadamard(device):
    H = torch.ones(1, 1, dtype=torch.float64, device=device)
    while H.shape[0] < D:
        H = torch.cat((torch.cat((H, H), 1), torch.cat((H, -H), 1)), 0)
    return H


def _tree8(x):
    s01, s23, s45, s67 = (x[..., 2 * i] + x[..., 2 * i + 1] for i in range(4))
    return (s01 + s23) + (s45 + s67)


def _summary(keys, signs, levels, flags):
    """(ids [n][B], bins with sign [n][D], W [n][B]) of keys [n][D] by the stated operations in 64 bits."""
    tau, a = levels
    x = keys.double()
    y = x if flags & pk.NO_ROTATION else (x * signs) @ _hadamard(x.device)
    y = y.reshape(-1, B, M)
    ids = ((y < 0).long() << torch.arange(M, device=x.device)).sum(2)
    Y = y * y
    S = _tree8(Y)
    t = torch.zeros_like(y, dtype=torch.long)
    for v in tau:
        t += Y >= ((v * v) * S)[..., None]
    t *= (S > 0)[..., None]
    A = _tree8(torch.from_numpy(a).to(x.device)[t] * y.abs())
    W = torch.sqrt(S) if flags & pk.NO_ALPHA_CORRECTION else S / A
    W = torch.where(S > 0, W, torch.zeros_like(W)).float()
    return ids, ((y < 0).long() << 3 | t).reshape(-1, D), W


def _exact_index(case, seed):
    K, _, _, signs = _inputs(case, seed)
    sg, levels = torch.from_numpy(signs).to(K.device).double(), _levels()
    b, h, rows = K.shape[:3]
    ids8 = torch.zeros(b, h, rows, B, dtype=torch.uint8, device=K.device)
    rec = torch.zeros(b, h, rows, D, dtype=torch.uint8, device=K.device)
    counts = torch.zeros(b, h, B, CENTROIDS, dtype=torch.int32, device=K.device)
    shift = 4 * torch.arange(M, device=K.device)
    for i in range(b):
        for j in range(h):
            ids, codes, W = _summary(K[i, j], sg, levels, case["flags"])
            slot = ids ^ (ids >> 5 & 1) * 0x07 ^ (ids >> 6 & 1) * 0x19 ^ (ids >> 7 & 1) * 0x0E
            ids8[i, j] = slot.to(torch.uint8)
            word = (codes.reshape(-1, B, M) << shift).sum(2)
            word = torch.where(word >= 1 << 31, word - (1 << 32), word).int().reshape(-1, B // 2, 2)
            both = torch.cat((word, W.reshape(-1, B // 2, 2).view(torch.int32)), 2).contiguous()
            rec[i, j] = both.view(torch.uint8).reshape(-1, D)
            for s in range(B):
                counts[i, j, s] = torch.bincount(ids[:, s], minlength=CENTROIDS).int()
    return {"ids": ids8, "rec": rec, "counts": counts}


def _bonus(z, ids, cand, flags):
    """Tier weight [B][256] of every cluster for a transformed query z [D]."""
    dev = z.device
    bits = (torch.arange(CENTROIDS, device=dev)[:, None] >> torch.arange(M, device=dev)) & 1
    proxy = z.reshape(B, M) @ (1.0 - 2.0 * bits.double()).T.contiguous()
    order = torch.sort(proxy, dim=1, descending=True, stable=True).indices
    counts = torch.stack([torch.bincount(ids[:, s], minlength=CENTROIDS) for s in range(B)])
    ranked = torch.gather(counts, 1, order)
    before = ranked.cumsum(1) - ranked
    got = torch.zeros_like(before)
    for pct in (5, 15, 30, 50, 75, 100):
        got += before < (pct * 2 * cand + 99) // 100
    if flags & pk.BINARY_COLLISIONS:
        got = got.clamp(max=1)
    return torch.zeros_like(got).scatter_(1, order, got)


def exact(case, seed):
    if case["kind"] in ("encode", "append"):
        return _exact_index(case, seed)
    K, V, q, signs = _inputs(case, seed)
    dev, b, h, g, n, k = K.device, case["batch"], case["hkv"], case["g"], case["n"], case["k"]
    tau_a, sg = _levels(), torch.from_numpy(signs).to(dev).double()
    a = torch.from_numpy(np.concatenate((tau_a[1], -tau_a[1]))).to(dev)
    first = SINK if case["kind"] in ("window", "tiered") else 0
    dense = torch.zeros(0, dtype=torch.long, device=dev)
    if first:
        begin, end = _regions(case)
        dense = torch.cat((torch.arange(SINK, device=dev), torch.arange(begin, end, device=dev)))
    given = _some_rows(case, seed).long() if case["kind"] == "attend" else None
    H = _hadamard(dev)
    out = torch.zeros(b, h * g, D, dtype=torch.float64, device=dev)
    score = torch.zeros(b, h * g, k, dtype=torch.float64, device=dev)
    cand = min(case["cand"], n)
    for i in range(b):
        for j in range(h):
            if given is None:
                ids, codes, W = _summary(K[i, j, first:first + n], sg, tau_a, 0)
            for r in range(j * g, (j + 1) * g):
                qd = q[i, r].double()
                if given is None:
                    z = (qd * sg) @ H
                    w = _bonus(z, ids, case["cand"], case["flags"])
                    S = torch.zeros(n, dtype=torch.long, device=dev)
                    for s in range(B):
                        S += w[s][ids[:, s]]
                    at = torch.sort(S, descending=True, stable=True).indices[:cand].sort().values
                    part = (a[codes[at]] * (z / D)).reshape(-1, B, M).sum(2)
                    est = (part * W[at].double()).sum(1)
                    top = torch.sort(est, descending=True, stable=True).indices[:k].sort().values
                    score[i, r], won = est[top], at[top]
                else:
                    won = given[i, r]
                if V is not None:
                    rows = torch.cat((dense, first + won))
                    p = torch.softmax(SCALE * (K[i, j, rows].double() @ qd), 0)
                    out[i, r] = p @ V[i, j, rows].double()
    if case["kind"] == "retrieve":
        return {"idx": None, "score": score}
    if case["kind"] == "attend":
        return {"out": out}
    return {"idx": None, "out": out}
