"""The work a user of this library has it do, as cases that can be timed.

Trainer side: eviction-masked attention over compacted agent traces, as whole
training steps through autograd, as a scoring pass (forward alone, for
log-probabilities of an old policy) and as a backward alone.  Inference side:
decode over the streamed paged KV cache, and a turn of a rollout (append,
decode, evict).  Every case goes through the package's public entry points.

``listed`` names the cases, ``draw`` makes more of the same ranges.
"""
import math

import numpy as np
import torch

from paper_2609_35750_amd import inputs, kvs
from paper_2609_35750_amd.paged import PagedKVCache

DEV = "cuda"


# ---------------------------------------------------------------- the cases
def _attn(name, kind, Hq, Hkv, D, n, lo, hi, lseed, p, w, s, strategy, prescaled=False, varlen=False):
    return {"name": name, "kind": kind, "Hq": Hq, "Hkv": Hkv, "D": D, "n": n, "lo": lo, "hi": hi, "lseed": lseed,
            "p": p, "w": w, "s": s, "strategy": strategy, "prescaled": prescaled, "varlen": varlen}


def _cache(name, kind, Hq, Hkv, D, seqs, lo, hi, lseed, block, gone, turn=0, room=2):
    return {"name": name, "kind": kind, "Hq": Hq, "Hkv": Hkv, "D": D, "seqs": seqs, "lo": lo, "hi": hi,
            "lseed": lseed, "block": block, "gone": gone, "turn": turn, "room": room}


def listed():
    return [
        # the smallest trainer call: one 512-token trace of a tiny model; launches and latency
        _attn("train_512", "train", 4, 4, 64, 1, 512, 512, 0, 64, 128, 32, "keep_all"),
        # a packed minibatch of short, ragged tool-call traces (SFT); groups of 8
        _attn("train_short_varlen", "train", 16, 2, 128, 24, 100, 1500, 7, 64, 256, 32, "latest_only", varlen=True),
        # an ordinary step of two equal traces, one token past a power of two
        _attn("train_2x4k", "train", 32, 8, 128, 2, 4097, 4097, 0, 512, 1024, 128, "keep_all"),
        # head dimension 64, an odd group and an odd length, latest summary only
        _attn("train_8k_d64", "train", 24, 8, 64, 1, 8191, 8191, 0, 512, 1536, 128, "latest_only"),
        # scoring pass: forward over the 16k trace (old-policy log-probabilities)
        _attn("forward_16k", "forward", 32, 8, 128, 1, 16384, 16384, 0, 1024, 4096, 512, "keep_all", prescaled=True),
        # the backward of that trace by itself (activations kept from an earlier forward)
        _attn("backward_16k", "backward", 32, 8, 128, 1, 16384, 16384, 0, 1024, 4096, 512, "keep_all",
              prescaled=True),
        # 32k trace under a turn-level sliding window: a mask with many boundaries
        _attn("train_32k_sliding", "train", 32, 8, 128, 1, 32768, 32768, 0, 1024, 10, 0, "sliding_window"),
        # the largest: eight packed rollouts of 4k to 24k tokens, groups of 5
        _attn("train_varlen8_gqa5", "train", 40, 8, 128, 8, 4096, 24576, 39, 512, 2048, 256, "keep_all", varlen=True),
        # one decode step of 64 concurrent rollouts, 16-token blocks
        _cache("decode_64x4k", "decode", 32, 8, 128, 64, 4096, 4096, 0, 16, 4096),
        # one decode step of a single long rollout, block size 1: latency
        _cache("decode_1x16k", "decode", 32, 8, 128, 1, 16000, 16000, 0, 1, 4096),
        # ragged rollouts whose evictions leave partly empty blocks, head dimension 64
        _cache("decode_ragged_d64", "decode", 24, 8, 64, 24, 200, 9000, 11, 16, 1001),
        # a turn of eight rollouts: its tokens are cached, every rollout decodes, the compaction evicts the turn
        _cache("rollout_turn", "rollout", 32, 8, 128, 8, 1000, 6000, 5, 16, 500, turn=384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST_FLOPS = 14 * 128 * 40 * 251_210_050     # the largest listed case
_MOST_BYTES = 64 * 4096 * 8 * 128 * 4         # the largest listed cache


def draw(rng):
    kind = rng.choice(["train", "train", "train", "forward", "backward", "decode", "decode", "rollout"])
    D = rng.choice([64, 128, 128])
    Hkv = rng.choice([1, 2, 4, 8, 8])
    G = rng.choice([1, 2, 3, 4, 4, 5, 8, 16])
    while Hkv * G > 64:
        G //= 2
    lseed = rng.randrange(1 << 20)
    if kind in ("decode", "rollout"):
        block = rng.choice([1, 16, 16, 5])
        seqs = _log_int(rng, 1, 128 if kind == "decode" else 16)
        top = min(20000, max(64, _MOST_BYTES // (seqs * Hkv * D * 4)))
        hi = _log_int(rng, 64, top)
        lo = rng.choice([hi, max(1, hi // 8)])
        turn = _log_int(rng, 1, 1024) if kind == "rollout" else 0
        c = _cache("", kind, Hkv * G, Hkv, D, seqs, lo, hi, lseed, block, rng.randrange(0, hi), turn,
                   rng.choice([1, 2, 4]))
        del c["name"]
        return c
    form = rng.choice(["one", "one", "batch", "varlen"])
    while True:
        total = _log_int(rng, 256, 65536)
        n = 1 if form == "one" else rng.randint(2, 4) if form == "batch" else rng.randint(2, 32)
        hi = max(33, total // n)
        lo = hi if form != "varlen" else max(1, hi // rng.choice([2, 6, 20]))
        p = rng.randrange(0, max(1, hi // 8))
        strategy = rng.choice(["keep_all", "latest_only", "last2", "sliding_window"])
        w = rng.randint(2, 12) if strategy == "sliding_window" else _log_int(rng, 16, max(17, hi // 3))
        s = 0 if strategy == "sliding_window" else max(1, w // rng.randint(4, 16))
        c = _attn("", kind, Hkv * G, Hkv, D, n, lo, hi, lseed, p, w, s, strategy, rng.random() < 0.3, form == "varlen")
        del c["name"]
        if work(c)["flops"] <= _MOST_FLOPS:
            return c


# ---------------------------------------------------------------- attention inputs
def _lengths(c):
    """Trace lengths: fixed by the case, uniform on [lo, hi]."""
    if c["lo"] == c["hi"]:
        return (c["hi"],) * c["n"]
    return inputs.varlen_lengths(c["n"], c["lo"], c["hi"], c["lseed"])


def _evict(c):
    """evict_at of every trace (trace-local), as a list."""
    out = []
    for b, L in enumerate(_lengths(c)):
        p = min(c["p"], L)
        if c["strategy"] == "sliding_window":
            # turns of 1/8 to 2 times a typical length, padded to the engine's 16-token blocks
            typ = max(32, min(512, L // (3 * c["w"])))
            e = inputs.turn_trace(L, p, "sliding_window", c["w"], 1, 0, max(1, typ // 8), 2 * typ, 16, c["lseed"], b)[0]
        else:
            e = inputs.evict_at_layout(L, p, c["w"], c["s"], c["strategy"])
        out.append(e)
    return out


def _pairs(c):
    """Visible (query, key) pairs of one head over all traces."""
    return sum(int((e.astype(np.int64) - np.arange(len(e))).sum()) for e in _evict(c))


def _scale(c):
    return 1.0 if c.get("prescaled") else 1.0 / math.sqrt(c["D"])


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32).to(torch.bfloat16)


def _tensors(c, seed):
    """Packed bf16 q, k, v, do: unit-variance activations, Q scaled by 1/sqrt(D) where the case says so."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    n = sum(_lengths(c))
    q = torch.randn(n, c["Hq"], c["D"], generator=gen, device=DEV, dtype=torch.float32)
    if c["prescaled"]:
        q *= 1.0 / math.sqrt(c["D"])
    q = q.to(torch.bfloat16)
    return q, _randn(gen, n, c["Hkv"], c["D"]), _randn(gen, n, c["Hkv"], c["D"]), _randn(gen, n, c["Hq"], c["D"])


# ---------------------------------------------------------------- cache inputs
def _cache_plan(c):
    """Per sequence: (entries cached, first evicted position, one past the last evicted position)."""
    rng = np.random.default_rng([c["lseed"], 1])
    out = []
    for _ in range(c["seqs"]):
        live = int(rng.integers(c["lo"], c["hi"], endpoint=True))
        gone = c["gone"]
        a = live // 3
        out.append((live + gone, a, a + gone))
    return out


def _cache_tensors(c, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    Hkv, D = c["Hkv"], c["D"]
    q = _randn(gen, c["seqs"], c["Hq"], D)
    kv = [(_randn(gen, m, Hkv, D), _randn(gen, m, Hkv, D)) for m, _, _ in _cache_plan(c)]
    turn = [(_randn(gen, c["turn"], Hkv, D), _randn(gen, c["turn"], Hkv, D)) for _ in range(c["seqs"])]
    return q, kv, turn


# ---------------------------------------------------------------- prepare and run
def prepare(case, seed):
    c = case
    if c["kind"] in ("decode", "rollout"):
        q, kv, turn = _cache_tensors(c, seed)
        plan = _cache_plan(c)
        need = max(-(-(m + c["turn"]) // c["block"]) + 1 for m, _, _ in plan)
        total = sum(-(-(m + c["turn"]) // c["block"]) + 2 for m, _, _ in plan)
        cache = PagedKVCache(total, c["block"], c["seqs"], need * c["room"], c["Hkv"], c["D"], DEV)
        # the rollouts' entries arrive interleaved; a compaction fires before the last part of each
        cut = lambda m, a, z, i: (0, a, z, m)[i]  # noqa: E731
        for part in range(3):
            for s, (m, a, z) in enumerate(plan):
                x, y = cut(m, a, z, part), cut(m, a, z, part + 1)
                if y > x:
                    cache.append(s, np.arange(x, y), kv[s][0][x:y], kv[s][1][x:y])
            if part == 1:
                for s, (m, a, z) in enumerate(plan):
                    if z > a:
                        cache.evict(s, np.arange(a, z))
        st = {"kind": c["kind"], "cache": cache, "q": q}
        if c["kind"] == "rollout":
            st["turn"] = [(np.arange(m, m + c["turn"]), tk, tv) for (m, _, _), (tk, tv) in zip(plan, turn)]
        else:
            cache.device_tables()
        return st

    q, k, v, do = _tensors(c, seed)
    L = _lengths(c)
    e = torch.from_numpy(np.concatenate(_evict(c))).to(DEV)
    kw = {}
    if c["varlen"]:
        kw = {"cu_seqlens": torch.from_numpy(np.concatenate([[0], np.cumsum(L)]).astype(np.int32)).to(DEV),
              "max_seqlen": max(L)}
    else:
        q, k, v, do = (x.view(c["n"], L[0], x.shape[1], x.shape[2]) for x in (q, k, v, do))
        e = e.view(c["n"], L[0])
    st = {"kind": c["kind"], "q": q, "k": k, "v": v, "do": do, "e": e, "scale": _scale(c), "kw": kw}
    if c["kind"] == "train":
        for n in ("q", "k", "v"):
            st[n].requires_grad_(True)
    if c["kind"] == "backward":
        st["o"], st["lse"] = kvs.kvs_evict_attn_fwd(q, k, v, e, st["scale"], **kw)
    return st


def run(state):
    s = state
    if s["kind"] == "train":
        o, lse = kvs.evict_attn(s["q"], s["k"], s["v"], s["e"], s["scale"], **s["kw"])
        dq, dk, dv = torch.autograd.grad(o, (s["q"], s["k"], s["v"]), s["do"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if s["kind"] == "forward":
        o, lse = kvs.kvs_evict_attn_fwd(s["q"], s["k"], s["v"], s["e"], s["scale"], **s["kw"])
        return {"o": o, "lse": lse}
    if s["kind"] == "backward":
        dq, dk, dv = kvs.kvs_evict_attn_bwd(s["do"], s["q"], s["k"], s["v"], s["o"], s["lse"], s["e"], s["scale"],
                                            **s["kw"])
        return {"dq": dq, "dk": dk, "dv": dv}
    cache = s["cache"]
    if s["kind"] == "decode":
        o, lse = cache.decode(s["q"])
        return {"o": o, "lse": lse}
    for i, (pos, tk, tv) in enumerate(s["turn"]):
        cache.append(i, pos, tk, tv)
    o, lse = cache.decode(s["q"])
    for i, (pos, _, _) in enumerate(s["turn"]):
        cache.evict(i, pos)
    return {"o": o, "lse": lse, "slot_pos": cache.slot_pos, "k": cache.k, "v": cache.v}


# ---------------------------------------------------------------- work and tolerance
def work(case):
    c = case
    D, Hq, Hkv = c["D"], c["Hq"], c["Hkv"]
    if c["kind"] in ("decode", "rollout"):
        new = c["turn"] * c["seqs"]
        live = sum(m - (z - a) for m, a, z in _cache_plan(c)) + new
        b = live * (Hkv * D * 4 + 4) + c["seqs"] * Hq * (4 * D + 4)
        # a turn: its K and V are read and written to the cache, its slots marked live and evicted again
        b += new * (Hkv * D * 8 + 16)
        return {"bytes": b, "flops": 4 * D * Hq * live}
    n = sum(_lengths(c))
    qb, kb, lb = 2 * n * Hq * D, 2 * n * Hkv * D, 4 * n * Hq
    fwd, bwd = (qb + 2 * kb + 4 * n) + (qb + lb), (3 * qb + 2 * kb + lb + 4 * n) + (qb + 2 * kb)
    pairs = _pairs(c) * Hq * D
    per, byt = {"train": (14, fwd + bwd), "forward": (4, fwd), "backward": (10, bwd)}[c["kind"]]
    return {"bytes": byt, "flops": per * pairs}


def tolerance(case):
    # bf16 results of bf16 inputs with fp32 sums and 16-bit probabilities in the products: 1.3e-3 to 3.5e-3
    # (2-norm) from the 64-bit values over the listed and drawn cases; about four times that
    return {"rel": 1e-2}


# ---------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    c = case
    if c["kind"] in ("decode", "rollout"):
        return _exact_decode(c, seed)
    q, k, v, do = _tensors(c, seed)
    Hq, Hkv, D, G = c["Hq"], c["Hkv"], c["D"], c["Hq"] // c["Hkv"]
    n, scale = q.shape[0], _scale(c)
    back = c["kind"] != "forward"
    f64 = dict(dtype=torch.float64, device=DEV)
    o, lse = torch.empty(n, Hq, D, **f64), torch.empty(Hq, n, **f64)
    dq, dk, dv = (torch.zeros(x, **f64) for x in ((n, Hq, D), (n, Hkv, D), (n, Hkv, D)))
    t0 = 0
    for e_np in _evict(c):
        L = len(e_np)
        e = torch.from_numpy(e_np.astype(np.int64)).to(DEV)
        j = torch.arange(L, device=DEV)
        step = max(16, min(1024, (1 << 26) // (G * max(L, 1))))
        for i0 in range(0, L, step):
            i1 = min(i0 + step, L)
            cols = torch.nonzero((j < i1) & (e > i0)).squeeze(1)     # keys some row of the block sees
            i = torch.arange(i0, i1, device=DEV)
            hidden = ~((cols[None, :] <= i[:, None]) & (i[:, None] < e[cols][None, :]))
            hidden = hidden.repeat(G, 1)
            for g in range(Hkv):
                heads = slice(g * G, (g + 1) * G)
                rows = lambda x: x[t0 + i0:t0 + i1, heads].transpose(0, 1).reshape(-1, D).double()  # noqa: E731,B023
                qs, ks, vs = rows(q), k[t0 + cols, g].double(), v[t0 + cols, g].double()
                sc = (qs @ ks.t().contiguous()).mul_(scale).masked_fill_(hidden, -math.inf)
                ls = torch.logsumexp(sc, 1)
                p = sc.sub_(ls[:, None]).exp_()
                os_ = p @ vs
                o[t0 + i0:t0 + i1, heads] = os_.view(G, i1 - i0, D).transpose(0, 1)
                lse[heads, t0 + i0:t0 + i1] = ls.view(G, i1 - i0)
                if back:
                    dos = rows(do)
                    dv[t0 + cols, g] += p.t().contiguous() @ dos
                    ds = (dos @ vs.t().contiguous()).sub_((dos * os_).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    dq[t0 + i0:t0 + i1, heads] = (ds @ ks).view(G, i1 - i0, D).transpose(0, 1)
                    dk[t0 + cols, g] += ds.t().contiguous() @ qs
        t0 += L
    if not c["varlen"]:
        B, T = c["n"], n // c["n"]
        o, dq, dk, dv = (x.view(B, T, *x.shape[1:]) for x in (o, dq, dk, dv))
        lse = lse.view(Hq, B, T).transpose(0, 1).contiguous()
    out = {"o": o, "lse": lse} if c["kind"] != "backward" else {}
    if back:
        out.update(dq=dq, dk=dk, dv=dv)
    return out


def _exact_decode(c, seed):
    q, kv, turn = _cache_tensors(c, seed)
    Hkv, G, D = c["Hkv"], c["Hq"] // c["Hkv"], c["D"]
    o = torch.empty(c["seqs"], c["Hq"], D, dtype=torch.float64, device=DEV)
    lse = torch.empty(c["seqs"], c["Hq"], dtype=torch.float64, device=DEV)
    for s, (m, a, z) in enumerate(_cache_plan(c)):
        k = torch.cat([kv[s][0][:a], kv[s][0][z:], turn[s][0]]).double()
        v = torch.cat([kv[s][1][:a], kv[s][1][z:], turn[s][1]]).double()
        for g in range(Hkv):
            sc = (q[s, g * G:(g + 1) * G].double() @ k[:, g].t().contiguous()) * _scale(c)
            lse[s, g * G:(g + 1) * G] = torch.logsumexp(sc, 1)
            o[s, g * G:(g + 1) * G] = torch.softmax(sc, 1) @ v[:, g].contiguous()
    out = {"o": o, "lse": lse}
    if c["kind"] == "rollout":
        out.update(slot_pos=None, k=None, v=None)
    return out
