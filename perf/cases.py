"""The work whose time is measured: calls of the library as a serving program makes them.

Every case is one pass through the public entry points on state that such a
program holds in device memory.  The kinds:

  step     voxzip_decode_evict: one generation step of one sequence at its
           budget (append, attention, decayed score, one row evicted)
  decode   voxzip_decode_attend_score: the same without eviction, e.g. a
           sequence whose cache is not (yet) compressed
  ragged   voxzip_decode_attend_score_ragged: one decode step of a batch of
           sequences of mixed lengths in one packed cache
  loop     DecodeLoop.replay(): one token of every slot, each layer's call
           waiting for the previous layer's output, as in a model's forward
           pass, replayed from a HIP graph, evicting every `interval` tokens
  fuse     voxzip_fuse_spans over the prefill's K and V
  embed    voxzip_fuse_spans over audio-token embeddings with text anchors
  prefill  fusion of a long prefill, its attention mass as scores, and the
           eviction down to the budget before the first token

Positions advance by one on every pass, as they do in a decode loop.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_08569_amd as vz
from paper_2608_08569_amd.loop import DecodeLoop

GAMMA = 0.95
N_SINK = 4
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: a toy decoder's one float32 layer, 128 slots
        {"name": "step_f32_tiny", "kind": "step", "dtype": "f32", "L": 1, "Hq": 4, "Hkv": 1, "d": 64, "budget": 128},
        # one layer of a 4x-compressed 4k-token cache (a model that calls layer by layer)
        {"name": "step_layer", "kind": "step", "dtype": "bf16", "L": 1, "Hq": 32, "Hkv": 4, "d": 128, "budget": 1024},
        # the 32k-context cache at its 8192-slot budget, every layer in one call: the headline step
        {"name": "step_long32k", "kind": "step", "dtype": "bf16", "L": 48, "Hq": 32, "Hkv": 4, "d": 128,
         "budget": 8192},
        # a float32 cache: a model evaluated in full precision
        {"name": "step_f32", "kind": "step", "dtype": "f32", "L": 16, "Hq": 16, "Hkv": 4, "d": 128, "budget": 2048},
        # a small decoder with head size 64
        {"name": "decode_d64", "kind": "decode", "dtype": "bf16", "L": 24, "Hq": 14, "Hkv": 2, "d": 64, "T": 4001},
        # the fused 64k-token cache before its first eviction: longer than one part
        {"name": "decode_13k", "kind": "decode", "dtype": "bf16", "L": 48, "Hq": 32, "Hkv": 4, "d": 128, "T": 13181},
        # a batch of eight requests, every layer in one call
        {"name": "ragged_8", "kind": "ragged", "dtype": "bf16", "L": 48, "Hq": 32, "Hkv": 4, "d": 128, "n": 8,
         "lo": 1000, "hi": 8000},
        # one layer of a batch of sixteen requests (the model calls layer by layer)
        {"name": "ragged_16_layer", "kind": "ragged", "dtype": "bf16", "L": 1, "Hq": 32, "Hkv": 4, "d": 128, "n": 16,
         "lo": 1200, "hi": 8100},
        # one token of one request through a 48-layer model, layer after layer
        {"name": "loop_layers", "kind": "loop", "dtype": "bf16", "L": 48, "Hq": 32, "Hkv": 4, "d": 128, "n": 1,
         "budget": 8192, "interval": 16},
        # the start of a 32k-token request
        {"name": "fuse_long32k", "kind": "fuse", "dtype": "bf16", "L": 48, "Hq": 32, "Hkv": 4, "d": 128,
         "T": 32768, "mean": 4.02},
        # the same request fused before the model: audio embeddings of width 3584
        {"name": "embed_long32k", "kind": "embed", "dtype": "bf16", "L": 1, "Hq": 1, "Hkv": 1, "d": 3584,
         "T": 32768, "mean": 4.02},
        # one layer's 64k-token prefill, fused and cut to 5 % as the prefill passes that layer
        {"name": "prefill_64k", "kind": "prefill", "dtype": "bf16", "L": 1, "Hq": 32, "Hkv": 4, "d": 128,
         "T": 65536, "mean": 4.97, "budget": 3277},
    ]


# ---- drawn cases ----

HEADS = [(4, 1), (8, 2), (14, 2), (16, 2), (16, 4), (32, 4), (32, 8), (64, 4), (64, 8)]
MOST_BYTES = 4e9


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "decode", "decode", "ragged", "ragged", "loop", "fuse", "embed", "prefill"])
    Hq, Hkv = rng.choice(HEADS)
    dtype = rng.choice(["bf16", "bf16", "f32"]) if kind != "loop" else "bf16"
    d = rng.choice([64, 128, 128])
    c = {"kind": kind, "dtype": dtype, "L": _logint(rng, 1, 48), "Hq": Hq, "Hkv": Hkv, "d": d}
    if kind == "step":
        c["budget"] = _logint(rng, 96, 8192)
    elif kind == "decode":
        c["T"] = _logint(rng, 200, 32768)
    elif kind == "ragged":
        c["n"] = rng.randint(2, 24)
        c["lo"] = _logint(rng, 100, 3000)
        c["hi"] = c["lo"] + _logint(rng, 10, 8000)
    elif kind == "loop":
        c.update(L=rng.randint(4, 48), d=128, n=rng.randint(1, 4), budget=_logint(rng, 500, 8192), interval=16)
    elif kind == "embed":
        c.update(L=1, Hq=1, Hkv=1, d=8 * rng.randint(128, 1024), T=_logint(rng, 1500, 65536),
                 mean=round(rng.uniform(1.5, 8.0), 2))
    else:
        c["T"] = _logint(rng, 1500, 65536)
        c["mean"] = round(rng.uniform(1.5, 8.0), 2)
        if kind == "prefill":
            c["L"] = rng.randint(1, 8)
            c["budget"] = max(96, int(_spans(c) * rng.uniform(0.1, 0.9)))
    while c["L"] > 1 and work(c)["bytes"] > MOST_BYTES:
        c["L"] = (c["L"] + 1) // 2
    return c


# ---- sizes ----

def _spans(case):
    return max(1, int(round(case["T"] / case["mean"])))


def _lens(case):
    """Resident keys of a batch's sequences, spread over [lo, hi] by their
    logarithm, the longest neither first nor last."""
    n = case["n"]
    x = np.exp(np.linspace(math.log(case["lo"]), math.log(case["hi"]), n)).astype(np.int64)
    x += np.arange(n) % 7  # not all of one parity
    return x[np.argsort((np.arange(n) * 7919 + 3) % (n + 1), kind="stable")]


def _keys(case):
    """Keys per layer that one pass attends over (the appended ones included)."""
    if case["kind"] == "step":
        return case["budget"] + 1
    if case["kind"] == "decode":
        return case["T"]
    if case["kind"] == "ragged":
        return int((_lens(case) + 1).sum())
    return case["n"] * (case["budget"] + 1)


def work(case):
    s = 2 if case["dtype"] == "bf16" else 4
    L, Hq, Hkv, d = case["L"], case["Hq"], case["Hkv"], case["d"]
    row = 2 * Hkv * d * s  # K and V of one token in one layer
    if case["kind"] in ("fuse", "embed", "prefill"):
        n, T = _spans(case), case["T"]
        if case["kind"] == "embed":  # one tensor and its anchors
            return {"bytes": (T + 2 * n) * d * s, "flops": T * d}
        b = L * (T + n) * row
        if case["kind"] == "prefill":  # moved rows read and written (the kept share of the slots past the budget)
            kept = case["budget"] * max(0, n - case["budget"]) / n
            b += L * (8 * n + 2 * kept * (row + 8))
        return {"bytes": b, "flops": 2 * L * T * Hkv * d}
    n = case.get("n", 1)
    T = _keys(case)
    b = L * (T * (row + 8) + n * (row + 2 * Hq * d * s))
    if case["kind"] == "step":
        b += L * (8 * T + 2 * (row + 8))
    return {"bytes": b, "flops": 4 * L * T * Hq * d}


# ---- inputs ----

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape, dtype):
    return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)


def _kv(g, L, Hkv, T, d, dtype):
    """Keys or values: normal, with a scale per channel between 1/2 and 4."""
    x = _normal(g, L, Hkv, T, d, dtype=dtype)
    u = torch.rand(L, Hkv, 1, d, generator=g, device="cuda")
    return x.mul_(torch.exp(math.log(0.5) + u * math.log(8.0)).to(dtype))


def _scores(g, *shape):
    """Decayed attention sums: a heavy-tailed mass of about a few hundredths per key."""
    return torch.exp(2.0 * torch.randn(*shape, generator=g, device="cuda")).mul_(0.01)


def _positions(g, L, n, next_pos, recent):
    """Resident positions of a cache after evictions: the sinks, the recent
    window and a random choice of the others, in mixed slot order."""
    out = torch.empty(L, n, dtype=torch.int32, device="cuda")
    mid = n - N_SINK - recent
    first = torch.arange(N_SINK, device="cuda")
    last = torch.arange(next_pos - recent, next_pos, device="cuda")
    for l in range(L):
        m = torch.randperm(next_pos - N_SINK - recent, generator=g, device="cuda")[:mid] + N_SINK
        p = torch.cat([first, m, last])
        out[l] = p[torch.randperm(n, generator=g, device="cuda")]
    return out


def _offsets(seed, T, n):
    """n contiguous spans over T tokens, cut at random: lengths about geometric."""
    cuts = np.random.default_rng(seed).choice(T - 1, size=n - 1, replace=False) + 1
    off = np.concatenate([[0], np.sort(cuts), [T]]).astype(np.int32)
    return torch.from_numpy(off).cuda()


def _i32(a):
    return torch.from_numpy(np.asarray(a, dtype=np.int32)).cuda()


def _i64(a):
    return torch.from_numpy(np.asarray(a, dtype=np.int64)).cuda()


def prepare(case, seed):
    g, dt = _gen(seed), DTYPE[case["dtype"]]
    kind, L, Hq, Hkv, d = case["kind"], case["L"], case["Hq"], case["Hkv"], case["d"]
    st = {"case": case}
    if kind in ("step", "decode"):
        n = case["budget"] if kind == "step" else case["T"] - 1
        cap = n + 2
        st.update(n=n, q=_normal(g, L, Hq, d, dtype=dt), kn=_kv(g, L, Hkv, 1, d, dt)[:, :, 0].contiguous(),
                  vn=_kv(g, L, Hkv, 1, d, dt)[:, :, 0].contiguous(), k=_kv(g, L, Hkv, cap, d, dt),
                  v=_kv(g, L, Hkv, cap, d, dt), s=_scores(g, L, cap),
                  p=torch.zeros(L, cap, dtype=torch.int32, device="cuda"),
                  out=torch.zeros(L, Hq, d, dtype=dt, device="cuda"))
        st["next"] = 2 * n if kind == "step" else n
        st["p"][:, :n] = (_positions(g, L, n, 2 * n, n // 5) if kind == "step"
                          else torch.arange(n, dtype=torch.int32, device="cuda"))
        st["ws"] = vz.workspace(vz.VZ_OP_DECODE_EVICT if kind == "step" else vz.VZ_OP_DECODE, L, Hq, Hkv, d, cap)
    elif kind == "ragged":
        lens = _lens(case)
        n, caps = case["n"], lens + 17
        total = int(caps.sum())
        base = np.concatenate([[0], np.cumsum(caps)[:-1]])
        st.update(q=_normal(g, n, L, Hq, d, dtype=dt), kn=_normal(g, n, L, Hkv, d, dtype=dt),
                  vn=_normal(g, n, L, Hkv, d, dtype=dt), k=_kv(g, L, Hkv, total, d, dt),
                  v=_kv(g, L, Hkv, total, d, dt), s=_scores(g, L, total),
                  p=torch.zeros(L, total, dtype=torch.int32, device="cuda"),
                  out=torch.zeros(n, L, Hq, d, dtype=dt, device="cuda"), base=_i64(base), cap=_i32(caps),
                  len=_i32(lens), next=_i32(lens),
                  ws=vz.workspace_ragged(vz.VZ_OP_DECODE, L, Hq, Hkv, d, total, n))
        for b, m in zip(base, lens):
            st["p"][:, int(b): int(b + m)] = torch.arange(int(m), dtype=torch.int32, device="cuda")
    elif kind == "loop":
        n, B, iv = case["n"], case["budget"], case["interval"]
        lp = DecodeLoop(L, Hq, Hkv, d, [B + iv + 1] * n, [B] * n, GAMMA, interval=iv)
        lp.k.copy_(_kv(g, L, Hkv, lp.total, d, dt))
        lp.v.copy_(_kv(g, L, Hkv, lp.total, d, dt))
        lp.score.copy_(_scores(g, L, lp.total))
        for i in range(n):
            lp.pos[:, i * (B + iv + 1): i * (B + iv + 1) + B] = _positions(g, L, B, 2 * B, B // 5)
        lp.set_lengths([B] * n, [2 * B] * n)
        q = _normal(g, L, n, 1, Hq, d, dtype=dt)
        kn, vn = (_normal(g, L, n, 1, Hkv, d, dtype=dt) for _ in range(2))
        mixed = torch.zeros_like(q)

        def layer_query(l, q, outs):
            return q[0] if l == 0 else torch.add(q[l], outs[l - 1], out=mixed[l])

        lp.capture(q, kn, vn, layer_query)
        st.update(lp=lp, q=q, kn=kn, vn=vn)
    elif kind == "embed":
        T, n = case["T"], _spans(case)
        st.update(x=_normal(g, 1, 1, T, d, dtype=dt), anchor=_normal(g, 1, 1, n, d, dtype=dt),
                  y=torch.zeros(1, 1, n, d, dtype=dt, device="cuda"), off=_offsets(seed, T, n),
                  s=torch.zeros(1, n, device="cuda"), p=torch.zeros(1, n, dtype=torch.int32, device="cuda"))
        # background spans carry no text: their anchors are zero rows
        st["anchor"].mul_((torch.rand(1, 1, n, 1, generator=g, device="cuda") < 0.7).to(dt))
    else:
        T, n = case["T"], _spans(case)
        st.update(ki=_kv(g, L, Hkv, T, d, dt), vi=_kv(g, L, Hkv, T, d, dt), off=_offsets(seed, T, n),
                  k=torch.zeros(L, Hkv, n + 2, d, dtype=dt, device="cuda"),
                  v=torch.zeros(L, Hkv, n + 2, d, dtype=dt, device="cuda"),
                  s=torch.zeros(L, n + 2, device="cuda"),
                  p=torch.zeros(L, n + 2, dtype=torch.int32, device="cuda"))
        if kind == "prefill":
            st["mass"] = _scores(g, L, n)
            st["ws"] = vz.workspace(vz.VZ_OP_EVICT, L, Hq, Hkv, d, n + 2)
    return st


# ---- one pass ----

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        vz.voxzip_decode_evict(st["q"], st["kn"], st["vn"], st["k"], st["v"], st["s"], st["p"], st["out"], st["n"],
                               st["next"], GAMMA, case["budget"], n_sink=N_SINK, workspace=st["ws"])
        st["next"] += 1
    elif kind == "decode":
        vz.voxzip_decode_attend_score(st["q"], st["kn"], st["vn"], st["k"], st["v"], st["s"], st["p"], st["out"],
                                      st["n"], st["next"], GAMMA, workspace=st["ws"])
        st["next"] += 1
    elif kind == "ragged":
        vz.voxzip_decode_attend_score_ragged(st["q"], st["kn"], st["vn"], st["k"], st["v"], st["s"], st["p"],
                                             st["out"], st["base"], st["cap"], st["len"], st["next"], GAMMA,
                                             workspace=st["ws"])
        st["next"].add_(1)
    elif kind == "loop":
        lp = st["lp"]
        lp.replay()
        return {"out": list(lp.out_layers), "k": lp.k, "v": lp.v, "score": lp.score, "pos": lp.pos, "len": lp.length}
    elif kind == "embed":
        vz.voxzip_fuse_spans(st["x"], None, st["off"], st["y"], None, st["s"], st["p"], anchor_k=st["anchor"])
        return {"y": st["y"], "score": st["s"], "pos": st["p"]}
    else:
        vz.voxzip_fuse_spans(st["ki"], st["vi"], st["off"], st["k"], st["v"], st["s"], st["p"])
        if kind == "prefill":
            n = st["mass"].shape[1]
            st["s"][:, :n] = st["mass"]
            vz.voxzip_evict_compact(st["k"], st["v"], st["s"], st["p"], n, case["budget"], n, n_sink=N_SINK,
                                    workspace=st["ws"])
        return {"k": st["k"], "v": st["v"], "score": st["s"], "pos": st["p"]}
    return {"out": st["out"], "k": st["k"], "v": st["v"], "score": st["s"], "pos": st["p"]}


def tolerance(case):
    """bfloat16 caches: outputs rounded to 8 bits (and, in the MFMA paths,
    probabilities too); float32: sums of up to a few thousand terms in another
    order.  Each about four times the error measured against 64 bits."""
    if case["kind"] == "loop":  # a rounding travels through every later layer's query
        return {"rel": 0.016, "max": 0.3}
    if case["kind"] in ("fuse", "embed", "prefill"):
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 8e-3, "max": 2e-2}
    return {"rel": 1e-5, "max": 1e-3} if case["dtype"] == "f32" else {"rel": 8e-3, "max": 8e-2}


# ---- the same in 64 bits ----

def _attend(q, kn, vn, k, v, s, n):
    """One layer of one sequence: keys 0 .. n - 1 and the new one; output and
    decayed scores of the n + 1 slots."""
    Hq, d = q.shape
    Hkv = kn.shape[0]
    q = q.double().view(Hkv, Hq // Hkv, d)
    K = torch.cat([k[:, :n].double(), kn.double()[:, None]], 1)
    V = torch.cat([v[:, :n].double(), vn.double()[:, None]], 1)
    a = torch.softmax(torch.bmm(q, K.transpose(1, 2).contiguous()) / math.sqrt(d), -1)
    new = torch.zeros(n + 1, dtype=torch.float64, device=q.device)
    new[:n] = GAMMA * s[:n].double()
    return torch.bmm(a, V).view(Hq, d), new + a.sum((0, 1))


def _kept_moves(score, pos, n, budget, next_pos):
    """Slots to fill and the slots that fill them (Sec. 3.2.2, Eq. 7-9), in slot order."""
    p = pos[:n].long()
    mid = (p >= N_SINK) & (p < next_pos - budget // 5)
    order = np.lexsort((-p.cpu().numpy(), score[:n].cpu().numpy()))  # smallest score first, then the larger position
    order = torch.from_numpy(order).to(p.device)
    gone = torch.zeros(n, dtype=torch.bool, device=p.device)
    gone[order[mid[order]][: n - budget]] = True
    return gone[:budget].nonzero()[:, 0], (~gone[budget:]).nonzero()[:, 0] + budget


def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    L = case["L"]
    if kind == "loop":
        lp, prev, outs = st["lp"], None, []
        s, B = lp.score.double(), case["budget"]
        for l in range(L):
            # the program's own bfloat16 query; everything after it in 64 bits
            ql = st["q"][0] if l == 0 else st["q"][l] + prev.to(torch.bfloat16)
            prev = torch.zeros_like(ql, dtype=torch.float64)
            for i, b in enumerate(lp.seq_base.tolist()):
                prev[i, 0], s[l, b: b + B + 1] = _attend(ql[i, 0], st["kn"][l, i, 0], st["vn"][l, i, 0],
                                                        lp.k[l, :, b: b + B], lp.v[l, :, b: b + B],
                                                        lp.score[l, b: b + B], B)
            outs.append(prev)
        return {"out": outs, "k": None, "v": None, "score": s, "pos": None, "len": None}
    if kind == "ragged":
        out, s = torch.zeros_like(st["out"], dtype=torch.float64), st["s"].double()
        for i, (b, n) in enumerate(zip(st["base"].tolist(), st["len"].tolist())):
            for l in range(L):
                out[i, l], s[l, b: b + n + 1] = _attend(st["q"][i, l], st["kn"][i, l], st["vn"][i, l],
                                                       st["k"][l, :, b: b + n], st["v"][l, :, b: b + n],
                                                       st["s"][l, b: b + n], n)
        return {"out": out, "k": None, "v": None, "score": s, "pos": None}
    if kind in ("step", "decode"):
        n = st["n"]
        out, s = torch.zeros_like(st["out"], dtype=torch.float64), st["s"].double()
        for l in range(L):
            out[l], s[l, : n + 1] = _attend(st["q"][l], st["kn"][l], st["vn"][l], st["k"][l], st["v"][l], st["s"][l],
                                            n)
            if kind == "step":
                pos = torch.cat([st["p"][l, :n], torch.tensor([st["next"]], dtype=torch.int32, device="cuda")])
                holes, movers = _kept_moves(s[l], pos, n + 1, case["budget"], st["next"] + 1)
                s[l, holes] = s[l, movers]
        return {"out": out, "k": None, "v": None, "score": s, "pos": None}
    n, off = _spans(case), st["off"].long()
    length = (off[1:] - off[:-1]).double()[:, None]
    span = torch.repeat_interleave(torch.arange(n, device="cuda"), off[1:] - off[:-1])

    def mean(x):
        y = torch.zeros(n, x.shape[-1], dtype=torch.float64, device="cuda")
        return y.index_add_(0, span, x.double()) / length

    if kind == "embed":
        return {"y": (mean(st["x"][0, 0]) + st["anchor"][0, 0].double())[None, None], "score": None, "pos": None}
    k, v = (torch.zeros_like(x, dtype=torch.float64) for x in (st["k"], st["v"]))
    for l in range(L):
        for h in range(case["Hkv"]):
            k[l, h, :n], v[l, h, :n] = mean(st["ki"][l, h]), mean(st["vi"][l, h])
        if kind == "prefill":
            pos = torch.arange(n, dtype=torch.int32, device="cuda")
            holes, movers = _kept_moves(st["mass"][l], pos, n, case["budget"], n)
            k[l][:, holes], v[l][:, holes] = k[l][:, movers], v[l][:, movers]
    return {"k": k, "v": v, "score": None, "pos": None}
