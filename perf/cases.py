"""The work that users of this package give it, as measured cases.

A case is one call (or one chain of calls) through the package's public entry points at one set of sizes:

  score   msa_score_topk: routing of queries against a resident routing index
  attend  msa_sparse_attend: attention over selected documents and the local context
  encode  msa_build_routing_keys + msa_pool_kv: the offline encoding of a bank
  step    msa_score_topk chained into msa_sparse_attend: one routed layer on its un-pooled bank
  layers  LayerStack.step: several routed layers on their pooled banks

Sizes follow the package's own configurations (documents of 512 tokens in chunks of 64, 32 query and 8 KV heads of 128
dimensions, banks of 32 thousand to 50 million tokens, 4 to 32 selected documents) and the ranges around them.
"""
import math

import torch

import paper_2603_23516_amd as msa
from paper_2603_23516_amd.layers import LayerStack

DEV = "cuda"


# ---- cases --------------------------------------------------------------------------------------------------
def _score(name, **kw):
    c = dict(op="score", B=1, M=1, N=2048, G=512, P=64, Hq=32, Hkv=8, d=128, k=16, sim="cos", scope="group", pool=False)
    c.update(kw)
    return dict(name=name, **c)


def _attend(name, **kw):
    c = dict(op="attend", B=1, M=1, N=2048, G=512, P=64, Hq=32, Hkv=8, d=128, k=16, Lloc=2048, scope="group",
             pool=False, ragged=False, base=1e6)
    c.update(kw)
    return dict(name=name, **c)


def listed():
    return [
        # one query token against a small bank: the shortest call chain, launches and latency
        dict(name="step_tiny_32k", op="step", B=1, M=1, N=64, G=512, P=64, Hq=8, Hkv=2, d=64, k=4, Lloc=256,
             scope="group", base=1e4),
        # single-stream decoding over one million tokens
        _score("score_decode_1m", B=1, N=2048, k=16),
        # a GPU's share of a 100M-token memory, eight streams decoding: the longest index
        _score("score_decode_50m", B=8, N=97656, k=32),
        # concurrent decoding with the head mean over every head (Eq. 2 as printed), one selection for all heads
        _score("score_batch_all_heads_4m", B=24, N=8192, k=16, scope="all"),
        # a question of 150 tokens routed as printed (max over its tokens, mean over all heads) against the 50M share
        _score("score_question_50m", M=150, N=97656, k=32, scope="all", pool=True),
        # a long prompt, every token with a selection of its own, against 16M tokens
        _score("score_prefill_16m", M=2048, N=32768, k=8),
        # forty streams decoding over a bank of documents of different lengths
        _attend("attend_decode_batch_ragged", B=40, N=8192, k=16, Lloc=1800, ragged=True),
        # eight streams, the large selection of the 50M share
        _attend("attend_decode_k32", B=8, N=8192, k=32, Lloc=2048),
        # a prompt of 512 tokens, every token attends its own documents and the prompt before it
        _attend("attend_prefill_tokens", M=512, N=4096, k=8, Lloc=512),
        # a question of 1000 tokens that share one selection (one for all heads)
        _attend("attend_prefill_question", M=1000, N=2048, k=16, Lloc=1000, scope="all", pool=True),
        # the offline stage: routing index and pooled bank of two million tokens
        dict(name="encode_2m", op="encode", N=4096, G=512, P=64, Hq=32, Hkv=8, d=128, ragged=False, base=1e6),
        # four routed layers on their pooled banks, four million tokens each, eight streams decoding
        dict(name="layers_pooled_4m", op="layers", L=4, B=8, M=1, N=8192, G=512, P=64, Hq=32, Hkv=8, d=128, k=16,
             Lloc=1024, base=1e6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    Hq, Hkv, d = rng.choice([(32, 8, 128)] * 5 + [(8, 2, 64), (16, 8, 128), (32, 4, 128), (8, 8, 64)])
    G, P = rng.choice([(512, 64)] * 5 + [(256, 64), (512, 32), (128, 64), (1024, 64), (64, 64)])
    base = rng.choice([1e4, 1e6])
    scope = rng.choice(["group", "group", "all"])
    op = rng.choice(["score"] * 4 + ["attend"] * 4 + ["encode", "step", "layers"])
    shape = dict(G=G, P=P, Hq=Hq, Hkv=Hkv, d=d)
    if op == "score":
        many = rng.random() < 0.4
        B, M = (rng.randint(1, 3), _log_int(rng, 2, 2048)) if many else (_log_int(rng, 1, 64), 1)
        return dict(op=op, B=B, M=M, N=_log_int(rng, 64, 97656 if G * Hkv >= 4096 else 20000), k=rng.randint(4, 32),
                    sim=rng.choice(["cos"] * 5 + ["dot"]), scope=scope, pool=many and rng.random() < 0.5, **shape)
    if op == "attend":
        many = rng.random() < 0.4
        B, M = (rng.randint(1, 2), _log_int(rng, 2, 1024)) if many else (_log_int(rng, 1, 64), 1)
        return dict(op=op, B=B, M=M, N=_log_int(rng, 64, 8192), k=rng.randint(4, 32),
                    Lloc=M if many else _log_int(rng, 1, 4096), scope=scope, pool=many and rng.random() < 0.5,
                    ragged=rng.random() < 0.3, base=base, **shape)
    if op == "encode":
        return dict(op=op, N=_log_int(rng, 64, 4096), ragged=rng.random() < 0.3, base=base, **shape)
    if op == "step":
        return dict(op=op, B=_log_int(rng, 1, 8), M=1, N=_log_int(rng, 64, 2048), k=rng.randint(4, 16),
                    Lloc=_log_int(rng, 16, 2048), scope=scope, base=base, **shape)
    return dict(op=op, L=rng.randint(2, 4), B=_log_int(rng, 1, 16), M=1, N=_log_int(rng, 256, 4096), G=512, P=64,
                Hq=Hq, Hkv=Hkv, d=d, k=rng.randint(4, 32), Lloc=_log_int(rng, 16, 2048), base=base)


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed()) * 0.9
    while True:
        c = _draw_once(rng)
        bank = c["N"] * c["G"] * c["Hkv"] * c["d"] * 4 if c["op"] != "score" else 0
        if _cost(c) <= most and bank <= 18e9 and c.get("k", 1) <= c["N"] // 2:
            return c


# ---- inputs -------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _normal(gen, shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _config(c, **kw):
    f = dict(sim=msa.MSA_SIM_DOT if c.get("sim") == "dot" else msa.MSA_SIM_COS,
             select_scope=msa.MSA_SCOPE_ALL if c.get("scope") == "all" else msa.MSA_SCOPE_GROUP,
             token_pool=int(bool(c.get("pool"))))
    f.update(kw)
    return msa.MsaConfig(c["N"], c["G"], c["P"], c["Hq"], c["Hkv"], c["d"], c.get("base", 1e6), **f)


def _queries(c, seed):
    """Query tokens of B sequences; the tokens of a sequence have its topic in common."""
    gen = _gen(seed, 1)
    topic = _normal(gen, (c["B"], 1, c["Hq"], c["d"]))
    q = _normal(gen, (c["B"], c["M"], c["Hq"], c["d"]))
    return (q.float() + 0.5 * topic.float()).to(torch.bfloat16), topic[:, 0].float()


def _index(c, seed, topic):
    """Plain routing keys bf16 [Hkv][N*C][d]: chunk means of normal keys; some documents carry a sequence's topic."""
    gen = _gen(seed, 2)
    N, C, Hkv, d, k = c["N"], c["G"] // c["P"], c["Hkv"], c["d"], c["k"]
    keys = torch.empty((Hkv, N, C, d), dtype=torch.bfloat16, device=DEV)
    for g in range(Hkv):
        keys[g] = _normal(gen, (N, C, d)) * (c["P"] ** -0.5)
    u = topic.reshape(c["B"], Hkv, c["Hq"] // Hkv, d).sum(2)
    u = u / u.norm(dim=-1, keepdim=True) * math.sqrt(d)
    per_seq = min(2 * k, N // (2 * c["B"]))
    if per_seq > 0:
        docs = torch.randperm(N, generator=gen, device=DEV)[:c["B"] * per_seq]
        ch = torch.randint(0, C, (docs.numel(),), generator=gen, device=DEV)
        a = torch.rand((docs.numel(),), generator=gen, device=DEV) * 0.12 + 0.03
        add = (u.repeat_interleave(per_seq, 0) * a[:, None, None]).transpose(0, 1)     # [Hkv][docs][d]
        keys[:, docs, ch] = (keys[:, docs, ch].float() + add).to(torch.bfloat16)
    return keys.reshape(Hkv, N * C, d)


def _tiled(keys):
    """(KR, inv_norm) in the documented layout: tiles of 16 keys, [Hkv][tiles][d/8][16][8], zero past the last key."""
    Hkv, n, d = keys.shape
    tiles = (n + 15) // 16
    KR = torch.zeros((Hkv, tiles, d // 8, 16, 8), dtype=torch.bfloat16, device=DEV)
    inv = torch.zeros((Hkv, tiles * 16), dtype=torch.float32, device=DEV)
    for g in range(Hkv):
        full = torch.zeros((tiles * 16, d), dtype=torch.bfloat16, device=DEV)
        full[:n] = keys[g]
        KR[g] = full.reshape(tiles, 16, d // 8, 8).transpose(1, 2)
        inv[g, :n] = 1.0 / keys[g].float().norm(dim=-1).clamp_min(1e-12)
    return KR, inv


def _selection(c, seed):
    """Selected documents int32 [B][M'][S][k]: half of a token's documents are among those of its sequence's topic
    (4 k documents), half are its own; no document twice."""
    gen = _gen(seed, 3)
    B, M, N, k = c["B"], 1 if c.get("pool") else c["M"], c["N"], c["k"]
    S = 1 if c.get("scope") == "all" else c["Hkv"]
    n_pool, n_hot = min(4 * k, N // 2), k // 2
    out = torch.empty((B, M, S, k), dtype=torch.int32, device=DEV)
    for b in range(B):
        for s in range(S):
            topic = torch.randperm(N, generator=gen, device=DEV)[:n_pool]
            hot = topic[torch.rand((M, n_pool), generator=gen, device=DEV).topk(n_hot, dim=1).indices]
            own = torch.rand((M, N), generator=gen, device=DEV)
            own[:, topic] = -1.0
            own = own.topk(k - n_hot, dim=1).indices
            mix = torch.cat([hot, own], dim=1)
            order = torch.rand((M, k), generator=gen, device=DEV).argsort(dim=1)
            out[b, :, s] = mix.gather(1, order).to(torch.int32)
    return out


def _lens(c, seed):
    if not c.get("ragged"):
        return None
    return torch.randint(c["G"] // 8, c["G"] + 1, (c["N"],), generator=_gen(seed, 4), device=DEV, dtype=torch.int32)


def _bank(c, seed, salt):
    gen = _gen(seed, salt)
    out = torch.empty((c["N"], c["Hkv"], c["G"], c["d"]), dtype=torch.bfloat16, device=DEV)
    step = max(1, (1 << 28) // (c["Hkv"] * c["G"] * c["d"]))
    for i in range(0, c["N"], step):
        out[i:i + step].normal_(generator=gen)
    return out


def _local(c, seed, salt=5):
    gen = _gen(seed, salt)
    shape = (c["B"], c["Hkv"], c["Lloc"], c["d"])
    return _normal(gen, shape), _normal(gen, shape)


def _positions(c, pos0):
    if c["M"] == 1:
        pos = torch.full((c["B"], 1), pos0 + c["Lloc"] - 1, dtype=torch.int32, device=DEV)
    else:   # the local context is the prompt itself: token m sees tokens 0 .. m
        pos = (pos0 + torch.arange(c["M"], dtype=torch.int32, device=DEV)).repeat(c["B"], 1)
    return pos.contiguous()


def _score_buffers(c, cfg):
    S = 1 if c.get("scope") == "all" else c["Hkv"]
    shape = (c["B"], 1 if c.get("pool") else c["M"], S, c["k"])
    return dict(idx=torch.empty(shape, dtype=torch.int32, device=DEV),
                val=torch.empty(shape, dtype=torch.float32, device=DEV),
                ws_s=torch.empty(msa.score_topk_workspace_bytes(cfg, c["B"], c["M"], c["k"]), dtype=torch.uint8,
                                 device=DEV))


def _attend_buffers(c, cfg, q):
    return dict(out=torch.empty_like(q),
                lse=torch.empty((c["B"], c["M"], c["Hq"]), dtype=torch.float32, device=DEV),
                ws_a=torch.empty(msa.sparse_attend_workspace_bytes(cfg, c["B"], c["M"], c["k"], c["Lloc"]),
                                 dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    c = case
    op = c["op"]
    s = dict(case=c, op=op)
    if op == "score":
        cfg = _config(c)
        q, topic = _queries(c, seed)
        KR, inv = _tiled(_index(c, seed, topic))
        s.update(cfg=cfg, q=q, KR=KR, inv=inv if c["sim"] == "cos" else None, **_score_buffers(c, cfg))
    elif op == "attend":
        cfg = _config(c, doc_lens=_lens(c, seed))
        q, _ = _queries(c, seed)
        Kl, Vl = _local(c, seed)
        s.update(cfg=cfg, q=q, K=_bank(c, seed, 6), V=_bank(c, seed, 7), idx=_selection(c, seed), Kl=Kl, Vl=Vl,
                 pos0=c["G"], pos=_positions(c, c["G"]), **_attend_buffers(c, cfg, q))
    elif op == "encode":
        cfg = _config(c, doc_lens=_lens(c, seed))
        C = c["G"] // c["P"]
        KR, inv = msa.alloc_routing_index(cfg, DEV)
        pooled = torch.empty((2, c["N"], c["Hkv"], C, c["d"]), dtype=torch.bfloat16, device=DEV)
        lens = torch.empty(c["N"], dtype=torch.int32, device=DEV) if c["ragged"] else None
        s.update(cfg=cfg, K=_bank(c, seed, 6), V=_bank(c, seed, 7), KR=KR, inv=inv, Kbar=pooled[0], Vbar=pooled[1],
                 pooled_lens=lens)
    elif op == "step":
        cfg = _config(c)
        q, _ = _queries(c, seed)
        K = _bank(c, seed, 6)
        KR, inv = msa.msa_build_routing_keys(cfg, K)
        Kl, Vl = _local(c, seed)
        s.update(cfg=cfg, q=q, K=K, V=_bank(c, seed, 7), KR=KR, inv=inv, Kl=Kl, Vl=Vl, pos0=c["G"],
                 pos=_positions(c, c["G"]), **_score_buffers(c, cfg), **_attend_buffers(c, cfg, q))
    else:
        cfg = _config(c)
        stack = LayerStack(cfg, c["L"], c["B"], c["M"], c["k"], c["Lloc"])
        s.update(stack=stack, pos0=c["k"], pos=_positions(c, c["k"]), q=[], Kl=[], Vl=[], out=[], lse=[])
        for l in range(c["L"]):
            stack.set_layer_keys(l, _bank(c, seed, 100 + 10 * l))
            stack.set_layer_values(l, _bank(c, seed, 101 + 10 * l))
            q, _ = _queries(c, seed + 7919 * (l + 1))
            Kl, Vl = _local(c, seed, 102 + 10 * l)
            s["q"].append(q)
            s["Kl"].append(Kl)
            s["Vl"].append(Vl)
            s["out"].append(torch.empty_like(q))
            s["lse"].append(torch.empty((c["B"], c["M"], c["Hq"]), dtype=torch.float32, device=DEV))
    return s


# ---- one pass -----------------------------------------------------------------------------------------------
def run(s):
    op = s["op"]
    if op in ("score", "step"):
        idx, val = msa.msa_score_topk(s["cfg"], s["q"], s["KR"], s["inv"], s["case"]["k"], s["idx"], s["val"], s["ws_s"])
        if op == "score":
            return dict(idx=idx, score=val)
    if op in ("attend", "step"):
        out, lse = msa.msa_sparse_attend(s["cfg"], s["q"], s["K"], s["V"], s["idx"], s["Kl"], s["Vl"], s["pos0"], s["pos"],
                                         s["out"], s["lse"], s["ws_a"])
        return dict(out=out, lse=lse) if op == "attend" else dict(idx=idx, score=val, out=out, lse=lse)
    if op == "encode":
        KR, inv = msa.msa_build_routing_keys(s["cfg"], s["K"], KR=s["KR"], inv_norm=s["inv"])
        pooled = msa.msa_pool_kv(s["cfg"], s["K"], s["V"], Kbar=s["Kbar"], Vbar=s["Vbar"], pooled_lens=s["pooled_lens"])
        return dict(KR=KR, inv_norm=inv, Kbar=pooled[0], Vbar=pooled[1])
    stack = s["stack"]
    stack.step(s["q"], s["Kl"], s["Vl"], s["pos0"], s["pos"], s["out"], s["lse"])
    return dict(idx=list(stack.idx), out=list(s["out"]), lse=list(s["lse"]))


# ---- what a pass cannot do without --------------------------------------------------------------------------
def _score_work(c):
    NC, BM = c["N"] * (c["G"] // c["P"]), c["B"] * c["M"]
    per_key = c["d"] * 2 + (0 if c.get("sim") == "dot" else 4)
    sel = c["B"] * (1 if c.get("pool") else c["M"]) * (1 if c.get("scope") == "all" else c["Hkv"]) * c["k"]
    # the head mean folds the heads of a group into one query per group
    return c["Hkv"] * NC * per_key + BM * c["Hq"] * c["d"] * 2 + sel * 8, 2.0 * BM * c["Hkv"] * NC * c["d"]


def _attend_work(c, rows_per_doc=None):
    """Every selected (document, KV head) once: half of the selections of a sequence fall on its 4 k topic documents."""
    G = rows_per_doc or c["G"]
    rows = G * (0.5625 if c.get("ragged") else 1.0)
    M = 1 if c.get("pool") else c["M"]
    hot, own = c["k"] // 2, c["k"] - c["k"] // 2
    n_pool = min(4 * c["k"], c["N"] // 2)
    rest = max(1, c["N"] - n_pool)
    uniq = n_pool * (1 - (1 - hot / n_pool) ** M) + rest * (1 - (1 - own / rest) ** M) if M > 1 else c["k"]
    docs = min(uniq * c["B"], c["N"])
    local = c["B"] * c["Lloc"]
    bytes_ = (docs * rows + local) * c["Hkv"] * c["d"] * 4 + 4.0 * c["B"] * c["M"] * c["Hq"] * (c["d"] + 1)
    seen = c["k"] * rows + (c["Lloc"] if c["M"] == 1 else c["Lloc"] / 2)
    return bytes_, 4.0 * c["B"] * c["M"] * c["Hq"] * seen * c["d"]


def work(case):
    c = case
    if c["op"] == "score":
        b, f = _score_work(c)
    elif c["op"] == "attend":
        b, f = _attend_work(c)
    elif c["op"] == "encode":
        rows = c["N"] * c["G"] * (0.5625 if c["ragged"] else 1.0)
        chunks = c["N"] * (c["G"] // c["P"])
        b, f = c["Hkv"] * (rows * c["d"] * 4 + chunks * (c["d"] * 6 + 4)), rows * c["Hkv"] * c["d"] * 6.0
    elif c["op"] == "step":
        (b, f), (b2, f2) = _score_work(c), _attend_work(c)
        b, f = b + b2, f + f2
    else:
        (b, f), (b2, f2) = _score_work(c), _attend_work(c, c["G"] // c["P"])
        b, f = c["L"] * (b + b2), c["L"] * (f + f2)
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    op = case["op"]
    if op == "score":     # fp32 scores of bf16 keys; neighbours closer than a rounding may change places
        return {"rel": 1e-5, "max": 4e-4, "differ": 5e-3}
    if op == "encode":    # bf16 means of fp32 sums: a sum next to a rounding boundary moves by one bf16 step
        return {"rel": 2e-3, "max": 2e-2}
    return {"rel": 8e-3, "max": 0.1, "differ": 1e-2}


# ---- the same in 64 bits, in plain torch --------------------------------------------------------------------
def _exact_score(c, q, keys):
    """keys bf16 [Hkv][N*C][d] -> (idx, score)."""
    B, M, Hq, d = q.shape
    Hkv, N, C, k = c["Hkv"], c["N"], c["G"] // c["P"], c["k"]
    r = Hq // Hkv
    x = q.double().reshape(B * M, Hkv, r, d)
    if c.get("sim") != "dot":
        x = x / x.norm(dim=-1, keepdim=True).clamp_min(1e-12)
    x = x.mean(2)
    every = c.get("scope") == "all"
    S = 1 if every else Hkv
    docs = torch.empty((B, 1 if c.get("pool") else M, S, N), dtype=torch.float64, device=DEV)
    step = max(16, (1 << 27) // (B * M * C) // 16 * 16)
    for n0 in range(0, N, step):
        n1 = min(N, n0 + step)
        acc = None
        for g in range(Hkv):
            kg = keys[g, n0 * C:n1 * C].double()
            sc = x[:, g] @ kg.t()
            if c.get("sim") != "dot":
                sc /= kg.norm(dim=-1).clamp_min(1e-12)
            if every:
                acc = sc if acc is None else acc.add_(sc)
                if g < Hkv - 1:
                    continue
                sc = acc / Hkv
            sc = sc.reshape(B, M, n1 - n0, C).amax(-1)
            docs[:, :, 0 if every else g, n0:n1] = sc.amax(1, keepdim=True) if c.get("pool") else sc
    val, idx = docs.topk(k, dim=-1)
    return idx.to(torch.int32), val


def _rope(x, pos, base):
    d = x.shape[-1]
    theta = base ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=DEV) / d)
    ang = pos.double()[..., None] * theta
    co, si = ang.cos(), ang.sin()
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * co - b * si, b * co + a * si], dim=-1)


def _exact_attend(c, q, K, V, idx, Kl, Vl, pos0, pos, base, lens=None, rotated=False):
    B, M, Hq, d = q.shape
    N, Hkv, G, _ = K.shape
    r, k = Hq // Hkv, idx.shape[-1]
    out = torch.empty((B, M, Hq, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((B, M, Hq), dtype=torch.float64, device=DEV)
    rows = torch.arange(G, device=DEV)
    lpos = pos0 + torch.arange(Kl.shape[2], device=DEV)
    shared = idx.shape[1] == 1
    step = M if shared else max(1, (1 << 26) // (k * G * d))
    for b in range(B):
        for g in range(Hkv):
            kl, vl = _rope(Kl[b, g].double(), lpos, base), Vl[b, g].double()
            for m0 in range(0, M, step):
                m1 = min(M, m0 + step)
                qt = _rope(q[b, m0:m1, g * r:(g + 1) * r].double(), pos[b, m0:m1, None].expand(m1 - m0, r), base)
                ids = idx[b, (slice(0, 1) if shared else slice(m0, m1)), 0 if idx.shape[2] == 1 else g].long()
                kk, vv = K[ids, g].double(), V[ids, g].double()                  # [T'][k][G][d]
                if not rotated:
                    kk = _rope(kk, rows, base)
                T = ids.shape[0]
                z = torch.matmul(qt.reshape(T, -1, d), kk.reshape(T, k * G, d).transpose(1, 2).contiguous())
                if lens is not None:
                    live = (rows < lens[ids].long()[..., None]).reshape(T, 1, k * G)
                    z = z.masked_fill(~live, -math.inf)
                zl = torch.matmul(qt, kl.t().contiguous())                         # [T][r][Lloc]
                zl = zl.masked_fill((lpos > pos[b, m0:m1, None])[:, None], -math.inf)
                z = torch.cat([z.reshape(m1 - m0, r, k * G), zl], dim=-1) / math.sqrt(d)
                ls = z.logsumexp(-1)
                w = (z - ls[..., None]).exp()
                o = torch.matmul(w[..., :k * G].reshape(T, -1, k * G), vv.reshape(T, k * G, d)).reshape(m1 - m0, r, d)
                out[b, m0:m1, g * r:(g + 1) * r] = o + torch.matmul(w[..., k * G:], vl)
                lse[b, m0:m1, g * r:(g + 1) * r] = ls
    return out, lse


def _exact_pool(c, X, lens=None, rotate=False):
    """Chunk means [N][Hkv][C][d] and the number of rows of every chunk [N][C]."""
    N, Hkv, G, d = X.shape
    P, C = c["P"], G // c["P"]
    out = torch.empty((N, Hkv, C, d), dtype=torch.float64, device=DEV)
    rows = torch.arange(G, device=DEV)
    have = torch.full((N, C), P, device=DEV)
    if lens is not None:
        have = (lens.long()[:, None] - torch.arange(C, device=DEV) * P).clamp(0, P)
    step = max(1, (1 << 26) // (Hkv * G * d))
    for i in range(0, N, step):
        x = X[i:i + step].double()
        if rotate:
            x = _rope(x, rows, c["base"])
        if lens is not None:
            x = x * (rows < lens[i:i + step].long()[:, None])[:, None, :, None]
        out[i:i + step] = x.reshape(-1, Hkv, C, P, d).sum(3) / have[i:i + step].clamp_min(1)[:, None, :, None]
    return out, have


def _exact_index(c, K, lens=None):
    """Plain routing keys in 64 bits [Hkv][N*C][d]; a chunk that a document does not have repeats its first."""
    mean, have = _exact_pool(c, K, lens)
    mean = torch.where((have > 0)[:, None, :, None], mean, mean[:, :, :1])
    return mean.transpose(0, 1).reshape(c["Hkv"], -1, c["d"])


def exact(case, seed):
    c, op = case, case["op"]
    if op == "score":
        q, topic = _queries(c, seed)
        idx, val = _exact_score(c, q, _index(c, seed, topic))
        return dict(idx=idx, score=val)
    if op == "encode":
        K, lens = _bank(c, seed, 6), _lens(c, seed)
        keys = _exact_index(c, K, lens)
        n, d = keys.shape[1], c["d"]
        tiles = (n + 15) // 16
        full = torch.zeros((c["Hkv"], tiles * 16, d), dtype=torch.float64, device=DEV)
        full[:, :n] = keys
        inv = torch.zeros((c["Hkv"], tiles * 16), dtype=torch.float64, device=DEV)
        inv[:, :n] = 1.0 / keys.to(torch.bfloat16).double().norm(dim=-1).clamp_min(1e-12)
        Kbar = _exact_pool(c, K, lens, rotate=True)[0]
        del K
        Vbar = _exact_pool(c, _bank(c, seed, 7), lens)[0]
        return dict(KR=full.reshape(c["Hkv"], tiles, 16, d // 8, 8).transpose(2, 3).contiguous(), inv_norm=inv,
                    Kbar=Kbar, Vbar=Vbar)
    if op == "attend":
        if c["B"] * c["M"] * c["k"] * c["G"] * c["Hkv"] > 1 << 26 and not c["pool"]:
            return None
        q, _ = _queries(c, seed)
        Kl, Vl = _local(c, seed)
        out, lse = _exact_attend(c, q, _bank(c, seed, 6), _bank(c, seed, 7), _selection(c, seed), Kl, Vl, c["G"],
                                 _positions(c, c["G"]), c["base"], _lens(c, seed))
        return dict(out=out, lse=lse)
    if op == "step":
        q, _ = _queries(c, seed)
        K = _bank(c, seed, 6)
        idx, val = _exact_score(c, q, _exact_index(c, K).to(torch.bfloat16))
        Kl, Vl = _local(c, seed)
        out, lse = _exact_attend(c, q, K, _bank(c, seed, 7), idx, Kl, Vl, c["G"], _positions(c, c["G"]), c["base"])
        return dict(idx=idx, score=val, out=out, lse=lse)
    res = dict(idx=[], out=[], lse=[])
    for l in range(c["L"]):
        q, _ = _queries(c, seed + 7919 * (l + 1))
        K = _bank(c, seed, 100 + 10 * l)
        idx, _ = _exact_score(c, q, _exact_index(c, K).to(torch.bfloat16))
        Kbar = _exact_pool(c, K, rotate=True)[0].to(torch.bfloat16)
        del K
        Vbar = _exact_pool(c, _bank(c, seed, 101 + 10 * l))[0].to(torch.bfloat16)
        Kl, Vl = _local(c, seed, 102 + 10 * l)
        out, lse = _exact_attend(c, q, Kbar, Vbar, idx, Kl, Vl, c["k"], _positions(c, c["k"]), c["base"], rotated=True)
        res["idx"].append(idx)
        res["out"].append(out)
        res["lse"].append(lse)
    return res
