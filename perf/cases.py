"""The calls whose speed matters: MALA training steps, prefills and decode steps through
the package's public functions, over the sizes that the workloads, tests and benchmark
of this repository use.

Inputs are the planted-needle inputs of the workloads (Q_i = noise + beta K_{r(i)},
optionally a local key, needles shared by blocks of rows and an attention sink), drawn
on the GPU.  tau = 1 is the method's canonical tolerance, on which a part of the tiles
is skipped on language-model-like inputs; tau <= 1e-3 keeps nearly every tile.
"""
import math

import torch

import paper_2609_32712_amd as mala

_TILE = 32        # decision tiles are 32 x 32 (decode: 1 x 32 per query head)
_LOG = math.log


# ------------------------------------------------------------------ the cases
def listed():
    train = dict(kind="train", stats=False, bf16_out=False, local=0.0, block=1, sink=0.0)
    lm = dict(beta=2.0, local=2.0, block=32, sink=1.5, tau=1.0)
    return [
        # one head over 1024 tokens: the smallest workload, in the form of the README's
        # example (statistics on, as the functions default to); launches and latency
        dict(train, name="train_1k_d64", B=1, Hq=1, Hkv=1, N=1024, D=64, beta=2.0, tau=1e-3,
             stats=True),
        # a small ragged batch (a fine-tuning micro-batch), bf16 outputs and gradients
        dict(train, name="train_700_gqa_bf16", B=2, Hq=4, Hkv=2, N=700, D=128, beta=2.5,
             local=2.0, tau=1e-3, bf16_out=True),
        # language-model-like inputs at the canonical tolerance: 4096-token sequences, and
        # one 8192-token sequence of a tensor-parallel rank
        dict(train, name="train_lm_4k_batch8", B=8, Hq=8, Hkv=2, N=4096, D=128, **lm),
        # multi-head attention over 8192 tokens
        dict(train, name="train_mha16_8k", B=1, Hq=16, Hkv=16, N=8192, D=128, beta=2.0,
             local=1.0, tau=1e-4),
        # long-context training: GQA over 32768 tokens, heads of every sharpness (beta < 0:
        # each head draws its own from [0.5, 3])
        dict(train, name="train_gqa32x8_32k", B=1, Hq=32, Hkv=8, N=32768, D=128, beta=-1.0,
             tau=1e-4),
        # one tensor-parallel rank's share of a 131072-token step
        dict(train, name="train_gqa8x2_128k", B=1, Hq=8, Hkv=2, N=131072, D=128, beta=2.0,
             tau=1e-4),
        # a packed training batch of sequences of very different lengths
        dict(kind="varlen", name="train_packed_32k", Hq=8, Hkv=2, D=128, stats=False,
             lens="16384,8192,4096,1500,1024,1000,500,68,4", **lm),
        # serving: a prompt of 2000 tokens, all heads of one layer, bf16 output
        dict(kind="prefill", name="prefill_2000", B=1, Hq=32, Hkv=8, Nq=2000, Nk=2000, D=128,
             beta=2.0, local=2.0, block=1, sink=1.5, tau=1e-3),
        # serving: the next 512 tokens of a chunked prefill against 16384 cached keys, one
        # tensor-parallel rank's heads
        dict(kind="prefill", name="prefill_chunk512_16k", B=1, Hq=8, Hkv=2, Nq=512, Nk=16384,
             D=128, beta=2.0, local=2.0, block=1, sink=1.5, tau=1e-3),
        # decode of one sequence (interactive use): latency
        dict(kind="decode", name="decode_1x4k", B=1, Hq=32, Hkv=8, Nk=4096, D=128, beta=3.0,
             needles=4, tau=1e-4, splits=0, ragged=False, noalloc=False),
        # decode of a serving batch with caches of different lengths, no allocation
        dict(kind="decode", name="decode_16x8k_ragged", B=16, Hq=32, Hkv=8, Nk=8192, D=128,
             beta=3.0, needles=4, tau=1e-3, splits=16, ragged=True, noalloc=True),
        # decode over long caches: bandwidth
        dict(kind="decode", name="decode_16x128k", B=16, Hq=32, Hkv=8, Nk=131072, D=128,
             beta=3.0, needles=4, tau=1e-4, splits=16, ragged=False, noalloc=False),
    ]


def _logsize(rng, lo, hi):
    return int(round(math.exp(rng.uniform(_LOG(lo), _LOG(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "varlen", "prefill", "decode", "decode"])
    D = rng.choice([64, 128, 128])
    Hkv = rng.choice([1, 2, 4, 8])
    Hq = Hkv * rng.choice([1, 2, 4, 4, 8])
    tau = rng.choice([0.0, 1e-4, 1e-3, 1.0])
    shape = dict(beta=round(rng.uniform(1.0, 3.0), 2), local=rng.choice([0.0, 1.0, 2.0]),
                 block=rng.choice([1, 32]), sink=rng.choice([0.0, 1.5]))
    if kind == "train":
        N = _logsize(rng, 64, 16384)
        B = max(1, min(_logsize(rng, 1, 32), 32768 // N))
        return dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, N=N, D=D, tau=tau, stats=rng.random() < 0.25,
                    bf16_out=rng.random() < 0.4, **shape)
    if kind == "varlen":
        total, lens = _logsize(rng, 512, 24576), []
        while sum(lens) < total and len(lens) < 24:
            lens.append(_logsize(rng, 8, 8192))
        return dict(kind=kind, Hq=Hq, Hkv=Hkv, D=D, tau=tau, stats=False,
                    lens=",".join(map(str, lens)), **shape)
    if kind == "prefill":
        Nq = _logsize(rng, 16, 8192)
        Nk = Nq + rng.choice([0, 1]) * _logsize(rng, 64, 24576)
        return dict(kind=kind, B=rng.choice([1, 1, 2, 4]), Hq=Hq, Hkv=Hkv, Nq=Nq, Nk=Nk, D=D,
                    tau=tau, **shape)
    B, Nk = _logsize(rng, 1, 32), _logsize(rng, 128, 65536)
    return dict(kind="decode", B=B, Hq=Hq, Hkv=Hkv, Nk=Nk, D=D, tau=tau,
                beta=round(rng.uniform(2.0, 4.0), 2), needles=4, splits=rng.choice([0, 0, 4, 16]),
                ragged=rng.random() < 0.4, noalloc=False)


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _queries(case, g, k, Hq):
    """Planted-needle queries of rows off .. Nk - 1 of the keys k [H, Nk, D] (one batch
    element): row i mixes noise with a key at or before it, its predecessor and key 0."""
    Hkv, Nk, D = k.shape
    Nq = case.get("Nq", Nk)
    off = Nk - Nq
    kf = k.float().repeat_interleave(Hq // Hkv, 0)
    rows = torch.arange(off, Nk, device="cuda")
    u = torch.rand((Hq, Nq), generator=g, device="cuda")
    start = rows
    if case["block"] > 1:     # rows of a block share a needle that all of them see
        start = rows // case["block"] * case["block"]
        first = (start - off).clamp_(min=0)
        u = u.gather(1, first.expand(Hq, Nq))
    r = (u * (start + 1)).long().minimum(start)
    beta = torch.full((Hq, 1, 1), case["beta"], device="cuda")
    if case["beta"] < 0:
        beta = 0.5 + 2.5 * torch.rand((Hq, 1, 1), generator=g, device="cuda")
    q = _randn(g, Hq, Nq, D) + beta * kf.gather(1, r[..., None].expand(Hq, Nq, D))
    if case["local"]:
        q += case["local"] * torch.where(rows[:, None] > 0, kf[:, (rows - 1).clamp(min=0)], 0.0)
    if case["sink"]:
        q += case["sink"] * kf[:, :1]
    return q.bfloat16()


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _splits(case):
    return case["splits"] or mala.default_num_splits(case["B"], case["Hkv"], case["Nk"])


def prepare(case, seed):
    g = _gen(seed)
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    st = dict(case=case, scale=D ** -0.5, tau=case["tau"])
    if case["kind"] == "varlen":
        lens = _lens(case)
        total = sum(lens)
        k = _randn(g, Hkv, total, D).bfloat16()
        v = _randn(g, Hkv, total, D).bfloat16()
        do = _randn(g, Hq, total, D).bfloat16()
        q, p = torch.empty_like(do), 0
        for n in lens:
            q[:, p:p + n] = _queries(case, g, k[:, p:p + n], Hq)
            p += n
        cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32,
                          device="cuda")
        st.update(q=q, k=k, v=v, do=do, cu=cu, max_len=max(lens))
        return st
    B, Nk = case["B"], case.get("Nk", case.get("N"))
    k = _randn(g, B, Hkv, Nk, D).bfloat16()
    v = _randn(g, B, Hkv, Nk, D).bfloat16()
    st.update(k=k, v=v)
    if case["kind"] == "decode":
        lens = torch.full((B,), Nk, device="cuda", dtype=torch.int64)
        if case["ragged"]:
            lens = torch.randint(1, Nk + 1, (B,), generator=g, device="cuda")
            lens[0] = Nk
        u = torch.rand((B, Hq, case["needles"]), generator=g, device="cuda")
        pos = (u * lens[:, None, None]).long().minimum(lens[:, None, None] - 1)
        q = _randn(g, B, Hq, D)
        for b in range(B):
            for hk in range(Hkv):
                hs = slice(hk * (Hq // Hkv), (hk + 1) * (Hq // Hkv))
                q[b, hs] += case["beta"] * k[b, hk][pos[b, hs]].float().sum(1)
        S = _splits(case)
        st.update(q=q.bfloat16(), splits=S, lens=lens.int() if case["ragged"] else None,
                  o=torch.empty((B, Hq, D), device="cuda"), lse=torch.empty((B, Hq), device="cuda"))
        if not case["noalloc"]:
            st["workspace"] = torch.empty(mala.mala_decode_workspace_size(B, Hq, D, S),
                                          dtype=torch.uint8, device="cuda")
        return st
    st["q"] = torch.stack([_queries(case, g, k[b], Hq) for b in range(B)])
    if case["kind"] == "train":
        st["do"] = _randn(g, B, Hq, Nk, D).bfloat16()
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    case, scale, tau = st["case"], st["scale"], st["tau"]
    q, k, v = st["q"], st["k"], st["v"]
    if case["kind"] == "train":
        dt = torch.bfloat16 if case["bf16_out"] else torch.float32
        f = mala.fwd(q, k, v, scale, tau, stats=case["stats"], out_dtype=dt)
        b = mala.bwd(q, k, v, f["o"], f["lse"], st["do"], scale, tau, stats=case["stats"],
                     grad_dtype=dt)
        return dict(fwd=f, bwd=b)
    if case["kind"] == "varlen":
        f = mala.fwd_varlen(q, k, v, st["cu"], st["max_len"], scale, tau, stats=case["stats"])
        b = mala.bwd_varlen(q, k, v, st["cu"], st["max_len"], f["o"], f["lse"], st["do"], scale,
                            tau, stats=case["stats"])
        return dict(fwd=f, bwd=b)
    if case["kind"] == "prefill":
        return mala.fwd(q, k, v, scale, tau, stats=False, out_dtype=torch.bfloat16)
    # decode into buffers that a serving loop keeps
    if case["noalloc"]:
        mala.mala_decode_noalloc(q, k, v, st["o"], st["lse"], None, None, st["splits"], scale, tau,
                                 cache_lens=st["lens"])
    else:
        mala.mala_decode(q, k, v, st["o"], st["lse"], None, None, st["splits"], st["workspace"],
                         scale, tau, cache_lens=st["lens"])
    return dict(o=st["o"], lse=st["lse"])


# ------------------------------------------------------------------ work and tolerance
def _retained(case):
    """Shares of the legal tiles that the forward and the backward retain: about all of
    them below tau = 1; at tau = 1 on these inputs 25-50% and 8-15% (language-model-like),
    98% and 20-50% (needles alone)."""
    if case["tau"] < 0.1:
        return 1.0, 1.0
    return (0.4, 0.12) if case.get("block", 1) > 1 else (0.98, 0.3)


def work(case):
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    keep_f, keep_b = _retained(case)
    if case["kind"] == "decode":
        B, Nk = case["B"], case["Nk"]
        share = 0.5 + 0.5 / B if case["ragged"] else 1.0     # mean cache length over Nk
        kv = 2.0 * B * Hkv * Nk * D * share                  # one cache, bytes
        return dict(bytes=2 * kv + B * Hq * (D * 6.0 + 4), flops=4.0 * B * Hq * Nk * D * share)
    if case["kind"] == "varlen":
        seqs = [(n, n) for n in _lens(case)]
    elif case["kind"] == "prefill":
        seqs = [(case["Nq"], case["Nk"])] * case["B"]
    else:
        seqs = [(case["N"], case["N"])] * case["B"]
    pairs = sum(nq * (nk - nq) + nq * (nq + 1) / 2 for nq, nk in seqs) * Hq
    tq, tk = sum(s[0] for s in seqs), sum(s[1] for s in seqs)
    bf16 = case.get("bf16_out", case["kind"] == "prefill")
    e = 2 if bf16 else 4                                     # bytes of an output value
    q_in, kv_in, lse = 2.0 * Hq * tq * D, 4.0 * Hkv * tk * D, 4.0 * Hq * tq
    fwd_bytes = q_in + kv_in + e * Hq * tq * D + lse
    fwd_flops = pairs * 2 * D * (1 + keep_f)
    if case["kind"] == "prefill":
        return dict(bytes=fwd_bytes, flops=fwd_flops)
    # backward: Q, K, V, dO, O and LSE in; dQ, dK, dV out
    bwd_bytes = 2 * q_in + kv_in + e * Hq * tq * D + lse + e * Hq * tq * D + 2.0 * e * Hkv * tk * D
    return dict(bytes=fwd_bytes + bwd_bytes, flops=fwd_flops + pairs * 2 * D * (1 + 4 * keep_b))


def tolerance(case):
    """About four times the largest error against exact() that the listed and a few drawn
    cases show: decode 1.4e-6; 1.7e-3 where outputs are rounded to bf16; 3e-4 for fp32
    outputs (dQ and dK, whose operands enter the matrix cores as one or two bf16 terms)."""
    if case["kind"] == "decode":
        return dict(rel=6e-6)
    if case.get("bf16_out", case["kind"] == "prefill"):
        return dict(rel=7e-3, differ=0.01)
    return dict(rel=1.2e-3, differ=0.01)


# ------------------------------------------------------------------ 64-bit results
def _neg(x):
    return torch.full_like(x, -math.inf)


def _exact_fwd(q, k, v, scale, tau):
    """MALA forward of H heads (k, v one per query head): q [H, Nq, D], k, v [H, Nk, D] in
    float64.  Returns O, LSE, the retained tiles per row."""
    H, Nq, D = q.shape
    Nk = k.shape[1]
    off, T = Nk - Nq, -(-Nk // _TILE)
    nqt = -(-Nq // _TILE)
    rows = torch.arange(Nq, device=q.device)
    mt = q.new_full((H, nqt * _TILE, T), -math.inf)      # tile maxima and log-sum-exps of
    lt = q.new_full((H, nqt * _TILE, T), -math.inf)      # each row over each key tile
    chunk = max(_TILE, min(1024, (1 << 28) // (Nk * 8) // _TILE * _TILE))

    def scores(h, r0, r1):
        n = min(Nk, r1 + off)
        s = (q[h, r0:r1] @ k[h, :n].t()) * scale
        return s.masked_fill_(torch.arange(n, device=q.device) > (rows[r0:r1, None] + off), -math.inf)

    for h in range(H):
        for r0 in range(0, Nq, chunk):
            r1 = min(Nq, r0 + chunk)
            s = scores(h, r0, r1)
            t = -(-s.shape[1] // _TILE)
            s = torch.nn.functional.pad(s, (0, t * _TILE - s.shape[1]), value=-math.inf)
            s = s.view(r1 - r0, t, _TILE)
            mt[h, r0:r1, :t] = s.amax(2)
            lt[h, r0:r1, :t] = torch.logsumexp(s, 2)
    # the online test over each 32-row query tile's key tiles, from the last one down
    run = q.new_full((H, nqt * _TILE), -math.inf)        # log of the retained normalizer
    thr = torch.full((nqt * _TILE,), math.inf, device=q.device, dtype=q.dtype)
    thr[:Nq] = (_LOG(tau) if tau > 0 else -math.inf) - torch.log((rows + off + 1).to(q.dtype))
    keep = torch.zeros((H, nqt, T), dtype=torch.bool, device=q.device)
    for j in range(T - 1, -1, -1):
        m = mt[:, :, j]
        vote = (m > -math.inf) & ((run == -math.inf) | (m - run >= thr))
        kj = vote.view(H, nqt, _TILE).any(2)
        keep[:, :, j] = kj
        on = kj.repeat_interleave(_TILE, 1)
        run = torch.where(on, torch.logaddexp(run, lt[:, :, j]), run)
    lse = run[:, :Nq].contiguous()
    tiles = ((mt > -math.inf) & keep.repeat_interleave(_TILE, 1)).sum(2)[:, :Nq]
    del mt, lt
    o = torch.empty_like(q)
    for h in range(H):
        for r0 in range(0, Nq, chunk):
            r1 = min(Nq, r0 + chunk)
            s = scores(h, r0, r1)
            kc = keep[h, r0 // _TILE:-(-r1 // _TILE)].repeat_interleave(_TILE, 0)[:r1 - r0]
            on = kc.repeat_interleave(_TILE, 1)[:, :s.shape[1]]
            p = torch.exp(s - lse[h, r0:r1, None]).mul_(on)
            o[h, r0:r1] = p @ v[h, :s.shape[1]]
    return o, lse, tiles


def _exact_bwd(q, k, v, o, lse, do, scale, tau):
    """MALA backward of H heads (offline test against lse): dQ, dK, dV per query head."""
    H, Nq, D = q.shape
    Nk = k.shape[1]
    off = Nk - Nq
    rows = torch.arange(Nq, device=q.device)
    thr = (_LOG(tau) if tau > 0 else -math.inf) - torch.log((rows + off + 1).to(q.dtype))
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    dsum = (o * do).sum(2)
    chunk = max(_TILE, min(1024, (1 << 28) // (Nk * 8) // _TILE * _TILE))
    for h in range(H):
        for r0 in range(0, Nq, chunk):
            r1 = min(Nq, r0 + chunk)
            n, r = min(Nk, r1 + off), r1 - r0
            s = (q[h, r0:r1] @ k[h, :n].t()) * scale
            s.masked_fill_(torch.arange(n, device=q.device) > (rows[r0:r1, None] + off), -math.inf)
            s -= lse[h, r0:r1, None]
            hit = (s >= thr[r0:r1, None]) & (s > -math.inf)
            tr, tc = -(-r // _TILE), -(-n // _TILE)
            hit = torch.nn.functional.pad(hit, (0, tc * _TILE - n, 0, tr * _TILE - r))
            hit = hit.view(tr, _TILE, tc, _TILE).any(3).any(1)
            on = hit.repeat_interleave(_TILE, 0)[:r].repeat_interleave(_TILE, 1)[:, :n]
            p = torch.exp(s).mul_(on)
            dv[h, :n] += p.t() @ do[h, r0:r1]
            ds = (do[h, r0:r1] @ v[h, :n].t()).sub_(dsum[h, r0:r1, None]).mul_(p)
            dq[h, r0:r1] = (ds @ k[h, :n]) * scale
            dk[h, :n] += (ds.t() @ q[h, r0:r1]) * scale
    return dq, dk, dv


def _exact_seq(case, q, k, v, do, scale, tau):
    """One sequence: q, do [Hq, Nq, D], k, v [Hkv, Nk, D] in bf16."""
    Hq, Hkv, D = q.shape[0], k.shape[0], q.shape[2]
    grp = Hq // Hkv
    o, lse, dq = [], [], []
    dk = torch.zeros(k.shape, dtype=torch.float64, device=k.device)
    dv = torch.zeros_like(dk)
    per = max(1, (1 << 33) // (q.shape[1] * k.shape[1]))     # heads at once
    for h0 in range(0, Hq, per):
        hs = torch.arange(h0, min(Hq, h0 + per), device=k.device)
        qh, kh, vh = q[hs].double(), k[hs // grp].double(), v[hs // grp].double()
        oh, lh, _ = _exact_fwd(qh, kh, vh, scale, tau)
        o.append(oh)
        lse.append(lh)
        if do is not None:
            ob = oh.bfloat16().double() if case.get("bf16_out") else oh
            a, b, c = _exact_bwd(qh, kh, vh, ob, lh, do[hs].double(), scale, tau)
            dq.append(a)
            dk.index_add_(0, hs // grp, b)
            dv.index_add_(0, hs // grp, c)
    return torch.cat(o), torch.cat(lse), torch.cat(dq) if do is not None else None, dk, dv


def _exact_decode(case, st):
    B, Hq, Hkv, D, Nk = case["B"], case["Hq"], case["Hkv"], case["D"], case["Nk"]
    S, scale, tau, grp = st["splits"], st["scale"], st["tau"], Hq // Hkv
    o = torch.zeros((B, Hq, D), dtype=torch.float64, device="cuda")
    lse = torch.full((B, Hq), -math.inf, dtype=torch.float64, device="cuda")
    for b in range(B):
        n = int(st["lens"][b]) if st["lens"] is not None else Nk
        T = -(-n // _TILE)
        tps = -(-T // S)
        k, v = st["k"][b, :, :n].double(), st["v"][b, :, :n].double()
        s = torch.cat([st["q"][b, h * grp:(h + 1) * grp].double() @ k[h].t() for h in range(Hkv)])
        s = torch.nn.functional.pad(s * scale, (0, S * tps * _TILE - n), value=-math.inf)
        s = s.view(Hq, S, tps, _TILE)
        m, lt = s.amax(3), torch.logsumexp(s, 3)
        thr = (_LOG(tau) if tau > 0 else -math.inf) - _LOG(n)
        run = torch.full((Hq, S), -math.inf, dtype=torch.float64, device="cuda")
        keep = torch.zeros((Hq, S, tps), dtype=torch.bool, device="cuda")
        for t in range(tps - 1, -1, -1):
            kt = (m[:, :, t] > -math.inf) & ((run == -math.inf) | (m[:, :, t] - run >= thr))
            keep[:, :, t] = kt
            run = torch.where(kt, torch.logaddexp(run, lt[:, :, t]), run)
        lse[b] = torch.logsumexp(run, 1)
        p = torch.exp(s - lse[b][:, None, None, None]) * keep[..., None]
        p = p.view(Hq, -1)[:, :n]
        o[b] = torch.cat([p[h * grp:(h + 1) * grp] @ v[h] for h in range(Hkv)])
    return dict(o=o, lse=lse)


def exact(case, seed):
    st = prepare(case, seed)
    scale, tau = st["scale"], st["tau"]
    if case["kind"] == "decode":
        return _exact_decode(case, st)
    if work(case)["flops"] > 1e14:      # 131072 tokens: too long in 64 bits
        return None
    if case["kind"] == "varlen":
        out, p = [], 0
        for n in _lens(case):
            a = slice(p, p + n)
            out.append(_exact_seq(case, st["q"][:, a], st["k"][:, a], st["v"][:, a], st["do"][:, a],
                                  scale, tau))
            p += n
        o, lse, dq, dk, dv = (torch.cat(x, 1) for x in zip(*out))
    else:
        do = st.get("do")
        out = [_exact_seq(case, st["q"][b], st["k"][b], st["v"][b], None if do is None else do[b],
                          scale, tau) for b in range(case["B"])]
        o, lse = (torch.stack([x[i] for x in out]) for i in (0, 1))
        if case["kind"] == "prefill":
            return dict(o=o, lse=lse, row_tiles=None, counters=None)
        dq, dk, dv = (torch.stack([x[i] for x in out]) for i in (2, 3, 4))
    none = dict(row_tiles=None, counters=None)
    return dict(fwd=dict(o=o, lse=lse, **none), bwd=dict(dq=dq, dk=dk, dv=dv, **none))
