"""Performance cases: the calls a speculative-decoding engine makes into this
library, one layer at a time, through the public binding.

Each case names its operation (`op`) and sizes:
  verify   md_verify_attn: gamma + 1 query tokens over the whole KV cache, the
           call every decoding step makes once per layer;
  draft    md_draft_attn: the StreamingLLM-style draft over sinks + window;
  listed   md_draft_attn_indexed: the draft over a SnapKV selection;
  votes    md_snapkv_votes: the prompt-time scoring that the selection reads;
  collect  md_snapkv_select, then md_kv_gather of the selection into a draft
           cache of its own, once per prompt;
  step     one whole speculative step of a layer: per drafted token an append
           and a draft call, then append, verify, acceptance and commit.

Sizes are the repository's own workloads (Llama-3.1-8B and 70B head shapes)
plus the small and ragged calls around them.  Inputs are seeded N(0, 1); with
k_outlier four K channels are scaled by 8, as trained models' keys are, which
makes the softmax peaky.  Prompt votes are lognormal: a few keys hold most of
the mass.
"""
import math
import random

import numpy as np
import torch

import paper_2408_11049_amd as md

DEV = "cuda:0"
VOCAB = 128256
MAX_CACHE_ELEMS = 1 << 31      # K (or V) elements of a drawn case: the largest listed cache
MAX_VOTE_SCORES = 1 << 30      # scores of a drawn votes case: half the largest listed one
F32_SHARE = 4                  # fp32 matrix operations are slower: a quarter of these sizes


def _case(op, name, **kw):
    c = dict(op=op, name=name, B=1, Hq=32, Hkv=8, d=128, dtype="bf16", q_len=1, s_lo=4096,
             s_hi=4096, page=0, n_sink=0, window=0, budget=0, n_obs=32, gamma=0, k_outlier=False)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: a unit-test-sized fp32 model, bound by latency and the host path.
        _case("verify", "verify_tiny_f32", B=2, Hq=4, Hkv=1, d=64, dtype="f32", q_len=4, s_lo=256,
              s_hi=256),
        # One interactive user, a short chat context, paged serving cache.
        _case("verify", "verify_b1_4k", B=1, q_len=5, s_lo=4001, s_hi=4001, page=16),
        # A medium batch at 8k, contiguous cache.
        _case("verify", "verify_b32_8k", B=32, q_len=4, s_lo=8192, s_hi=8192),
        # A continuous-batching server: ragged lengths, paged, trained-model-like keys.
        _case("verify", "verify_b64_ragged", B=64, q_len=5, s_lo=16384, s_hi=32768, page=16,
              k_outlier=True),
        # Long documents on the 70B layer shape; the largest attention call.
        _case("verify", "verify_70b_b16_128k", B=16, Hq=64, q_len=5, s_lo=131072, s_hi=131072),
        # One drafted token, small streaming budget.
        _case("draft", "draft_b32_8k", B=32, q_len=1, s_lo=8192, s_hi=8192, n_sink=16, window=496),
        # gamma + 1 tokens over sinks + window of the long paged cache.
        _case("draft", "draft_b64_32k", B=64, q_len=5, s_lo=32768, s_hi=32768, page=16, n_sink=16,
              window=1008),
        # One drafted token over the SnapKV selection, read in place.
        _case("listed", "listed_b64_16k", B=64, q_len=1, s_lo=8192, s_hi=16384, page=16,
              budget=2049),
        # Prompt-time scoring of a full batch of long prompts (the 8B group: 128 rows a head).
        _case("votes", "votes_b64_32k", B=64, s_lo=32768, s_hi=32768, page=16),
        # The same for four ragged prompts on the 70B group (256 rows a head), contiguous.
        _case("votes", "votes_70b_b4", B=4, Hq=64, s_lo=5000, s_hi=12000),
        # Selection and collection of the draft cache for a batch of prompts.
        _case("collect", "collect_b32_32k", B=32, s_lo=24000, s_hi=32768, page=16, budget=2049),
        # A whole speculative step of a medium batch with listed drafts.
        _case("step", "step_b16_8k", B=16, q_len=5, gamma=4, s_lo=6000, s_hi=8000, page=16,
              budget=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the listed ranges: batches of 1 to 128, contexts of 256
    to 131072 tokens, both head dims and dtypes, groups of 1 to 8 query heads,
    contiguous and paged, uniform and ragged."""
    op = rng.choice(["verify", "verify", "draft", "listed", "votes", "collect", "step"])
    Hkv = rng.choice([1, 2, 4, 8, 8, 8])
    G = rng.choice([1, 2, 4, 4, 7, 8])
    d = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    page = rng.choice([0, 16, 16, 64])
    share = F32_SHARE if dtype == "f32" else 1
    while True:
        B = _log_int(rng, 1, 128)
        s_hi = _log_int(rng, 256, 131072)
        if op in ("votes", "collect", "step"):
            s_hi = min(s_hi, 32768)
        ok = B * s_hi * Hkv * d <= MAX_CACHE_ELEMS // share
        if op == "votes":
            ok = ok and B * s_hi * Hkv * G * 32 <= MAX_VOTE_SCORES // share
        if ok:
            break
    s_lo = s_hi if rng.random() < 0.4 else max(64, int(s_hi * rng.uniform(0.3, 1.0)))
    q_len = rng.randint(1, 8)
    n_sink, window = rng.choice([4, 16, 64]), _log_int(rng, 64, 2048)
    budget = _log_int(rng, 128, 2049)
    gamma = rng.randint(1, 5)
    if op == "step":
        q_len = gamma + 1
    if op == "listed":
        q_len = rng.choice([1, 1, q_len])
    c = _case(op, "", B=B, Hq=Hkv * G, Hkv=Hkv, d=d, dtype=dtype, q_len=q_len, s_lo=s_lo,
              s_hi=s_hi, page=page, n_sink=n_sink if op == "draft" else 0,
              window=window if op == "draft" else 0,
              budget=budget if op in ("listed", "collect", "step") else 0,
              gamma=gamma if op == "step" else 0, k_outlier=rng.random() < 0.3)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs --

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 128 + stream)
    return g


def _randn(shape, case, seed, stream):
    t = torch.empty(shape, dtype=_dtype(case), device=DEV)
    return t.normal_(generator=_gen(seed, stream))


def _lens(case):
    """Committed context lengths on the host (shape-defining: fixed per case, so
    that states of other seeds hold the same work)."""
    lo, hi, B = case["s_lo"], case["s_hi"], case["B"]
    n = np.random.default_rng([lo, hi, B]).integers(lo, hi + 1, size=B)
    if B:
        n[0] = hi
    return n.astype(np.int32)


def _cache(case, seed, cap, want_v=True):
    """K (and V) of `cap` tokens a sequence, contiguous or in pages of one pool
    placed in seeded random order, with the page table."""
    B, Hkv, d, ps = case["B"], case["Hkv"], case["d"], case["page"]
    pt = None
    if ps:
        n = -(-cap // ps)
        perm = torch.randperm(B * n, generator=_gen(seed, 4), device=DEV)
        pt = perm.to(torch.int32).reshape(B, n).contiguous()
        shape = (B * n, ps, Hkv, d)
    else:
        shape = (B, cap, Hkv, d)
    k = _randn(shape, case, seed, 1)
    if case["k_outlier"]:
        ch = np.random.default_rng(seed).permutation(d)[:4].tolist()
        k[..., ch] *= 8
    v = _randn(shape, case, seed, 2) if want_v else None
    return k, v, pt


def _lists(case, seed, lens):
    """Per (sequence, kv head) budget distinct ascending prompt positions: a
    seeded stand-in for a selection."""
    B, Hkv, n = case["B"], case["Hkv"], case["budget"]
    smax = int(lens.max())
    r = torch.rand((B, Hkv, smax), generator=_gen(seed, 5), device=DEV)
    dev_lens = torch.from_numpy(lens).to(DEV)
    r.masked_fill_(torch.arange(smax, device=DEV)[None, None] >= dev_lens[:, None, None], -1.0)
    k = min(n, smax)
    idx = r.topk(k, dim=2).indices.to(torch.int32)
    idx_len = torch.clamp(dev_lens, max=n).to(torch.int32)
    # short sequences: the entries past their length sort to the end and are not counted
    pad = torch.arange(k, device=DEV)[None, None] >= idx_len[:, None, None]
    idx = idx.masked_fill(pad, 2 ** 31 - 1).sort(dim=2).values
    if k < n:
        idx = torch.nn.functional.pad(idx, (0, n - k), value=-1)
    return idx.masked_fill(idx == 2 ** 31 - 1, -1).contiguous(), idx_len


def prepare(case, seed):
    op, B, L, Hq, Hkv, d = (case[x] for x in ("op", "B", "q_len", "Hq", "Hkv", "d"))
    lens = _lens(case)
    st = dict(case=case, lens_np=lens, lens=torch.from_numpy(lens.copy()).to(DEV), smax=int(lens.max()))
    if op in ("verify", "draft", "listed"):
        st["k"], st["v"], st["pt"] = _cache(case, seed, st["smax"])
        st["q"] = _randn((B, L, Hq, d), case, seed, 0)
        if op == "listed":
            st["idx"], st["idx_len"] = _lists(case, seed, np.maximum(lens - L, 1))
    elif op == "votes":
        st["k"], _, st["pt"] = _cache(case, seed, st["smax"], want_v=False)
        st["q"] = _randn((B, case["n_obs"], Hq, d), case, seed, 0)
    elif op == "collect":
        st["k"], st["v"], st["pt"] = _cache(case, seed, st["smax"])
        stride = max(1, st["smax"] - case["n_obs"])
        st["votes"] = torch.exp(2 * torch.randn((B, Hkv, stride), generator=_gen(seed, 6), device=DEV))
        rows = max(case["budget"], case["n_obs"]) + 8
        st["dk"] = torch.zeros((B, rows, Hkv, d), dtype=_dtype(case), device=DEV)
        st["dv"] = torch.zeros_like(st["dk"])
    else:
        g = case["gamma"]
        st["k"], st["v"], st["pt"] = _cache(case, seed, st["smax"] + L)
        st["idx"], st["idx_len"] = _lists(case, seed, lens)
        st["qd"] = [_randn((B, 1, Hq, d), case, seed, 20 + i) for i in range(g)]
        st["kd"] = [_randn((B, 1, Hkv, d), case, seed, 40 + i) for i in range(g)]
        st["vd"] = [_randn((B, 1, Hkv, d), case, seed, 60 + i) for i in range(g)]
        st["pos"] = [st["lens"] + i for i in range(g)]
        st["q"] = _randn((B, L, Hq, d), case, seed, 0)
        st["kn"] = _randn((B, L, Hkv, d), case, seed, 7)
        st["vn"] = _randn((B, L, Hkv, d), case, seed, 8)
        st["logits"] = _randn((B, L, VOCAB), case, seed, 9)
        # drafts that match the target for a seeded number of positions
        tgt = st["logits"].argmax(dim=2).to(torch.int32)[:, :g]
        keep = torch.randint(0, g + 1, (B, 1), generator=_gen(seed, 10), device=DEV)
        ok = torch.arange(g, device=DEV)[None] < keep
        st["draft"] = torch.where(ok, tgt, (tgt + 1) % VOCAB).to(torch.int32).contiguous()
    return st


# ---------------------------------------------------------------- one pass --

def run(st):
    c = st["case"]
    op = c["op"]
    kw = dict(max_kv_len=st["smax"], page_table=st.get("pt"))
    if op == "verify":
        return md.md_verify_attn(st["q"], st["k"], st["v"], st["lens"], **kw)
    if op == "draft":
        return md.md_draft_attn(st["q"], st["k"], st["v"], st["lens"], c["n_sink"], c["window"], **kw)
    if op == "listed":
        return md.md_draft_attn_indexed(st["q"], st["k"], st["v"], st["lens"], st["idx"],
                                        st["idx_len"], **kw)
    if op == "votes":
        return md.md_snapkv_votes(st["q"], st["k"], st["lens"], max_prompt_len=st["smax"],
                                  page_table=st["pt"])
    if op == "collect":
        idx, idx_len = md.md_snapkv_select(st["votes"], st["lens"], c["n_obs"],
                                           max(c["budget"], c["n_obs"]))
        dlen = md.md_kv_gather(st["dk"], st["dv"], st["k"], st["v"], idx, idx_len, st["lens"],
                               src_page_table=st["pt"])
        return idx, idx_len, dlen, st["dk"], st["dv"]
    # One speculative step; the committed lengths are a copy, so that every
    # pass speculates from the same context.
    L, cap = c["q_len"], st["smax"] + c["q_len"]
    k, v, pt = st["k"], st["v"], st["pt"]
    lens = st["lens"].clone()
    outs = []
    for i in range(c["gamma"]):
        kv_lens = md.md_kv_append(k, v, st["kd"][i], st["vd"][i], st["pos"][i], page_table=pt)
        outs.append(md.md_draft_attn_indexed(st["qd"][i], k, v, kv_lens, st["idx"], st["idx_len"],
                                             max_kv_len=cap, page_table=pt))
    kv_lens = md.md_kv_append(k, v, st["kn"], st["vn"], lens, page_table=pt)
    outs.append(md.md_verify_attn(st["q"], k, v, kv_lens, max_kv_len=cap, page_table=pt))
    accepted, tokens, target = md.md_greedy_accept(st["logits"], st["draft"])
    md.md_kv_commit(lens, accepted, L)
    return {"attn": outs, "accepted": accepted, "tokens": tokens, "target": target, "lens": lens,
            "k": k, "v": v}


# -------------------------------------------------------------------- work --

def _attn_work(case, lens, vis, L):
    """Bytes and operations of one attention call: vis[b] visible tokens."""
    es = 4 if case["dtype"] == "f32" else 2
    n = float(np.sum(vis))
    qo = 2 * case["B"] * L * case["Hq"] * case["d"] * es + 4 * case["B"] * L * case["Hq"]
    pages = 4 * n / case["page"] if case["page"] else 0
    return (2 * n * case["Hkv"] * case["d"] * es + qo + pages,
            4 * n * L * case["Hq"] * case["d"])


def work(case):
    op, B, L, Hq, Hkv, d = (case[x] for x in ("op", "B", "q_len", "Hq", "Hkv", "d"))
    es = 4 if case["dtype"] == "f32" else 2
    lens = _lens(case).astype(np.float64)
    row = Hkv * d * es  # one token's K (or V)
    if op == "verify":
        b, f = _attn_work(case, lens, lens, L)
    elif op == "draft":
        b, f = _attn_work(case, lens, np.minimum(lens, case["n_sink"] + case["window"] + L - 1), L)
    elif op == "listed":
        vis = np.minimum(np.maximum(lens - L, 1), case["budget"]) + L
        b, f = _attn_work(case, lens, vis, L)
        b += 4 * float(np.sum(vis)) * Hkv
    elif op == "votes":
        n, R = float(lens.sum()), case["n_obs"] * Hq
        b = n * row + R * B * d * es + 4 * Hkv * B * max(1, lens.max() - case["n_obs"])
        f = 2 * n * R * d
    elif op == "collect":
        n = float(np.sum(np.minimum(lens, max(case["budget"], case["n_obs"]))))
        b = 4 * Hkv * float(np.sum(lens - case["n_obs"])) + 4 * Hkv * n + 4 * n * row
        f = 6 * Hkv * float(lens.sum())
    else:
        b = f = 0.0
        for i in range(case["gamma"]):
            vis = np.minimum(lens, case["budget"]) + 1
            x, y = _attn_work(case, lens, vis, 1)
            b, f = b + x + 4 * float(np.sum(vis)) * Hkv + 4 * B * row, f + y
        x, y = _attn_work(case, lens, lens + L, L)
        b += x + 4 * B * L * row + B * L * VOCAB * es
        f += y + B * L * VOCAB
    return {"bytes": int(b), "flops": int(f)}


def tolerance(case):
    if case["op"] == "collect":
        return "exact"          # positions and copied rows
    if case["op"] == "votes":
        return {"rel": 1e-5}    # fp32 sums of fp32 softmax weights
    if case["dtype"] == "f32":
        return {"rel": 1e-5}    # fp32 throughout
    return {"rel": 1e-2}        # bf16 outputs, bf16 softmax weights


# ------------------------------------------------------------------- exact --

def _tokens(t, pt, b, n):
    """The first n tokens of sequence b, [Hkv, n, d] in float64."""
    if pt is None:
        x = t[b, :n]
    else:
        ps = t.shape[1]
        x = t[pt[b, : -(-n // ps)].long()].reshape(-1, t.shape[2], t.shape[3])[:n]
    return x.permute(1, 0, 2).to(torch.float64).contiguous()


def _exact_attn(case, q, k, v, pt, lens, mode, idx=None, idx_len=None):
    """softmax(q k^T / sqrt(d) + mask) v in float64, one sequence at a time."""
    B, L, Hq, d = q.shape
    Hkv = case["Hkv"]
    G = Hq // Hkv
    o = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.zeros(q.shape[:3], dtype=torch.float64, device=DEV)
    for b in range(B):
        S = int(lens[b])
        kb, vb = _tokens(k, pt, b, S), _tokens(v, pt, b, S)
        pos = torch.arange(S, device=DEV)[None].expand(Hkv, S)      # [Hkv, n]
        if mode == "listed":
            n = int(idx_len[b])
            spec = torch.arange(S - L, S, device=DEV)[None].expand(Hkv, L)
            pos = torch.cat([idx[b, :, :n].long(), spec], 1)
            kb = kb.gather(1, pos[..., None].expand(-1, -1, d))
            vb = vb.gather(1, pos[..., None].expand(-1, -1, d))
        qp = S - L + torch.arange(L, device=DEV)                     # query positions
        vis = pos[:, None] <= qp[None, :, None]                      # [Hkv, L, n]
        if mode == "draft":
            vis = vis & ((pos[:, None] < case["n_sink"]) |
                         (pos[:, None] >= qp[None, :, None] - case["window"] + 1))
        qb = q[b].reshape(L, Hkv, G, d).permute(1, 0, 2, 3).reshape(Hkv, L * G, d).to(torch.float64)
        s = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(d)
        s = s.masked_fill(~vis.repeat_interleave(G, dim=1), -math.inf)
        lb = torch.logsumexp(s, 2)
        ob = torch.matmul(torch.exp(s - lb[..., None]), vb)
        o[b] = ob.reshape(Hkv, L, G, d).permute(1, 0, 2, 3).reshape(L, Hq, d)
        lse[b] = lb.reshape(Hkv, L, G).permute(1, 0, 2).reshape(L, Hq)
    return o, lse


def _exact_votes(case, st):
    B, n_obs, Hq, d = st["q"].shape
    Hkv, S_max = case["Hkv"], st["smax"]
    G = Hq // Hkv
    out = torch.zeros((B, Hkv, max(1, S_max - n_obs)), dtype=torch.float64, device=DEV)
    for b in range(B):
        S = int(st["lens_np"][b])
        kb = _tokens(st["k"], st["pt"], b, S)
        qb = (st["q"][b].reshape(n_obs, Hkv, G, d).permute(1, 0, 2, 3)
              .reshape(Hkv, n_obs * G, d).to(torch.float64))
        s = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(d)
        qp = S - n_obs + torch.arange(n_obs, device=DEV).repeat_interleave(G)
        s = s.masked_fill(torch.arange(S, device=DEV)[None, None] > qp[None, :, None], -math.inf)
        out[b, :, : S - n_obs] = torch.softmax(s, 2).sum(1)[:, : S - n_obs]
    return out


def _put(t, pt, lens, rows):
    """rows [B, n, Hkv, d] written at positions lens[b] + i of the cache, in place."""
    for b in range(rows.shape[0]):
        for i in range(rows.shape[1]):
            p = int(lens[b]) + i
            if pt is None:
                t[b, p] = rows[b, i]
            else:
                t[int(pt[b, p // t.shape[1]]), p % t.shape[1]] = rows[b, i]


def exact(case, seed):
    st = prepare(case, seed)
    op = case["op"]
    if op in ("verify", "draft", "listed"):
        return _exact_attn(case, st["q"], st["k"], st["v"], st["pt"], st["lens_np"], op,
                           st.get("idx"), st.get("idx_len"))
    if op == "votes":
        return _exact_votes(case, st)
    if op == "collect":
        return None             # positions and copies: no 64-bit value
    L, k, v, pt, lens = case["q_len"], st["k"], st["v"], st["pt"], st["lens_np"]
    pt_host = None if pt is None else pt.cpu().numpy()
    outs = []
    for i in range(case["gamma"]):
        _put(k, pt_host, lens + i, st["kd"][i])
        _put(v, pt_host, lens + i, st["vd"][i])
        outs.append(_exact_attn(case, st["qd"][i], k, v, pt, lens + i + 1, "listed", st["idx"],
                                st["idx_len"]))
    _put(k, pt_host, lens, st["kn"])
    _put(v, pt_host, lens, st["vn"])
    outs.append(_exact_attn(case, st["q"], k, v, pt, lens + L, "verify"))
    return {"attn": outs, "accepted": None, "tokens": None, "target": None, "lens": None,
            "k": None, "v": None}
