"""What the speed of this library is measured on: the calls a serving loop makes on one GPU.

A case is a dict of plain values; its "kind" says which calls it makes:

  attend    the new K/V rows into the paged cache, then the verification attention over it
  accept    acceptance from target and draft logits
  probs     softmax of the target and draft rows, then acceptance from the probabilities
  fused     acceptance from logits whose statistics and gathered entries the LM head left
  head      the LM head of the verifying stage: gather columns, logits, statistics, gathers
  adapter   the drafting adapter's linear layers (input, stacked q/k/v, output with residual)
  schedule  what follows a drafting step: the draw with its confidence, the selection of drafts,
            the look-ahead memory estimate
  step      one whole verification step (VerifyStep)
  draft     one whole drafting step (DraftStep)

Sizes are those of this repository's workloads (Llama-3-8B/70B and Qwen3 head shapes and
vocabularies, 1 to 512 sequences) and of the range between them.  All inputs are drawn here, from
the seed alone; `exact` computes the same results with plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2609_34370_amd import spexis as sx
from paper_2609_34370_amd import workloads as wl
from paper_2609_34370_amd.draft import DraftStep
from paper_2609_34370_amd.step import VerifyStep

DEV = "cuda"

# the largest drawn case stays below the largest listed one
_MAX_CACHE_BYTES = 1.4e9
_MAX_LOGIT_BYTES = 2.5e9
_MAX_HEAD_FLOPS = 4.5e12


def listed():
    return [
        # a test or development server: a handful of short sequences, a small vocabulary; all
        # launches and host work
        dict(name="step_tiny", kind="step", batch=4, hq=8, hkv=2, dim=64, block=16, ctx_lo=32, ctx_hi=256, k_lo=4,
             k_hi=4, vocab=1024, std=2.0, noise=0.5, temp=1.0),
        # one user with a long document: a single sequence split over the whole chip
        dict(name="attend_one_long", kind="attend", batch=1, hq=32, hkv=8, dim=128, block=16, ctx_lo=16000,
             ctx_hi=16384, k_lo=4, k_hi=4),
        # the ordinary serving batch of an 8B model (this repository's headline workload)
        dict(name="attend_batch", kind="attend", batch=64, hq=32, hkv=8, dim=128, block=16, ctx_lo=1024, ctx_hi=4096,
             k_lo=4, k_hi=4),
        # a large batch with many drafts: 63 query rows per KV head, blocks of 32, seven heads a group
        dict(name="attend_stress", kind="attend", batch=512, hq=28, hkv=4, dim=128, block=32, ctx_lo=512, ctx_hi=2048,
             k_lo=8, k_hi=8),
        # acceptance of the ordinary batch from logits
        dict(name="accept_logits", kind="accept", batch=64, k_lo=4, k_hi=4, vocab=128256, std=3.0, noise=1.0, temp=1.0),
        # a caller that keeps probabilities: ragged draft counts (none among them), a 32K vocabulary
        dict(name="accept_probs", kind="probs", batch=128, k_lo=0, k_hi=8, vocab=32000, std=3.0, noise=1.0, temp=1.0),
        # acceptance behind the fused LM head, ordinary batch
        dict(name="accept_fused", kind="fused", batch=64, k_lo=4, k_hi=4, vocab=128256, std=3.0, noise=1.0, temp=1.0),
        # the verifying LM head of the ordinary batch: 320 rows
        dict(name="head_verify", kind="head", batch=64, k_lo=4, k_hi=4, vocab=128256, hidden=4096),
        # and of the large batch: 4608 rows
        dict(name="head_stress", kind="head", batch=512, k_lo=8, k_hi=8, vocab=152064, hidden=3584),
        # the adapter's linear layers at the large batch (28 query and 4 KV heads of 128)
        dict(name="adapter_512", kind="adapter", batch=512, hidden=3584, q_out=3584, kv_out=512),
        # after a drafting step of the ordinary batch
        dict(name="schedule_64", kind="schedule", batch=64, k_lo=4, k_hi=4, vocab=128256, alpha=0.15, iters=64, pp=4),
        # a whole drafting step of the ordinary batch
        dict(name="draft_step", kind="draft", model=2, batch=64, ctx_lo=1024, ctx_hi=4096, vocab=128256),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _vocab(rng):
    # the vocabularies of the workloads, or any size between a test's and a large model's
    return rng.choice([32000, 128256, 152064, _log(rng, 1000, 152064), _log(rng, 1000, 152064)])


def _drafts(rng, most):
    """Draft counts: the same for every sequence, or ragged."""
    hi = rng.randint(1, most)
    return (hi, hi) if rng.random() < 0.5 else (rng.randint(0, hi), hi)


def draw(rng):
    kind = rng.choice(["attend", "attend", "accept", "probs", "fused", "head", "head", "adapter", "schedule", "step",
                       "draft"])
    if kind in ("attend", "step"):
        hkv, group, dim = rng.choice([2, 4, 8]), rng.choice([4, 7, 8]), rng.choice([64, 128])
        block = rng.choice([16, 32])
        k_lo, k_hi = _drafts(rng, min(8, 64 // group - 1))
        batch = _log(rng, 1, 512 if kind == "attend" else 16)
        most = int(min(16384, _MAX_CACHE_BYTES / (batch * hkv * dim * 4)))
        hi = _log(rng, 128, most) if kind == "attend" else _log(rng, 64, 1024)
        c = dict(kind=kind, batch=batch, hq=hkv * group, hkv=hkv, dim=dim, block=block, ctx_lo=max(1, hi // 4),
                 ctx_hi=hi, k_lo=k_lo, k_hi=k_hi)
        if kind == "step":
            c.update(vocab=_log(rng, 1000, 32000), std=2.0, noise=0.5, temp=1.0)
        return c
    if kind in ("accept", "probs", "fused"):
        vocab = _vocab(rng)
        k_lo, k_hi = _drafts(rng, 8)
        most = int(_MAX_LOGIT_BYTES / ((2 * k_hi + 1) * vocab * 4))
        noise = rng.choice([1.0, 2.0])
        return dict(kind=kind, batch=_log(rng, 1, max(1, min(512, most))), k_lo=k_lo, k_hi=k_hi, vocab=vocab,
                    std=3.0 if noise == 1.0 else 4.0, noise=noise, temp=1.0 if noise == 1.0 else 0.7)
    if kind == "head":
        vocab, hidden, k = _vocab(rng), 256 * rng.choice([2, 8, 10, 14, 16]), rng.randint(0, 8)
        most = int(_MAX_HEAD_FLOPS / (2.0 * vocab * hidden * (k + 1)))
        return dict(kind=kind, batch=_log(rng, 1, max(1, min(512, most))), k_lo=k, k_hi=k, vocab=vocab, hidden=hidden)
    if kind == "adapter":
        hidden = 256 * rng.choice([2, 6, 8, 10, 14, 16])
        return dict(kind=kind, batch=_log(rng, 1, 512), hidden=hidden, q_out=hidden,
                    kv_out=128 * rng.choice([1, 2, 4, 8]))
    if kind == "schedule":
        k_lo, k_hi = _drafts(rng, 8)
        return dict(kind=kind, batch=_log(rng, 1, 512), k_lo=k_lo, k_hi=k_hi, vocab=_vocab(rng),
                    alpha=round(rng.uniform(0.05, 0.5), 3), iters=rng.randint(16, 128), pp=rng.randint(1, 8))
    hi = _log(rng, 128, 4096)
    return dict(kind=kind, model=rng.choice([2, 5]), batch=_log(rng, 1, 256), ctx_lo=max(1, hi // 4), ctx_hi=hi,
                vocab=rng.choice([32000, 128256]))


# ------------------------------------------------------------------------------------- inputs


def _rng(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + stream)
    return g


def _randn_bf16(shape, g, std=1.0):
    x = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = x.view(-1)
    for s in range(0, flat.numel(), 1 << 27):
        e = min(flat.numel(), s + (1 << 27))
        flat[s:e] = torch.randn(e - s, generator=g, device=DEV) * std
    return x


def _batch(case, seed):
    """Lengths, draft counts and randomly placed blocks of a batch (the attention kinds); only the
    draft counts for the others.  A case's sequences are the same for every seed, in another order,
    so that its sizes don't change with it."""
    B = case["batch"]
    fixed, r = np.random.default_rng(B), np.random.default_rng([int(seed), 7])
    order = r.permutation(B)
    k = fixed.integers(case.get("k_lo", 0), case.get("k_hi", 0) + 1, size=B).astype(np.int32)[order]
    qsl = np.zeros(B + 1, dtype=np.int32)
    qsl[1:] = np.cumsum(k + 1)
    if "ctx_hi" not in case:
        return k, qsl
    ctx = fixed.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=B).astype(np.int32)[order]
    S = ctx + k + 1
    nblk = -(-S // case["block"])
    perm = r.permutation(int(nblk.sum())).astype(np.int32)
    tables = np.zeros((B, int(nblk.max())), dtype=np.int32)
    ends = np.cumsum(nblk)
    for b in range(B):
        tables[b, : nblk[b]] = perm[ends[b] - nblk[b]: ends[b]]
    return k, qsl, ctx, S.astype(np.int32), tables, int(nblk.sum())


def _spec(case):
    if case["kind"] == "draft":
        return wl.spec_with(case["model"], batch=case["batch"], k=("fixed", 0), vocab=case["vocab"],
                            ctx=("uniform", case["ctx_lo"], case["ctx_hi"]))
    return wl.WorkloadSpec(0, "case", case["batch"], case["hq"], case["hkv"], case["dim"], case["block"],
                           ("uniform", case["ctx_lo"], case["ctx_hi"]), ("uniform", case["k_lo"], case["k_hi"]),
                           case.get("vocab", 1), case.get("std", 1.0), ("fixed", case.get("noise", 1.0)),
                           temperature=case.get("temp", 1.0))


def _cache(case, seed):
    """The batch and what the attention reads, N(0, 1) as after a normalisation."""
    s = _spec(case)
    k, qsl, ctx, S, tables, blocks = _batch(dict(case, block=s.block_size), seed)
    batch = wl.Batch(s, ctx, k, qsl, S, tables, blocks)
    g = _rng(seed, 0)
    pool = (blocks * s.num_kv_heads * s.block_size * s.head_dim,)
    k_pool, v_pool = _randn_bf16(pool, g), _randn_bf16(pool, g)
    q = _randn_bf16((batch.T, s.num_q_heads, s.head_dim), g)
    new = (batch.T, s.num_kv_heads, s.head_dim)
    return batch, wl.AttentionInputs(k_pool, v_pool, q, _randn_bf16(new, g), _randn_bf16(new, g))


def _logits(case, seed):
    """Target logits, draft logits (target + noise), drafts drawn from the draft rows, uniforms."""
    k, qsl = _batch({n: case[n] for n in ("batch", "k_lo", "k_hi")}, seed)
    B, T, V = case["batch"], int(qsl[-1]), case["vocab"]
    g = _rng(seed, 1)
    target = torch.randn((T, V), generator=g, device=DEV).mul_(case["std"])
    src = np.concatenate([np.arange(qsl[b], qsl[b] + k[b]) for b in range(B)]).astype(np.int64)
    draft = torch.empty((T - B, V), dtype=torch.float32, device=DEV)
    ids = torch.empty(T - B, dtype=torch.int32, device=DEV)
    for s in range(0, T - B, 512):
        e = min(T - B, s + 512)
        draft[s:e] = target[torch.as_tensor(src[s:e], device=DEV)]
        draft[s:e] += torch.randn((e - s, V), generator=g, device=DEV).mul_(case["noise"])
        # Gumbel-max draw from softmax(draft / T)
        gumbel = torch.empty((e - s, V), device=DEV).exponential_(generator=g).log_().neg_()
        ids[s:e] = torch.argmax(draft[s:e] / case["temp"] + gumbel, dim=1).to(torch.int32)
    u = torch.randint(0, 1 << 24, (T,), generator=g, device=DEV).to(torch.float32) / (1 << 24)
    return k, qsl, wl.AcceptInputs(target, draft, ids, u[: T - B].contiguous(), u[T - B:].contiguous(), case["temp"])


def _tile_stats(x, temp):
    """What the LM head leaves of logit rows: (max, sum of 2^(x c - max)) over every 128 columns."""
    tiles = -(-x.shape[1] // 128)
    out = torch.empty((x.shape[0], tiles, 2), dtype=torch.float32, device=DEV)
    c = 1.4426950408889634 / temp
    for s in range(0, x.shape[0], 256):
        y = torch.nn.functional.pad(x[s: s + 256] * c, (0, tiles * 128 - x.shape[1]), value=-math.inf)
        y = y.view(-1, tiles, 128)
        m = y.amax(dim=2)
        out[s: s + 256, :, 0] = m
        out[s: s + 256, :, 1] = torch.exp2(y - m.unsqueeze(2)).sum(dim=2)
    return out


def _hidden(case, seed):
    k, qsl = _batch(case, seed)
    T, d, V, g = int(qsl[-1]), case["hidden"], case["vocab"], _rng(seed, 2)
    h = _randn_bf16((T, d), g)
    w = _randn_bf16((V, d), g, 2.0 / d ** 0.5)   # logits of standard deviation about 2
    ids = torch.randint(0, V, (max(T - case["batch"], 0),), generator=g, device=DEV).to(torch.int32)
    return k, qsl, h, w, ids


def _layers(case, seed):
    B, d, g = case["batch"], case["hidden"], _rng(seed, 3)
    h, o = _randn_bf16((B, d), g), _randn_bf16((B, case["q_out"]), g)
    w_in = _randn_bf16((d, d), g, d ** -0.5)
    w_q = _randn_bf16((case["q_out"], d), g, d ** -0.5)
    w_k = _randn_bf16((case["kv_out"], d), g, d ** -0.5)
    w_v = _randn_bf16((case["kv_out"], d), g, d ** -0.5)
    w_o = _randn_bf16((d, case["q_out"]), g, case["q_out"] ** -0.5)
    return h, o, w_in, w_q, w_k, w_v, w_o


def _adapter(case, seed):
    s = _spec(case)
    d = s.num_q_heads * s.head_dim
    h, _, w_in, w_q, w_k, w_v, w_o = _layers(
        dict(batch=case["batch"], hidden=d, q_out=d, kv_out=s.num_kv_heads * s.head_dim), seed)
    w_lm = _randn_bf16((s.vocab, d), _rng(seed, 4), 2.0 / d ** 0.5)
    u = torch.rand(case["batch"], generator=_rng(seed, 5), device=DEV)
    return wl.AdapterInputs(h, w_in, w_q, w_k, w_v, w_o, w_lm, u, s.temperature)


def _schedule(case, seed):
    k, qsl = _batch(case, seed)
    B, g = case["batch"], _rng(seed, 6)
    logits = torch.randn((B, case["vocab"]), generator=g, device=DEV).mul_(3.0)
    u = torch.rand(B, generator=g, device=DEV)
    conf = torch.rand(int(qsl[-1]) - B, generator=g, device=DEV).sqrt_()
    cur = torch.randint(32, 4096, (B,), generator=g, device=DEV)
    rem = (torch.randint(1, 18, (B,), generator=g, device=DEV) * 4).to(torch.int32)
    prec = torch.rand(B, generator=g, device=DEV, dtype=torch.float64)
    return k, qsl, logits, u, conf, cur, rem, prec


# ---------------------------------------------------------------------------------- prepare, run


def _ints(*shape):
    return torch.zeros(shape, dtype=torch.int32, device=DEV)


def _bytes(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "attend":
        batch, a = _cache(case, seed)
        st["step"] = VerifyStep(batch, a, None)
    elif kind == "step":
        batch, a = _cache(case, seed)
        st["step"] = VerifyStep(batch, a, _logits(case, seed)[2])
    elif kind in ("accept", "probs", "fused"):
        k, qsl, a = _logits(case, seed)
        B, max_k = case["batch"], int(k.max())
        st.update(acc=a, max_k=max_k, qsl=torch.as_tensor(qsl, device=DEV), a=_ints(B), tok=_ints(B, max_k + 1),
                  status=_ints(B), ws=_bytes(sx.spexis_accept_workspace_size(B, case["vocab"], max_k)))
        if kind == "probs":
            st.update(p=torch.empty_like(a.target_logits), q=torch.empty_like(a.draft_logits))
        if kind == "fused":
            cols = torch.full((int(qsl[-1]),), -1, dtype=torch.int64, device=DEV)
            rows = np.concatenate([np.arange(qsl[b], qsl[b] + k[b]) for b in range(B)]).astype(np.int64)
            cols[torch.as_tensor(rows, device=DEV)] = a.draft_ids.long()
            st.update(ts=_tile_stats(a.target_logits, case["temp"]), ds=_tile_stats(a.draft_logits, case["temp"]),
                      tg=a.target_logits.gather(1, cols.clamp(min=0).unsqueeze(1)).squeeze(1).contiguous(),
                      dg=a.draft_logits.gather(1, a.draft_ids.long().unsqueeze(1)).squeeze(1).contiguous())
    elif kind == "head":
        k, qsl, h, w, ids = _hidden(case, seed)
        T, V = int(qsl[-1]), case["vocab"]
        st.update(qsl=torch.as_tensor(qsl, device=DEV), h=h, w=sx.spexis_pack_weight(w), ids=ids, cols=_ints(T),
                  gathered=torch.zeros(T, device=DEV), logits=torch.empty((T, V), device=DEV),
                  stats=torch.empty((T, sx.spexis_lm_head_tiles(V), 2), device=DEV))
    elif kind == "adapter":
        h, o, w_in, w_q, w_k, w_v, w_o = _layers(case, seed)
        B, d, nq, nkv = case["batch"], case["hidden"], case["q_out"], case["kv_out"]
        bf = dict(dtype=torch.bfloat16, device=DEV)
        ws = max(sx.spexis_linear_workspace_size(B, d, d), sx.spexis_linear_workspace_size(B, d, nq),
                 sx.spexis_linear_split_workspace_size(B, nq + 2 * nkv, d))
        st.update(h=h, o=o, w_in=sx.spexis_pack_weight(w_in), w_o=sx.spexis_pack_weight(w_o),
                  w_qkv=sx.spexis_pack_weight(torch.cat([w_q, w_k, w_v], dim=0)), x=torch.empty((B, d), **bf),
                  q=torch.empty((B, nq), **bf), k=torch.empty((B, nkv), **bf), v=torch.empty((B, nkv), **bf),
                  y=torch.empty((B, d), **bf), ws=_bytes(ws))
    elif kind == "schedule":
        k, qsl, logits, u, conf, cur, rem, prec = _schedule(case, seed)
        B, V = case["batch"], case["vocab"]
        st.update(qsl=torch.as_tensor(qsl, device=DEV), logits=logits, stats=_tile_stats(logits, 1.0), u=u, conf=conf,
                  tok=_ints(B), status=_ints(B), prob=torch.zeros(B, device=DEV), kept_k=_ints(B),
                  kept_qsl=_ints(B + 1), keep=_ints(conf.shape[0]), cur=cur, rem=rem, prec=prec,
                  mem=torch.zeros(case["iters"], dtype=torch.float64, device=DEV),
                  ws=_bytes(sx.spexis_sample_workspace_size(B, V)))
    else:
        batch, cache = _cache(case, seed)
        st["step"] = DraftStep(batch, cache, _adapter(case, seed))
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind in ("attend", "step"):
        s = st["step"]
        s.run()
        got = dict(out=s.out, k_pool=s.attn.k_pool, v_pool=s.attn.v_pool)
        if kind == "step":
            got.update(accepted=s.accepted_len, tokens=s.out_tokens, status=s.row_status)
        return got
    if kind in ("accept", "probs", "fused"):
        a = st["acc"]
        got = dict(accepted=st["a"], tokens=st["tok"], status=st["status"])
        if kind == "fused":
            sx.spexis_accept_with_stats(st["qsl"], a.target_logits, a.draft_logits, st["ts"], st["ds"], a.draft_ids,
                                        a.u_accept, a.u_sample, st["max_k"], st["a"], st["tok"], st["status"], st["ws"],
                                        temperature=a.temperature, target_gathered=st["tg"], draft_gathered=st["dg"])
            return got
        p, q, which = a.target_logits, a.draft_logits, sx.SPEXIS_INPUT_LOGITS
        if kind == "probs":
            sx.spexis_softmax_rows(p, st["p"], a.temperature)
            sx.spexis_softmax_rows(q, st["q"], a.temperature)
            p, q, which = st["p"], st["q"], sx.SPEXIS_INPUT_PROBS
            got.update(p=p, q=q)
        sx.spexis_accept(which, st["qsl"], p, q, a.draft_ids, a.u_accept, a.u_sample, st["max_k"], st["a"], st["tok"],
                         st["status"], st["ws"], temperature=a.temperature)
        return got
    if kind == "head":
        sx.spexis_verify_gather_columns(st["qsl"], st["ids"], st["cols"])
        sx.spexis_lm_head_gather(st["h"], st["w"], st["stats"], st["cols"], st["gathered"], logits=st["logits"])
        return dict(logits=st["logits"], stats=st["stats"], gathered=st["gathered"])
    if kind == "adapter":
        sx.spexis_linear(st["h"], st["w_in"], st["x"], workspace=st["ws"])
        sx.spexis_linear_split(st["x"], st["w_qkv"], [st["q"], st["k"], st["v"]], st["ws"])
        sx.spexis_linear(st["o"], st["w_o"], st["y"], residual=st["x"], workspace=st["ws"])
        return {n: st[n] for n in "xqkvy"}
    if kind == "schedule":
        sx.spexis_sample_tokens(sx.SPEXIS_INPUT_LOGITS, st["logits"], st["u"], st["tok"], st["status"], st["ws"],
                                token_prob=st["prob"], stats=st["stats"])
        sx.spexis_select_drafts(st["qsl"], st["conf"], case["alpha"], st["kept_k"], st["kept_qsl"], st["keep"])
        sx.spexis_lookahead_memory(st["cur"], st["rem"], st["prec"], case["pp"], 0.6, st["mem"])
        return {n: st[n] for n in ("tok", "status", "prob", "kept_k", "kept_qsl", "keep", "mem")}
    # The draws of a drafting step aren't compared: a bf16 rounding that differs in one layer moves
    # a row's cumulative distribution by more than a token's own share of it now and then.  The
    # schedule cases compare the draw, from given logits.
    s = st["step"]
    s.run()
    return dict(logits=s.logits, y=s.y, k_pool=s.cache.k_pool, v_pool=s.cache.v_pool)


# ------------------------------------------------------------------------------- work, tolerance


def _accepted(case):
    """Drafts accepted per sequence on average: measured acceptance rates of the two noise levels."""
    k = (case["k_lo"] + case["k_hi"]) / 2
    r = 0.7 if case["noise"] <= 1.0 else 0.3
    return r * (1 - r ** k) / (1 - r), k


def work(case):
    kind = case["kind"]
    B = case["batch"]
    out = dict(bytes=0.0, flops=0.0)

    def add(b, f=0.0):
        out["bytes"] += b
        out["flops"] += f

    if kind in ("attend", "step", "draft"):
        s = _spec(case)
        n = 1 + (case.get("k_lo", 0) + case.get("k_hi", 0)) / 2
        S = (case["ctx_lo"] + case["ctx_hi"]) / 2 + n
        D = s.head_dim
        # every cached row once, the queries and outputs, the new rows read and written
        add(B * (S * s.num_kv_heads * D * 4 + n * s.num_q_heads * D * 4 + n * s.num_kv_heads * D * 8),
            4.0 * B * n * S * s.num_q_heads * D)
    if kind in ("accept", "step"):
        # target rows 0..a and draft rows 0..min(a, k-1): the normalisers of the tests, the sampled rows
        a, k = _accepted(case)
        add(B * 4.0 * case["vocab"] * (a + 1 + min(a + 1, k)))
    if kind == "probs":
        a, k = _accepted(case)
        rows = B * (2 * k + 1)
        add(rows * case["vocab"] * 8.0 + 2 * B * case["vocab"] * 4.0)   # both softmaxes, the sampled rows
    if kind == "fused":
        a, k = _accepted(case)
        add(B * (2 * k + 1) * -(-case["vocab"] // 128) * 8.0 + 2 * B * case["vocab"] * 4.0)
    if kind == "schedule":
        add(B * (case["vocab"] * 4.0 + -(-case["vocab"] // 128) * 8.0))
    if kind == "head":
        T, V, d = B * (1 + (case["k_lo"] + case["k_hi"]) / 2), case["vocab"], case["hidden"]
        add(2.0 * V * d + 2.0 * T * d + 4.0 * T * V, 2.0 * T * V * d)
    if kind in ("adapter", "draft"):
        if kind == "draft":
            d = nq = s.num_q_heads * s.head_dim
            nkv = s.num_kv_heads * s.head_dim
            add(2.0 * s.vocab * d + 4.0 * B * s.vocab, 2.0 * B * s.vocab * d)
        else:
            d, nq, nkv = case["hidden"], case["q_out"], case["kv_out"]
        weights = d * d + (nq + 2 * nkv) * d + d * nq
        add(2.0 * weights + 2.0 * B * (3 * d + 2 * nq + 2 * nkv), 2.0 * B * weights)
    return out


def tolerance(case):
    """Relative errors, each about four times what was measured against 64 bits; whole numbers (the
    decisions of acceptance and selection) are the same but for a uniform that falls between two
    roundings of a boundary."""
    kind = case["kind"]
    if kind in ("attend", "step"):
        return {"rel": 1e-2, "differ": 0.0}      # bf16 probabilities and output
    if kind == "adapter":
        return {"rel": 1e-2}                     # bf16 output of a layer on bf16 outputs
    if kind == "draft":
        return {"rel": 1e-2}                     # a chain of bf16 layers
    if kind == "head":
        return {"rel": 4e-6}                     # fp32 sums of up to 4096 products
    if kind in ("probs", "schedule"):
        return {"rel": 1e-6, "differ": 0.0}      # fp32 exponentials and sums
    return "exact"                               # accept, fused: whole numbers only


# ------------------------------------------------------------------------------------- 64 bits


def _exact_attention(batch, a, q, new_k, new_v):
    """[T][Hq][D] in 64 bits: every query row over its sequence's blocks, the new rows in place."""
    s = batch.spec
    hkv, D, bs = s.num_kv_heads, s.head_dim, s.block_size
    G = s.num_q_heads // hkv
    kp = a.k_pool.view(-1, hkv, D // 8, bs, 8)
    vp = a.v_pool.view(-1, hkv, D, bs)
    slot = torch.arange(bs, device=DEV)
    slot = (slot & ~12) | ((slot >> 2 & 1) << 3) | ((slot >> 3 & 1) << 2)
    out = torch.empty((batch.T, s.num_q_heads, D), dtype=torch.float64, device=DEV)
    for b in range(batch.B):
        S, q0, n = int(batch.seq_lens[b]), int(batch.qsl[b]), int(batch.k[b]) + 1
        blocks = torch.as_tensor(batch.block_tables[b, : -(-S // bs)].astype(np.int64), device=DEV)
        k = kp[blocks].permute(1, 0, 3, 2, 4).reshape(hkv, -1, D)[:, :S].double()
        v = vp[blocks][..., slot].permute(1, 0, 3, 2).reshape(hkv, -1, D)[:, :S].double()
        k[:, S - n:] = new_k[q0: q0 + n].double().transpose(0, 1)
        v[:, S - n:] = new_v[q0: q0 + n].double().transpose(0, 1)
        x = q[q0: q0 + n].double().view(n, hkv, G, D).permute(1, 0, 2, 3).reshape(hkv, n * G, D)
        sc = torch.matmul(x, k.transpose(1, 2).contiguous()) / math.sqrt(D)
        lim = torch.arange(S - n, S, device=DEV).repeat_interleave(G)
        sc.masked_fill_(torch.arange(S, device=DEV)[None, :] > lim[:, None], -math.inf)
        o = torch.matmul(torch.softmax(sc, dim=2), v.contiguous())
        out[q0: q0 + n] = o.view(hkv, n, G, D).permute(1, 0, 2, 3).reshape(n, hkv * G, D)
    return out


def _exact_head(h, w):
    out = torch.empty((h.shape[0], w.shape[0]), dtype=torch.float64, device=DEV)
    hd = h.double()
    for s in range(0, w.shape[0], 16384):
        out[:, s: s + 16384] = hd @ w[s: s + 16384].double().t()
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("attend", "step"):
        batch, a = _cache(case, seed)
        return dict(out=_exact_attention(batch, a, a.q, a.new_k, a.new_v), k_pool=None, v_pool=None)
    if kind == "probs":
        a = _logits(case, seed)[2]
        p = torch.softmax(a.target_logits.double() / case["temp"], dim=1)
        q = torch.softmax(a.draft_logits.double() / case["temp"], dim=1)
        return dict(p=p, q=q, accepted=None, tokens=None, status=None)
    if kind == "head":
        k, qsl, h, w, ids = _hidden(case, seed)
        T, V = int(qsl[-1]), case["vocab"]
        logits = _exact_head(h, w)
        tiles = -(-V // 128)
        stats = torch.empty((T, tiles, 2), dtype=torch.float64, device=DEV)
        gathered = torch.zeros(T, dtype=torch.float64, device=DEV)
        for s in range(0, T, 256):
            y = torch.nn.functional.pad(logits[s: s + 256] * 1.4426950408889634, (0, tiles * 128 - V), value=-math.inf)
            y = y.view(-1, tiles, 128)
            stats[s: s + 256, :, 0] = y.amax(dim=2)
            stats[s: s + 256, :, 1] = torch.exp2(y - stats[s: s + 256, :, :1]).sum(dim=2)
        rows = np.concatenate([np.arange(qsl[b], qsl[b] + k[b]) for b in range(case["batch"])]).astype(np.int64)
        rows = torch.as_tensor(rows, device=DEV)
        gathered[rows] = logits[rows, ids.long()]
        return dict(logits=logits, stats=stats, gathered=gathered)
    if kind == "adapter":
        h, o, w_in, w_q, w_k, w_v, w_o = (t.double() for t in _layers(case, seed))
        x = h @ w_in.t()
        return dict(x=x, q=x @ w_q.t(), k=x @ w_k.t(), v=x @ w_v.t(), y=o @ w_o.t() + x)
    if kind == "schedule":
        _, _, logits, u, _, cur, rem, prec = _schedule(case, seed)
        p = torch.softmax(logits.double(), dim=1)
        at = torch.searchsorted(p.cumsum(dim=1), u.double().unsqueeze(1), right=True).clamp_(max=case["vocab"] - 1)
        mem, theta, n = [], 0.6, case["batch"]
        for i in range(1, case["iters"] + 1):
            e_gen, fin = 0.0, torch.zeros(n, dtype=torch.float64, device=DEV)
            for w in range(i // case["pp"] + 1):
                t = i - case["pp"] * w
                term = math.comb(t + w, t) * theta ** t * (1 - theta) ** w
                e_gen += (t + w) * term
                fin += (rem <= t + w).double() * term
            fin = fin * prec
            mem.append(cur.double().sum() + (n - fin.sum()) * e_gen - (cur.double() * fin).sum())
        return dict(prob=p.gather(1, at).squeeze(1), mem=torch.stack(mem), tok=None, status=None, kept_k=None,
                    kept_qsl=None, keep=None)
    if kind == "draft":
        batch, cache = _cache(case, seed)
        ad = _adapter(case, seed)
        s, B = batch.spec, case["batch"]
        x = ad.h.double() @ ad.w_in.double().t()
        q = (x @ ad.w_q.double().t()).view(B, s.num_q_heads, s.head_dim)
        k = (x @ ad.w_k.double().t()).view(B, s.num_kv_heads, s.head_dim)
        v = (x @ ad.w_v.double().t()).view(B, s.num_kv_heads, s.head_dim)
        y = _exact_attention(batch, cache, q, k, v).view(B, -1) @ ad.w_o.double().t() + x
        return dict(logits=_exact_head(y, ad.w_lm), y=y, k_pool=None, v_pool=None)
    return None   # accept, fused: whole numbers
