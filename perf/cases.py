"""The work that a serving or training program has this library do, as cases that can be timed and compared.

Kinds of cases (the sizes are those of the repository's own configurations, or lie around them):

draft    K recursive draft steps and the greedy acceptance for a batch of sequences, from one sequence (latency) to
         batches; long contexts are bound by the KV cache, short ones by the weights.
lists    the same with one id list per sequence (a batch in several languages).
extend   the first draft step over a block of new positions per sequence: the tokens a verification has confirmed
         (a few positions) or a prompt (hundreds).
cycle    one turn of the drafting loop: the block of confirmed positions, the recursive steps from its last output,
         the acceptance.
train    the teacher-forced forward over one sequence and its weighted cross-entropy, full vocabulary.
build    the high-frequency id list of a token stream.

A case holds plain values; `shape` names a head, `rows` the size of the compressed vocabulary (0: the full one).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_18362_amd import binding, synth

DEVICE = "cuda:0"

SHAPES = {
    "tiny": synth.TINY,
    "mid": synth.HeadShape(2048, 16, 8, 128, 6144, 65536),   # a head of a small model: half the width, G = 2
    "7b": synth.SEVEN_B,
}


def listed():
    return [
        # the smallest call: a toy head, where launches and latency are everything
        dict(name="draft_tiny_b1", kind="draft", shape="tiny", batch=1, steps=3, ctx_lo=128, ctx_hi=128, rows=1024),
        # one user, the headline: 32768 of 151680 rows, 2k context
        dict(name="draft_7b_b1", kind="draft", shape="7b", batch=1, steps=3, ctx_lo=2048, ctx_hi=2048, rows=32768),
        # one user without the compressed vocabulary, 8k context
        dict(name="draft_7b_b1_full_8k", kind="draft", shape="7b", batch=1, steps=3, ctx_lo=8192, ctx_hi=8192, rows=0),
        # a handful of users with ragged contexts
        dict(name="draft_7b_b5", kind="draft", shape="7b", batch=5, steps=3, ctx_lo=200, ctx_hi=3000, rows=16384),
        # a small serving batch
        dict(name="draft_7b_b16", kind="draft", shape="7b", batch=16, steps=3, ctx_lo=512, ctx_hi=4096, rows=32768),
        # a large batch of long contexts, five steps
        dict(name="draft_7b_b64_32k", kind="draft", shape="7b", batch=64, steps=5, ctx_lo=8192, ctx_hi=32768, rows=32768),
        # several languages in one batch
        dict(name="lists_7b_b24", kind="lists", shape="7b", batch=24, steps=3, ctx_lo=512, ctx_hi=4096, rows=32768),
        # the loop of one user: four confirmed positions, two recursive steps, acceptance
        dict(name="cycle_7b_b1", kind="cycle", shape="7b", batch=1, steps=3, ctx_lo=2048, ctx_hi=2048, rows=32768, block=4),
        # the confirmed positions of a serving batch
        dict(name="extend_7b_b16x4", kind="extend", shape="7b", batch=16, ctx_lo=512, ctx_hi=4096, rows=32768, block=4),
        # a prompt of odd length into an empty cache
        dict(name="prompt_7b_509", kind="extend", shape="7b", batch=1, ctx_lo=0, ctx_hi=0, rows=32768, block=509),
        # the training objective over 512 positions
        dict(name="train_7b_512", kind="train", shape="7b", positions=512, steps=3),
        # the id list of a corpus shard
        dict(name="build_64m", kind="build", vocab=151680, tokens=1 << 26, rows=32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["draft", "draft", "draft", "lists", "extend", "extend", "cycle", "train", "build"])
    if kind == "build":
        vocab = rng.choice([4096, 65536, 151680, 200001])
        return dict(kind=kind, vocab=vocab, tokens=_log_int(rng, 1 << 18, 1 << 26),
                    rows=rng.choice([vocab // 9, vocab // 5, vocab // 2 + 1]))
    shape = rng.choice(["tiny", "mid", "7b", "7b", "7b"])
    vocab = SHAPES[shape].vocab_size
    if kind == "train":
        return dict(kind=kind, shape=shape, positions=_log_int(rng, 24, 512), steps=rng.randint(1, 3))
    rows = rng.choice([vocab // 9, vocab // 5, vocab // 2 + 1, 0])
    if kind == "extend" and rng.random() < 0.5:  # a prompt, or a piece of one
        lo = rng.choice([0, 0, rng.randint(1, 2048)])
        return dict(kind=kind, shape=shape, batch=1, ctx_lo=lo, ctx_hi=lo, rows=rows, block=_log_int(rng, 16, 512))
    batch = {"cycle": 1, "lists": _log_int(rng, 3, 48)}.get(kind) or _log_int(rng, 1, 64 if kind == "draft" else 32)
    lo = _log_int(rng, 16, 8192)
    hi = min(lo * rng.choice([1, 2, 4]), 32768)
    case = dict(kind=kind, shape=shape, batch=batch, ctx_lo=lo, ctx_hi=hi, rows=rows)
    if kind != "extend":
        case["steps"] = rng.randint(2, 5)
    if kind in ("extend", "cycle"):
        case["block"] = rng.randint(2, 6)
    while work(case)["bytes"] > 3e10:  # no more than the largest listed case
        case["ctx_lo"], case["ctx_hi"] = case["ctx_lo"] // 2, case["ctx_hi"] // 2
    return case


# ------------------------------------------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed) * 7919 + 17)


def _normal(g, shape, mean=0.0, std=1.0):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEVICE).normal_(mean, std, generator=g)


def _lists(case):
    """Sizes of the call's id lists; 0: the full vocabulary."""
    if case["kind"] != "lists":
        return [case["rows"]]
    vocab = SHAPES[case["shape"]].vocab_size
    base = case["rows"] or vocab // 4
    return [base, base // 2, base // 4 + 3]


def _inputs(case, seed):
    """Weights, id lists, caches and tokens of a case, as the tensors a program holds."""
    g, rng = _generator(seed), np.random.default_rng(int(seed) + 101)
    x = {}
    if case["kind"] == "build":
        # long-tailed ids, P(rank r) ~ 1/(r+1)^1.1, ranks scattered over the vocabulary; a few ids out of range
        V, n = case["vocab"], case["tokens"]
        w = 1.0 / np.power(np.arange(V, dtype=np.float64) + 1.0, 1.1)
        cdf = torch.from_numpy(np.cumsum(w) / w.sum()).to(DEVICE)
        perm = torch.from_numpy(rng.permutation(V).astype(np.int32)).to(DEVICE)
        out = torch.empty(n, dtype=torch.int32, device=DEVICE)
        for lo in range(0, n, 1 << 24):
            hi = min(n, lo + (1 << 24))
            u = torch.rand(hi - lo, dtype=torch.float64, device=DEVICE, generator=g)
            out[lo:hi] = perm[torch.searchsorted(cdf, u).clamp_(max=V - 1)]
        out[4095::65536] = -1
        x["tokens"] = out
        return x
    s = SHAPES[case["shape"]]
    x["w"] = {}
    for name, shp in synth.weight_shapes(s).items():
        x["w"][name] = _normal(g, shp, 1.0 if name.startswith("g_") else 0.0, 0.02)
    if case["kind"] == "train":
        n, K = case["positions"], case["steps"]
        x["hidden"] = _normal(g, (n, s.d_model))
        x["tokens"] = torch.from_numpy(rng.integers(0, s.vocab_size, n + K + 1).astype(np.int32)).to(DEVICE)
        return x
    # compressed vocabularies: weighted draws without replacement, weight 1/(id+1), ascending, nested
    key = np.log(np.maximum(rng.random(s.vocab_size), 1e-300)) * (np.arange(s.vocab_size) + 1.0)
    order = np.argsort(-key, kind="stable")
    x["lists"] = [np.sort(order[:n]).astype(np.int32) for n in _lists(case) if n > 0]
    B, m = case["batch"], case.get("block", 0)
    ctx = rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, B).astype(np.int32)
    x["cap"] = -(-(case["ctx_hi"] + m + case.get("steps", 0)) // 64) * 64
    x["ctx"] = ctx
    x["kv_len"] = torch.from_numpy(ctx).to(DEVICE)
    x["k_cache"] = _normal(g, (B, s.n_kv_heads, x["cap"], s.head_dim))
    x["v_cache"] = _normal(g, (B, s.n_kv_heads, x["cap"], s.head_dim))
    rows = (m, B) if m else (B,)
    x["hidden"] = _normal(g, rows + (s.d_model,))
    x["token"] = torch.from_numpy(rng.integers(0, s.vocab_size, rows).astype(np.int32)).to(DEVICE)
    if m:
        x["ext_len"] = torch.full((B,), m, dtype=torch.int32, device=DEVICE)
        if B > 1:  # a verification confirms one to `block` tokens of each sequence
            x["ext_len"].copy_(torch.from_numpy(rng.integers(1, m + 1, B).astype(np.int32)))
    K = case.get("steps", 0)
    if K:
        x["target"] = torch.from_numpy(rng.integers(0, s.vocab_size, (B, K + 1)).astype(np.int32)).to(DEVICE)
        # Large batches draft along given tokens: one near-tie among hundreds of argmaxes, taken the other way by
        # another order of summation, would change all that follows in its sequence.  Small ones draft freely.
        if B > 16:
            x["forced"] = torch.from_numpy(rng.integers(0, s.vocab_size, (B, K - 1)).astype(np.int32)).to(DEVICE)
    if case["kind"] == "lists":  # sequences sorted by list, as the library asks for
        x["seq_list"] = [min(3 * b // B, 2) for b in range(B)]
    return x


def _rows_of(case):
    """(position, sequence) rows of the largest call."""
    return case["positions"] if case["kind"] == "train" else case["batch"] * case.get("block", 1)


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "build":
        return {"case": case, "x": x}
    s = SHAPES[case["shape"]]
    cap = -(-case["positions"] // 64) * 64 if case["kind"] == "train" else x["cap"]
    eng = binding.DraftEngine(s, x["w"], x.get("lists", []), _rows_of(case), cap, case.get("steps", 1), device=DEVICE)
    st = {"case": case, "x": x, "eng": eng}
    if "kv_len" in x:
        st["kv"] = x["kv_len"].clone()
    if case["kind"] == "extend" and case["batch"] > 1:
        live = torch.arange(case["block"], device=DEVICE)[:, None] < x["ext_len"][None, :]
        st["live"] = live[:, :, None].float()
    return st


# --------------------------------------------------------------------------------------------- one pass
def run(st):
    case, x = st["case"], st["x"]
    kind = case["kind"]
    if kind == "build":
        out = binding.build_subset(x["tokens"], case["vocab"], case["rows"], want_counts=True)
        return {"ids": out["ids"], "counts": out["counts"], "invalid": out["invalid"]}
    eng = st["eng"]
    if kind == "train":
        loss, logits = eng.train_loss(x["hidden"], x["tokens"], case["steps"], 0.6, want_logits=True)
        return {"loss": loss, "logits": logits}
    subset = 0 if x["lists"] else -1
    kc, vc, kv = x["k_cache"], x["v_cache"], st["kv"]
    if kind == "extend":
        kv.copy_(x["kv_len"])  # the call advances the lengths
        out = eng.extend(subset, x["hidden"], x["token"], x["ext_len"], kc, vc, kv, want_logits=True, want_hidden=True)
        if "live" in st:  # rows of positions a sequence does not have are unspecified
            out["logits"].mul_(st["live"])
            out["hidden"].mul_(st["live"])
        return dict(out, kv_len=kv, k_cache=kc, v_cache=vc)
    if kind == "cycle":
        kv.copy_(x["kv_len"])
        blk = eng.extend(subset, x["hidden"], x["token"], x["ext_len"], kc, vc, kv, want_logits=True, want_hidden=True)
        first = blk["draft"][-1].clone()
        out = eng.draft_continue(case["steps"] - 1, subset, blk["hidden"][-1], first, kc, vc, kv, want_logits=True,
                                 want_hidden=True)
        draft = torch.cat([first[:, None], out["draft"]], dim=1)
        acc = eng.accept(draft, x["target"], kv, mode=1)
        return {"draft": draft, "block": blk["draft"], "block_logits": blk["logits"], "block_hidden": blk["hidden"],
                "logits": out["logits"], "hidden": out["hidden"], "accept_len": acc["accept_len"],
                "out_tokens": acc["out_tokens"], "kv_len": kv, "k_cache": kc, "v_cache": vc}
    forced = x.get("forced")
    if kind == "lists":
        out = eng.draft_lists(case["steps"], x["seq_list"], x["hidden"], x["token"], kc, vc, kv, forced=forced,
                              want_logits=True, want_hidden=True)
    else:
        out = eng.draft(case["steps"], subset, x["hidden"], x["token"], kc, vc, kv, forced=forced, want_logits=True,
                        want_hidden=True)
    # mode 1: the confirmed tokens come back as the next block, so the drafted slots are discarded
    acc = eng.accept(out["draft"], x["target"], kv, mode=1)
    return dict(out, accept_len=acc["accept_len"], out_tokens=acc["out_tokens"], kv_len=kv, k_cache=kc, v_cache=vc)


# ---------------------------------------------------------------------------------------- what it cannot do without
def work(case):
    if case["kind"] == "build":
        return {"bytes": 4.0 * case["tokens"] + 4 * case["vocab"] + 4 * case["rows"], "flops": float(case["tokens"])}
    s = SHAPES[case["shape"]]
    params = synth.head_param_count(s)
    d, V = s.d_model, s.vocab_size
    if case["kind"] == "train":
        n, K = case["positions"], case["steps"]
        flops = K * (2.0 * n * (params + V * d) + 2.0 * n * n * s.q_dim)
        return {"bytes": K * 2.0 * (params + V * d) + 4.0 * n * V + 2 * n * d, "flops": flops}
    B, m, K = case["batch"], case.get("block", 1), case.get("steps", 1)
    ctx = 0.5 * (case["ctx_lo"] + case["ctx_hi"])  # contexts are uniform in the range
    kv_token = 4.0 * s.kv_dim                      # key and value of a token, bf16
    sizes = [n or V for n in _lists(case)]
    head = float(sum(sizes))                       # rows of the output head that some sequence uses
    per_row = head / len(sizes)                    # logits of one row
    live = 0.5 * (m + 1) if B > 1 and m > 1 else m  # positions of a block that exist
    # A step needs the result of the step before, and the weights of one step are larger than the chip's caches: they
    # are read once per step.
    steps = [(B * live, ctx + live)] if m > 1 else []
    if case["kind"] != "extend":
        steps += [(B, ctx + (live if m > 1 else 0) + k) for k in range(len(steps), K)]
    byts = flops = 0.0
    for rows, length in steps:
        byts += 2.0 * (params + head * d) + B * length * kv_token + rows * (4 * per_row + 6 * d)
        flops += 2.0 * rows * (params + per_row * d) + 4.0 * rows * length * s.q_dim
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "build":
        return "exact"
    # Sums in another order move hidden states and logits by about 1e-5 (activations are carried to 16 bits of mantissa,
    # sums are 32-bit), and with them a few new cache entries to the neighbouring bf16 value, 2^-8 away.  From an empty
    # cache (a prompt, the training forward) such entries are all that a position attends: 6e-5 on the logits against
    # 64 bits, 4e-4 after the recursion of the training forward.
    rel = {"train": 2e-3, "extend": 1e-3}.get(case["kind"], 2e-4)
    return {"rel": rel, "max": 2e-2 if rel < 2e-3 else 5e-2, "differ": 0.01}


# ----------------------------------------------------------------------------------------------- in 64 bits
def _norm(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x [..., hd] at positions pos (broadcast over the leading dimensions but the first)."""
    hd = x.shape[-1]
    inv = theta ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=x.device) / hd)
    a = pos.double()[:, None, None] * inv
    c, sn = torch.cos(a), torch.sin(a)
    lo, hi = x[..., : hd // 2], x[..., hd // 2:]
    return torch.cat([lo * c - hi * sn, hi * c + lo * sn], dim=-1)


def _lin(x, w):
    return x @ w.double().t()


class _Exact:
    """The head in 64 bits; only cache entries are rounded to bf16, as the interface says."""

    def __init__(self, s, w, caches):
        self.s, self.w = s, w
        self.kc, self.vc = caches                       # bf16, read by the attention
        self.new = []                                   # (sequence, slot, key, value) before rounding

    def step(self, h, token, seq, pos):
        """One application: rows r with hidden h[r], token[r], sequence seq[r] and cache slot pos[r] (host arrays)."""
        s, w = self.s, self.w
        p = torch.as_tensor(np.asarray(pos), device=DEVICE)
        c = torch.cat([_norm(h, w["g_hnorm"], s.rms_eps),
                       _norm(w["embed"][token.long()].double(), w["g_enorm"], s.rms_eps)], dim=-1)
        x = _lin(c, w["w_proj"])
        y = _norm(x, w["g_attn_norm"], s.rms_eps)
        n = x.shape[0]
        q = (_lin(y, w["w_q"]) + w["b_q"].double()).view(n, s.n_q_heads, s.head_dim)
        k = (_lin(y, w["w_k"]) + w["b_k"].double()).view(n, s.n_kv_heads, s.head_dim)
        v = (_lin(y, w["w_v"]) + w["b_v"].double()).view(n, s.n_kv_heads, s.head_dim)
        q, k = _rope(q, p, s.rope_theta), _rope(k, p, s.rope_theta)
        seq_t = torch.as_tensor(np.asarray(seq), device=DEVICE)
        self.kc[seq_t, :, p] = k.to(torch.bfloat16)
        self.vc[seq_t, :, p] = v.to(torch.bfloat16)
        self.new.append((seq_t, p, k, v))
        att = torch.empty(n, s.q_dim, dtype=torch.float64, device=DEVICE)
        G = s.n_q_heads // s.n_kv_heads
        for b in sorted(set(int(i) for i in seq)):
            rows = [r for r in range(n) if int(seq[r]) == b]
            top = max(int(pos[r]) for r in rows) + 1
            kb, vb = self.kc[b, :, :top].double(), self.vc[b, :, :top].double()
            lens = torch.as_tensor([int(pos[r]) + 1 for r in rows], device=DEVICE)
            dead = torch.arange(top, device=DEVICE)[None, :] >= lens[:, None]
            for kh in range(s.n_kv_heads):
                qq = q[rows][:, kh * G:(kh + 1) * G].reshape(-1, s.head_dim)
                sc = (qq @ kb[kh].t().contiguous()) / math.sqrt(s.head_dim)
                sc = sc.view(len(rows), G, top).masked_fill(dead[:, None], -math.inf)
                o = torch.softmax(sc, -1).view(-1, top) @ vb[kh]
                att[torch.as_tensor(rows, device=DEVICE), kh * G * s.head_dim:(kh + 1) * G * s.head_dim] = \
                    o.view(len(rows), -1)
        x1 = x + _lin(att, w["w_o"])
        y2 = _norm(x1, w["g_mlp_norm"], s.rms_eps)
        x2 = x1 + _lin(torch.nn.functional.silu(_lin(y2, w["w_gate"])) * _lin(y2, w["w_up"]), w["w_down"])
        return _norm(x2, w["g_final_norm"], s.rms_eps)

    def logits(self, hh, ids):
        return _lin(hh, self.w["lm_head"] if ids is None else self.w["lm_head"][ids.long()])

    def caches(self, k_cache, v_cache):
        """The caches after the call with the new entries unrounded; None where that would take too much memory."""
        if k_cache.numel() > 1 << 28:
            return None, None
        kx, vx = k_cache.double(), v_cache.double()
        for seq, p, k, v in self.new:
            kx[seq, :, p], vx[seq, :, p] = k, v
        return kx, vx


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        return None
    s, x = SHAPES[case["shape"]], _inputs(case, seed)
    w = x["w"]
    if kind == "train":
        n, K = case["positions"], case["steps"]
        h, ces, z = x["hidden"].double(), [], None
        for k in range(1, K + 1):
            shape = (1, s.n_kv_heads, n, s.head_dim)
            e = _Exact(s, w, [torch.zeros(shape, dtype=torch.bfloat16, device=DEVICE) for _ in range(2)])
            h = e.step(h, x["tokens"][k:k + n], [0] * n, range(n))
            z = e.logits(h, None)
            ces.append(torch.nn.functional.cross_entropy(z, x["tokens"][k + 1:k + 1 + n].long()))
        a = torch.tensor([0.6 ** k for k in range(K)], dtype=torch.float64, device=DEVICE)
        ce = torch.stack(ces)
        return {"loss": torch.cat([ce, ((a * ce).sum() / a.sum())[None]]), "logits": z}
    B, K, m = case["batch"], case.get("steps", 1), case.get("block", 0)
    ids = [torch.from_numpy(i).to(DEVICE) for i in x["lists"]]
    e = _Exact(s, w, (x["k_cache"].clone(), x["v_cache"].clone()))
    ctx, out = x["ctx"].astype(np.int64), {}
    h = tok = None
    if m:
        lens = x["ext_len"].cpu().numpy()
        rows = [(j, b) for j in range(m) for b in range(B) if j < lens[b]]
        at = torch.as_tensor([j * B + b for j, b in rows], device=DEVICE)
        hh = e.step(x["hidden"].view(m * B, -1)[at].double(), x["token"].view(-1)[at], [b for _, b in rows],
                    [int(ctx[b]) + j for j, b in rows])
        z = e.logits(hh, ids[0] if ids else None)
        hidden = torch.zeros(m * B, s.d_model, dtype=torch.float64, device=DEVICE)
        logits = torch.zeros(m * B, z.shape[1], dtype=torch.float64, device=DEVICE)
        hidden[at], logits[at] = hh, z
        hidden, logits = hidden.view(m, B, -1), logits.view(m, B, -1)
        pre = "block_" if kind == "cycle" else ""
        out[pre + "hidden"], out[pre + "logits"] = hidden, logits
        if kind == "cycle":
            h = hidden[-1]
            best = logits[-1].argmax(-1)
            tok = ids[0][best] if ids else best
            ctx, K = ctx + m, K - 1
    if kind != "extend":
        if h is None:
            h, tok = x["hidden"].double(), x["token"]
        groups = [[b for b in range(B) if x["seq_list"][b] == i] for i in range(3)] if kind == "lists" else [list(range(B))]
        n_max = max(len(ids[i]) if ids else s.vocab_size for i, g in enumerate(groups) if g)
        logits = torch.zeros(B, K, n_max, dtype=torch.float64, device=DEVICE)
        hidden = torch.zeros(B, K, s.d_model, dtype=torch.float64, device=DEVICE)
        for k in range(K):
            h = e.step(h, tok, list(range(B)), [int(c) + k for c in ctx])
            hidden[:, k] = h
            tok = torch.zeros(B, dtype=torch.int32, device=DEVICE)
            for i, g in enumerate(groups):
                if not g:
                    continue
                at = torch.as_tensor(g, device=DEVICE)
                z = e.logits(h[at], ids[i] if ids else None)
                logits[at, k, : z.shape[1]] = z
                best = z.argmax(-1)
                tok[at] = (ids[i][best] if ids else best).int()
            if "forced" in x and k < K - 1:
                tok = x["forced"][:, k]
        out["hidden"], out["logits"] = hidden, logits
    out["k_cache"], out["v_cache"] = e.caches(x["k_cache"], x["v_cache"])
    return out
