"""The calls that a user of this library makes, as measurable cases.

A case is a plain dict; ``prepare`` builds what a serving program (or a data
pipeline) holds before the call, ``run`` makes ONE pass through the public
entry points (``binding.Engine``, or ``pard_cod_build`` for the training data),
``exact`` computes the same logits in float64 with plain torch.

Kinds
  prefill   a prompt into a free slot: both models ingest it, first token
  draft     the granular drafting call: one parallel draft pass
  verify    the granular verification call: one target pass over K + 1 rows
  generate  the fused device loop over one or several slots (draft, verify,
            accept, roll back), greedy or with speculative sampling; K = 0 is
            plain target decoding
  request   prefill, then the fused loop: a whole request
  cod       COD training-data processing of a batch of samples

Models keep the width, heads, feed-forward size and vocabulary family of
``pard_inputs.WORKLOADS``; most cases run a few layers of them over a small
vocabulary, so that a pass is its decode layers (blocks) rather than the copy
of the logits to the host.  Two cases run the full vocabulary, one of them at
full depth.

Weights are seeded normals like the library's other inputs, with tied
embeddings and a spread (``std_t``, ``std_d``) at which a token's own embedding
row keeps a clear lead in its logits (5 to 50 standard deviations of the
others; wider spreads let the layers swamp it).  Greedy choices then have wide
margins, as a trained model's have: the token path of a pass does not hang on
the last bit of a sum, each step accepts its first candidate (two tokens a
step), and rewinding a slot (``kv_truncate``) restores exactly the state the
pass began with.  The margins are below 2 in logit units, so the sampled
cases' temperature is small in proportion.
"""
from __future__ import annotations

import ctypes as C
import math
import random
from dataclasses import replace

import numpy as np
import torch

import pard_inputs as pi
from paper_2504_18583_amd import binding as B

BLOCK_VOCAB = 4096                 # vocabulary of the block cases
RETAIN, RETAIN_MIN = 0.7, 0.2      # COD retention (the library's benchmark setting)


def listed():
    return [
        # The smallest engine call: the tiny pair's loop, where launches and
        # the chain of a step are all there is.
        dict(name="tiny_generate", kind="generate", pair="tiny", lt=2, ld=1, vocab=1024, std_t=0.007, std_d=0.007,
             n_seq=1, lo=32, hi=32, k=4, steps=16, temp=0.0),
        # A host-driven scheduler's drafting call on the whole 1B-shaped draft.
        dict(name="draft_1b", kind="draft", pair="llama8b_1b", lt=1, ld=16, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=1, lo=512, hi=512, k=8, steps=1, temp=0.0),
        # Its verification call: 8B-shaped layers, 9 rows, ordinary context.
        dict(name="verify_8b", kind="verify", pair="llama8b_1b", lt=8, ld=1, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=1, lo=600, hi=600, k=8, steps=1, temp=0.0),
        # The same at a long context (16k keys, chunked attention).
        dict(name="verify_8b_16k", kind="verify", pair="llama8b_1b", lt=4, ld=1, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=1, lo=16384, hi=16384, k=8, steps=1, temp=0.0),
        # Time to first token of an ordinary prompt, an odd length.
        dict(name="prefill_8b_517", kind="prefill", pair="llama8b_1b", lt=8, ld=4, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=1, lo=517, hi=517, k=8, steps=1, temp=0.0),
        # Time to first token of a long document.
        dict(name="prefill_8b_8k", kind="prefill", pair="llama8b_1b", lt=4, ld=2, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=1, lo=8192, hi=8192, k=8, steps=1, temp=0.0),
        # A small server: four conversations stepped together.
        dict(name="batch4_8b", kind="generate", pair="llama8b_1b", lt=8, ld=4, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=4, lo=256, hi=1024, k=8, steps=8, temp=0.0),
        # A loaded server: 32 ragged conversations stepped together.
        dict(name="batch32_8b", kind="generate", pair="llama8b_1b", lt=8, ld=4, vocab=BLOCK_VOCAB, std_t=0.001,
             std_d=0.001, n_seq=32, lo=256, hi=2048, k=8, steps=8, temp=0.0),
        # Speculative sampling, Qwen2.5-shaped pair (QKV bias), the longest K
        # of the paper's sweep, the full vocabulary.
        dict(name="sampled_qwen_k12", kind="generate", pair="qwen7b_05b", lt=4, ld=4, vocab=152064, std_t=0.001,
             std_d=0.002, n_seq=1, lo=1024, hi=1024, k=12, steps=16, temp=0.01),
        # A whole request on the whole 8B/1B pair: prompt in, 64 tokens out.
        dict(name="request_8b_1b", kind="request", pair="llama8b_1b", lt=32, ld=16, vocab=128256, std_t=0.0006,
             std_d=0.001, n_seq=1, lo=512, hi=512, k=8, steps=32, temp=0.0),
        # Training data: a packing worker's small batch with long samples, and
        # a dataset shard at the paper's lengths.
        dict(name="cod_48", kind="cod", samples=48, lo=512, hi=6000, k=8),
        dict(name="cod_4096", kind="cod", samples=4096, lo=256, hi=1024, k=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["prefill", "prefill", "draft", "verify", "verify", "generate", "generate", "generate", "cod",
                       "cod"])
    if kind == "cod":
        if rng.random() < 0.5:
            return dict(kind="cod", samples=_log_int(rng, 8, 4000), lo=rng.randint(20, 300), hi=rng.randint(301, 1024),
                        k=rng.choice([4, 8, 8, 12]))
        return dict(kind="cod", samples=_log_int(rng, 2, 64), lo=rng.randint(300, 2000), hi=rng.randint(2001, 8193),
                    k=rng.choice([4, 8, 8, 12]))
    pair = rng.choice(["llama8b_1b", "llama8b_1b", "qwen7b_05b"])
    c = dict(kind=kind, pair=pair, lt=rng.randint(2, 8), ld=rng.randint(1, 4), vocab=BLOCK_VOCAB,
             std_t=0.001 if pair == "llama8b_1b" else 0.0007, std_d=0.001, n_seq=1, lo=0, hi=0, k=rng.choice([1, 2, 4, 5, 8, 8, 12, 16]),
             steps=1, temp=0.0)
    if kind == "prefill":
        n = _log_int(rng, 9, 8192)
        c.update(lt=rng.randint(2, 4) if n > 2048 else c["lt"], ld=min(c["ld"], 2), lo=n, hi=n)
    elif kind in ("draft", "verify"):
        n = _log_int(rng, 33, 16384)
        c.update(lt=rng.randint(2, 4) if n > 2048 or kind == "draft" else c["lt"], lo=n, hi=n)
        if kind == "draft":
            c.update(ld=rng.randint(4, 16))
    else:
        n_seq = _log_int(rng, 1, 32)
        k = rng.choice([0, 2, 4, 8, 8] if n_seq > 16 else [0, 2, 4, 5, 8, 8, 12])
        lo = _log_int(rng, 20, 900)
        c.update(n_seq=n_seq, k=k, lo=lo, hi=lo + rng.randint(0, 1100), steps=rng.randint(3, 8),
                 temp=0.01 if rng.random() < 0.25 else 0.0)
    return c


# --------------------------------------------------------------------------
# specs, prompts
# --------------------------------------------------------------------------

def _specs(case, seed):
    wl = pi.WORKLOADS[case["pair"]]
    s = seed % (1 << 40)
    t = replace(wl.target, n_layers=case["lt"], vocab=case["vocab"], init_std=case["std_t"], tied=True, seed=s,
                dtype="bf16")
    d = replace(wl.draft, n_layers=case["ld"], vocab=case["vocab"], init_std=case["std_d"], tied=True, seed=s,
                dtype="bf16")
    return t, d


def _prompt_lengths(case):
    """Prompt lengths (part of the case, not of the seed: all seeds are the
    same amount of work)."""
    return [int(n) for n in pi.gen_prompt_lengths(4, case["n_seq"], case["lo"], case["hi"])]


def _prompts(case, seed):
    return [[int(x) for x in pi.gen_prompt(seed % (1 << 40), case["vocab"], n, b)]
            for b, n in enumerate(_prompt_lengths(case))]


def _cod_lengths(case):
    """The shard's sample lengths (part of the case, too)."""
    return pi.gen_prompt_lengths(case["samples"], case["samples"], case["lo"], case["hi"]).astype(np.int64)


def _tokens_per_step(case):
    return 2 if case["k"] > 0 else 1   # the first candidate is accepted, the second is not


# --------------------------------------------------------------------------
# prepare / run
# --------------------------------------------------------------------------

def _prepare_cod(case, seed):
    lens = _cod_lengths(case)
    offs = np.zeros(len(lens) + 1, np.int64)
    offs[1:] = np.cumsum(lens)
    vocab = pi.WORKLOADS["llama8b_1b"].target.vocab
    tokens = torch.from_numpy(pi.gen_prompt(seed % (1 << 40), vocab, int(offs[-1]))).cuda()
    i64p = C.POINTER(C.c_int64)
    out_offs = np.zeros(len(offs), np.int64)
    n = len(lens)
    total = B.lib.pard_cod_layout(offs.ctypes.data_as(i64p), n, case["k"], RETAIN, RETAIN_MIN,
                                  out_offs.ctypes.data_as(i64p))
    out = {name: torch.zeros(total, dtype=torch.int32, device="cuda")
           for name in ("ids", "labels", "pos", "section", "column")}
    out["len"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    ws_bytes = int(B.lib.pard_cod_workspace_bytes(n))
    ws = torch.empty(ws_bytes + 256, dtype=torch.uint8, device="cuda")
    args = (C.c_void_p(tokens.data_ptr()), offs.ctypes.data_as(i64p), n, case["k"], RETAIN, RETAIN_MIN, vocab - 1,
            seed % (1 << 40), out_offs.ctypes.data_as(i64p),
            *[C.c_void_p(out[name].data_ptr()) for name in ("ids", "labels", "pos", "section", "column", "len")],
            C.c_void_p(ws.data_ptr() + (-ws.data_ptr()) % 256), ws_bytes, None,
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    return dict(case=case, out=out, args=args, keep=(tokens, offs, out_offs, ws))


def prepare(case, seed):
    if case["kind"] == "cod":
        return _prepare_cod(case, seed)
    t, d = _specs(case, seed)
    prompts = _prompts(case, seed)
    k, steps = case["k"], case["steps"]
    longest = max(len(p) for p in prompts)
    max_k = max(k, 1)
    eng = B.Engine(t, d, case["vocab"] - 1, max_ctx=longest + (steps + 2) * (max_k + 1) + 2 * max_k + 16, max_k=max_k,
                   max_batch=case["n_seq"])
    s = dict(case=case, eng=eng, prompts=prompts, slots=list(range(case["n_seq"])))
    if case["kind"] in ("draft", "verify", "generate"):
        firsts = [eng.prefill(p, seq=i) for i, p in enumerate(prompts)]
        s["prefix"] = prompts[0] + [firsts[0]]
        s["cand"] = [int(x) for x in pi.gen_prompt((seed + 1) % (1 << 40), case["vocab"], max_k, 99)]
        if case["temp"] > 0.0:
            eng.set_sampling(case["temp"], seed % (1 << 40))
    return s


def _steps(case):
    """Arguments of the loop: enough tokens that max_steps ends it."""
    return case["steps"] * (case["k"] + 1) + 2, case["steps"]


def run(s):
    case = s["case"]
    kind, k = case["kind"], case["k"]
    if kind == "cod":
        rc = B.lib.pard_cod_build(*s["args"])
        if rc != B.PARD_OK:
            raise RuntimeError(f"pard_cod_build: {rc}")
        return s["out"]
    eng, prompts = s["eng"], s["prompts"]
    if kind == "prefill":
        first = eng.prefill(prompts[0])
        return {"first": first, "logits": eng.read_logits(B.PARD_TARGET, 1)}
    if kind == "draft":
        cand = eng.draft(s["prefix"], k)
        return {"cand": np.asarray(cand), "logits": eng.read_logits(B.PARD_DRAFT, k)}
    if kind == "verify":
        eng.kv_truncate(B.PARD_TARGET, len(prompts[0]))
        a, bonus = eng.verify(s["cand"][:k])
        return {"a": a, "bonus": bonus, "logits": eng.read_logits(B.PARD_TARGET, k + 1)}
    if kind == "request":
        eng.prefill(prompts[0])
    else:                                  # generate: back to the prompt's end
        for i, p in zip(s["slots"], prompts):
            eng.kv_truncate(B.PARD_TARGET, len(p), seq=i)
            eng.kv_truncate(B.PARD_DRAFT, len(p), seq=i)
    n_tokens, max_steps = _steps(case)
    tokens, _ = eng.generate_batch(s["slots"], k, n_tokens, max_steps=max_steps)
    return {"tokens": [np.asarray(t) for t in tokens] if len(tokens) <= 24 else np.asarray(tokens),
            "logits": [eng.read_logits(B.PARD_TARGET, k + 1, seq=i) for i in s["slots"]]}


# --------------------------------------------------------------------------
# work
# --------------------------------------------------------------------------

def _layer_params(s):
    return s.d_model * (2 * s.q_dim + 2 * s.kv_dim) + 3 * s.d_model * s.ffn_dim


def _pass_work(s, seqs, lm_rows):
    """(bytes, flops) of one pass: seqs = (committed length, rows) per sequence."""
    rows = sum(r for _, r in seqs)
    weights = s.n_layers * _layer_params(s) + (s.vocab * s.d_model if lm_rows else 0)
    kv = 2 * s.n_layers * s.kv_dim * 2
    n_bytes = 2 * weights + sum(kv * (l + 2 * r) for l, r in seqs) + rows * s.d_model * 2 + lm_rows * s.vocab * 4
    pairs = sum(r * l + r * (r + 1) / 2 for l, r in seqs)
    flops = 2 * rows * s.n_layers * _layer_params(s) + 2 * lm_rows * s.vocab * s.d_model
    return n_bytes, flops + 4 * pairs * s.n_layers * s.q_dim


def _add(works):
    works = list(works)
    return {"bytes": float(sum(w[0] for w in works)), "flops": float(sum(w[1] for w in works))}


def work(case):
    if case["kind"] == "cod":
        cols = _cod_lengths(case) - 1
        packed, gamma = int(cols.sum()), 1.0
        for _ in range(2, case["k"] + 1):
            gamma *= RETAIN
            packed += int(np.floor(cols * max(gamma, RETAIN_MIN) + 0.5).sum())
        return {"bytes": 4.0 * int((cols + 1).sum()) + 20.0 * packed + 4.0 * len(cols), "flops": 0.0}
    t, d = _specs(case, 0)
    kind, k = case["kind"], case["k"]
    lens = _prompt_lengths(case)
    n = lens[0]
    if kind == "prefill":
        return _add([_pass_work(t, [(0, n)], 1), _pass_work(d, [(0, n)], 0)])
    if kind == "draft":
        return _add([_pass_work(d, [(n, k)], k)])
    if kind == "verify":
        return _add([_pass_work(t, [(n, k + 1)], k + 1)])
    works = [_pass_work(t, [(0, n)], 1), _pass_work(d, [(0, n)], 0)] if kind == "request" else []
    m = case["n_seq"]
    for i in range(case["steps"]):
        at = [n + i * _tokens_per_step(case) for n in lens]
        if k > 0:
            works.append(_pass_work(d, [(l, k + (1 if i else 0)) for l in at], m * k))
        works.append(_pass_work(t, [(l, k + 1) for l in at], m * (k + 1)))
    return _add(works)


def tolerance(case):
    if case["kind"] == "cod":
        return "exact"
    # fp16 activations (2^-11 per rounding, several per layer), fp32 sums: the
    # cases are 1.5e-4 to 5.3e-4 (largest 2.3e-3) off float64
    return {"rel": 2e-3, "max": 1e-2}


# --------------------------------------------------------------------------
# exact: the decoder in float64, plain torch
# --------------------------------------------------------------------------

_M1, _M2, _G = 0xBF58476D1CE4E5B9, 0x94D049BB133111EB, 0x9E3779B97F4A7C15


def _i64(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _shr(z, n):
    return (z >> n) & ((1 << (64 - n)) - 1)


def _mix(z):
    z = (z ^ _shr(z, 30)) * _i64(_M1)
    z = (z ^ _shr(z, 27)) * _i64(_M2)
    return z ^ _shr(z, 31)


def _mix_int(z):
    z &= (1 << 64) - 1
    z = ((z ^ (z >> 30)) * _M1) & ((1 << 64) - 1)
    z = ((z ^ (z >> 27)) * _M2) & ((1 << 64) - 1)
    return z ^ (z >> 31)


def _tensor(spec, ordinal, shape):
    """One weight tensor of the published generator (SplitMix64, Box-Muller,
    rounded to bf16), as float64 on the GPU."""
    key = _mix_int((spec.seed << 20) + (spec.stream << 16) + ordinal)
    n = int(np.prod(shape))
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    step = 1 << 25
    for a in range(0, n, step):
        m = min(step, n - a)
        i = torch.arange(a // 2, (a + m + 1) // 2, dtype=torch.int64, device="cuda")
        z0 = _mix((2 * i + 1) * _i64(_G) + _i64(key))
        z1 = _mix((2 * i + 2) * _i64(_G) + _i64(key))
        r = torch.sqrt(-2.0 * torch.log((_shr(z0, 11) + 1).double() * 2.0 ** -53))
        th = _shr(z1, 11).double() * (2.0 ** -53 * 2.0 * math.pi)
        v = torch.stack([r * torch.cos(th), r * torch.sin(th)], 1).reshape(-1)[:m] * spec.init_std
        out[a:a + m] = v.float().bfloat16().double()
    return out.reshape(shape)


def _rms(x, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps)


def _rotate(x, spec):
    """Rotary embedding of [n, heads, hd], rotate-half pairs, positions 0..n-1."""
    half = spec.head_dim // 2
    w = spec.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / spec.head_dim)
    a = torch.arange(x.shape[0], dtype=torch.float64, device="cuda")[:, None] * w
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _attend(q, k, v):
    """Causal grouped attention of the last rows of q's sequence: q [r, H, hd]
    are positions n - r .. n - 1 of k, v [n, Hkv, hd]."""
    n, r = k.shape[0], q.shape[0]
    group = q.shape[1] // k.shape[1]
    kt = k.permute(1, 2, 0).contiguous()
    vt = v.permute(1, 0, 2).contiguous()
    pos = torch.arange(n, device="cuda")
    out = torch.empty_like(q)
    for a in range(0, r, 256):
        b = min(r, a + 256)
        qq = q[a:b].permute(1, 0, 2).reshape(k.shape[1], group * (b - a), -1).contiguous()
        sc = torch.matmul(qq, kt).reshape(q.shape[1], b - a, n) / math.sqrt(q.shape[2])
        sc.masked_fill_(pos[None, None, :] > (pos[n - r + a:n - r + b])[None, :, None], -math.inf)
        p = torch.softmax(sc, -1).reshape(k.shape[1], group * (b - a), n)
        out[a:b] = torch.matmul(p, vt).reshape(q.shape[1], b - a, -1).permute(1, 0, 2)
    return out


def _logits64(spec, seqs, rows):
    """Float64 logits of the last `rows` positions of each token sequence."""
    embed = _tensor(spec, 0, (spec.vocab, spec.d_model))
    lens = [len(s) for s in seqs]
    x = embed[torch.tensor([t for s in seqs for t in s], device="cuda")]
    cuts = np.concatenate([[0], np.cumsum(lens)])
    d, q_dim, kv, f = spec.d_model, spec.q_dim, spec.kv_dim, spec.ffn_dim
    for l in range(spec.n_layers):
        w = lambda j, *shape: _tensor(spec, 16 * (l + 1) + j, shape)  # noqa: E731
        h = _rms(x, spec.rms_eps)
        q, k, v = (torch.matmul(h, w(j, m, d).T) for j, m in ((0, q_dim), (1, kv), (2, kv)))
        if spec.qkv_bias:
            q, k, v = q + w(7, q_dim), k + w(8, kv), v + w(9, kv)
        att = torch.empty_like(q)
        for a, b in zip(cuts[:-1], cuts[1:]):
            qs, ks, vs = (z[a:b].reshape(b - a, -1, spec.head_dim) for z in (q, k, v))
            att[a:b] = _attend(_rotate(qs, spec), _rotate(ks, spec), vs).reshape(b - a, -1)
        x = x + torch.matmul(att, w(3, d, q_dim).T)
        del q, k, v, att
        h = _rms(x, spec.rms_eps)
        g = torch.matmul(h, w(4, f, d).T)
        u = torch.matmul(h, w(5, f, d).T)
        x = x + torch.matmul(torch.nn.functional.silu(g) * u, w(6, d, f).T)
        del g, u
    return [torch.matmul(_rms(x[b - rows:b], spec.rms_eps), embed.T).cpu().numpy() for b in cuts[1:]]


def exact(case, seed):
    """The logits that `run` returns, in float64 (tokens have no 64-bit form).

    The token path is the one that the weights' wide margins fix: the target
    and the draft repeat the last token, mask rows propose the mask token."""
    if case["kind"] == "cod":
        return None
    t, d = _specs(case, seed)
    prompts = _prompts(case, seed)
    kind, k, mask = case["kind"], case["k"], case["vocab"] - 1
    if kind == "prefill":
        return {"first": None, "logits": _logits64(t, prompts[:1], 1)[0]}
    if kind == "draft":
        return {"cand": None, "logits": _logits64(d, [prompts[0] + [prompts[0][-1]] + [mask] * (k - 1)], k)[0]}
    if kind == "verify":
        cand = [int(x) for x in pi.gen_prompt((seed + 1) % (1 << 40), case["vocab"], max(k, 1), 99)][:k]
        return {"a": None, "bonus": None, "logits": _logits64(t, [prompts[0] + [prompts[0][-1]] + cand], k + 1)[0]}
    # the last step's verify rows: [p, p, m, ..., m] after the tokens before it
    done = (case["steps"] - 1) * _tokens_per_step(case)
    seqs = [p + [p[-1]] * done + ([p[-1]] + ([p[-1]] + [mask] * (k - 1) if k else [])) for p in prompts]
    tokens = None if len(prompts) > 24 else [None] * len(prompts)
    return {"tokens": tokens, "logits": _logits64(t, seqs, k + 1)}
