"""GPU parity of multi-sequence passes (the batch-32 workload's regime).

* 32 independent slots with ragged prompt lengths (uniform in [256, 2048], as
  the batch-32 workload draws them), each with its own acceptance and KV
  rollback: stepped one slot at a time (granular calls), and stepped together
  by the fused loop, whose draft and verify passes then hold every slot's
  rows (256-512 and 288 rows at K = 8: the row-block GEMM, split inputs,
  per-sequence attention, tails and next-pass staging).  Each slot is checked
  against its own oracle run every step.
* The same at the full width of the 8B/1B-shaped pair (2 / 1 layers), with
  shorter ragged prompts so that the fp64 oracle keeps up.
* Small batches (skinny GEMMs with several sequences), plain target steps
  (K = 0) over many slots, and whole fused generations against the target's
  greedy decoding (lossless, Sec. 2.1 eq. 2)."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
import pard_inputs as pi
from gpu_common import MARGIN, BatchLockstep, Lockstep, margins, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    require_gpu()
    from paper_2504_18583_amd import binding
    return binding


def _tiny():
    wl = pi.WORKLOADS["tiny"]
    return wl, pi.with_dtype(wl.target, "bf16"), pi.with_dtype(wl.draft, "bf16")


def _ragged_prompts(seed, batch, lo, hi, vocab):
    lens = pi.gen_prompt_lengths(seed, batch, lo, hi)
    return [[int(x) for x in pi.gen_prompt(seed, vocab, int(n), b)] for b, n in enumerate(lens)]


@pytest.fixture(scope="module")
def tiny_models():
    wl, t_spec, d_spec = _tiny()
    return oracle.build_model(t_spec), oracle.build_model(d_spec)


def test_32_ragged_slots_interleaved_lockstep(B, tiny_models):
    wl, t_spec, d_spec = _tiny()
    bw = pi.WORKLOADS["llama8b_1b_batch32"]
    lo, hi = bw.prompt_len_range
    prompts = _ragged_prompts(bw.seed, bw.batch, lo, hi, t_spec.vocab)
    target, draft = tiny_models
    k = bw.k
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=hi + 64, max_k=k, max_batch=bw.batch)
    try:
        slots = [Lockstep(eng, target, draft, p, k, wl.mask_id, seq=b, tag=f"slot {b} (L={len(p)})")
                 for b, p in enumerate(prompts)]
        for b, ls in enumerate(slots):
            if b % 8 == 0:
                say(f"[gpu] batch: prefill slots {b}..{b + 7}")
            ls.prefill()
        for step in range(2):
            say(f"[gpu] batch: step {step} over {len(slots)} slots, one at a time")
            for ls in slots:
                ls.step()
        say(f"    max |logit err| {max(ls.worst for ls in slots):.3g}")
        for b, ls in enumerate(slots):
            assert eng.kv_len(B.PARD_TARGET, seq=b) == ls.cache_t.length
            assert eng.kv_len(B.PARD_DRAFT, seq=b) == ls.cache_d.length
    finally:
        eng.close()


def test_32_ragged_slots_batched_passes_lockstep(B, tiny_models):
    wl, t_spec, d_spec = _tiny()
    bw = pi.WORKLOADS["llama8b_1b_batch32"]
    lo, hi = bw.prompt_len_range
    prompts = _ragged_prompts(bw.seed, bw.batch, lo, hi, t_spec.vocab)
    target, draft = tiny_models
    k = bw.k
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=hi + 128, max_k=k, max_batch=bw.batch)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, k, wl.mask_id, tag="batched")
        say("[gpu] batched passes: prefill 32 slots")
        bl.prefill()
        for step in range(3):
            say(f"[gpu] batched passes: fused step {step} ({len(prompts) * (k + 1)} verify rows)")
            bl.step(n_tokens=64)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()


@pytest.mark.parametrize("n_slots,k", [(3, 4), (5, 6)])
def test_small_batches_skinny_path_lockstep(B, tiny_models, n_slots, k):
    wl, t_spec, d_spec = _tiny()
    prompts = _ragged_prompts(11 + n_slots, n_slots, 20, 90, t_spec.vocab)
    target, draft = tiny_models
    # non-contiguous slots, listed out of order
    slots = [2 * i + 1 for i in range(n_slots)][::-1]
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=256, max_k=k, max_batch=2 * n_slots + 2)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, k, wl.mask_id, slots=slots, tag=f"{n_slots} slots")
        bl.prefill()
        for step in range(3):
            say(f"[gpu] {n_slots} slots, K={k}: fused step {step}")
            bl.step(n_tokens=40)
    finally:
        eng.close()


def test_plain_target_steps_over_40_slots(B, tiny_models):
    wl, t_spec, d_spec = _tiny()
    prompts = _ragged_prompts(21, 40, 8, 70, t_spec.vocab)
    target, draft = tiny_models
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=160, max_k=4, max_batch=40)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, 0, wl.mask_id, tag="K=0")
        bl.prefill()
        for step in range(3):
            say(f"[gpu] 40 slots, K=0: fused step {step}")
            bl.step(n_tokens=16)
    finally:
        eng.close()


def test_batched_generation_equals_greedy_decoding(B, tiny_models):
    """Greedy PARD is lossless: every slot's output equals the target's own
    greedy continuation, up to the first near-tie of the oracle."""
    wl, t_spec, d_spec = _tiny()
    prompts = _ragged_prompts(31, 24, 12, 60, t_spec.vocab)
    target, draft = tiny_models
    n_tokens, k = 24, wl.k
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=128, max_k=k, max_batch=24)
    try:
        firsts = [eng.prefill(p, seq=b) for b, p in enumerate(prompts)]
        say("[gpu] 24 slots: one fused batched generation")
        res, stats = eng.generate_batch(list(range(24)), k, n_tokens)
        assert stats.tokens == 24 * n_tokens
        for b, p in enumerate(prompts):
            toks = res[b]
            assert len(toks) == n_tokens and toks[0] == firsts[b]
            ref = oracle.greedy_ar(target, p, n_tokens)
            # compare up to the first position whose oracle margin is small
            cache = oracle.KVCache(target)
            lg = oracle.forward_cached(target, cache, p, logits_rows=[len(p) - 1])
            for i in range(n_tokens):
                if margins(lg)[-1] <= MARGIN:
                    break
                assert toks[i] == ref[i], f"slot {b} token {i}: gpu {toks[i]} oracle {ref[i]}"
                lg = oracle.forward_cached(target, cache, [ref[i]])
            assert eng.kv_len(B.PARD_TARGET, seq=b) >= len(p) + n_tokens - 1
    finally:
        eng.close()


@pytest.mark.timeout(900)
def test_llama_8b_1b_full_width_slice_32_slots_batched(B):
    wl = pi.WORKLOADS["llama8b_1b_batch32"]
    t_spec = replace(pi.with_dtype(wl.target, "bf16"), n_layers=2)
    d_spec = replace(pi.with_dtype(wl.draft, "bf16"), n_layers=1)
    # ragged, but short enough for the fp64 oracle's prefill at full width
    prompts = _ragged_prompts(wl.seed, wl.batch, 16, 80, t_spec.vocab)
    say("[gpu] 8B/1B full-width slice, 32 slots: oracle build")
    target, draft = oracle.build_model(t_spec), oracle.build_model(d_spec)
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=160, max_k=wl.k, max_batch=wl.batch)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, wl.k, wl.mask_id, tag="8B/1B x32")
        say("[gpu] 8B/1B full-width slice, 32 slots: prefill")
        bl.prefill()
        for step in range(2):
            say(f"[gpu] 8B/1B full-width slice, 32 slots: fused step {step}")
            bl.step(n_tokens=48)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()


@pytest.mark.parametrize("pair,n_slots", [("llama8b_1b", 2), ("llama8b_1b", 4), ("llama8b_1b", 7), ("qwen7b_05b", 3)])
def test_full_width_small_batches_lockstep(B, pair, n_slots):
    """18 to 63 rows (two to four row tiles) at full widths: the wide gate/up,
    split down and lm_head tiles of passes of 17 to 64 rows."""
    wl = pi.WORKLOADS[pair]
    vocab, k = 36864, 8
    t_spec = replace(pi.with_dtype(wl.target, "bf16"), n_layers=1, vocab=vocab)
    d_spec = replace(pi.with_dtype(wl.draft, "bf16"), n_layers=1, vocab=vocab)
    prompts = _ragged_prompts(41, n_slots, 8, 40, vocab)
    say(f"[gpu] {pair} widths, {n_slots} slots: oracle build")
    target, draft = oracle.build_model(t_spec), oracle.build_model(d_spec)
    eng = B.Engine(t_spec, d_spec, vocab - 1, max_ctx=96, max_k=k, max_batch=n_slots)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, k, vocab - 1, tag=f"{pair} x{n_slots}")
        bl.prefill()
        for step in range(2):
            bl.step(n_tokens=40)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()


@pytest.mark.parametrize("heads,kv,hd,n_slots,lo,hi", [
    (32, 8, 128, 32, 200, 700),      # whole contexts, three query tiles, four wavefronts
    (32, 8, 64, 20, 100, 600),       # whole contexts, eight wavefronts
    (16, 4, 128, 16, 900, 1500),     # key chunks of 384 and their merge; slots that end chunks early
    (28, 4, 64, 12, 900, 1500),      # two query groups of four and less tiles
    (8, 4, 128, 24, 300, 900),       # two query tiles
])
def test_batched_attention_chunks_lockstep(B, heads, kv, hd, n_slots, lo, hi):
    """Batched decode attention over key chunks longer than 256 keys: ragged
    contexts that end inside a tile, a wavefront's share and a chunk."""
    wl, t_spec, d_spec = _tiny()
    t_spec = replace(t_spec, n_layers=1, n_heads=heads, n_kv_heads=kv, head_dim=hd)
    d_spec = replace(d_spec, n_layers=1, n_heads=heads, n_kv_heads=kv, head_dim=hd)
    prompts = _ragged_prompts(51, n_slots, lo, hi, t_spec.vocab)
    target, draft = oracle.build_model(t_spec), oracle.build_model(d_spec)
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=hi + 96, max_k=8, max_batch=n_slots)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, 8, wl.mask_id, tag=f"{heads}/{kv}x{hd}")
        bl.prefill()
        for step in range(2):
            say(f"[gpu] batched attention {heads}/{kv} heads of {hd}, {n_slots} slots: step {step}")
            bl.step(n_tokens=40)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()


@pytest.mark.parametrize("heads,kv,hd", [
    (32, 32, 128),    # 768 QKV strips: four per workgroup at one row tile
    (64, 8, 128),     # 640
    (40, 40, 64),     # 480: two
    (33, 33, 128),    # 792
    (43, 43, 64),     # 516, the narrowest that takes four
    (48, 48, 128),    # 1152: two, beyond one round of four
])
@pytest.mark.parametrize("n_slots", [1, 3])
def test_wide_qkv_weights_lockstep(B, heads, kv, hd, n_slots):
    """QKV weights wider than 512 strips (many-headed models): one and two row
    tiles, and a prompt of up to 16 tokens through the skinny GEMM."""
    wl, t_spec, d_spec = _tiny()
    t_spec = replace(t_spec, n_layers=1, n_heads=heads, n_kv_heads=kv, head_dim=hd)
    d_spec = replace(d_spec, n_layers=1, n_heads=heads, n_kv_heads=kv, head_dim=hd)
    prompts = _ragged_prompts(71, n_slots, 5, 16, t_spec.vocab)
    target, draft = oracle.build_model(t_spec), oracle.build_model(d_spec)
    eng = B.Engine(t_spec, d_spec, wl.mask_id, max_ctx=96, max_k=8, max_batch=n_slots)
    try:
        bl = BatchLockstep(eng, target, draft, prompts, 8, wl.mask_id, tag=f"{heads}/{kv}x{hd} x{n_slots}")
        bl.prefill()
        for step in range(2):
            say(f"[gpu] wide QKV {heads}/{kv} heads of {hd}, {n_slots} slots: step {step}")
            bl.step(n_tokens=40)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()


@pytest.mark.parametrize("pair", ["llama8b_1b", "qwen7b_05b"])
def test_rows_do_not_depend_on_the_pass(B, pair):
    """Up to 64 rows a row's sums have one order whatever the pass holds beside
    it: full-width layers give a slot bitwise the same logits stepped alone (one
    row tile, the one-launch layer) and with 2, 4 or 7 slots (two to four row
    tiles; draft passes hold up to 2 K rows a slot), and the first rows of a verify
    pass of 8 candidates are those of one of 24."""
    wl = pi.WORKLOADS[pair]
    vocab = 36864
    t_spec = replace(pi.with_dtype(wl.target, "bf16"), n_layers=2, vocab=vocab)
    d_spec = replace(pi.with_dtype(wl.draft, "bf16"), n_layers=2, vocab=vocab)
    prompts = _ragged_prompts(81, 7, 8, 60, vocab)

    def logits(eng, s, k):
        return eng.read_logits(B.PARD_DRAFT, k, seq=s), eng.read_logits(B.PARD_TARGET, k + 1, seq=s)

    one, many = (B.Engine(t_spec, d_spec, vocab - 1, max_ctx=160, max_k=24, max_batch=7) for _ in range(2))
    try:
        for n, k in ((2, 8), (4, 8), (7, 4)):
            say(f"[gpu] {pair}: {n} slots together and alone, K={k}")
            for s in range(n):
                assert one.prefill(prompts[s], seq=s) == many.prefill(prompts[s], seq=s)
            for step in range(2):
                toks, _ = many.generate_batch(list(range(n)), k, 40, max_steps=1)
                for s in range(n):
                    alone, _ = one.generate_batch([s], k, 40, max_steps=1)
                    assert list(alone[0]) == list(toks[s]), f"{n} slots, step {step}, slot {s}: tokens"
                    for got, ref, what in zip(logits(many, s, k), logits(one, s, k), ("draft", "verify")):
                        assert np.array_equal(got, ref), f"{n} slots, step {step}, slot {s}: {what} logits"
        cand = [int(x) for x in pi.gen_prompt(82, vocab, 24)]
        one.verify(cand, seq=0)               # the same state in both engines
        many.verify(cand[:8], seq=0)
        assert np.array_equal(one.read_logits(B.PARD_TARGET, 25, seq=0)[:9], many.read_logits(B.PARD_TARGET, 9, seq=0))
    finally:
        one.close()
        many.close()


@pytest.mark.parametrize("d,heads,kv,hd,ffn,vocab", [
    (320, 5, 1, 64, 1000, 1040),       # 20 and 28 strips, an lm_head of 65 (odd)
    (1056, 9, 3, 128, 2740, 4112),     # 66 and 120 strips, 257 of lm_head
    (288, 43, 43, 64, 96, 1024),       # QKV 516 strips, O 86 k-blocks over 18 strips
    (2080, 8, 8, 64, 4096, 2064),      # 130 strips, QKV 96
    (64, 1, 1, 64, 32, 64),            # four strips, one and two k-blocks
])
def test_row_block_widths_lockstep(B, d, heads, kv, hd, ffn, vocab):
    """Row-block GEMMs (prefill chunks and batched passes of more than 64 rows)
    at widths that fill no tile: ragged last column tiles of every epilogue,
    row counts that end inside a row block, split inputs."""
    wl, t_spec, d_spec = _tiny()
    t_spec = replace(t_spec, n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=hd, ffn_dim=ffn, vocab=vocab)
    d_spec = replace(d_spec, n_layers=1, d_model=d, n_heads=heads, n_kv_heads=kv, head_dim=hd, ffn_dim=ffn, vocab=vocab)
    lens = [65, 97, 130, 144, 145, 200, 257, 290, 330]
    prompts = [[int(x) for x in pi.gen_prompt(91, vocab, n, b)] for b, n in enumerate(lens)]
    target, draft = oracle.build_model(t_spec), oracle.build_model(d_spec)
    eng = B.Engine(t_spec, d_spec, vocab - 1, max_ctx=420, max_k=8, max_batch=len(prompts))
    try:
        bl = BatchLockstep(eng, target, draft, prompts, 8, vocab - 1, tag=f"d{d} {heads}/{kv}x{hd} f{ffn} v{vocab}")
        bl.prefill()
        for step in range(2):
            say(f"[gpu] row-block widths d{d} {heads}/{kv}x{hd} ffn {ffn} vocab {vocab}: step {step}")
            bl.step(n_tokens=40)
        say(f"    max |logit err| {bl.worst:.3g}")
    finally:
        eng.close()
