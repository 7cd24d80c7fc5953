"""Products over many rows.  Prefill: a sequence that is prefilled whole must stand exactly where the same
sequence stands after it was decoded token by token (other kernels, the same additions in the same
order), so the next iteration's logits of both models are equal bit for bit.  Several sequences: each must
get the logits and tokens that it gets alone."""
import numpy as np
import pytest
import torch

from oracle import transformer as T
from paper_2211_17192_amd import synth

pytestmark = pytest.mark.gpu

# (arch, d_model, heads, kv heads, d_head, d_ff, layers, rows, enc_len): what each one reaches
CASES = {
    # fewer rows than two slabs, one K-step per wavefront: the smallest product over K-slices
    "gpt-17": (T.GPT, 128, 2, 2, 64, 512, 3, 17, 0),
    # odd row count, K of 23 k-steps (slices of 6, 6, 6, 5: three k-steps a block) and a 63-tile FFN
    "gqa-121-odd-k": (T.GQA, 736, 12, 6, 64, 1008 * 2, 2, 121, 0),
    # LayerNorm rows longer than what a wavefront holds in registers; K of eight slices
    "gpt-200-wide": (T.GPT, 2304, 4, 4, 64, 2080, 2, 200, 0),
    # position bias, cross-attention over a ragged number of encoder positions
    "t5-75-enc-61": (T.T5DEC, 256, 4, 4, 64, 704, 3, 75, 61),
    "t5-33-dh128": (T.T5DEC, 512, 4, 4, 128, 544, 2, 33, 17),
    # enough rows for the 64-row and the 128-row workgroups, four query heads per KV head
    "gqa-1050-medium-large": (T.GQA, 512, 16, 4, 64, 5120, 2, 1050, 0),
    # a context beyond 1024 positions: key ranges times row groups; two passes of the pass limit
    "gqa-2100-two-passes": (T.GQA, 256, 4, 2, 128, 512, 2, 2100, 0),
}


# Products whose tiles fill the rounds of 256 workgroups of eight wavefronts (256 features x 128 rows; a gated
# product's half as many features), rows no multiple of 128: QKV, gated, O / FFN-out; and with LayerNorm and biases
EIGHT = {
    "gqa-1999-eight": (T.GQA, 4096, 32, 16, 64, 2048, 2, 1999, 0),
    "gpt-2017-eight": (T.GPT, 4096, 32, 32, 64, 4096, 2, 2017, 0),
}


def takes_eight_wavefronts(rows, n, gated=False):
    """The rule of the launcher on a device of 256 CUs."""
    wgs = -(-(n // 16) // (8 if gated else 16)) * -(-(-(-rows // 16)) // 8)
    return rows > 128 and 100 * wgs >= 85 * 256 * -(-wgs // 256)


@pytest.mark.parametrize("name", list(EIGHT))
def test_prefill_with_eight_wavefront_products_equals_token_by_token(name):
    arch, d, heads, kv, dh, ff, layers, rows, enc = EIGHT[name]
    assert takes_eight_wavefronts(rows, d) and takes_eight_wavefronts(rows, ff, arch == T.GQA)
    assert arch != T.GQA or takes_eight_wavefronts(rows, (heads + 2 * kv) * dh)
    prefill_equals_token_by_token(EIGHT[name], False)


@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_prefill_equals_token_by_token(name, scatter):
    if scatter and CASES[name][7] > 300:
        pytest.skip("the page table's order is covered by the small cases")
    prefill_equals_token_by_token(CASES[name], scatter)


def prefill_equals_token_by_token(case, scatter, gamma=3):
    from paper_2211_17192_amd import binding
    arch, d, heads, kv, dh, ff, layers, rows, enc = case
    vocab = 512
    kw = dict(n_kv_heads=kv) if arch == T.GQA else {}
    cfg = synth.model_cfg(arch, layers, d, heads, ff, vocab, rows + 40, d_head=dh, enc_len=enc, dtype="bf16", logit_scale=4.0, **kw)
    w = synth.random_weights(cfg, 5, "cuda", 0.04)
    cfg_q, w_q = synth.truncated_noisy_copy(cfg, w, layers - 1, 9, 0.004)
    enc_out = synth.counter_normal((enc, d), 3, 1.0, 0.0, "cuda").to(torch.bfloat16) if enc else None
    flags = binding.SD_FLAG_GRAPH | (binding.SD_FLAG_SCATTER_PAGES if scatter else 0)
    dec = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=gamma, flags=flags)
    tokens = [int(t) for t in synth.random_tokens(7, 9, vocab)]
    u = synth.uniform_stream(11, (rows + 8) * (2 * gamma + 1)).reshape(-1, 2 * gamma + 1)
    dec.prefill(tokens, enc_out, enc_out)            # 8 rows: the decoding kernels
    it = 0
    while len(tokens) < rows + 1:
        tokens += dec.step(gamma, 1.0, u[it])[1]
        it += 1
    n1, t1 = dec.step(gamma, 1.0, u[it])
    p1, q1 = dec.logits(0, gamma + 1), dec.logits(1, gamma)
    dec.reset()
    dec.prefill(tokens, enc_out, enc_out)            # len(tokens) - 1 >= rows rows at once
    n2, t2 = dec.step(gamma, 1.0, u[it])
    p2, q2 = dec.logits(0, gamma + 1), dec.logits(1, gamma)
    dec.close()
    assert np.isfinite(p1).all() and np.ptp(p1) > 1.0
    assert np.array_equal(p1, p2) and np.array_equal(q1, q2)
    assert (n1, t1) == (n2, t2)


# Every chunk length and loop of the one-slab product (k-steps of 32 a wavefront; four wavefronts below K 2048, else
# eight), with k-steps past a slice's end: K of d_model, of heads x 64 and of d_ff; several tiles a workgroup in the
# LM head and, where d_ff is large, in FFN-in.
SLICES = {
    "gpt-2-3-5": (T.GPT, 160, 3, 3, 64, 544, 2, 18, 0),                      # a slice without k-steps; 3 and 5 of them
    "gpt-9-8-12": (T.GPT, 1056, 16, 16, 64, 1536, 2, 18, 0),                 # LayerNorm rows in two halves
    "gpt-15-9-17": (T.GPT, 1888, 33, 33, 64, 4128, 2, 18, 0),                # LayerNorm over chunks; eight wavefronts
    "gpt-13-16-20": (T.GPT, 3104, 64, 64, 64, 5120, 2, 18, 0),
    "gqa-16-11-24": (T.GQA, 1984, 22, 11, 64, 6112, 2, 18, 0),
    "gqa-13-16-40": (T.GQA, 3104, 32, 8, 128, 10240, 2, 18, 0),
    "gqa-18-24-8": (T.GQA, 4576, 48, 12, 128, 2016, 2, 18, 0),               # RMSNorm of more partial sums than are staged
    "t5-6-7-14": (T.T5DEC, 736, 13, 13, 64, 1760, 2, 18, 20),
}


@pytest.mark.parametrize("name", list(SLICES))
def test_k_slices_of_every_length_equal_the_products_over_many_rows(name):
    prefill_equals_token_by_token(SLICES[name], False)


# Contexts over several key ranges (512 keys): decoded tokens come from ranges merged by the last workgroup to arrive, or,
# with more KV heads than there are tickets (252), taken in turn; a prompt's from ranges taken in turn.
RANGES = {                                           # case, gamma
    "gqa-1100-two-row-tiles": ((T.GQA, 256, 16, 4, 128, 512, 2, 1100, 0), 7),            # (eight rows of four heads)
    "gqa-2700-six-ranges": ((T.GQA, 256, 16, 4, 128, 512, 2, 2700, 0), 7),               # two row tiles of 128 features: four ranges are merged at a time,
    "gqa-4700-ten-ranges": ((T.GQA, 128, 4, 2, 64, 256, 2, 4700, 0), 3),                 # else eight
    "gpt-1060-64-heads": ((T.GPT, 128, 64, 64, 64, 256, 2, 1060, 0), 3),                 # heads 63 and 0 share a ticket's word
    "gpt-1060-253-heads": ((T.GPT, 128, 253, 253, 64, 256, 2, 1060, 0), 3),
    "t5-1040-bias": ((T.T5DEC, 256, 4, 4, 64, 512, 2, 1040, 20), 3),
    "t5-1100-bias-dh128": ((T.T5DEC, 256, 4, 4, 128, 512, 2, 1100, 20), 3),
}


@pytest.mark.parametrize("name", list(RANGES))
def test_key_ranges_merged_by_ticket_equal_key_ranges_in_turn(name):
    case, gamma = RANGES[name]
    prefill_equals_token_by_token(case, False, gamma)


def test_decoding_with_64_kv_heads_spreads_its_key_ranges():
    """The attention of 64 KV heads over 8000 keys reads twice what 32 read.  (3.7 times their time when each of the 64 took
    its 16 ranges in turn.)"""
    from paper_2211_17192_amd import binding
    us = {}
    for heads in (32, 64):
        cfg = synth.model_cfg(T.GPT, 2, 128, heads, 256, 512, 8192, d_head=64, dtype="bf16", logit_scale=4.0)
        w = synth.random_weights(cfg, 5, "cuda", 0.04)
        cfg_q, w_q = synth.truncated_noisy_copy(cfg, w, 1, 9, 0.004)
        dec = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=4, flags=binding.SD_FLAG_GRAPH)
        dec.prefill(synth.random_tokens(7, 8000, 512))
        whole, rest = (min(dec.time_forward(0, 1, skip, 20) for _ in range(5)) for skip in (0, binding.SD_OP["attn"]))
        us[heads] = (whole - rest) / 2
        dec.close()
    print(us)
    assert us[64] <= 2.6 * us[32]


# (arch, d_model, heads, kv heads, d_head, d_ff, vocab, sequences, gamma, temperature): rows = sequences x (gamma + 1)
BATCHES = {
    # LayerNorm rows: two slabs and a ragged one, the smallest products
    "gpt-3x6": (T.GPT, 128, 2, 2, 64, 512, 512, 3, 5, 1.0),
    # five slabs, argmax; key ranges are tested by the 8B-class shapes
    "gpt-20x4-argmax": (T.GPT, 768, 12, 12, 64, 3072, 512, 20, 3, 0.0),
    # the most rows of a draft and of a verify forward, d_head 128
    "gpt-64x3": (T.GPT, 256, 2, 2, 128, 1024, 512, 64, 2, 1.0),
    "gqa-48x4": (T.GQA, 512, 8, 4, 64, 1408, 512, 48, 3, 1.0),
    # residual products of 64 MB over five slabs: K chunks over workgroups
    "gqa-16x5-split": (T.GQA, 2048, 8, 2, 128, 16384, 512, 16, 4, 1.0),
    # LM head over 144 rows: workgroups of eight wavefronts
    "gqa-16x9-head": (T.GQA, 256, 4, 4, 64, 512, 32000, 16, 8, 1.0),
    # contexts of one and of two key ranges, which 512 workgroups take in turn and 64, alone, do not
    "gpt-8x3-ranges": (T.GPT, 128, 64, 64, 64, 256, 512, 8, 2, 1.0),
}

@pytest.mark.parametrize("name", list(BATCHES))
def test_sequences_together_equal_each_alone(name):
    from paper_2211_17192_amd import binding
    arch, d, heads, kv, dh, ff, vocab, B, gamma, temperature = BATCHES[name]
    assert "head" not in name or takes_eight_wavefronts(B * (gamma + 1), vocab)
    kw = dict(n_kv_heads=kv) if arch == T.GQA else {}
    max_len, more = (1100, 540) if "ranges" in name else (160, 0)
    cfg = synth.model_cfg(arch, 2, d, heads, ff, vocab, max_len, d_head=dh, dtype="bf16", logit_scale=4.0, **kw)
    w = synth.random_weights(cfg, 5, "cuda", 0.04)
    cfg_q, w_q = synth.truncated_noisy_copy(cfg, w, 1, 9, 0.004)
    together = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=gamma, flags=binding.SD_FLAG_GRAPH, batch=B)
    alone = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=gamma, flags=binding.SD_FLAG_GRAPH)
    prompts = [[int(t) for t in synth.random_tokens(40 + b, 4 + 37 * b % 50 + more * (b % 2), vocab)] for b in range(B)]
    iterations = 3
    u = synth.uniform_stream(13, iterations * B * (2 * gamma + 1)).reshape(iterations, B, 2 * gamma + 1)
    for b, p in enumerate(prompts):
        together.prefill(p, row=b)
    got = []
    for it in range(iterations):
        res = together.step(gamma, temperature, u[it])
        got.append((res, together.logits(0, B * (gamma + 1)).reshape(B, gamma + 1, vocab), together.logits(1, B * gamma).reshape(B, gamma, vocab)))
    assert np.isfinite(got[0][1]).all() and np.ptp(got[0][1]) > 1.0
    for b, p in enumerate(prompts):
        alone.reset()
        alone.prefill(p)
        for it in range(iterations):
            assert alone.step(gamma, temperature, u[it, b]) == got[it][0][b], (it, b)
            assert np.array_equal(alone.logits(0, gamma + 1), got[it][1][b]), (it, b)
            assert np.array_equal(alone.logits(1, gamma), got[it][2][b]), (it, b)
    together.close()
    alone.close()


# (arch, d_model, heads, kv heads, d_head, d_ff, vocab, max_len, enc_len, max_gamma, sequences), and the bytes of a
# workspace without room for prompt passes of more than 16 rows (what the pair needs otherwise, with 31 KB of row
# statistics a sequence beside the activations: sizes that loaded before those passes existed)
WORKSPACES = {
    "gqa-key-ranges": ((T.GQA, 256, 4, 2, 64, 512, 512, 1500, 0, 3, 1), 7933184),
    "gqa-key-ranges-6": ((T.GQA, 256, 4, 2, 64, 512, 512, 1500, 0, 3, 6), 24270592),          # 24 rows in two slabs
    "gpt-gamma-15": ((T.GPT, 128, 2, 2, 64, 256, 50256, 300, 0, 15, 1), 59184640),
    "t5": ((T.T5DEC, 256, 4, 4, 64, 512, 512, 200, 100, 3, 1), 7660800),
}


@pytest.mark.parametrize("name", list(WORKSPACES))
def test_smaller_workspaces_give_the_same_results(name, monkeypatch):
    """Whatever room a workspace leaves for prompt passes, down to none."""
    from paper_2211_17192_amd import binding
    (arch, d, heads, kv, dh, ff, vocab, max_len, enc, gamma, B), least = WORKSPACES[name]
    kw = dict(n_kv_heads=kv) if arch == T.GQA else {}
    cfg = synth.model_cfg(arch, 2, d, heads, ff, vocab, max_len, d_head=dh, enc_len=enc, dtype="bf16", logit_scale=4.0, **kw)
    w = synth.random_weights(cfg, 5, "cuda", 0.04)
    cfg_q, w_q = synth.truncated_noisy_copy(cfg, w, 1, 9, 0.004)
    enc_out = synth.counter_normal((enc, d), 3, 1.0, 0.0, "cuda").to(torch.bfloat16) if enc else None
    prompt = [int(t) for t in synth.random_tokens(7, max_len - 3 * (gamma + 1), vocab)]
    u = synth.uniform_stream(11, 2 * B * (2 * gamma + 1)).reshape(2, B, 2 * gamma + 1)

    def decode(nbytes):
        with monkeypatch.context() as mp:
            if nbytes:
                mp.setattr(binding.lib, "sd_workspace_bytes", lambda *a: nbytes)
            dec = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=gamma, flags=binding.SD_FLAG_GRAPH, batch=B)
        for b in range(B):
            dec.prefill(prompt[: len(prompt) - 5 * b], enc_out, enc_out, row=b)
        out = []
        for it in range(2):
            out += [dec.step(gamma, 1.0, u[it] if B > 1 else u[it, 0]), dec.logits(0, B * (gamma + 1)), dec.logits(1, B * gamma)]
        size = dec.workspace_bytes
        dec.close()
        return size, out

    full, ref = decode(0)
    assert least < full
    for nbytes in (least, (least + full) // 2, full - 256):
        _, got = decode(nbytes)
        for a, b in zip(ref, got):
            assert np.array_equal(a, b) if isinstance(a, np.ndarray) else a == b
    with pytest.raises(binding.SdError, match="workspace too small"):
        decode(least // 2)


def test_last_prompt_rows_of_both_models_beside_each_other():
    """A pass of 2048 rows and one of 9, whose key ranges both models merge by tickets, on a stream and with tickets each."""
    prefill_equals_token_by_token((T.GQA, 256, 4, 2, 128, 512, 3, 2057, 0), False)


@pytest.mark.parametrize("layers_q", [1, 3])        # a draft of fewer layers than the target, and of more
def test_prompt_waits_for_the_callers_stream(layers_q, monkeypatch):
    """sd_prefill on a stream of the caller's that still computes the encoder outputs: both models' launches come behind it."""
    import ctypes as C
    from paper_2211_17192_amd import binding
    cfg = synth.model_cfg(T.T5DEC, 2, 256, 4, 704, 512, 200, d_head=64, enc_len=61, dtype="bf16", logit_scale=4.0)
    w = synth.random_weights(cfg, 5, "cuda", 0.04)
    cfg_q = dict(cfg, n_layers=layers_q)
    w_q = synth.random_weights(cfg_q, 6, "cuda", 0.04)
    enc = synth.counter_normal((61, 256), 3, 1.0, 0.0, "cuda").to(torch.bfloat16)
    tokens = np.asarray(synth.random_tokens(40, 9, 512), dtype=np.int32)
    u = synth.uniform_stream(11, 7)

    def logits(dec):
        dec.step(3, 1.0, u)
        return dec.logits(0, 4), dec.logits(1, 3)

    dec = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=3)
    dec.prefill(tokens, enc, enc)
    want = logits(dec)
    stream = torch.cuda.Stream()
    plain = binding._RuntimeCfg
    monkeypatch.setattr(binding, "_RuntimeCfg", lambda **kw: plain(**{**kw, "stream": stream.cuda_stream}))
    dec = binding.SpecDecoder(cfg, w, cfg_q, w_q, max_gamma=3)
    big = torch.zeros(4096, 4096, device="cuda")
    late = [torch.zeros_like(enc), torch.zeros_like(enc)]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(20):
            big = big @ big
        for t in late:
            t.copy_(enc)
    ptr = lambda t: C.c_void_p(t.data_ptr())         # noqa: E731
    st = binding.lib.sd_prefill(dec._ctx, 0, tokens.ctypes.data_as(C.POINTER(C.c_int32)), len(tokens), ptr(late[0]), ptr(late[1]))
    assert st == 0
    got = logits(dec)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
