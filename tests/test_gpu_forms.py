"""GPU: the kernels' forms at the sizes where they can go wrong -- whole and ragged tiles of the matrix products with two to a
few K steps, decode steps on either side of the rules that divide an attention job inside a block, norms with a
wave or a block to a row, and a joined output product whose K is not whole K blocks."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import decoder as O
from workloads import ModelShape
from gpu_util import (GPU_SHAPES, LONG_SHAPES, TOL_LOGITS, TOL_LOGPROB, R, dev_f32, dev_i32, long_context_weights, make_policy, padded,
                      reference_decoder, report, scaled_bf16_weights)
from rounding_model import DEFAULT_FORMATS, RoundedDecoder

pytestmark = pytest.mark.gpu

# K = d: two, three and five K steps of 64; d_ffn + d: 8 to 15 (a ring of up to six stages fills and drains); widths that are
# no multiple of a 64-, 128- or 256-column tile; the vocabulary odd
TILES = {
    "neox-d128": ModelShape(0, 1, 128, 2, 2, 64, 384, 515, rotary_dim=16),
    "neox-d192": ModelShape(0, 1, 192, 4, 4, 48, 608, 333, rotary_dim=12),
    "llama-d320": ModelShape(1, 1, 320, 4, 2, 80, 640, 700, rotary_dim=80, rope_theta=500000.0),
}


@pytest.mark.parametrize("precise", [0, 1])
@pytest.mark.parametrize("name", list(TILES))
def test_every_tile_shape_returns_the_same_bits_on_whole_and_ragged_tiles(name, precise):
    """One chunk of 611 rows (two whole 256-row tiles and a ragged one) through every tile shape, forced on all layers of the
    prompt pass: the same bits for all of them, and those within tolerance of the reference."""
    m = TILES[name]
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m, precise)
    rng = np.random.default_rng(17)
    seqs = [rng.integers(0, m.vocab, size=n) for n in (256, 1, 255, 99)]
    arr, lens = padded(seqs)
    r = R()
    pol = make_policy(W, max_seqs=4, max_seq_len=256, max_batch_tokens=1024, precise=precise)
    outs = []
    try:
        for v in [0, 3, 5, 7] if precise else range(11):
            for which in range(5):
                wide_only = which == 4 or (which == 2 and m.arch == 1)
                r.rlgen_debug_set_gemm(pol, 1, which, 0 if wide_only and 6 <= v <= 9 else v)
            outs.append((r.rlgen_score(pol, dev_i32(arr), lens, 0.7).cpu(), r.rlgen_debug_logits(pol, dev_i32(arr), lens).cpu()))
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for o in outs[1:]:
        assert torch.equal(o[0], outs[0][0]) and torch.equal(o[1], outs[0][1])
    ref = np.stack([O.last_logits(dec, s) for s in seqs])
    assert np.abs(outs[0][1].numpy() - ref).max() < (TOL_LOGITS / 20 if precise else TOL_LOGITS)
    for n in (0, 3):
        assert np.abs(outs[0][0][n, :lens[n]].numpy() - O.score(dec, seqs[n], 0.7)).max() < TOL_LOGPROB


# capacities on either side of the rules: decode attention shares a job among eight or four waves while capacity x kv heads x
# max(head size, 64) is at most 32768 (256 jobs of head sizes 80 and 96, 16384 for wider heads) or 131072
@pytest.mark.parametrize("max_seqs", [6, 17, 128, 129, 300, 2100])
@pytest.mark.parametrize("name", ["neox-h16-raggedV", "neox-h80", "neox-h256", "llama-gqa4-h16", "llama-gqa2-h128"])
def test_decode_forms_match_the_reference(name, max_seqs):
    m = GPU_SHAPES[name]
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m)
    rng = np.random.default_rng(23)
    lens = [1, 31, 32, 33, 97, 150]
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in lens])
    T = 5
    forced = rng.integers(0, m.vocab, size=(6, 1, T)).astype(np.int32)
    r = R()
    pol = make_policy(W, max_seqs=max_seqs, max_seq_len=160, max_kv_tokens=max(6 * 160, 32 * max_seqs), max_batch_tokens=160)
    try:
        u = dev_f32(np.zeros((6, 1, T)))
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, u, dev_i32(forced))
        # a smaller batch of the same context takes its sums in the same order
        _, one = r.rlgen_generate(pol, dev_i32(arr[4:5]), lens[4:5], 1, T, 0.7, u[:1].contiguous(), dev_i32(forced[4:5]))
        assert r.rlgen_status(pol) == 0
        assert torch.equal(one[0], lp[4])
        lp = lp.cpu().numpy()
    finally:
        pol.close()
    for b in range(6):
        want = O.score(dec, np.concatenate([arr[b, :lens[b]], forced[b, 0]]), 0.7, score_from=int(lens[b]))[lens[b]:]
        assert np.abs(lp[b, 0] - want).max() < TOL_LOGPROB


# widths whose 16-byte pieces fill one wave's share and part of the next (80), the second round of all four (264) and the third (640);
# the 1056-wide shapes end a K block half full.  1037 rows of 1056 cut the products into the residual in two or three parts
NORM_SHAPES = {
    "neox-d320": ModelShape(0, 2, 320, 5, 5, 64, 640, 300, rotary_dim=16),          # the output products are one
    "neox-d1056": ModelShape(0, 2, 1056, 33, 33, 32, 1024, 300, rotary_dim=8),      # they are two
    "llama-d1056": ModelShape(1, 2, 1056, 33, 11, 32, 1024, 300, rotary_dim=32, rope_theta=500000.0),
    "neox-d2560": ModelShape(0, 2, 2560, 40, 40, 64, 512, 300, rotary_dim=16),
}


@pytest.mark.parametrize("precise", [0, 1])
@pytest.mark.parametrize("name", list(NORM_SHAPES))
def test_norms_return_the_same_bits_with_a_wave_or_a_block_to_a_row(name, precise):
    """A sequence scored on its own (few rows: a block to each, which also adds up the parts of a split product) and among others
    (1037 rows: a wave to each, and the parts are added by the product's second pass)."""
    m = NORM_SHAPES[name]
    W = scaled_bf16_weights(m, scale=1.5)
    rng = np.random.default_rng(29)
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in [100] * 10 + [37]])
    r = R()
    pol = make_policy(W, max_seqs=12, max_seq_len=100, max_batch_tokens=1056, precise=precise)
    try:
        assert r.rlgen_debug_get_gemm(pol, 1, 3)[1] > 1          # the product into the residual is split
        many = r.rlgen_score(pol, dev_i32(arr), lens, 1.0)
        for i in (3, 10):
            one = r.rlgen_score(pol, dev_i32(arr[i:i + 1]), lens[i:i + 1], 1.0)
            assert torch.equal(many[i, :lens[i]], one[0, :lens[i]])
        assert (many[10, 1:37] < 0).all()
    finally:
        pol.close()


@pytest.mark.parametrize("precise", [0, 1])
def test_joined_output_product_with_half_a_k_block(precise):
    """d_ffn % 64 = 32: the joined attention-output and FFN-down product ends on half a K block."""
    m = ModelShape(0, 2, 64, 4, 4, 16, 160, 200, rotary_dim=4)
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m, precise)
    rng = np.random.default_rng(37)
    seqs = [rng.integers(0, m.vocab, size=n) for n in (5, 64, 33)]
    arr, lens = padded(seqs)
    r = R()
    pol = make_policy(W, max_seqs=3, max_seq_len=70, precise=precise)
    try:
        z = r.rlgen_debug_logits(pol, dev_i32(arr), lens).cpu().numpy()
        forced = rng.integers(0, m.vocab, size=(3, 1, 4)).astype(np.int32)
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, 4, 1.0, dev_f32(np.zeros((3, 1, 4))), dev_i32(forced))
        lp = lp.cpu().numpy()
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    assert np.abs(z - np.stack([O.last_logits(dec, s) for s in seqs])).max() < (TOL_LOGITS / 20 if precise else TOL_LOGITS)
    for b in range(3):
        want = O.score(dec, np.concatenate([seqs[b], forced[b, 0]]), 1.0, score_from=len(seqs[b]))[len(seqs[b]):]
        assert np.abs(lp[b, 0] - want).max() < TOL_LOGPROB


@pytest.mark.parametrize("V", [63, 131072, 131073, 200001])
def test_sampler_draws_in_order_at_any_vocabulary(V):
    """Up to 131072 columns a thread holds its run of column groups in registers, beyond it reads the rest again; 63 columns are
    one group for 256 threads.  Every draw must lie in the reference's CDF bucket (up to the 1e-4 that the 16-bit rows move the
    CDF by) and carry its log-prob."""
    m = ModelShape(0, 1, 64, 4, 4, 16, 64, V, rotary_dim=4)
    W = scaled_bf16_weights(m, scale=4.0)
    dec = O.Decoder(W, m, np.float64)
    rng = np.random.default_rng(V)
    hidden = rng.normal(size=(9, 64)).astype(np.float32)
    u = np.array([0.0, 1e-6, 0.1, 0.3, 0.5, 0.7, 0.9, 0.999, 0.99999994], np.float32)
    r = R()
    pol = make_policy(W, max_seqs=9, max_seq_len=32)
    try:
        tok, lp = (x.cpu().numpy() for x in r.rlgen_debug_sample(pol, dev_f32(hidden), 0.7, dev_f32(u)))
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    logp = O.tempered_log_softmax(dec.logits(hidden.astype(np.float64)), 0.7)
    for i in range(9):
        lo, hi = O.cdf_bucket(logp[i], int(tok[i]))
        assert lo - 1e-4 <= u[i] <= hi + 1e-4, (i, tok[i])
        assert abs(lp[i] - logp[i, tok[i]]) < TOL_LOGPROB


def test_a_vocabulary_beyond_two_to_the_24():
    """A weight row of 64 K values is 128 bytes: from row 2^24 on a K block's rows lie past the 2 GiB that a 32-bit distance with a
    buffer's bounds reaches.  The LM head repeats with a period that divides no power of two, the rows from 2^24 on sixteen
    times as large (exact in fp16 and fp32), so every logit is known from those of the first period bit for bit, and the last
    columns decide log Z: every tile shape must return the log-probs that the logits give, and the same bits."""
    r = R()
    V, P, d = (1 << 24) + 777, 4099, 128
    m = ModelShape(0, 1, d, 2, 2, 64, 128, V, rotary_dim=16)
    small = scaled_bf16_weights(ModelShape(0, 1, d, 2, 2, 64, 128, P, rotary_dim=16), scale=2.5)
    dev = r.upload_weights(small.tensors)
    scale = torch.ones(V, 1, dtype=torch.bfloat16, device="cuda")
    scale[1 << 24:] = 16.0
    head = ((dev["lm_head"].float() * 64).round() / 64).to(torch.bfloat16)       # no value is subnormal in fp16
    dev["lm_head"] = head.repeat((V + P - 1) // P, 1)[:V] * scale
    dev["embed_in"] = dev["embed_in"].repeat((V + P - 1) // P, 1)[:V].contiguous()
    rng = np.random.default_rng(3)
    seqs = rng.integers(0, V, size=(3, 9)).astype(np.int32)
    seqs[:, -1] = (5, V - 1, (1 << 24) + 3)
    lens = [9, 9, 9]
    cfg = r.make_cfg(m, weight_dtype=r.DTYPE_BF16, max_seqs=3, max_seq_len=32, max_kv_tokens=96)
    pol = r.Policy(cfg, dev)
    del dev
    try:
        z = r.rlgen_debug_logits(pol, dev_i32(seqs), [8, 8, 8])
        want = torch.cat([z[:, :P].repeat(1, (V + P - 1) // P)[:, :1 << 24],
                          16 * z[:, torch.arange(1 << 24, V, device="cuda") % P]], dim=1)
        assert torch.equal(z, want)
        want_lp = torch.log_softmax(z.double() / 0.7, dim=1)[torch.arange(3), torch.from_numpy(seqs[:, -1]).cuda().long()]
        hidden = dev_f32(rng.normal(size=(3, d)))
        u = dev_f32(np.array([0.1, 0.5, 0.9]))
        outs = []
        for v in (0, 1, 2, 3, 4, 5, 10):
            for mode in (0, 1):
                r.rlgen_debug_set_gemm(pol, mode, 4, v)
            score = r.rlgen_score(pol, dev_i32(seqs), lens, 0.7)
            assert (score[:, -1].double() - want_lp).abs().max() < 1e-4, v       # fp32 sums of the same logits
            outs.append((score, *r.rlgen_debug_sample(pol, hidden, 0.7, u)))
        for o in outs[1:]:
            assert all(torch.equal(a, b) for a, b in zip(o, outs[0])), o
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()


@pytest.mark.parametrize("temperature,precise", [(0.7, 1), (1e-38, 0), (1e-38, 1), (1e-40, 0), (1e-40, 1)])
def test_lm_head_statistics_with_infinite_logits(temperature, precise):
    """Logits of -infinity (a precise-mode weight row whose product overflows, or any negative logit over a tiny temperature)
    have probability zero, also where they fill whole groups of 64 columns and whole tiles.  Columns 37 and 700 have logit 0, and
    a row's draw is one of the two at log-prob -log 2."""
    from workloads import f32_to_bf16_bits
    r = R()
    V, d, rows = 1000, 64, 300
    m = ModelShape(0, 1, d, 4, 4, 16, 64, V, rotary_dim=4)
    W = scaled_bf16_weights(m)
    low = -3e38 if temperature > 0.1 else -0.05
    head = np.full((V, d), low, np.float32)
    head[[37, 700]] = 0.0
    W.tensors.update({"final_norm_g": f32_to_bf16_bits(np.full(d, 0.1, np.float32)),
                      "final_norm_b": f32_to_bf16_bits(np.full(d, 3.0, np.float32)), "lm_head": f32_to_bf16_bits(head)})
    rng = np.random.default_rng(5)
    u = rng.random(rows, dtype=np.float32)
    pol = make_policy(W, max_seqs=rows, max_seq_len=32, precise=precise)
    try:
        for v in (0, 3, 5) if precise else (0, 1, 2, 3, 4, 5, 10):
            r.rlgen_debug_set_gemm(pol, 0, 4, v)
            tok, lp = (x.cpu().numpy() for x in r.rlgen_debug_sample(pol, dev_f32(rng.normal(size=(rows, d))), temperature, dev_f32(u)))
            np.testing.assert_array_equal(tok, np.where(u < 0.5, 37, 700), err_msg=str(v))
            assert np.abs(lp + np.log(2.0)).max() < 1e-6, v
    finally:
        pol.close()


@pytest.mark.parametrize("precise", [0, 1])
def test_swiglu_at_large_gates(precise):
    """Gates from where exp(-gate) overflows to where it vanishes.  Every token embeds to ones, attention adds nothing, gate f is
    the f-th value and its activation, scaled to order one, reaches residual f, which the LM head reads out."""
    from workloads import f32_to_bf16_bits
    gates = [-6e4, -1e3, -103.5, -89.0, -88.5, -88.0, -87.0, -40.0, -9.0, -1.0, -0.01, 0.0, 0.01, 1.0, 9.0, 40.0, 88.5, 1e3, 6e4]
    d, F = 64, 32
    m = ModelShape(1, 1, d, 4, 2, 16, F, d, rotary_dim=16)
    W = scaled_bf16_weights(m)
    g = np.zeros(F, np.float32)
    g[:len(gates)] = gates
    down = np.zeros((d, F), np.float32)
    down[np.arange(F), np.arange(F)] = 1.0 / np.maximum(np.abs(g), 0.25)
    ones = f32_to_bf16_bits(np.ones(d, np.float32))
    W.tensors.update({"embed_in": f32_to_bf16_bits(np.ones((d, d), np.float32)), "lm_head": f32_to_bf16_bits(4 * np.eye(d, dtype=np.float32)),
                      "layers.0.wo": f32_to_bf16_bits(np.zeros((d, d), np.float32)), "layers.0.norm2_g": ones, "final_norm_g": ones,
                      "layers.0.w_gate": f32_to_bf16_bits(np.repeat(g[:, None] / d, d, 1)),
                      "layers.0.w_up": f32_to_bf16_bits(np.full((F, d), 1.0 / d, np.float32)), "layers.0.w_down": f32_to_bf16_bits(down)})
    dec = reference_decoder(W, m, precise)
    r = R()
    pol = make_policy(W, max_seqs=2, max_seq_len=32, precise=precise)
    try:
        z = r.rlgen_debug_logits(pol, dev_i32(np.array([[1, 2, 3]])), [3]).cpu().numpy()
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    with np.errstate(over="ignore"):
        want = O.last_logits(dec, np.array([1, 2, 3]))
    assert np.abs(z[0] - want).max() < (TOL_LOGITS / 20 if precise else TOL_LOGITS)


@pytest.mark.parametrize("share", [0, 1])
@pytest.mark.parametrize("name,max_seqs,waves", [(n, s, w) for n in ("neox-h64", "llama-gqa2-h128", "neox-h256")
                                                 for s, w in ((12, 8), (300, 4), (1100, 1))])
def test_decode_attention_over_several_turns_of_the_key_loop(name, max_seqs, waves, share):
    """A job's waves take super-blocks of 32 keys in turn and request one or two turns ahead: contexts of one turn of eight waves less,
    exactly and more (255 to 257 keys), of two (513) and of three and a part (797, where the steps cross into a new super-block).
    Tolerance: the reference rounds where the library does, and its own log-probs move by at most 1.3e-3 on these models when its
    sums are taken in fp64 instead of fp32 (roundings that fall the other way); with two blocks of the Llama shape that is
    1.1e-2, so it has one here."""
    m = LONG_SHAPES[name]
    r = R()
    assert r.lib["_Z25rl_attention_decode_splitxi"](C.c_longlong(max_seqs * m.n_kv_heads), m.head_dim) == waves
    W = long_context_weights(name)
    dec = RoundedDecoder(W, m, DEFAULT_FORMATS)
    rng = np.random.default_rng(41)
    prompts = [rng.integers(0, m.vocab, size=n) for n in (31, 255, 256, 257, 513, 797)]
    arr, lens = padded(prompts)
    k, T = 2, 5
    forced = rng.integers(0, m.vocab, size=(6, k, T)).astype(np.int32)
    pol = make_policy(W, max_seqs=max_seqs, max_seq_len=832, max_kv_tokens=5000, max_batch_tokens=832, share_prompt_kv=share)
    try:
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, k, T, 0.7, dev_f32(np.zeros((6, k, T))), dev_i32(forced))
        assert r.rlgen_status(pol) == 0
        lp = lp.cpu().numpy()
    finally:
        pol.close()
    worst = 0.0
    for b in range(6):
        for j in range(k):
            want = O.score(dec, np.concatenate([prompts[b], forced[b, j]]), 0.7, score_from=int(lens[b]))[lens[b]:]
            worst = max(worst, np.abs(lp[b, j] - want).max())
    report("decode-attention-turns", err=worst, waves=waves, h=m.head_dim, share=share)
    assert worst < TOL_LOGPROB


# FFN-down is cut into parts, and the GPT-NeoX shape's FFN-up too
DECODE_TILES = {
    "neox-d512": ModelShape(0, 2, 512, 8, 8, 64, 1024, 515, rotary_dim=16),
    "llama-d256": ModelShape(1, 2, 256, 4, 2, 64, 512, 700, rotary_dim=64, rope_theta=500000.0),
}


@pytest.mark.parametrize("precise", [0, 1])
@pytest.mark.parametrize("name", list(DECODE_TILES))
def test_decode_steps_return_the_same_bits_on_every_tile_shape(name, precise):
    """Every tile shape forced on all layers of a decode step of 131 sequences (ragged in every tile), taken whole and as two
    halves: the QKV product's writes into the cache, split and whole products, the LM head.  The same tokens and log-probs bit
    for bit, and those within tolerance of the reference."""
    m = DECODE_TILES[name]
    W = scaled_bf16_weights(m, scale=2.0)
    rng = np.random.default_rng(53)
    prompts = [rng.integers(0, m.vocab, size=n) for n in rng.integers(1, 40, size=131)]
    arr, lens = padded(prompts)
    T = 5
    u = dev_f32(rng.random((131, 1, T), dtype=np.float32))
    r = R()
    pol = make_policy(W, max_seqs=131, max_seq_len=45, precise=precise)
    outs = []
    try:
        splits = [r.rlgen_debug_get_gemm(pol, 0, which)[1] for which in range(5)]
        assert splits[3] > 1 and (m.arch == 1 or splits[2] > 1), splits
        for v in [0, 3, 5, 7] if precise else range(11):
            for halves in (0, 1):
                r.rlgen_set_decode_split_min(pol, 2 if halves else 0)
                for which in range(5):
                    wide_only = which == 4 or (which == 2 and m.arch == 1)
                    r.rlgen_debug_set_gemm(pol, 2 if halves else 0, which, 0 if wide_only and 6 <= v <= 9 else v)
                outs.append(r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, u))
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for t, lp in outs[1:]:
        assert torch.equal(t, outs[0][0]) and torch.equal(lp, outs[0][1])
    t, lp = (x.cpu().numpy() for x in outs[0])
    dec = reference_decoder(W, m, precise)
    for b in (0, 64, 130):
        want = O.score(dec, np.concatenate([prompts[b], t[b, 0]]), 0.7, score_from=int(lens[b]))[lens[b]:]
        assert np.abs(lp[b, 0] - want).max() < TOL_LOGPROB


# every way a key's and a value's head dims divide in the cache: steps of 32 dims with and without a rest of 16, whole groups of
# 64 dims and 0 to 3 tiles behind them; rotary pairs inside a step and across steps
@pytest.mark.parametrize("precise", [0, 1])
@pytest.mark.parametrize("h, rot", [(16, 16), (32, 8), (48, 48), (64, 16), (64, 6), (80, 20), (96, 96), (112, 28), (128, 128), (256, 64)])
def test_decode_steps_read_what_the_prompt_pass_and_they_wrote(h, rot, precise):
    """Prompts of 27 and 32 tokens and 40 decoded ones (pairs, groups of eight and super-blocks begin and end in both): the
    same log-probs as one prompt pass over all of them."""
    if precise and (h == 256 or rot % 4):
        pytest.skip("no precise mode for this shape")
    m = ModelShape(0, 2, 2 * h, 2, 2, h, 128, 210, rotary_dim=rot)
    W = scaled_bf16_weights(m)
    rng = np.random.default_rng(41)
    lens, T = [27, 32], 40
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in lens])
    forced = rng.integers(0, m.vocab, size=(2, 1, T)).astype(np.int32)
    r = R()
    pol = make_policy(W, max_seqs=2, max_seq_len=72, precise=precise)
    try:
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, dev_f32(np.zeros((2, 1, T))), dev_i32(forced))
        full = np.zeros((2, 72), np.int32)
        for b in range(2):
            full[b, :lens[b] + T] = np.concatenate([arr[b, :lens[b]], forced[b, 0]])
        sc = r.rlgen_score(pol, dev_i32(full), [n + T for n in lens], 0.7).cpu().numpy()
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for b in range(2):
        assert np.abs(lp.cpu().numpy()[b, 0] - sc[b, lens[b]:lens[b] + T]).max() < (TOL_LOGPROB / 20 if precise else TOL_LOGPROB)


# one launch for QKV and FFN-up: widths of both that are no multiple of any tile, with and without a joined output product, prompt
# pass and decode; the Llama shape has no such launch
@pytest.mark.parametrize("m", [ModelShape(0, 2, 192, 4, 4, 48, 608, 333, rotary_dim=12), ModelShape(0, 1, 256, 1, 1, 256, 1056, 130, rotary_dim=64),
                               ModelShape(0, 1, 96, 2, 2, 48, 160, 100, rotary_dim=12)])
def test_qkv_and_ffn_up_in_one_launch_match_the_reference(m):
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m)
    rng = np.random.default_rng(61)
    lens = [1, 63, 64, 65, 130]
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in lens])
    T = 6
    forced = rng.integers(0, m.vocab, size=(5, 1, T)).astype(np.int32)
    r = R()
    outs = []
    for shape in (None, 1, 6, 2, 3):             # the rule's tile, the smallest, 64x64, 128x128, 256x256
        pol = make_policy(W, max_seqs=5, max_seq_len=140)
        try:
            for mode in (0, 1):
                assert r.rlgen_debug_get_gemm(pol, mode, 2)[0] == -2          # (FFN-up has no launch of its own)
                if shape is not None:
                    r.rlgen_debug_set_gemm(pol, mode, 0, shape)
            _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, dev_f32(np.zeros((5, 1, T))), dev_i32(forced))
            assert r.rlgen_status(pol) == 0
            outs.append(lp.cpu())
        finally:
            pol.close()
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
    for b in range(5):
        want = O.score(dec, np.concatenate([arr[b, :lens[b]], forced[b, 0]]), 0.7, score_from=int(lens[b]))[lens[b]:]
        assert np.abs(outs[0].numpy()[b, 0] - want).max() < TOL_LOGPROB


# contexts with room for enough rows that the waves of a block share the super-blocks of a prompt pass: every division of the head
# dims among them, waves along the tokens, the heads of a group or both; a group of three has no heads to share
@pytest.mark.parametrize("hq, hkv, h", [(4, 4, 16), (3, 3, 32), (2, 2, 48), (2, 2, 64), (2, 2, 80), (2, 2, 96), (2, 2, 112), (2, 2, 128), (1, 1, 256),
                                        (4, 1, 64), (4, 2, 80), (3, 1, 32), (8, 2, 128), (4, 1, 112), (2, 1, 256)])
def test_prompt_attention_with_shared_super_blocks_matches_the_reference(hq, hkv, h):
    """Sequences of 1 to 200 tokens (ends inside and at the end of query blocks, blocks of waves and super-blocks), on their own and as
    completions behind a shared prompt."""
    m = ModelShape(0 if hq == hkv else 1, 1, hq * h, hq, hkv, h, 96, 150, rotary_dim=h // 4 * 4 if h < 64 else 16 if hq == hkv else h)
    W = scaled_bf16_weights(m)
    dec = RoundedDecoder(W, m, DEFAULT_FORMATS)       # with the formats applied: on widths of 64 and 96 they alone are up to 0.012 off
    rng = np.random.default_rng(67)
    lens = [1, 15, 16, 17, 32, 33, 64, 65, 127, 128, 129, 200]
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in lens])
    r = R()
    pol = make_policy(W, max_seqs=12, max_seq_len=300, max_kv_tokens=12 * 320, max_batch_tokens=40000)
    try:
        lp = r.rlgen_score(pol, dev_i32(arr), lens, 0.7).cpu().numpy()
        for n in range(12):
            if lens[n] > 1:
                assert np.abs(lp[n, :lens[n]] - O.score(dec, arr[n, :lens[n]], 0.7)).max() < TOL_LOGPROB
        P, tails = 77, [1, 16, 33, 90]
        full = np.zeros((4, P + 90), np.int32)
        full[:, :P] = arr[11, :P]
        for j, n in enumerate(tails):
            full[j, P:P + n] = rng.integers(0, m.vocab, size=n)
        total = [P + n for n in tails]
        plain = r.rlgen_score(pol, dev_i32(full), total, 0.7, [P] * 4).cpu().numpy()
        r.rlgen_set_score_groups(pol, 4)
        grouped = r.rlgen_score(pol, dev_i32(full), total, 0.7, [P] * 4).cpu().numpy()
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for j, n in enumerate(tails):
        want = O.score(dec, full[j, :P + n], 0.7, score_from=P)[P:]
        assert np.abs(plain[j, P:P + n] - want).max() < TOL_LOGPROB
        assert np.abs(grouped[j, P:P + n] - want).max() < TOL_LOGPROB


@pytest.mark.parametrize("h", [16, 48, 80, 112])
def test_both_prompt_forms_agree_on_queries_that_an_infinite_key_does_not_reach(h):
    """Queries and keys are biases alone, the keys' large enough that the rotation (by the position itself, theta is 1) takes them
    beyond bf16 at some positions: the head's last dim at position 1, its partner h / 2 before it at 2.  The queries of the first
    four positions score such keys at minus infinity, weight zero, and their rows stay what they are without them: in a small
    context, where the waves of a block share a job, and in a large one, where they share super-blocks and head sizes that are no
    multiple of 32 end on half a step."""
    from workloads import f32_to_bf16_bits
    m = ModelShape(0, 1, 2 * h, 2, 2, h, 96, 150, rotary_dim=h, rope_theta=1.0)
    W = scaled_bf16_weights(m)
    pair = [h // 2 - 1, h - 1]
    bq, bk = np.zeros(2 * h, np.float32), np.zeros(2 * h, np.float32)
    bq[pair] = np.cos(-3.2), np.sin(-3.2)
    bk[pair] = 2.9e38
    zero = f32_to_bf16_bits(np.zeros((2 * h, 2 * h), np.float32))
    W.tensors.update({"layers.0.wq": zero, "layers.0.wk": zero, "layers.0.bq": f32_to_bf16_bits(bq), "layers.0.bk": f32_to_bf16_bits(bk)})
    pos = np.arange(4)
    k0, k2 = 2.9 * (np.cos(pos) - np.sin(pos)), 2.9 * (np.cos(pos) + np.sin(pos))
    q0, q2 = np.cos(pos - 3.2), np.sin(pos - 3.2)
    assert list(np.abs(k0) > 3.39) == [False, False, True, False] and list(np.abs(k2) > 3.39) == [False, True, False, False]
    assert (q2[1:] * k2[1] < 0).all() and (q0[2:] * k0[2] < 0).all()
    rng = np.random.default_rng(71)
    seqs = dev_i32(rng.integers(0, m.vocab, size=(6, 5)))
    r = R()
    outs = []
    for rows in (64, 40000):
        pol = make_policy(W, max_seqs=6, max_seq_len=32, max_batch_tokens=rows)
        try:
            outs.append(r.rlgen_score(pol, seqs, [5] * 6, 0.7).cpu().numpy())
            assert r.rlgen_status_bits(pol) == 8
        finally:
            pol.close()
    assert np.isfinite(outs[0]).all() and np.abs(outs[1][:, 1:] - outs[0][:, 1:]).max() < TOL_LOGPROB


@pytest.mark.parametrize("name", ["neox-d128", "neox-d192", "llama-d320"])
def test_a_tile_shape_for_ffn_up_takes_it_out_of_the_qkv_launch(name):
    """Small GPT-NeoX contexts report FFN-up as part of QKV's launch.  A shape set for it gives it a launch of its own, -2 takes it
    back, and every shape of either form returns the same bits: prompt pass (611 rows) and decode, whole and in halves."""
    m = TILES[name]
    W = scaled_bf16_weights(m)
    rng = np.random.default_rng(73)
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in (256, 1, 255, 99)])
    T = 3
    forced = dev_i32(rng.integers(0, m.vocab, size=(4, 1, T)))
    u = dev_f32(np.zeros((4, 1, T)))
    r = R()
    pol = make_policy(W, max_seqs=4, max_seq_len=256 + T, max_batch_tokens=1024)
    try:
        if m.arch == 1:
            for mode in range(3):
                assert r.rlgen_debug_get_gemm(pol, mode, 2)[0] != -2
                with pytest.raises(r.RlgenError):
                    r.rlgen_debug_set_gemm(pol, mode, 2, -2)
            return
        with pytest.raises(r.RlgenError):
            r.rlgen_debug_set_gemm(pol, 1, 0, -2)
        outs = []
        for v in range(11):
            for joined in (1, 0):
                for mode in range(3):
                    r.rlgen_debug_set_gemm(pol, mode, 0, v)
                    assert r.rlgen_debug_get_gemm(pol, mode, 2) == (-2, 1)
                    if not joined:
                        r.rlgen_debug_set_gemm(pol, mode, 2, v)
                        assert r.rlgen_debug_get_gemm(pol, mode, 2) == (v, 1)
                for halves in (0, 2):
                    r.rlgen_set_decode_split_min(pol, halves)
                    outs.append(r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, u, forced)[1].cpu())
                for mode in range(3):
                    r.rlgen_debug_set_gemm(pol, mode, 2, -2)
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


@pytest.mark.parametrize("max_seqs", [1, 64])
def test_narrow_models_of_few_rows_take_ffn_up_whole(max_seqs):
    """An FFN of a few tile columns, which would be cut into parts on its own, shares QKV's launch in decode steps of up to 64 rows."""
    m = ModelShape(0, 2, 512, 8, 8, 64, 2048, 200, rotary_dim=16)
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m)
    rng = np.random.default_rng(79)
    B, T = min(max_seqs, 3), 5
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in (33, 1, 20)[:B]])
    forced = rng.integers(0, m.vocab, size=(B, 1, T)).astype(np.int32)
    r = R()
    pol = make_policy(W, max_seqs=max_seqs, max_seq_len=40)
    try:
        assert r.rlgen_debug_get_gemm(pol, 0, 2) == (-2, 1)
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, dev_f32(np.zeros((B, 1, T))), dev_i32(forced))
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for b in range(B):
        want = O.score(dec, np.concatenate([arr[b, :lens[b]], forced[b, 0]]), 0.7, score_from=int(lens[b]))[lens[b]:]
        assert np.abs(lp.cpu().numpy()[b, 0] - want).max() < TOL_LOGPROB


@pytest.mark.parametrize("name", ["neox-d128", "neox-d192", "llama-d320", "neox-d512"])
def test_the_two_stage_tile_of_64_rows_returns_the_same_bits(name):
    """Two stages of 64x128 (no shape of the SwiGLU and LM-head products) on every layer that takes it, against 128x128: a prompt
    pass of 611 rows and decode steps, FFN-up in QKV's launch and on its own; 611 rows end in a ragged tile, 512 x 1536 is cut
    into parts."""
    m = {**TILES, **DECODE_TILES}[name]
    W = scaled_bf16_weights(m)
    rng = np.random.default_rng(83)
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in (256, 1, 255, 99)])
    T = 3
    forced, u = dev_i32(rng.integers(0, m.vocab, size=(4, 1, T))), dev_f32(np.zeros((4, 1, T)))
    r = R()
    pol = make_policy(W, max_seqs=4, max_seq_len=256 + T, max_batch_tokens=1024)
    outs = []
    try:
        with pytest.raises(r.RlgenError):
            r.rlgen_debug_set_gemm(pol, 1, 4, 11)
        for v in (0, 11):
            for apart in (0, 1):
                for mode in range(3):
                    for which in (0, 1, 2, 3):
                        if which == 2 and not (apart and m.arch == 0):
                            continue
                        r.rlgen_debug_set_gemm(pol, mode, which, v)
                outs.append((r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, u, forced)[1].cpu(), r.rlgen_score(pol, dev_i32(arr), lens, 0.7).cpu()))
                for mode in range(3):
                    if m.arch == 0 and apart:
                        r.rlgen_debug_set_gemm(pol, mode, 2, -2)
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for o in outs[1:]:
        assert torch.equal(o[0], outs[0][0]) and torch.equal(o[1], outs[0][1])


@pytest.mark.parametrize("max_seqs", [1, 64, 65])
def test_an_unfused_qkv_product_of_few_rows_stays_whole(max_seqs):
    """A rotary dim that is no multiple of 4 keeps QKV apart from its rotation; up to 64 rows its K is not cut."""
    m = ModelShape(0, 2, 512, 8, 8, 64, 1024, 200, rotary_dim=6)
    W = scaled_bf16_weights(m)
    dec = reference_decoder(W, m)
    rng = np.random.default_rng(89)
    B, T = min(max_seqs, 3), 5
    arr, lens = padded([rng.integers(0, m.vocab, size=n) for n in (33, 1, 20)[:B]])
    forced = rng.integers(0, m.vocab, size=(B, 1, T)).astype(np.int32)
    r = R()
    pol = make_policy(W, max_seqs=max_seqs, max_seq_len=40)
    try:
        assert (r.rlgen_debug_get_gemm(pol, 0, 0)[1] == 1) == (max_seqs <= 64)
        _, lp = r.rlgen_generate(pol, dev_i32(arr), lens, 1, T, 0.7, dev_f32(np.zeros((B, 1, T))), dev_i32(forced))
        assert r.rlgen_status(pol) == 0
    finally:
        pol.close()
    for b in range(B):
        want = O.score(dec, np.concatenate([arr[b, :lens[b]], forced[b, 0]]), 0.7, score_from=int(lens[b]))[lens[b]:]
        assert np.abs(lp.cpu().numpy()[b, 0] - want).max() < TOL_LOGPROB
