"""Incremental decoding on the GPU against the decoding oracle (the full decoder recomputed over each prefix)."""
import numpy as np
import pytest

from oracle.decoding import DecodingOracle, top_k
from synth import ModelShape, init_params
from synth.batches import zipf_ids

pytestmark = pytest.mark.gpu

SHAPES = {
    "width_768": ModelShape(0, 1, 768, 12, 3072, 96, pre_norm=1),
    "long_ffn": ModelShape(0, 1, 64, 1, 18432, 96),
    "post": ModelShape(2, 2, 32, 2, 64, 96),
    "pre": ModelShape(1, 2, 32, 4, 48, 80, pre_norm=1),
    "lm": ModelShape(0, 2, 32, 2, 64, 96, pre_norm=1),
    "half": ModelShape(2, 2, 128, 2, 256, 512),         # head width 64: the MFMA GEMMs serve rows that are a multiple of 8
    # the fp32 slices of a sub-layer's last product are summed by the LayerNorm kernel, those of the cross-attention query projection
    # by the attention kernel (head width 64) or, where the general attention kernel runs (head width 32), by a reduction in front
    # of it: a single slice with 9 to 64 rows at width 512, two with more rows or at width 1024
    "wide": ModelShape(1, 1, 512, 8, 1024, 96),
    "wide_dh32": ModelShape(1, 1, 512, 16, 1024, 96),
    "wider": ModelShape(1, 1, 1024, 16, 2048, 96),
    "wider_dh32": ModelShape(1, 1, 1024, 32, 2048, 96),
    # adaptive inputs + adaptive softmax: clusters of 24 / 32 / 40 tokens (generic kernels) and of 126 (+2 entries) / 128 / 256
    # tokens, every table a multiple of 8 rows (matrix-core GEMMs)
    "adaptive": ModelShape(0, 2, 32, 2, 64, 96, pre_norm=1, cutoffs=(24, 56), factor=2),
    "adaptive_half": ModelShape(0, 2, 128, 2, 256, 510, pre_norm=1, cutoffs=(126, 254)),
}


def rounded(params, prec):
    import torch
    import paper_1904_01038_amd as T
    tdt = {T.FP32: torch.float32, T.FP16: torch.float16, T.BF16: torch.bfloat16}[prec]
    return {k: torch.tensor(v, dtype=torch.float32).to(tdt).to(torch.float64).numpy() for k, v in params.items()}


def make(shape, prec, max_rows, max_steps, max_src, topk, seed=0):
    import paper_1904_01038_amd as T
    params = rounded(init_params(shape, seed, generic=True), prec)
    cfg = T.make_config(shape, precision=prec, max_sentences=16, max_len=max(max_steps, 24), max_tokens=256, dropout=0.3,
                        label_smoothing=0.0 if shape.cutoffs else 0.1)
    ctx = T.Tfm(cfg)
    ctx.set_params(params)
    return ctx, T.Decoder(ctx, max_rows, max_steps, max_src, topk), DecodingOracle(shape, params)


def sources(shape, rng, B, lo, hi):
    if not shape.enc_layers:
        return None, None
    lens = rng.integers(lo, hi + 1, B).astype(np.int32)
    src = np.full((B, lens.max()), shape.pad_id, np.int32)
    for b in range(B):
        src[b, :lens[b]] = np.append(zipf_ids(rng, lens[b] - 1, shape.vocab), shape.eos_id)
    return src, lens


def check_step(lp_gpu, top_lp, top_id, lp_ref, tol):
    """Full distribution within tol; the reported candidates are sorted, carry the right values, and nothing that was
    left out beats the last one by more than rounding."""
    assert np.max(np.abs(lp_gpu - lp_ref)) <= tol
    k = top_lp.shape[1]
    for r in range(lp_ref.shape[0]):
        assert len(set(top_id[r])) == k
        assert np.all(np.diff(top_lp[r]) <= 0.0)
        assert np.max(np.abs(top_lp[r] - lp_ref[r, top_id[r]])) <= tol
        assert np.allclose(top_lp[r], lp_gpu[r, top_id[r]], atol=1e-6)
        # exact on the GPU's own distribution: the same values, ties in ascending id order
        assert [i for _, i in top_k(lp_gpu[r], k)] == top_id[r].tolist()
        rest = np.delete(lp_ref[r], top_id[r])
        assert rest.max() <= top_lp[r, -1] + 2 * tol


@pytest.mark.parametrize("name,prec,tol", [("post", "fp32", 2e-4), ("pre", "fp32", 2e-4), ("lm", "fp32", 2e-4),
                                           ("half", "fp16", 3e-2), ("half", "bf16", 2e-1),
                                           ("wide", "fp16", 3e-2), ("wide", "bf16", 2e-1), ("wide_dh32", "fp16", 3e-2),
                                           ("wider", "fp16", 3e-2), ("wider", "bf16", 2e-1), ("wider_dh32", "fp16", 3e-2),
                                           ("adaptive", "fp32", 2e-4), ("adaptive_half", "fp16", 3e-2), ("adaptive_half", "bf16", 2e-1)])
def test_steps_with_reordered_beams_match_the_full_decoder(name, prec, tol, B=4, beam=4):
    import paper_1904_01038_amd as T
    shape = SHAPES[name]
    p = {"fp32": T.FP32, "fp16": T.FP16, "bf16": T.BF16}[prec]
    steps, topk = 7, 8
    ctx, dec, oracle = make(shape, p, B * beam, steps, 16 * B, topk)
    rng = np.random.default_rng(5)
    src, lens = sources(shape, rng, B, 1, 11)
    for attempt in range(2):                               # a second batch re-uses the decoder: caches start over
        dec.begin(src, lens, beam, n_sentences=B)
        mems = [oracle.encode(src[b, :lens[b]]) if src is not None else None for b in range(B)]
        hist = [[] for _ in range(B * beam)]
        for t in range(steps):
            prev = np.full(B * beam, shape.eos_id, np.int32) if t == 0 else rng.integers(4, shape.vocab, B * beam).astype(np.int32)
            if t == 2 and shape.cutoffs:
                prev[:] = rng.integers(4, shape.cutoffs[0], B * beam)     # a step that feeds head tokens only
            parent = None
            if t:
                parent = np.array([r // beam * beam + rng.integers(0, beam) for r in range(B * beam)], np.int32)
                if t == 3:
                    parent = None                           # identity is allowed at any step
            par = parent if parent is not None else np.arange(B * beam)
            hist = [hist[par[r]] + [int(prev[r])] for r in range(B * beam)]
            top_lp, top_id = dec.step(prev, parent)
            ref = np.stack([oracle.next_logprobs(mems[r // beam], hist[r]) for r in range(B * beam)])
            check_step(dec.logprobs(), top_lp, top_id, ref, tol)
        src, lens = sources(shape, rng, B, 2, 9)
    ctx.close()


@pytest.mark.parametrize("name,prec,tol", [("wide", "fp16", 3e-2), ("wide", "bf16", 2e-1), ("wide_dh32", "fp16", 3e-2), ("wide_dh32", "bf16", 2e-1)])
def test_steps_of_more_than_64_rows_match_the_full_decoder(name, prec, tol):
    test_steps_with_reordered_beams_match_the_full_decoder(name, prec, tol, B=16, beam=5)


@pytest.mark.parametrize("prec,tol", [("fp16", 3e-2), ("bf16", 2e-1)])
@pytest.mark.parametrize("name,B,beam", [("width_768", 16, 5), ("long_ffn", 1, 4)])
def test_contractions_long_enough_for_more_slices_than_the_next_kernel_adds(name, B, beam, prec, tol):
    """80 rows x 768 columns leave room for 10 slices of K = 3072 and 4 rows x 64 columns for 72 of K = 18432 on the tiled kernel, which must leave
    no more than the next kernel adds (a few-row product would need 9 for the latter, and is refused)."""
    test_steps_with_reordered_beams_match_the_full_decoder(name, prec, tol, B=B, beam=beam)


def test_beam_search_on_both_sides_finds_the_same_hypotheses():
    import paper_1904_01038_amd as T
    from tests.beam_search import beam_search
    shape = SHAPES["post"]
    B, beam, steps = 3, 3, 8
    ctx, dec, oracle = make(shape, T.FP32, B * beam, steps, 64, 2 * beam, seed=2)
    rng = np.random.default_rng(9)
    src, lens = sources(shape, rng, B, 3, 9)
    dec.begin(src, lens, beam)
    got = beam_search(dec.step, B, beam, steps, shape.eos_id)

    mems = [oracle.encode(src[b, :lens[b]]) for b in range(B)]
    state = {"hist": [[] for _ in range(B * beam)]}

    def oracle_step(prev, parent):
        par = parent if parent is not None else np.arange(B * beam)
        state["hist"] = [state["hist"][par[r]] + [int(prev[r])] for r in range(B * beam)]
        lp = np.empty((B * beam, 2 * beam), np.float32)
        ids = np.empty((B * beam, 2 * beam), np.int32)
        for r in range(B * beam):
            best = top_k(oracle.next_logprobs(mems[r // beam], state["hist"][r]), 2 * beam)
            lp[r], ids[r] = [v for v, _ in best], [i for _, i in best]
        return lp, ids

    want = beam_search(oracle_step, B, beam, steps, shape.eos_id)
    for s in range(B):
        assert len(got[s]) == len(want[s]) == beam
        # the best hypothesis of each side is a valid hypothesis of the other with the same score
        assert got[s][0][1] == want[s][0][1]
        for (sg, tg), (sw, tw) in zip(got[s], want[s]):
            assert abs(sg - sw) <= 1e-3
    ctx.close()


def test_decoder_argument_checks_and_limits():
    import paper_1904_01038_amd as T
    shape = SHAPES["post"]
    ctx, dec, _ = make(shape, T.FP32, 8, 3, 32, 4)
    eos = np.full(8, shape.eos_id, np.int32)
    with pytest.raises(T.TfmError) as e:
        dec.rows = 8
        dec.step(eos)                                       # no batch has been started
    assert e.value.code == -4
    src, lens = sources(shape, np.random.default_rng(0), 2, 1, 1)    # one-token sources
    with pytest.raises(T.TfmError):
        dec.begin(src, lens, 5)                             # 2 x 5 rows > 8
    with pytest.raises(T.TfmError):
        dec.begin(None, None, 4, n_sentences=2)             # the model has an encoder
    dec.begin(src, lens, 4)
    dec.step(eos)
    bad = np.arange(8, dtype=np.int32)
    bad[0] = 4                                              # row 0 cannot continue a row of the other sentence
    with pytest.raises(T.TfmError):
        dec.step(eos, bad)
    with pytest.raises(T.TfmError):
        dec.step(np.full(8, shape.vocab, np.int32))
    dec.step(eos)
    dec.step(eos)
    with pytest.raises(T.TfmError) as e:
        dec.step(eos)                                       # created for 3 steps
    assert e.value.code == -4
    with pytest.raises(T.TfmError):
        T.Decoder(ctx, 8, 10 ** 6, 32, 4)                   # more steps than the position table holds
    with pytest.raises(T.TfmError):
        T.Decoder(ctx, 8, 3, 32, 17)
    ctx.close()


def test_training_and_decoding_share_one_context():
    """A training step, an update, then decoding: the decoder sees the updated parameters."""
    import paper_1904_01038_amd as T
    from tests.test_oracle_model import small_batch
    from oracle.transformer import OracleTransformer, TrainConfig
    shape = ModelShape(1, 1, 32, 2, 64, 48)
    params = init_params(shape, 0, generic=True)
    cfg = T.make_config(shape, precision=T.FP32, max_sentences=8, max_len=16, max_tokens=64, init_loss_scale=1.0)
    ctx = T.Tfm(cfg)
    ctx.set_params(params)
    trainer = OracleTransformer(shape, params, TrainConfig(init_loss_scale=1.0, fp16_overflow=False, dynamic_scale=False))
    b = small_batch(shape, 1)
    ctx.train_step(b.src, b.tgt, b.src_lens, b.tgt_lens, sync=False)
    ctx.apply_update(1e-2, sync=False)
    trainer.train_step(b.src, b.tgt, b.src_lens, b.tgt_lens)
    trainer.apply_update(1e-2)
    dec = T.Decoder(ctx, 3, 4, 32, 4)
    dec.begin(b.src, b.src_lens, 1)
    dec.step(np.full(3, shape.eos_id, np.int32))
    oracle = DecodingOracle(shape, trainer.p)
    ref = np.stack([oracle.next_logprobs(oracle.encode(b.src[i, :b.src_lens[i]]), [shape.eos_id]) for i in range(3)])
    assert np.max(np.abs(dec.logprobs() - ref)) <= 1e-3
    stale = DecodingOracle(shape, params)
    ref0 = np.stack([stale.next_logprobs(stale.encode(b.src[i, :b.src_lens[i]]), [shape.eos_id]) for i in range(3)])
    assert np.max(np.abs(ref - ref0)) > 1e-2                # the update mattered
    ctx.close()


def test_a_batch_in_flight_is_invalidated_by_training_and_parameter_changes():
    """A decoding batch is tied to the parameters it began under: a training step, an update or a parameter write on
    the context makes the next decoding step fail with TFM_ESTATE instead of reading re-used encoder state; a new
    tfm_decoder_begin recovers.  Two decoders of one context keep their own source offsets and projected keys/values,
    so beginning a batch on one does not disturb the other."""
    import paper_1904_01038_amd as T
    from tests.test_oracle_model import small_batch
    shape = ModelShape(1, 1, 32, 2, 64, 48)
    params = init_params(shape, 0, generic=True)
    cfg = T.make_config(shape, precision=T.FP32, max_sentences=8, max_len=16, max_tokens=64, init_loss_scale=1.0)
    ctx = T.Tfm(cfg)
    ctx.set_params(params)
    oracle = DecodingOracle(shape, params)
    b = small_batch(shape, 1)
    eos3 = np.full(3, shape.eos_id, np.int32)
    dec = T.Decoder(ctx, 3, 4, 32, 4)

    def expect_estate():
        with pytest.raises(T.TfmError) as e:
            dec.step(eos3)
        assert e.value.code == -4

    dec.begin(b.src, b.src_lens, 1)
    dec.step(eos3)
    ctx.train_step(b.src, b.tgt, b.src_lens, b.tgt_lens)                      # re-uses the encoder buffers
    expect_estate()
    expect_estate()                                                           # stays refused until a new batch begins
    dec.begin(b.src, b.src_lens, 1)
    dec.step(eos3)
    ctx.apply_update(0.0)                                                     # (lr 0: the parameters keep their values)
    expect_estate()
    dec.begin(b.src, b.src_lens, 1)
    ctx.set_params({"embed": params["embed"]})
    expect_estate()

    # two decoders: the second one's batch has other sentences and lengths
    rng = np.random.default_rng(3)
    src2, lens2 = sources(shape, rng, 2, 5, 9)
    dec2 = T.Decoder(ctx, 2, 4, 32, 4)
    dec.begin(b.src, b.src_lens, 1)
    dec2.begin(src2, lens2, 1)
    dec.step(eos3)
    ref = np.stack([oracle.next_logprobs(oracle.encode(b.src[i, :b.src_lens[i]]), [shape.eos_id]) for i in range(3)])
    assert np.max(np.abs(dec.logprobs() - ref)) <= 2e-4
    dec2.step(np.full(2, shape.eos_id, np.int32))
    ref2 = np.stack([oracle.next_logprobs(oracle.encode(src2[i, :lens2[i]]), [shape.eos_id]) for i in range(2)])
    assert np.max(np.abs(dec2.logprobs() - ref2)) <= 2e-4
    ctx.close()


def test_big_model_fp16_beam4_full_size_steps():
    """The decoding benchmark's configuration (big Transformer, fp16, beam 4) at its real widths: 2 sentences x 4 rows,
    4 steps with re-ordered beams, whole distribution against the full-prefix oracle.  The row count is what a small
    decoding batch has; the GEMM, cache and attention kernels are the ones the benchmark runs."""
    import paper_1904_01038_amd as T
    from synth import PRESETS
    shape = PRESETS["big"]
    params = rounded(init_params(shape, 0), T.FP16)
    B, beam, steps, topk = 2, 4, 4, 8
    cfg = T.make_config(shape, precision=T.FP16, max_sentences=8, max_len=32, max_tokens=256, dropout=0.1)
    ctx = T.Tfm(cfg)
    ctx.set_params(params)
    dec = T.Decoder(ctx, B * beam, steps, 64, topk)
    oracle = DecodingOracle(shape, params)
    rng = np.random.default_rng(11)
    src, lens = sources(shape, rng, B, 10, 24)
    dec.begin(src, lens, beam)
    mems = [oracle.encode(src[b, :lens[b]]) for b in range(B)]
    hist = [[] for _ in range(B * beam)]
    for t in range(steps):
        prev = np.full(B * beam, shape.eos_id, np.int32) if t == 0 else zipf_ids(rng, B * beam, shape.vocab)
        parent = None if t == 0 else np.array([r // beam * beam + rng.integers(0, beam) for r in range(B * beam)], np.int32)
        par = parent if parent is not None else np.arange(B * beam)
        hist = [hist[par[r]] + [int(prev[r])] for r in range(B * beam)]
        top_lp, top_id = dec.step(prev, parent)
        ref = np.stack([oracle.next_logprobs(mems[r // beam], hist[r]) for r in range(B * beam)])
        check_step(dec.logprobs(), top_lp, top_id, ref, 3e-2)
    ctx.close()


@pytest.mark.parametrize("vocab,k,distinct,prec", [
    (4096, 16, 0, "fp16"), (4097, 1, 0, "fp16"), (4104, 8, 0, "fp32"),          # one block per row, and one value / vector more
    (300, 8, 0, "fp16"), (12290, 5, 0, "bf16"), (32808, 16, 0, "fp16"),         # a last block with fewer lanes than k
    (65536, 1, 0, "fp16"), (32769, 4, 0, "fp16"),
    (12288, 8, 40, "fp16"), (12288, 16, 1, "fp32"),                             # hundreds of equal values: nothing to filter by
    (8392704, 16, 0, "fp16")])                                                  # more lists than one block merges
def test_candidates_are_the_top_of_the_distribution(vocab, k, distinct, prec):
    """Exactly the k best of the distribution the decoder itself reports, equal values in ascending id order.  distinct: the
    embedding rows are copies of that many vectors, so that whole groups of tokens have equal scores."""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 8, 1, 8, vocab, pre_norm=1)
    params = init_params(shape, 3, generic=True)
    if distinct:
        params["embed"] = params["embed"][np.random.default_rng(0).integers(0, distinct, vocab)]
    p = {"fp32": T.FP32, "fp16": T.FP16, "bf16": T.BF16}[prec]
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=4, max_len=4, max_tokens=16))
    ctx.set_params(params)
    dec = T.Decoder(ctx, 3, 2, 1, k)
    dec.begin(None, None, 1, 3)
    top_lp, top_id = dec.step(np.full(3, shape.eos_id, np.int32))
    top_lp, top_id = dec.step(np.array([5, 6, 7], np.int32))
    lp = dec.logprobs()
    for r in range(3):
        order = np.lexsort((np.arange(vocab), -lp[r]))[:k]
        assert top_id[r].tolist() == order.tolist()
        assert np.array_equal(top_lp[r], lp[r, order])
    assert np.allclose(np.exp(lp.astype(np.float64)).sum(axis=1), 1.0, atol=1e-4)


@pytest.mark.parametrize("cutoffs,vocab,k,distinct,prec", [
    ((24,), 32, 8, 0, "fp32"), ((4,), 9, 8, 0, "fp16"),                          # fewer tokens than k in every cluster
    ((4093, 8189), 12287, 16, 0, "fp16"), ((4097, 4099), 16399, 5, 0, "bf16"),   # blocks of odd rows, one value in a last block, a cluster of two tokens
    ((5000, 13192), 21384, 8, 3, "fp16"), ((50, 60, 5000), 9096, 4, 2, "fp32"),  # equal values in and across clusters
    ((24, 600000), 1100000, 16, 0, "fp16")])                                     # more lists than one block merges
def test_candidates_of_an_adaptive_softmax_are_the_top_of_the_distribution(cutoffs, vocab, k, distinct, prec):
    """As above, and the distribution against the oracle's, within what the other decoding tests allow."""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 32, 1, 32, vocab, pre_norm=1, cutoffs=cutoffs, factor=2)
    params = init_params(shape, 3, generic=True)
    if distinct:
        for name in list(params):
            if name.startswith("embed") and not name.endswith("proj"):
                params[name] = params[name][np.random.default_rng(0).integers(0, distinct, len(params[name]))]
    p, tol = {"fp32": (T.FP32, 2e-4), "fp16": (T.FP16, 3e-2), "bf16": (T.BF16, 2e-1)}[prec]
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=4, max_len=4, max_tokens=16, label_smoothing=0.0))
    ctx.set_params(params)
    dec = T.Decoder(ctx, 3, 2, 1, k)
    dec.begin(None, None, 1, 3)
    fed = np.array([[shape.eos_id] * 3, [3, vocab - 1, cutoffs[0]]], np.int32)
    dec.step(fed[0])
    top_lp, top_id = dec.step(fed[1])
    lp = dec.logprobs()
    oracle = DecodingOracle(shape, params)
    for r in range(3):
        order = np.lexsort((np.arange(vocab), -lp[r]))[:k]
        assert np.array_equal(top_lp[r], lp[r, order])
        assert top_id[r].tolist() == order.tolist()
        assert np.max(np.abs(lp[r] - oracle.next_logprobs(None, list(fed[:, r])))) <= tol
    assert np.allclose(np.exp(lp.astype(np.float64)).sum(axis=1), 1.0, atol=2e-3)


@pytest.mark.parametrize("vocab", [60, 9000])                   # one block of a tail's scores and three
def test_candidates_whose_scores_differ_by_less_than_the_sum_resolves(vocab):
    """fp32, a tail with many more than topk scores a few units in the last place apart around 1/16, which log-probabilities of -3.6 and -9.1 do
    not tell apart: the values are the largest of the distribution, every id has the value that is returned with it, no id comes twice."""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 32, 1, 32, vocab, pre_norm=1, cutoffs=(24,), factor=2)
    params, k = init_params(shape, 3, generic=True), 8
    # the state is some 1 in every column, the head's tokens score -15, the entry of the tail 0 and its tokens around 1/16
    params["dec.ln_final.g"], params["dec.ln_final.b"] = np.full(32, 1e-2), np.ones(32)
    params["embed"][:24], params["embed"][24:] = -15.0 / 32, 0.0
    u = params["embed.1.proj"].sum(axis=0)
    params["embed.1"] = u / (u @ u) / 16 * (1.0 + np.arange(vocab - 24)[::-1, None] % 23 * 2.0 ** -23)
    ctx = T.Tfm(T.make_config(shape, precision=T.FP32, max_sentences=4, max_len=4, max_tokens=16, label_smoothing=0.0))
    ctx.set_params(params)
    dec = T.Decoder(ctx, 3, 2, 1, k)
    dec.begin(None, None, 1, 3)
    top_lp, top_id = dec.step(np.array([shape.eos_id, 3, 7], np.int32))
    lp = dec.logprobs()
    for r in range(3):
        assert top_id[r].min() >= 24 and len(set(top_id[r].tolist())) == k
        assert np.sum(lp[r] >= top_lp[r, -1]) > k                   # (there is something to choose from)
        assert np.array_equal(top_lp[r], np.sort(lp[r])[::-1][:k]) and np.array_equal(lp[r, top_id[r]], top_lp[r])


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("cutoffs,vocab", [((93, 1030), 9222), ((94, 1031), 9223), ((93, 1000, 4096), 9222)])
def test_scores_of_a_tail_do_not_depend_on_the_rows_beside_it_nor_on_other_tails(cutoffs, vocab, prec):
    """To the bit, with 1 to 8 rows: a first tail of 937 or 907 tokens must not take a second one of 8192 (8192, 3096 and 5126) tokens off the
    16-byte boundary that its matrix-core product needs, whatever rows x 937 comes to.  (The few-row kernel sums a row in the
    same order for any number of them.)"""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 256, 4, 256, vocab, pre_norm=1, cutoffs=cutoffs, factor=2)
    p = {"fp16": T.FP16, "bf16": T.BF16}[prec]
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=8, max_len=4, max_tokens=16, label_smoothing=0.0))
    ctx.set_params(init_params(shape, 3, generic=True))
    fed = np.array([shape.eos_id, 3, cutoffs[0], vocab - 1, 7, cutoffs[1], 92, 5], np.int32)
    got = {}
    for rows in (8, 5, 3, 2, 1):
        dec = T.Decoder(ctx, rows, 2, 1, 16)
        dec.begin(None, None, 1, rows)
        got[rows] = (*dec.step(fed[:rows]), dec.logprobs())
        order = [np.lexsort((np.arange(vocab), -r))[:16] for r in got[rows][2]]
        assert np.array_equal(got[rows][1], order) and np.array_equal(got[rows][0], np.take_along_axis(got[rows][2], np.array(order), 1))
        for a, b in zip(got[rows], got[8]):
            assert np.array_equal(a, b[:rows]), rows


@pytest.mark.parametrize("where", ["tail", "head"])
def test_nan_scores_of_an_adaptive_softmax_reach_every_log_probability_and_no_candidate_hides(where):
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 16, 1, 16, 9000, pre_norm=1, cutoffs=(100, 5000), factor=2)
    params = init_params(shape, 3, generic=True)
    tables = [n for n in params if n.startswith("embed") and not n.endswith("proj")]
    params[tables[0 if where == "head" else -1]][7] = np.nan
    ctx = T.Tfm(T.make_config(shape, precision=T.FP16, max_sentences=4, max_len=4, max_tokens=16, label_smoothing=0.0))
    ctx.set_params(params)
    dec = T.Decoder(ctx, 2, 2, 1, 4)
    dec.begin(None, None, 1, 2)
    top_lp, top_id = dec.step(np.full(2, shape.eos_id, np.int32))
    assert np.isnan(top_lp).all() and all(len(set(row)) == 4 for row in top_id.tolist())
    assert ((top_id >= 0) & (top_id < (5000 if where == "tail" else 9000)) & ((top_id != 7) | (where == "tail"))).all()


@pytest.mark.parametrize("prec,tol", [("fp16", 0.006), ("bf16", 0.03)])
@pytest.mark.parametrize("d,heads,rows", [(d, h, r) for d, h in ((256, 4), (400, 5), (576, 9), (784, 7), (1024, 16)) for r in (1, 8, 9, 64)]
                         + [(576, 9, 80), (1024, 16, 80)])
def test_a_sub_layers_result_is_added_to_the_residual_in_32_bits(d, heads, rows, prec, tol):
    """The attention's output projection cancels the residual down to 2e-4 of it; rounded to 2 bytes before the sum, nothing of the
    difference is left.  sqrt(d) is whole and the fed token's embedding has small whole numbers, so that the residual itself, the
    values (the bias alone) and everything but the sum are exact.  Tolerance: two logits of at most 4 rounded to 2 bytes, plus six
    standard deviations of the rounding of the two normalised states."""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, d, heads, 64, 96)
    rng = np.random.default_rng(d + rows)
    params = {k: np.zeros_like(v) if k.startswith("dec") else v for k, v in init_params(shape, 1).items()}
    root = int(round(d ** 0.5))
    params["embed"][shape.eos_id] = rng.integers(1, 5, d) * rng.choice([-1, 1], d)
    x = root * params["embed"][shape.eos_id] + np.arange(d) % 2                  # position 0: sin 0, cos 0
    params["dec.0.self.bqkv"][2 * d:] = rng.standard_normal(d)
    params["dec.0.self.wo"] = rng.standard_normal((d, d)) * 0.02 / root
    params["dec.0.self.bo"] = -x
    params["dec.0.ln_self.g"][:] = params["dec.0.ln_ffn.g"][:] = 1.0
    p = {"fp16": T.FP16, "bf16": T.BF16}[prec]
    params = rounded(params, p)
    assert np.array_equal(params["dec.0.self.bo"], -x)
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=rows, max_len=4, max_tokens=64))
    ctx.set_params(params)
    dec = T.Decoder(ctx, rows, 2, 1, 4)
    dec.begin(None, None, 1, rows)
    dec.step(np.full(rows, shape.eos_id, np.int32))
    got, ref = dec.logprobs().astype(np.float64), DecodingOracle(shape, params).next_logprobs(None, [shape.eos_id])
    assert np.max(np.abs((got[:, 5:] - got[:, 4:5]) - (ref[5:] - ref[4]))) <= tol
    ctx.close()


EDGES = (31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 130)   # where a chunk of 32 or 64 positions ends


def peaked(shape, prec, seed):
    """Parameters whose attention scores spread over several units, so that single positions matter."""
    params = init_params(shape, seed, generic=True)
    d = shape.d_model
    for k in params:
        if k.endswith("self.wqkv") and k.startswith("dec"):
            params[k][:2 * d] *= 2.5
        if k.endswith("cross.wq") or k.endswith("cross.wkv"):
            params[k][:d] *= 2.5
    return rounded(params, prec)


@pytest.mark.parametrize("prec,tol", [("fp16", 3e-2), ("bf16", 2e-1)])
@pytest.mark.parametrize("d,heads,beam,copies", [
    (128, 2, 1, 1), (128, 2, 5, 1), (128, 2, 9, 1),        # a row, the beams of a sentence (odd), or, above 8, again a row per block
    (256, 4, 5, 15), (256, 4, 9, 9)])                      # more than 2048 wavefronts: chunks of 32 positions
def test_attention_over_several_chunks_of_positions(d, heads, beam, copies, prec, tol):
    """Head width 64: histories and sources around the ends of the chunks, with re-ordered beams.  copies: how often each source
    length occurs; of many rows a sample is compared."""
    import paper_1904_01038_amd as T
    shape = ModelShape(1, 1, d, heads, 2 * d, 96)
    p = {"fp16": T.FP16, "bf16": T.BF16}[prec]
    params = peaked(shape, p, 4)
    lens = np.array([1, 31, 32, 33, 64, 65, 130] * copies, np.int32)
    B, R, steps = len(lens), len(lens) * beam, EDGES[-1]
    assert (R * heads > 2048) == (copies > 1)
    rng = np.random.default_rng(beam)
    src = rng.integers(4, shape.vocab, (B, lens.max())).astype(np.int32)
    src[np.arange(lens.max())[None, :] >= lens[:, None]] = shape.pad_id
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=B, max_len=steps, max_tokens=(int(lens.sum()) + 63) // 64 * 64))
    ctx.set_params(params)
    dec, oracle = T.Decoder(ctx, R, steps, int(lens.sum()), 4), DecodingOracle(shape, params)
    dec.begin(src, lens, beam)
    sample = np.arange(R) if R <= 64 else np.sort(rng.choice(R, 24, replace=False))
    mems = {b: oracle.encode(src[b, :lens[b]]) for b in set(sample // beam)}
    base = np.arange(R) // beam * beam
    hist = np.zeros((R, 0), np.int32)
    for t in range(steps):
        prev = np.full(R, shape.eos_id, np.int32) if t == 0 else rng.integers(4, shape.vocab, R).astype(np.int32)
        parent = None if t == 0 else (base + rng.integers(0, beam, R)).astype(np.int32)
        hist = np.concatenate([hist if parent is None else hist[parent], prev[:, None]], axis=1)
        dec.step(prev, parent)
        if t + 1 in EDGES:
            ref = np.stack([oracle.next_logprobs(mems[r // beam], hist[r]) for r in sample])
            assert np.max(np.abs(dec.logprobs()[sample] - ref)) <= tol, t + 1
    ctx.close()


@pytest.mark.parametrize("prec,tol", [("fp16", 3e-2), ("bf16", 2e-1)])
@pytest.mark.parametrize("beam", [1, 5, 9])
def test_attention_over_few_positions(prec, tol, beam):
    """Histories of 1 to 50 positions, at every step, and sources around the ends of a tile of 16 positions, with re-ordered beams."""
    import paper_1904_01038_amd as T
    shape = ModelShape(1, 1, 128, 2, 256, 96)
    p = {"fp16": T.FP16, "bf16": T.BF16}[prec]
    params = peaked(shape, p, 9)
    lens = np.array([1, 15, 16, 17, 47, 49], np.int32)
    B, R, steps = len(lens), len(lens) * beam, 50
    rng = np.random.default_rng(beam)
    src = rng.integers(4, shape.vocab, (B, lens.max())).astype(np.int32)
    src[np.arange(lens.max())[None, :] >= lens[:, None]] = shape.pad_id
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=B, max_len=steps, max_tokens=(int(lens.sum()) + 63) // 64 * 64))
    ctx.set_params(params)
    dec, oracle = T.Decoder(ctx, R, steps, int(lens.sum()), 4), DecodingOracle(shape, params)
    dec.begin(src, lens, beam)
    mems = [oracle.encode(src[b, :lens[b]]) for b in range(B)]
    base, hist = np.arange(R) // beam * beam, np.zeros((R, 0), np.int32)
    for t in range(steps):
        prev = np.full(R, shape.eos_id, np.int32) if t == 0 else rng.integers(4, shape.vocab, R).astype(np.int32)
        parent = None if t == 0 else (base + rng.integers(0, beam, R)).astype(np.int32)
        hist = np.concatenate([hist if parent is None else hist[parent], prev[:, None]], axis=1)
        dec.step(prev, parent)
        row = t % R                                        # (one row a step, each in turn)
        assert np.max(np.abs(dec.logprobs()[row] - oracle.next_logprobs(mems[row // beam], hist[row]))) <= tol, t + 1
    ctx.close()


def _thirty_steps():
    """The candidates of 30 steps of a small fp16 model, as (values, ids); the tokens fed depend on the step before."""
    import paper_1904_01038_amd as T
    shape = SHAPES["half"]
    ctx = T.Tfm(T.make_config(shape, precision=T.FP16, max_sentences=4, max_len=32, max_tokens=64))
    ctx.set_params(init_params(shape, 0, generic=True))
    dec = T.Decoder(ctx, 12, 30, 64, 4)
    rng = np.random.default_rng(1)
    src, lens = sources(shape, rng, 4, 3, 9)
    dec.begin(src, lens, 3)
    prev, out = np.full(12, shape.eos_id, np.int32), []
    for t in range(30):
        out.append(dec.step(prev, None if t == 0 else (np.arange(12) // 3 * 3 + rng.integers(0, 3, 12)).astype(np.int32)))
        prev = out[-1][1][:, t % 4].copy()
    ctx.close()
    return np.stack([v for v, _ in out]), np.stack([i for _, i in out])


def test_steps_do_not_depend_on_the_default_coherence_of_pinned_memory(tmp_path):
    """A step's kernels read tokens from, and write candidates to, pinned host memory that is used again at the next step."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = str(tmp_path / "steps.npz")
    code = ("import sys, numpy as np; sys.path.insert(0, %r); from tests.test_gpu_decode import _thirty_steps; "
            "v, i = _thirty_steps(); np.savez(%r, v=v, i=i)" % (root, out))
    subprocess.run([sys.executable, "-c", code], check=True, timeout=100, env=dict(os.environ, HIP_HOST_COHERENT="0"))
    got, (v, i) = np.load(out), _thirty_steps()
    assert np.array_equal(got["v"], v) and np.array_equal(got["i"], i)


@pytest.mark.parametrize("prec", ["fp16", "fp32"])
@pytest.mark.parametrize("vocab", [300, 4099, 32768, 40001, 65536])
@pytest.mark.parametrize("finite,nans,k", [(1, 0, 1), (1, 0, 8), (5, 0, 16), (2000, 0, 8), (20, 200, 16), (3, 200, 8), (1, -3, 8)])
def test_candidates_among_infinite_and_undefined_logits(vocab, finite, nans, k, prec):
    """`finite` tokens have finite logits, the others overflow to -infinity: those follow in ascending id order.  nans > 0: that many
    tokens side by side are NaN, nans < 0: all but that many; they are never returned, and the row's log-probabilities are NaN."""
    import paper_1904_01038_amd as T
    finite = min(finite, vocab // 2)
    shape = ModelShape(0, 1, 8, 1, 8, vocab, pre_norm=1)
    rng = np.random.default_rng(vocab + finite)
    params = {n: np.zeros_like(v) for n, v in init_params(shape, 3).items()}
    params["dec.ln_final.b"][:] = 1.0                      # the final state is all ones: a logit is the sum of its token's row
    z = np.full(vocab, -np.inf)
    ids = np.append(rng.choice(np.setdiff1d(np.arange(vocab), [shape.eos_id]), finite - 1, replace=False), shape.eos_id)
    z[ids] = 8 * rng.integers(-64, 64, finite) / 64.0      # (several equal ones among many)
    if nans:
        kept = np.concatenate([[shape.eos_id], np.arange(vocab - 2, vocab)])
        gone = np.setdiff1d(np.arange(vocab // 3, min(vocab, vocab // 3 + nans)) if nans > 0 else np.arange(vocab), kept)
        z[gone] = np.nan
    params["embed"][:] = np.where(np.isneginf(z), {"fp16": -60000.0, "fp32": -3e38}[prec], z / 8)[:, None]
    ctx = T.Tfm(T.make_config(shape, precision={"fp16": T.FP16, "fp32": T.FP32}[prec], max_sentences=4, max_len=4, max_tokens=16))
    ctx.set_params(params)
    dec = T.Decoder(ctx, 3, 2, 1, k)
    dec.begin(None, None, 1, 3)
    top_lp, top_id = dec.step(np.full(3, shape.eos_id, np.int32))
    there = np.flatnonzero(~np.isnan(z))
    want = there[np.lexsort((there, -z[there]))][:k]
    want_id = np.concatenate([want, np.full(k - len(want), 0x7fffffff)])
    lse = np.nan if nans else np.log(np.exp(z[np.isfinite(z)]).sum())
    for r in range(3):
        assert top_id[r].tolist() == want_id.tolist()
        if nans:
            assert np.isnan(top_lp[r]).all()
        else:
            assert np.array_equal(np.isneginf(top_lp[r]), np.isneginf(z[want]))
            assert np.allclose(top_lp[r][np.isfinite(z[want])], (z[want] - lse)[np.isfinite(z[want])], atol=1e-5)
    ctx.close()


@pytest.mark.parametrize("vocab", [40, 4104])
def test_more_rows_than_the_second_axis_of_a_grid_holds(vocab):
    """70000 rows: every row's candidates are those of the same row decoded in a batch of few."""
    import paper_1904_01038_amd as T
    shape = ModelShape(0, 1, 8, 1, 8, vocab, pre_norm=1)
    ctx = T.Tfm(T.make_config(shape, precision=T.FP32, max_sentences=35000, max_len=4, max_tokens=64))
    ctx.set_params(init_params(shape, 3, generic=True))
    prev = np.random.default_rng(0).integers(4, shape.vocab, 70000).astype(np.int32)
    many, few = T.Decoder(ctx, 70000, 2, 1, 3), T.Decoder(ctx, 64, 2, 1, 3)
    many.begin(None, None, 2, 35000)
    lp, ids = many.step(prev)
    for r in (0, 32768, 65472, 69936):
        few.begin(None, None, 2, 32)
        want_lp, want_id = few.step(prev[r:r + 64])
        assert np.array_equal(ids[r:r + 64], want_id) and np.array_equal(lp[r:r + 64], want_lp)
    ctx.close()


def _normed(d, heads, pre, enc, vocab=96, cutoffs=()):
    return ModelShape(enc, 2, d, heads, 2 * d, vocab, pre_norm=pre, cutoffs=cutoffs)


@pytest.mark.parametrize("prec,tol", [("fp16", 3e-2), ("bf16", 2e-1)])
@pytest.mark.parametrize("rows", [1, 3, 7, 8])
@pytest.mark.parametrize("shape", [
    _normed(72, 9, 0, 1), _normed(72, 9, 1, 0), _normed(520, 5, 1, 1), _normed(520, 5, 0, 0, 8200), _normed(1024, 16, 1, 1),
    _normed(1024, 16, 1, 0, 8200), _normed(1536, 24, 0, 1), _normed(1536, 24, 1, 0, 8200), SHAPES["adaptive_half"]],
    ids=lambda s: "d%d_%s%s_v%d" % (s.d_model, "pre" if s.pre_norm else "post", "_enc" if s.enc_layers else "", s.vocab))
def test_layernorm_inside_the_product_of_a_few_rows(shape, rows, prec, tol):
    """At most 8 rows are normalised by the product that reads them: against the oracle, and, where the other products are the same
    ones (no cross-attention, whose query is cut into slices), against a batch of 16 rows, which has a LayerNorm kernel: to the bit
    in bf16 with a small vocabulary.  In fp16 the compiler fuses some of the last multiply-adds with the conversion, not the same
    ones in both kernels, and a large vocabulary's scores of 16 rows may come from the tiled kernel: now and then a value is rounded
    the other way, which moves a logit below 8 by at most two of its steps (2^-8 and 2^-5)."""
    import paper_1904_01038_amd as T
    p = {"fp16": T.FP16, "bf16": T.BF16}[prec]
    params = rounded(init_params(shape, 7, generic=True), p)
    ctx = T.Tfm(T.make_config(shape, precision=p, max_sentences=16, max_len=32, max_tokens=256, label_smoothing=0.0 if shape.cutoffs else 0.1))
    ctx.set_params(params)
    few, many, oracle = T.Decoder(ctx, rows, 3, 64, 8), T.Decoder(ctx, 16, 3, 64, 8), DecodingOracle(shape, params)
    rng = np.random.default_rng(rows)
    src, lens = sources(shape, rng, rows, 1, 8)
    few.begin(src, lens, 1, rows)
    mems = [oracle.encode(src[r, :lens[r]]) if src is not None else None for r in range(rows)]
    fed = np.concatenate([np.full((1, 16), shape.eos_id), rng.integers(4, shape.vocab, (2, 16))]).astype(np.int32)
    same = src is None
    if same:
        many.begin(None, None, 1, 16)
    for t in range(3):
        top_lp, top_id = few.step(fed[t, :rows])
        lp = few.logprobs()
        check_step(lp, top_lp, top_id, np.stack([oracle.next_logprobs(mems[r], list(fed[:t + 1, r])) for r in range(rows)]), tol)
        if same:
            many.step(fed[t])
            assert np.max(np.abs(many.logprobs()[:rows] - lp)) <= (2 * 2.0 ** -8 if p == T.FP16 else 2 * 2.0 ** -5 if shape.vocab > 4096 else 0.0)
    ctx.close()


@pytest.mark.parametrize("heads,rows", [(1, 3), (16, 144)])                  # chunks of 64 and (more than 2048 wavefronts) of 32 positions
def test_positions_whose_score_is_minus_infinity_have_no_weight(heads, rows):
    """One token's key overflows to infinity, against which every query gives -infinity.  64 such positions, whole chunks, come first;
    the steps after them must attend to the others alone.  Tolerance: the fp16 one, and half a step each (2^-5) for a token's logit and
    for the largest, which token 5 brings up to 64-128."""
    import paper_1904_01038_amd as T
    d = 64 * heads
    shape = ModelShape(0, 1, d, heads, 64, 96)
    params = init_params(shape, 5, generic=True)
    params["embed"][5] *= 0.5
    params["embed"][5, ::64] = 3.0                                             # token 5, and no other, is large in every 64th place
    params["embed"][6:] *= 4.0
    params["embed"][6:, ::64] = 0.0
    first = np.arange(0, d, 64)                                                # the heads' first features
    params["dec.0.self.wqkv"][first] = 0.0
    params["dec.0.self.bqkv"][first] = -0.01                                   # queries: a constant
    params["dec.0.self.wqkv"][d + first] = 0.0
    params["dec.0.self.wqkv"][d + first, first] = 4000.0                       # keys: 92000 and more for token 5, at most 4000 else
    params = rounded(params, T.FP16)
    ctx = T.Tfm(T.make_config(shape, precision=T.FP16, max_sentences=rows, max_len=72, max_tokens=64))
    ctx.set_params(params)
    dec, oracle = T.Decoder(ctx, rows, 72, 1, 4), DecodingOracle(shape, params)
    dec.begin(None, None, 1, rows)
    fed = np.random.default_rng(0).integers(6, 96, (72, rows)).astype(np.int32)
    fed[:64] = 5
    for t in range(72):
        dec.step(fed[t])
        if t >= 64:
            lp = dec.logprobs()
            for r in (0, rows - 1):
                assert np.max(np.abs(lp[r] - oracle.next_logprobs(None, list(fed[:t + 1, r])))) <= 3e-2 + 2 * 2.0 ** -5
    ctx.close()
