"""Client forward passes (Session.loss, row losses) through the attention kernels at the edges of their blocks of 32 queries and keys."""
import numpy as np
import pytest

import zgr_inputs as I
from tests.util import inputs_of, make_batch_arrays, make_session, session_batch

pytestmark = pytest.mark.gpu


def _model(arch, dtype, head, batch, seq, **kw):
    n_head = max(1, 64 // head) if dtype == "bf16" else 2
    base = dict(name="attention", arch=arch, dtype=dtype, n_class=3 if arch == I.ARCH_ENCODER_CLS else 0, n_layer=2, d_model=head * n_head, n_head=n_head,
                d_ff=128, vocab=307, max_pos=seq + 3, batch=batch, seq=seq, k=4, k_full=4, tokens="uniform")
    return I.shrink(I.CONFIGS["cfg2"], **dict(base, **kw))


LN_GAINS = (I.ROLE_LN1_G, I.ROLE_LN2_G, I.ROLE_LNF_G)


def _check_row_losses(cfg, lengths=None):
    """Row losses of one client forward against the oracle's, matrices scaled up so that the softmax is far from uniform.  fp32: a few hundred
    roundings of 2^-24 through two blocks, amplified by the 1 / sigma of the LayerNorms; bf16: the tolerance of the step tests."""
    from oracle import forward as F
    from tests.test_gpu_step import LOSS_RTOL
    specs, values, bases = inputs_of(cfg)
    values = [v if s.role in LN_GAINS else v * np.float32(4) for s, v in zip(specs, values)]
    arrays = make_batch_arrays(cfg)
    if lengths is not None:
        arrays["lengths"] = np.asarray(lengths, dtype=np.int32)
    sess = make_session(cfg, specs, values, bases)
    sess.loss(session_batch(sess, cfg, arrays))
    P = {s.name: sess.get_theta(i).astype(np.float64).reshape(s.rows, s.cols) for i, s in enumerate(specs)}
    if cfg.arch == I.ARCH_DECODER_LM:
        got = sess.last_row_losses(cfg.batch * cfg.seq).reshape(cfg.batch, cfg.seq)
        assert np.all(got[:, -1] == 0)
        got = got[:, :-1]
        want = F.lm_token_losses(P, arrays["x"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
    else:
        got = sess.last_row_losses(cfg.batch)
        want = F.cls_row_losses(P, arrays["x"], arrays["lengths"], arrays["y"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
    sess.close()
    tol = 2e-5 if cfg.dtype == "f32" else LOSS_RTOL["bf16"]
    assert np.abs(got - want).max() <= tol * np.abs(want).max(), np.abs(got - want).max() / np.abs(want).max()


@pytest.mark.parametrize("seq", [1 + 1, 31, 32, 33, 64, 65, 77, 128])
@pytest.mark.parametrize("dtype,head", [("f32", 8), ("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 8), ("bf16", 16), ("bf16", 32)])
def test_decoder_rows_at_the_edges_of_the_attention_blocks(dtype, head, seq):
    _check_row_losses(_model(I.ARCH_DECODER_LM, dtype, head, 3, seq))


@pytest.mark.parametrize("seq,lengths", [(33, [1, 31, 32, 33]), (64, [32, 33, 63, 64]), (65, [1, 32, 64, 65]), (77, [33, 64, 65, 77]), (100, [96, 97, 2, 100])])
@pytest.mark.parametrize("dtype,head", [("f32", 8), ("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 8), ("bf16", 16), ("bf16", 32)])
def test_encoder_rows_with_lengths_inside_and_at_the_edges_of_key_blocks(dtype, head, seq, lengths):
    _check_row_losses(_model(I.ARCH_ENCODER_CLS, dtype, head, len(lengths), seq), lengths)


@pytest.mark.parametrize("seq", [2, 33, 63, 64, 65, 127, 128, 129, 160, 255, 256, 257, 384, 385])
@pytest.mark.parametrize("arch", [I.ARCH_DECODER_LM, I.ARCH_ENCODER_CLS], ids=["decoder", "encoder"])
def test_heads_of_64_in_bf16_at_the_edges_of_the_key_stages(arch, seq):
    """Keys arrive in stages of 64 (up to 128 tokens) or 128: sequences and padding lengths that end inside, at and just behind one."""
    _check_row_losses(_model(arch, "bf16", 64, 4, seq), [max(1, seq // 2), max(1, min(seq, 64)), max(1, seq - 1), seq] if arch == I.ARCH_ENCODER_CLS else None)


@pytest.mark.parametrize("arch", [I.ARCH_DECODER_LM, I.ARCH_ENCODER_CLS], ids=["decoder", "encoder"])
@pytest.mark.parametrize("act,post_ln", [("gelu", False), ("relu", True)])
@pytest.mark.parametrize("batch,seq,d_ff", [(1, 29, 2048), (3, 21, 2052), (2, 64, 4096)])
def test_long_feed_forward_sums_split_over_blocks(arch, act, post_ln, batch, seq, d_ff):
    """fp32 projections back from a feed-forward width of 2048 and more: the sum is split over blocks and its parts lie in an activation
    buffer that the pass has no use for at that moment."""
    _check_row_losses(_model(arch, "f32", 32, batch, seq, d_model=96, n_head=3, d_ff=d_ff, act=act, post_ln=post_ln))


@pytest.mark.parametrize("dtype,head,batch,seq", [
    ("f32", 8, 2, 20), ("f32", 16, 2, 33), ("f32", 32, 1, 64), ("f32", 64, 2, 45), ("f32", 64, 1, 96),
    ("bf16", 8, 2, 40), ("bf16", 16, 2, 40), ("bf16", 32, 1, 71)])
def test_a_query_does_not_see_what_a_later_position_holds(dtype, head, batch, seq):
    """Causal mask: a position whose activations are not finite leaves the losses of earlier ones as they are, bit for bit, and with
    them the whole loss when it is the last position, which carries no target."""
    from paper_2601_12917_amd import binding as B
    cfg = _model(I.ARCH_DECODER_LM, dtype, head, batch, seq)
    specs, values, bases = inputs_of(cfg)
    sess = make_session(cfg, specs, values, bases)
    b = session_batch(sess, cfg, make_batch_arrays(cfg))
    pos = next(i for i, s in enumerate(specs) if s.role == I.ROLE_POS_EMB)
    clean = sess.loss(b)
    rows = sess.last_row_losses(batch * seq).reshape(batch, seq)
    for p in sorted({seq - 1, seq - 2, seq // 2, 1}):
        for bad in (np.inf, np.nan):
            wild = np.array(values[pos], dtype=np.float32)
            wild[p, 3] = bad
            sess.set_theta(pos, wild)
            if p == seq - 1:
                assert sess.loss(b) == clean
            else:
                with pytest.raises(B.ZgrError) as e:
                    sess.loss(b)
                assert e.value.status == B.ZGR_ERR_NONFINITE
            got = sess.last_row_losses(batch * seq).reshape(batch, seq)
            assert np.array_equal(got[:, :p], rows[:, :p]), (p, bad)
            assert np.all(np.isnan(got[:, p:seq - 1])), (p, bad)
    sess.close()


@pytest.mark.parametrize("dtype,seq,batch,heads", [("f32", 1030, 32, 6), ("f32", 1024, 36, 6), ("bf16", 70, 5, 8), ("bf16", 33, 40, 8)])
def test_heads_of_eight_by_either_kernel(dtype, seq, batch, heads):
    """Heads of 8 take one of two kernels by storage type, mask, length and how many there are: a sequence's loss is the same alone and among
    others (the sums run in another order: 2^-24 per term of a few hundred, amplified by 1 / sigma of two LayerNorms), and the oracle's."""
    from oracle import forward as F
    from tests.test_gpu_step import LOSS_RTOL
    cfg = _model(I.ARCH_ENCODER_CLS, dtype, 8, batch, seq, n_layer=1, d_model=8 * heads, n_head=heads, d_ff=64)
    specs, values, bases = inputs_of(cfg)
    arrays = make_batch_arrays(cfg)
    sess = make_session(cfg, specs, values, bases)
    sess.loss(session_batch(sess, cfg, arrays))
    together = sess.last_row_losses(batch)
    P = {s.name: np.asarray(v, dtype=np.float64) for s, v in zip(specs, values)}
    for i in (0, batch // 2, batch - 1):
        one = {k: v[i:i + 1] for k, v in arrays.items()}
        alone = sess.loss(sess.make_batch(one["x"], one["y"], one["lengths"], seq))
        want = F.cls_loss(P, one["x"], one["lengths"], one["y"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
        assert abs(alone - together[i]) <= (1e-5 if dtype == "f32" else 0.0) * abs(alone), (i, alone, together[i])
        assert abs(alone - want) <= LOSS_RTOL[dtype] * abs(want), (i, alone, want)
    sess.close()


@pytest.mark.parametrize("vocab", [2, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 51200, 51201])
def test_row_losses_at_the_edges_of_the_cross_entropy_forms(vocab):
    """fp32 logits: each row's loss against the oracle's at vocabularies where the block or the number of entries it holds changes
    (sums of `vocab` exponentials in fp32: 2^-24 sqrt(vocab) of the loss at most, and a few roundings of the model's own)."""
    from oracle import forward as F
    cfg = _model(I.ARCH_DECODER_LM, "f32", 8, 2, 5, n_layer=1, d_model=16, n_head=2, d_ff=32, vocab=vocab)
    specs, values, bases = inputs_of(cfg)
    values = [v * np.float32(20) if s.role == I.ROLE_TOK_EMB else v for s, v in zip(specs, values)]          # logits of a few units
    arrays = make_batch_arrays(cfg)
    sess = make_session(cfg, specs, values, bases)
    sess.loss(session_batch(sess, cfg, arrays))
    got = sess.last_row_losses(10).reshape(2, 5)
    want = F.lm_token_losses({s.name: np.asarray(v, dtype=np.float64) for s, v in zip(specs, values)}, arrays["x"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
    assert np.all(got[:, 4] == 0)
    assert np.abs(got[:, :4] - want.reshape(2, 4)).max() <= (2.0 ** -24 * np.sqrt(vocab) + 4e-6) * np.abs(want).max()
    sess.close()


@pytest.mark.parametrize("vocab,batch,seq", [(307, 1, 2), (1000, 1, 64), (1025, 1, 65), (127, 2, 64), (4000, 1, 128), (300, 1, 129), (129, 3, 43)])
def test_bf16_row_losses_of_short_prompts(vocab, batch, seq):
    """The vocabulary product on tiles for up to 64, up to 128 and more tokens, vocabularies on either side of a tile of 128."""
    from oracle import forward as F
    from tests.test_gpu_step import LOSS_RTOL
    cfg = _model(I.ARCH_DECODER_LM, "bf16", 64, batch, seq, n_layer=1, d_model=128, n_head=2, vocab=vocab)
    specs, values, bases = inputs_of(cfg)
    arrays = make_batch_arrays(cfg)
    sess = make_session(cfg, specs, values, bases)
    sess.loss(session_batch(sess, cfg, arrays))
    got = sess.last_row_losses(batch * seq).reshape(batch, seq)
    P = {s.name: sess.get_theta(i).astype(np.float64) for i, s in enumerate(specs)}
    want = F.lm_token_losses(P, arrays["x"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
    assert np.all(got[:, -1] == 0)
    assert np.abs(got[:, :-1] - want).max() <= LOSS_RTOL["bf16"] * np.abs(want).max()
    sess.close()
