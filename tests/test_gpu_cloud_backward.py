"""HIP path vs CPU oracle for the cloud's backward pass (cloud block of Algorithm 1: back-propagation on the public
dataset, whose gradients build the basis): zgr_cloud_backward against oracle.cloud on the same seeded parameters and batches, tensor by tensor.

Tolerances.  fp32 models: every intermediate result is fp32 on the device and fp64 in the oracle, sums run over at
most a few thousand terms, so a gradient entry differs by a few 1e-6 of the tensor's largest entry; the bound is
2e-4 of it (rounding in the softmax and LayerNorm chains is amplified by their 1 / sigma factors).  bf16 models: the
forward half keeps what the client's forward keeps, bf16-rounded activations (2^-9 relative each), and the weights
are bf16 values the oracle reads exactly; over two blocks that is a few per cent of a tensor's norm, so the test
asks for the direction (cosine >= 0.995) and the norm (within 5 %) of every matrix's gradient, not its entries."""
import numpy as np
import pytest

import zgr_inputs as I
from oracle import cloud as C

pytestmark = pytest.mark.gpu

LN_GAINS = (I.ROLE_LN1_G, I.ROLE_LN2_G, I.ROLE_LNF_G)


def _setup(cfg, scale=4.0, data_seed=0):
    """Session and oracle parameters: the seeded initial values, matrices scaled up so that attention and GELU leave
    their linear regime (the gradient rules of softmax and LayerNorm then carry weight)."""
    from tests.util import make_session
    specs = I.tensor_specs(cfg)
    values = [v if s.role in LN_GAINS else (v * scale).astype(np.float32) for s, v in zip(specs, I.make_params(cfg, data_seed, specs))]
    if cfg.dtype == "bf16":
        import torch
        values = [torch.from_numpy(v).bfloat16().float().numpy() for v in values]
    sess = make_session(cfg, specs, values, [None] * len(specs))
    P = {s.name: v.astype(np.float64) for s, v in zip(specs, values)}
    return sess, specs, P


def _batch(cfg, data_seed):
    from tests.util import make_batch_arrays
    return make_batch_arrays(cfg, data_seed)


def _oracle(cfg, P, arrays):
    if cfg.arch == I.ARCH_DECODER_LM:
        return C.lm_loss_and_gradients(P, arrays["x"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)
    return C.cls_loss_and_gradients(P, arrays["x"], arrays["lengths"], arrays["y"], cfg.n_layer, cfg.n_head, cfg.ln_eps, cfg.act, cfg.post_ln)


def _device(sess, cfg, arrays):
    from tests.util import session_batch
    loss, grads = sess.cloud_backward(session_batch(sess, cfg, arrays))
    return loss, [g.cpu().numpy().astype(np.float64) for g in grads]


TINY_LM = dict(name="bw_lm", n_layer=2, d_model=64, n_head=4, d_ff=192, vocab=211, max_pos=40, batch=3, seq=37, k=8, k_full=8)
TINY_CLS = dict(name="bw_cls", arch=I.ARCH_ENCODER_CLS, n_class=3, n_layer=2, d_model=64, n_head=2, d_ff=128, vocab=157, max_pos=48, batch=5, seq=41, k=8, k_full=8)


VARIANT_KW = {"lm_relu": dict(TINY_LM, name="bw_lm_relu", act="relu"), "cls_postln": dict(TINY_CLS, name="bw_cls_postln", post_ln=True),
              "lm_relu_postln": dict(TINY_LM, name="bw_lm_relu_postln", act="relu", post_ln=True),
              # sequences past 256 tokens: a thread of the row-wise softmax rule holds two entries of a row, the [T, T] buffers span
              # five 64-wide tiles with a ragged last one
              "lm_long": dict(TINY_LM, name="bw_lm_long", n_layer=1, d_model=32, n_head=2, d_ff=64, vocab=101, max_pos=320, batch=2, seq=300),
              "cls_long": dict(TINY_CLS, name="bw_cls_long", n_layer=1, d_model=32, n_head=2, d_ff=64, vocab=101, max_pos=320, batch=3, seq=290)}


@pytest.mark.parametrize("which", ["lm", "cls", "cfg2", "lm_relu", "cls_postln", "lm_relu_postln", "lm_long", "cls_long"])
def test_fp32_gradients_match_the_oracle_entry_by_entry(which, say):
    """The default model (pre-LayerNorm, erf-GELU) and the two switches of the paper's model families."""
    cfg = I.CONFIGS["cfg2"] if which == "cfg2" else I.shrink(I.CONFIGS["cfg2"], **(VARIANT_KW[which] if which in VARIANT_KW else TINY_LM if which == "lm" else TINY_CLS))
    sess, specs, P = _setup(cfg)
    theta_before = [sess.get_theta(i).copy() for i in range(len(specs))]
    arrays = _batch(cfg, 1)
    say(f"cloud backward fp32 {which}: {len(specs)} tensors")
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= 2e-5 * max(1.0, abs(loss_or))
    from tests.util import session_batch
    assert abs(loss - sess.loss(session_batch(sess, cfg, arrays))) <= 1e-6 * max(1.0, abs(loss_or))   # the client's own forward
    # the key bias has an identically zero gradient (softmax does not see it): what the device returns there is the
    # rounding of sums that cancel, bounded against the largest gradient entry of the model instead of its own
    floor = 1e-6 * max(np.abs(g).max() for g in grads_or.values())
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        assert grads[i].shape == want.shape, s.name
        scale = np.abs(want).max()
        err = np.abs(grads[i] - want).max()
        assert err <= 2e-4 * scale + floor, (s.name, err, scale)
        assert np.array_equal(sess.get_theta(i), theta_before[i]), s.name          # parameters untouched
    # something flows everywhere except into the key bias (softmax is invariant to it)
    assert all(np.abs(grads[i]).max() > 0 for i, s in enumerate(specs) if s.role != I.ROLE_BK)


@pytest.mark.parametrize("kw", [
    dict(d_model=32, n_head=2, d_ff=64, vocab=5, max_pos=540, batch=2, seq=530),       # a lane of the softmax rule holds nine entries of a row; each token some 200 times
    dict(d_model=1032, n_head=129, d_ff=40, vocab=67, max_pos=9, batch=1, seq=2),      # LayerNorm rows of 258 four-wide pieces, fewer rows than a block's waves
    dict(d_model=2056, n_head=257, d_ff=36, vocab=70, max_pos=7, batch=3, seq=5),      # rows past what a wave holds
    dict(d_model=24, n_head=3, d_ff=35, vocab=33, max_pos=33, batch=7, seq=33),        # odd feed-forward width: entries left over by the four-wide activation
    dict(d_model=8, n_head=1, d_ff=8, vocab=52001, max_pos=4, batch=2, seq=3),         # more logits per row than a block of the cross-entropy rule holds
    dict(d_model=64, n_head=1, d_ff=32, vocab=90, max_pos=66, batch=3, seq=33),        # head size 64: the attention rule's products over 33, 64 and 65 keys
    dict(d_model=128, n_head=2, d_ff=32, vocab=90, max_pos=66, batch=2, seq=64),
    dict(arch=I.ARCH_ENCODER_CLS, n_class=3, d_model=64, n_head=1, d_ff=32, vocab=90, max_pos=66, batch=6, seq=65),   # and with padded keys, no causal mask
], ids=lambda k: f"d{k['d_model']}h{k['n_head']}t{k['seq']}")
def test_fp32_gradients_at_the_edges_of_the_row_rules(kw):
    """Same comparison and bound as above, one block, at the sizes where the row-wise rules change form.  (The forward half of this pass takes
    attention key by key; test_gpu_attention.py has the client's attention kernels.)"""
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_LM, name="bw_rows", n_layer=1, **kw))
    sess, specs, P = _setup(cfg)
    arrays = _batch(cfg, 3)
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= 2e-5 * max(1.0, abs(loss_or))
    floor = 1e-6 * max(np.abs(g).max() for g in grads_or.values())
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        assert np.abs(grads[i] - want).max() <= 2e-4 * np.abs(want).max() + floor, s.name


# per head size: batches on either side of the line between attention's kernels and the products with [T, T] buffers (blocks of 32 rows x heads)
LONG = [(1, 257, 113, 114), (1, 1100, 29, 30), (2, 257, 28, 29), (2, 1100, 7, 8), (4, 257, 14, 15), (4, 2047, 2, 3)]


@pytest.mark.parametrize("few", [True, False], ids=["few", "many"])
@pytest.mark.parametrize("n_head,seq,few_batch,many_batch", LONG)
def test_key_bias_gradient_is_zero_but_for_rounding(n_head, seq, few_batch, many_batch, few):
    """Scores shifted by one number leave the softmax as it is, so the key bias has no gradient: what comes out is the rounding of dS and of the sums over it.  dK rows
    meet LayerNorm rows of norm sqrt(d) in Wk's gradient, so sqrt(sum |dK_j|^2) is its norm / sqrt(d); four roundings an entry of dS (scores, exponential, 1 / sum,
    dP - p dP), independent, and as much again at most for the sums, whose chains must not grow with the sequence."""
    cfg = I.shrink(I.CONFIGS["cfg2"], name="bw_sums", n_layer=1, d_model=64, n_head=n_head, d_ff=64, vocab=101, max_pos=2048, batch=few_batch if few else many_batch, seq=seq,
                   k=4, k_full=4, tokens="uniform")
    sess, specs, _ = _setup(cfg, 1.0)
    _, got = _device(sess, cfg, _batch(cfg, 0))
    g = {s.role: x for s, x in zip(specs, got)}
    assert np.linalg.norm(g[I.ROLE_BK]) <= 4.5 * 2.0 ** -24 * np.linalg.norm(g[I.ROLE_WK]) / 8
    sess.close()


@pytest.mark.parametrize("few", [True, False], ids=["few", "many"])
@pytest.mark.parametrize("dtype,arch", [("f32", "dec"), ("f32", "enc"), ("bf16", "dec"), ("bf16", "enc")])
@pytest.mark.parametrize("n_head", [1, 2, 4], ids=["head64", "head32", "head16"])
def test_attention_on_long_sequences_either_way(n_head, dtype, arch, few):
    """330 tokens (bf16 models with heads of 16 or 32 have their line from 321 on), both sides of it; products of fp32 operands as above, of bf16 ones by direction."""
    waves = 2048 if dtype == "f32" and n_head == 1 and arch == "enc" else 1024 if dtype == "f32" and n_head == 1 else 512
    batch = waves // (11 * n_head) + (0 if few else 1)
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_CLS if arch == "enc" else TINY_LM, name="bw_line", n_layer=1, d_model=64, n_head=n_head, d_ff=64, vocab=67, max_pos=332, batch=batch, seq=330, dtype=dtype))
    sess, specs, P = _setup(cfg)
    arrays = _batch(cfg, 5)
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    floor = 1e-6 * max(np.abs(g).max() for g in grads_or.values())
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        if dtype == "f32":
            assert np.abs(grads[i] - want).max() <= 2e-4 * np.abs(want).max() + floor, s.name
        elif want.ndim == 2 and s.rows > 1:
            assert (grads[i] * want).sum() >= 0.995 * np.linalg.norm(grads[i]) * np.linalg.norm(want), s.name
    sess.close()


@pytest.mark.parametrize("dtype,n_head", [("f32", 1), ("f32", 4), ("bf16", 1), ("bf16", 2), ("f32", 8)])
@pytest.mark.parametrize("arch", [I.ARCH_DECODER_LM, I.ARCH_ENCODER_CLS], ids=["dec", "enc"])
def test_workspace_of_a_batch_holds_every_smaller_one(dtype, n_head, arch):
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_CLS if arch == I.ARCH_ENCODER_CLS else TINY_LM, arch=arch, name="bw_ws", n_layer=1, d_model=64, n_head=n_head, d_ff=64, max_pos=2048,
                                             batch=64, seq=2048, dtype=dtype))
    sess, _, _ = _setup(cfg)
    need = lambda b, t: sess.lib.zgr_cloud_backward_workspace(sess.ctx, b, t)
    for t in (64, 128, 192, 256, 320, 512, 1024, 2048):            # multiples of 64: bf16 models keep one form of the products
        sizes = [need(b, t) for b in range(1, 65)]
        assert all(0 < a <= b for a, b in zip(sizes, sizes[1:])), t
    for b in (1, 5, 17, 64):
        sizes = [need(b, t) for t in range(64, 2049, 64)]
        assert all(0 < x <= y for x, y in zip(sizes, sizes[1:])), b
    sess.close()


@pytest.mark.parametrize("arch,dtype,d,ff", [(I.ARCH_ENCODER_CLS, "bf16", 256, 1024), (I.ARCH_DECODER_LM, "bf16", 128, 1024), (I.ARCH_ENCODER_CLS, "f32", 64, 64)])
def test_workspace_of_a_batch_holds_every_shorter_one(arch, dtype, d, ff):
    """Every length, not only whole ones: bf16 models keep three planes of each gradient where the token count is no multiple of 64, the transposed weights where it is."""
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_CLS if arch == I.ARCH_ENCODER_CLS else TINY_LM, arch=arch, name="bw_ws", n_layer=1, d_model=d, n_head=d // 64, d_ff=ff, max_pos=700,
                                             batch=16, seq=700, dtype=dtype))
    sess, _, _ = _setup(cfg)
    need = lambda b, t: sess.lib.zgr_cloud_backward_workspace(sess.ctx, b, t)
    for b in (1, 3, 16):
        sizes = [need(b, t) for t in range(1, 701)]
        assert all(0 < x <= y for x, y in zip(sizes, sizes[1:])), b
    for t in (1, 63, 64, 129):
        sizes = [need(b, t) for b in range(1, 130)]
        assert all(0 < x <= y for x, y in zip(sizes, sizes[1:])), t
    sess.close()


def test_a_shorter_ragged_batch_runs_in_the_room_of_a_whole_one():
    import ctypes as Ct
    import torch
    from paper_2601_12917_amd import binding as B
    from tests.util import session_batch
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_CLS, name="bw_room", dtype="bf16", d_model=256, n_head=4, d_ff=1024, max_pos=512, batch=1, seq=512))
    sess, specs, _ = _setup(cfg, scale=2.0)
    grads = [torch.zeros(s.rows, s.cols, device="cuda:0") for s in specs]
    ptrs = (Ct.c_void_p * len(grads))(*[g.data_ptr() for g in grads])
    work = torch.empty(sess.lib.zgr_cloud_backward_workspace(sess.ctx, 1, 512), dtype=torch.uint8, device="cuda:0")
    short = I.shrink(cfg, name="bw_short", seq=511)
    batch, loss = session_batch(sess, short, _batch(short, 3)), Ct.c_double()
    B.check(sess.lib.zgr_cloud_backward(sess.ctx, Ct.byref(batch), ptrs, len(grads), Ct.byref(loss), work.data_ptr(), work.numel()), sess.ctx)
    want_loss, want = sess.cloud_backward(batch)
    assert loss.value == want_loss and all(torch.equal(a.flatten(), b.flatten()) for a, b in zip(grads, want))
    sess.close()


@pytest.mark.parametrize("batch,seq,act,post_ln", [(4, 48, "gelu", False), (3, 37, "gelu", False), (4, 48, "relu", True)])
def test_bf16_gradients_point_where_the_oracle_gradients_point(batch, seq, act, post_ln, say):
    """192 tokens: the backward products run on the matrix cores; 111 tokens (not a multiple of 64): on the fp32 kernel."""
    cfg = I.shrink(I.CONFIGS["cfg3"], name="bw_bf16", n_layer=2, d_model=128, n_head=2, d_ff=256, vocab=389, max_pos=64, batch=batch, seq=seq, k=8, k_full=8,
                   act=act, post_ln=post_ln)
    sess, specs, P = _setup(cfg, scale=3.0)
    arrays = _batch(cfg, 2)
    say("cloud backward bf16 decoder")
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= 2e-2 * max(1.0, abs(loss_or))
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        if min(want.shape) == 1 and s.role == I.ROLE_BK:
            continue
        cos = float((grads[i] * want).sum() / (np.linalg.norm(grads[i]) * np.linalg.norm(want)))
        ratio = float(np.linalg.norm(grads[i]) / np.linalg.norm(want))
        assert cos >= 0.995 and abs(ratio - 1.0) <= 0.05, (s.name, cos, ratio)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name,batch", [("cfg3", 2), ("cfg5", 1)])
def test_bf16_gradients_at_the_size_of_a_real_model(name, batch, say):
    """cfg3 (12 blocks of d = 768) on two of its sequences and cfg5 (24 blocks of d = 2048, the benchmark's model) on one,
    both with the 50272-word vocabulary: every tensor's gradient against the oracle's.  The blocks' bf16-rounded
    activations leave a few per cent: direction and norm are what is asked."""
    cfg = I.shrink(I.CONFIGS[name], name="bw_" + name, batch=batch)
    sess, specs, P = _setup(cfg, scale=1.0)
    arrays = _batch(cfg, 0)
    say(f"cloud backward at {name}, {batch} sequence(s): device")
    loss, grads = _device(sess, cfg, arrays)
    say(f"cloud backward at {name}, {batch} sequence(s): oracle")
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= 1e-2 * abs(loss_or)
    worst = (1.0, None)
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        if s.role == I.ROLE_BK:
            continue
        cos = float((grads[i] * want).sum() / (np.linalg.norm(grads[i]) * np.linalg.norm(want)))
        ratio = float(np.linalg.norm(grads[i]) / np.linalg.norm(want))
        worst = min(worst, (cos, s.name))
        assert cos >= 0.99 and abs(ratio - 1.0) <= 0.05, (s.name, cos, ratio)
    say(f"worst cosine {worst[0]:.5f} at {worst[1]}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_two_runs_agree_bit_for_bit(dtype):
    """No sum of the backward pass depends on scheduling: the same call twice gives the same bits."""
    from tests.util import session_batch
    cfg = I.shrink(I.CONFIGS["cfg3"], name="bw_det", dtype=dtype, n_layer=2, d_model=128, n_head=2, d_ff=256, vocab=389, max_pos=64, batch=4, seq=64, k=8, k_full=8)
    sess, specs, P = _setup(cfg, scale=3.0)
    batch = session_batch(sess, cfg, _batch(cfg, 5))
    l1, g1 = sess.cloud_backward(batch)
    l2, g2 = sess.cloud_backward(batch)
    assert l1 == l2
    for a, b, s_ in zip(g1, g2, specs):
        assert bool((a == b).all()), s_.name


@pytest.mark.parametrize("kw", [
    dict(dtype="bf16", n_layer=8, d_model=64, n_head=1, d_ff=64, batch=4, seq=16),                       # ten sums a block: more than 64 of them
    dict(dtype="bf16", n_layer=8, d_model=64, n_head=1, d_ff=128, batch=4, seq=16, post_ln=True, act="relu"),
    dict(dtype="f32", n_layer=4, d_model=2048, n_head=32, d_ff=64, batch=64, seq=16),                    # few sums, whose chunks fill the arena (2^23 floats)
], ids=["jobs", "jobs post-LN", "room"])
def test_sums_over_rows_of_more_blocks_than_are_kept_back(kw):
    """Bias and LayerNorm gradients of every block where their chunk sums are added up in the middle of the pass and the space used again."""
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_LM, name="bw_sums_kept", vocab=37, max_pos=16, **kw))
    sess, specs, P = _setup(cfg, scale=2.0)
    arrays = _batch(cfg, 4)
    _, grads = _device(sess, cfg, arrays)
    _, want = _oracle(cfg, P, arrays)
    floor = 1e-6 * max(np.abs(g).max() for g in want.values())
    for g, s in zip(grads, specs):
        w = want[s.name]
        if s.rows > 1 or s.role == I.ROLE_BK:
            continue
        if cfg.dtype == "f32":
            assert np.abs(g - w).max() <= 2e-4 * np.abs(w).max() + floor, s.name
        else:
            assert (g * w).sum() >= 0.99 * np.linalg.norm(g) * np.linalg.norm(w) and abs(np.linalg.norm(g) / np.linalg.norm(w) - 1) <= 0.1, s.name
    sess.close()


def test_workspace_of_a_small_model_is_small():
    """Nothing in it is sized for large models: 3 x 37 tokens of a 2-block, 64-wide decoder, where split sums (4.3 MB) take the most."""
    sess, _, _ = _setup(I.shrink(I.CONFIGS["cfg2"], **TINY_LM))
    assert 0 < sess.lib.zgr_cloud_backward_workspace(sess.ctx, 3, 37) <= 6 << 20
    sess.close()


@pytest.mark.parametrize("dtype,d,n_head,batch,seq", [("f32", 768, 12, 4, 128), ("f32", 512, 8, 1, 2048), ("bf16", 512, 8, 1, 2047), ("bf16", 512, 8, 4, 128), ("f32", 40, 5, 2, 19)])
def test_gradients_do_not_depend_on_where_they_are_written(dtype, d, n_head, batch, seq):
    """Adjacent gradients of Wq, Wk, Wv (and of their biases) are one product: the sums take the order of three all the same.  (Undivided sums in one launch; parts that the
    scratch has no room for all at once; bf16 operands.)"""
    import ctypes
    import torch
    cfg = I.shrink(I.CONFIGS["cfg2"], name="bw_places", n_layer=1, d_model=d, n_head=n_head, d_ff=64, vocab=101, max_pos=2048, batch=batch, seq=seq, k=4, k_full=4, dtype=dtype)
    from tests.util import session_batch
    sess, specs, _ = _setup(cfg)
    b = session_batch(sess, cfg, _batch(cfg, 0))
    need = sess.lib.zgr_cloud_backward_workspace(sess.ctx, batch, seq)
    work, out = torch.empty(need, dtype=torch.uint8, device="cuda"), []
    for gap in (0, 64):
        at = np.cumsum([0] + [s.numel + gap for s in specs])
        slab, loss = torch.zeros(int(at[-1]), device="cuda"), ctypes.c_double()
        ptrs = (ctypes.c_void_p * len(specs))(*[slab.data_ptr() + 4 * int(a) for a in at[:-1]])
        assert sess.lib.zgr_cloud_backward(sess.ctx, ctypes.byref(b), ptrs, len(specs), ctypes.byref(loss), work.data_ptr(), need) == 0
        out.append([slab[int(a):int(a) + s.numel].clone() for a, s in zip(at, specs)])
    for x, y, s in zip(*out, specs):
        assert torch.equal(x, y), s.name
    sess.close()


def test_lsq_gradient_through_the_same_entry_point():
    cfg = I.CONFIGS["cfg1"]
    sess, specs, P = _setup(cfg, scale=1.0)
    arrays = _batch(cfg, 0)
    loss, grads = _device(sess, cfg, arrays)
    want = C.lsq_gradient(P[specs[0].name], arrays["x"], arrays["y"])
    assert np.abs(grads[0] - want).max() <= 1e-5 * np.abs(want).max()
    from tests.util import oracle_loss_fn
    assert abs(loss - oracle_loss_fn(cfg, arrays)({"W": P[specs[0].name]})) <= 1e-5 * abs(loss)


def test_descent_along_the_device_gradient_lowers_the_loss():
    """What a gradient is for: theta - lr dL/dtheta has a lower loss, by about lr |dL/dtheta|^2 for a small step."""
    from tests.util import oracle_loss_fn
    cfg = I.shrink(I.CONFIGS["cfg2"], **TINY_LM)
    sess, specs, P = _setup(cfg)
    arrays = _batch(cfg, 3)
    loss, grads = _device(sess, cfg, arrays)
    g2 = sum(float((g * g).sum()) for g in grads)
    lr = 1e-3 / np.sqrt(g2)
    loss_fn = oracle_loss_fn(cfg, arrays)
    stepped = {s.name: P[s.name] - lr * grads[i] for i, s in enumerate(specs)}
    drop = loss_fn(P) - loss_fn(stepped)
    assert abs(drop - lr * g2) <= 0.05 * lr * g2, (drop, lr * g2)


def test_gradient_agrees_with_the_clients_own_directional_estimate(say):
    """At a size the oracle does not reach: along the client's perturbation Z of a step, the two-point estimate of
    Eq. (11), (L(W + h Z) - L(W - h Z)) / 2h from the client's forward, is the directional derivative <dL/dW, Z> up
    to O(h^2); Z itself is read back as (W + h Z - W) / h."""
    from tests.util import session_batch
    cfg = I.shrink(I.CONFIGS["cfg2"], name="bw_mid", n_layer=4, d_model=256, n_head=4, d_ff=1024, vocab=4096, max_pos=128, batch=4, seq=128, k=8, k_full=8)
    sess, specs, P = _setup(cfg, scale=2.0)
    batch = session_batch(sess, cfg, _batch(cfg, 4))
    say("cloud backward, 4 blocks of d = 256")
    loss, grads = sess.cloud_backward(batch)
    h, step = 2e-3, 7
    before = [sess.get_theta(i).astype(np.float64) for i in range(len(specs))]
    sess.perturb(step, h)
    lp = sess.loss(batch)
    dot = sum(float((g.cpu().numpy().astype(np.float64) * ((sess.get_theta(i).astype(np.float64) - before[i]) / h)).sum()) for i, g in enumerate(grads))
    sess.perturb(step, -2.0 * h)
    lm = sess.loss(batch)
    sess.perturb(step, h)
    est = (lp - lm) / (2.0 * h)
    assert abs(loss - 0.5 * (lp + lm)) <= 1e-3 * loss
    assert abs(est - dot) <= 2e-2 * abs(dot) + 1e-3, (est, dot)


def test_basis_from_device_gradients_captures_what_the_oracle_basis_captures():
    """The cloud block end to end on the device: three backward passes give the snapshots of a matrix, zgr_cloud_basis
    their basis; it must capture as much of the ORACLE's gradients as the oracle's own basis does."""
    from paper_2601_12917_amd.session import cloud_basis
    cfg = I.shrink(I.CONFIGS["cfg2"], **TINY_LM)
    sess, specs, P = _setup(cfg, scale=8.0)
    dev, ora = [], []
    for b in range(3):
        arrays = _batch(cfg, 10 + b)
        dev.append(_device(sess, cfg, arrays)[1])
        ora.append(_oracle(cfg, P, arrays)[1])
    k = cfg.k
    for name in ("l0.wq", "l1.w1", "l1.w2", "l0.wo"):
        i = [s.name for s in specs].index(name)
        snaps_dev = [g[i].astype(np.float32) for g in dev]
        snaps_or = [g[name] for g in ora]
        omega = np.random.default_rng(5).standard_normal((snaps_dev[0].shape[1], k)).astype(np.float32)
        U, dep = cloud_basis(snaps_dev, k, omega, 40)
        assert dep == 0
        U0, _ = C.gradient_basis(snaps_or, k)
        assert C.captured_energy(U[:, :k], snaps_or) >= C.captured_energy(U0, snaps_or) * (1.0 - 1e-3), name


def test_argument_errors_are_reported_not_executed():
    import ctypes as Ct
    from paper_2601_12917_amd import binding as B
    from tests.util import session_batch
    cfg = I.shrink(I.CONFIGS["cfg2"], **TINY_LM)
    sess, specs, P = _setup(cfg)
    lib = sess.lib
    batch = session_batch(sess, cfg, _batch(cfg, 0))
    need = lib.zgr_cloud_backward_workspace(sess.ctx, cfg.batch, cfg.seq)
    assert need > 0 and lib.zgr_cloud_backward_workspace(sess.ctx, 0, cfg.seq) == 0
    import torch
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    grads = [torch.empty(*v.shape, dtype=torch.float32, device="cuda:0") for v in P.values()]
    ptrs = (Ct.c_void_p * len(grads))(*[g.data_ptr() for g in grads])
    v = Ct.c_double()
    assert lib.zgr_cloud_backward(sess.ctx, Ct.byref(batch), ptrs, len(grads) - 1, Ct.byref(v), ws.data_ptr(), need) == B.ZGR_ERR_SHAPE
    assert lib.zgr_cloud_backward(sess.ctx, Ct.byref(batch), ptrs, len(grads), Ct.byref(v), ws.data_ptr(), need - 256) == B.ZGR_ERR_WORKSPACE
    assert lib.zgr_cloud_backward(sess.ctx, Ct.byref(batch), ptrs, len(grads), Ct.byref(v), ws.data_ptr() + 64, need) == B.ZGR_ERR_WORKSPACE
    ptrs[3] = None
    assert lib.zgr_cloud_backward(sess.ctx, Ct.byref(batch), ptrs, len(grads), Ct.byref(v), ws.data_ptr(), need) == B.ZGR_ERR_NULL


@pytest.mark.parametrize("dtype,d,n_head,ff,batch,seq", [
    ("f32", 128, 2, 2048, 1, 33),      # FC1's sum in two parts
    ("f32", 704, 11, 5120, 2, 19),     # in several, rows of 704; Q, K, V's in two
    ("bf16", 128, 2, 2048, 1, 33),     # four parts, all requested at once
    ("bf16", 576, 9, 4608, 1, 70),     # nine of FC1's, three of Q, K, V's
    ("bf16", 1088, 17, 2048, 1, 31),   # wide rows, where they are requested one by one; the weight gradients' third tile size
    ("bf16", 512, 8, 4096, 9, 64),     # whole k-tiles of tokens: slices of the products on bf16 operands, three of FC1's and four of the head's
])
def test_layernorm_adds_the_parts_of_a_split_product(dtype, d, n_head, ff, batch, seq):
    """Long sums over few rows: the products in front of the LayerNorm rules leave parts.  Bounds as above."""
    cfg = I.shrink(I.CONFIGS["cfg3"], name="bw_parts", dtype=dtype, n_layer=2, d_model=d, n_head=n_head, d_ff=ff, vocab=6001 if batch * seq % 64 == 0 else 203, max_pos=80, batch=batch, seq=seq, k=8, k_full=8)
    sess, specs, P = _setup(cfg, scale=2.0)
    arrays = _batch(cfg, 3)
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= (1e-4 if dtype == "f32" else 2e-2) * max(1.0, abs(loss_or))
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        if s.role == I.ROLE_BK:
            continue
        if dtype == "f32":
            assert np.abs(grads[i] - want).max() <= 2e-4 * np.abs(want).max(), s.name
        else:
            cos = float((grads[i] * want).sum() / (np.linalg.norm(grads[i]) * np.linalg.norm(want)))
            ratio = float(np.linalg.norm(grads[i]) / np.linalg.norm(want))
            assert cos >= 0.995 and abs(ratio - 1.0) <= 0.05, (s.name, cos, ratio)
    sess.close()


@pytest.mark.parametrize("vocab,d,seq,batch", [(4, 8, 530, 3), (1500, 520, 257, 4), (3, 16, 15, 1)])
def test_embedding_rows_of_frequent_and_of_rare_tokens(vocab, d, seq, batch):
    """Rows of a token are listed 1024 tokens at a time and requested sixteen at a time: lists over two pieces, lists of one row, and fewer rows
    than one request; 520 columns take a second block.  Bounds as above."""
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_LM, name="bw_embed", n_layer=1, d_model=d, n_head=d // 8, d_ff=16, vocab=vocab, max_pos=540, batch=batch, seq=seq))
    sess, specs, P = _setup(cfg)
    arrays = _batch(cfg, 3)
    _, grads = _device(sess, cfg, arrays)
    _, grads_or = _oracle(cfg, P, arrays)
    floor = 1e-6 * max(np.abs(g).max() for g in grads_or.values())
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        assert np.abs(grads[i] - want).max() <= 2e-4 * np.abs(want).max() + floor, s.name
    sess.close()


@pytest.mark.parametrize("batch,seq,d,ff,act,post_ln", [(5, 307, 64, 128, "gelu", False), (29, 53, 64, 128, "gelu", False), (2, 1025, 64, 64, "relu", False), (41, 50, 128, 256, "relu", True)])
def test_ragged_counts_on_either_side_of_the_planes(batch, seq, d, ff, act, post_ln):
    """1535, 1537 and 2050 tokens: the last count whose weight gradients are taken on planes, and counts that take them on fp32 gradients as they lie.  Bounds as above."""
    cfg = I.shrink(I.CONFIGS["cfg2"], **dict(TINY_CLS, name="bw_long_ragged", dtype="bf16", n_layer=1, d_model=d, n_head=d // 32, d_ff=ff, max_pos=2050, batch=batch, seq=seq, act=act, post_ln=post_ln))
    sess, specs, P = _setup(cfg, scale=2.0)
    arrays = _batch(cfg, 3)
    loss, grads = _device(sess, cfg, arrays)
    loss_or, grads_or = _oracle(cfg, P, arrays)
    assert abs(loss - loss_or) <= 2e-2 * max(1.0, abs(loss_or))
    for i, s in enumerate(specs):
        want = grads_or[s.name]
        if s.role == I.ROLE_BK or not want.any():
            continue
        cos = float((grads[i] * want).sum() / (np.linalg.norm(grads[i]) * np.linalg.norm(want)))
        ratio = float(np.linalg.norm(grads[i]) / np.linalg.norm(want))
        assert cos >= 0.995 and abs(ratio - 1.0) <= 0.05, (s.name, cos, ratio)
    sess.close()
