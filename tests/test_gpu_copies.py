"""zgr_step with room for two copies of the parameters (Z generated once for both forward passes and the restoration) against
the same step with the smallest workspace, where the three perturbations are applied in place one after the other: the
parameters and the losses come out the same bit for bit, and a loss of the perturbed parameters is the step's."""
import numpy as np
import pytest

import zgr_inputs as I
from paper_2601_12917_amd import binding as B
from paper_2601_12917_amd.session import ParamSpec, Session
from tests.util import inputs_of, make_batch_arrays, make_session, session_batch

pytestmark = pytest.mark.gpu

_SMALL = dict(n_layer=3, vocab=211, max_pos=40, batch=3, seq=17)
CASES = {
    # few tiles: blocks of 8 rows, a column strip that ends early, a rank below the matrix-core kernel's
    "linear": (I.shrink(I.CONFIGS["cfg1"], lsq_out=37, lsq_in=132, batch=5), 32),
    "f32 rank 5": (I.shrink(I.CONFIGS["cfg2"], d_model=96, n_head=3, d_ff=200, k=5, k_full=9, **_SMALL), 32),
    # matrix-core kernel: whole and ragged tiles, both group sizes, both types
    "f32 rank 20": (I.shrink(I.CONFIGS["cfg2"], d_model=160, n_head=5, d_ff=328, k=20, k_full=20, **_SMALL), 16),
    # both models' projections on the bf16 instructions' planes (160 tiles of 64 x 64 at K = 256)
    "f32 planes": (I.shrink(I.CONFIGS["cfg2"], d_model=256, n_head=4, d_ff=1024, k=16, k_full=16, n_layer=2, vocab=900, max_pos=40, batch=8, seq=40), 32),
    "bf16 rank 16": (I.shrink(I.CONFIGS["cfg3"], d_model=256, n_head=4, d_ff=576, k=16, k_full=24, **_SMALL), 32),
    "bf16 rank 16 by 8": (I.shrink(I.CONFIGS["cfg3"], d_model=256, n_head=4, d_ff=576, k=16, k_full=16, **_SMALL), 16),
    "bf16 many tiles": (I.shrink(I.CONFIGS["cfg3"], d_model=512, n_head=8, d_ff=1088, k=8, k_full=8, **_SMALL), 32),
    # sizes at which two models' tiles would cross a line of the fp32 projections that one's don't, sums split over blocks, and heads of 8
    "f32 two products": (I.shrink(I.CONFIGS["cfg2"], d_model=96, n_head=12, d_ff=4096, k=4, k_full=4, n_layer=1, vocab=300, max_pos=40, batch=1, seq=29), 32),
    "f32 shared": (I.shrink(I.CONFIGS["cfg2"], d_model=256, n_head=4, d_ff=768, k=4, k_full=4, n_layer=1, vocab=4500, max_pos=70, batch=16, seq=64), 32),
    "f32 wide": (I.shrink(I.CONFIGS["cfg2"], d_model=768, n_head=12, d_ff=3072, k=4, k_full=4, n_layer=1, vocab=3000, max_pos=40, batch=2, seq=33), 32),
    "f32 odd": (I.shrink(I.CONFIGS["cfg2"], d_model=72, n_head=9, d_ff=140, k=4, k_full=4, n_layer=2, vocab=300, max_pos=40, batch=7, seq=31), 32),
    "encoder post-LN": (I.shrink(I.CONFIGS["cfg4"], d_model=128, n_head=2, d_ff=192, k=16, k_full=16, post_ln=True, act="relu", **_SMALL), 32),
}


def _sessions(monkeypatch, cfg, bits, fuse_lr=None, stream=False, shares=(0.25, 0.0)):
    specs, values, bases = inputs_of(cfg)
    arrays = make_batch_arrays(cfg)
    out = []
    for share in shares:
        monkeypatch.setattr(Session, "COPIES_SHARE", share)
        sess = make_session(cfg, specs, values, bases, bits=bits, fuse_lr=fuse_lr)
        if stream:
            sess.set_stage_tiles(1)
            for i, u in enumerate(bases):
                if u is not None:
                    sess.set_basis_host(i, u, cfg.k)
        out.append((sess, session_batch(sess, cfg, arrays)))
    assert out[0][0].workspace.numel() > out[1][0].workspace.numel()
    return out


@pytest.mark.parametrize("stream", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_step_with_copies_equals_step_in_place(monkeypatch, name, stream):
    cfg, bits = CASES[name]
    (a, ba), (b, bb), (c, bc) = _sessions(monkeypatch, cfg, bits, stream=stream, shares=(0.25, 0.0, 0.25))
    for step in range(2):
        ra, rb = a.step(step, ba), b.step(step, bb)
        assert ra == rb
        c.perturb(step, cfg.eps)                          # the step by hand
        assert c.loss(bc) == ra[0]
        c.perturb(step, -2 * np.float32(cfg.eps))
        assert c.loss(bc) == ra[1]
        c.perturb(step, cfg.eps)
        for i in range(len(a.params)):
            assert np.array_equal(a.get_theta(i), b.get_theta(i)), (step, a.params[i].name)
        for sess in (a, b, c):
            sess.apply_update(step, 0.7, 1e-3)
    # what reads the caller's parameters between the steps reads the restored ones
    assert a.loss(ba) == b.loss(bb) == c.loss(bc)
    a.close(); b.close(); c.close()


@pytest.mark.parametrize("name", ["linear", "f32 rank 20", "bf16 rank 16"])
def test_fused_step_with_copies(monkeypatch, name):
    """Learning rate 0 makes the fused last pass, which starts from the second copy, independent of g: the same bits."""
    cfg, bits = CASES[name]
    (a, ba), (b, bb) = _sessions(monkeypatch, cfg, bits, fuse_lr=0.0)
    for step in range(2):
        a.step(step, ba), b.step(step, bb)
        for i in range(len(a.params)):
            assert np.array_equal(a.get_theta(i), b.get_theta(i)), (step, a.params[i].name)
    a.close(); b.close()


def test_least_squares_context_with_tensors_of_other_roles(monkeypatch):
    """Tensors the model does not read, of roles that a transformer's copies keep behind Wq and bq: each has a place of its own in the copies."""
    rng = np.random.default_rng(5)
    table = [("w", I.ROLE_LSQ_W, (24, 40)), ("k", I.ROLE_WK, (64, 48)), ("v", I.ROLE_WV, (33, 20)), ("bk", I.ROLE_BK, (1, 13)), ("q", I.ROLE_WQ, (5, 3)), ("k2", I.ROLE_WK, (5, 3))]
    params = [ParamSpec(n, r, 0, i, rng.standard_normal(s).astype(np.float32)) for i, (n, r, s) in enumerate(table)]
    x, y = rng.standard_normal((6, 40)).astype(np.float32), rng.standard_normal((6, 24)).astype(np.float32)
    out = []
    for share in (0.25, 0.0):
        monkeypatch.setattr(Session, "COPIES_SHARE", share)
        sess = Session(B.ZGR_ARCH_LINEAR_LSQ, "f32", params, seed=9, eps=1e-2, alpha=1.0, max_batch=6)
        batch = sess.make_batch(x, y)
        losses = []
        for step in range(2):
            losses.append(sess.step(step, batch)[:2])
            sess.apply_update(step, 0.7, 1e-2)
        out.append((losses, [sess.get_theta(i) for i in range(len(params))], sess.workspace.numel()))
        sess.close()
    (la, ta, na), (lb, tb, nb) = out
    assert na > nb
    assert np.allclose(la, lb, rtol=1e-5), (la, lb)
    for a, b, (name, _, _) in zip(ta, tb, table):
        assert np.array_equal(a, b), name


@pytest.mark.parametrize("name", ["linear", "f32 rank 20", "bf16 rank 16", "encoder post-LN"])
def test_row_losses_of_a_step_outlive_a_later_loss(name):
    """A loss of more rows than the step's writes to the first forward's row losses alone: those of L- stay."""
    cfg, bits = CASES[name]
    specs, values, bases = inputs_of(cfg)
    sess, a = make_session(cfg, specs, values, bases, bits=bits), make_batch_arrays(cfg)
    assert sess.with_copies
    one = sess.make_batch(a["x"][:1], None if a["y"] is None else a["y"][:1], None if a["lengths"] is None else a["lengths"][:1], cfg.seq)
    keep = sess._batch_keep
    n = cfg.seq if cfg.arch == I.ARCH_DECODER_LM else 1
    sess.step(0, one)
    before = sess.step_row_losses(1, n)
    assert np.all(before[:max(1, n - 1)] > 0)
    sess.loss(session_batch(sess, cfg, a))
    assert np.array_equal(sess.step_row_losses(1, n), before)
    del keep
    sess.close()


def test_copies_are_the_callers_choice(monkeypatch):
    """Asked for or refused by the caller; left to the session, a device too full for them is no error."""
    import torch
    params = [ParamSpec("w", I.ROLE_LSQ_W, 0, 0, np.ones((8, 12), np.float32))]
    make = lambda **kw: Session(B.ZGR_ARCH_LINEAR_LSQ, "f32", params, seed=9, eps=1e-2, alpha=1.0, max_batch=6, **kw)
    sizes = {}
    for copies in (None, True, False):
        sess = make(copies=copies)
        sizes[copies] = sess.workspace.numel()
        assert sess.with_copies == (copies is not False)
        sess.close()
    assert sizes[None] == sizes[True] > sizes[False]
    empty = torch.empty

    def full(n, *a, **kw):
        if n == sizes[True]:
            raise torch.cuda.OutOfMemoryError("full")
        return empty(n, *a, **kw)
    monkeypatch.setattr(torch, "empty", full)
    sess = make()
    assert not sess.with_copies and sess.workspace.numel() == sizes[False]
    sess.close()
    with pytest.raises(torch.cuda.OutOfMemoryError):
        make(copies=True)
