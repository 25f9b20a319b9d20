"""HIP path vs CPU oracle for the perturbation itself: Z = a G + b U R of every
kind of tensor, and the in-place passes theta <- rnd(theta + c Z) in fp32 and
bf16.  Tolerances: parameters within 1e-5 (fp32) / 1e-2 (bf16) relative."""
import numpy as np
import pytest

import zgr_inputs as I
from oracle import dtc as D
from oracle import perturbation as P
from tests.util import make_session

pytestmark = pytest.mark.gpu

F32_RTOL, BF16_RTOL = 1e-5, 1e-2
PARAM_SCALE = 0.02          # std of the random init: the scale 'relative' refers to for values near zero


def _basis(rows, k, seed=0):
    q, r = np.linalg.qr(np.random.default_rng(seed).standard_normal((rows, k)))
    return (q * np.sign(np.diag(r))).astype(np.float32)


def _single_tensor_cfg(rows, cols, k, dtype="f32", scale_mode=0, ldu=None):
    return I.shrink(I.CONFIGS["cfg1"], name=f"t{rows}x{cols}k{k}", dtype=dtype, lsq_out=rows, lsq_in=cols, k=k,
                    k_full=ldu or k, scale_mode=scale_mode)


def _session_for(rows, cols, k, dtype="f32", bits=32, scale_mode=0, ldu=None, tensor_id=3):
    cfg = _single_tensor_cfg(rows, cols, k, dtype, scale_mode, ldu)
    spec = I.TensorSpec("W", I.ROLE_LSQ_W, -1, rows, cols, tensor_id, k > 0)
    rng = np.random.default_rng(rows * 131 + cols)
    W = (rng.standard_normal((rows, cols)) * PARAM_SCALE).astype(np.float32)
    if dtype == "bf16":
        W = P.bf16_round(W)
    U = _basis(rows, ldu or k, seed=rows + k) if k > 0 else None
    sess = make_session(cfg, [spec], [W], [U], bits=bits, arch=-1)
    return sess, cfg, W, U


def _z_bound(cfg, G, R, U, k, rows, cols, mode):
    """|Z_gpu - Z_oracle| allowed: 2 ulp on each Gaussian plus fp32 accumulation of the k-term dot."""
    if U is None or k == 0:
        return 2.0 * np.spacing(np.abs(G)) + 1e-45
    a, b = P.mix_coefficients(cfg.alpha, rows, cols, k, mode)
    absdot = np.abs(U[:, :k]).astype(np.float64) @ np.abs(R).astype(np.float64)
    return 2.0 ** -23 * (float(a) * np.abs(G) * 2 + (k + 4) * float(b) * absdot) + 1e-30


SHAPES = [
    # rows, cols, k, ldu
    (256, 512, 4, 4),       # cfg1
    (100, 72, 5, 5),        # ragged in both directions, odd k
    (300, 136, 16, 16),     # two row blocks of a tile, ragged tail
    (130, 256, 64, 64),     # maximum k
    (300, 136, 20, 20),     # matrix-core kernel with a rank that is no multiple of 8: the padded contraction steps are masked
    (200, 264, 36, 40),     # the same with a truncated basis (36 of 40 columns) and ragged tiles in both directions
    (70, 128, 17, 17),      # one step past the smallest matrix-core rank
    (64, 128, 8, 24),       # truncated basis: first 8 of 24 columns
    (1, 1000, 0, 0),        # 1-D, isotropic
    (1, 7, 0, 0),           # shorter than two Philox calls
    (3, 5, 0, 0),           # rows of a matrix straddling Philox calls
    (2, 1024, 0, 0),        # classification head: rows < k keeps it isotropic
]


@pytest.mark.parametrize("rows,cols,k,bits", [
    (1021, 1016, 5, 32),     # 8 strips x 8 row tiles of 128: the most tiles that still take 8 rows each, the last with five
    (1025, 1024, 5, 32),     # one row more: tiles of 128 rows, the last with one
    (1100, 2056, 8, 16),     # the same with eight Gaussians per call, a ragged strip
    (1021, 1016, 18, 32),    # matrix-core kernel on tiles of 64 rows
])
def test_z_on_either_side_of_the_small_tiles(rows, cols, k, bits):
    sess, cfg, W, U = _session_for(rows, cols, k, bits=bits)
    got = sess.fill_z(0, 7)
    G, R, Z = P.hybrid_z(cfg.seed, 7, 3, rows, cols, U, k, cfg.alpha, 0, bits, parts=True)
    assert np.all(np.abs(got.astype(np.float64) - Z) <= _z_bound(cfg, G, R, U, k, rows, cols, 0))
    c = np.float32(1e-3)                      # and the pass itself: one fp32 FMA per entry
    sess.perturb(7, float(c))
    want = W.astype(np.float64) + float(c) * Z
    assert np.all(np.abs(sess.get_theta(0) - want) <= F32_RTOL * (np.abs(want) + PARAM_SCALE))


@pytest.mark.parametrize("bits", [32, 16])
@pytest.mark.parametrize("rows,cols,k,ldu", SHAPES)
def test_z_matches_oracle(rows, cols, k, ldu, bits):
    if k > 0 and cols % (4 if bits == 32 else 8):
        pytest.skip("guided tensors need cols to be a multiple of the Philox group")
    for mode in (P.SCALE_UNIT, P.SCALE_PAPER):
        sess, cfg, W, U = _session_for(rows, cols, k, bits=bits, scale_mode=mode, ldu=ldu)
        step = 11
        got = sess.fill_z(0, step)
        G, R, Z = P.hybrid_z(cfg.seed, step, 3, rows, cols, U, k, cfg.alpha, mode, bits, parts=True)
        assert got.shape == Z.shape and np.all(np.isfinite(got))
        assert np.all(np.abs(got.astype(np.float64) - Z) <= _z_bound(cfg, G, R, U, k, rows, cols, mode))
        sess.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols,k,ldu", SHAPES)
def test_inplace_pass_matches_oracle(rows, cols, k, ldu, dtype):
    sess, cfg, W, U = _session_for(rows, cols, k, dtype=dtype, ldu=ldu)
    step, c = 4, np.float32(1e-3)
    Z = P.hybrid_z(cfg.seed, step, 3, rows, cols, U, k, cfg.alpha, P.SCALE_UNIT, 32)
    want = W
    for coef in (c, np.float32(-2) * c, c, np.float32(-3.7e-4)):        # the four passes of a step + update
        sess.perturb(step, float(coef))
        want = P.axpy_inplace_value(want, coef, Z, dtype)
        got = sess.get_theta(0)
        if dtype == "f32":
            assert np.all(np.abs(got - want) <= F32_RTOL * (np.abs(want) + PARAM_SCALE))
            assert np.abs(got - want).max() <= 4e-9 + 4 * np.spacing(np.abs(want)).max()   # in fact within an ulp or two
        else:
            assert np.all(np.abs(got - want) <= BF16_RTOL * np.abs(want) + 1e-30)
            assert np.mean(got == want) > 0.98
        want = got          # later passes start from what the device holds, so errors do not compound in the check
    sess.close()


def test_set_basis_switches_between_guided_and_non_guided_rounds():
    rows, cols, k = 96, 64, 8
    sess, cfg, W, U = _session_for(rows, cols, k)
    G = P.gauss_field(cfg.seed, 2, 3, 0, rows, cols)
    Zg = P.hybrid_z(cfg.seed, 2, 3, rows, cols, U, k, cfg.alpha)
    assert np.allclose(sess.fill_z(0, 2), Zg, atol=2e-6)
    sess.set_basis(0, None, 0)                       # non-guided round: Z = G
    assert np.all(np.abs(sess.fill_z(0, 2) - G) <= 2 * np.spacing(np.abs(G)))
    U2 = _basis(rows, 4, seed=77)
    sess.set_basis(0, U2, 4)                         # a new basis from the cloud
    Z2 = P.hybrid_z(cfg.seed, 2, 3, rows, cols, U2, 4, cfg.alpha)
    assert np.allclose(sess.fill_z(0, 2), Z2, atol=2e-6)
    sess.close()


def test_alpha_one_and_identity_basis_special_cases():
    rows, cols = 32, 64
    cfg = I.shrink(_single_tensor_cfg(rows, cols, rows), alpha=0.36)
    spec = I.TensorSpec("W", I.ROLE_LSQ_W, -1, rows, cols, 3, True)
    W = np.zeros((rows, cols), np.float32)
    sess = make_session(cfg, [spec], [W], [np.eye(rows, dtype=np.float32)], arch=-1)
    G = P.gauss_field(cfg.seed, 0, 3, 0, rows, cols)
    R = P.gauss_field(cfg.seed, 0, 3, 1, rows, cols)
    assert np.allclose(sess.fill_z(0, 0), 0.6 * G + 0.8 * R, atol=3e-6)      # k = rows, U = I
    sess.close()
    cfg1 = I.shrink(cfg, alpha=1.0, k=4, k_full=4)
    sess = make_session(cfg1, [spec], [W], [_basis(rows, 4)], arch=-1)
    assert np.all(np.abs(sess.fill_z(0, 0) - G) <= 2 * np.spacing(np.abs(G)))  # alpha = 1: plain ZO-SGD direction
    sess.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ranks", [(8, 16), (16, 4), (20, 5, 64)])
def test_mixed_ranks_in_one_context(ranks, dtype):
    """Tensors with ranks on both sides of 16 in one table: each rank class is served by its own kernel (matrix
    cores from 16 on, vector FMAs below), and every tensor's Z and in-place pass match the oracle."""
    from paper_2601_12917_amd.session import ParamSpec, Session
    rng = np.random.default_rng(sum(ranks))
    shapes = [(192, 256), (150, 136), (256, 128)][:len(ranks)]
    params, Ws, Us = [], [], []
    for j, ((rows, cols), k) in enumerate(zip(shapes, ranks)):
        W = (rng.standard_normal((rows, cols)) * PARAM_SCALE).astype(np.float32)
        if dtype == "bf16":
            W = P.bf16_round(W)
        U = _basis(rows, k, seed=40 + j)
        params.append(ParamSpec(f"W{j}", I.ROLE_LSQ_W, -1, 10 + j, W, U, k))
        Ws.append(W); Us.append(U)
    # plus an isotropic tensor, so the flat kernel runs in the same pass
    b = (rng.standard_normal((1, 300)) * PARAM_SCALE).astype(np.float32)
    if dtype == "bf16":
        b = P.bf16_round(b)
    params.append(ParamSpec("b", I.ROLE_B1, 0, 20, b))
    cfg = _single_tensor_cfg(1, 1, 1, dtype)
    sess = Session(-1, dtype, params, cfg.seed, cfg.eps, cfg.alpha, P.SCALE_UNIT, 32)
    step, c = 6, np.float32(1e-3)
    for j, ((rows, cols), k) in enumerate(zip(shapes, ranks)):
        G, R, Z = P.hybrid_z(cfg.seed, step, 10 + j, rows, cols, Us[j], k, cfg.alpha, P.SCALE_UNIT, 32, parts=True)
        got = sess.fill_z(j, step)
        assert np.all(np.abs(got.astype(np.float64) - Z) <= _z_bound(cfg, G, R, Us[j], k, rows, cols, P.SCALE_UNIT)), (j, k)
    sess.perturb(step, float(c))
    for j, ((rows, cols), k) in enumerate(zip(shapes, ranks)):
        Z = P.hybrid_z(cfg.seed, step, 10 + j, rows, cols, Us[j], k, cfg.alpha, P.SCALE_UNIT, 32)
        want = P.axpy_inplace_value(Ws[j], c, Z, dtype)
        got = sess.get_theta(j)
        if dtype == "f32":
            assert np.all(np.abs(got - want) <= F32_RTOL * (np.abs(want) + PARAM_SCALE)), (j, k)
        else:
            assert np.all(np.abs(got - want) <= BF16_RTOL * np.abs(want) + 1e-30) and np.mean(got == want) > 0.98, (j, k)
    want_b = P.axpy_inplace_value(b, c, P.gauss_field(cfg.seed, step, 20, 0, 1, 300), dtype)
    assert np.all(np.abs(sess.get_theta(len(ranks)) - want_b) <= (F32_RTOL if dtype == "f32" else BF16_RTOL) * (np.abs(want_b) + PARAM_SCALE))
    sess.close()


@pytest.mark.parametrize("rows,cols,k,ldu,bits,dtype", [
    (17, 128, 16, 17, 32, "f32"),       # a second slab of one row; rows of U on 4-byte boundaries
    (144, 132, 24, 24, 32, "bf16"),     # three eights (a step of 32 terms with eight zeros); a second tile of one whole slab, a strip of 4 columns
    (129, 256, 40, 43, 16, "bf16"),     # a step of 32 terms and one of 8; eight Gaussians per call
    (257, 264, 48, 48, 16, "f32"),      # steps of 32 and 16 terms, two vectors of theta per round
    (256, 128, 56, 56, 32, "f32"),      # 32 and 24
    (2304, 512, 32, 32, 32, "bf16"),    # several tiles of a strip per block
])
def test_matrix_core_tiles_at_their_edges(rows, cols, k, ldu, bits, dtype):
    sess, cfg, W, U = _session_for(rows, cols, k, dtype=dtype, bits=bits, ldu=ldu)
    step, c = 9, np.float32(1e-3)
    for quantised in (False, True):
        if quantised:
            lam, delta = D.affine_params(U[:, :k], 4)
            codes = D.quantize(U[:, :k], lam, delta, 4)
            U = D.dequantize(codes, lam, delta)
            sess.set_basis_q4(0, D.pack_nibbles(codes), k, lam, delta)
        G, R, Z = P.hybrid_z(cfg.seed, step, 3, rows, cols, U, k, cfg.alpha, P.SCALE_UNIT, bits, parts=True)
        assert np.all(np.abs(sess.fill_z(0, step).astype(np.float64) - Z) <= _z_bound(cfg, G, R, U, k, rows, cols, P.SCALE_UNIT))
        before = sess.get_theta(0)
        sess.perturb(step, float(c))
        want, got = P.axpy_inplace_value(before, c, Z, dtype), sess.get_theta(0)
        if dtype == "f32":
            assert np.all(np.abs(got - want) <= F32_RTOL * (np.abs(want) + PARAM_SCALE))
        else:
            assert np.all(np.abs(got - want) <= BF16_RTOL * np.abs(want) + 1e-30) and np.mean(got == want) > 0.98
    sess.close()


@pytest.mark.parametrize("k", [16, 40])
def test_basis_entries_beyond_bf16(k):
    """Entries that bf16 does not hold, and an infinite one, give what fp32 products give; their rows alone are concerned."""
    rows, cols = 160, 128
    sess, cfg, W, U = _session_for(rows, cols, k, scale_mode=P.SCALE_PAPER)
    U = U.copy()
    U[5, 3], U[70, k - 1], U[130, 0] = 3.4e38, np.inf, -np.inf
    sess.set_basis(0, U, k)
    with np.errstate(invalid="ignore", over="ignore"):
        G, R, Z = P.hybrid_z(cfg.seed, 1, 3, rows, cols, U, k, cfg.alpha, P.SCALE_PAPER, 32, parts=True)
        bound = _z_bound(cfg, G, R, U, k, rows, cols, P.SCALE_PAPER)
    got = sess.fill_z(0, 1).astype(np.float64)
    for r, l, sign in ((70, k - 1, 1.0), (130, 0, -1.0)):
        assert np.array_equal(got[r], sign * np.sign(R[l]) * np.inf)
    rest = np.setdiff1d(np.arange(rows), [70, 130])
    assert np.all(np.abs(got[rest] - Z[rest]) <= bound[rest])
    sess.close()


@pytest.mark.parametrize("rows,cols,k,dtype,bits", [
    (16, 128, 16, "f32", 32),       # a tile with rows for one wave of eight
    (33, 132, 16, "bf16", 32),      # for three, the last with one row; a strip of 4 columns
    (80, 128, 24, "f32", 32),       # tiles of 64 and of 16 rows, or one of 80
    (193, 256, 40, "bf16", 32),     # four tiles of 64, the last of one row; of 128 and of 65
    (200, 264, 16, "f32", 16),
    (129, 256, 64, "bf16", 16),
    (256, 260, 24, "bf16", 32),     # whole tiles of 128 rows, which a launch without ragged ones takes by themselves
    (128, 264, 40, "f32", 16),
    (384, 512, 16, "f32", 32),
])
def test_bits_do_not_depend_on_the_height_of_the_tiles(rows, cols, k, dtype, bits):
    """The same tensor alone (tiles of 64 rows), with a vector beside it (both in one launch) and in contexts of many tiles (128 rows), one of them with a ragged last: single passes and sums of
    several perturbations leave the same bits, and every entry is moved once."""
    cfg = _single_tensor_cfg(rows, cols, k, dtype)
    rng = np.random.default_rng(rows + cols)

    def values(r, c):
        w = (rng.standard_normal((r, c)) * PARAM_SCALE).astype(np.float32)
        return P.bf16_round(w) if dtype == "bf16" else w
    W, U = values(rows, cols), _basis(rows, k)
    vector = (I.TensorSpec("b", I.ROLE_BQ, -1, 1, 333, 5, False), values(1, 333), None)
    many, whole = ((I.TensorSpec("V", I.ROLE_LSQ_W, -1, n, 2304, 9, True), values(n, 2304), _basis(n, k, 2)) for n in (1100, 1152))
    c = np.float32(1e-3)
    want = P.axpy_inplace_value(W, c, P.hybrid_z(cfg.seed, 4, 3, rows, cols, U, k, cfg.alpha, P.SCALE_UNIT, bits), dtype)
    seen = []
    for others in ([], [vector], [many], [whole]):
        sess = make_session(cfg, [I.TensorSpec("W", I.ROLE_LSQ_W, -1, rows, cols, 3, True)] + [o[0] for o in others], [W] + [o[1] for o in others], [U] + [o[2] for o in others], bits=bits, arch=-1)
        sess.perturb(4, float(c))
        once = sess.get_theta(0)
        sess.apply_updates([7, 8, 9], [0.5, -0.25, 1.0], 1e-3)
        seen.append((once, sess.get_theta(0)))
        sess.close()
    assert np.all(np.abs(seen[0][0] - want) <= (F32_RTOL if dtype == "f32" else BF16_RTOL) * (np.abs(want) + PARAM_SCALE))
    assert all(np.array_equal(a, b) for one in seen[1:] for a, b in zip(one, seen[0]))


@pytest.mark.parametrize("k,bits", [(16, 32), (40, 32), (24, 16)])
def test_basis_rows_and_coefficients_too_small_for_planes(k, bits):
    """Rows of U around 2^-114 and 2^-130, whose last bits no plane of normal bf16 numbers holds, and a sum of perturbations with coefficients around 2^-112: within the norm of fp32
    products (a sum of k terms rounds k times by 2^-24 of its size at most, R by 2 2^-23), each row by itself."""
    rows, cols = 160, 128
    cfg = I.shrink(_single_tensor_cfg(rows, cols, k), alpha=0.0)
    spec = I.TensorSpec("W", I.ROLE_LSQ_W, -1, rows, cols, 3, True)
    U = _basis(rows, k)
    U[40:50] *= np.float32(2.0 ** -111)
    U[50:60] *= np.float32(2.0 ** -127)                             # subnormal ones: results with 2^-22 of their size
    off = lambda got, want: np.linalg.norm(got - want.astype(np.float64), axis=1) / np.linalg.norm(want.astype(np.float64), axis=1)
    sess = make_session(cfg, [spec], [np.zeros((rows, cols), np.float32)], [U], bits=bits, arch=-1)
    Z = P.hybrid_z(cfg.seed, 1, 3, rows, cols, U, k, 0.0, P.SCALE_UNIT, bits)
    assert off(sess.fill_z(0, 1).astype(np.float64), Z).max() <= (k + 4) * 2.0 ** -24
    sess.set_basis(0, _basis(rows, k), k)
    lr, gs = np.float32(1e-30), np.float32([2e-4, -3e-4])
    sess.apply_updates([1, 2], gs, float(lr))
    want = sum(-float(np.float32(lr * g)) * P.hybrid_z(cfg.seed, s, 3, rows, cols, _basis(rows, k), k, 0.0, P.SCALE_UNIT, bits).astype(np.float64) for s, g in zip((1, 2), gs))
    assert off(sess.get_theta(0).astype(np.float64), want).max() <= (k + 8) * 2.0 ** -24
    sess.close()


@pytest.mark.parametrize("k", [8, 16, 64])
@pytest.mark.parametrize("blocks", ["one a CU", "two a CU", "more"])
def test_lists_share_a_launch_while_their_blocks_are_resident(k, blocks):
    """A block per entry of either list, two a CU at most: with one entry more the lists take a launch each, with the same bits."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    per_item = 256 * 4 * 4                                                     # fp32: 256 threads of four calls of four Gaussians
    rows, cols = 64, 128
    tiles = 1 if k >= 16 else 8
    flat = {"one a CU": cus - tiles, "two a CU": 2 * cus - tiles, "more": 2 * cus - tiles + 1}[blocks]
    cfg = _single_tensor_cfg(rows, cols, k)
    rng = np.random.default_rng(k)
    W, U = (rng.standard_normal((rows, cols)) * PARAM_SCALE).astype(np.float32), _basis(rows, k)
    v = (rng.standard_normal((1, flat * per_item)) * PARAM_SCALE).astype(np.float32)
    spec = I.TensorSpec("W", I.ROLE_LSQ_W, -1, rows, cols, 3, True)
    sess = make_session(cfg, [spec, I.TensorSpec("b", I.ROLE_BQ, -1, 1, flat * per_item, 5, False)], [W, v], [U, None], arch=-1)
    sess.profile_enable()
    sess.perturb(4, 1e-3)
    assert [n for _, n in sess.profile_read().values()][:2] == ([1, 1] if blocks == "more" else [1, 0])
    alone = make_session(cfg, [spec], [W], [U], arch=-1)
    alone.perturb(4, 1e-3)
    assert np.array_equal(sess.get_theta(0), alone.get_theta(0))
    want = P.axpy_inplace_value(v, np.float32(1e-3), P.gauss_field(cfg.seed, 4, 5, 0, 1, v.size), "f32")
    assert np.all(np.abs(sess.get_theta(1) - want) <= F32_RTOL * (np.abs(want) + PARAM_SCALE))
    sess.close(); alone.close()
