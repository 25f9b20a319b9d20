"""Performance cases of the ZGR library: the work its users have it do, through its public entry points.

Five kinds of work, after the three roles of Algorithm 1:
  step      a client's step and the update that follows it: Session.step (two losses) and Session.apply_update
            (with a fused learning rate the step updates by itself)
  loss      a client that only evaluates its model: Session.loss
  updates   the edge server: Session.apply_updates, a context without a model that replays (step, g) pairs
  backward  the cloud's gradients of every tensor: zgr_cloud_backward over memory the program keeps
  basis     the cloud's basis of one matrix from its gradient snapshots: session.cloud_basis_device

Sizes are those of the repository's configurations and benchmark lines (zgr_inputs.CONFIGS, bench.py) and generic ones
between them.  Weights are N(0, 0.02^2) in one slab, LayerNorm gains 1 + N(0, 0.02^2), tokens Zipf(1.1) or uniform, padding
lengths uniform, bases orthonormal: the distributions of zgr_inputs, drawn on the GPU where they are large.
"""
import ctypes as C
import math

import numpy as np
import torch

import zgr_inputs as I
from paper_2601_12917_amd import binding as B
from paper_2601_12917_amd.session import ParamSpec, Session, cloud_basis_device
from paper_2601_12917_amd.workloads import PACK_AFTER_ROLES, make_batch_arrays

_ARCH = {"linear": I.ARCH_LINEAR_LSQ, "decoder": I.ARCH_DECODER_LM, "encoder": I.ARCH_ENCODER_CLS}


def _model_case(kind, arch, dtype, layers, d, heads, ff, vocab, max_pos, batch, seq, k, k_full=None, **more):
    case = dict(kind=kind, arch=arch, dtype=dtype, layers=layers, d=d, heads=heads, ff=ff, vocab=vocab, max_pos=max_pos, batch=batch, seq=seq,
                k=k, k_full=k_full or k, bits=32, bases="device", act="gelu", post_ln=False, fused=False, updates=0, lr=1e-6)
    case.update(more)
    return case


_D125 = dict(layers=12, d=768, heads=12, ff=3072, vocab=50272, max_pos=2048)       # OPT-125m-shaped
_D1P3 = dict(layers=24, d=2048, heads=32, ff=8192, vocab=50272, max_pos=2048)      # OPT-1.3B-shaped
_E350 = dict(layers=24, d=1024, heads=16, ff=4096, vocab=50265, max_pos=512)       # RoBERTa-large-shaped


def listed():
    return [
        # The smallest thing a user runs: one least-squares layer, where launches and the host's wait are everything.
        dict(name="linear step", kind="step", arch="linear", dtype="f32", rows=256, cols=512, batch=32, k=4, bits=32, lr=1e-2),
        # A toy decoder in fp32, the model people debug with: short kernels, many of them.
        dict(_model_case("step", "decoder", "f32", 2, 128, 4, 512, 1024, 64, 8, 64, 8, lr=1e-4), name="tiny decoder step"),
        # The small language model at its configured batch: ordinary work of a phone-sized client.
        dict(_model_case("step", "decoder", "bf16", batch=16, seq=128, k=16, **_D125), name="125m decoder step"),
        # The same model kept in fp32 with a ragged batch: the fp32 matrix products and fp32 logits.
        dict(_model_case("step", "decoder", "f32", batch=5, seq=77, k=16, **_D125), name="125m decoder step f32 ragged"),
        # The encoder classifier with padded sequences: key masks, a classification head, rank 32.
        dict(_model_case("step", "encoder", "bf16", batch=16, seq=256, k=32, **_E350), name="350m encoder step"),
        # The benchmark's own step.
        dict(_model_case("step", "decoder", "bf16", batch=16, seq=256, k=16, k_full=64, **_D1P3), name="1.3b decoder step"),
        # Two long odd documents instead of sixteen short ones, ReLU model, 4-bit bases streamed layer by layer, 16-bit
        # uniforms, restore and update in one pass: the options a memory-bound client turns on together.
        dict(_model_case("step", "decoder", "bf16", batch=2, seq=2047, k=16, bits=16, bases="stream4", act="relu", fused=True, **_D1P3), name="1.3b decoder step long"),
        # The edge server folding four clients' scalars into its copy of the model.
        dict(_model_case("updates", "decoder", "bf16", batch=1, seq=2, k=16, k_full=64, updates=4, **_D1P3), name="1.3b server updates"),
        # Evaluating one short prompt: the model is read once for a handful of tokens.
        dict(_model_case("loss", "decoder", "bf16", batch=1, seq=33, k=16, **_D125), name="125m decoder loss short"),
        # The cloud's gradients for the small decoder, whole k-tiles of tokens.
        dict(_model_case("backward", "decoder", "bf16", batch=16, seq=128, k=16, **_D125), name="125m decoder backward"),
        # The cloud's gradients for the encoder on a few odd sequences.
        dict(_model_case("backward", "encoder", "bf16", batch=3, seq=77, k=32, **_E350), name="350m encoder backward ragged"),
        # The basis as it is transmitted for the largest matrix: 64 columns from three snapshots of a feed-forward weight.
        dict(name="basis 8192x2048", kind="basis", rows=8192, cols=2048, k=64, snapshots=3, sweeps=3),
    ]


def _log_int(rng, lo, hi, multiple=1):
    """An integer of [lo, hi], uniform over its logarithm, a multiple of `multiple`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // multiple * multiple, max(-(-lo // multiple) * multiple, int(v / multiple + 0.5) * multiple))


def _draw_linear(rng):
    rows, cols = _log_int(rng, 16, 2048), _log_int(rng, 16, 2048, 4)
    return dict(kind="step", arch="linear", dtype="f32", rows=rows, cols=cols, batch=_log_int(rng, 1, 512), k=min(rows, _log_int(rng, 1, 32)),
                bits=32, lr=1e-3)


def _draw_model(rng, kind):
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    arch = "encoder" if rng.random() < 0.3 else "decoder"
    head = rng.choice([64, 64, 64, 32]) if dtype == "bf16" else rng.choice([64, 32, 16])
    d = _log_int(rng, 64, 2048, 64)
    seq = _log_int(rng, 2, 2048)
    k = _log_int(rng, 4, 64)
    case = _model_case(kind, arch, dtype, _log_int(rng, 1, 24), d, d // head, _log_int(rng, 2 * d, 4 * d, 64), _log_int(rng, 500, 50272), 2048,
                       _log_int(rng, 1, 32), seq, min(k, d), lr=1e-6,
                       act=rng.choice(["gelu", "relu"]), post_ln=rng.random() < 0.3)
    if kind == "step":
        case["fused"] = rng.random() < 0.2
    if kind in ("step", "updates"):
        case["bits"] = rng.choice([32, 32, 16])
        case["bases"] = rng.choice(["device", "device", "device4", "stream", "stream4", "none"])
    if kind == "updates":
        case["updates"] = rng.randint(1, 8)
    return case


def draw(rng):
    """One more case of the same ranges, never dearer than the listed ones of its kind."""
    kind = rng.choice(["linear", "step", "step", "step", "step", "loss", "updates", "backward", "backward", "basis"])
    dearest = {k: max(_cost(c) for c in listed() if c["kind"] == k and c.get("arch") != "linear") for k in ("step", "updates", "basis")}
    dearest["loss"] = dearest["step"] / 2
    dearest["backward"] = dearest["step"] / 2
    while True:
        if kind == "linear":
            return _draw_linear(rng)
        if kind == "basis":
            rows = _log_int(rng, 64, 8192)
            case = dict(kind="basis", rows=rows, cols=_log_int(rng, 64, 8192), k=_log_int(rng, 4, 64), snapshots=rng.randint(1, 4), sweeps=rng.randint(1, 4))
        else:
            case = _draw_model(rng, kind)
        if _cost(case) <= dearest[kind]:
            return case


def _cost(case):
    """A rough time: what bounds a pass on the matrix cores, the vector units and the memory, in arbitrary units."""
    w = work(case)
    if case["kind"] == "basis":
        return float(case["rows"]) * case["k"] ** 2 * (case["sweeps"] + 1)
    if case["arch"] == "linear":
        return w["flops"]
    slow = 8.0 if case["dtype"] == "f32" else 1.0
    if case["kind"] == "backward" and (case["dtype"] == "f32" or case["batch"] * case["seq"] % 64):
        slow = 16.0
    long_rows = case["batch"] * case["heads"] * float(case["seq"]) ** 2 * case["d"] / case["heads"] * case["layers"]      # attention off the matrix cores
    other = 40.0 * long_rows if case["dtype"] == "f32" or case["d"] // case["heads"] != 64 or case["kind"] == "backward" else 0.0
    return slow * w["flops"] + other + 200.0 * w["bytes"] * max(1, case["updates"])


# ---------------------------------------------------------------------------------------------------------- preparation
def _generator(seed):
    return torch.Generator(device="cuda:0").manual_seed(int(seed) * 7919 + 13)


def _orthonormal(rows, k, gen):
    """[rows, k] with orthonormal columns: a Gaussian block, orthonormalised twice through its Gram matrix."""
    q = torch.randn(rows, k, generator=gen, device="cuda:0", dtype=torch.float64)
    for _ in range(2):
        chol = torch.linalg.cholesky(q.T @ q)
        q = torch.linalg.solve_triangular(chol, q.T, upper=False).T
    return q.float().contiguous()


def _config(case):
    if case["arch"] == "linear":
        return I.Config("case", I.ARCH_LINEAR_LSQ, "f32", lsq_out=case["rows"], lsq_in=case["cols"], batch=case["batch"], k=case["k"], k_full=case["k"])
    return I.Config("case", _ARCH[case["arch"]], case["dtype"], n_layer=case["layers"], d_model=case["d"], n_head=case["heads"], d_ff=case["ff"], vocab=case["vocab"],
                    max_pos=case["max_pos"], n_class=2 if case["arch"] == "encoder" else 0, batch=case["batch"], seq=case["seq"], k=case["k"], k_full=case["k_full"],
                    tokens="zipf", act=case["act"], post_ln=case["post_ln"])


class _State:
    pass


def _session(case, seed, gen):
    """The model of a case in a Session: parameters, bases and workspace on the GPU."""
    cfg = _config(case)
    specs = I.tensor_specs(cfg)
    linear = case["arch"] == "linear"
    guided = [s.guided and case.get("bases") != "none" for s in specs]
    ldu = case.get("k_full", case["k"])
    # the Session copies host arrays to the device; the values drawn on the device follow
    zeros = np.zeros(max(max(s.numel for s in specs), max(s.rows for s in specs) * ldu), np.float32)
    params = [ParamSpec(s.name, s.role, s.layer, s.tensor_id, zeros[:s.numel].reshape(s.rows, s.cols),
                        zeros[:s.rows * ldu].reshape(s.rows, ldu) if on else None, case["k"] if on else 0) for s, on in zip(specs, guided)]
    sess = Session(B.ZGR_ARCH_NONE if case["kind"] == "updates" else cfg.arch, case["dtype"], params, seed=1000 + seed, eps=1e-3, alpha=0.5,
                   scale_mode=B.ZGR_SCALE_PAPER if linear else B.ZGR_SCALE_UNIT, gauss_bits=case["bits"], n_layer=cfg.n_layer, d_model=cfg.d_model,
                   n_head=cfg.n_head, d_ff=cfg.d_ff, vocab=cfg.vocab, max_pos=cfg.max_pos, n_class=cfg.n_class, ln_eps=cfg.ln_eps, max_batch=cfg.batch,
                   max_seq=max(cfg.seq, 2), pack_after=tuple(s.name for s in specs if s.role in PACK_AFTER_ROLES),
                   fuse_lr=case["lr"] if case.get("fused") else None, act=cfg.act, post_ln=cfg.post_ln)
    sess.slab.normal_(0.0, 0.02, generator=gen)
    for i, s in enumerate(specs):
        if s.role in (I.ROLE_LN1_G, I.ROLE_LN2_G, I.ROLE_LNF_G):
            sess.theta[i].add_(1.0)
        if guided[i]:
            sess.U[i].copy_(_orthonormal(s.rows, ldu, gen))
    bases = case.get("bases")
    if bases == "device4":
        for i in range(len(specs)):
            if guided[i]:
                sess.compress_basis(i)
    if bases in ("stream", "stream4"):
        for layer in sorted({s.layer for s, on in zip(specs, guided) if on}):
            idx = [i for i, s in enumerate(specs) if guided[i] and s.layer == layer]
            if bases == "stream4":
                q = [sess.quantize_basis(sess.U[i].cpu().numpy(), case["k"]) for i in idx]
                sess.set_layer_bases_host(idx, [x[0] for x in q], case["k"], codes=True, lams=[x[1] for x in q], deltas=[x[2] for x in q])
            else:
                sess.set_layer_bases_host(idx, [sess.U[i].cpu().numpy() for i in idx], case["k"])
    return cfg, specs, sess


def prepare(case, seed):
    gen = _generator(seed)
    s = _State()
    s.case, s.count = case, 0
    if case["kind"] == "basis":
        # gradients of one matrix over rounds: a common decaying subspace, a part of their own, and noise
        rows, cols = case["rows"], case["cols"]
        r = min(rows, cols, 2 * case["k"])
        left = torch.randn(rows, r, generator=gen, device="cuda:0") * (0.9 ** torch.arange(r, device="cuda:0")) / math.sqrt(rows)
        s.snaps = [(left @ torch.randn(r, cols, generator=gen, device="cuda:0") + 0.02 / math.sqrt(rows) * torch.randn(rows, cols, generator=gen, device="cuda:0")).contiguous()
                   for _ in range(case["snapshots"])]
        s.omega = torch.randn(cols, case["k"], generator=gen, device="cuda:0")
        return s
    cfg, specs, s.sess = _session(case, seed, gen)
    if case["kind"] == "updates":
        s.g = [float(v) for v in torch.randn(case["updates"], generator=torch.Generator().manual_seed(seed)) * 5]
        return s
    a = make_batch_arrays(cfg, seed)
    s.batch = s.sess.make_batch(a["x"], a["y"], a["lengths"], cfg.seq)
    if case["kind"] == "backward":
        nbytes = B.lib().zgr_cloud_backward_workspace(s.sess.ctx, cfg.batch, cfg.seq)
        s.work = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
        offs, off = [], 0
        for sp in specs:
            offs.append(off)
            off += -(-sp.numel // 64) * 64
        s.grads = torch.zeros(off, dtype=torch.float32, device="cuda:0")
        s.ptrs = (C.c_void_p * len(offs))(*[s.grads.data_ptr() + 4 * o for o in offs])
    return s


# ---------------------------------------------------------------------------------------------------------------- a pass
def run(s):
    kind = s.case["kind"]
    if kind == "basis":
        U, dependent = cloud_basis_device(s.snaps, s.case["k"], s.omega, s.case["sweeps"])
        return [U, dependent]
    sess, step = s.sess, s.count
    s.count += 1
    if kind == "loss":
        return sess.loss(s.batch)
    if kind == "updates":
        n = len(s.g)
        sess.apply_updates([step * n + i for i in range(n)], s.g, s.case["lr"])
        return sess.slab
    if kind == "backward":
        loss = C.c_double()
        B.check(B.lib().zgr_cloud_backward(sess.ctx, C.byref(s.batch), s.ptrs, len(s.ptrs), C.byref(loss), s.work.data_ptr(), s.work.numel()), sess.ctx)
        return [loss.value, s.grads]
    loss_plus, loss_minus, g = sess.step(step, s.batch)
    if not s.case.get("fused"):
        sess.apply_update(step, g, s.case["lr"])
    # g is (loss_plus - loss_minus) / (2 eps): it has no relative accuracy of its own, the losses and the weights have
    return [loss_plus, loss_minus, sess.slab]


# ------------------------------------------------------------------------------------------------------ work, tolerances
def work(case):
    """Each parameter, basis and input once in, each result once out; multiply-adds of the products counted as two."""
    if case["kind"] == "basis":
        rows, cols, k, n, sweeps = (float(case[x]) for x in ("rows", "cols", "k", "snapshots", "sweeps"))
        return {"bytes": 4 * (n * rows * cols + cols * k + rows * k), "flops": 2 * n * rows * cols * k * (1 + 2 * sweeps) + (sweeps + 1) * 2 * rows * k * k}
    specs = I.tensor_specs(_config(case))
    params = float(sum(s.numel for s in specs))
    es = 4.0 if case["dtype"] == "f32" else 2.0
    basis = 0.0
    if case.get("bases") != "none":
        per = 0.5 if case.get("bases") in ("device4", "stream4") else 4.0
        basis = sum(s.rows * case["k"] * per for s in specs if s.guided)
    if case["arch"] == "linear":
        batch, mat = float(case["batch"]), params
        return {"bytes": 2 * params * es + basis + 4 * batch * (case["rows"] + case["cols"]), "flops": 2 * 2 * batch * mat + 2 * 2 * case["k"] * mat}
    tokens, d, layers, seq = float(case["batch"] * case["seq"]), case["d"], case["layers"], case["seq"]
    contraction = 2 * case["k"] * sum(s.numel for s in specs if s.guided) if basis else 0.0          # U R, once per set of updates
    if case["kind"] == "updates":
        return {"bytes": 2 * params * es + basis, "flops": contraction}
    forward = 2 * tokens * layers * (4 * d * d + 2 * d * case["ff"])
    forward += 4 * tokens * seq * d * layers * (0.5 if case["arch"] == "decoder" else 1.0)
    forward += 2 * tokens * d * case["vocab"] if case["arch"] == "decoder" else 0.0
    inputs = 4 * tokens
    embeddings = case["vocab"] * d + case["max_pos"] * d
    read = params - (embeddings if case["arch"] == "encoder" else case["max_pos"] * d) + 2 * tokens * d * (1 if case["arch"] == "encoder" else 0.5)
    if case["kind"] == "loss":
        return {"bytes": min(read, params) * es + inputs, "flops": forward}
    if case["kind"] == "backward":
        return {"bytes": min(read, params) * es + 4 * params + inputs, "flops": 3 * forward}
    return {"bytes": 2 * params * es + basis + inputs, "flops": 2 * forward + contraction}


def tolerance(case):
    """About four times what was seen between this path and a build of it with its sums in another order: vector-unit attention
    and products instead of the matrix cores' (each bf16 activation then rounds elsewhere), block-wide LayerNorm reductions,
    fp32 instead of bf16 operands in the backward products, undivided sums in the basis."""
    if case["kind"] == "basis":
        return {"rel": 8e-4, "max": 1.2e-2}                 # seen: 1.9e-4 and 3e-3
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}                   # seen: steps 4.5e-7 and 2.1e-6, gradients 1.7e-6 and 8.9e-6 on small models
    # bf16: "max" is the spacing of bf16 around one weight that rounded the other way, and again in a later pass (2^-6)
    if case["kind"] == "updates":
        return {"rel": 1e-4, "max": 1.6e-2}                 # seen: the same bits; a rounding of Z moves one weight in a few thousand
    if case["arch"] == "encoder":                           # one short row of logits per sequence: a loss averages little
        if case["kind"] == "backward":
            return {"rel": 0.03, "max": 0.99}               # seen: 1e-2 and 0.9 (single entries, against the rms of all gradients)
        return {"rel": 4e-3, "max": 5e-2}                   # seen: 8.6e-4 and 1.3e-2
    if case["kind"] == "backward":
        return {"rel": 3e-3, "max": 0.3}                    # seen: 7.1e-4 and 7.5e-2
    return {"rel": 7e-4, "max": 4.5e-2}                     # seen: 1.6e-4 and 1.1e-2
