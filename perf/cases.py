"""Performance cases of the library: the calls that a training program makes of it, with the sizes
such programs have.

A case is a dict of plain values.  `kind` says which part of a training step it is:

  backward   one backward action of a pipeline stage: tf_stage_backward, or its microbatch, row-block
             and shared-input forms (`form`)
  optimizer  one masked AdamW step, with the stability averages and their sums
  step       both, one after the other, as a small model's training loop calls them
  norms      one AutoFreeze stability check
  reconcile  one budget reconciliation of an element mask

The tensors are those of LLaMA blocks (q, k, v, o, gate, up, down): `blocks` of them with widths d,
kv and ffn, T tokens per call.
"""
import math
import random

import numpy as np
import torch

import paper_2602_05754_amd as tf

DEV = "cuda"
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
CODE = {"bf16": tf.TF_BF16, "f32": tf.TF_F32}
HYPER = dict(lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
EMA_DECAY = 0.99
B1 = dict(d=2048, kv=512, ffn=8192)          # LLaMA-3.2-1B widths
B8 = dict(d=4096, kv=1024, ffn=14336)        # LLaMA-3-8B widths

_ctx = None


def _context():
    """The one context that a program keeps for its GPU."""
    global _ctx
    if _ctx is None:
        _ctx = tf.Context(0)
    return _ctx


def listed():
    return [
        # The smallest training step there is use for: the fp32 tiny stage (2 blocks of width 256, two
        # sequences of 128 tokens), half of its tensors frozen.  Launches and latency.
        dict(name="step_tiny_f32", kind="step", io="f32", dw="f32", blocks=2, d=256, kv=256, ffn=688, T=256, r=0.5),
        # The LLaMA-1B-shaped stage at its full batch of four sequences of 2048 tokens.
        dict(name="stage_1b", kind="backward", form="plain", io="bf16", dw="bf16", blocks=4, T=8192, r=0.5, **B1),
        # Four blocks of the LLaMA-8B-shaped stage, one sequence of 4096 tokens: the largest backward.
        dict(name="stage_8b", kind="backward", form="plain", io="bf16", dw="bf16", blocks=4, T=4096, r=0.5, **B8),
        # A packed batch of instruction data: its token count is whatever the samples add up to.
        dict(name="stage_1b_packed", kind="backward", form="plain", io="bf16", dw="bf16", blocks=2, T=3001, r=0.25, **B1),
        # A single short sample, 200 tokens: fewer rows than one tile of a large product.
        dict(name="stage_1b_short", kind="backward", form="plain", io="bf16", dw="bf16", blocks=2, T=200, r=0.5, **B1),
        # An fp32 stage of a small model (width 1024, odd feed-forward width, 1000 tokens).
        dict(name="stage_f32", kind="backward", form="plain", io="f32", dw="f32", blocks=2, d=1024, kv=256, ffn=2731, T=1000, r=0.5),
        # One of the later microbatches of an 8-microbatch step of the 8B stage: 1024 tokens, weight
        # gradients added to fp32 accumulators.
        dict(name="microbatch_8b", kind="backward", form="microbatch", io="bf16", dw="f32", blocks=2, T=1024, r=0.4, **B8),
        # Sub-tensor freezing (256-row blocks) with q/k/v and gate/up sharing their input gradients.
        dict(name="rows_shared_1b", kind="backward", form="rows", io="bf16", dw="bf16", blocks=2, T=4096, r=0.5, **B1),
        # The optimizer over one 8B block, tensors frozen whole, bf16 gradients.
        dict(name="adamw_8b", kind="optimizer", mask="tensor", grad="bf16", r=0.3, **B8),
        # The optimizer over one 1B block, random elements frozen, fp32 gradient accumulators of 8 microbatches.
        dict(name="adamw_1b_elements", kind="optimizer", mask="element", grad="f32", r=0.3, **B1),
        # A stability check over one 8B block.
        dict(name="norms_8b", kind="norms", blocks=1, **B8),
        # The freeze budget of the whole 8B stage: 1.74e9 mask bits brought from 30 % to 50 % ones.
        dict(name="reconcile_8b", kind="reconcile", blocks=8, density=0.3, ratio=0.5, seed=7, **B8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds: any token count from a few to 8192, widths of small to
    8B-sized models (feed-forward widths that are no multiple of a tile among them), every form."""
    what = rng.choice(["bf16", "bf16", "bf16", "bf16", "f32", "f32", "step", "optimizer", "optimizer", "norms", "reconcile"])
    r = rng.choice([0.0, 0.25, 0.3, 0.5, 0.75, 0.9])
    if what == "bf16":
        form = rng.choice(["plain", "plain", "microbatch", "rows"])
        d = 256 * rng.randint(1, 16)
        heads = rng.choice([1, 2, 4])
        ffn = int(d * rng.uniform(2.6, 4.0))
        ffn -= ffn % rng.choice([8, 64, 256])
        kv = max(64, d // heads)
        T = _log_int(rng, 32, 8192)
        if rng.random() < 0.4:
            T = max(64, T - T % 64)
        if form == "rows":                           # shared input gradients are for whole tiles of bf16
            T, ffn = max(256, T), ffn - ffn % 64
        params = 2 * d * d + 2 * d * kv + 3 * d * ffn
        blocks = max(1, min(4, int(1.2e12 / (T * params))))
        while T * params * blocks > 2.4e12:
            T = T // 2
        dw = "f32" if form == "microbatch" else rng.choice(["bf16", "bf16", "f32"])
        return dict(kind="backward", form=form, io="bf16", dw=dw, blocks=blocks, d=d, kv=kv, ffn=ffn, T=T, r=r)
    if what in ("f32", "step"):
        d = 32 * rng.randint(4, 40 if what == "f32" else 16)
        ffn = int(d * rng.uniform(2.6, 4.0))
        kv = max(32, d // rng.choice([1, 2, 4]))
        T = _log_int(rng, 16, 2048 if what == "f32" else 512)
        case = dict(kind="backward", form="plain") if what == "f32" else dict(kind="step")
        r = min(r, 0.75) if what == "step" else r    # of seven tensors, 0.9 freezes all
        return dict(case, io="f32", dw="f32", blocks=rng.choice([1, 2]) if what == "f32" else 1, d=d, kv=kv, ffn=ffn, T=T, r=r)
    d = 64 * rng.randint(2, 64)
    kv = max(64, d // rng.choice([1, 2, 4]))
    ffn = int(d * rng.uniform(2.6, 3.5))
    if what == "optimizer":
        return dict(kind="optimizer", mask=rng.choice(["tensor", "element"]), grad=rng.choice(["bf16", "f32"]), r=min(r, 0.75), d=d, kv=kv, ffn=ffn)
    if what == "norms":
        return dict(kind="norms", blocks=rng.choice([1, 2]), d=d, kv=kv, ffn=ffn)
    return dict(kind="reconcile", blocks=rng.choice([1, 2, 4, 8]), d=d, kv=kv, ffn=ffn, density=rng.choice([0.1, 0.3, 0.5, 0.8]),
                ratio=rng.choice([0.2, 0.4, 0.7, 0.9]), seed=rng.randrange(1 << 60))


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _shapes(case):
    d, kv, f = case["d"], case["kv"], case["ffn"]
    return [(d, d), (d, kv), (d, kv), (d, d), (d, f), (d, f), (f, d)] * case.get("blocks", 1)


def _frozen(case):
    """Whole tensors frozen at ratio r: the first ceil(r L) of a fixed permutation."""
    L = len(_shapes(case))
    order = list(range(L))
    random.Random(41).shuffle(order)
    mask = np.zeros(L, np.uint8)
    mask[order[: math.ceil(case["r"] * L - 1e-9)]] = 1
    return mask


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype="f32"):
    return (torch.randn(shape, generator=g, device=DEV) * std).to(TORCH[dtype])


def _words(g, n, p):
    """n random 32-bit mask words whose bits are 1 with probability p (to 2^-16)."""
    rand = lambda: torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
    if p <= 0 or p >= 1:
        return torch.full((n,), -1 if p >= 1 else 0, dtype=torch.int32, device=DEV)
    k = int(round(p * 65536))
    out = torch.zeros(n, dtype=torch.int32, device=DEV)
    for b in range(16):
        out = (out | rand()) if (k >> b) & 1 else (out & rand())
    return out


def _backward_inputs(case, g):
    sh, T = _shapes(case), case["T"]
    io = case["io"]
    W = [_normal(g, s, 0.02, io) for s in sh]
    X = [_normal(g, (T, k), 1.0, io) for k, n in sh]
    dY = [_normal(g, (T, n), 1e-3, io) for k, n in sh]
    if case.get("form") == "rows":
        for l in range(0, len(sh), 7):               # q, k, v read one input, gate and up another
            X[l + 1] = X[l + 2] = X[l]
            X[l + 5] = X[l + 4]
    dW0 = None
    if case.get("form") == "microbatch":             # what earlier microbatches have left in the accumulators
        dW0 = [_normal(g, s, 1e-3 * math.sqrt(T)) for s in sh]
    return W, X, dY, dW0


def _row_masks(case):
    """256-row blocks frozen at ratio r; tensors whose rows do not divide so are left whole."""
    sh = _shapes(case)
    rnd = random.Random(43)
    return [np.array([rnd.random() < case["r"] for _ in range(k // 256)], np.uint8) if k % 256 == 0 else None for k, n in sh]


def _groups(case):
    return np.array([g for b in range(case["blocks"]) for g in (7 * b, 7 * b, 7 * b, -1, 7 * b + 4, 7 * b + 4, -1)], np.int32)


def _prepare_backward(case, g):
    sh, T = _shapes(case), case["T"]
    W, X, dY, dW0 = _backward_inputs(case, g)
    s = dict(case=case, shapes=sh, mask=_frozen(case))
    dX = [torch.empty((T, k), dtype=TORCH[case["io"]], device=DEV) for k, n in sh]
    if case.get("form") == "rows":
        s["rows"], s["groups"], s["mask"] = _row_masks(case), _groups(case), None
        dX = [dX[q if grp < 0 else grp] for q, grp in enumerate(s["groups"])]
    dW = dW0 or [torch.zeros(t, dtype=TORCH[case["dw"]], device=DEV) for t in sh]
    s["tables"] = [tf.PtrTable(t) for t in (W, X, dY, dX, dW)]
    s["dX"], s["dW"] = dX, dW
    s["add"] = np.ones(len(sh), np.uint8)
    return s


def _backward(s):
    case, sh = s["case"], s["shapes"]
    W, X, dY, dX, dW = s["tables"]
    T, io, dw = case["T"], CODE[case["io"]], CODE[case["dw"]]
    form = case.get("form", "plain")
    if form == "microbatch":
        tf.tf_stage_backward_microbatch(_context(), sh, T, io, W, X, dY, s["mask"], dX, dW, dw, s["add"])
    elif form == "rows":
        tf.tf_stage_backward_shared(_context(), sh, T, io, W, X, dY, None, s["rows"], 256, s["groups"], dX, dW, dw)
    else:
        tf.tf_stage_backward(_context(), sh, T, io, W, X, dY, s["mask"], dX, dW, dw)
    return _backward_out(case, s["mask"], s["dX"], s["dW"])


def _backward_out(case, mask, dX, dW):
    """Every input gradient once, and the weight gradients of tensors that are not frozen whole."""
    grp = _groups(case) if case.get("form") == "rows" else [-1] * len(dX)
    out = {"dX%d" % l: x for l, x in enumerate(dX) if grp[l] in (-1, l)}
    out.update({"dW%d" % l: w for l, w in enumerate(dW) if mask is None or not mask[l]})
    return out


def _prepare_optimizer(case, g, grads=None):
    sh = _shapes(case)
    n = [k * m for k, m in sh]
    s = dict(case=case, numel=n, mask=_frozen(case), bits=None)
    p = [_normal(g, q, 0.02) for q in n]
    m = [_normal(g, q, 3e-4) for q in n]
    v = [_normal(g, q, 1e-3).square_() for q in n]
    E = [_normal(g, q, 1e-5) for q in n]
    A = [_normal(g, q, 1e-4).abs_() for q in n]
    grad = grads or [_normal(g, q, 1e-3, case["grad"]) for q in n]
    low = [t.to(torch.bfloat16) for t in p] if grads is None else None
    if case.get("mask") == "element":
        s["bits"] = [_words(g, (q + 31) // 32, case["r"]) for q in n]
        s["mask"] = np.zeros(len(n), np.uint8)
    s["buffers"] = dict(p=p, m=m, v=v, E=E, A=A)
    if low is not None:
        s["buffers"]["low"] = low
    s["grad"] = grad
    s["tables"] = {k: tf.PtrTable(t) for k, t in s["buffers"].items()}
    s["grad_table"] = tf.PtrTable(grad)
    s["sums"] = torch.zeros(2 * len(n), dtype=torch.float64, device=DEV)
    s["step"] = np.full(len(n), 10, np.int32)
    s["scale"] = 1.0 if case.get("grad") != "f32" else 0.125
    return s


def _optimizer(s):
    t = s["tables"]
    grad_dtype = CODE[s["case"].get("grad", "f32")]
    tf.tf_masked_adamw(_context(), s["numel"], t["p"], t["m"], t["v"], s["grad_table"], grad_dtype, s["step"],
                       grad_scale=s["scale"], p_lowp=t.get("low"), tensor_freeze_mask=s["mask"], elem_freeze_bits=s["bits"],
                       ema=t["E"], ema_abs=t["A"], ema_decay=EMA_DECAY, score_sums=s["sums"], **HYPER)
    s["step"] = s["step"] + 1
    out = {"%s%d" % (k, i): x for k, seq in s["buffers"].items() for i, x in enumerate(seq) if not s["mask"][i]}
    out["sums"] = s["sums"]
    return out


def _prepare_step(case, g):
    back = _prepare_backward(case, g)
    return dict(case=case, back=back, opt=_prepare_optimizer(dict(case, grad="f32", mask="tensor"), g, grads=back["dW"]))


def _prepare_norms(case, g):
    n = [k * m for k, m in _shapes(case)]
    snap = [_normal(g, q, 0.02) for q in n]
    p = [[t + _normal(g, t.shape, 1e-4) for t in snap] for _ in range(2)]      # the weights at two checks in turn
    return dict(case=case, numel=n, p=p, snap=snap, turn=0, out=torch.zeros(len(n), dtype=torch.float64, device=DEV))


def _norms(s):
    p = s["p"][s["turn"]]
    s["turn"] ^= 1
    tf.tf_autofreeze_norms(_context(), s["numel"], p, s["snap"], s["out"])
    return {"norms": s["out"], "snapshot": list(s["snap"])}


def _prepare_reconcile(case, g):
    n = [k * m for k, m in _shapes(case)]
    base = [_words(g, (q + 31) // 32, case["density"]) for q in n]
    return dict(case=case, numel=n, base=base, bits=[torch.empty_like(b) for b in base], budget=int(case["ratio"] * sum(n)),
                stats=torch.zeros(3, dtype=torch.int64, device=DEV))


def _reconcile(s):
    for b, w in zip(s["base"], s["bits"]):           # the check's fresh mask; the entry point works in place
        w.copy_(b)
    tf.tf_reconcile_mask(_context(), s["numel"], s["bits"], s["budget"], s["case"]["seed"], s["stats"])
    return {"bits": list(s["bits"]), "stats": s["stats"]}


def prepare(case, seed):
    g = _gen(seed)
    _context()
    make = dict(backward=_prepare_backward, optimizer=_prepare_optimizer, step=_prepare_step, norms=_prepare_norms, reconcile=_prepare_reconcile)
    return make[case["kind"]](case, g)


def run(state):
    kind = state["case"]["kind"]
    if kind == "backward":
        return _backward(state)
    if kind == "optimizer":
        return _optimizer(state)
    if kind == "norms":
        return _norms(state)
    if kind == "reconcile":
        return _reconcile(state)
    out = _backward(state["back"])
    out.update(_optimizer(state["opt"]))
    return out


# ---------------------------------------------------------------------------------------------
# what a case cannot do without, and what it should give
# ---------------------------------------------------------------------------------------------
def _backward_work(case):
    sh, T = _shapes(case), case["T"]
    e, w = (2 if case["io"] == "bf16" else 4), (2 if case["dw"] == "bf16" else 4)
    rows = case.get("form") == "rows"
    keep = [1.0 if m is None else 1.0 - float(m.mean()) for m in _row_masks(case)] if rows else [1.0 - float(f) for f in _frozen(case)]
    grp = _groups(case) if rows else [-1] * len(sh)
    b = f = 0.0
    for l, (k, n) in enumerate(sh):
        lead = grp[l] in (-1, l)
        f += 2.0 * T * k * n * (1 + keep[l])
        b += e * (k * n + T * n) + (e * T * k if lead else 0)                       # W, dY, dX
        b += (e * T * k * keep[l] if lead or not rows else 0)                       # X
        b += w * k * n * keep[l] * (2 if case.get("form") == "microbatch" else 1)   # dW, read as well where it is added to
    return b, f


def _optimizer_work(case, low=True):
    keep = [1.0 - float(f) for f in _frozen(case)] if case.get("mask") != "element" else None
    g = 2 if case.get("grad") == "bf16" else 4
    b = 0.0
    for i, (k, n) in enumerate(_shapes(case)):
        # p, m, v, E, A read and written, the gradient read, the bf16 copy written.  With random
        # elements frozen nearly every line of memory still holds elements that are not.
        b += k * n * ((keep[i] if keep else 1.0) * (40 + g + (2 if low else 0)) + (1 / 8 if keep is None else 0))
    return b, 20.0 * b / 44


def work(case):
    kind = case["kind"]
    n = sum(k * m for k, m in _shapes(case))
    if kind == "backward":
        b, f = _backward_work(case)
    elif kind == "optimizer":
        b, f = _optimizer_work(case)
    elif kind == "step":
        (b, f), (b2, f2) = _backward_work(case), _optimizer_work(dict(case, grad="f32"), low=False)
        b, f = b + b2, f + f2
    elif kind == "norms":
        b, f = 12.0 * n, 3.0 * n
    else:
        # the base mask copied in, then read and written once; a key of the keyed permutation (6
        # rounds of 4 integer operations) for every element of the mask
        b, f = n / 8 * 4.0, 24.0 * n
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "reconcile":
        return "exact"
    if kind == "norms":
        return {"rel": 1e-10}
    if kind == "optimizer":
        # fp32 arithmetic per element, without sums; the bf16 copy may round to the next value
        return {"rel": 5e-5, "max": 1e-2}
    if kind == "step":
        # the averages take an update m / sqrt(v) whose m may have cancelled: 6e-6 (single values 9e-5)
        # seen against 64 bits where the gradients are 1e-6 off
        return {"rel": 3e-5, "max": 5e-4}
    if case["io"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}             # fp32 sums of up to 4000 products: 9e-7 and 9e-6 seen against 64 bits
    return {"rel": 4e-3, "max": 1.6e-2}               # fp32 sums rounded to bf16 once: 1.7e-3 and 3.9e-3 seen


# ---------------------------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------
def _exact_backward(case, g):
    W, X, dY, dW0 = _backward_inputs(case, g)
    mask = _frozen(case) if case.get("form") != "rows" else None
    rows = _row_masks(case) if case.get("form") == "rows" else None
    grp = _groups(case) if rows else [-1] * len(W)
    dX, dW = [], []
    for l in range(len(W)):
        y = dY[l].double()
        x = y @ W[l].double().t().contiguous()
        if grp[l] in (-1, l):
            dX.append(x)
        else:
            dX[grp[l]] += x
            dX.append(None)
        if mask is not None and mask[l]:
            dW.append(None)
            continue
        w = X[l].double().t().contiguous() @ y
        if rows and rows[l] is not None:
            w *= torch.from_numpy(1.0 - np.repeat(rows[l], 256)).to(DEV)[:, None]
        dW.append(w if dW0 is None else w + dW0[l].double())
    return dX, dW, mask


def _exact_optimizer(case, s, grad):
    out, sums = {}, torch.zeros_like(s["sums"])
    lr, b1, b2, eps, wd, a = (float(np.float32(x)) for x in (*HYPER.values(), EMA_DECAY))      # as the library receives them
    for i in range(len(s["numel"])):
        if s["mask"][i]:
            continue
        b = {k: seq[i].double() for k, seq in s["buffers"].items()}
        t = int(s["step"][i])
        gr = grad[i].double().reshape(-1) * s["scale"]
        m = b1 * b["m"] + (1 - b1) * gr
        v = b2 * b["v"] + (1 - b2) * gr * gr
        u = -lr * wd * b["p"] - lr * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + eps)
        new = dict(m=m, v=v, p=b["p"] + u, E=a * b["E"] + (1 - a) * u, A=a * b["A"] + (1 - a) * u.abs())
        if "low" in b:
            new["low"] = new["p"]
        if s["bits"] is not None:
            n = s["numel"][i]
            keep = ((s["bits"][i][:, None] >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1).reshape(-1)[:n].bool()
            new = {k: torch.where(keep, b[k], x) for k, x in new.items()}
        out.update({"%s%d" % (k, i): x for k, x in new.items()})
        sums[2 * i], sums[2 * i + 1] = new["E"].abs().sum(), new["A"].sum()
    out["sums"] = sums
    return out


def exact(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind == "reconcile":
        return None
    if kind == "backward":
        dX, dW, mask = _exact_backward(case, g)
        return _backward_out(case, mask, dX, dW)
    if kind == "optimizer":
        s = _prepare_optimizer(case, g)
        return _exact_optimizer(case, s, s["grad"])
    if kind == "norms":
        s = _prepare_norms(case, g)
        p = s["p"][0]
        return {"norms": torch.stack([(a.double() - b.double()).square().sum() for a, b in zip(p, s["snap"])]), "snapshot": [t.double() for t in p]}
    dX, dW, mask = _exact_backward(case, g)
    out = _backward_out(case, mask, dX, dW)
    s = _prepare_optimizer(dict(case, grad="f32", mask="tensor"), g, grads=[torch.empty(0)] * len(_shapes(case)))
    out.update(_exact_optimizer(case, s, dW))
    return out
