"""GPU parity at the sizes the benchmark and the larger configurations run at.
The fp64 oracle cannot produce these outputs in full, so it computes sampled
elements one by one (at least two per 256 x 256 output tile of every layer) and
whole tensors where that is affordable (the elementwise pass).  Bounds: per
element |gpu - exact| <= 2^-8 |exact| + 1e-3 rms (one bf16 rounding of an
fp32-accumulated sum), relative Frobenius error over each layer's sample
<= 1e-2 (bf16) / 1e-5-class bounds for the fp32 optimizer state; frozen buffers
bit-identical; dX independent of the mask (Sec. 3.2.1; App. D.1; Sec. 2.3)."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2602_05754_amd as tf
from gpu_util import GENERIC, WHOLE_256, canary, dev, host64, kinds_of, raw_bytes, rel_fro, route

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tf.Context(0)
    yield c
    c.close()


def _gen(cfg, microbatch=0):
    with ThreadPoolExecutor(max_workers=8) as ex:
        return list(ex.map(lambda l: wl.gen_layer(cfg, l, microbatch=microbatch), range(cfg.n_layers)))


def _tile_samples(rs, rows, cols, per_tile=2, tile=256):
    r, c = [], []
    for tr in range(0, rows, tile):
        for tc in range(0, cols, tile):
            r.append(rs.integers(tr, min(tr + tile, rows), per_tile))
            c.append(rs.integers(tc, min(tc + tile, cols), per_tile))
    return np.concatenate(r), np.concatenate(c)


def _gather(t, r, c):
    ri = torch.from_numpy(np.asarray(r, dtype=np.int64)).cuda()
    ci = torch.from_numpy(np.asarray(c, dtype=np.int64)).cuda()
    return t[ri, ci].to(torch.float64).cpu().numpy()


def _check(got, exact, label, tol_fro=1e-2):
    rms = np.sqrt(np.mean(exact ** 2))
    bad = np.abs(got - exact) > 2.0 ** -8 * np.abs(exact) + 1e-3 * rms
    assert not bad.any(), f"{label}: {bad.sum()} of {bad.size} sampled elements off, worst {np.abs(got - exact).max():.3e} (rms {rms:.3e})"
    e = rel_fro(got, exact)
    assert e <= tol_fro, f"{label}: rel_fro over the sample {e:.3e}"
    return e


def _prepare(cfg):
    """Host arrays (W, X, dY per layer) and their device copies."""
    host = _gen(cfg)
    gW = [dev(h[0], "bf16") for h in host]
    gX = [dev(h[1], "bf16") for h in host]
    gdY = [dev(h[2], "bf16") for h in host]
    return host, gW, gX, gdY


def _backward_case(ctx, cfg, r, seed, prepared=None):
    sh, T, L = cfg.shapes, cfg.T, cfg.n_layers
    host, gW, gX, gdY = prepared if prepared is not None else _prepare(cfg)
    mask = wl.permutation_mask(cfg, r)
    gdX = [canary((T, k), torch.bfloat16) for k, n in sh]
    gdW = [canary((k, n), torch.bfloat16) for k, n in sh]
    before = [t.clone() for t in gdW]
    tf.tf_stage_backward(ctx, sh, T, tf.TF_BF16, gW, gX, gdY, mask, gdX, gdW, tf.TF_BF16)
    torch.cuda.synchronize()
    rs = np.random.default_rng(seed)
    worst = 0.0
    for l, (k, n) in enumerate(sh):
        W, X, dY = host[l]
        ts, ks = _tile_samples(rs, T, k)
        worst = max(worst, _check(_gather(gdX[l], ts, ks), oracle.sample_dx(dY, W, ts, ks), f"dX[{l}] {sh[l]}"))
        if mask[l]:
            assert torch.equal(gdW[l].view(torch.int16), before[l].view(torch.int16)), f"frozen dW[{l}] was touched"
        else:
            kk, nn = _tile_samples(rs, k, n)
            worst = max(worst, _check(_gather(gdW[l], kk, nn), oracle.sample_dw(X, dY, kk, nn), f"dW[{l}] {sh[l]}"))
    # the input gradients do not depend on the mask: r = 1 gives the same bytes
    gdX1 = [torch.empty((T, k), dtype=torch.bfloat16, device="cuda") for k, n in sh]
    tf.tf_stage_backward(ctx, sh, T, tf.TF_BF16, gW, None, gdY, np.ones(L, np.uint8), gdX1, None, tf.TF_BF16)
    torch.cuda.synchronize()
    for l in range(L):
        assert torch.equal(gdX[l].view(torch.int16), gdX1[l].view(torch.int16)), f"dX[{l}] depends on the mask"
    # Freivalds-style projection of two whole outputs: u^T dW v = (X u)^T (dY v), a^T dX b = (a^T dY)(W^T b)
    for l in [i for i in range(L) if not mask[i]][:2]:
        W, X, dY = host[l]
        k, n = sh[l]
        u = rs.choice([-1.0, 1.0], k); v = rs.choice([-1.0, 1.0], n)
        a = rs.choice([-1.0, 1.0], T); b = rs.choice([-1.0, 1.0], k)
        G = host64(gdW[l]); D = host64(gdX[l])
        exact_w = float((X.astype(np.float64) @ u) @ (dY.astype(np.float64) @ v))
        exact_x = float((a @ dY.astype(np.float64)) @ (W.astype(np.float64).T @ b))
        # a random-sign projection of an error field E has standard deviation ||E||_F
        assert abs(float(u @ G @ v) - exact_w) <= 6 * 1e-2 * np.linalg.norm(G)
        assert abs(float(a @ D @ b) - exact_x) <= 6 * 1e-2 * np.linalg.norm(D)
    return worst


def test_llama1b_stage_full_size_as_benchmarked(ctx):
    # BASELINE configs[1]: 4 blocks, d=2048, kv=512, ffn=8192, 4 x 2048 tokens, 28 layers in one grouped launch
    worst = _backward_case(ctx, wl.CONFIGS[2], 0.5, seed=21)
    print(f"cfg2 worst sampled rel_fro {worst:.2e}")


def test_llama8b_stage_all_eight_blocks(ctx):
    """BASELINE configs[2] in full: 8 blocks, 56 layers (d=4096, kv=1024, ffn=14336, 4096 tokens) - one
    grouped launch of 19,456 input-gradient tiles and one of up to 26,624 weight-gradient tiles, 15 GB of
    operands and outputs (tensors lie on both sides of several 4 GiB address boundaries) - at
    r = 0, 0.5 and 0.9 (28 and 51 of 56 tensors frozen); at least two sampled elements per output tile."""
    cfg = wl.CONFIGS[3]
    prepared = _prepare(cfg)
    for r, n_frozen in ((0.0, 0), (0.5, 28), (0.9, 51)):
        assert int(wl.permutation_mask(cfg, r).sum()) == n_frozen
        worst = _backward_case(ctx, cfg, r, seed=22 + int(10 * r), prepared=prepared)
        print(f"cfg3 r={r} worst sampled rel_fro {worst:.2e}")


@pytest.mark.parametrize("which,kind", [(WHOLE_256, "mfma"), (GENERIC, "generic")])
def test_operands_and_outputs_that_cross_a_4gib_address_boundary(ctx, which, kind):
    """Every tensor of a layer in turn is laid across a multiple of 2^32 in the device address
    space, so that the fill addresses of some tile (inputs) or the rows of some tile's epilogue
    (outputs) carry into the high word; whole outputs against the oracle."""
    from gpu_util import assert_elementwise
    k, n, T = 1024, 512, 512
    cfg = wl.scaled(wl.CONFIGS[2], blocks=1, d=k, kv=n, ffn=256, T=T)
    W, X, dY = wl.gen_layer(cfg, 1)                       # layer 1 is the (d, kv) projection
    assert W.shape == (k, n)
    f64 = lambda a: np.asarray(a, dtype=np.float64)
    ref_dX = [np.zeros((T, k))]; ref_dW = [np.zeros((k, n))]
    oracle.stage_backward([(k, n)], T, [f64(W)], [f64(X)], [f64(dY)], np.zeros(1, np.uint8), ref_dX, ref_dW)
    span = (1 << 32) + (64 << 20)
    pool = torch.empty(span, dtype=torch.uint8, device="cuda")
    base = pool.data_ptr()
    edge = (-base) % (1 << 32)                            # offset of the first multiple of 2^32 inside the pool
    if edge < (2 << 20):                                  # too close to the start for a tensor to begin before it
        edge += 1 << 32
    assert edge + (32 << 20) <= span
    sizes = {"W": k * n, "X": T * k, "dY": T * n, "dX": T * k, "dW": k * n}
    shapes = {"W": (k, n), "X": (T, k), "dY": (T, n), "dX": (T, k), "dW": (k, n)}
    src = {"W": W, "X": X, "dY": dY}
    for across in ("W", "X", "dY", "dX", "dW"):
        # the chosen tensor starts 16 (mod 32) bytes before the middle of its bytes reaches the edge,
        # so the edge falls inside a row; the others are packed well away from it
        off = {}
        cursor = 0 if edge > (32 << 20) else edge + (16 << 20)
        for name in sizes:
            if name == across:
                off[name] = edge - ((sizes[name] * 2 // 2 + 16) // 16) * 16
            else:
                off[name] = cursor
                cursor += sizes[name] * 2 + 256
        view = {name: pool[off[name]: off[name] + 2 * sizes[name]].view(torch.bfloat16).view(shapes[name]) for name in sizes}
        lo, hi = base + off[across], base + off[across] + 2 * sizes[across]
        assert lo >> 32 != (hi - 1) >> 32, "the tensor does not cross the boundary"
        for name in src:
            view[name].copy_(dev(src[name], "bf16"))
        view["dX"].copy_(canary((T, k), torch.bfloat16)); view["dW"].copy_(canary((k, n), torch.bfloat16))
        with route(ctx, which):
            kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(
                ctx, [(k, n)], T, tf.TF_BF16, [view["W"]], [view["X"]], [view["dY"]], np.zeros(1, np.uint8),
                [view["dX"]], [view["dW"]], tf.TF_BF16))
        assert kinds == ["dx_" + kind, "dw_" + kind]
        assert_elementwise(host64(view["dX"]), ref_dX[0], "bf16", f"dX with {across} across the boundary")
        assert_elementwise(host64(view["dW"]), ref_dW[0], "bf16", f"dW with {across} across the boundary")
    del pool


@pytest.mark.parametrize("per_layer", [False, True])
def test_llama8b_microbatch_accumulation_then_masked_update(ctx, per_layer):
    # BASELINE configs[4]: 8 sequential calls of 1024 tokens accumulating dW in fp32 for unfrozen
    # tensors only, a different ratio per call; then one optimizer step with grad_scale = 1/M.
    # per_layer: through tf_stage_backward_microbatch, as bench.py times it - nothing is cleared, a
    # layer's first unfrozen microbatch overwrites the canaries its accumulator starts with.
    cfg = wl.scaled(wl.CONFIGS[5], blocks=1)
    sh, T, L, M = cfg.shapes, cfg.T, cfg.n_layers, cfg.microbatches
    ratios = wl.microbatch_ratios(cfg)
    assert len(ratios) == 8 and set(ratios) <= {0.2, 0.4, 0.6, 0.8}
    masks = [wl.permutation_mask(cfg, ratios[m], microbatch=m) for m in range(M)]
    all_frozen = np.minimum.reduce(masks)
    W = [wl.gen_layer(cfg, l, T=8)[0] for l in range(L)]          # weights do not change between microbatches
    gW = [dev(w, "bf16") for w in W]
    acc = [canary((k, n), torch.float32) if all_frozen[l] or per_layer else torch.zeros((k, n), device="cuda")
           for l, (k, n) in enumerate(sh)]
    adds, never = tf.tf_microbatch_plan(np.stack(masks))
    assert np.array_equal(never, all_frozen)
    before = [t.clone() for t in acc]
    rs = np.random.default_rng(23)
    samples = [_tile_samples(rs, k, n, per_tile=1) for k, n in sh]
    exact = [np.zeros(len(s[0])) for s in samples]
    for m in range(M):
        host = _gen(cfg, microbatch=m)
        gX = [dev(h[1], "bf16") for h in host]
        gdY = [dev(h[2], "bf16") for h in host]
        gdX = [torch.empty((T, k), dtype=torch.bfloat16, device="cuda") for k, n in sh]
        if per_layer:
            tf.tf_stage_backward_microbatch(ctx, sh, T, tf.TF_BF16, gW, gX, gdY, masks[m], gdX, acc, tf.TF_F32, adds[m])
        else:
            tf.tf_stage_backward(ctx, sh, T, tf.TF_BF16, gW, gX, gdY, masks[m], gdX, acc, tf.TF_F32, accumulate=True)
        torch.cuda.synchronize()
        for l in range(L):
            if not masks[m][l]:
                exact[l] += oracle.sample_dw(host[l][1], host[l][2], *samples[l])
            if m == 0:
                ts, ks = _tile_samples(rs, T, sh[l][0], per_tile=1)
                _check(_gather(gdX[l], ts, ks), oracle.sample_dx(host[l][2], W[l], ts, ks), f"dX[{l}] microbatch 0")
    for l in range(L):
        if all_frozen[l]:
            assert torch.equal(acc[l].view(torch.int32), before[l].view(torch.int32))
        else:
            _check(_gather(acc[l], *samples[l]), exact[l], f"accumulator[{l}]", tol_fro=1e-4)
    # masked update: a tensor is skipped only if it was frozen in every microbatch; the gradient is sum / M
    hp = {k: float(np.float32(getattr(cfg, k))) for k in ("lr", "beta1", "beta2", "eps", "weight_decay")}
    sizes = [k * n for k, n in sh]
    P = [wl.gen_weight(cfg, l).reshape(-1) for l in range(L)]
    dp = [dev(p, "f32") for p in P]
    dm = [torch.zeros(n, device="cuda") for n in sizes]; dv = [torch.zeros(n, device="cuda") for n in sizes]
    tf.tf_masked_adamw(ctx, sizes, dp, dm, dv, acc, tf.TF_F32, [1] * L, hp["lr"], hp["beta1"], hp["beta2"], hp["eps"],
                       hp["weight_decay"], grad_scale=1.0 / M, tensor_freeze_mask=all_frozen, p_lowp=gW)
    torch.cuda.synchronize()
    for l in range(L):
        if all_frozen[l]:
            assert np.array_equal(dp[l].cpu().numpy(), P[l])
            continue
        idx = rs.integers(0, sizes[l], 200_000)
        g = acc[l].reshape(-1)[torch.from_numpy(idx).cuda()].to(torch.float64).cpu().numpy()   # the bytes the GPU consumed
        p = P[l][idx].astype(np.float64); m_ = np.zeros(idx.size); v_ = np.zeros(idx.size); low = np.zeros(idx.size)
        oracle.masked_adamw(p, m_, v_, g, step=1, grad_scale=1.0 / M, p_lowp=low, **hp)
        got = dp[l][torch.from_numpy(idx).cuda()].to(torch.float64).cpu().numpy()
        assert rel_fro(got, p) <= 1e-5
        assert rel_fro(gW[l].reshape(-1)[torch.from_numpy(idx).cuda()].to(torch.float64).cpu().numpy(), low) <= 1e-2


def test_llama8b_elementwise_pass_with_bernoulli_masks(ctx):
    # BASELINE configs[3] tensors (one block of the 8: 218 M elements, largest tensor 58.7 M): fp32 state,
    # bf16 gradients, element masks Bernoulli(0.3) on the first step (zero state) and Bernoulli(0.7) on the second.
    cfg = wl.scaled(wl.CONFIGS[4], blocks=1)
    L = cfg.n_layers
    sizes = [k * n for k, n in cfg.shapes]
    hp = {k: float(np.float32(getattr(cfg, k))) for k in ("lr", "beta1", "beta2", "eps", "weight_decay")}
    decay = float(np.float32(cfg.ema_decay))
    P = [wl.gen_weight(cfg, l).reshape(-1) for l in range(L)]
    d = {k: [dev(P[l], "f32") if k == "p" else torch.zeros(sizes[l], device="cuda") for l in range(L)] for k in "pmvEA"}
    d["low"] = [dev(P[l], "bf16") for l in range(L)]
    h = [{k: (P[l].astype(np.float64) if k == "p" else np.zeros(sizes[l])) for k in "pmvEA"} for l in range(L)]
    for l in range(L):
        h[l]["low"] = wl.round_to_bf16(P[l]).astype(np.float64)
    sums = torch.zeros(2 * L, dtype=torch.float64, device="cuda")
    for step, r in ((1, 0.3), (2, 0.7)):
        cfg_r = wl.scaled(cfg, cfg_id=40 + step)                  # a different mask and gradient draw per step
        elem = [wl.bernoulli_elem_mask(cfg_r, l, sizes[l], r) for l in range(L)]
        bits = [torch.from_numpy(wl.pack_mask_bits(e).view(np.int32)).cuda() for e in elem]
        grads = [wl.gen_grad(cfg_r, l, step) for l in range(L)]
        before = {k: [t.clone() for t in d[k]] for k in d}
        tf.tf_masked_adamw(ctx, sizes, d["p"], d["m"], d["v"], [dev(g, "bf16") for g in grads], tf.TF_BF16, [step] * L,
                           hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["weight_decay"], p_lowp=d["low"],
                           elem_freeze_bits=bits, ema=d["E"], ema_abs=d["A"], ema_decay=decay, score_sums=sums)
        torch.cuda.synchronize()
        got_sums = sums.cpu().numpy().reshape(L, 2)
        for l in range(L):
            oracle.masked_adamw(h[l]["p"], h[l]["m"], h[l]["v"], grads[l].astype(np.float64), step=step, p_lowp=h[l]["low"],
                                elem_frozen=elem[l], ema=h[l]["E"], ema_abs=h[l]["A"], ema_decay=decay, **hp)
            fz = torch.from_numpy(elem[l]).cuda().bool()
            assert abs(float(fz.float().mean()) - r) < 2e-3
            for k in d:
                e = rel_fro(host64(d[k][l]), h[l][k])
                assert e <= (1e-2 if k == "low" else 1e-5), f"step {step} tensor {l} {k}: rel_fro {e:.3e}"
                a = d[k][l].view(torch.int16 if k == "low" else torch.int32)
                b = before[k][l].view(torch.int16 if k == "low" else torch.int32)
                assert torch.equal(a[fz], b[fz]), f"step {step} tensor {l} {k}: frozen elements changed"
            se, sa = oracle.score_sums(h[l]["E"], h[l]["A"])
            assert np.isclose(got_sums[l, 0], se, rtol=1e-5) and np.isclose(got_sums[l, 1], sa, rtol=1e-5)


def test_llama8b_stage_selection_steps_at_full_size(ctx):
    """AutoFreeze norms and the Alg. 2 reconciliation over all 56 tensors of the 8B stage
    (1.74e9 elements).  Inputs are drawn on the device (the host could not draw them in
    reasonable time); the oracle checks whole tensors where affordable and properties plus
    sampled elements elsewhere."""
    cfg = wl.CONFIGS[3]
    sizes = [k * n for k, n in cfg.shapes]
    L, P = len(sizes), sum(sizes)
    g = torch.Generator(device="cuda").manual_seed(wl.SEED_BASE + 66)
    # --- norms: oracle on the first block's seven tensors in full, the snapshots of all
    p = [torch.randn(n, generator=g, device="cuda") * 0.02 for n in sizes]
    snap = [x + torch.randn(x.numel(), generator=g, device="cuda") * 1e-4 for x in p]
    host = [(p[i].cpu().numpy(), snap[i].cpu().numpy()) for i in range(7)]
    norms = torch.zeros(L, dtype=torch.float64, device="cuda")
    tf.tf_autofreeze_norms(ctx, sizes, p, snap, norms)
    got = norms.cpu().numpy()
    for i in range(7):
        assert got[i] == pytest.approx(oracle.autofreeze_sqnorm(*host[i]), rel=1e-12), i
    for i in range(L):
        assert torch.equal(snap[i], p[i])                                   # snapshot renewed, bit for bit
        assert got[i] == pytest.approx(sizes[i] * 1e-8, rel=0.01)           # E||d||^2 = n sigma^2
    del snap, host
    # --- reconciliation
    base = [(torch.rand((n + 31) // 32 * 32, generator=g, device="cuda") < 0.3).view(-1, 32).to(torch.int64)
            .mul_(2 ** torch.arange(32, device="cuda", dtype=torch.int64)).sum(1).to(torch.int32) for n in sizes]
    base_host = [b.cpu().numpy().view("<u4") for b in base]
    base_ones = sum(int(np.bitwise_count(w).sum()) for w in base_host)
    offs = np.concatenate([[0], np.cumsum(sizes)])
    rs = np.random.default_rng(12)
    for r, seed in ((0.5, 424242), (0.1, 99)):
        nf = int(r * P)
        work = [b.clone() for b in base]
        stats = torch.zeros(3, dtype=torch.int64, device="cuda")
        tf.tf_reconcile_mask(ctx, sizes, work, nf, seed, stats=stats)
        st = stats.cpu().numpy()
        new_host = [w.cpu().numpy().view("<u4") for w in work]
        assert st[0] == base_ones and st[1] == (1 if base_ones < nf else 2)
        assert sum(int(np.bitwise_count(w).sum()) for w in new_host) == nf           # the budget, exactly
        for b, w in zip(base_host, new_host):                                        # superset / subset of the base mask
            assert np.array_equal(w & b, b) if st[1] == 1 else np.array_equal(w | b, b)
        # sampled elements: drawn exactly when a candidate's key does not exceed the largest key drawn
        for t in rs.integers(0, L, 40):
            j = rs.integers(0, sizes[t], 2000)
            key = oracle.perm32(offs[t] + j, seed).astype(np.int64)
            was = (base_host[t][j >> 5] >> (j & 31).astype(np.uint32)) & 1
            now = (new_host[t][j >> 5] >> (j & 31).astype(np.uint32)) & 1
            if st[1] == 1:
                expect = was | ((was == 0) & (key <= st[2]))
            else:
                expect = was & ~((was == 1) & (key <= st[2])).astype(was.dtype)
            assert np.array_equal(now, expect), (r, t)


def test_llama1b_stage_with_row_block_freezing_at_full_size(ctx):
    """cfg 2 at full size with 256-row blocks drawn under the budget 0.5 P: the frozen parameter
    fraction is 0.5 to within one block; sampled dW elements of unfrozen rows against one-by-one
    oracle dots, rows of frozen blocks untouched, dX equal to the unmasked run's."""
    cfg = wl.CONFIGS[2]
    sh, T, L = cfg.shapes, cfg.T, cfg.n_layers
    masks, frozen = tf.tf_select_row_blocks(sh, 256, 0.5, 77)
    ref_masks, ref_frozen = oracle.select_row_blocks(sh, 256, 0.5, 77)
    assert frozen == ref_frozen and all(np.array_equal(a, b) for a, b in zip(masks, ref_masks))
    assert abs(frozen / cfg.n_params - 0.5) < 256 * 8192 / cfg.n_params
    host = _gen(cfg)
    gW = [dev(h[0], "bf16") for h in host]
    gX = [dev(h[1], "bf16") for h in host]
    gdY = [dev(h[2], "bf16") for h in host]
    gdX = [canary((T, k), torch.bfloat16) for k, n in sh]
    gdW = [canary((k, n), torch.bfloat16) for k, n in sh]
    before = [t.clone() for t in gdW]
    tf.tf_stage_backward_blocks(ctx, sh, T, tf.TF_BF16, gW, gX, gdY, None, masks, 256, gdX, gdW, tf.TF_BF16)
    torch.cuda.synchronize()
    rs = np.random.default_rng(31)
    for l, (k, n) in enumerate(sh):
        W, X, dY = host[l]
        ts, ks = _tile_samples(rs, T, k, per_tile=1)
        _check(_gather(gdX[l], ts, ks), oracle.sample_dx(dY, W, ts, ks), f"dX[{l}]")
        kk, nn = _tile_samples(rs, k, n)
        fr = masks[l][kk // 256].astype(bool)
        got = _gather(gdW[l], kk, nn)
        if (~fr).any():
            _check(got[~fr], oracle.sample_dw(X, dY, kk[~fr], nn[~fr]), f"dW[{l}] unfrozen rows")
        for b in np.flatnonzero(masks[l]):
            rows = slice(b * 256, (b + 1) * 256)
            assert torch.equal(gdW[l][rows].view(torch.int16), before[l][rows].view(torch.int16)), f"frozen rows of dW[{l}] touched"


def test_llama1b_stage_with_shared_inputs_at_full_size(ctx):
    """cfg 2 at full size with q/k/v and gate/up of every block sharing their input: sampled
    elements of the grouped dX against the sum of one-by-one oracle dots over the members."""
    cfg = wl.CONFIGS[2]
    sh, T, L = cfg.shapes, cfg.T, cfg.n_layers
    groups = []
    for b in range(cfg.blocks):
        groups += [2 * b, 2 * b, 2 * b, -1, 2 * b + 1, 2 * b + 1, -1]
    host = _gen(cfg)
    gW = [dev(h[0], "bf16") for h in host]
    gdY = [dev(h[2], "bf16") for h in host]
    bufs, gdX = {}, []
    for l, (k, n) in enumerate(sh):
        key = groups[l] if groups[l] >= 0 else -(l + 1)
        if key not in bufs:
            bufs[key] = canary((T, k), torch.bfloat16)
        gdX.append(bufs[key])
    tf.tf_stage_backward_shared(ctx, sh, T, tf.TF_BF16, gW, None, gdY, np.ones(L, np.uint8), None, 0, groups, gdX, None, tf.TF_BF16)
    torch.cuda.synchronize()
    rs = np.random.default_rng(41)
    seen = set()
    for l, (k, n) in enumerate(sh):
        key = groups[l] if groups[l] >= 0 else -(l + 1)
        if key in seen:
            continue
        seen.add(key)
        members = [q for q in range(L) if (groups[q] if groups[q] >= 0 else -(q + 1)) == key]
        ts, ks = _tile_samples(rs, T, k, per_tile=1)
        exact = sum(oracle.sample_dx(host[q][2], host[q][0], ts, ks) for q in members)
        _check(_gather(gdX[l], ts, ks), exact, f"grouped dX of layers {members}")
