"""GPU parity of the generic matrix-core GEMM (Sec. 3.2.1, both halves of the backward) where it can
go wrong: extents around its tiles and contraction steps, rows shorter than one 16-byte piece,
pitches that leave rows on any element address, every launch shape, both types.  Outputs lie inside
guard bands, which must come back untouched."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2602_05754_amd as tf
from gpu_util import ALL_256, BY_ESTIMATE, CODE, F32_TILES, GENERIC, NARROW, SHORT, SPLIT, TDT, WHOLE_256, assert_elementwise, canary, common_tiles, dev, host64, kinds_of, raw_bytes, rel_fro, route

pytestmark = pytest.mark.gpu
GUARD = 64


@pytest.fixture(scope="module")
def ctx():
    c = tf.Context(0)
    yield c
    c.close()


def _expected(M, N, Kc, io):
    """Tile of the generic kernel's launch shape for these problems."""
    n = len(M)
    arr = lambda v: (ctypes.c_int64 * n)(*v)
    tile, us = (ctypes.c_int32 * 2)(), ctypes.c_double()
    tf.load_library().tf_internal_generic_shape(n, arr(M), arr(N), arr(Kc), CODE[io], tile, ctypes.byref(us))
    return tuple(tile)


class Guarded:
    """An output of a stage backward between two guard bands."""

    def __init__(self, shape, dtype, fill=None):
        self.n, self.shape = int(np.prod(shape)), shape
        self.all = canary((self.n + 2 * GUARD,), TDT[dtype])
        self.t = self.all[GUARD:GUARD + self.n].view(shape)
        if fill is not None:
            self.t.copy_(fill)
        self.before = raw_bytes(self.all[:GUARD]), raw_bytes(self.all[GUARD + self.n:])

    def check(self, what):
        assert (raw_bytes(self.all[:GUARD]), raw_bytes(self.all[GUARD + self.n:])) == self.before, f"{what}: written outside"


def _case(ctx, shapes, T, io, dw, accumulate=False, seed=0):
    rs = np.random.default_rng(seed)
    L = len(shapes)
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    low = (lambda a: wl.round_to_bf16(f32(a))) if io == "bf16" else f32
    W = [low(rs.standard_normal(s) * 0.02) for s in shapes]
    X = [low(rs.standard_normal((T, k))) for k, n in shapes]
    dY = [low(rs.standard_normal((T, n)) * 1e-3) for k, n in shapes]
    old = [f32(rs.standard_normal(s) * 1e-2) for s in shapes]
    f64 = lambda t: [np.asarray(a, dtype=np.float64) for a in t]
    rX = [np.zeros((T, k)) for k, n in shapes]
    rW = f64(old) if accumulate else [np.zeros(s) for s in shapes]
    if T * sum(k * n for k, n in shapes) < 2e8:
        oracle.stage_backward(shapes, T, f64(W), f64(X), f64(dY), np.zeros(L, np.uint8), rX, rW, accumulate=accumulate)
    else:                                                            # the same in numpy, for the oracle's loops too much
        rX = [y @ w.T for y, w in zip(f64(dY), f64(W))]
        rW = [r + x.T @ y for r, x, y in zip(rW, f64(X), f64(dY))]
    gX = [Guarded((T, k), io) for k, n in shapes]
    gW = [Guarded(s, dw, torch.from_numpy(o) if accumulate else None) for s, o in zip(shapes, old)]
    gin = [[dev(a, io) for a in t] for t in (W, X, dY)]
    kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, shapes, T, CODE[io], *gin, None, [g.t for g in gX], [g.t for g in gW],
                                                       CODE[dw], accumulate=accumulate))
    for l in range(L):
        # one rounding of a sum in 32 bits: the bounds of assert_elementwise
        assert_elementwise(host64(gX[l].t), rX[l], io, f"dX[{l}] {shapes[l]} T={T} {io}")
        assert_elementwise(host64(gW[l].t), rW[l], dw, f"dW[{l}] {shapes[l]} T={T} {io}->{dw}")
        gX[l].check(f"dX[{l}] {shapes[l]} T={T}")
        gW[l].check(f"dW[{l}] {shapes[l]} T={T}")
    return kinds


# steps of 64 (bf16) / 32 (fp32) contraction values, tiles of 32, 64, 128, pieces of 8 / 4 elements
@pytest.mark.parametrize("io,dw,accumulate", [("f32", "f32", False), ("f32", "f32", True), ("bf16", "bf16", False),
                                              ("bf16", "f32", False), ("bf16", "f32", True)])
@pytest.mark.parametrize("T,shapes", [
    (1, [(1, 1), (3, 2), (8, 9), (33, 64)]),                       # outer products, rows shorter than a piece
    (2, [(1, 7), (7, 1), (5, 130)]),
    (31, [(31, 33), (32, 32), (65, 7), (64, 129)]),
    (64, [(128, 64), (127, 63), (129, 65), (4, 200)]),
    (65, [(66, 257), (192, 320), (2, 3)]),
    (191, [(72, 136), (100, 385), (260, 31)]),                     # three bf16 steps less one value
])
def test_edges_of_tiles_steps_and_pieces(ctx, io, dw, accumulate, T, shapes):
    _case(ctx, shapes, T, io, dw, accumulate, seed=T)


@pytest.mark.parametrize("half,io,T,shapes,tile", [
    ("dX", "f32", 130, [(97, 161), (160, 96)], (32, 32)),
    ("dX", "f32", 643, [(1290, 399), (1283, 395)], (32, 64)),
    ("dX", "f32", 2033, [(2047, 731), (2046, 733)] * 3, (64, 64)),
    ("dX", "bf16", 130, [(97, 161), (160, 96)], (64, 64)),
    ("dX", "bf16", 770, [(1027, 1101), (1101, 2030), (1027, 2003)], (128, 64)),
    ("dX", "bf16", 1531, [(1027, 1101), (1101, 2030), (2047, 1003)], (128, 128)),
    ("dW", "f32", 130, [(97, 161), (160, 96)], (32, 32)),
    ("dW", "f32", 391, [(1290, 643), (1283, 643)], (32, 64)),
    ("dW", "f32", 815, [(2047, 2001), (2046, 2005), (2047, 2001)], (64, 64)),
    ("dW", "bf16", 130, [(97, 161), (160, 96)], (64, 64)),
    ("dW", "bf16", 1101, [(1027, 771), (2030, 773)], (128, 64)),
    ("dW", "bf16", 770, [(1027, 1101), (1101, 2030), (1027, 2003)], (128, 128)),
])
def test_every_launch_shape(ctx, half, io, T, shapes, tile):
    K, N = zip(*shapes)
    problems = ([T] * len(K), K, N) if half == "dX" else (K, N, [T] * len(K))
    assert _expected(*problems, io) == tile
    _case(ctx, shapes, T, io, "f32" if io == "f32" else "bf16", seed=3)


@pytest.mark.parametrize("dw,accumulate", [("bf16", False), ("f32", False), ("f32", True)])
@pytest.mark.parametrize("T,shapes", [
    # contractions of the weight gradients with 1, 63, 1, 8 and 1 values more than whole steps; ragged last tiles
    (1025, [(4096, 4096), (4096, 2048)]),
    (1087, [(4104, 2048), (4096, 4104)]),
    (577, [(4096, 4104), (4104, 2056)]),
    (264, [(4096, 2056), (2568, 4096), (2048, 2376)]),
    (65, [(8192, 4104), (8192, 4104)]),
])
def test_contractions_that_are_no_multiple_of_a_step_on_256_tiles(ctx, T, shapes, dw, accumulate):
    with route(ctx, ALL_256):
        kinds = _case(ctx, shapes, T, "bf16", dw, accumulate, seed=T)
    assert "dw_mfma" in kinds and "dw_generic" not in kinds


def test_input_gradients_over_ragged_feature_counts_on_256_tiles(ctx):
    T, shapes = 2048, [(4096, 1032), (4104, 1096), (4096, 328)]
    kinds = _case(ctx, shapes, T, "bf16", "bf16", seed=5)
    assert "dx_mfma" in kinds and "dx_generic" not in kinds


@pytest.mark.parametrize("io,T,K,N,which", [
    ("f32", 37, 45, 70, GENERIC), ("bf16", 37, 45, 70, GENERIC), ("bf16", 577, 4096, 8200, GENERIC), ("bf16", 2048, 4096, 1096, GENERIC),
    # 256 x 256 tiles: contractions of 8 and 1, of 8 and 1, of 8 and none values more than whole steps
    ("bf16", 321, 264, 1096, ALL_256), ("bf16", 577, 4096, 8200, ALL_256), ("bf16", 2048, 4096, 1096, ALL_256),
])
def test_infinities_stay_where_they_are(ctx, io, T, K, N, which):
    """What a last step takes from outside the contraction, or a second time, must not meet an infinity
    or a zero: in either operand, in both layouts."""
    dt = TDT[io]
    for t, n in ((T - 1, N - 1), (T - 64, N - 64)):
        if t < 0:
            continue
        for inf in ("dY", "W and X"):
            W, X, dY = torch.ones(K, N), torch.ones(T, K), torch.ones(T, N)
            rX, rW = torch.full((T, K), float(N)).to(dt).float(), torch.full((K, N), float(T)).to(dt).float()
            if inf == "dY":
                dY[t, n] = float("inf")
                rX[t], rW[:, n] = float("inf"), float("inf")
            else:
                W[K - 1, n] = X[t, K - 1] = float("inf")
                rX[:, K - 1], rW[K - 1] = float("inf"), float("inf")
            dX, dW = torch.empty(T, K, device="cuda", dtype=dt), torch.empty(K, N, device="cuda", dtype=dt)
            gin = [[a.to(dt).cuda()] for a in (W, X, dY)]
            with route(ctx, which):
                kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, [(K, N)], T, CODE[io], *gin, None, [dX], [dW], CODE[io]))
            assert kinds == (["dx_generic", "dw_generic"] if which == GENERIC else ["dx_mfma", "dw_mfma"])
            assert torch.equal(dX.float().cpu(), rX) and torch.equal(dW.float().cpu(), rW)


@pytest.mark.parametrize("T,shapes,which,dx,dw", [
    (256, [(256, 256)], BY_ESTIMATE, "dx_generic", "dw_generic"),       # 256 x 256 tiles fit, the smaller ones are faster
    (256, [(256, 256)], WHOLE_256, "dx_mfma", "dw_mfma"),
    (257, [(256, 256)], WHOLE_256, "dx_mfma", "dw_generic"),
    (257, [(256, 264)], ALL_256, "dx_mfma", "dw_mfma"),
    (4096, [(4096, 4096)] * 2, BY_ESTIMATE, "dx_mfma", "dw_mfma"),
    (2048, [(4096, 4096)], GENERIC, "dx_generic", "dw_generic"),
    (4097, [(4096, 4096)] * 2, BY_ESTIMATE, "dx_mfma", "dw_mfma"),
])
def test_profile_kinds_name_the_kernel_that_ran(ctx, T, shapes, which, dx, dw):
    """The kinds follow the kernel, whatever the shape would allow: the other tests go by them."""
    z = lambda s: [torch.zeros(q, dtype=torch.bfloat16, device="cuda") for q in s]
    W, dW, X, dX, dY = z(shapes), z(shapes), z([(T, k) for k, n in shapes]), z([(T, k) for k, n in shapes]), z([(T, n) for k, n in shapes])
    with route(ctx, which):
        kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, shapes, T, tf.TF_BF16, W, X, dY, None, dX, dW, tf.TF_BF16))
    assert kinds == [dx, dw]


def _random(shapes, T, io, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda s, std: (torch.randn(s, generator=g, device="cuda") * std).to(TDT[io])
    return [rnd(s, 0.02) for s in shapes], [rnd((T, k), 1.0) for k, n in shapes], [rnd((T, n), 1e-3) for k, n in shapes]


@pytest.mark.parametrize("dw,accumulate", [("bf16", False), ("f32", True)])
@pytest.mark.parametrize("T,shapes", [
    (320, [(256, 320), (264, 256)]),                       # whole steps
    (321, [(256, 264), (264, 328), (520, 1096)]),          # 1 value more; 8, 8 and 8
    (127, [(256, 264), (312, 256)]),                       # 63 more (input gradients: fewer rows than a tile)
    (577, [(264, 3000), (256, 2040)]),
])
def test_both_kernels_give_the_same_bf16_bits(ctx, T, shapes, dw, accumulate):
    """Which kernel takes a layer depends on what else is in the launch: its bits must not."""
    W, X, dY = _random(shapes, T, "bf16", T)
    old = [torch.randn(s, device="cuda").to(TDT[dw]) for s in shapes]
    out = []
    for which in (ALL_256, GENERIC):
        dX, dW = [torch.empty_like(x) for x in X], [o.clone() for o in old]
        with route(ctx, which):
            kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, shapes, T, tf.TF_BF16, W, X, dY, None, dX, dW, CODE[dw], accumulate=accumulate))
        assert ("dw_mfma" in kinds) == (which == ALL_256) and ("dw_generic" in kinds) == (which == GENERIC)
        out.append([raw_bytes(t) for t in dX + dW])
    assert out[0] == out[1]


@pytest.mark.parametrize("io,T,others", [("bf16", 577, [(4096, 4096)] * 5), ("bf16", 576, [(4096, 4096)] * 5), ("f32", 500, [(1536, 2048)] * 2)])
def test_a_layers_gradient_does_not_depend_on_the_other_layers(ctx, io, T, others):
    """With the other layers unfrozen the launch takes another kernel or another launch shape.  bf16: the same
    bits.  fp32: the sums are 64-bit ones where the launch is short, in 32 bits otherwise, both
    within the bound of a sum in 32 bits."""
    shapes = [(256, 264)] + others
    W, X, dY = _random(shapes, T, io, T)
    exact = (X[0].double().t().contiguous() @ dY[0].double()).cpu().numpy()
    got = []
    for frozen in (0, 1):
        dX, dW = [torch.empty_like(x) for x in X], [torch.zeros(s, dtype=TDT[io], device="cuda") for s in shapes]
        mask = np.array([0] + [frozen] * len(others), np.uint8)
        kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, shapes, T, CODE[io], W, X, dY, mask, dX, dW, CODE[io]))
        if io == "bf16":
            assert [k for k in kinds if k.startswith("dw")] == ["dw_generic" if frozen else "dw_mfma"]
        assert_elementwise(host64(dW[0]), exact, io, f"dW[0] with the other layers {'frozen' if frozen else 'unfrozen'}")
        got.append((raw_bytes(dX[0]), raw_bytes(dW[0]), host64(dW[0])))
    assert got[0][0] == got[1][0]
    if io == "bf16":
        assert got[0][1] == got[1][1]
    else:
        # chains of at most 32 fp32 products and 16 partial sums against one rounding: 2^-24 (32 + 16)^(1/2) each way,
        # of terms as large as the result's root mean square times sqrt(T) / sqrt(T)
        assert 0 < rel_fro(got[0][2], got[1][2]) <= 2 * 2.0 ** -24 * 48 ** 0.5


@pytest.mark.parametrize("tile", sorted(NARROW))
@pytest.mark.parametrize("T", [1, 63, 65, 128, 200, 257])
def test_input_gradients_of_few_rows(ctx, T, tile):
    """The kernel for few rows where it can go wrong: rows and columns around its tiles, contractions of one step, of
    fewer steps than it has stages, of as many and of more, and 8, 16 or 56 values more than whole steps.  The bits are
    the generic kernel's; an infinity stays in its row and column."""
    shapes = [(64, 64), (1, 72), (130, 128), (63, 136), (129, 320), (65, 376), (257, 1096), (7, 64)]
    with route(ctx, NARROW[tile]):
        kinds = _case(ctx, shapes, T, "bf16", "bf16", seed=T)
    assert kinds[0] == "dx_generic"
    W, X, dY = _random(shapes, T, "bf16", T)
    W[6][5, 1095] = dY[4][T - 1, 319] = float("inf")
    got = {}
    for which in (NARROW[tile], GENERIC):
        out = [Guarded((T, k), "bf16") for k, n in shapes]
        with route(ctx, which):
            tf.tf_stage_backward(ctx, shapes, T, tf.TF_BF16, W, X, dY, np.ones(len(shapes), np.uint8), [g.t for g in out],
                                 [torch.empty(s, dtype=torch.bfloat16, device="cuda") for s in shapes], tf.TF_BF16)
        for l, g in enumerate(out):
            g.check(f"dX[{l}] {shapes[l]} T={T} {tile}")
        got[which] = [raw_bytes(g.t) for g in out]
        assert not torch.isfinite(out[6].t[:, 5]).any() and torch.isfinite(out[6].t[:, :5]).all() and torch.isfinite(out[4].t[:T - 1]).all()
    assert got[NARROW[tile]] == got[GENERIC]


def _across_4_gib(*shape):
    """Zeros in bf16, a 4 GiB boundary of addresses in their middle."""
    size = 2 * int(np.prod(shape))
    room = torch.empty((1 << 32) + size + 16, dtype=torch.uint8, device="cuda")
    half = size // 2 & ~15
    boundary = -(-(room.data_ptr() + half) >> 32) << 32
    first = boundary - half - room.data_ptr()
    t = room[first:first + size].view(torch.bfloat16).view(*shape).zero_()
    assert t.data_ptr() >> 32 != (t.data_ptr() + size - 1) >> 32 and t.data_ptr() % 16 == 0
    return t


def test_few_rows_of_pitches_across_4_gib(ctx):
    """Operands that cross a 4 GiB boundary of addresses, whose rows are far apart: 64-bit base addresses,
    32-bit offsets in a tile."""
    K, N, T = 300, 1 << 19, 65
    W, dY = _across_4_gib(K, N), _across_4_gib(T, N)
    cols = torch.arange(0, N, 4099, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    W[:, cols] = torch.randn((K, cols.numel()), generator=g, device="cuda").bfloat16()
    dY[:, cols] = torch.randn((T, cols.numel()), generator=g, device="cuda").bfloat16()
    ref = dY[:, cols].double() @ W[:, cols].double().t().contiguous()
    X = torch.empty(T, K, dtype=torch.bfloat16, device="cuda")
    for tile in NARROW.values():
        dX = torch.full((T, K), 7.0, dtype=torch.bfloat16, device="cuda")
        with route(ctx, tile):
            tf.tf_stage_backward(ctx, [(K, N)], T, tf.TF_BF16, [W], [X], [dY], np.ones(1, np.uint8), [dX], [torch.empty_like(W)], tf.TF_BF16)
        assert rel_fro(host64(dX), ref.cpu().numpy()) < 4e-3


def test_few_tokens_of_pitches_across_4_gib(ctx):
    """The same for the weight gradients' operands, and gradients that cross a boundary."""
    K, N, T = 72, 1 << 19, 100
    X, dY = torch.randn((T, K), device="cuda").bfloat16(), _across_4_gib(T, N)
    dY[:, ::3] = torch.randn((T, -(-N // 3)), device="cuda").bfloat16()
    W, dX, dW = torch.zeros(K, N, dtype=torch.bfloat16, device="cuda"), torch.empty(T, K, dtype=torch.bfloat16, device="cuda"), _across_4_gib(K, N)
    ref = X.float().t().contiguous() @ dY.float()
    for tile in SHORT.values():
        dW.fill_(7.0)
        with route(ctx, tile):
            tf.tf_stage_backward(ctx, [(K, N)], T, tf.TF_BF16, [W], [X], [dY], None, [dX], [dW], tf.TF_BF16)
        assert float((dW.float() - ref).norm() / ref.norm()) < 4e-3


@pytest.mark.parametrize("tile,dw,accumulate", [(tile, dw, add) for tile in sorted(SHORT) for dw, add in (("bf16", False), ("f32", False), ("f32", True))
                                                if not (add and tile == (256, 128))])          # (that tile does not add)
@pytest.mark.parametrize("T", [64, 65, 96, 97, 128, 200, 257, 1000])
def test_weight_gradients_of_few_tokens(ctx, T, tile, dw, accumulate):
    """The kernel for few tokens where it can go wrong: rows and columns around its tiles, contractions of two steps (fewer
    than it has stages), of three and more, 1, 8, 32 or 33 values more than whole ones.  The bits are the generic kernel's; an
    infinity stays in its row and column; nothing outside the outputs is written."""
    shapes = [(8, 8), (64, 136), (128, 128), (136, 64), (120, 264), (264, 120), (1096, 72), (256, 512)]
    W, X, dY = _random(shapes, T, "bf16", T)
    X[5][T - 1, 263], dY[5][T - 1, :] = float("inf"), dY[5][T - 1, :].abs() + 1e-3
    got = {}
    for which in (SHORT[tile], GENERIC):
        out = [Guarded(s, dw) for s in shapes]
        for g, s in zip(out, shapes):
            g.t.copy_(torch.arange(s[0] * s[1], device="cuda").reshape(s) % 97 * 1e-3)
        dX = [torch.empty_like(x) for x in X]
        with route(ctx, which):
            kinds = kinds_of(ctx, lambda: tf.tf_stage_backward(ctx, shapes, T, tf.TF_BF16, W, X, dY, None, dX, [g.t for g in out], CODE[dw], accumulate=accumulate))
        assert "dw_generic" in kinds and "dw_mfma" not in kinds
        if which != GENERIC:
            assert kinds.count("dw_generic") == 1                        # one launch, whichever could go elsewhere
        for l, g in enumerate(out):
            g.check(f"dW[{l}] {shapes[l]} T={T} {tile}")
        got[which] = [raw_bytes(g.t) for g in out]
    assert got[SHORT[tile]] == got[GENERIC]
    assert torch.isinf(out[5].t[263]).all() and torch.isfinite(out[5].t[:263]).all()
    for l in (2, 6):
        ref = X[l].double().t().contiguous() @ dY[l].double()
        if accumulate:
            ref += (torch.arange(ref.numel(), device="cuda").reshape(ref.shape) % 97 * 1e-3).double()
        assert rel_fro(host64(out[l].t), ref.cpu().numpy()) < (4e-3 if dw == "bf16" else 4e-6)


def test_weight_gradients_of_few_tokens_in_row_runs(ctx):
    """Runs of unfrozen 64-row blocks: operands with the tensor's pitch, rows around the run's own; frozen rows stay."""
    K, N, T = 576, 200, 100
    W, X, dY = _random([(K, N)], T, "bf16", 5)
    rows = [np.array([0, 1, 0, 0, 0, 1, 1, 0, 0], np.uint8)]
    keep = torch.from_numpy(np.repeat(rows[0], 64)).bool()
    got = []
    for which in (*SHORT.values(), GENERIC):
        out = Guarded((K, N), "bf16")
        out.t.fill_(7.0)
        with route(ctx, which):
            tf.tf_stage_backward_blocks(ctx, [(K, N)], T, tf.TF_BF16, W, X, dY, None, rows, 64, [torch.empty_like(X[0])], [out.t], tf.TF_BF16)
        out.check(f"dW {which}")
        assert (out.t.cpu()[keep] == 7.0).all()
        got.append(raw_bytes(out.t))
    assert all(g == got[0] for g in got)
    ref = (X[0].double().t().contiguous() @ dY[0].double()).cpu()
    assert rel_fro(host64(out.t)[~keep.numpy()], ref[~keep].numpy()) < 4e-3


def _both_halves(ctx, T, shapes, form, tiles):
    """An fp32 call launches its two halves together, in tiles that `tiles` accepts (-1: not together); a call that is
    profiled launches them one by one.  The same bits in every gradient."""
    W, X, dY = _random(shapes, T, "f32", T)
    old = [torch.randn(s, device="cuda") for s in shapes]
    L = len(shapes)
    mask = np.array([(form == "frozen" and l != 1) for l in range(L)], np.uint8)
    got = []
    for profiled in (False, True):
        gX, gW = [Guarded((T, k), "f32") for k, n in shapes], [Guarded(s, "f32", o) for s, o in zip(shapes, old)]
        out = [g.t for g in gX], [g.t for g in gW]
        if form == "microbatch":
            add = np.array([l % 2 for l in range(L)], np.uint8)
            call = lambda: tf.tf_stage_backward_microbatch(ctx, shapes, T, tf.TF_F32, W, X, dY, None, *out, tf.TF_F32, add)
        else:
            call = lambda: tf.tf_stage_backward(ctx, shapes, T, tf.TF_F32, W, X, dY, mask, *out, tf.TF_F32, accumulate=form == "add")
        if profiled:
            kinds = kinds_of(ctx, call)
            assert "dx_generic" in kinds and "dw_generic" in kinds and common_tiles(ctx) == -1
        else:
            call()
            torch.cuda.synchronize()
            assert tiles(common_tiles(ctx)), common_tiles(ctx)
        for l in range(L):
            gX[l].check(f"dX[{l}]")
            gW[l].check(f"dW[{l}]")
            if mask[l]:
                assert torch.equal(gW[l].t, old[l])
        got.append([raw_bytes(g.t) for g in gX + gW])
    assert got[0] == got[1]
    ref = dY[1].double() @ W[1].double().t().contiguous()
    assert rel_fro(host64(gX[1].t), ref.cpu().numpy()) < 4e-6
    ref = X[1].double().t().contiguous() @ dY[1].double()
    if form == "add" or form == "microbatch":
        ref += old[1].double()
    assert rel_fro(host64(gW[1].t), ref.cpu().numpy()) < 4e-6


@pytest.mark.parametrize("form", ["set", "add", "microbatch", "frozen"])
@pytest.mark.parametrize("T,shapes", [
    (1, [(1, 1), (33, 70)]),
    (256, [(256, 256), (256, 688), (688, 256)]),                   # both halves in 64 bits
    (391, [(1290, 643), (643, 1283), (31, 5)]),
    (815, [(2047, 1001), (1046, 1005), (1047, 1001)] * 2),
    (40, [(96, 40 + l) for l in range(40)]),                       # more problems than one launch holds, but for `microbatch` and `frozen`
])
def test_both_halves_in_one_launch_give_the_same_bits(ctx, T, shapes, form):
    too_many = len(shapes) == 40 and form in ("set", "add")
    _both_halves(ctx, T, shapes, form, lambda tiles: (tiles == -1) == too_many)


@pytest.mark.parametrize("form", ["set", "add"])
@pytest.mark.parametrize("pair", range(9))
def test_both_halves_in_every_pair_of_tiles(ctx, pair, form):
    """The halves' tiles differ, and the larger ones' stages make the LDS: every pair, at sizes around the tiles of each and a
    contraction shorter than a step."""
    with route(ctx, F32_TILES + pair):
        _both_halves(ctx, 65, [(31, 33), (129, 63), (64, 200), (3, 7), (95, 257)], form, lambda tiles: tiles == pair)
        _both_halves(ctx, 20, [(33, 12), (70, 129)], form, lambda tiles: tiles == pair)


@pytest.mark.parametrize("tile", sorted(SPLIT))
@pytest.mark.parametrize("T", [32, 33, 61, 95, 128, 160, 191, 257])
def test_fp32_calls_of_bf16_pieces(ctx, T, tile):
    """The kernel that splits fp32 values into three bf16 pieces where it can go wrong: rows and columns around its tiles, rows that
    end inside a 16-byte load, contractions of one step to more than are on their way, 1 to 31 values more than whole ones.  The same
    bits in both tiles, in one launch and two; no less exact than sums of fp32 products in 32 bits."""
    shapes = [(4, 33), (5, 32), (127, 95), (128, 129), (130, 64), (255, 34), (258, 63), (64, 261), (7, 385)]
    for accumulate in (False, True):
        with route(ctx, SPLIT[tile]):
            kinds = _case(ctx, shapes, T, "f32", "f32", accumulate, seed=T)
        assert kinds == ["dx_generic", "dw_generic"]
    W, X, dY = _random(shapes, T, "f32", T)
    got, errors = {}, {}
    for which in (*SPLIT.values(), F32_TILES + 4):
        out = [[Guarded((T, k), "f32") for k, n in shapes], [Guarded(s, "f32") for s in shapes]]
        with route(ctx, which):
            tf.tf_stage_backward(ctx, shapes, T, tf.TF_F32, W, X, dY, None, *[[g.t for g in half] for half in out], tf.TF_F32)
        assert common_tiles(ctx) == (4 if which == F32_TILES + 4 else 9 + which - min(SPLIT.values()))
        got[which] = [raw_bytes(g.t) for half in out for g in half]
        exact = [y.double() @ w.double().t().contiguous() for y, w in zip(dY, W)] + [x.double().t().contiguous() @ y.double() for x, y in zip(X, dY)]
        errors[which] = sum(rel_fro(host64(g.t), e.cpu().numpy()) ** 2 for g, e in zip(out[0] + out[1], exact)) ** 0.5
        for g in out[0] + out[1]:
            g.check(f"T={T} {which}")
    assert got[20] == got[21]
    assert errors[20] <= 1.05 * errors[F32_TILES + 4]              # (of 18 outputs, some of a few values: a rounding more or less)


def _against_64_bits(ctx, which, W, X, dY):
    """dX and dW of one layer on that route: relative rms and mean error (towards larger magnitudes) and the largest relative one of both."""
    dX, dW = [torch.empty_like(X)], [torch.empty_like(W)]
    with route(ctx, which):
        tf.tf_stage_backward(ctx, [tuple(W.shape)], X.shape[0], tf.TF_F32, [W], [X], [dY], None, dX, dW, tf.TF_F32)
    out = []
    for got, exact in ((dX[0], dY.double() @ W.double().t().contiguous()), (dW[0], X.double().t().contiguous() @ dY.double())):
        d = got.double() - exact
        out.append([float(d.norm() / exact.norm()), float((d * exact.sign()).mean() / exact.abs().mean()), float((d / exact).abs().max())])
    return np.array(out)


@pytest.mark.parametrize("tile", sorted(SPLIT))
@pytest.mark.parametrize("T", [64, 200, 1000])
@pytest.mark.parametrize("operands", ["absolute values of normal ones", "1 to 1.01", "1 to 2"])
def test_fp32_products_of_one_sign_have_no_error_of_one_sign(ctx, operands, T, tile):
    """What the three pieces of two values leave out of their product is as often too much as too little: sums of products of one sign are no
    further off than sums of fp32 products in 32 bits.  (Mean of some 10^5 errors of 2^-24 and less, each row's and column's in common: 2^-30;
    pieces cut off and not rounded are off by 2^-25 to 2^-24 on average.)"""
    rs = np.random.default_rng(T)
    draw = {"absolute values of normal ones": lambda *s: np.abs(rs.standard_normal(s)), "1 to 1.01": lambda *s: rs.uniform(1, 1.01, s),
            "1 to 2": lambda *s: rs.uniform(1, 2, s)}[operands]
    W, X, dY = (dev(draw(*s).astype(np.float32), "f32") for s in ((260, T), (T, 260), (T, T)))         # both contractions are of T
    pieces, generic = (_against_64_bits(ctx, which, W, X, dY) for which in (SPLIT[tile], F32_TILES + 4))
    assert (pieces[:, 0] <= 1.02 * generic[:, 0]).all(), (pieces, generic)
    assert (np.abs(pieces[:, 1]) <= 2.0 ** -27).all(), pieces


@pytest.mark.parametrize("tile", sorted(SPLIT))
@pytest.mark.parametrize("T", [64, 200])
@pytest.mark.parametrize("value", [1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -17 - 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -17 + 2.0 ** -23])
def test_fp32_products_of_the_worst_mantissas(ctx, value, T, tile):
    """Equal operands, so that all errors add up.  Cut off, pieces lose most where the lower 16 bits are all ones, 2^-21 of the product;
    rounded, where the first two are off by half of their last places: 2 * 2^-8 * 2^-17.  Besides, in units of 2^-24 of the result: a step's last
    instruction rounds at 1/4, 1/2, 3/4 and all of its sum, the five before it at 2^-7 of that; S steps' sums are added, at (S + 1) / 2 of the result."""
    W, X, dY = (torch.full(s, value, device="cuda") for s in ((260, T), (T, 260), (T, T)))
    bound = 2.0 ** -24 * (1.01 + 2.5 + 5 * 4 * 2.0 ** -7 + ((T + 31) // 32 + 1) / 2)
    got = _against_64_bits(ctx, SPLIT[tile], W, X, dY)
    assert (got[:, 2] <= bound).all(), (got, bound)


@pytest.mark.parametrize("tile", sorted(SPLIT))
@pytest.mark.parametrize("T", [64, 200])
@pytest.mark.parametrize("first,second", [(-106, 0), (-110, 0), (-58, -58), (-64, -64)])
def test_fp32_pieces_and_products_below_the_smallest_normal_number(ctx, first, second, T, tile):
    """Third pieces of values of 2^-110 and more, and products of pieces whose whole product is a normal number, may be subnormal; the
    matrix instructions keep them.  Nothing is computed again (other bits than the generic kernel's), and no error is larger than that
    kernel's - all operands are +-(1 .. 2) 2^first and 2^second, so that all of them lie in that range."""
    rs = np.random.default_rng(T)
    draw = lambda s, e: dev((rs.uniform(1, 2, s) * rs.choice([-1, 1], s) * 2.0 ** e).astype(np.float32), "f32")
    W, X, dY = draw((260, T), first), draw((T, 260), first), draw((T, T), second)
    pieces, generic = (_against_64_bits(ctx, which, W, X, dY) for which in (SPLIT[tile], F32_TILES + 4))
    assert (pieces[:, 0] <= generic[:, 0]).all() and (pieces[:, 0] != generic[:, 0]).all(), (pieces, generic)


def _whole_blocks(odd):
    """The blocks of 32 x 64 that have one."""
    all_of = torch.zeros_like(odd)
    for m in range(0, odd.shape[0], 32):
        for n in range(0, odd.shape[1], 64):
            all_of[m:m + 32, n:n + 64] = odd[m:m + 32, n:n + 64].any()
    return all_of


@pytest.mark.parametrize("tile", sorted(SPLIT))
@pytest.mark.parametrize("what", ["infinity", "overflow", "tiny"])
def test_values_that_bf16_pieces_cannot_hold(ctx, what, tile):
    """An infinity meets the zeros among another value's pieces, a sum of pieces may leave the range where the sum does not, and pieces of
    values below 2^-110 lose bits: blocks of 32 x 64 outputs that have such ones are computed from fp32 products, with the bits of the generic kernel."""
    T, shapes = 100, [(300, 200)]
    W, X, dY = _random(shapes, T, "f32", 3)
    if what == "infinity":
        dY[0][T - 1, 150], W[0][17, 3], X[0][50, 299] = float("inf"), float("-inf"), float("inf")
    elif what == "overflow":
        X[0] *= 1e38
        dY[0] *= 1e35
        W[0] *= 1e38
    else:
        X[0] *= 2.0 ** -115
        W[0] *= 2.0 ** -112
    got = []
    for which in (SPLIT[tile], F32_TILES + 4):
        dX, dW = [torch.zeros_like(X[0])], [torch.zeros_like(W[0])]
        with route(ctx, which):
            tf.tf_stage_backward(ctx, shapes, T, tf.TF_F32, W, X, dY, None, dX, dW, tf.TF_F32)
        got.append((dX[0], dW[0]))
    for a, b in zip(*got):
        redone = torch.ones_like(a, dtype=torch.bool)
        if what == "infinity":                                     # only blocks with a sum that is not finite
            redone = _whole_blocks(~torch.isfinite(b))
            assert redone.any()
        elif what == "overflow":
            redone = ~torch.isfinite(b)
            assert redone.any()
        assert torch.equal(a[redone].view(torch.int32), b[redone].view(torch.int32))
        assert torch.equal(torch.isfinite(a), torch.isfinite(b))


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("T,where", [(70, 69), (257, 3), (300, 130)])
@pytest.mark.parametrize("what", ["infinity", "nan", "a tiny value", "a tiny row"])
def test_odd_values_change_the_bits_of_their_own_blocks_only(ctx, what, T, where, accumulate):
    """One infinity per layer in dY: its row of dX and its column of dW are computed again, in blocks of 32 x 64 that are the same in both
    tiles (two at a time, of an odd number the last beside one beyond the matrix), and nothing else changes a bit; with `accumulate` what
    was there is added to once.  A row of tiny values is computed again where it is all that a sum consists of: in dX.  A NaN, and a
    tiny value that loses bits (2^-120 + 2^-140: the 2^-140) among ordinary ones, have nothing computed again."""
    shapes = [(300, 200), (257, 330), (70, 129)]
    W, X, clean = _random(shapes, T, "f32", T)
    old = [torch.randn(s, device="cuda") for s in shapes]
    dY = [y.clone() for y in clean]
    for y, c in zip(dY, clean):
        at = slice(None) if what == "a tiny row" else y.shape[1] - 1
        y[where, at] = {"infinity": float("inf"), "nan": float("nan")}.get(what, 2.0 ** -120 + 2.0 ** -140)
        if what.startswith("a tiny"):
            c[where, at] = 2.0 ** -120

    def run(which, dY):
        dX, dW = [Guarded((T, k), "f32") for k, n in shapes], [Guarded(s, "f32", o) for s, o in zip(shapes, old)]
        with route(ctx, which):
            tf.tf_stage_backward(ctx, shapes, T, tf.TF_F32, W, X, dY, None, [g.t for g in dX], [g.t for g in dW], tf.TF_F32, accumulate=accumulate)
        for g in dX + dW:
            g.check(f"T={T} {which}")
        return [g.t for g in dX + dW]

    plain, fp32 = run(20, clean), run(F32_TILES + 4, dY)
    for which in SPLIT.values():
        for i, (got, without, generic) in enumerate(zip(run(which, dY), plain, fp32)):
            odd = ~torch.isfinite(generic)
            assert odd.any() == (what in ("infinity", "nan")) and not odd.all()
            blocks = _whole_blocks(odd)
            if what == "nan":                                      # (which NaN it is nobody promises)
                assert torch.equal(torch.isnan(got), odd)
                blocks[:] = False
                got, without = torch.where(odd, 0, got), torch.where(odd, 0, without)
            if what == "a tiny row" and i < len(shapes):
                odd[where] = True
                blocks = _whole_blocks(odd)
            assert torch.equal(got.view(torch.int32), torch.where(blocks, generic, without).view(torch.int32)), (which, i, tuple(got.shape))


@pytest.mark.parametrize("form", ["set", "add", "microbatch", "frozen"])
def test_both_halves_of_bf16_pieces_give_the_same_bits(ctx, form):
    """Both halves in one launch of the kernel of bf16 pieces, by the estimates: the bits of a launch each."""
    _both_halves(ctx, 1000, [(1024, 1024), (1024, 2731), (2731, 1024)], form, lambda tiles: tiles >= 9)
