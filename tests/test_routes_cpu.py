"""Which kernel a GEMM launch takes (no GPU: the choice is made from the sizes, for 256 compute units).
The launches named here were timed on both kernels; the slower one must not be chosen."""
import ctypes

import pytest

import paper_2602_05754_amd as tf

TILES_256 = -1
GENERIC, FEW_ROWS, FEW_TOKENS = range(3), range(3, 7), range(7, 10)                # launch shapes of the other kernels


def kernels(M, N, Kc, tn, io=tf.TF_BF16, out=tf.TF_BF16, accumulate=False, after=None):
    n = len(M)
    arr = lambda v: (ctypes.c_int64 * n)(*v)
    kernel = (ctypes.c_int32 * n)(*([99] * n))
    assert tf.load_library().tf_internal_kernels(n, arr(M), arr(N), arr(Kc), after and arr(after), int(tn), io, out, int(accumulate), kernel) == 0
    return list(kernel)


def block(d, kv, ffn, blocks=1):
    return [(d, d), (d, kv), (d, kv), (d, d), (d, ffn), (d, ffn), (ffn, d)] * blocks


def without_kv(d, ffn):
    return [(d, d), (d, d), (d, ffn), (d, ffn), (ffn, d)]


# (shapes, tokens, "bf16" / fp32 "set" / fp32 "add", kernel); us on 256 x 256 tiles, on the generic kernel and on the best
# shape of the kernel for few tokens, three sets of buffers in turn
@pytest.mark.parametrize("shapes,T,dw,fastest", [
    (block(1024, 256, 2816), 128, "add", FEW_TOKENS),            # 28.9, 29.7, 21.7
    (block(1024, 256, 2816), 256, "add", FEW_TOKENS),            # 30.4, 37.4, 24.4
    (block(1024, 256, 2816), 200, "add", FEW_TOKENS),            # 30.4, 34.3, 23.5: a contraction that is no multiple of 64
    (block(512, 256, 1536, 3), 256, "add", FEW_TOKENS),          # 31.3, 34.9, 23.1
    (block(512, 256, 1536, 3), 1000, "add", FEW_TOKENS),         # 45.7, 63.9, 37.4
    (block(1024, 256, 2816), 256, "bf16", FEW_TOKENS),           # 16.1, 23.0, 13.5
    (block(1024, 256, 2816), 456, "bf16", FEW_TOKENS),           # 20.6, 27.6, 18.7
    (block(512, 256, 1536, 3), 1024, "set", FEW_TOKENS),         # 39.2, 43.0, 33.4
    (block(512, 256, 1536, 3), 1024, "bf16", FEW_TOKENS),        # 36.5, 40.4, 30.1
    (block(2048, 512, 8192), 256, "add", FEW_TOKENS),            # 120, 176, 97
    (block(512, 256, 1536), 1000, "add", FEW_TOKENS),            # 34.9, 24.2, 18.0
    (block(512, 256, 1536), 128, "add", FEW_TOKENS),             # 21.0, 12.5, 10.4
    (block(256, 256, 768), 1024, "add", FEW_TOKENS),             # 32.5, 14.0, 12.3
    (block(768, 384, 2304), 256, "bf16", FEW_TOKENS),            # 16.1, 14.6, 10.4
    (block(768, 384, 2304), 128, "add", FEW_TOKENS),             # 44.9, 18.4, 16.1
    (block(2048, 512, 8192, 2), 64, "set", FEW_TOKENS),          # 110, 110, 85
    (block(2048, 512, 8192, 2), 200, "add", FEW_TOKENS),         # 214, 321, 176
    (block(2048, 512, 8192, 2), 512, "bf16", [TILES_256]),       # 135, 214, 142
    (block(2048, 512, 8192, 2), 1024, "add", [TILES_256]),       # 307, 484, 334
    (block(4096, 1024, 14336), 512, "bf16", [TILES_256]),        # 213, 376, 243
    (block(2816, 1408, 8200), 512, "add", FEW_TOKENS),           # 227, 310, 181
    (block(1024, 256, 2816, 2), 200, "bf16", FEW_TOKENS),        # 29, 35, 21
    (block(256, 256, 688, 2), 1000, "bf16", FEW_TOKENS),         # 29.9, 15.9, 12.6
    # narrow layers, many tokens: one long chain per unit
    (block(64, 64, 176, 2), 1024, "bf16", FEW_TOKENS),           # -, 12.3, 11.6
    (block(64, 64, 176, 2), 4096, "bf16", GENERIC),              # -, 26.2, 30.0
    (block(128, 64, 344, 2), 8192, "add", GENERIC),              # -, 48.8, 57.5
    (block(192, 96, 512), 3001, "set", GENERIC),                 # -, 21.5, 23.8
    (block(256, 64, 688), 3001, "bf16", GENERIC),                # -, 22.4, 24.9
    (block(384, 128, 1024, 2), 3001, "bf16", FEW_TOKENS),        # 97, 45.9, 37.5
    # many tokens: whole rounds of tiles
    (block(1024, 256, 2816), 3001, "bf16", [TILES_256]),         # 73, 99, 89
    (block(1024, 256, 2816), 4096, "set", [TILES_256]),          # 102, 140, 123
    (without_kv(1024, 4096), 2048, "add", [TILES_256]),          # 71, 131, 89
    (block(512, 256, 1536), 6000, "bf16", FEW_TOKENS),           # 123, 88, 68
    (block(512, 512, 1408, 2), 4096, "bf16", FEW_TOKENS),        # 96, 85, 72
    # large layers, masked last steps: with and without k and v (a frozen pair must not turn the choice)
    (block(3328, 832, 11000), 200, "add", FEW_TOKENS),           # 337, 384, 239
    (without_kv(3328, 11000), 200, "add", FEW_TOKENS),           # 315, -, 232
    (without_kv(2816, 8200), 65, "set", FEW_TOKENS),             # 112, -, 89
    (without_kv(2816, 8200), 200, "add", FEW_TOKENS),            # 184, -, 138
    (without_kv(4096, 14336), 200, "add", FEW_TOKENS),           # 330, -, 308
    (without_kv(4096, 14336), 264, "add", FEW_TOKENS),           # 338, -, 319
    (without_kv(4096, 14336), 200, "bf16", [TILES_256]),         # 142, -, 147
    # few tokens, bf16: large layers take as long on either, and these longer
    (block(4096, 1024, 14336), 100, "bf16", [TILES_256]),        # 109, 160, 118
    (without_kv(4096, 14336), 100, "bf16", [TILES_256]),         # 108, -, 113
    (block(3328, 832, 11000), 100, "bf16", [TILES_256]),         # 92.5, 113, 95.9
])
def test_weight_gradients_take_the_faster_kernel(shapes, T, dw, fastest):
    K, N = zip(*shapes)
    got = kernels(K, N, [T] * len(K), True, out=tf.TF_BF16 if dw == "bf16" else tf.TF_F32, accumulate=dw == "add")
    assert set(got) <= set(fastest), got


# runs of unfrozen row blocks of one block's tensors (widths 1024 / 256 / 2816 and 512 / 256 / 1536)
RUNS_128 = ([128, 256, 256, 128, 128, 256, 128, 128, 128, 128, 128, 128, 384, 384, 128, 128, 128], [1024] * 3 + [256] * 3 + [2816] * 5 + [1024] * 6)
RUNS_64 = ([128] + [64] * 11 + [128, 64, 128, 128, 64, 64, 128, 64], [512] + [256] * 5 + [512] + [1536] * 7 + [512] * 6)
RUNS_256 = ([512, 512, 512, 256, 512, 256, 512, 768, 1280, 1280], [1024, 256, 256, 1024, 1024, 2816, 2816, 2816, 1024, 1024])


# us on 256 x 256 tiles, on the generic kernel and on the best shape of the kernel for few tokens
@pytest.mark.parametrize("runs,T,accumulate,fastest", [
    (RUNS_128, 512, False, FEW_TOKENS),                  # 24.1, 15.0, 11.2
    (RUNS_64, 512, False, FEW_TOKENS),                   # 24.2, 11.4, 9.0
    (RUNS_256, 200, True, FEW_TOKENS),                   # 28.6, 33.7, 19.5
])
def test_row_runs_take_the_faster_kernel(runs, T, accumulate, fastest):
    M, N = runs
    got = kernels(M, N, [T] * len(M), True, out=tf.TF_F32 if accumulate else tf.TF_BF16, accumulate=accumulate, after=[256] * len(M))
    assert set(got) <= set(fastest), got


@pytest.mark.parametrize("shapes,T,on256", [
    (block(1024, 256, 2816), 512, False),                # input gradients: 54.6, 29.1
    (block(2048, 512, 8192), 1024, False),               # 196, 151
    (block(2048, 512, 8192, 3), 1024, True),
    (block(4096, 1024, 14336), 512, False),              # 354, 299
    (block(4096, 1024, 14336), 2048, True),
    (block(2440, 1216, 8744), 928, False),               # 294, 242: partly filled tiles
])
def test_input_gradients_take_the_faster_kernel(shapes, T, on256):
    K, N = zip(*shapes)
    got = kernels([T] * len(K), K, N, False)
    assert len(set(got)) == 1 and (got[0] == TILES_256) == on256, got


# us on the kernel for few rows and on the better one of the others
@pytest.mark.parametrize("shapes,T,few", [
    (block(1024, 256, 2816), 32, True),                  # 13.5, 21.9
    (block(2048, 512, 8192, 2), 200, True),              # 71, 103
    (block(2048, 512, 8192, 4), 256, True),              # 132, 161
    (block(4096, 1024, 14336), 1024, True),              # 382, 434
    (block(2048, 512, 8192, 2), 1536, False),            # 340, 300 on 256 x 256 tiles
    (block(2048, 512, 8192, 4), 1024, False),            # 433, 356
])
def test_few_rows_take_their_own_kernel(shapes, T, few):
    K, N = zip(*shapes)
    got = set(kernels([T] * len(K), K, N, False))
    assert len(got) == 1 and (got <= set(FEW_ROWS)) == few


def test_few_rows_that_their_kernel_cannot_take():
    """A contraction below 64 or no multiple of 8 and fp32 go to the generic kernel, weight gradients to their own."""
    for M, N, Kc, tn, io in ([32, 256, 56, 0, 1], [32, 256, 100, 0, 1], [32, 256, 128, 0, 0]):
        assert 0 <= kernels([M], [N], [Kc], tn, io=io, out=io)[0] < 3
    assert kernels([32], [256], [128], True)[0] in FEW_TOKENS
    assert kernels([32, 32], [256, 256], [128, 100], False) == kernels([32, 32], [256, 256], [100, 100], False)


def test_few_tokens_that_their_kernel_cannot_take():
    """Fewer than 64, extents that are no multiple of 8 and fp32 go to the generic kernel, input gradients to their own; what it
    can take in the same launch goes to it."""
    for M, N, Kc, tn, io in ([256, 256, 63, 1, 1], [36, 256, 128, 1, 1], [256, 36, 128, 1, 1], [256, 256, 128, 1, 0]):
        assert 0 <= kernels([M], [N], [Kc], tn, io=io, out=io)[0] < 3
    assert kernels([64], [256], [128], False)[0] in FEW_ROWS
    assert kernels([256, 128], [256, 64], [128, 128], True)[0] in FEW_TOKENS
    for T, apart in ((128, False), (320, False), (1024, True), (4096, True)):           # whole calls, us, apart and together: 21.6 and 19.2,
        mixed = kernels([2048, 36], [2048, 256], [T, T], True)                          # 26.6 and 25.1, 40.2 and 41.7, 96 and 106
        assert mixed[0] in (FEW_TOKENS if apart else GENERIC) and mixed[1] in GENERIC


TILES = {tf.TF_F32: [(32, 32), (32, 64), (64, 64)], tf.TF_BF16: [(64, 64), (128, 64), (128, 128)]}


@pytest.mark.parametrize("io", [tf.TF_F32, tf.TF_BF16])
@pytest.mark.parametrize("M,N", [((1 << 29) + 5, 4), (4, (1 << 29) + 5), ((1 << 30) - 64, 1), (1, (1 << 30) - 64), (1 << 18, 1 << 17), ((1 << 31) - 128, 1)])
def test_a_launch_has_fewer_than_2_to_the_32_threads(io, M, N):
    """One block of 256 threads per tile: what fits with one of the launch shapes gets it."""
    tiles = [-(-M // m) * -(-N // n) for m, n in TILES[io]]
    if min(tiles) * 256 >= 1 << 32:
        return                                                       # refused, as it was with 64 x 64 tiles
    shape = kernels([M], [N], [3], False, io=io, out=io)[0]
    assert shape >= 0 and tiles[shape] * 256 < 1 << 32


PIECES = range(10, 12)                                             # launch shapes of the fp32 kernel of bf16 pieces


# fp32 launches of one half, us on the generic kernel and in the better tiles of the one of bf16 pieces, three sets of buffers in turn
@pytest.mark.parametrize("shapes,T,tn,fastest", [
    (block(1024, 256, 2731, 2), 1001, False, PIECES),              # 379, 237
    (block(1024, 256, 2731, 2), 1001, True, PIECES),               # 368, 248
    (block(1024, 256, 2731, 2), 350, False, PIECES),               # 152, 119
    (block(1280, 320, 4900), 2048, True, PIECES),                  # 739, 486
    (block(640, 640, 2000, 2), 512, False, PIECES),                # 104, 81
    (block(512, 256, 1700), 2048, False, PIECES),                  # 129, 89
    (block(512, 256, 1700), 512, False, GENERIC),                  # 40, 64: chains of 54 steps in few tiles
    (block(1024, 256, 2731, 2), 100, False, GENERIC),              # 62, 100
    (block(1280, 320, 4900), 37, False, GENERIC),                  # 81, 171
    (block(1024, 256, 2731, 2), 20, True, GENERIC),                # -, 57: less than a step of 32 tokens
    (block(256, 256, 688, 2), 200, True, [0]),                     # 14, 15: short, so in 64 bits
    (block(256, 256, 688, 2), 200, False, [0]),                    # 19, 30: the same
])
def test_fp32_launches_take_the_fastest_kernel(shapes, T, tn, fastest):
    K, N = zip(*shapes)
    M, N, Kc = (K, N, [T] * len(K)) if tn else ([T] * len(K), K, N)
    got = kernels(M, N, Kc, tn, io=tf.TF_F32, out=tf.TF_F32)
    assert len(set(got)) == 1 and got[0] in fastest, got


def test_fp32_problems_that_the_kernel_of_bf16_pieces_does_not_take():
    """Pitches past its 32-bit offsets, contractions past its 32-bit indices, rows shorter than a load: the generic kernel."""
    big = 1 << 22
    assert kernels([2048], [2048], [big], False, io=tf.TF_F32, out=tf.TF_F32)[0] in PIECES
    assert kernels([2048], [2048], [big + 1], False, io=tf.TF_F32, out=tf.TF_F32)[0] in GENERIC      # (packed: the pitch)
    assert kernels([2048], [2048], [(1 << 30) + 1], True, io=tf.TF_F32, out=tf.TF_F32)[0] in GENERIC
    assert kernels([1 << 20], [260], [4096], True, io=tf.TF_F32, out=tf.TF_F32)[0] in PIECES
    assert kernels([1 << 20, 1 << 20], [3, 260], [4096, 4096], True, io=tf.TF_F32, out=tf.TF_F32)[0] in GENERIC
