"""Which kernel a GEMM launch takes (no GPU: the choice is made from the sizes, for 256 compute units).
The launches named here were timed on both kernels; the slower one must not be chosen."""
import ctypes

import pytest

import paper_2602_05754_amd as tf

TILES_256 = -1


def kernels(M, N, Kc, tn, io=tf.TF_BF16, out=tf.TF_BF16, accumulate=False, after=None, few=False):
    n = len(M)
    arr = lambda v: (ctypes.c_int64 * n)(*v)
    kernel = (ctypes.c_int32 * n)(*([99] * n))
    fn = tf.load_library().tf_internal_kernels_few if few else tf.load_library().tf_internal_kernels
    assert fn(n, arr(M), arr(N), arr(Kc), after and arr(after), int(tn), io, out, int(accumulate), kernel) == 0
    return list(kernel)


def block(d, kv, ffn, blocks=1):
    return [(d, d), (d, kv), (d, kv), (d, d), (d, ffn), (d, ffn), (ffn, d)] * blocks


# (shapes, tokens, "bf16" / fp32 "set" / fp32 "add", faster on 256 x 256 tiles); us on 256 x 256 tiles and on the generic kernel
@pytest.mark.parametrize("shapes,T,dw,on256", [
    (block(1024, 256, 2816), 128, "add", True),          # 22.3, 39.3
    (block(1024, 256, 2816), 256, "add", True),          # 24.7, 43.0
    (block(1024, 256, 2816), 200, "add", True),          # 24.4, 42.3: a contraction that is no multiple of 64
    (block(512, 256, 1536, 3), 256, "add", True),        # 25.0, 42.1
    (block(512, 256, 1536, 3), 1000, "add", True),       # 38.6, 59.4
    (block(1024, 256, 2816), 256, "bf16", True),         # 16.9, 21.4
    (block(1024, 256, 2816), 456, "bf16", True),         # 22.3, 27.0
    (block(512, 256, 1536, 3), 1024, "set", True),       # 34.4, 41.7
    (block(512, 256, 1536, 3), 1024, "bf16", True),      # 35.5, 40.9
    (block(2048, 512, 8192), 256, "add", True),          # 109, 160
    (block(512, 256, 1536), 1000, "add", False),         # 30.8, 26.4
    (block(512, 256, 1536), 128, "add", False),          # 17.5, 15.1
    (block(256, 256, 768), 1024, "add", False),          # 30.3, 14.6
    (block(768, 384, 2304), 256, "bf16", False),         # 16.7, 13.8
    (block(768, 384, 2304), 128, "add", False),          # 36.6, 23.6
])
def test_weight_gradients_take_the_faster_kernel(shapes, T, dw, on256):
    K, N = zip(*shapes)
    got = kernels(K, N, [T] * len(K), True, out=tf.TF_BF16 if dw == "bf16" else tf.TF_F32, accumulate=dw == "add")
    assert len(set(got)) == 1 and (got[0] == TILES_256) == on256, got


# runs of unfrozen row blocks of one block's tensors (widths 1024 / 256 / 2816 and 512 / 256 / 1536)
RUNS_128 = ([128, 256, 256, 128, 128, 256, 128, 128, 128, 128, 128, 128, 384, 384, 128, 128, 128], [1024] * 3 + [256] * 3 + [2816] * 5 + [1024] * 6)
RUNS_64 = ([128] + [64] * 11 + [128, 64, 128, 128, 64, 64, 128, 64], [512] + [256] * 5 + [512] + [1536] * 7 + [512] * 6)
RUNS_256 = ([512, 512, 512, 256, 512, 256, 512, 768, 1280, 1280], [1024, 256, 256, 1024, 1024, 2816, 2816, 2816, 1024, 1024])


@pytest.mark.parametrize("runs,T,accumulate,on256", [
    (RUNS_128, 512, False, False),                       # 23.8, 14.1
    (RUNS_64, 512, False, False),                        # 24.5, 10.4
    (RUNS_256, 200, True, True),                         # 22.3, 40.0
])
def test_row_runs_take_the_faster_kernel(runs, T, accumulate, on256):
    M, N = runs
    got = kernels(M, N, [T] * len(M), True, out=tf.TF_F32 if accumulate else tf.TF_BF16, accumulate=accumulate, after=[256] * len(M))
    assert len(set(got)) == 1 and (got[0] == TILES_256) == on256, got


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


FEW_ROWS = range(3, 7)


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
    """A contraction below 64 or no multiple of 8, fp32, and weight gradients go where they went."""
    for M, N, Kc, tn, io in ([32, 256, 56, 0, 1], [32, 256, 100, 0, 1], [32, 256, 128, 0, 0], [32, 256, 128, 1, 1]):
        assert kernels([M], [N], [Kc], tn, io=io, out=io)[0] < 3
    assert kernels([32, 32], [256, 256], [128, 100], False) == kernels([32, 32], [256, 256], [100, 100], False)


# us on the kernel for few tokens and on the better one of the others
@pytest.mark.parametrize("shapes,T,dw,few", [
    (block(2048, 512, 8192, 2), 64, "set", True),        # 85, 110
    (block(2048, 512, 8192, 2), 200, "add", True),       # 176, 214
    (block(2048, 512, 8192, 2), 512, "bf16", False),     # 142, 135
    (block(2048, 512, 8192, 2), 1024, "add", False),     # 334, 307
    (block(4096, 1024, 14336), 512, "bf16", False),      # 243, 213
    (block(2816, 1408, 8200), 512, "add", True),         # 181, 227
    (block(1024, 256, 2816, 2), 200, "bf16", True),      # 21, 29
    (block(256, 256, 688, 2), 1000, "bf16", True),       # 12.6, 15.9
])
def test_few_tokens_take_their_own_kernel(shapes, T, dw, few):
    K, N = zip(*shapes)
    got = set(kernels(K, N, [T] * len(K), True, out=tf.TF_BF16 if dw == "bf16" else tf.TF_F32, accumulate=dw == "add", few=True))
    assert (got <= {7, 8, 9}) if few else (got == {TILES_256}), got


def test_few_tokens_that_their_kernel_cannot_take():
    """Fewer than 64, extents that are no multiple of 8, fp32 and input gradients go where they went; what it can take in the
    same launch goes to it."""
    for M, N, Kc, tn, io in ([256, 256, 63, 1, 1], [36, 256, 128, 1, 1], [256, 36, 128, 1, 1], [256, 256, 128, 1, 0], [64, 256, 128, 0, 1]):
        assert kernels([M], [N], [Kc], tn, io=io, out=io, few=True) == kernels([M], [N], [Kc], tn, io=io, out=io)
    assert kernels([256, 128], [256, 64], [128, 128], True, few=True)[0] >= 7
    mixed = kernels([256, 36], [256, 256], [128, 128], True, few=True)
    assert mixed[0] >= 7 and 0 <= mixed[1] < 3


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
