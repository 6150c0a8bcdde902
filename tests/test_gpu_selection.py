"""GPU parity of the AutoFreeze norms (Sec. 2.3) and of the Alg. 2 budget
reconciliation (App. "Hybrid Variants Algorithm") against the oracle.
Bounds: squared norms within 1e-12 relative (fp64 sums of exact differences;
only the order of summation differs); snapshots, masks, counts and the largest
key drawn bit-exact."""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2602_05754_amd as tf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tf.Context(0)
    yield c
    c.close()


def _f32(a):
    return np.ascontiguousarray(a, dtype=np.float32)


# ---------------------------------------------------------------- AutoFreeze
@pytest.mark.parametrize("update", [True, False])
def test_autofreeze_norms_and_snapshot(ctx, update):
    rs = np.random.default_rng(260205754 + int(update))
    numel = [1, 3, 4096, 4097, 5 * 4096 + 1234, 256 * 688, 100003]     # one element ... several blocks and ragged tails
    p = [_f32(rs.standard_normal(n) * 0.02) for n in numel]
    snap = [_f32(a + rs.standard_normal(a.size) * 1e-4) for a in p]
    mask = np.zeros(len(numel), np.uint8)
    mask[2] = 1                                                       # one tensor skipped
    dp = [torch.from_numpy(a).cuda() for a in p]
    ds = [torch.from_numpy(a).cuda() for a in snap]
    out = torch.full((len(numel),), -7.0, dtype=torch.float64, device="cuda")
    tf.tf_autofreeze_norms(ctx, numel, dp, ds, out, tensor_freeze_mask=mask, update_snapshot=update)
    got = out.cpu().numpy()
    for i, n in enumerate(numel):
        if mask[i]:
            assert got[i] == -7.0                                      # skipped: untouched
            assert np.array_equal(ds[i].cpu().numpy(), snap[i])
            continue
        ref = oracle.autofreeze_sqnorm(p[i], snap[i])
        assert got[i] == pytest.approx(ref, rel=1e-12), (i, n)
        assert np.array_equal(ds[i].cpu().numpy(), p[i] if update else snap[i])      # bit-exact snapshot
        assert np.array_equal(dp[i].cpu().numpy(), p[i])                             # parameters only read
    if update:      # a second check right away sees no movement at all
        tf.tf_autofreeze_norms(ctx, numel, dp, ds, out, tensor_freeze_mask=mask, update_snapshot=True)
        got2 = out.cpu().numpy()
        assert all(got2[i] == 0.0 for i in range(len(numel)) if not mask[i])


def test_autofreeze_norms_with_more_tensors_than_one_launch_holds(ctx):
    """75 tensors need three launches of the norm pass; the per-tensor sums are gathered through
    slots that every launch must leave zero for the next one (also for the optimizer's score sums,
    which share them).  Sizes from one element to many one-wave blocks per slot."""
    rs = np.random.default_rng(260205754 + 77)
    numel = [int(n) for n in rs.integers(1, 3000, size=72)] + [64 * 512 * 3 + 5, 700001, 2]
    p = [_f32(rs.standard_normal(n) * 0.02) for n in numel]
    snap = [_f32(a + rs.standard_normal(a.size) * 1e-4) for a in p]
    mask = np.zeros(len(numel), np.uint8)
    mask[[5, 40, 73]] = 1
    dp = [torch.from_numpy(a).cuda() for a in p]
    ds = [torch.from_numpy(a).cuda() for a in snap]
    out = torch.full((len(numel),), -7.0, dtype=torch.float64, device="cuda")
    for rep in range(2):            # the second call finds the slots as the first left them
        tf.tf_autofreeze_norms(ctx, numel, dp, ds, out, tensor_freeze_mask=mask, update_snapshot=False)
        got = out.cpu().numpy()
        for i, n in enumerate(numel):
            if mask[i]:
                assert got[i] == -7.0
            else:
                assert got[i] == pytest.approx(oracle.autofreeze_sqnorm(p[i], snap[i]), rel=1e-12), (rep, i, n)
    # the optimizer's score sums go through the same slots: still exact after the norm passes
    n = 3000
    E = _f32(rs.standard_normal(n) * 1e-5)
    A = _f32(np.abs(rs.standard_normal(n)) * 1e-4)
    d = _f32(rs.standard_normal(n) * 1e-5)
    dE, dA, dd = (torch.from_numpy(x.copy()).cuda() for x in (E, A, d))
    sums = torch.zeros(2, dtype=torch.float64, device="cuda")
    tf.tf_stability_update(ctx, [n], [dd], [dE], [dA], 0.99, score_sums=sums)
    E64, A64 = E.astype(np.float64), A.astype(np.float64)
    oracle.stability_update(d.astype(np.float64), E64, A64, 0.99)
    assert sums.cpu().numpy() == pytest.approx(np.array(oracle.score_sums(E64, A64)), rel=1e-5)


def test_autofreeze_check_sequence_matches_the_oracle_rule(ctx):
    """Three checks of a 14-layer stage whose early layers move less and less: norms -> scores ->
    prefix selection, every step against the oracle."""
    rs = np.random.default_rng(99)
    L = 14
    numel = [256 * 256] * 8 + [256 * 688] * 6
    p = [_f32(rs.standard_normal(n) * 0.02) for n in numel]
    dp = [torch.from_numpy(a.copy()).cuda() for a in p]
    ds = [torch.from_numpy(a.copy()).cuda() for a in p]
    host_snap = [a.copy() for a in p]
    out = torch.zeros(L, dtype=torch.float64, device="cuda")
    sq_prev = sq_prev_ref = None
    frozen = 0
    for check in range(3):
        for l in range(L):                                            # the interval's cumulative update
            scale = 1e-3 * (1.0 if l >= 5 else 0.5 ** check) * (1.0 + 0.3 * rs.random())
            p[l] = _f32(p[l] + rs.standard_normal(numel[l]) * scale)
            dp[l].copy_(torch.from_numpy(p[l]))
        tf.tf_autofreeze_norms(ctx, numel, dp, ds, out)
        sq = out.cpu().numpy().copy()
        sq_ref = np.array([oracle.autofreeze_sqnorm(p[l], host_snap[l]) for l in range(L)])
        assert np.allclose(sq, sq_ref, rtol=1e-12, atol=0)
        host_snap = [a.copy() for a in p]
        if sq_prev is not None:
            sc = tf.tf_autofreeze_scores(sq_prev, sq)
            sc_ref = np.array([oracle.autofreeze_score(a, b) for a, b in zip(sq_prev_ref, sq_ref)])
            assert np.allclose(sc, sc_ref, rtol=1e-9)
            m = tf.tf_autofreeze_select(sc, frozen, 80.0)
            assert np.array_equal(m, oracle.autofreeze_select(sc_ref, frozen, 80.0))
            frozen = int(m.sum())
        sq_prev, sq_prev_ref = sq, sq_ref
    assert frozen >= 1                                                 # the slowing prefix did get frozen


# -------------------------------------------------------------------- Alg. 2
def _run_reconcile(ctx, base, numel, n_freeze, seed):
    words = [torch.from_numpy(oracle.pack_bits(b).view(np.int32)).cuda() for b in base]
    stats = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    tf.tf_reconcile_mask(ctx, numel, words, n_freeze, seed, stats=stats)
    got = [oracle.unpack_bits(w.cpu().numpy().view("<u4"), n) for w, n in zip(words, numel)]
    raw = [w.cpu().numpy().view("<u4") for w in words]
    return got, raw, stats.cpu().numpy()


@pytest.mark.parametrize("density", [0.0, 0.3, 0.7, 1.0])
def test_reconcile_matches_the_oracle_bit_for_bit(ctx, density):
    rs = np.random.default_rng(int(density * 10) + 40)
    numel = [1, 31, 32, 33, 4097, 32768, 32769, 100003, 5]           # word / block boundaries and ragged tails
    N = sum(numel)
    base = [(rs.random(n) < density).astype(np.uint8) for n in numel]
    c = int(sum(int(b.sum()) for b in base))
    for r in (0.0, 0.25, 0.5, 0.9, 1.0):
        nf = math.floor(r * N)
        seed = 0xC0FFEE ^ (nf * 7919)
        got, raw, stats = _run_reconcile(ctx, base, numel, nf, seed)
        ref, count = oracle.reconcile_mask(base, numel, nf, seed)
        for g, e in zip(got, ref):
            assert np.array_equal(g, e)
        assert stats[0] == count == c
        assert stats[1] == (0 if c == nf else 1 if c < nf else 2)
        assert sum(int(g.sum()) for g in got) == nf
        for w, n in zip(raw, numel):                                   # bits past the end of a tensor stay clear
            if n % 32:
                assert int(w[-1]) >> (n % 32) == 0
    got, _, stats = _run_reconcile(ctx, base, numel, c, 5)             # budget already met
    assert all(np.array_equal(g, b) for g, b in zip(got, base)) and stats[1] == 0


def test_reconcile_more_tensors_than_one_launch_holds(ctx):
    rs = np.random.default_rng(8)
    numel = [int(n) for n in rs.integers(1, 3000, size=70)]           # 70 tensors: two launches per pass
    base = [(rs.random(n) < 0.4).astype(np.uint8) for n in numel]
    N = sum(numel)
    for nf in (N // 5, (4 * N) // 5):
        got, _, stats = _run_reconcile(ctx, base, numel, nf, 123456789)
        ref, _ = oracle.reconcile_mask(base, numel, nf, 123456789)
        assert all(np.array_equal(g, e) for g, e in zip(got, ref))


@pytest.mark.parametrize("first", [7, 32, 65535])
@pytest.mark.parametrize("r", [0.2, 0.6])
def test_reconcile_where_indices_cross_65536_inside_a_word(ctx, first, r):
    """Tensors of more than 16 rows of 2^16 elements (a task of the keyed passes) that start anywhere in the
    stage's index space: low halves of the indices wrap inside a word, and with 3.4e6 keys some fifty
    share the top half of the threshold."""
    rs = np.random.default_rng(first)
    numel = [first, 17 * 65536 + 5, 3, 2200001]
    base = [(rs.random(n) < 0.4).astype(np.uint8) for n in numel]
    base[3][600000:800000] = 1                                          # stretches without a candidate
    base[3][900000:1100000] = 0
    nf = math.floor(r * sum(numel))
    got, _, stats = _run_reconcile(ctx, base, numel, nf, 9 + first)
    ref, count = oracle.reconcile_mask(base, numel, nf, 9 + first)
    assert all(np.array_equal(g, e) for g, e in zip(got, ref)) and stats[0] == count


@pytest.mark.parametrize("candidate", [0, 1])
@pytest.mark.parametrize("per_word", [(0, 1), (7,), (0, 7, 8), (1, 2, 32)])
def test_reconcile_words_with_few_candidates(ctx, per_word, candidate):
    """Waves whose words have at most seven candidates each look at them one by one, others at all 32
    elements: stretches of 64 words (a wave's) with every number around that limit, and stretches that mix them."""
    rs = np.random.default_rng(len(per_word))
    n_words = 64 * 70
    numel = [32 * n_words, 32 * n_words - 13, 77]
    base = []
    for n in numel:
        c = rs.choice(per_word, size=(n + 31) // 32)
        rank = rs.random((len(c), 32)).argsort(axis=1)               # c random places of a word are candidates
        bits = np.where(rank < c[:, None], candidate, 1 - candidate).astype(np.uint8).reshape(-1)[:n]
        base.append(np.ascontiguousarray(bits))
    ones, have = sum(int(b.sum()) for b in base), sum(int((b == candidate).sum()) for b in base)
    for share in (0.0, 0.4, 1.0):
        nf = ones + int(share * have) * (-1 if candidate else 1)
        got, _, stats = _run_reconcile(ctx, base, numel, nf, 31 + int(10 * share))
        ref, count = oracle.reconcile_mask(base, numel, nf, 31 + int(10 * share))
        assert all(np.array_equal(g, e) for g, e in zip(got, ref)) and stats[0] == count == ones
        assert sum(int(g.sum()) for g in got) == nf


def test_reconcile_threshold_is_the_largest_key_drawn(ctx):
    rs = np.random.default_rng(3)
    numel = [50000, 70001]
    base = [(rs.random(n) < 0.5).astype(np.uint8) for n in numel]
    flat = np.concatenate(base)
    c, N = int(flat.sum()), sum(numel)
    keys = oracle.perm32(np.arange(N), 77).astype(np.int64)
    got, _, stats = _run_reconcile(ctx, base, numel, c + 1234, 77)
    new = np.concatenate(got)
    added = np.flatnonzero((new == 1) & (flat == 0))
    assert added.size == 1234 and stats[2] == keys[added].max()
    got, _, stats = _run_reconcile(ctx, base, numel, c - 999, 77)
    new = np.concatenate(got)
    dropped = np.flatnonzero((new == 0) & (flat == 1))
    assert dropped.size == 999 and stats[2] == keys[dropped].max()


# ---- large masks: the threshold is guessed, and the general passes are there where the guess does not hold
GUESS_FROM = 1 << 28


def _random_words(g, n, p):
    words = torch.zeros(n, dtype=torch.int32, device="cuda")
    for b in range(16):
        r = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
        words = (words | r) if (int(p * 65536) >> b) & 1 else (words & r)
    return words


def _key_words(numel, seed, test):
    """Words whose bit e says test(key of element e), the elements counted from the first tensor on."""
    mul, mask, k = 0x9E3779B1, 0xffffffff, [(seed >> (16 * r)) & 0xffff for r in range(4)]
    s2 = seed * 0xD1342543DE82EF95 % (1 << 64)
    k += [(s2 >> 32) & 0xffff, (s2 >> 48) & 0xffff]
    place = (1 << torch.arange(32, device="cuda", dtype=torch.int64))
    out, first = [], 0
    for n in numel:
        parts = []
        for a in range(0, n, 1 << 25):
            x = first + a + torch.arange(min(1 << 25, n - a), device="cuda", dtype=torch.int64)
            hi, lo = x >> 16, x & 0xffff
            for r in range(6):
                hi, lo = lo, hi ^ ((((lo ^ k[r]) + 1) * mul & mask) >> 16)
            bits = torch.nn.functional.pad(test(hi << 16 | lo).to(torch.int64), (0, -x.numel() % 32))
            parts.append((bits.view(-1, 32) * place).sum(1).to(torch.int32))
        out.append(torch.cat(parts))
        first += n
    return out


def _outcome(ctx):
    """How the context's last reconciliation went: (window of top halves of keys, candidates in the probe, drawn below
    the window, the guess held)."""
    out = (ctypes.c_int64 * 5)()
    assert tf.load_library().tf_internal_reconcile_outcome(ctx.handle, out) == 0
    return (out[0], out[1]), out[2], out[3], bool(out[4])


@pytest.mark.parametrize("what", ["added", "removed", "all", "same seed", "little more", "too few below", "too many below", "few candidates"])
def test_reconcile_large_masks_against_the_general_passes(ctx, what):
    """tf_reconcile_mask guesses the threshold of a large mask, tf_reconcile_mask_static never does.  Masks
    whose candidates have to do with the keys: so much that the probe sees it (`same seed`, `little more`: every candidate has a key
    above the last threshold), and so little that only the count shows it and the mask has to be put back.  And one with so
    few candidates that the window would be too wide.  The guess is made, dropped by the probe and held or not as it should be."""
    seed = 0x1234_5678_9ABC_DEF1
    numel = [GUESS_FROM - 77_000_003, 5, 77_000_005, 64]
    N = sum(numel)
    g = torch.Generator(device="cuda")
    g.manual_seed(len(what))
    base = [_random_words(g, (n + 31) // 32, 0.3) for n in numel]
    for w, n in zip(base, numel):
        if n % 32:
            w[-1] &= (1 << n % 32) - 1
    ones = lambda words: sum(int(((w >> b) & 1).sum()) for w in words for b in range(32))
    nf = N // 2
    if what == "removed":
        nf = N // 10
    elif what == "few candidates":                                     # one bit in 16
        base = [w & _random_words(g, w.numel(), 0.2) for w in base]
        nf = N // 32
    elif what == "all":
        nf = N                                                         # every candidate is drawn
    elif what in ("same seed", "little more"):                         # 83 % and 25 % of those expected below the threshold are none
        tf.tf_reconcile_mask_static(ctx, numel, base, int((0.4 if what == "same seed" else 0.33) * N), seed)
        nf = N // 2 if what == "same seed" else int(0.43 * N)
    elif what != "added":                                              # 5 % of the candidates on one side are none
        limit = int((0.5 - 0.3) / 0.7 * (1 << 32))
        side = _key_words(numel, seed, (lambda k: k < limit) if what == "too few below" else (lambda k: k >= limit))
        some = [_random_words(g, (n + 31) // 32, 0.05) for n in numel]
        base = [w | (s & x) for w, s, x in zip(base, side, some)]
    got = [w.clone() for w in base]
    ref = [w.clone() for w in base]
    stats, stats_ref = (torch.full((3,), -1, dtype=torch.int64, device="cuda") for _ in range(2))
    for _ in range(2):                                                 # the second call finds what the first has left
        for a, b in zip(got, base):
            a.copy_(b)
        tf.tf_reconcile_mask(ctx, numel, got, nf, seed, stats=stats)
        tf.tf_reconcile_mask_static(ctx, numel, ref, nf, seed, stats=stats_ref)
        assert all(torch.equal(a, b) for a, b in zip(got, ref)) and ones(got) == nf
        assert torch.equal(stats, stats_ref)
        for a, b in zip(ref, base):
            a.copy_(b)
        (lo, hi), probe, drawn, held = _outcome(ctx)
        need = abs(nf - int(stats[0]))
        expected = 32768 * need / max((lo + hi) << 15, 1)
        probe_fits = abs(probe - expected) <= 6 * expected ** 0.5 + 8
        if what == "few candidates":
            assert hi == 0 and not held
            continue
        assert 0 < lo < hi <= lo + 64
        assert probe_fits == (what not in ("same seed", "little more")) and held == (what in ("added", "removed", "all"))
        if held:
            assert drawn < need and lo <= int(stats[2]) >> 16 < hi
        elif not probe_fits:
            assert drawn == 0
        else:                                                          # 5 % of them in the way: far outside the window
            assert drawn < 0.98 * need if what == "too few below" else drawn > 1.02 * need


def test_reconcile_of_a_large_mask_in_a_graph():
    """A captured call makes no guess (a graph would keep the address of a copy) and allocates nothing; replays between
    eager calls, which do guess."""
    c = tf.Context(0)
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(11)
        numel = [GUESS_FROM, 1000]
        base = [_random_words(g, (n + 31) // 32, 0.3) for n in numel]
        base[1][-1] &= (1 << 1000 % 32) - 1
        words, ref = [w.clone() for w in base], [w.clone() for w in base]
        nf = sum(numel) // 2
        tf.tf_reconcile_mask_static(c, numel, ref, nf, 5)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            tf.tf_reconcile_mask(c, numel, words, nf, 5)
        assert torch.cuda.mem_get_info()[0] >= free - (32 << 20)       # (the smallest copy is 71 MB)
        for replay in range(3):
            for w, b in zip(words, base):
                w.copy_(b)
            graph.replay()
            assert _outcome(c)[0] == (0, 0) and not _outcome(c)[3]
            assert all(torch.equal(w, r) for w, r in zip(words, ref)), f"replay {replay}"
            eager = [w.clone() for w in base]
            tf.tf_reconcile_mask(c, numel, eager, nf, 5)
            assert _outcome(c)[3] and all(torch.equal(w, r) for w, r in zip(eager, ref))
        del graph
    finally:
        c.close()


def test_reconcile_large_mask_of_many_tensors(ctx):
    """140 tensors: three launches per pass, the keys of a window spread over them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    numel = [GUESS_FROM // 140 + 1 + 17 * i for i in range(140)]
    base = [_random_words(g, (n + 31) // 32, 0.4) for n in numel]
    got, ref = [w.clone() for w in base], [w.clone() for w in base]
    tf.tf_reconcile_mask(ctx, numel, got, sum(numel) // 4, 99)
    tf.tf_reconcile_mask_static(ctx, numel, ref, sum(numel) // 4, 99)
    assert all(torch.equal(a, b) for a, b in zip(got, ref)) and _outcome(ctx)[3]


def test_reconcile_never_waits_for_the_device():
    """The first large mask of a context, and a larger one after it, while another stream is busy: the call
    is back long before that stream is."""
    c = tf.Context(0)
    try:
        torch.cuda._sleep(1000)
        cycles, ms = 1 << 20, 0.0
        while ms < 300:                                                # how many cycles are 0.3 s
            cycles *= 2
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            torch.cuda._sleep(cycles)
            b.record()
            b.synchronize()
            ms = a.elapsed_time(b)
        busy, own = torch.cuda.Stream(), torch.cuda.Stream()
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        for n in (GUESS_FROM, 2 * GUESS_FROM + 1, 5 * GUESS_FROM):
            words = [_random_words(g, (n + 31) // 32, 0.3)]
            if n % 32:
                words[0][-1] &= (1 << n % 32) - 1
            ref = [w.clone() for w in words]
            tf.tf_reconcile_mask_static(c, [n], ref, n // 2, 17)
            torch.cuda.synchronize()
            done = torch.cuda.Event()
            with torch.cuda.stream(busy):
                torch.cuda._sleep(cycles)
                done.record()
            tf.tf_reconcile_mask(c, [n], words, n // 2, 17, stream=own)
            assert not done.query(), f"{n} elements: the call waited"
            torch.cuda.synchronize()
            assert torch.equal(words[0], ref[0]) and _outcome(c)[3]
    finally:
        c.close()
