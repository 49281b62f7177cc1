"""GPU parity of the nearest-codeword search on the shapes that select each screen variant.

Long top-1 searches (at least 2048 codewords and 5e8 pairs of a row and a codeword) run on 32 x 32 tiles under a power-of-two codebook scale: one fp16 MFMA per tile, exact for
bf16 operands, and for fp32 operands a second, split-fp16 screen of the rows the first leaves
uncertain (the split form at once below 3e9 pairs); shorter ones on 16 x 16 tiles with split-bf16 operands.  Whatever the variant, the certified screen plus the
exact rescue must return the oracle's codes (the fp64 definition of Eq. 3, ties to the lower index)
and its distances, including rows the scaled screen cannot represent (forced to the exact rescue),
codebooks of extreme magnitude and ragged tails."""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_09282_amd import crvq as C
from paper_2412_09282_amd import inputs
from paper_2412_09282_amd.crvq import VecSet

from gpu_util import dev, say, search_plan

pytestmark = pytest.mark.gpu


def rv(n, d, seed, scale=0.02):
    return inputs.random_vectors(n, d, seed, scale)


def assign_both(V, Cb, dtype="f32"):
    Vt = dev(V, dtype)
    Ct = dev(Cb, dtype)
    n = V.shape[0]
    codes = torch.empty(n, dtype=torch.int32, device="cuda")
    dist = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign(VecSet.of_vectors(Vt), Ct, codes, dist)
    torch.cuda.synchronize()
    exp, ed = oracle.assign(V, Cb, dtype, dtype)
    return codes.cpu().numpy(), dist.cpu().numpy(), exp, ed


def check(V, Cb, dtype="f32"):
    got, gd, exp, ed = assign_both(V, Cb, dtype)
    bad = np.flatnonzero(got != exp)
    assert len(bad) == 0, f"{len(bad)} codes differ, e.g. rows {bad[:5]} got {got[bad[:5]]} want {exp[bad[:5]]}"
    np.testing.assert_array_equal(gd, ed.astype(np.float32))


def check_pruned(V, Cb, dtype="f32"):
    """A call whose plan prunes: the codes and distances of every row against those of the same rows in pieces whose
    plan does not, and of a sample of the rows against the oracle."""
    n, d = V.shape
    K, piece = Cb.shape[0], 131072
    assert search_plan(n, d, K).prune == 1, f"n={n} K={K} does not prune"
    assert search_plan(piece, d, K).prune == 0
    Vt, Ct = dev(V, dtype), dev(Cb, dtype)
    codes, ref = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    dist, refd = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(2))
    C.crvq_assign(VecSet.of_vectors(Vt), Ct, codes, dist)
    for a in range(0, n, piece):
        b = min(n, a + piece)
        C.crvq_assign(VecSet.of_vectors(Vt[a:b]), Ct, ref[a:b], refd[a:b])
    torch.cuda.synchronize()
    assert torch.equal(codes, ref), f"{int((codes != ref).sum())} codes differ from the unpruned search"
    assert torch.equal(dist, refd)
    S = np.random.default_rng(1).choice(n, 40000, replace=False)
    exp, ed = oracle.assign(V[S], Cb, dtype, dtype)
    np.testing.assert_array_equal(codes.cpu().numpy()[S], exp)
    np.testing.assert_array_equal(dist.cpu().numpy()[S], ed.astype(np.float32))


@pytest.mark.parametrize("n,K,d", [(65536, 65536, 8), (65536 + 37, 65536 - 5, 8), (70001, 32768 + 17, 5)])
def test_long_search_f32(n, K, d):
    say(f"long top-1 search fp32 n={n} K={K} d={d}")
    check(rv(n, d, 31 + d), rv(K, d, 32 + K))


def test_long_search_bf16():
    say("long top-1 search bf16 n=65536 K=65536")
    V = inputs.f32_to_bf16_bits(rv(65536, 8, 33))
    Cb = inputs.f32_to_bf16_bits(rv(65536, 8, 34))
    check(V, Cb, "bf16")


@pytest.mark.parametrize("case", ["ties", "outliers", "tiny", "huge"])
def test_long_search_bf16_exact_operands(case):
    """bf16 rows against a bf16 codebook take the one-MFMA screen (exact fp16 operands)."""
    say(f"long top-1 search bf16, exact-operand screen: {case}")
    g = np.random.default_rng(44)
    if case == "ties":
        base = rv(16384, 8, 45)
        Cb = np.ascontiguousarray(np.concatenate([base, base, base[::-1], base])[g.permutation(65536)])
        V = np.concatenate([base[g.integers(0, 16384, 40000)], rv(25536 + 11, 8, 46)])
    elif case == "outliers":
        Cb = (g.standard_t(4.0, size=(65536 - 3, 8)) * 0.02).astype(np.float32)
        Cb[:, 5] *= np.float32(10.0)
        V = (g.standard_t(4.0, size=(65536 + 29, 8)) * 0.02).astype(np.float32)
        big = g.choice(len(V), 300, replace=False)
        V[big, g.integers(0, 8, 300)] *= np.float32(1e5)   # beyond the scaled fp16 range
        tiny = g.choice(len(V), 300, replace=False)
        V[tiny] *= np.float32(1e-9)                        # below the fp16 normal range once scaled
    else:
        s = np.float32(1e-30 if case == "tiny" else 1e30)
        V, Cb = rv(65536, 8, 47) * s, rv(65536, 8, 48) * s
    check(inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb), "bf16")


def test_long_search_outlier_rows_and_heavy_tails():
    say("long top-1 search: t4 codebook with outlier columns, rows far outside the codebook range")
    g = np.random.default_rng(35)
    K, n = 65536, 65536
    Cb = (g.standard_t(4.0, size=(K, 8)) * 0.02).astype(np.float32)
    Cb[:, 3] *= np.float32(10.0)
    V = (g.standard_t(4.0, size=(n, 8)) * 0.02).astype(np.float32)
    big = g.choice(n, 300, replace=False)
    V[big, g.integers(0, 8, 300)] *= np.float32(1e5)   # beyond the scaled fp16 range: exact rescue
    tiny = g.choice(n, 300, replace=False)
    V[tiny] *= np.float32(1e-6)                       # far below the codebook scale
    check(V, Cb)


@pytest.mark.parametrize("scale", [1e-30, 1e30])
def test_long_search_extreme_magnitude(scale):
    say(f"long top-1 search at magnitude {scale:g}")
    s = np.float32(scale)
    check(rv(65536, 8, 36) * s, rv(65536, 8, 37) * s)


def test_long_search_duplicates_and_ties():
    say("long top-1 search with duplicated codewords and rows equal to codewords")
    g = np.random.default_rng(38)
    base = rv(16384, 8, 39)
    Cb = np.ascontiguousarray(np.concatenate([base, base, base[::-1], base])[g.permutation(65536)])
    V = np.concatenate([base[g.integers(0, 16384, 40000)], rv(25536, 8, 40)])
    check(V, Cb)


def test_beam_width_one_long_codebook():
    say("residual beam, width 1, over a K=65536 basic and K=256 extended codebook")
    n = 65536
    V = rv(n, 8, 41)
    books = [rv(65536, 8, 42), rv(256, 8, 43, 0.005)]
    Vt = dev(V)
    bt = [dev(b) for b in books]
    codes = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in books]
    err = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign_residual_beam(VecSet.of_vectors(Vt), bt, 1, codes, err)
    torch.cuda.synchronize()
    exp_codes, exp_err = oracle.beam(V, books, 1)
    for t in range(2):
        got = codes[t].cpu().numpy()
        bad = np.flatnonzero(got != exp_codes[t])
        assert len(bad) == 0, f"book {t}: {len(bad)} codes differ, e.g. rows {bad[:5]}"
    np.testing.assert_array_equal(err.cpu().numpy(), np.asarray(exp_err, dtype=np.float64).astype(np.float32))


@pytest.mark.parametrize("n", [65536 + 37, (1 << 20) + 37])
def test_beam_width_one_long_extended_book(n):
    """Width 1 over a K=4096 basic and a K=65536 extended book: the extended step searches the fp64
    residuals on the 32 x 32 fp16 screens (unpruned with codebook splits at 65,573 rows, pruned in key
    order at 1,048,613), whose operands are the residuals rounded to fp32; the certificate adds that
    rounding to each row's own fp16 remainder."""
    say(f"residual beam, width 1, K=4096 basic + K=65536 extended over fp64 residuals, n={n}")
    assert search_plan(n, 8, 65536).prune == (1 if n > 1000000 else 0)
    V = rv(n, 8, 81)
    books = [rv(4096, 8, 82), rv(65536, 8, 83, 0.006)]
    codes = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in books]
    err = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign_residual_beam(VecSet.of_vectors(dev(V)), [dev(b) for b in books], 1, codes, err)
    torch.cuda.synchronize()
    exp_codes, exp_err = oracle.beam(V, books, 1)
    for t in range(2):
        got = codes[t].cpu().numpy()
        bad = np.flatnonzero(got != exp_codes[t])
        assert len(bad) == 0, f"book {t}: {len(bad)} codes differ, e.g. rows {bad[:5]}"
    np.testing.assert_array_equal(err.cpu().numpy(), np.asarray(exp_err, dtype=np.float64).astype(np.float32))


# Long searches on fp32 operands (here 262144 rows x 65536 codewords, four codebook splits) get two
# screens: one MFMA per tile on fp16-rounded operands with the wider certificate, then the split form
# on the rows it left uncertain, then the exact rescue of what is left.
@pytest.mark.parametrize("case", ["plain", "ties", "mixed_bf16_book"])
def test_two_pass_screen(case):
    n, K, d = 262144 + 37, 65536, 8
    say(f"two-pass screen fp32 n={n} K={K} ({case})")
    g = np.random.default_rng(44)
    if case == "ties":
        base = rv(16384, 8, 45)
        Cb = np.ascontiguousarray(np.concatenate([base, base, base[::-1], base])[g.permutation(K)])
        V = np.concatenate([base[g.integers(0, 16384, n // 2)], rv(n - n // 2, 8, 46)])
        check(V, Cb)
    elif case == "mixed_bf16_book":
        V = rv(n, d, 47)
        Cb = inputs.f32_to_bf16_bits(rv(K, d, 48))
        Vt, Ct = dev(V), dev(Cb, "bf16")
        codes = torch.empty(n, dtype=torch.int32, device="cuda")
        dist = torch.empty(n, dtype=torch.float32, device="cuda")
        C.crvq_assign(VecSet.of_vectors(Vt), Ct, codes, dist)
        torch.cuda.synchronize()
        exp, ed = oracle.assign(V, Cb, "f32", "bf16")
        np.testing.assert_array_equal(codes.cpu().numpy(), exp)
        np.testing.assert_array_equal(dist.cpu().numpy(), ed.astype(np.float32))
    else:
        # codewords drawn near the rows, as K-means leaves them: many near-ties for the first screen
        V = rv(n, d, 49)
        Cb = np.ascontiguousarray(V[g.choice(n, K, replace=False)] + rv(K, d, 50, 0.002))
        check(V, Cb)


# The first screen on fp16-rounded operands certifies each row with its own fp16 remainder: with
# a = alpha c and y = -2 alpha x = y1 + y2 the dropped terms are sum_t a_t y2_t + sum_t a2_t y1_t, bounded
# by R (||y2|| + 2^-11 (1 + 2^-11) ||y||) / alpha.  Here every row sits just below the midpoint between
# two fp16 values after the power-of-two scale (each y2_t positive and 2^-13 short of half a spacing,
# the largest it can be), and the codewords share the rows' signs, so sum_t a_t y2_t is close to its
# Cauchy-Schwarz bound; the codewords come in near-tied pairs, so many rows stay uncertain.  Codes
# and distances must remain the oracle's (unpruned in one and in four codebook splits; pruned: one split, key
# order).
@pytest.mark.parametrize("n,K,splits,prune", [(262144 + 37, 65536, 4, 0), ((1 << 20) + 37, 16384, 1, 0),
                                              (400037, 65536, 1, 1), (1600037, 16384, 1, 1)])
def test_first_screen_aligned_remainders(n, K, splits, prune):
    d = 8
    p = search_plan(n, d, K)
    assert (p.s32, p.splits, p.prune) == (1, splits, prune)
    say(f"first screen, remainders aligned with the codewords: n={n} K={K}")
    g = np.random.default_rng(71)
    # -2^12 x in [256, 512), where fp16 values are 0.25 apart: 256 + 0.25 j + (0.125 - 2^-13), exact in fp32
    j = g.integers(0, 1024, size=(n, d)).astype(np.float64)
    V = (-(256.0 + 0.25 * j + (0.125 - 2.0 ** -13)) / 4096.0).astype(np.float32)
    base = V[g.choice(n, K // 2, replace=False)]
    e1 = (g.random((K // 2, d)) * 2e-6).astype(np.float32)
    e2 = (g.random((K // 2, d)) * 2e-6).astype(np.float32)
    Cb = np.ascontiguousarray(np.concatenate([base - e1, base - e2])[g.permutation(K)])
    assert (Cb < 0).all() and (V < 0).all()
    (check_pruned if prune else check)(V, Cb)


@pytest.mark.parametrize("K", [4096, 16384])
def test_second_screen_own_rows_full(K):
    """From 2^23 rows up the second (split) screen of fp32 rows gives every wave rows of its own
    instead of sharing them across a workgroup.  Every row of a (2^23 + 37)-row search against codewords drawn
    next to the rows (so several percent of the rows reach the second screen) is compared with the oracle (4096
    codewords, unpruned) or with the unpruned search (16384, pruned)."""
    n, d = (1 << 23) + 37, 8
    say(f"two-pass screen fp32 n={n} K={K}: second screen with rows per wave, full comparison")
    g = np.random.default_rng(51)
    V = rv(n, d, 52)
    Cb = np.ascontiguousarray(V[g.choice(n, K, replace=False)] + rv(K, d, 53, 0.002))
    (check if K == 4096 else check_pruned)(V, Cb)


# From 2.5e10 pairs and 16384 codewords up the first screen visits the codebook in the order
# of a key (norm, then two coordinates, each binned over a robust range of the codebook) and skips
# pairs of tiles whose norms or coordinates are certified too far from every row of a wave; the
# results must stay the oracle's exactly.  "constant": both key coordinates constant over the codebook
# (no spread to bin); "outlier_cols": heavy tails with 10x outlier coordinates in 8 % of the vectors
# (the bins follow the bulk, the outliers fall into the end bins); "d1": one dimension (both key
# coordinates are the same one).
@pytest.mark.parametrize("case,n,K", [("near", (1 << 20) + 4133, 65536), ("bf16", 1600037, 16384),
                                      ("outliers", 1600037, 16384), ("ties", 400037, 65536), ("tiny", 400037, 65536),
                                      ("constant", 400037, 65536), ("outlier_cols", 1600037, 16384),
                                      ("d1", 400037, 65536)])
def test_pruned_first_screen(case, n, K):
    d = 1 if case == "d1" else 8
    say(f"pruned first screen n={n} K={K} ({case})")
    g = np.random.default_rng(60)
    if case in ("near", "bf16"):
        V = rv(n, d, 61)
        Cb = np.ascontiguousarray(V[g.choice(n, K, replace=False)] + rv(K, d, 62, 0.002))
        if case == "bf16":
            check_pruned(inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb), "bf16")
            return
    elif case == "outliers":
        Cb = (g.standard_t(4.0, size=(K, d)) * 0.02).astype(np.float32)
        Cb[:, 0] *= np.float32(10.0)                       # the coordinate of the second band
        V = (g.standard_t(4.0, size=(n, d)) * 0.02).astype(np.float32)
        big = g.choice(n, 500, replace=False)
        V[big, g.integers(0, d, 500)] *= np.float32(1e5)   # beyond the scaled fp16 range: rescued exactly
        tiny = g.choice(n, 500, replace=False)
        V[tiny] *= np.float32(1e-6)
    elif case == "ties":
        base = rv(K // 4, d, 63)
        Cb = np.ascontiguousarray(np.concatenate([base, base, base[::-1], base])[g.permutation(K)])
        V = np.concatenate([base[g.integers(0, K // 4, n // 2)], rv(n - n // 2, d, 64)])
    elif case == "constant":
        V = rv(n, d, 67)
        Cb = rv(K, d, 68)
        Cb[:, 0] = np.float32(0.01)
        Cb[:, 1] = np.float32(-0.02)
        V[: n // 2, 0] = np.float32(0.01)
    elif case == "outlier_cols":
        V = (g.standard_t(4.0, size=(n, d)) * 0.02).astype(np.float32)
        hit = g.random(n) < 0.08
        V[hit, g.integers(0, d, int(hit.sum()))] *= np.float32(10.0)
        Cb = np.ascontiguousarray(V[g.choice(n, K, replace=False)])
    elif case == "d1":
        V = rv(n, d, 69)
        Cb = rv(K, d, 70)
    else:  # magnitudes far below one: the bands are kept in units of the codebook scale
        V = rv(n, d, 65) * np.float32(1e-30)
        Cb = rv(K, d, 66) * np.float32(1e-30)
    check_pruned(V, Cb)


def hard_inputs(case, n, K, d, g):
    """Rows and codewords of one of: plain, outliers (rows past the scaled fp16 range, tiny rows), ties
    (codewords four times over), constant (no spread in the key coordinates), tiny magnitudes."""
    if case == "ties":
        base = rv((K + 3) // 4, d, 81)
        Cb = np.ascontiguousarray(np.concatenate([base] * 4)[g.permutation(4 * base.shape[0])[:K]])
        return np.concatenate([base[g.integers(0, base.shape[0], n // 2)], rv(n - n // 2, d, 82)]), Cb
    V, Cb = rv(n, d, 83), rv(K, d, 84)
    if case == "outliers":
        big = g.choice(n, 300, replace=False)
        V[big, g.integers(0, d, 300)] *= np.float32(1e6)
        V[g.choice(n, 300, replace=False)] *= np.float32(1e-6)
    elif case == "constant":
        Cb[:, :2] = np.float32(0.01)
    elif case == "tiny":
        V, Cb = V * np.float32(1e-30), Cb * np.float32(1e-30)
    return V, Cb


@pytest.mark.parametrize("case,n,K,d", [
    ("bf16", 400037, 65531, 8), ("outliers", 400037, 65531, 8), ("ties", 381600, 65536, 8), ("tiny", 400037, 65531, 8),
    ("constant", 400037, 65531, 8), ("plain", 400037, 65531, 1)])
def test_pruned_long_books(case, n, K, d):
    """The pruned screen just above the pairs it starts at."""
    say(f"pruned screen n={n} K={K} d={d} ({case})")
    assert search_plan(n, d, K).prune == 1
    V, Cb = hard_inputs(case, n, K, d, np.random.default_rng(80))
    if case == "bf16":
        check(inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb), "bf16")
    else:
        check(V, Cb)


@pytest.mark.parametrize("case,n,K,d", [
    ("plain", 250007, 2053, 8), ("bf16", 262111, 2048, 8), ("outliers", 122077, 4096, 8), ("ties", 131071, 4100, 5),
    ("tiny", 200003, 3001, 8), ("plain", 9001, 65536, 8), ("bf16", 8011, 65535, 3),  # 28 and more splits
    ("constant", 183251, 16384, 8), ("ties", 190003, 16400, 8),  # the last of the split form, the first of two screens
    ("plain", 243001, 2048, 8), ("plain", 600011, 2047, 8)])  # below the fewest pairs, the fewest codewords
def test_split_form_at_once(case, n, K, d):
    """Middle lengths: 32 x 32 tiles in the split form for every row, around the lines of the dispatch."""
    say(f"split form at once n={n} K={K} d={d} ({case})")
    p = search_plan(n, d, K)
    assert (p.s32, p.prune) == (0 if (n, K) in ((243001, 2048), (600011, 2047)) else 1, 0)
    V, Cb = hard_inputs(case, n, K, d, np.random.default_rng(85))
    if case == "bf16":
        check(inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb), "bf16")
    else:
        check(V, Cb)


def test_beam_width_one_split_form():
    """A width-1 beam's fp64 residual rows through the split form at once (second book), fp32 rows first."""
    n, d = 130003, 8
    say("width-1 beam, two books of 4096 over 130003 rows")
    V, books = rv(n, d, 86), [rv(4096, d, 87), rv(4096, d, 88, 0.01)]
    codes = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in books]
    err = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign_residual_beam(VecSet.of_vectors(dev(V)), [dev(b) for b in books], 1, codes, err)
    torch.cuda.synchronize()
    exp_codes, exp_err = oracle.beam(V, books, 1)
    np.testing.assert_array_equal(np.stack([c.cpu().numpy() for c in codes]), exp_codes)
    np.testing.assert_array_equal(err.cpu().numpy(), exp_err.astype(np.float32))


def test_rescue_of_most_rows():
    """Rows equal to codewords that the book holds four times (exact ties on every row, so nearly every
    row reaches the exact rescue) over 1,048,579 rows: more listed rows than the parted rescue has
    room for, so the rescue scans the whole codebook per row batch; sampled rows against the oracle."""
    say("long top-1 search, 1048579 rows that all tie: whole-codebook rescue")
    g = np.random.default_rng(44)
    base = rv(16384, 8, 45)
    Cb = np.ascontiguousarray(np.concatenate([base, base, base, base])[g.permutation(65536)])
    n = 1048579
    assert search_plan(n, 8, 65536).prune == 1
    V = np.ascontiguousarray(base[g.integers(0, 16384, n)])
    codes = torch.empty(n, dtype=torch.int32, device="cuda")
    dist = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign(VecSet.of_vectors(dev(V)), dev(Cb), codes, dist)
    torch.cuda.synchronize()
    S = np.sort(g.choice(n, 3000, replace=False))
    S[-1] = n - 1
    exp, ed = oracle.assign(V[S], Cb)
    np.testing.assert_array_equal(codes.cpu().numpy()[S], exp)
    np.testing.assert_array_equal(dist.cpu().numpy()[S], ed.astype(np.float32))


# Small codebooks (K <= 256) at row counts that take the wide top-1 kernel (128 rows per wave): fp32 and
# bf16 rows packed at a 16-byte aligned base take its fast forms, any other layout the generic form;
# codes and distances must equal the oracle's, including exact ties (duplicated codewords, rescued)
# and a last tile of padding codewords (K = 37).
@pytest.mark.parametrize("case", ["f32", "f32_k37", "bf16", "unaligned", "ties"])
def test_small_book_wide_forms(case):
    n, d = 600_001, 8
    say(f"small-book top-1, wide form: {case}, n={n}")
    K = 37 if case == "f32_k37" else 256
    V = rv(n, d, 71)
    Cb = rv(K, d, 72)
    if case == "ties":
        Cb[128:] = Cb[:128]
        V[: n // 3] = Cb[np.random.default_rng(73).integers(0, 128, n // 3)]
    if case == "bf16":
        check(inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb), "bf16")
        return
    if case == "unaligned":
        buf = torch.empty(n * d + 1, dtype=torch.float32, device="cuda")
        buf[1:] = torch.from_numpy(V.reshape(-1)).cuda()
        Vt = buf[1:].view(n, d)  # base 4 bytes past a 16-byte boundary
        codes = torch.empty(n, dtype=torch.int32, device="cuda")
        dist = torch.empty(n, dtype=torch.float32, device="cuda")
        C.crvq_assign(VecSet.of_vectors(Vt), dev(Cb), codes, dist)
        torch.cuda.synchronize()
        exp, ed = oracle.assign(V, Cb)
        np.testing.assert_array_equal(codes.cpu().numpy(), exp)
        np.testing.assert_array_equal(dist.cpu().numpy(), ed.astype(np.float32))
        return
    check(V, Cb)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [1, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n,K", [(1000, 60), (3000, 1100), (250013, 2050)])
def test_row_lengths_at_any_element(n, K, d, dtype):
    """Rows and codewords of every length up to 8 whose memory starts at an odd element, the last row at the end
    of its allocation: whole and overlapping vector loads, element loads."""
    say(f"row lengths n={n} K={K} d={d} {dtype}")
    V, Cb = rv(n, d, 110 + d), rv(K, d, 120 + d)
    if dtype == "bf16":
        V, Cb = inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(Cb)
    held = []
    for a in (V, Cb):
        flat = torch.empty(a.size + 1, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        held.append(flat[1:].view(*a.shape))
        held[-1].copy_(dev(a, dtype))
    codes = torch.empty(n, dtype=torch.int32, device="cuda")
    dist = torch.empty(n, dtype=torch.float32, device="cuda")
    C.crvq_assign(VecSet.of_vectors(held[0]), held[1], codes, dist)
    torch.cuda.synchronize()
    exp, ed = oracle.assign(V, Cb, dtype, dtype)
    np.testing.assert_array_equal(codes.cpu().numpy(), exp)
    np.testing.assert_array_equal(dist.cpu().numpy(), ed.astype(np.float32))


def test_short_rows_time():
    """Rows of 7 in the 32 x 32 screen, whose winners' 64 codewords are read again exactly: no slower than rows of 8
    by much (3072 codewords x 1 M rows: measured 1.05 times; 1.6 times with element loads)."""
    n, K = 1000000, 3072

    def us(d):
        vs, Ct = VecSet.of_vectors(dev(rv(n, d, 130))), dev(rv(K, d, 131))
        codes = torch.empty(n, dtype=torch.int32, device="cuda")
        C.crvq_assign(vs, Ct, codes)
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                C.crvq_assign(vs, Ct, codes)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / 5)
        return min(times)

    t7, t8 = us(7), us(8)
    say(f"short rows: d=7 {t7:.1f} us, d=8 {t8:.1f} us")
    assert t7 <= 1.3 * t8


def repeated_book(K, d, share, seed):
    """K codewords of which the given share are copies of others, copies and originals in any order."""
    u = int(K * (1 - share))
    B = rv(u, d, seed)
    B[u // 2] = 0.0  # zeros of either sign are equal
    order = np.random.default_rng(seed + 1).permutation(K)
    full = np.concatenate([B, B[np.arange(K - u) % u]])
    full[-1] = -0.0
    return full[order]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,K,d,share", [(250000, 2048, 8, 0.5), (200003, 4000, 5, 0.75), (61440, 8192, 8, 0.5),
                                         (800000, 4096, 7, 0.3), (20000, 32771, 8, 0.9), (131072, 16384, 1, 0.5)])
def test_repeated_codewords_unpruned(n, K, d, share, dtype):
    """The codes are the lowest copies, whatever the scratch held before (it is full of entries for random codewords at
    first, then of what the first call left)."""
    p = search_plan(n, d, K)
    assert p.s32 and not p.prune
    V, B = rv(n, d, 140), repeated_book(K, d, share, 141)
    V[:50] = B[np.arange(50) * (K // 50)]
    if dtype == "bf16":
        V, B = inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(B)
    Vt, Bt = dev(V, dtype), dev(B, dtype)
    vs = VecSet.of_vectors(Vt)
    Bh = oracle.widen(B, dtype)
    _, back = np.unique(Bh + 0.0, axis=0, return_inverse=True)
    first = np.full(back.max() + 1, K)
    np.minimum.at(first, back, np.arange(K))
    say(f"repeated codewords: n={n} K={K} d={d} {dtype}")
    codes = torch.empty(n, dtype=torch.int32, device="cuda")
    dist = torch.empty(n, device="cuda")
    need = C.lib().crvq_assign_workspace_size(n, d, K)
    ws = ~torch.randint(0, K, (need // 4 + 1,), dtype=torch.int32, device="cuda")
    seen = []
    for _ in range(2):
        assert C.lib().crvq_assign(*vs.args(), C._ptr(Bt), C.dtype_code(Bt), K, C._ptr(codes), C._ptr(dist), C._ptr(ws),
                                   ws.numel() * 4, C._stream(None)) == 0
        got = codes.cpu().numpy()
        np.testing.assert_array_equal(got, first[back[got]])
        seen.append((got, dist.cpu().numpy()))
    np.testing.assert_array_equal(seen[0][0], seen[1][0])
    np.testing.assert_array_equal(seen[0][1], seen[1][1])
    m = min(n, 2000)
    exp, ed = oracle.assign(V[:m], B, dtype, dtype)
    np.testing.assert_array_equal(seen[0][0][:m], exp)
    np.testing.assert_array_equal(seen[0][1][:m], ed.astype(np.float32))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_repeated_codewords_pruned(dtype):
    """The pruned form takes the copies out of its key-ordered book as well."""
    V, B = rv(1600000, 8, 145), repeated_book(16384, 8, 0.5, 146)
    V[:100] = B[np.arange(100) * 160]
    say(f"repeated codewords, pruned, {dtype}")
    if dtype == "bf16":
        V, B = inputs.f32_to_bf16_bits(V), inputs.f32_to_bf16_bits(B)
    check_pruned(V, B, dtype)


def test_repeated_codewords_time():
    """Half of a book's codewords being copies costs the search little (2048 codewords x 262,144 rows: measured
    1.06 times; 11 times with the copies in the screen)."""
    n, K = 262144, 2048
    vs = VecSet.of_vectors(dev(rv(n, 8, 150)))
    codes = torch.empty(n, dtype=torch.int32, device="cuda")

    def us(B):
        Bt = dev(B)
        C.crvq_assign(vs, Bt, codes)
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                C.crvq_assign(vs, Bt, codes)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / 5)
        return min(times)

    plain, copies = us(rv(K, 8, 151)), us(repeated_book(K, 8, 0.5, 152))
    say(f"repeated codewords: {copies:.1f} us, without {plain:.1f} us")
    assert copies <= 1.6 * plain
