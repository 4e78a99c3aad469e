"""The 64 x 64 / 128 x 128-tile product kernel (fp32 through bf16 pieces, ragged and unaligned bf16) against fp64.

Tolerance, per symbol: every product is formed to 2^-24 of itself (fp32: the terms that are left out add up to less
than 2^-24 of it, a piece is the nearest bf16 to what it stands for; bf16: products are exact) and k of them are
added in fp32, so |C - C64| <= (k + 4) 2^-24 (|A| |B|)."""
import numpy as np
import pytest

from paper_2508_04355_amd import gecc, inputs

pytestmark = pytest.mark.gpu


def _product(A, B, dtype, trans=(0, 0), pad=0, shift=0):
    """plain product of (batch, n, k) and (batch, k, m); `pad`: extra elements per stored row, `shift`: elements
    the operands start behind a 16-byte boundary."""
    import torch
    import gpu_harness as H
    batch, n, k = A.shape
    m = B.shape[2]
    lda, ldb, ldc = (n if trans[0] else k) + pad, (k if trans[1] else m) + pad, m + pad

    def put(x, tr, ld):
        t = H.to_dev(x, dtype, tr, ld)
        flat = torch.zeros(t.numel() + 8, dtype=t.dtype, device=t.device)
        flat[shift:shift + t.numel()] = t.reshape(-1)
        return flat[shift:shift + t.numel()]

    dA, dB = put(A, trans[0], lda), put(B, trans[1], ldb)
    ctx = gecc.Context(n, k, m, gecc.BF16 if dtype == "bf16" else gecc.F32, gecc.noise_thresholds(n, k, m, 1.0, 1.0),
                       batch=batch, trans_a=trans[0], trans_b=trans[1], lda=lda, ldb=ldb, ldc=ldc)
    C = ctx.alloc_c()
    C.fill_(float("nan"))
    ctx.plain_gemm(dA, dB, C)
    torch.cuda.synchronize()
    out = C.cpu().numpy().astype(np.float64)
    assert np.isnan(out[:, :, m:]).all()                 # what lies between m and ldc is left alone
    return out[:, :, :m]


def _check(C, A, B):
    A, B = A.astype(np.float64), B.astype(np.float64)
    assert not np.isnan(C).any()
    ref, mag = A @ B, np.abs(A) @ np.abs(B)
    assert (np.abs(C - ref) <= (A.shape[2] + 4) * 2.0 ** -24 * mag).all(), np.max(np.abs(C - ref) / (mag + 1e-300))


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,batch", [((1, 1, 1), 1), ((2, 33, 1), 2), ((1, 65, 3), 1), ((63, 31, 65), 1), ((64, 64, 64), 3),
                                         ((65, 129, 63), 1), ((127, 300, 129), 1),
                                         ((250, 257, 250), 64),      # 128 x 128 tiles, fp32: k split in two
                                         ((500, 321, 381), 48)])     # 128 x 128 tiles, one workgroup each
def test_tiles_layouts_and_tails(shape, batch, dtype, trans):
    n, k, m = shape
    rng = inputs.rng_for(80, n + k)
    law = ("normal", 1.0)
    A, B = [np.stack(x) for x in zip(*[inputs.operands(rng, n, k, m, law, law, dtype) for _ in range(batch)])]
    _check(_product(A, B, dtype, trans), A, B)
    _check(_product(A, B, dtype, trans, pad=3, shift=1), A, B)       # rows that start at any element


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,m", [(1, 66), (65, 2), (3, 1), (70, 131)])
def test_ends_of_the_k_range(n, m, dtype, trans):
    """The last k-tile is loaded from the end of the range, whatever lies before it: ranges shorter than a vector or a thread's
    share of k (below 16), one more and one less than a share, a k-tile and two of them."""
    law = ("normal", 1.0)
    for k in (2, 7, 8, 15, 16, 17, 31, 32, 34, 47, 63, 66, 95, 127, 128, 130, 193):
        A, B = [x[None] for x in inputs.operands(inputs.rng_for(83, k), n, k, m, law, law, dtype)]
        _check(_product(A, B, dtype, trans, pad=k % 3, shift=k % 2), A, B)


# Batches that go in tiles of 128 x 256 (test_launch_plans.py holds them to it): every remainder of the k loop (three k-tiles of
# 32 in flight), few rows, a second half with a single column, more tile columns than one, of which the last has no second half
WIDE_CASES = [((128, 256, 256), 250), ((120, 257, 250), 250), ((127, 287, 1541), 73), ((128, 288, 193), 250), ((65, 319, 200), 250),
              ((121, 320, 385), 125)]
# ... and in tiles of 64 x 64, for the same values and faults
SMALL_CASES = [((128, 128, 256), 250), ((127, 129, 249), 250), ((100, 160, 200), 250), ((1, 191, 129), 250)]


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape,batch", WIDE_CASES + SMALL_CASES)
def test_fp32_tiles_of_128_by_256(shape, batch, trans):
    """Rounds of such tiles, and products too short for them: every remainder of the k loop, rows and columns past the end,
    operands the pieces cannot hold, faults in either half of a tile."""
    import torch
    import gpu_harness as H
    n, k, m = shape
    rng = inputs.rng_for(81, n + k)
    A, B = rng.standard_normal((batch, n, k)).astype(np.float32), rng.standard_normal((batch, k, m)).astype(np.float32)
    A[7, :, 3] *= np.float32(2.0 ** -120)
    B[7, 3, :] *= np.float32(2.0 ** 120)
    _check(_product(A, B, "f32", trans), A, B)
    _check(_product(A, B, "f32", trans, pad=3, shift=1), A, B)
    A[7, :, 3] *= np.float32(2.0 ** 120)
    B[7, 3, :] *= np.float32(2.0 ** -120)
    ctx = gecc.Context(n, k, m, gecc.F32, gecc.noise_thresholds(n, k, m, 1.0, 1.0), batch=batch, trans_a=trans[0], trans_b=trans[1])
    dA, dB, C = H.to_dev(A, "f32", trans[0]), H.to_dev(B, "f32", trans[1]), ctx.alloc_c()
    A_par, B_par, C_par = ctx.alloc_parities()
    rep = ctx.alloc_report()
    planted = {5: (n - 1, m - 1, 40.0), 11: (0, min(m - 1, 130), -25.0), batch - 1: (n // 2, 3, 60.0)}
    ctx.encode_a(dA, A_par)
    ctx.encode_b(dB, B_par)
    ctx.multiply(dA, A_par, dB, B_par, C, C_par, *gecc.make_faults([(b,) + f for b, f in planted.items()]))
    ctx.verify(C, C_par, rep, fused=True)
    ctx.correct(dA, A_par, dB, B_par, C, C_par, rep)
    torch.cuda.synchronize()
    _check(C.cpu().numpy().astype(np.float64).reshape(batch, n, m), A, B)
    for b, r in enumerate(ctx.report_to_host(rep)):
        assert r.status == (gecc.CORRECTED if b in planted else gecc.CLEAN), (b, r.status)
        if b in planted:
            assert [e[:3] for e in r.errors()] == [(2,) + planted[b][:2]]


HALVES_SHAPES = [(128, 256, 256), (120, 289, 250)]
HALVES_OTHER_BATCH = 300      # too many for one round of 128 x 256 tiles: the same products in 128 x 128 ones


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", HALVES_SHAPES)
def test_halves_of_an_fp32_tile_are_as_in_tiles_of_their_own(shape, trans):
    """Which columns go through native fp32 (values the pieces cannot hold) does not depend on the tile: 128 x 256 and
    128 x 128 tiles give the same bits."""
    n, k, m = shape
    rng = inputs.rng_for(82, n + k)
    A = rng.standard_normal((HALVES_OTHER_BATCH, n, k)).astype(np.float32)
    B = rng.standard_normal((HALVES_OTHER_BATCH, k, m)).astype(np.float32)
    tiny = np.float32(2.0 ** -120)
    B[3, 5, 200] = tiny                 # the second half
    B[4, k - 1, 17] = -tiny             # the first
    B[5, 0, 127] = B[5, 1, 128] = tiny  # both
    A[6, n - 1, 4] = tiny               # a row of A: both
    B[7, 9, m - 1] = np.float32(np.inf)
    A[8, 3, 7] = np.float32(3.4e38)     # rounds to an infinite bf16
    B[8, 7, 100] = np.float32(2.0)
    B[9, 8, 40] = np.float32(np.nan)
    wide, other = _product(A[:256], B[:256], "f32", trans), _product(A, B, "f32", trans)
    for b in range(256):
        assert np.array_equal(wide[b], other[b], equal_nan=True), (b, np.argwhere(wide[b] != other[b])[:4])
    assert np.isnan(wide[9, :, 40]).all() and np.isinf(wide[7, :, m - 1]).all() and np.isfinite(wide[3:7]).all()


def test_values_the_bf16_pieces_cannot_hold():
    """Infinities, NaN, magnitudes beyond the largest bf16 and values below 2^-110 go through native fp32
    arithmetic: the same result as a chain of fp32 multiplications and additions would have."""
    n, k, m = 200, 96, 150
    rng = inputs.rng_for(81, 0)
    A, B = inputs.operands(rng, n, k, m, ("normal", 1.0), ("normal", 1.0), "f32")
    B[7, 3], B[7, 4], B[:, 5] = 1.0, 0.0, 1.0        # (exact in bf16; zero; exact in bf16)
    X = A.copy()
    X[10, 7] = np.inf
    X[150, 2] = np.nan
    X[60, 9] = np.float32(3.4e38)                    # finite, but rounds to an infinite bf16
    Y = B.copy()
    Y[9, :] *= np.float32(0.25)
    C = _product(X[None], Y[None], "f32")[0]
    with np.errstate(all="ignore"):
        ref = X.astype(np.float64) @ Y.astype(np.float64)
    assert np.isnan(C[150]).all() and np.isnan(C[10, 4])
    cols = [j for j in range(m) if Y[7, j] != 0.0]
    assert np.array_equal(C[10, cols], np.sign(Y[7, cols]) * np.inf)
    rows = [i for i in range(n) if i not in (10, 150)]
    mag = np.abs(X[rows].astype(np.float64)) @ np.abs(Y.astype(np.float64))
    fine = mag < 3.3e38
    assert np.isfinite(C[rows][fine]).all()
    assert (np.abs(C[rows] - ref[rows])[fine] <= (k + 4) * 2.0 ** -24 * mag[fine]).all()
    # rows of tiny operands: their low pieces would be below the smallest normal number
    X = A.copy()
    X[33] *= np.float32(1e-36)
    X[180] = np.float32(2.0 ** -120)
    _check(_product(X[None], (B * np.float32(2.0 ** 40))[None], "f32"), X[None], (B * np.float32(2.0 ** 40))[None])
    Z = B * np.float32(1e-36)
    _check(_product((A * np.float32(2.0 ** 30))[None], Z[None], "f32"), (A * np.float32(2.0 ** 30))[None], Z[None])
    # zeros are no tiny operands, and an all-zero operand gives zeros
    assert not _product(np.zeros((1, n, k), np.float32), B[None], "f32").any()


@pytest.mark.parametrize("trans", [(0, 0), (1, 1)])
@pytest.mark.parametrize("e", [100, 103, 108, 112, 120, 124])
def test_tiny_values_beside_ordinary_ones(e, trans):
    """Columns of A scaled by 2^-e against rows of B scaled by 2^e, every other one: a row holds values whose low pieces
    bf16 cannot hold beside ordinary ones, and both kinds of products count alike.  And where only such products count."""
    n, k, m = 200, 96, 150
    rng = inputs.rng_for(86, e)
    A, B = inputs.operands(rng, n, k, m, ("normal", 1.0), ("normal", 1.0), "f32")
    d = np.ones(k, np.float32)
    d[::2] = np.float32(2.0 ** -e)
    X, Y = A * d, B / d[:, None]
    _check(_product(X[None], Y[None], "f32", trans), X[None], Y[None])
    Y[1::2] = 0.0
    _check(_product(X[None], Y[None], "f32", trans), X[None], Y[None])
    X[:, 2::2], Y[2::2] = 0.0, 0.0                   # one product a symbol: rounded once (and what k - 1 zeros cannot add)
    C, ref = _product(X[None], Y[None], "f32", trans)[0], X.astype(np.float64) @ Y.astype(np.float64)
    assert (np.abs(C - ref) <= 2.0 ** -23 * np.abs(ref)).all()


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("k", [1, 2, 5, 31, 32])
def test_short_fp32_sums_are_rounded_once(k, trans):
    """k <= 32: summed in fp64, so what is left is one rounding to fp32, 2^-24 of the result or half the smallest number
    (and 2^-45 of |A| |B|, k roundings to 2^-53).  On values spread over 17 decades, near the smallest numbers, and on
    mantissas just above 1 + 2^-8, whose second and third bf16 pieces are the largest."""
    n, m = 200, 150
    rng = inputs.rng_for(87, 100 * k + trans[0] * 2 + trans[1])
    spread = [(rng.standard_normal(s) * np.exp(rng.uniform(-20, 20, s))).astype(np.float32) for s in ((n, k), (k, m))]
    above_one = [(rng.uniform(1.0035, 1.0042, s) * rng.choice([-1.0, 1.0], s)).astype(np.float32) for s in ((n, k), (k, m))]
    for A, B in (spread, above_one):
        for e in (0, 50, 58, 64, 72):
            X, Y = A * np.float32(2.0 ** -e), B * np.float32(2.0 ** -e)
            C = _product(X[None], Y[None], "f32", trans)[0]
            X, Y = X.astype(np.float64), Y.astype(np.float64)
            ref = X @ Y
            assert (np.abs(C - ref) <= np.maximum(2.0 ** -24 * np.abs(ref), 2.0 ** -150) + 2.0 ** -45 * (np.abs(X) @ np.abs(Y))).all(), e


@pytest.mark.parametrize("law", [("normal", 1.0), ("uniform", -1.0, 1.0), ("uniform", 0.0, 1.0)])
@pytest.mark.parametrize("shape", [(128, 48, 128), (512, 512, 512), (300, 1031, 129), (1024, 1024, 1024)])
def test_fp32_products_through_pieces_are_as_close_as_native_ones(shape, law):
    """Relative distance from the fp64 product, next to what native fp32 MFMAs gave on such operands with the
    sums over k split the same way: 1e-7 (k = 32 to 48), 2.0e-7 (k = 128 to 512), 2.9e-7 (k = 1024); all-positive
    operands: 8e-8 to 1.6e-7."""
    n, k, m = shape
    rng = inputs.rng_for(82, k)
    A, B = inputs.operands(rng, n, k, m, law, law, "f32")
    C = _product(A[None], B[None], "f32")[0]
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.linalg.norm(C - ref) <= (1.0e-7 if k < 128 or law[1] == 0.0 else 2.0e-7) * np.linalg.norm(ref)


@pytest.mark.parametrize("trans", [(0, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,batch", [((5, 3, 7), 2),            # rows shorter than a vector
                                         ((64, 9, 8), 600), ((33, 259, 41), 520),   # a wavefront per rows, and the last vector overlapped
                                         ((131, 260, 77), 1), ((70, 2053, 515), 1), ((515, 1027, 2051), 1)])
def test_scans_of_rows_at_any_alignment(shape, batch, dtype, trans):
    """Operand parities and parity blocks (fp64 sums) to 1e-12 and 1e-11, and an audit that finds the one wrong symbol
    (it re-forms the stored parities bit for bit), where rows start at any element and end in mid-vector."""
    import gpu_harness as H
    n, k, m = shape
    rng = inputs.rng_for(83, n + k)
    law = ("normal", 1.0)
    A, B = [np.stack(x) for x in zip(*[inputs.operands(rng, n, k, m, law, law, dtype) for _ in range(batch)])]
    A2 = A.copy()
    A2[-1, n - 1, k - 1] += 4.0
    A2 = inputs.store(A2, dtype)
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    g = H.run_gpu(A, B, A2, B, [], tau, dtype, trans[0], trans[1], ld_pad=1)
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    wn, wm = np.arange(1, n + 1), np.arange(1, m + 1)
    AP = np.stack([A64.sum(1), np.einsum("bnk,n->bk", A64, wn)], 1)
    BP = np.stack([B64.sum(2), np.einsum("bkm,m->bk", B64, wm)], 1)
    assert np.allclose(g.A_par, AP, rtol=1e-12, atol=1e-12 * np.abs(AP).max())
    assert np.allclose(g.B_par, BP, rtol=1e-12, atol=1e-12 * np.abs(BP).max())
    ref = np.concatenate([np.matmul(A64, BP.transpose(0, 2, 1)).transpose(0, 2, 1).reshape(batch, -1), np.matmul(AP, B64).reshape(batch, -1),
                          np.matmul(AP, BP.transpose(0, 2, 1)).reshape(batch, -1)], 1)
    assert np.allclose(g.C_par, ref, rtol=1e-11, atol=1e-12 * np.abs(ref).max())
    assert all(r.status == gecc.CLEAN for r in g.reports[:-1])
    assert g.reports[-1].status == gecc.CORRECTED and [e[:3] for e in g.reports[-1].errors()] == [(0, n - 1, k - 1)]
    assert np.array_equal(g.A, A64)


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(256, 2176, 256), (384, 3904, 768),     # 64 x 64 tiles, k split
                                   (1536, 4224, 768), (1000, 3584, 1000)])  # 128 x 128 tiles, k split
def test_bf16_products_of_few_tiles_and_long_k(shape, trans):
    """Aligned bf16 products that leave most compute units of the 256 x 256-tile kernel idle: product, decisions and
    located errors (one in the last tile of C, one in A) next to the fp64 product."""
    import gpu_harness as H
    n, k, m = shape
    rng = inputs.rng_for(84, n)
    law = ("normal", 1.0)
    A, B = inputs.operands(rng, n, k, m, law, law, "bf16")
    _check(_product(A[None], B[None], "bf16", trans), A[None], B[None])
    A2 = A.copy()
    A2[n - 1, k - 1] = inputs.store(A2[n - 1, k - 1:k] + 4.0, "bf16")[0]
    g = H.run_gpu(A, B, A2, B, [(0, n - 2, m - 1, 50.0)], gecc.noise_thresholds(n, k, m, 1.0, 1.0), "bf16", trans[0], trans[1])
    assert g.reports[0].status == gecc.CORRECTED
    assert [e[:3] for e in g.reports[0].errors()] == [(0, n - 1, k - 1), (2, n - 2, m - 1)]
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.abs(g.C[0] - ref).max() <= 1e-5 * np.abs(ref).max() and np.array_equal(g.A[0], A)


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("pad", [0, 24])
def test_ragged_tiles_in_the_kernel_with_256_by_256_tiles(pad, trans, monkeypatch):
    """(GECC_CU_COUNT keeps the plan with 256 x 256 tiles for a product this small.)"""
    import gpu_harness as H
    monkeypatch.setenv("GECC_CU_COUNT", "256")
    n, k, m = 520, 256, 264
    rng = inputs.rng_for(85, pad)
    A, B = inputs.operands(rng, n, k, m, ("normal", 1.0), ("normal", 1.0), "bf16")
    cf = [(0, n - 1, m - 1, 37.5), (0, 256, 0, -12.25)]
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    g = H.run_gpu(A, B, A, B, cf, tau, "bf16", trans[0], trans[1], ld_pad=pad)
    H.compare(g, H.run_oracle(A, B, A, B, cf, tau), 1e-5, what="256 tiles, pad %d" % pad)
    assert g.pad_untouched and [e[:3] for e in g.reports[0].errors()] == [(2, 256, 0), (2, n - 1, m - 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("trans", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("shape", [(129, 130, 131), (255, 513, 3), (5, 640, 257), (96, 4133, 71),
                                   (260, 300, 16200)])      # the most workgroups of these (vectors of 8 bytes)
def test_column_scans_at_their_ends(shape, dtype, trans):
    """Rows that end in the middle of a vector of 8 or 16 bytes, chunks whose last rows are no whole batch, rows shorter than a
    vector: operand parities and parity blocks in fp64, rounded k times (n, m times) at most, in any order."""
    import torch
    import gpu_harness as H
    n, k, m = shape
    law = ("normal", 1.0)
    A, B = inputs.operands(inputs.rng_for(84, n + k), n, k, m, law, law, dtype)
    g = H.run_gpu(A, B, A, B, [], gecc.noise_thresholds(n, k, m, 1.0, 1.0), dtype, trans[0], trans[1])
    A, B = A.astype(np.float64), B.astype(np.float64)
    wn, wm = np.arange(1, n + 1.0), np.arange(1, m + 1.0)
    aP, bP = np.stack([A.sum(0), wn @ A]), np.stack([B.sum(1), B @ wm])
    mag_a, mag_b = np.stack([np.abs(A).sum(0), wn @ np.abs(A)]), np.stack([np.abs(B).sum(1), np.abs(B) @ wm])
    eps = 2.0 ** -52
    assert (np.abs(g.A_par[0] - aP) <= n * eps * mag_a).all() and (np.abs(g.B_par[0] - bP) <= m * eps * mag_b).all()
    pr, pc = (A @ bP.T).T, aP @ B
    mr, mc = (np.abs(A) @ mag_b.T).T, mag_a @ np.abs(B)
    got = g.C_par[0]
    assert (np.abs(got[:2 * n].reshape(2, n) - pr) <= 2 * (k + m) * eps * mr).all()
    assert (np.abs(got[2 * n:2 * n + 2 * m].reshape(2, m) - pc) <= 2 * (k + n) * eps * mc).all()


def _check_parities(g, A, B):
    """Operand parities and parity blocks in fp64, rounded k times (n, m times) at most, in any order."""
    (_, n, k), m = A.shape, B.shape[2]
    eps = 2.0 ** -52
    wn, wm = np.arange(1, n + 1.0), np.arange(1, m + 1.0)
    for b in range(A.shape[0]):
        X, Y = A[b].astype(np.float64), B[b].astype(np.float64)
        aP, bP = np.stack([X.sum(0), wn @ X]), np.stack([Y.sum(1), Y @ wm])
        mag_a, mag_b = np.stack([np.abs(X).sum(0), wn @ np.abs(X)]), np.stack([np.abs(Y).sum(1), np.abs(Y) @ wm])
        assert (np.abs(g.A_par[b] - aP) <= n * eps * mag_a).all() and (np.abs(g.B_par[b] - bP) <= m * eps * mag_b).all()
        pr, pc = (X @ bP.T).T, aP @ Y
        mr, mc = (np.abs(X) @ mag_b.T).T, mag_a @ np.abs(Y)
        got = g.C_par[b]
        assert (np.abs(got[:2 * n].reshape(2, n) - pr) <= 2 * (k + m) * eps * mr).all()
        assert (np.abs(got[2 * n:2 * n + 2 * m].reshape(2, m) - pc) <= 2 * (k + n) * eps * mc).all()


# Batches whose column scans go in vectors of 16 bytes, in launches of their own (test_launch_plans.py holds them to it): rows that end
# in the middle of one, a second chunk whose rows are no whole batch
WIDE_SCANS = ((141, 139, 133), 520)


@pytest.mark.parametrize("staged", [True, False])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("trans", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_column_scans_of_many_workgroups_at_their_ends(trans, dtype, staged):
    import gpu_harness as H
    (n, k, m), batch = WIDE_SCANS
    rng = inputs.rng_for(89, n)
    A, B = [inputs.store(rng.standard_normal(x), dtype) for x in ((batch, n, k), (batch, k, m))]
    g = H.run_gpu(A, B, A, B, [], gecc.noise_thresholds(n, k, m, 1.0, 1.0), dtype, trans[0], trans[1], staged=staged)
    _check_parities(g, A, B)


# (test_launch_plans.py holds them to the tiles and ranges, and to the scans in the product's launch)
BESIDE_CASES = [((1530, 4222, 760), 128, 7),        # 128 x 128 tiles, seven ranges of k
                ((256, 64, 256), 64, 1)]            # the smallest that the 256 x 256-tile kernel could take


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(1280, 2176, 1408),       # aligned, tiles of 64 in one range
                                   (1300, 1750, 1211),       # ragged, scans before or behind the product's workgroups
                                   (192, 64, 256)] +         # too small for the 256 x 256-tile kernel
                                  [x[0] for x in BESIDE_CASES])
def test_bf16_products_with_their_scans_beside_them(shape, trans):
    import gpu_harness as H
    n, k, m = shape
    law = ("normal", 1.0)
    A, B = inputs.operands(inputs.rng_for(85, n + k), n, k, m, law, law, "bf16")
    A2, B2, cf, eff = inputs.apply_operand_faults(A, B, [inputs.Fault(inputs.MAT_B, k - 1, 0, 5.0), inputs.Fault(inputs.MAT_C, n - 1, m - 1, 60.0)], "bf16")
    cfb = [(0,) + c for c in cf]
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    g = H.run_gpu(A, B, A2, B2, cfb, tau, "bf16", trans[0], trans[1])
    H.compare(g, H.run_oracle(A, B, A2, B2, cfb, tau), 1e-5, what="%s, trans %s" % (shape, trans))
    clean, one = [H.run_gpu(A, B, A, B, [], tau, "bf16", trans[0], trans[1], staged=x) for x in (True, False)]
    assert clean.reports[0].status == one.reports[0].status == gecc.CLEAN
    assert np.array_equal(clean.C, one.C) and np.array_equal(clean.A_par, one.A_par)
    assert np.allclose(clean.C_par, one.C_par, rtol=1e-12, atol=1e-13 * np.abs(clean.C_par).max())


@pytest.mark.parametrize("trans", [(0, 0), (1, 1)])
def test_the_256_tile_kernel_at_sizes_that_gemm_tile_has_taken_over(trans, monkeypatch):
    """Multiples of 64 go to gemm_tile where that saves launches; the other kernel keeps its results there."""
    import gpu_harness as H
    monkeypatch.setenv("GECC_CU_COUNT", "256")
    n, k, m = 576, 192, 320
    law = ("normal", 1.0)
    A, B = inputs.operands(inputs.rng_for(86, 1), n, k, m, law, law, "bf16")
    cfb = [(0, n - 1, m - 1, 60.0), (0, 5, 7, -30.0)]
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    H.compare(H.run_gpu(A, B, A, B, cfb, tau, "bf16", trans[0], trans[1]), H.run_oracle(A, B, A, B, cfb, tau), 1e-5, what=str(trans))


# bf16 products of 449 x 450 in fewer ranges of k than they could have, whose sums are put aside every 128 or 256 terms
# (test_launch_plans.py holds them to that kernel): pieces of which the last is a single term, a k-tile, one and a half, a whole one; two ranges
FOLD_KS = (256, 257, 320, 383, 384, 385, 449, 513, 640, 901, 1100, 2049, 2500)


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("k", FOLD_KS)
def test_sums_put_aside(k, trans):
    A, B = [x[None] for x in inputs.operands(inputs.rng_for(90, k), 449, k, 450, ("normal", 1.0), ("normal", 1.0), "bf16")]
    _check(_product(A, B, "bf16", trans), A, B)
    _check(_product(A, B, "bf16", trans, pad=3, shift=1), A, B)


@pytest.mark.parametrize("dtype,shape,trans,limit", [("bf16", (700, 700, 700), (0, 0), 7.5e-8), ("bf16", (128, 896, 640), (0, 0), 7.7e-8),
                                                     ("bf16", (1313, 1220, 2578), (0, 0), 1.48e-7), ("bf16", (3440, 240, 2496), (1, 1), 6.7e-8),
                                                     ("bf16", (2509, 3866, 266), (1, 0), 1.49e-7), ("bf16", (776, 3240, 1496), (0, 1), 1.47e-7),
                                                     ("f32", (256, 512, 256), (0, 0), 7.05e-8), ("f32", (512, 512, 512), (0, 0), 7.1e-8)])
def test_distance_from_fp64(dtype, shape, trans, limit):
    """What the order of a product's sums leaves, as |C - C64| / |C64| in 2-norms.  With the whole range of k in as few chains as tiles and
    ranges alone would give, the bf16 ones are 1.05e-7, 1.19e-7, 2.04e-7, 8.3e-8, 1.83e-7 and 1.52e-7; their limits are 5 % above 7.1e-8, 7.3e-8,
    1.41e-7, 6.4e-8, 1.42e-7 and 1.40e-7, the distances of plans with more ranges.  fp32 in eight ranges that are added up one by one: 7.27e-8
    and 7.31e-8, in four 6.92e-8 and 7.00e-8.  Over 65 000 symbols and more all of this varies by less than 1 %."""
    n, k, m = shape
    A, B = [x[None] for x in inputs.operands(inputs.rng_for(87, n), n, k, m, ("normal", 1.0), ("normal", 1.0), dtype)]
    C = _product(A, B, dtype, trans)
    _check(C, A, B)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.linalg.norm(C - ref) <= limit * np.linalg.norm(ref)


@pytest.mark.parametrize("shape,trans,limit", [((1258, 2122, 1110), (1, 0), 1.43e-7), ((768, 2816, 1408), (0, 1), 1.46e-7), ((256, 2688, 4480), (0, 1), 1.45e-7)])
def test_distance_from_fp64_where_tiles_of_128_would_have_shorter_ranges(shape, trans, limit):
    """5 % above the distances of tiles of 128 in four and five ranges, 1.36e-7, 1.39e-7 and 1.38e-7; tiles of 64 with two chains over one range
    (1258 x 2122 x 1110) or two are 1.90e-7, 1.54e-7 and 1.50e-7 from the fp64 product."""
    test_distance_from_fp64("bf16", shape, trans, limit)


ALONE_SHAPE = (448, 192, 18624)


@pytest.mark.parametrize("trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("pad,shift", [(0, 0), (8, 0), (0, 1)])
def test_a_product_on_its_own_in_another_kernel_than_its_plan_has(pad, shift, trans):
    """Planned in tiles of 64 (NN), on its own in tiles of 256 x 256 (test_launch_plans.py holds it to both); off a 16-byte boundary
    the plan's kernel takes it after all."""
    A, B = [x[None] for x in inputs.operands(inputs.rng_for(88, pad), *ALONE_SHAPE, ("normal", 1.0), ("normal", 1.0), "bf16")]
    _check(_product(A, B, "bf16", trans, pad=pad, shift=shift), A, B)
