"""The kernels that turn factors between column-major and row-major order, rebuild the
residual from them and sum held-out errors, at the edges of their tiles: features
around multiples of 4, 16, 32 and 64, rows around 64, held-out sets that turn neither,
one or both factors, few and many values, entries and windows.

Tolerances: the rebuilt residual is a float64 sum (k terms, below 1e-15 k of the
summed magnitudes) rounded once to the value type, so it lies within one rounding of
numpy's float64 value; the RMSE is a float64 sum of at most 20,000 squares: 1e-12.
"""
import numpy as np
import pytest

import paper_1511_02433_amd.ccdpp as C
from paper_1511_02433_amd import synth
from paper_1511_02433_amd.ccdpp import CCDPP, make_options

pytestmark = pytest.mark.gpu

LAYOUTS = {
    "tiled": dict(gather_mode=(2, 2), cache=(1, 1)),            # 16-bit indices, delta-coded
    "several_tiles": dict(gather_mode=(2, 2), tile_width=(64, 64)),
    "hot": dict(gather_mode=(3, 3), tile_width=(64, 64)),       # 32-bit indices
    "global": dict(gather_mode=(1, 1)),
}


@pytest.mark.parametrize("k", [1, 3, 4, 5, 16, 17, 32, 33, 64, 67, 130])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("precision", [0, 1])
def test_factors_residual_and_rmse(k, layout, precision):
    m, n = 193, 130
    row, col, val, _ = synth.small_random(m, n, 6_000, k, seed=500 + k)
    rng = np.random.default_rng(900 + k)
    dt = np.float64 if precision else np.float32
    W = rng.standard_normal((m, k)).astype(dt)
    H = rng.standard_normal((n, k)).astype(dt)
    kw = dict(LAYOUTS[layout], precision=precision)
    print(f"case: k {k} precision {precision} {layout}", flush=True)
    g = CCDPP(m, n, k, 0.1, row, col, val, opts=make_options(**kw))
    (g.set_factors_f64 if precision else g.set_factors)(W, H)
    W2, H2 = g.factors_f64() if precision else g.factors()
    assert np.array_equal(W, W2) and np.array_equal(H, H2)
    Wd, Hd = W.astype(np.float64), H.astype(np.float64)
    dot = (Wd[row] * Hd[col]).sum(1)
    mag = (np.abs(Wd[row]) * np.abs(Hd[col])).sum(1) + np.abs(val)
    want = val.astype(np.float64) - dot
    got = g.residual_f64()
    bound = np.abs(want) * (2.0 ** -24 if precision == 0 else 0.0) * 1.001 + mag * 4e-16 * (k + 2)
    assert (np.abs(got - want) <= bound).all()
    assert g.check_consistency() == 0
    for entries in (1, 100, 8 * n, 8 * m, 20_000):
        r = rng.integers(0, m, entries).astype(np.int32)
        c = rng.integers(0, n, entries).astype(np.int32)
        a = rng.standard_normal(entries).astype(np.float32)
        ref = np.sqrt(np.mean((a.astype(np.float64) - (Wd[r] * Hd[c]).sum(1)) ** 2))
        assert abs(g.rmse(r, c, a) - ref) <= 1e-12 * ref
    g.close()


@pytest.mark.parametrize("m,n,turned", [(3_000, 2_000, "both"), (40_000, 2_000, "H"), (2_000, 40_000, "W"),
                                        (1_800, 1_800, "neither")])
@pytest.mark.parametrize("precision", [0, 1])
def test_rmse_from_turned_factors(m, n, turned, precision):
    # 120,000 entries times 70 features turn a factor of at least 2^17 values and at most
    # 15,000 rows; with triplets that may not be used, each variant names the first.
    k, entries = 70, 120_000
    row, col, val, _ = synth.small_random(m, n, 9_000, k, seed=m)
    rng = np.random.default_rng(n)
    W = rng.standard_normal((m, k)).astype(np.float32)
    H = rng.standard_normal((n, k)).astype(np.float32)
    print(f"case: {m} x {n}, turned {turned}, precision {precision}", flush=True)
    g = CCDPP(m, n, k, 0.1, row, col, val, opts=make_options(precision=precision))
    g.set_factors(W, H)
    r = rng.integers(0, m, entries).astype(np.int32)
    c = rng.integers(0, n, entries).astype(np.int32)
    a = rng.standard_normal(entries).astype(np.float32)
    err = a.astype(np.float64)
    for t in range(k):
        err -= W[:, t].astype(np.float64)[r] * H[:, t].astype(np.float64)[c]
    ref = np.sqrt(np.mean(err ** 2))
    got = g.rmse(r, c, a)
    assert abs(got - ref) <= 1e-12 * ref
    for arr, x in ((r, m), (c, -1), (a, np.nan)):
        keep = arr[777], arr[-1]
        arr[777] = arr[-1] = x
        with pytest.raises(C.CCDPPError) as ei:
            g.rmse(r, c, a)
        assert ei.value.code == C.CCDPP_EINVAL and "777" in str(ei.value)
        arr[777], arr[-1] = keep
        assert g.rmse(r, c, a) == got
    _, hist = g.run_until(1, 1, -1.0, (r, c, a))
    assert hist[0, 2] == g.rmse(r, c, a)
    g.close()


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (1, 64, 2), (63, 65, 31), (64, 1, 33), (65, 63, 65), (200, 250, 500),
                                   (64, 65, 4_100), (3, 2, 100_003), (6_000, 70, 60), (70_000, 40, 40),
                                   (70_000, 129, 3)])
@pytest.mark.parametrize("precision", [0, 1])
def test_turns_of_few_rows_or_many_features(m, n, k, precision):
    # Up to 2^18 values, or four to a row, are turned value by value; few rows of more have
    # their tiles shared out over several workgroups; 70,000 rows and k = 40 fill the chip
    # alone and a workgroup takes both tiles of its rows.
    rng = np.random.default_rng(m + k)
    row = np.arange(m, dtype=np.int32)
    col = (row % n).astype(np.int32)
    g = CCDPP(m, n, k, 0.1, row, col, np.ones(m, np.float32), opts=make_options(precision=precision))
    print(f"case: {m} x {n}, k {k}, precision {precision}", flush=True)
    W = rng.standard_normal((m, k)).astype(np.float32)
    H = rng.standard_normal((n, k)).astype(np.float32)
    g.set_factors(W, H)
    for x, y in zip((W, H, W, H), g.factors() + g.factors_f64()):
        assert np.array_equal(x, y)
    H = H[::-1].copy()
    g.set_factors(None, H)
    for x, y in zip((W, H), g.factors()):
        assert np.array_equal(x, y)
    g.close()


def test_factors_at_the_largest_k():
    # The features of a turn are counted past 2^31 - 32 without overflow (8.6 GB per factor).
    k = 2**31 - 1
    g = CCDPP(1, 1, k, 0.1, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32), seed=3)
    H = np.empty((1, k), np.float32)
    print("case: k 2^31 - 1", flush=True)
    assert C.lib().ccdpp_get_factors(g._h, None, C._p(H)) == 0
    g.close()
    for at in (0, k // 2, k - 64):
        part = H[0, at:at + 64].astype(np.float64)
        assert np.isfinite(part).all() and 0.04 < part.std() < 0.2  # N(0, 0.01)


@pytest.mark.parametrize("k,nnz", [(6, 820_000), (9, 480_000), (16, 300_000), (20, 250_000), (32, 150_000),
                                   (67, 70_000), (130, 36_000)])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("precision", [0, 1])
def test_rebuild_in_rows(k, nnz, layout, precision):
    # From 2^22 entries times features the rebuild reads rows of H, 4, 8 or 16 lanes to a
    # row; 820,000 entries give every wave a window, fewer share a window out.
    m, n = 2_900, 701
    rng = np.random.default_rng(k)
    key = rng.choice(m * n, nnz, replace=False)
    row, col = (key // n).astype(np.int32), (key % n).astype(np.int32)
    val = rng.standard_normal(nnz).astype(np.float32)
    dt = np.float64 if precision else np.float32
    W, H = rng.standard_normal((m, k)).astype(dt), rng.standard_normal((n, k)).astype(dt)
    kw = dict(LAYOUTS[layout], precision=precision)
    if layout != "global":
        kw["tile_width"] = (192, 320)
    print(f"case: k {k} nnz {nnz} {layout} precision {precision}", flush=True)
    g = CCDPP(m, n, k, 0.1, row, col, val, opts=make_options(**kw))
    (g.set_factors_f64 if precision else g.set_factors)(W, H)
    Wd, Hd = W.astype(np.float64), H.astype(np.float64)
    dot, mag = np.zeros(nnz), np.abs(val).astype(np.float64)
    for t in range(k):
        x = Wd[:, t][row] * Hd[:, t][col]
        dot, mag = dot + x, mag + np.abs(x)
    want = val.astype(np.float64) - dot
    got = g.residual_f64()
    bound = np.abs(want) * (2.0 ** -24 if precision == 0 else 0.0) * 1.001 + mag * 4e-16 * (k + 2)
    assert (np.abs(got - want) <= bound).all()
    assert g.check_consistency() == 0
    g.close()
