"""The kernels that turn factors between column-major and row-major order, rebuild the
residual from them and sum held-out errors, at the edges of their tiles: features
around multiples of 4, 16, 32 and 64, rows around 64, held-out sets that turn neither,
one or both factors.

Tolerances: the rebuilt residual is a float64 sum (k terms, below 1e-15 k of the
summed magnitudes) rounded once to the value type, so it lies within one rounding of
numpy's float64 value; the RMSE is a float64 sum of at most 20,000 squares: 1e-12.
"""
import numpy as np
import pytest

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
@pytest.mark.parametrize("precision", [0, 1])
def test_factors_residual_and_rmse(k, precision):
    m, n = 193, 130
    layout = sorted(LAYOUTS)[k % 4]
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
    # Held-out sets that turn neither factor, H only (8 n <= entries < 8 m), or both.
    for entries in (1, 100, 8 * n, 8 * m, 20_000):
        r = rng.integers(0, m, entries).astype(np.int32)
        c = rng.integers(0, n, entries).astype(np.int32)
        a = rng.standard_normal(entries).astype(np.float32)
        ref = np.sqrt(np.mean((a.astype(np.float64) - (Wd[r] * Hd[c]).sum(1)) ** 2))
        assert abs(g.rmse(r, c, a) - ref) <= 1e-12 * ref
    g.close()
