"""The shares of small copies against the oracle: a workgroup per window, share bounds
moved to row starts (up to half a share), fewer workgroups (down to a window per wave)
where a bound would have to move further, and the combine kernel where neither will do.

Tolerance: float sums of up to 512 entries and one rounding per coordinate, over two
features and two inner iterations: 1e-3 of the largest coordinate of a feature, as for
every layout (about 1e-6 is seen).
"""
import numpy as np
import pytest

from oracle import Oracle
from paper_1511_02433_amd import synth
from paper_1511_02433_amd.ccdpp import CCDPP, make_options
from gpu_util import colscaled_max_rel_err

pytestmark = pytest.mark.gpu

# Row lengths, columns, and whether the user-major copy needs the combine kernel.
CASES = {
    "one_window": ([8] * 60, 64, False),            # less than one window: one workgroup
    "window_edge": ([64] * 16 + [8], 300, False),   # two windows and one lane group
    "bounds_move": ([700] * 40 + [40] * 100, 900, False),   # rows longer than a window
    "halved": ([1000] * 60, 1200, False),           # a bound a whole row away from its share
    "combine": ([9000, 7000, 5000] + [30] * 200, 9500, True),  # rows over many workgroups
    "many_rows": ([3] * 20_000, 500, False),        # 64 segment starts in every window
    "one_round": ([600] * 3600, 4000, False),       # past a window per wave of the chip
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_small_copy(name):
    lens, n, combined = CASES[name]
    m, k, lam = len(lens), 2, 0.3
    row, col, val, H0 = synth.lengths_problem(lens, n, k, seed=77)
    g = CCDPP(m, n, k, lam, row, col, val)
    info = g.info()
    print(f"case {name}: nnz {row.size} workgroups {info['u_workgroups']}/{info['v_workgroups']} "
          f"combined {info['u_rows_combined']}/{info['v_rows_combined']} finished in the pass "
          f"{info['u_rows_finished_in_pass']}/{info['v_rows_finished_in_pass']}", flush=True)
    assert (info["u_rows_combined"] > 0) == combined
    g.set_factors(np.zeros((m, k), np.float32), H0)
    o = Oracle(m, n, k, lam, row, col, val, H0)
    for _ in range(2):
        g.run(1, 2)
        o.run(1, 2)
        W, H = g.factors()
        Wo, Ho = o.factors()
        ew, eh = colscaled_max_rel_err(W, Wo), colscaled_max_rel_err(H, Ho)
        print(f"  W err {ew:.2e}  H err {eh:.2e}", flush=True)
        assert ew <= 1e-3 and eh <= 1e-3
    assert g.check_consistency() == 0
    g.close()
    o.close()


@pytest.mark.parametrize("kind", ["double_one_tile", "double_tiles", "double_hot", "float_hot"])
def test_cached_accesses_change_nothing(kind):
    # Hot and double copies whose streams fit the memory-side cache use cached accesses
    # and plain indices; a forced streaming policy gives the same bits.
    lens = [850, 700, 300, 40] + list(np.random.default_rng(31).integers(0, 80, 1496))
    m, n, k = len(lens), 900, 4
    row, col, val, H0 = synth.lengths_problem(lens, n, k, seed=32)
    kw = {"double_one_tile": dict(precision=1), "double_tiles": dict(precision=1, gather_mode=(2, 2), tile_width=(192, 128)),
          "double_hot": dict(precision=1, gather_mode=(3, 3), tile_width=(64, 96)),
          "float_hot": dict(gather_mode=(3, 3), tile_width=(64, 96))}[kind]
    print(f"case: cached accesses, {kind}", flush=True)
    outs = []
    for cache in ((0, 0), (1, 1)):
        g = CCDPP(m, n, k, 0.1, row, col, val, opts=make_options(cache=cache, **kw))
        g.set_factors(None, H0)
        g.run(2, 2)
        g.run(1, 1)
        g.ccd_run(1)
        outs.append(g.factors_f64() + (g.residual_f64(), g.train_rmse()))
        assert g.check_consistency() == 0
        g.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("per_row,tiled", [(60, True), (4, False)])
@pytest.mark.parametrize("precision", [0, 1])
def test_short_segments_are_tiled_where_gathers_cost_more(per_row, tiled, precision):
    # Rows spread evenly over 200,000 columns: of 60 entries, about 48 lie past the columns
    # that a hot layout stages, against ten segments in tiles; of 4 entries, as many
    # segments as entries.  The transposed problem takes the item-major copy there.
    m, n, k, lam = 2_000, 200_000, 2, 0.5
    row, col, val, H0 = synth.lengths_problem([per_row] * m, n, k, seed=per_row)
    print(f"case: {per_row} per row, precision {precision}", flush=True)
    for transposed in (False, True):
        a = (n, m, k, lam, col, row, val) if transposed else (m, n, k, lam, row, col, val)
        h0 = np.random.default_rng(3).standard_normal((a[1], k)).astype(np.float32) * 0.1
        g = CCDPP(*a, opts=make_options(precision=precision))
        info = g.info()
        side = "v" if transposed else "u"
        assert (info[f"{side}_gather"] == 2 and info[f"{side}_tiles"] > 1) == tiled
        g.set_factors(None, h0)
        o = Oracle(*a, h0)
        for step in range(2):
            g.run(1, 2)
            o.run(1, 2)
            W, H = g.factors_f64()
            Wo, Ho = o.factors()
            tol = 1e-9 if precision else 1e-3
            assert colscaled_max_rel_err(W, Wo) <= tol and colscaled_max_rel_err(H, Ho) <= tol
        assert g.check_consistency() == 0
        g.close()
        o.close()


@pytest.mark.parametrize("n", [32_768, 32_769])
def test_tile_counts_at_the_lds_limit(n):
    # The item-major copy's (tile, row) counts are taken in LDS for up to 32,768 rows; the
    # user-major copy's tiles put their order through several resets.
    m, k, lam = 3_000, 2, 0.5
    rng = np.random.default_rng(n)
    key = np.unique(rng.integers(0, m, 80_000) * n + rng.integers(0, n, 80_000))
    row, col = (key // n).astype(np.int32), (key % n).astype(np.int32)
    row[:3], col[:3] = [m - 1, m - 1, 0], [n - 1, 0, n - 1]
    _, first = np.unique(row.astype(np.int64) * n + col, return_index=True)
    row, col = row[first], col[first]
    val = rng.standard_normal(row.size).astype(np.float32)
    H0 = (rng.standard_normal((n, k)) * 0.1).astype(np.float32)
    for tile in ((0, 0), (9_024, 64)):
        print(f"case: n {n} tile widths {tile}", flush=True)
        g = CCDPP(m, n, k, lam, row, col, val, opts=make_options(gather_mode=(2, 2), tile_width=tile))
        g.set_factors(None, H0)
        o = Oracle(m, n, k, lam, row, col, val, H0)
        g.run(1, 2)
        o.run(1, 2)
        W, H = g.factors()
        Wo, Ho = o.factors()
        assert colscaled_max_rel_err(W, Wo) <= 1e-3 and colscaled_max_rel_err(H, Ho) <= 1e-3
        assert g.check_consistency() == 0
        g.close()
        o.close()


def _one_share_per_8192_snaps(lens):
    """Whether shares of 8,192 entries (a window per wave) can start on rows with no bound
    moved by more than an eighth of a share: the work of a range is its entries plus 4
    per row, rows start at multiples of 8."""
    start = np.concatenate([[0], np.cumsum((np.sort(lens)[::-1] + 7) // 8 * 8)])
    start, npad = start[:-1], -(-int(start[-1]) // 512) * 512
    work = start + 4 * (np.arange(start.size) + 1)
    total, shares = npad + 4 * start.size, -(-npad // 8192)
    for g in range(1, shares):
        t = total // shares * g + total % shares * g // shares
        s = int(np.searchsorted(work, t, side="right")) - 1
        near = [abs(int(work[x]) - t) for x in (s, s + 1) if 0 <= x < start.size]
        if min(near) > total // shares // 8:
            return False
    return True


def _long_rows(name):
    if name == "equal":
        return [1_500] * 40
    if name == "one_longer":
        return [3_200] + [449] * 200
    seed = int(name.rsplit("_", 1)[1])
    rng = np.random.default_rng(seed)
    nnz, rows = int(np.exp(rng.uniform(np.log(5e4), np.log(3e5)))), int(rng.integers(300, 6_000))
    w = (np.arange(rows) + rows / 200) ** -rng.choice([0.9, 1.001, 1.2])
    return np.clip(w / w.sum() * nnz, 1, 4_600).astype(int).tolist()


@pytest.mark.parametrize("name", ["equal", "one_longer"] + [f"power_law_{s}" for s in range(24)])
def test_long_rows_keep_the_finish_in_the_pass(name):
    # Where workgroups of one window each cannot start their shares on rows, fewer can: as
    # long as shares of a window per wave do, no combine runs.
    lens = _long_rows(name)
    m, n, k, lam = len(lens), 4_700, 2, 0.3
    row, col, val, H0 = synth.lengths_problem(lens, n, k, seed=78)
    g = CCDPP(m, n, k, lam, row, col, val)
    info = g.info()
    snaps = _one_share_per_8192_snaps(lens)
    print(f"case {name}: nnz {row.size} rows {m} longest {max(lens)} snaps {snaps} workgroups "
          f"{info['u_workgroups']} combined {info['u_rows_combined']}", flush=True)
    assert info["u_rows_combined"] == 0 or not snaps
    g.set_factors(np.zeros((m, k), np.float32), H0)
    o = Oracle(m, n, k, lam, row, col, val, H0)
    g.run(1, 2)
    o.run(1, 2)
    for x, y in zip(g.factors(), o.factors()):
        assert colscaled_max_rel_err(x, y) <= 1e-3
    g.close()
    o.close()


@pytest.mark.parametrize("m,tiles", [(90, 63), (90, 64), (90, 65), (1, 130), (700, 200), (16_383, 70), (16_384, 70)])
def test_many_tiles(m, tiles):
    # A row's tiles are walked by a wave from 64 tiles on, below 16,384 rows: partials of many
    # segments, of segments cut between workgroups, and of rows without entries.
    k, lam, n = 2, 0.3, tiles * 64
    rng = np.random.default_rng(m + tiles)
    key = np.unique(np.concatenate([rng.integers(0, m * n, 120_000),
                                    (m // 2) * n + rng.integers(0, n, 3_000)]))
    row, col = (key // n).astype(np.int32), (key % n).astype(np.int32)
    if m > 1:
        keep = row != m - 1  # the last row is empty
        row, col = row[keep], col[keep]
    val = rng.standard_normal(row.size).astype(np.float32)
    H0 = (rng.standard_normal((n, k)) * 0.1).astype(np.float32)
    print(f"case: {m} rows, {tiles} tiles", flush=True)
    for kw in (dict(tile_width=(64, 0)), dict(tile_width=(64, 0), workgroups=37, precision=1)):
        g = CCDPP(m, n, k, lam, row, col, val, opts=make_options(gather_mode=(2, 0), **kw))
        info = g.info()
        assert info["u_tiles"] == tiles
        g.set_factors(None, H0)
        o = Oracle(m, n, k, lam, row, col, val, H0)
        g.run(1, 2)
        o.run(1, 2)
        for x, y in zip(g.factors_f64(), o.factors()):
            assert colscaled_max_rel_err(x, y) <= (1e-9 if "precision" in kw else 1e-3)
        assert g.check_consistency() == 0
        g.close()
        o.close()
