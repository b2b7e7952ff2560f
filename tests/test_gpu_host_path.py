"""Caller memory on its way to the device and back: sizes around the staging chunks, and
arguments checked on the host (few) and on the device (many), which name the first
bad element and change nothing.
"""
import numpy as np
import pytest

import paper_1511_02433_amd.ccdpp as C
from paper_1511_02433_amd import synth
from paper_1511_02433_amd.ccdpp import CCDPP, CCDPPError, CCDPP_EINVAL

pytestmark = pytest.mark.gpu


# Values of W: below the staging limit (4 MiB), on and around whole chunks, and more
# chunks than slots (six workers with two each).
@pytest.mark.parametrize("values", [1000, (4 << 20) // 4 - 1, (4 << 20) // 4, (4 << 20) // 4 + 1,
                                    3 * (4 << 20) // 4 + 5, 14 * (4 << 20) // 4 + 17])
def test_factors_round_trip(values):
    m, n, k = values, 40, 1
    rng = np.random.default_rng(values)
    row = rng.integers(0, m, 500).astype(np.int32)
    col = (np.arange(500) % n).astype(np.int32)
    _, first = np.unique(row.astype(np.int64) * n + col, return_index=True)
    row, col = row[first], col[first]
    val = rng.standard_normal(row.size).astype(np.float32)
    print(f"case: round trip of {values} values", flush=True)
    g = CCDPP(m, n, k, 0.1, row, col, val)
    for seed in (1, 2):  # the second call finds the slots of the first
        W = np.random.default_rng(seed).standard_normal((m, k)).astype(np.float32)
        H = np.random.default_rng(seed + 5).standard_normal((n, k)).astype(np.float32)
        g.set_factors(W, H)
        W2, H2 = g.factors()
        assert np.array_equal(W, W2) and np.array_equal(H, H2)
    g.close()


def test_factors_round_trip_on_the_per_thread_stream():
    # hipStreamPerThread (2) is another stream in each thread, and so in a copy's workers.
    m, n, k = 14 * (4 << 20) // 4 + 17, 40, 1
    rng = np.random.default_rng(3)
    row, col = rng.permutation(m)[:500].astype(np.int32), (np.arange(500) % n).astype(np.int32)
    g = CCDPP(m, n, k, 0.1, row, col, rng.standard_normal(500).astype(np.float32))
    g.set_stream(2)
    for _ in range(3):
        W = rng.standard_normal((m, k)).astype(np.float32)
        H = rng.standard_normal((n, k)).astype(np.float32)
        g.set_factors(W, H)
        W2, H2 = g.factors()
        assert np.array_equal(W, W2) and np.array_equal(H, H2)
    g.close()


@pytest.mark.parametrize("entries", [50, 24_576, 24_577, 400_000])
def test_bad_held_out_triplets_are_named(entries):
    m, n, k = 700, 300, 3
    row, col, val, H0 = synth.small_random(m, n, 9_000, k, seed=8)
    g = CCDPP(m, n, k, 0.1, row, col, val)
    g.set_factors(None, H0)
    g.run(1, 2)
    rng = np.random.default_rng(entries)
    r = rng.integers(0, m, entries).astype(np.int32)
    c = rng.integers(0, n, entries).astype(np.int32)
    a = rng.standard_normal(entries).astype(np.float32)
    ref = g.rmse(r, c, a)
    W, H = g.factors()
    at = entries // 2
    for arr, x, text in ((r, m, f"test entry {at} out of range"), (r, -1, f"test entry {at} out of range"),
                         (c, n, f"test entry {at} out of range"), (a, np.nan, f"test value {at} is not finite"),
                         (a, np.inf, f"test value {at} is not finite")):
        keep = arr[at], arr[-1]
        arr[at] = arr[-1] = x
        for call in (lambda: g.rmse(r, c, a), lambda: g.run_until(2, 1, -1.0, (r, c, a))):
            with pytest.raises(CCDPPError) as ei:
                call()
            assert ei.value.code == CCDPP_EINVAL and text in str(ei.value)
        arr[at], arr[-1] = keep
    assert g.rmse(r, c, a) == ref
    for x, y in zip((W, H), g.factors()):
        assert np.array_equal(x, y)
    g.close()


@pytest.mark.parametrize("m", [200, 32_618, 32_619, 40_000])  # (2^17 values are checked on the host)
def test_factors_that_are_not_finite_change_nothing(m):
    n, k = 150, 4
    row, col, val, H0 = synth.small_random(m, n, 3_000, k, seed=9)
    g = CCDPP(m, n, k, 0.1, row, col, val)
    g.set_factors(None, H0)
    g.run(1, 2)
    W, H = g.factors()
    R = g.residual()
    bad = W.copy()
    bad[m // 2, 1] = bad[m - 1, 0] = np.inf
    with pytest.raises(CCDPPError) as ei:
        g.set_factors(bad, H)
    assert ei.value.code == CCDPP_EINVAL and f"W[{m // 2 * k + 1}] is not finite" in str(ei.value)
    bad_h = H.copy()
    bad_h[n - 1, 2] = np.nan
    with pytest.raises(CCDPPError) as ei:
        g.set_factors(W, bad_h)
    assert f"H[{(n - 1) * k + 2}] is not finite" in str(ei.value)
    for x, y in zip((W, H, R), g.factors() + (g.residual(),)):
        assert np.array_equal(x, y)
    g.close()


@pytest.mark.parametrize("entries", [1_000, 30_000])
@pytest.mark.parametrize("outer", [0, 1])
def test_held_out_arrays_are_read_before_the_call_returns(entries, outer):
    # Pinned caller memory is copied by the DMA engine, behind the stream's work: the call
    # waits for it, also where no iteration runs, and where the first pass fails.
    import torch

    m, n, k = 700, 300, 3
    row, col, val, H0 = synth.small_random(m, n, 9_000, k, seed=8)
    g = CCDPP(m, n, k, 0.1, row, col, val)
    side = torch.cuda.Stream()
    g.set_stream(side.cuda_stream)
    rng = np.random.default_rng(entries)
    pinned = [torch.from_numpy(x).pin_memory() for x in (rng.integers(0, m, entries).astype(np.int32),
                                                         rng.integers(0, n, entries).astype(np.int32),
                                                         rng.standard_normal(entries).astype(np.float32))]
    test = tuple(x.numpy() for x in pinned)
    print(f"case: {entries} entries, {outer} iterations", flush=True)
    for fails in (False, True):
        with torch.cuda.stream(side):
            torch.cuda._sleep(50_000_000)
        if fails and outer:
            C.ccdpp_debug_inject(1, 0)
            with pytest.raises(CCDPPError):
                g.run_until(outer, 1, -1.0, test)
        else:
            g.run_until(outer, 1, -1.0, test)
        assert side.query()
    C.ccdpp_debug_inject(1, -1)
    g.close()
