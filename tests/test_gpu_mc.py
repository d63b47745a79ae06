"""GPU parity of the App. B Monte-Carlo calibration: every simulated estimate
equals the oracle's (same counter-based generator, exact integer sums), and
the moments agree."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
sk = pytest.importorskip("paper_1808_10365_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,sigma,est", [(16, 256, 2.5, 1), (300, 64, 1.52, 0), (5, 1000, 3.5, 1)])
def test_mc_values_match_oracle(N, M, sigma, est):
    n_sim = 300
    m, vals = sk.calibrate_mc(N, M, sigma, n_sim, seed=19, estimator=est, return_values=True)
    g = vals.cpu().numpy()
    r = oracle.mc_calibrate(N, M, sigma, n_sim, seed=19, est=est)
    assert np.all(np.abs(g - r) <= 1e-12 * np.maximum(1.0, np.abs(r)))
    assert abs(m[0] - r.mean()) < 1e-12 and abs(m[1] / r.var(ddof=1) - 1) < 1e-9


def test_mc_large_run_moments():
    # CHIME-like: N = 2048 receivers, n = 256, RMS 1.52 counts (App. B).
    m = sk.calibrate_mc(2048, 256, 1.52, 2000, seed=3)
    K = 2048 * 256
    assert abs(m[0] - 1.0) < 0.01
    assert abs(m[1] / (4 / K) - 1) < 0.15


@pytest.mark.parametrize("N,M,sigma,n_sim,est", [
    (1, 2, 2.0, 1, 0),            # one lane, one estimate
    (1, 64, 0.3, 3000, 1),        # several thresholds in one bucket of the inverse-CDF table; 64 estimates a group
    (17, 33, 1.3, 4099, 1),       # pairs that do not fill the lanes, a short last group
    (2, 131, 3.0, 37, 0),         # few lanes: an input's samples split over lanes, a ragged last segment
    (256, 16, 2.0, 5, 1), (257, 17, 2.0, 5, 1),   # one and two inputs per summing lane
    (512, 16, 2.0, 3, 0), (513, 16, 2.0, 3, 0), (1300, 40, 1.52, 9, 1),   # one and several slabs of inputs
])
def test_mc_split_edges(N, M, sigma, n_sim, est):
    # The split over groups, slabs and segments leaves every estimate what the
    # oracle's plain loop gives: integer sums, then one FP64 sum over inputs
    # (error below N 2^-53 relative; 1e-12 covers N = 1300).
    print(f"case N={N} M={M} sigma={sigma} n_sim={n_sim}", flush=True)
    m, vals = sk.calibrate_mc(N, M, sigma, n_sim, seed=23, estimator=est, return_values=True)
    g = vals.cpu().numpy()
    r = oracle.mc_calibrate(N, M, sigma, n_sim, seed=23, est=est)
    assert np.array_equal(np.isnan(g), np.isnan(r))
    ok = ~np.isnan(r)
    assert np.all(np.abs(g[ok] - r[ok]) <= 1e-12 * np.maximum(1.0, np.abs(r[ok])))
    if ok.sum() > 1:
        assert abs(m[0] - r[ok].mean()) < 1e-12 and abs(m[1] / r[ok].var(ddof=1) - 1) < 1e-9
