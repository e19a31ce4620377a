"""The hyperparameter draw at the edges of its 32-row register tiles and 16-wide product
tiles, and its status: every input for which Lambda or its factors have no positive finite
pivots is reported.

Bar: 1e-9 relative against the fp64 oracle (both fp64; the matrices' condition numbers stay
below 1e4, so rounding gives about D * 1e4 * 2^-53 ~ 1e-10 at D = 128)."""
import numpy as np
import pytest

import oracle
import workload
from tests.test_gpu_bayes import HYPER_TOL, bartlett_variates, dev, small_matrix, spd

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def draw(als, side, X, mu0, beta0, W0inv, nu0, chi2, offd, zmu):
    als.set_nw_prior(side, mu0, beta0, W0inv, nu0)
    f = lambda a: dev(a, np.float64)
    return [t.cpu().numpy() for t in als.sample_hyper(side, dev(X), f(chi2), f(offd), f(zmu),
                                                      check=True)]


@pytest.mark.parametrize("D", [3, 15, 31, 32, 34, 63, 65, 96, 97, 127])
def test_tile_edges(D):
    from paper_1108_2580_amd import ALS

    M, N = 700, 300
    ptr, col, val = small_matrix(M, N, 3 + D, zero_users=0)
    rng = np.random.default_rng(70 + D)
    print(f"hyper edges D={D}", flush=True)
    with ALS(M, N, ptr, col, val, D) as als:
        X = rng.normal(0.2, 0.6, size=(M, D)).astype(np.float32)
        mu0, W0inv = rng.normal(0, 0.1, size=D), spd(rng, D, 0.3)
        chi2, offd, zmu = bartlett_variates(rng, D, D + 3.0 + M)
        mu_g, Lam_g = draw(als, "users", X, mu0, 2.0, W0inv, D + 3.0, chi2, offd, zmu)
    post = oracle.nw_posterior(X, mu0, 2.0, W0inv, D + 3.0)
    mu_o, Lam_o = oracle.nw_sample(post[0], post[1], post[2], chi2, offd, zmu)
    assert np.array_equal(Lam_g, Lam_g.T)
    assert np.linalg.norm(Lam_g - Lam_o) <= HYPER_TOL * np.linalg.norm(Lam_o)
    assert np.linalg.norm(mu_g - mu_o) <= HYPER_TOL * np.linalg.norm(mu_o)


@pytest.mark.parametrize("what", ["chi2_zero", "chi2_nan", "chi2_inf", "offdiag_nan", "indefinite",
                                  "x_nan"])
@pytest.mark.parametrize("D", [3, 40])
def test_failures_are_reported(D, what):
    from paper_1108_2580_amd import ALS, ALSError, ALS_ERR_NOT_SPD

    M, N = 50, 40
    ptr, col, val = small_matrix(M, N, 3 + D, zero_users=0)
    rng = np.random.default_rng(D)
    X = rng.normal(size=(M, D)).astype(np.float32)
    W0inv = np.eye(D)
    chi2, offd, zmu = bartlett_variates(rng, D, D + 3.0 + M)
    if what == "offdiag_nan":
        offd[D - 2] = np.nan
    elif what == "indefinite":
        W0inv[D // 2, D // 2] = -1e6
    elif what == "x_nan":
        X[7, D - 1] = np.nan
    else:
        chi2[D // 2] = {"chi2_zero": 0.0, "chi2_nan": np.nan, "chi2_inf": np.inf}[what]
    print(f"hyper failure {what} D={D}", flush=True)
    with ALS(M, N, ptr, col, val, D) as als:
        with pytest.raises(ALSError) as e:
            draw(als, "users", X, np.zeros(D), 2.0, W0inv, D + 3.0, chi2, offd, zmu)
        assert e.value.status == ALS_ERR_NOT_SPD
