"""The tuner's estimate of the series' error against the oracle's Fourier coefficients, over forced
and searched parameters."""
import math

import numpy as np
import pytest

from oracle import fastsum as F
from paper_2208_03120_amd import mot

POINTS = 97  # test points of the estimate over [0, diameter]


def series_error(d, M, eta, tau, eps_B, p, diag):
    kh = F.kappa_hat(1, M, eta, tau, eps_B, p)  # k = -M .. M - 1
    r = diag * np.arange(POINTS) / (POINTS - 1)
    s = np.cos(np.pi * np.outer(r, np.arange(-M, M)) / tau) @ kh
    return d * np.abs(s - np.exp(-r * r / eta)).max()


def window_error(m, sigma):
    a = 1.0 - 1.0 / sigma
    return 4 * math.pi * (math.sqrt(m) + m) * a ** 0.25 * math.exp(-2 * math.pi * m * math.sqrt(a))


@pytest.mark.parametrize("d,eta,half,kw", [
    (1, 0.1, 0.25, {}), (2, 0.05, 0.25, {}), (3, 0.3, 0.5, {}), (2, 5e-3, 0.25, {}),
    (2, 0.05, 0.25, {"M": 12}),   # a forced M is not given up however large its error
    (1, 0.02, 0.25, {"p": 5, "eps_B": 0.2}), (2, 0.1, 0.25, {"tau": 1.25, "M": 16, "n": 64, "m": 4}),
])
def test_estimate_matches_the_series(d, eta, half, kw):
    fs = mot.fastsum_params(**kw) if kw else None
    r = mot.tune_resolve(d, eta, 1000, half, fs)
    args = (eta, r["tau"], r["eps_B"], r["p"], 2 * half * math.sqrt(d))
    want = series_error(d, r["M"], *args) + window_error(r["m"], r["n"] / (2.0 * r["M"]))
    # both sides solve for the boundary polynomial and sum 2 M terms of size 1 in FP64
    assert abs(r["est_err"] - want) < 1e-11
    if "M" not in kw:  # no shorter series of the tuner's list reaches half the target
        shorter = [M for M in (4, 6, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 112) if M < r["M"]]
        assert all(series_error(d, M, *args) > 0.5 * r["target_rel_err"] for M in shorter)
