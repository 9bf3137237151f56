"""The two-sweep rank select of binary32 input against the oracle, where it can go wrong: ties
(all values of a set equal, a fifth of them zero, few distinct values), values close together
far from zero (the interval is narrow), heavy tails, sets smaller than the sample, several
batches of tokens, ties and other values in one bin, rows at element alignment,
the percentile base radius, 33 to 64 sets (256 bins), and the largest images of the route next
to the smallest ones past it."""
import numpy as np
import pytest

from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _data(kind, B, T, C, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    X = rng.laplace(0, 1, (B, T, C)) * rng.lognormal(0, 1.0, (B, T, 1))
    if kind == "equal":
        X[:] = 0.75
    elif kind == "relu":
        X = np.maximum(X, 0.0)
    elif kind == "levels":                       # 15 distinct magnitudes: every bin is all ties
        X = np.round(X * 7 / np.abs(X).max(axis=2, keepdims=True)) * np.float32(0.1)
    elif kind == "two":                          # the rank lies among ties next to other values
        X = np.where(rng.random((B, T, C)) < 0.3, 0.5, 0.5 + rng.random((B, T, C)) * 1e-4)
    elif kind == "offset":
        X = 250.0 + 0.25 * rng.normal(0, 1, (B, T, C))
    elif kind == "tails":
        X = 20.0 * rng.standard_t(2.0, (B, T, C))
    return X.astype(np.float32)


@pytest.mark.parametrize("kind", ["laplace", "equal", "relu", "levels", "two", "offset", "tails"])
@pytest.mark.parametrize("T,C,G", [(70, 40, 3), (1100, 257, 12), (4500, 130, 33), (300, 2052, 64)])
def test_two_sweep_select(kind, T, C, G):
    X = _data(kind, 2, T, C, T + C)
    p = tdq.default_params(G)
    for pct, pad, zr in ((0.0, 0, 0.2), (0.99, 1, 0.05)):
        p.base_pct, p.zr = pct, zr
        g = U.gpu_calibrate(X, p, ld_pad=pad)
        assert g["status"] == 0
        U.assert_calibration_matches(g, X, p)


def test_interval_holds_the_rank():
    """On ordinary data no set may need the fallback (it costs time, not accuracy)."""
    X = _data("laplace", 4, 1024, 768, 5)
    g = U.gpu_calibrate(X, tdq.default_params(16))
    U.assert_calibration_matches(g, X, tdq.default_params(16))
    assert g["exact_sets"] == 0


@pytest.mark.parametrize("B,T,C,G,sampled", [
    (1, 1023, 1024, 16, True), (1, 1024, 1024, 16, False),       # 1 Mi elements
    (1, 1023, 1024, 4, True), (1, 1024, 1024, 4, False),
    (1, 623, 1024, 64, True), (1, 624, 1024, 64, False),         # shorter lists
    (1, 32768, 9, 1, True), (1, 32769, 9, 1, False),             # many tokens, few sets
    (1, 49152, 5, 3, True), (1, 49153, 5, 3, False),
    (64, 30, 35, 32, True), (65, 30, 35, 32, False),             # many small sets
])
def test_limits_of_the_route(B, T, C, G, sampled):
    """The largest images of the sampled route and the smallest past it."""
    assert bool(tdq.lib().tdq_samples_rank(tdq.TDQ_F32, B, T, C, G)) == sampled
    X = _data("laplace", B, T, C, T + G)
    p = tdq.default_params(G)
    g = U.gpu_calibrate(X, p)
    U.assert_calibration_matches(g, X, p)
    assert g["exact_sets"] == 0


@pytest.mark.parametrize("T", [2912, 2913])
def test_images_of_three_million_elements(T):
    """Radix levels."""
    X = _data("laplace", 1, T, 1024, T)
    p = tdq.default_params(4)
    U.assert_calibration_matches(U.gpu_calibrate(X, p), X, p)
