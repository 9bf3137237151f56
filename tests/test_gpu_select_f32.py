"""The two-sweep rank select of binary32 input (the chain of kernels, which images take that the one kernel after the
statistics does not) against the oracle, where it can go wrong: ties
(all values of a set equal, a fifth of them zero, few distinct values), values close together
far from zero (the interval is narrow), heavy tails, sets smaller than the sample, several
batches of tokens, ties and other values in one bin, rows at element alignment,
the percentile base radius, 33 to 64 sets (256 bins), and the largest images of the route next
to the smallest ones past it.  Some of the shapes take the one kernel, and say so."""
import numpy as np
import pytest

from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _whole(B, T, C, G, pct=0.0):
    """Whether the one kernel after the statistics does it all."""
    return tdq.lib().tdq_whole_extra(tdq.TDQ_F32, B, T, C, G, tdq.C.c_double(pct)) >= 0


def _two_sweeps(B, T, C, G, pct=0.0):
    """Whether the chain of kernels that samples does."""
    return not _whole(B, T, C, G, pct) and bool(tdq.lib().tdq_samples_rank(tdq.TDQ_F32, B, T, C, G))


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
@pytest.mark.parametrize("T,C,G,chain", [
    (70, 40, 3, ""), (1100, 257, 12, "percentile"), (4500, 130, 33, "both"), (300, 2052, 64, "both"),
    (8193, 33, 3, "both"), (8200, 77, 12, "both"), (300, 1100, 1, "both")])
def test_two_sweep_select(kind, T, C, G, chain):
    """chain: which of the two calls take it."""
    X = _data(kind, 2, T, C, T + C)
    p = tdq.default_params(G)
    for pct, pad, zr in ((0.0, 0, 0.2), (0.99, 1, 0.05)):
        assert _two_sweeps(2, T, C, G, pct) == (chain == "both" or (chain == "percentile" and pct > 0))
        p.base_pct, p.zr = pct, zr
        g = U.gpu_calibrate(X, p, ld_pad=pad)
        assert g["status"] == 0
        U.assert_calibration_matches(g, X, p)


@pytest.mark.parametrize("T,C,G,whole", [(1024, 768, 16, True), (8300, 96, 16, False), (800, 768, 40, False)])
def test_interval_holds_the_rank(T, C, G, whole):
    """On ordinary data no set may need the fallback (it costs time, not accuracy)."""
    assert _whole(4, T, C, G) == whole and _two_sweeps(4, T, C, G) != whole
    X = _data("laplace", 4, T, C, 5)
    g = U.gpu_calibrate(X, tdq.default_params(G))
    U.assert_calibration_matches(g, X, tdq.default_params(G))
    assert g["exact_sets"] == 0


@pytest.mark.parametrize("B,T,C,G,sampled", [
    (1, 16383, 64, 16, True), (1, 16384, 64, 16, False),         # 1 Mi elements
    (1, 16383, 64, 4, True), (1, 16384, 64, 4, False),
    (1, 1024, 1023, 1, True), (1, 1024, 1024, 1, False),
    (1, 623, 1024, 64, True), (1, 624, 1024, 64, False),         # shorter lists
    (1, 32768, 9, 1, True), (1, 32769, 9, 1, False),             # many tokens, few sets
    (1, 49152, 5, 3, True), (1, 49153, 5, 3, False),
    (64, 30, 35, 32, True), (65, 30, 35, 32, False),             # many small sets
])
def test_limits_of_the_route(B, T, C, G, sampled):
    """The largest images of the sampled chain and the smallest past it, which take the radix levels."""
    assert not _whole(B, T, C, G) and _two_sweeps(B, T, C, G) == sampled
    X = _data("laplace", B, T, C, T + G)
    p = tdq.default_params(G)
    g = U.gpu_calibrate(X, p)
    U.assert_calibration_matches(g, X, p)
    assert g["exact_sets"] == 0


@pytest.mark.parametrize("G", [4, 16])
@pytest.mark.parametrize("T", [1023, 1024])
def test_a_million_elements_in_one_kernel(T, G):
    """The limits of the chain are not those of the one kernel."""
    assert _whole(1, T, 1024, G)
    X = _data("laplace", 1, T, 1024, T + G)
    p = tdq.default_params(G)
    g = U.gpu_calibrate(X, p)
    U.assert_calibration_matches(g, X, p)
    assert g["exact_sets"] == 0


@pytest.mark.parametrize("T,C,G,whole", [(2912, 1024, 4, True), (2913, 1024, 4, True), (2912, 1024, 33, False),
                                         (2913, 1024, 33, False), (8200, 364, 4, False)])
def test_images_of_three_million_elements(T, C, G, whole):
    """By one kernel, and by the radix levels."""
    assert _whole(1, T, C, G) == whole and not tdq.lib().tdq_samples_rank(tdq.TDQ_F32, 1, T, C, G)
    X = _data("laplace", 1, T, C, T)
    p = tdq.default_params(G)
    U.assert_calibration_matches(U.gpu_calibrate(X, p), X, p)
