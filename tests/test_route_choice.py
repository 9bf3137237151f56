"""Which images that the one kernel after the statistics does not take (tdq_whole_extra) go by the radix levels because
their sets are many and small, or have more tokens to look at than elements; the rule itself needs no GPU."""
import numpy as np
import pytest

from paper_2604_16855_amd import tdq

import parity_util as U

DTYPES = [tdq.TDQ_F16, tdq.TDQ_F32]


def _samples(dt, B, T, C, G):
    return bool(tdq.lib().tdq_samples_rank(dt, B, T, C, G))


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("B,T,C,G,sampled", [
    (256, 64, 512, 8, True), (257, 64, 512, 8, False), (257, 64, 513, 8, True),      # 2048 sets
    (64, 49, 2, 32, True), (65, 49, 2, 32, False), (65, 128, 1025, 32, True),
    (1024, 9, 24, 4, True), (1025, 9, 24, 4, False), (1025, 64, 257, 4, True),       # 4096 sets
    (64, 196, 384, 64, True), (65, 196, 384, 64, False),
    (33, 15888, 16, 16, False), (33, 15887, 16, 16, True), (33, 15888, 17, 16, True),  # 2^23 looks
    (32, 32768, 16, 16, True), (8, 1024, 768, 16, True), (2048, 1024, 64, 8, True),
])
def test_rule(dt, B, T, C, G, sampled):
    assert _samples(dt, B, T, C, G) == sampled


def test_a_type_alone():
    """The binary32 limits bind no binary16 image; more than 64 sets take the levels always."""
    for s in ((1, 1024, 1024, 16), (1, 624, 1024, 64), (1, 32769, 9, 1)):
        assert _samples(tdq.TDQ_F16, *s) and not _samples(tdq.TDQ_F32, *s)
    for dt in DTYPES:
        assert not _samples(dt, 1, 100, 64, 65)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("B,T,C,G", [(1025, 9, 24, 4), (257, 20, 33, 8), (66, 49, 2, 64), (33, 15888, 9, 16)])
def test_levels_of_many_sets(B, T, C, G, dtype):
    dt = tdq.TDQ_F16 if dtype is np.float16 else tdq.TDQ_F32
    assert not _samples(dt, B, T, C, G)
    rng = np.random.default_rng(B + T)
    X = (rng.laplace(0, 1, (B, T, C)) * np.exp(rng.normal(0, 0.7, (B, T, 1)))).astype(dtype)
    for pct in (0.0, 0.99):
        p = tdq.default_params(G)
        p.base_pct = pct
        g = U.gpu_calibrate(X, p)
        assert g["status"] == 0 and g["exact_sets"] == 0
        U.assert_calibration_matches(g, X, p)


@pytest.mark.gpu
def test_switch_searches_whatever_the_route():
    """The validation switch searches every set of a binary16 image whose sets would take the levels."""
    rng = np.random.default_rng(3)
    X = rng.laplace(0, 1, (257, 20, 33)).astype(np.float16)
    p = tdq.default_params(8)
    p.flags |= tdq.FLAG_EXACT_SELECT
    g = U.gpu_calibrate(X, p)
    assert g["exact_sets"] > 0
    U.assert_calibration_matches(g, X, p)
