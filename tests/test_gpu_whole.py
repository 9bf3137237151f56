"""Calibration by one kernel after the statistics: which images take it (CPU), and its results against the
oracle and the route that searches every set, at the edges of its rounds of keys, rows of odd length, one and
several workgroups per set, one and two ranks."""
import numpy as np
import pytest

from paper_2604_16855_amd import tdq

import parity_util as U


def _extra(dt, B, T, C, G, pct=0.0):
    return tdq.lib().tdq_whole_extra(dt, B, T, C, G, tdq.C.c_double(pct))


@pytest.mark.parametrize("dt,B,T,C,G,pct,extra", [
    (tdq.TDQ_F16, 8, 121, 512, 16, 0.0, 7), (tdq.TDQ_F16, 1, 7744, 64, 16, 0.0, 60),
    (tdq.TDQ_F16, 1, 8192, 8, 16, 0.0, 8), (tdq.TDQ_F16, 1, 8193, 8, 16, 0.0, -1),
    (tdq.TDQ_F16, 32, 1024, 512, 15, 0.0, -1), (tdq.TDQ_F16, 32, 80, 1024, 15, 0.0, 1),   # 512 groups
    (tdq.TDQ_F16, 32, 81, 1024, 15, 0.0, -1), (tdq.TDQ_F16, 64, 40, 1024, 16, 0.0, 0),
    (tdq.TDQ_F16, 32, 128, 1024, 15, 0.99, 1), (tdq.TDQ_F16, 32, 129, 1024, 15, 0.99, -1),
    (tdq.TDQ_F32, 64, 20, 64, 16, 0.0, 0), (tdq.TDQ_F32, 65, 20, 64, 16, 0.0, -1),
    (tdq.TDQ_F32, 32, 20, 64, 16, 0.99, 0), (tdq.TDQ_F32, 33, 20, 64, 16, 0.99, -1),
    (tdq.TDQ_F16, 1, 512, 64, 17, 0.99, -1), (tdq.TDQ_F16, 1, 512, 64, 16, 0.99, 4),       # words for two ranks
    (tdq.TDQ_F16, 96, 50, 32, 16, 0.0, 0), (tdq.TDQ_F16, 97, 50, 32, 16, 0.0, -1),          # 1536 sets
    (tdq.TDQ_F16, 1, 127, 64, 17, 0.99, 0), (tdq.TDQ_F16, 1, 100, 64, 65, 0.0, -1),
    (tdq.TDQ_F32, 2, 896, 64, 8, 0.0, 0), (tdq.TDQ_F32, 2, 897, 64, 8, 0.99, -1),
    (tdq.TDQ_F32, 2, 640, 64, 1, 0.0, 0), (tdq.TDQ_F32, 2, 641, 64, 1, 0.0, -1),
    (tdq.TDQ_F16, 1, 4095, 128, 1, 0.0, 63), (tdq.TDQ_F16, 1, 4096, 128, 1, 0.0, -1),      # many share a set
    (tdq.TDQ_F16, 1, 4096, 128, 2, 0.0, 64), (tdq.TDQ_F16, 3, 2125, 1669, 1, 0.99, 169),
    (tdq.TDQ_F16, 16, 58, 5470, 4, 0.0, 28), (tdq.TDQ_F16, 16, 57, 5470, 4, 0.0, -1),      # few rows for each
    (tdq.TDQ_F16, 16, 57, 5470, 4, 0.99, 28), (tdq.TDQ_F16, 1, 57, 5470, 4, 0.0, 38),
    (tdq.TDQ_F16, 58, 6152, 21, 1, 0.0, 7), (tdq.TDQ_F16, 58, 6152, 22, 1, 0.0, -1),       # many tokens in one set
    (tdq.TDQ_F16, 58, 4096, 44, 1, 0.0, 7), (tdq.TDQ_F16, 58, 6152, 44, 1, 0.99, 7),
    (tdq.TDQ_F16, 11, 1000, 1500, 15, 0.0, 31), (tdq.TDQ_F16, 11, 1000, 1500, 16, 0.0, -1),  # three to a set, fewer
    (tdq.TDQ_F16, 11, 1024, 1240, 16, 0.0, 30), (tdq.TDQ_F16, 11, 1024, 1241, 16, 0.0, -1),
    (tdq.TDQ_F16, 8, 7840, 512, 16, 0.0, 48), (tdq.TDQ_F16, 8, 7841, 512, 16, 0.0, -1),
    (tdq.TDQ_F16, 27, 2800, 79, 16, 0.0, -1), (tdq.TDQ_F16, 27, 166, 1095, 16, 0.0, -1),
])
def test_rule(dt, B, T, C, G, pct, extra):
    assert _extra(dt, B, T, C, G, pct) == extra


def test_groups_fit():
    """Never more than 512 workgroups, or one per set if there are more sets."""
    rng = np.random.default_rng(5)
    for _ in range(2000):
        B, T, C = (int(np.exp(rng.uniform(0, np.log(m)))) for m in (600, 9000, 5000))
        G = int(rng.integers(1, 65))
        e = _extra(tdq.TDQ_F16, B, T, C, G, float(rng.choice([0.0, 0.99])))
        assert e == -1 or B * (G + e) <= max(512, B * G)


def _data(kind, B, T, C, dtype, seed):
    rng = np.random.default_rng(seed)
    x = rng.laplace(0, 1, (B, T, C)) * np.exp(rng.normal(0, 0.8, (B, T, 1)))
    if kind == "relu":
        x = np.maximum(x, 0)
    elif kind == "pad":                              # tokens of zeros, one set of identical values
        x[:, ::3] = 0
    elif kind == "few":                              # a dozen values
        x = 0.5 * np.round(rng.normal(0, 3, (B, T, C)))
    elif kind == "near":                             # binary16: up to three values
        x = 1 + 1e-4 * rng.normal(0, 1, (B, T, C))
    elif kind == "one":                              # all tokens in one set
        x[:, :, 0] = 9.0
        x = np.clip(x, -9, 9)
    return x.astype(dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("pct", [0.0, 0.99])
@pytest.mark.parametrize("kind", ["lap", "relu", "pad", "few", "near", "one"])
@pytest.mark.parametrize("dtype,B,T,C,G,pad", [
    (np.float16, 2, 1, 1, 1, 0), (np.float16, 3, 511, 24, 16, 0), (np.float16, 2, 513, 33, 5, 2),
    (np.float16, 2, 1025, 17, 16, 1), (np.float16, 1, 2049, 56, 12, 0), (np.float16, 1, 4097, 40, 8, 0),
    (np.float16, 1, 8192, 9, 3, 0), (np.float16, 5, 70, 1031, 64, 0), (np.float16, 2, 300, 520, 16, 3), (np.float16, 49, 30, 40, 24, 0),
    (np.float32, 2, 1, 3, 2, 0), (np.float32, 2, 512, 66, 16, 0), (np.float32, 1, 1025, 37, 8, 3),
    (np.float32, 1, 8192, 7, 5, 0), (np.float32, 3, 20, 2049, 64, 0),
])
def test_against_oracle(dtype, B, T, C, G, pad, kind, pct):
    dt = tdq.TDQ_F16 if dtype is np.float16 else tdq.TDQ_F32
    X = _data(kind, B, T, C, dtype, T + C)
    p = tdq.default_params(G)
    p.base_pct = pct
    if not (pct and G > 16 and _extra(dt, B, T, C, G) > 0):
        assert _extra(dt, B, T, C, G, pct) >= 0
    g = U.gpu_calibrate(X, p, ld_pad=pad)
    assert g["status"] == 0
    U.assert_calibration_matches(g, X, p)
    p.flags |= tdq.FLAG_EXACT_SELECT                 # the general route
    h = U.gpu_calibrate(X, p, ld_pad=pad)
    assert np.array_equal(g["gid"], h["gid"]) and np.array_equal(g["stats"]["thr"], h["stats"]["thr"])
    assert np.array_equal(g["stats"]["c_base"], h["stats"]["c_base"])
    assert np.allclose(g["scale"], h["scale"], rtol=2e-7, atol=0)        # sigma: sums in another order


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,C,G", [(19, 167, 2056, 12), (2, 2231, 2752, 32), (42, 863, 29, 15),
                                     (51, 2213, 103, 4)])
def test_few_values_cost_little_more(B, T, C, G):
    """Keys that all meet in a few words of LDS: at most twice the time of ordinary data (1.1 to 1.5 times
    measured, 2 to 3.5 times where every addition went to one word)."""
    import torch

    from test_gpu_block_outputs import _time
    assert _extra(tdq.TDQ_F16, B, T, C, G) >= 0
    ms = {}
    for kind in ("lap", "near"):
        X = torch.from_numpy(_data(kind, B, T, C, np.float16, 2)).to(U.dev())
        p = tdq.default_params(G)
        ws = tdq.alloc_workspace(B, T, C, tdq.TDQ_F16, p, X.device)
        out = (torch.empty((B, T), dtype=torch.int32, device=X.device),
               *(torch.empty((B, G), device=X.device) for _ in range(2)))
        ms[kind] = _time(lambda: tdq.tdq_calibrate_groups(X, p, ws, out=out))
    print({k: f"{1e3 * t:.1f} us" for k, t in ms.items()}, flush=True)
    assert ms["near"] <= 2.0 * ms["lap"]


@pytest.mark.gpu
def test_status_is_this_calls():
    """The status area is cleared by each call, and one image that is not finite raises it."""
    import torch
    X = torch.from_numpy(_data("lap", 4, 300, 64, np.float16, 1)).cuda()
    p = tdq.default_params(8)
    ws = tdq.alloc_workspace(4, 300, 64, tdq.TDQ_F16, p, X.device)
    ws.fill_(255)
    Y = X.clone()
    Y[2, 7, 5] = float("inf")
    for x, want in ((X, 0), (Y, 1), (X, 0)):
        tdq.tdq_calibrate_groups(x, p, ws)
        torch.cuda.synchronize()
        assert tdq.device_status(ws) == want and (want or tdq.exact_select_sets(ws) == 0)
