"""Outputs of the contraction's tiles that an edge of Y cuts: wavefronts wholly inside, cut in rows, in columns or both,
and wholly outside, with rows of Y longer than its columns so that a store past them shows."""
import numpy as np
import pytest
import torch

from paper_2604_16855_amd import inputs as I
from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("with_bias", [False, True])
@pytest.mark.parametrize("M,K,N", [
    (1, 64, 1), (31, 64, 33), (33, 96, 63), (64, 32, 65), (95, 160, 129), (129, 64, 190),          # 64 x 64 tiles
    (7700, 64, 1250), (100000, 96, 70), (98337, 64, 321),                                         # 64 x 128
    (7713, 100, 1281), (7745, 33, 1313), (98400, 64, 63), (17000, 300, 1055),                     # 128 x 64
    (16990, 260, 1121), (16897, 256, 1100)])                                                      # 128 x 128
def test_cut_tiles(M, K, N, with_bias, out_dtype):
    _check(M, K, N, with_bias, out_dtype, 5)


@pytest.mark.parametrize("M,K,N,pad,out_dtype", [
    (83220, 40, 63, 2, torch.float32), (83221, 40, 63, 2, torch.float32), (83221, 40, 63, 1, torch.float32),
    (62914, 64, 100, 3, torch.float32), (62915, 64, 100, 3, torch.float32), (41943, 130, 300, 1, torch.float32),
    (41944, 130, 300, 1, torch.float32), (41944, 520, 321, 7, torch.float32), (41001, 96, 1223, 2, torch.float32),
    (233016, 33, 45, 0, torch.float16), (233017, 33, 45, 0, torch.float16), (125830, 96, 100, 0, torch.float16),
    (83887, 200, 301, 2, torch.float16), (41001, 96, 1223, 2, torch.float16)])
def test_stores_by_the_rule(M, K, N, pad, out_dtype):
    """Either side of the amounts of output (20, 24 and 48 MiB with less than 64, less than 128 and more columns) from
    which cut tiles store as usual at rows between 64-byte boundaries, and rows on such boundaries."""
    _check(M, K, N, True, out_dtype, pad)


@pytest.mark.parametrize("M,K,N,out_dtype", [(291908, 108, 63, torch.float32), (398437, 136, 59, torch.float32),
                                             (300000, 64, 61, torch.float16)])
def test_cut_tiles_of_many_rows(M, K, N, out_dtype):
    """A cut tile must cost little more than the whole one that it is part of: 1.09 to 1.43 times measured, 2.2 to 2.8 while
    all its stores went past the caches."""
    from test_gpu_block_outputs import _time
    d, us = U.dev(), {}
    for n in (N, 64):
        Q, Qw = (torch.randint(0, 256, (rows, tdq.packed_row_bytes(K)), dtype=torch.uint8, device=d) for rows in (M, n))
        scale, sw, Y = torch.rand((1, 1), device=d), torch.rand(n, device=d), torch.empty((M, n), dtype=out_dtype, device=d)
        us[n] = 1e3 * _time(lambda: tdq.tdq_w4a4_linear(Q, None, scale, 1, M, K, Qw, sw, out=Y))
    print({n: f"{t:.1f} us" for n, t in us.items()}, flush=True)
    assert us[N] <= 1.8 * us[64]


def _check(M, K, N, with_bias, out_dtype, pad):
    d = U.dev()
    qx, qw = I.random_codes((M, K), 3), I.random_codes((N, K), 4)
    rng = np.random.default_rng(M + N)
    scale = rng.uniform(0.5, 2.0, (1, 3)).astype(np.float32)
    gid = rng.integers(0, 3, (1, M)).astype(np.int32)
    ws = rng.uniform(0.01, 0.02, N).astype(np.float32)
    bias = rng.normal(0, 1, N).astype(np.float32) if with_bias else None
    buf = torch.full((M, N + pad), 77.0, dtype=out_dtype, device=d)
    t = lambda a: torch.from_numpy(a).to(d)
    tdq.tdq_w4a4_linear(U.pack_to_device(qx), t(gid), t(scale), 1, M, K, U.pack_to_device(qw), t(ws),
                        bias=None if bias is None else t(bias), out=buf[:, :N])
    torch.cuda.synchronize()
    acc = (t(qx.astype(np.float32)) @ t(qw.astype(np.float32)).t())                    # sums below 2^24: exact
    want = (acc * t(scale[0][gid[0]])[:, None]) * t(ws)
    if bias is not None:
        want = want + t(bias)
    assert torch.equal(buf[:, :N], want.to(out_dtype))
    assert bool((buf[:, N:] == 77.0).all())
