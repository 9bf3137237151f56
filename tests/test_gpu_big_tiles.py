"""The 256 x 256 contraction kernels where their tiles are not whole, or their stages are few, odd
and even in number: the bounds-checked output of the last row and column of tiles next to the fast
one of the others, bias, padded leading dimensions, the accumulator dump.  Bit for bit against the
oracle on sampled rows."""
import numpy as np
import pytest
import torch

from oracle import tdq_oracle as O
from paper_2604_16855_amd import inputs as I

from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,M,K,N,out_dtype,with_bias,pad,dump", [
    ("pipe", 16384, 640, 4096, torch.float16, True, 0, False),      # whole tiles, 5 stages
    ("pipe", 20000, 1152, 4096, torch.float32, False, 0, False),    # ragged rows, 9 stages
    ("pipe", 16383, 1408, 2047, torch.float32, True, 3, False),     # ragged rows and columns, 11 stages
    ("pipe", 16383, 1408, 2047, torch.float16, False, 0, True),
    ("wide", 8192, 1024, 4096, torch.float32, True, 4, False),      # whole tiles, 4 stages
    ("wide", 16383, 1280, 4095, torch.float16, True, 1, False),     # ragged rows and columns, 5 stages
    ("wide", 16383, 1280, 4095, torch.float32, False, 0, False),
    ("wide", 8191, 2048, 4095, torch.float32, True, 0, True),       # 8 stages
    ("wide", 32767, 2304, 1000, torch.float16, False, 0, False),    # 9 stages, 3.9 columns of tiles
])
def test_big_tile_edges(kernel, M, K, N, out_dtype, with_bias, pad, dump):
    assert U.linear_kernel(M, K, N) == kernel
    qx, qw = I.random_codes((M, K), M + K), I.random_codes((N, K), N + 3 * K)
    rng = np.random.default_rng(M * N)
    G = 6
    gid = rng.integers(0, G, (1, M)).astype(np.int32)
    scale = rng.uniform(0.01, 3.0, (1, G)).astype(np.float32)
    sw = rng.uniform(0.001, 0.1, N).astype(np.float32)
    bias = rng.normal(0, 0.5, N).astype(np.float32) if with_bias else None
    d = [None if a is None else torch.from_numpy(a).to(U.dev()) for a in (gid, scale, sw, bias)]
    buf = torch.full((M, N + pad), -77.0, dtype=out_dtype, device=U.dev())
    acc = torch.empty((M, N), dtype=torch.int32, device=U.dev()) if dump else None
    Y = tdq.tdq_w4a4_linear(U.pack_to_device(qx), d[0], d[1], 1, M, K, U.pack_to_device(qw), d[2], d[3],
                            out_dtype, out=buf[:, :N], acc_dump=acc)
    torch.cuda.synchronize()
    if pad:
        assert (buf[:, N:] == -77.0).all(), "wrote past the row end"
    rows = np.unique(np.concatenate([np.arange(3), np.arange(254, 258), rng.integers(0, M, 150),
                                     np.arange(M - 300, M)[::5], [M - 1]]))
    acc_ref, Y_ref = O.w4a4_linear(qx[rows], scale[0, gid[0, rows]], qw, sw, bias)
    at = torch.from_numpy(rows).to(U.dev())
    if out_dtype == torch.float16:
        Y_ref = Y_ref.astype(np.float16)
    assert np.array_equal(Y[at].cpu().numpy(), Y_ref)
    if dump:
        assert np.array_equal(acc[at].cpu().numpy(), acc_ref)
