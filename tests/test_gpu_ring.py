"""The ring contraction (tiles of 64 and 128) and the choice among tile sizes, at the edges of
both: one to many K stages and every kind of K tail (odd K, a tail of one code, a tail inside
the first 16-byte piece, whole pieces past the end of the rows), last tiles of one row or one
column, junk bytes past the rows' codes, rows strides wider than the codes -- accumulators and
outputs bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tdq_oracle as O
from paper_2604_16855_amd import inputs as I
from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _packed(codes, extra):
    """Device codes [R, ld] with junk in every byte past ceil(K / 2)."""
    R, K = codes.shape
    ld = tdq.packed_row_bytes(K) + extra
    buf = np.random.default_rng(K).integers(0, 256, (R, ld), dtype=np.uint8)
    pk = O.pack_nibbles(codes)
    buf[:, :pk.shape[1]] = pk
    return torch.from_numpy(buf).to(U.dev())


CASES = [(kernel, *c) for kernel, cases in {
    "64x64": [(1, 1, 1, 0), (63, 31, 65, 0), (65, 33, 64, 16), (64, 127, 63, 0), (129, 128, 129, 32),
              (200, 129, 72, 0), (130, 255, 250, 0), (257, 384, 40, 16), (100, 385, 130, 0), (70, 511, 90, 0),
              (66, 513, 70, 48), (90, 1025, 66, 0), (49999, 64, 60, 0)],
    "64x128": [(2000, 320, 2010, 0), (4100, 97, 1024, 0), (25000, 161, 321, 0), (8197, 289, 1021, 16),
               (8193, 1025, 1024, 0)],
    "128x64": [(16380, 256, 520, 0), (60000, 161, 190, 0), (50000, 33, 190, 16), (100001, 97, 33, 0),
               (60001, 511, 190, 0)],
    "128x128": [(8192, 289, 1021, 16), (8191, 513, 1021, 0), (8192, 385, 1024, 0), (30001, 641, 250, 48)],
    "staged": [(8200, 2049, 1000, 0)],                          # long K
}.items() for c in cases]


@pytest.mark.parametrize("kernel,M,K,N,extra", CASES)
def test_ring_tiles_and_tails(kernel, M, K, N, extra):
    assert U.linear_kernel(M, K, N) == kernel
    qx, qw = I.random_codes((M, K), M + K), I.random_codes((N, K), N + 3 * K)
    rng = np.random.default_rng(M * N)
    G = 5
    gid = rng.integers(0, G, (1, M)).astype(np.int32)
    scale = rng.uniform(0.01, 3.0, (1, G)).astype(np.float32)
    sw, bias = (rng.uniform(0.001, 0.1, N).astype(np.float32) for _ in range(2))
    d = [torch.from_numpy(a).to(U.dev()) for a in (gid, scale, sw, bias)]
    rows = np.unique(np.concatenate([np.arange(min(M, 3)), np.arange(M)[-3:], rng.integers(0, M, 400)]))
    acc_ref, Y_ref = O.w4a4_linear(qx[rows], scale[0, gid[0, rows]], qw, sw, bias)
    Qx, Qw = _packed(qx, extra), _packed(qw, 0)
    for out_dtype in (torch.float32, torch.float16):
        Y = tdq.tdq_w4a4_linear(Qx, d[0], d[1], 1, M, K, Qw, d[2], d[3], out_dtype)
        got = Y[torch.from_numpy(rows).to(U.dev())].cpu().numpy()
        want = Y_ref if out_dtype == torch.float32 else Y_ref.astype(np.float16)
        assert np.array_equal(got, want), out_dtype
        assert torch.isfinite(Y).all()
    acc, Y = U.gpu_linear(Qx, d[0], d[1], 1, M, K, Qw, d[2])
    assert np.array_equal(acc[rows], acc_ref)
    assert np.array_equal(Y[rows], O.w4a4_linear(qx[rows], scale[0, gid[0, rows]], qw, sw)[1])
