"""Block sums of the block-scaled linears at their largest magnitudes, with whole and with cut last stages of K
(a stage is 128 channels): unit steps and unit weight scales make every output the integer product itself, which
both kernels hold exactly (no sum here reaches 2^24), so the outputs have to be equal and not near."""
import numpy as np
import pytest
import torch

from paper_2604_16855_amd import inputs as I
from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _codes(shape, kind, seed):
    if kind == "random":
        return I.random_codes(shape, seed)
    q = np.full(shape, -8, dtype=np.int8)
    if kind == "mixed":                       # block sums of +2048, -1792 and 1568
        q[:, 32:64] = 7
        q[1::2] = -q[1::2] - 1
    return q


@pytest.mark.parametrize("six_bit", [False, True])
@pytest.mark.parametrize("kind", ["lowest", "mixed", "random"])
@pytest.mark.parametrize("M,K,N", [(33, 1, 5), (64, 32, 128), (65, 33, 129), (70, 127, 64), (128, 128, 128),
                                   (129, 129, 65), (40, 160, 200), (96, 256, 96), (200, 257, 130), (64, 1000, 72)])
def test_block_sums_are_exact(M, K, N, kind, six_bit):
    qx, qw = _codes((M, K), kind, 3), _codes((N, K), kind, 4)
    d, KB = U.dev(), -(-K // 32)
    Qx, Qw = U.pack_to_device(qx), U.pack_to_device(qw)
    step, ws = torch.ones((M, KB), device=d), torch.ones(N, device=d)
    if six_bit:
        Y = tdq.tdq_w4a4_linear_blocks_f6(tdq.tdq_pack_codes_f6(Qx, K), step, K, tdq.tdq_pack_codes_f6(Qw, K), N, ws,
                                          out_dtype=torch.float32)
    else:
        Y = tdq.tdq_w4a4_linear_blocks(Qx, step, K, Qw, ws, None, torch.float32)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), qx.astype(np.float64) @ qw.T.astype(np.float64))


def test_six_bit_rows_to_the_limit():
    """2^30 rows, the most an entry point takes: more tiles than one axis of a grid."""
    M, K, d = 1 << 30, 96, U.dev()
    if torch.cuda.mem_get_info()[0] < 130e9:
        pytest.skip("the operand alone is 103 GB")
    rows = I.random_codes((32, K), 5)
    frag = tdq.tdq_pack_codes_f6(U.pack_to_device(rows), K)               # 32 rows, repeated below
    Qx = torch.empty(M // 32 * frag.numel(), dtype=torch.uint8, device=d)
    Qx.view(-1, frag.numel()).copy_(frag)
    step = torch.ones((M, 1), device=d).expand(M, 3).clone()
    step[:, 0] = torch.arange(M, device=d) % 61 + 1
    qw = I.random_codes((2, K), 6)
    Y = tdq.tdq_w4a4_linear_blocks_f6(Qx, step, K, tdq.tdq_pack_codes_f6(U.pack_to_device(qw), K), 2,
                                      torch.ones(2, device=d), out_dtype=torch.float32)
    part = torch.from_numpy(np.stack([rows[:, 32 * b:32 * b + 32].astype(np.float32) @ qw[:, 32 * b:32 * b + 32].T
                                      for b in range(3)])).to(d)         # [3, 32, 2]
    for m in range(0, M, 1 << 27):
        got = Y[m:m + (1 << 27)].view(-1, 32, 2)
        s0 = step[m:m + (1 << 27), 0].view(-1, 32, 1)
        assert torch.equal(got, s0 * part[0] + (part[1] + part[2]))
