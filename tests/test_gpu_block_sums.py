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
