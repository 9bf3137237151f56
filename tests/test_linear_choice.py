"""Which contraction kernel a shape takes: the rule as a function of the sizes, no GPU."""
import os

import pytest

from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.skipif(not os.path.exists(tdq.LIB_PATH),
                                reason="libtdq.so not built (python -m paper_2604_16855_amd.build)")

TILE = {"64x64": (64, 64), "64x128": (64, 128), "128x64": (128, 64), "128x128": (128, 128),
        "staged": (128, 128), "pipe": (256, 256), "wide": (256, 256)}


def _threads(M, N, kernel):
    bm, bn = TILE[kernel]
    groups = (-(-M // bm) + 7) // 8
    return groups * 8 * -(-N // bn) * 256


@pytest.mark.parametrize("M,K,N,kernel", [
    (968, 512, 512, "64x64"), (7744, 320, 1280, "64x128"), (131072, 320, 320, "128x64"),
    (131072, 1000, 1024, "128x128"), (20000, 4096, 500, "staged"), (33000, 1152, 4096, "pipe"),
    (4096, 4096, 4096, "wide")])
def test_each_kernel_has_its_shapes(M, K, N, kernel):
    assert U.linear_kernel(M, K, N, 256) == kernel


@pytest.mark.parametrize("cus", [8, 64, 256, 304])
def test_every_launch_fits(cus):
    """A launch has fewer than 2^32 threads.  2^30 rows are allowed, and their outputs fit the
    device up to about a hundred columns."""
    for M in (1, 1 << 20, (1 << 30) - 65, (1 << 30) - 64, (1 << 30) - 63, 1 << 30):
        for K in (1, 32, 320, 4096):
            for N in (1, 63, 64, 65, 96, 127, 128):
                kernel = U.linear_kernel(M, K, N, cus)
                assert _threads(M, N, kernel) < 1 << 32, (M, K, N, kernel)
