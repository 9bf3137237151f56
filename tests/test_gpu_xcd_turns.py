"""The workgroups of one set of all images take turns on the chip: with all tokens of every image in one set, a
number of sets that is a multiple of 8 (the number of XCDs) costs no more than one more set an image (up to
twice as much where one set of all images ran on one XCD, or on one of its shader engines)."""
import pytest
import torch

from paper_2604_16855_amd import tdq

import parity_util as U
from test_gpu_block_outputs import _time

pytestmark = pytest.mark.gpu


def _one_set(B, T, C, dtype):
    """Tokens that share their range: all in one set, whatever their number."""
    X = torch.rand((B, T, C), device=U.dev(), generator=torch.Generator(device="cuda").manual_seed(1)) - 0.5
    X[:, :, 0] = 4.0
    return X.to(dtype)


@pytest.mark.parametrize("B,T,C,G,pct", [(46, 16, 1414, 32, 0.0), (41, 510, 45, 24, 0.99), (35, 24, 1024, 24, 0.0)])
def test_calibration(B, T, C, G, pct):
    X, ms = _one_set(B, T, C, torch.float16), {}
    for g in (G, G + 1):
        assert tdq.lib().tdq_whole_extra(tdq.TDQ_F16, B, T, C, g, tdq.C.c_double(pct)) == 0
        p = tdq.default_params(g)
        p.base_pct = pct
        ws = tdq.alloc_workspace(B, T, C, tdq.TDQ_F16, p, X.device)
        out = (torch.empty((B, T), dtype=torch.int32, device=X.device),
               *(torch.empty((B, g), device=X.device) for _ in range(2)))
        ms[g] = _time(lambda: tdq.tdq_calibrate_groups(X, p, ws, out=out))
    print({g: f"{1e3 * t:.1f} us" for g, t in ms.items()}, flush=True)
    assert ms[G] <= 1.2 * ms[G + 1]
