"""The stream that the binding hands to the library: the current one, by torch's raw look-up or,
in a build of torch without it, by the stream object."""
import types

import pytest
import torch

from paper_2604_16855_amd import inputs as I
from paper_2604_16855_amd import tdq


def test_without_the_raw_lookup(monkeypatch):
    monkeypatch.setattr(tdq, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    assert tdq._stream() == 4711


@pytest.mark.gpu
def test_both_lookups_name_the_current_stream(monkeypatch):
    """On the default stream and on one of the caller's; a calibration runs with either."""
    lc = I.case("cfg0")
    X = torch.from_numpy(I.make_activations(lc)[0]).cuda()
    p = tdq.default_params(lc.G)
    expect = tdq.tdq_calibrate_groups(X, p)[2].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for raw in (tdq._raw_stream, None):
        monkeypatch.setattr(tdq, "_raw_stream", raw)
        assert tdq._stream() == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert tdq._stream() == side.cuda_stream
            scale = tdq.tdq_calibrate_groups(X, p)[2]
        side.synchronize()
        assert torch.equal(scale, expect)
