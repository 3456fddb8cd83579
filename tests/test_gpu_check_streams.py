"""dbmp_check finds the errors of forwards on other streams that synchronise with the null stream (those
created without the non-blocking flag), whichever stream it is given."""
import ctypes

import pytest
import torch

from paper_2602_22625_amd import capi, synth
from paper_2602_22625_amd.render import Renderer

pytestmark = pytest.mark.gpu


@pytest.fixture
def blocking_stream():
    hip = ctypes.CDLL("libamdhip64.so.7")  # the runtime torch has loaded
    s = ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(s)) == 0
    yield s.value
    assert hip.hipStreamDestroy(s) == 0


def test_check_waits_for_blocking_streams(blocking_stream):
    a = torch.rand(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    p = torch.zeros(3, 8, device="cuda")
    p[:, :2], p[:, 2] = 8.0, 1.0
    atlas = torch.tensor(synth.soft_disk(16)[None], device="cuda")
    R = Renderer(check=False)
    good, bad = (torch.tensor(v, dtype=torch.int32, device="cuda") for v in ([0, 0, 0], [0, 9, 0]))
    R.render(p, good, atlas, 16, 16)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for other in (side.cuda_stream, 0):
        with torch.cuda.stream(torch.cuda.ExternalStream(blocking_stream)):
            for _ in range(20):
                torch.mm(a, a, out=b)  # some tens of milliseconds ahead of the forward
            R.render(p, bad, atlas, 16, 16)
        assert capi.dbmp_check(R.ctx, other) == capi.DBMP_EINVAL
        torch.cuda.synchronize()
        assert capi.dbmp_check(R.ctx, other) == capi.DBMP_OK  # reported once
