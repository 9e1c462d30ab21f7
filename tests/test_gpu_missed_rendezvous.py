"""A stream that may use half of the device's CUs (a CU mask): a team of 256
workgroups never meets there.  One call finds that out; the calls after it do
not wait for the same again, and teams are tried again later."""
import ctypes
import time

import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say
from tests.test_gpu_resident import fv  # noqa: F401

pytestmark = pytest.mark.gpu
CALLS, LIMIT_MS = 20, 20


@pytest.fixture
def half_stream():
    """Every other 16 CUs of 256: some on every XCD, however they are numbered."""
    import torch

    hip = ctypes.CDLL("libamdhip64.so.7")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the mask is for 256 CUs")
    mask = (ctypes.c_uint32 * 8)(*[0x0000FFFF] * 8)
    h = ctypes.c_void_p()
    if hip.hipExtStreamCreateWithCUMask(ctypes.byref(h), ctypes.c_uint32(8), mask) != 0:
        pytest.skip("no CU masks here")
    yield torch.cuda.ExternalStream(h.value)
    torch.cuda.synchronize()
    hip.hipStreamDestroy(h)


def test_missed_rendezvous_is_paid_once(fv, monkeypatch, half_stream):  # noqa: F811
    import torch

    monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", str(LIMIT_MS))
    dc = DevCase(fc.varcoef((128, 64, 128), seed=11, permute=False))

    def run():
        return fv.solve(dc.A, dc.b, x=torch.zeros_like(dc.b), tol=0.0, maxit=20)

    say("missed rendezvous: all CUs")
    want, st = run()
    assert st["one_launch"] == 1
    torch.cuda.synchronize()
    with torch.cuda.stream(half_stream):
        say("missed rendezvous: half of the CUs")
        x, st = run()  # waits, and allocates what the launches need
        assert st["one_launch"] == 0 and torch.equal(x, want)
        t0 = time.perf_counter()
        for _ in range(CALLS):
            x, st = run()
            assert st["one_launch"] == 0 and torch.equal(x, want)
        ms = (time.perf_counter() - t0) * 1e3
    say("missed rendezvous:", CALLS, "calls", round(ms, 1), "ms")
    assert ms < CALLS * LIMIT_MS / 2
    time.sleep(50 * LIMIT_MS / 1e3)
    x, st = run()
    assert st["one_launch"] == 1 and torch.equal(x, want)
    dc.close()
