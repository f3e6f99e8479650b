"""Round creation reports what its own calls report."""
import pytest

from paper_2604_03143_amd import workload as wl

pytestmark = pytest.mark.gpu


def test_an_error_left_behind_by_the_caller_is_not_the_rounds(tdo):
    """The runtime keeps a thread's last error until it is asked for: here that of a device that does not exist."""
    import torch
    from paper_2604_03143_amd import tdk
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    rnd = wl.make_round(wl.CONFIGS["tiny"])
    torch.zeros(1, device="cuda")
    hip = tdk.load()                                  # (the library's own runtime is found through it)
    assert hip.hipSetDevice(4096) != 0 and hip.hipPeekAtLastError() != 0
    try:
        tdk.round_from_workload(rnd).destroy()
    finally:
        hip.hipGetLastError()                         # nobody else is to find it either
