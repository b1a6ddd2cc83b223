"""The issue-rate microbenchmark behind the bench's ceiling of the bit-plane kernels."""
import ctypes

import pytest

import paper_2509_01654_amd as nw


def test_arguments_rejected_on_the_host():
    lib = nw.load_library()
    n = ctypes.c_uint64()
    assert lib.nw_function_issue_rate(0, 1, ctypes.byref(n), None) == nw.NW_EINVAL
    assert lib.nw_function_issue_rate(1, 0, ctypes.byref(n), None) == nw.NW_EINVAL
    assert lib.nw_function_issue_rate(1, 1, None, None) == nw.NW_EINVAL


@pytest.mark.gpu
def test_function_issue_rate():
    """Counts what it issues; the rate lies between the packed unit's floor and two a
    lane and clock (256 CUs x 64 lanes x 2.4 GHz)."""
    torch = pytest.importorskip("torch")
    print("[gpu case] function issue-rate microbenchmark", flush=True)
    assert nw.function_issue_rate(256, 16) == 256 * 256 * 16 * 64
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    n = nw.function_issue_rate(2048, 4096)
    e1.record()
    torch.cuda.synchronize()
    assert 5e12 < n / (e0.elapsed_time(e1) / 1e3) <= 2 * 256 * 64 * 2.4e9 * 1.02
