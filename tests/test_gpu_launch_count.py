"""Kernel launches of a call, counted as the nodes of its captured graph."""
import ctypes

import pytest

from paper_2109_05496_amd import _lib

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def launches(b, support, iters, **kw):
    """Nodes of ctv_denoise captured on a stream of its own; the graph is not run."""
    import paper_2109_05496_amd as ctv
    ctv.tune_cache_clear()
    hip = ctypes.CDLL("libamdhip64.so")
    m, n = b.shape
    ws = torch.empty(ctv.workspace_size(m, n, 1, iters=iters)[0], dtype=torch.uint8, device="cuda")
    out = torch.empty_like(b)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    handle, graph, count = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(handle, 2) == 0  # relaxed mode
        try:
            ctv.denoise(b, 0.05, support=support, iters=iters, out=out, workspace=ws, **kw)
        finally:
            assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("m,n", [(64, 64), (40, 64), (7, 9)])
@pytest.mark.parametrize("iters", [1, 5, 30])
def test_a_support_adds_no_launch_to_an_image_of_one_region(m, n, iters):
    b = torch.view_as_complex(torch.randn(m, n, 2, device="cuda")).contiguous()
    support = torch.zeros(m, n, dtype=torch.uint8, device="cuda")
    support[: m // 2 + 1] = 1
    assert launches(b, support, iters) == launches(b, None, iters)


def test_a_larger_image_lists_its_live_tiles():
    b = torch.view_as_complex(torch.randn(300, 300, 2, device="cuda")).contiguous()
    support = torch.zeros(300, 300, dtype=torch.uint8, device="cuda")
    support[:40, :40] = 1
    kw = dict(tile=(8, 8), fuse=8)
    # K = 16: launches of 8 (state) and 8 (x), two tilings with a scan and a list each
    assert launches(b, support, 16, **kw) == launches(b, None, 16, **kw) + 4 == 6
