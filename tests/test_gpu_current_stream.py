"""Calls without a stream run on the current stream of the current device: on a
side stream the result follows the work queued there before the call."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_call_follows_the_current_stream():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    assert ag._stream(None).value in (None, torch.cuda.current_stream().cuda_stream)
    d = ag.make_desc(0.0, 0.0, 1.0, 1.0, 300, 200)
    src = torch.zeros((200, 300), device="cuda")
    dst = torch.empty_like(src)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert ag._stream(None).value == side.cuda_stream
        a = torch.randn((2048, 2048), device="cuda")
        for _ in range(20):
            a = torch.mm(a, a) * 1e-3
        src.add_(7.0)                    # queued behind the products
        ag.auv_resample_bilinear(src, d, dst, d)
        out = dst.clone()
    side.synchronize()
    assert torch.equal(out, torch.full_like(out, 7.0))
