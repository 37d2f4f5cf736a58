"""The wrappers' argument checks and the stream they launch on."""
import pytest
import torch

from paper_2506_20686_amd import binding as B

pytestmark = pytest.mark.gpu


def test_launches_on_the_current_stream():
    dev = torch.device("cuda", torch.cuda.current_device())
    side = torch.cuda.Stream(dev)
    assert B._stream(dev) == torch.cuda.current_stream(dev).cuda_stream
    with torch.cuda.stream(side):
        assert B._stream(dev) == side.cuda_stream
        assert B._stream(torch.device("cuda")) == side.cuda_stream
    assert B._stream(dev) == torch.cuda.current_stream(dev).cuda_stream


@pytest.mark.parametrize("which", ["q", "k", "bias", "mask"])
@pytest.mark.parametrize("fault, error", [
    (lambda t: t.tolist(), TypeError),
    (lambda t: t.cpu(), ValueError),
    (lambda t: t.to(torch.float16), ValueError),
    (lambda t: t[:-1], ValueError),
    (lambda t: t.transpose(0, 1), ValueError),
])
def test_refused_arguments(which, fault, error):
    if which == "q" and error is TypeError:
        error = AttributeError  # q gives the shapes, before any check
    n, h, d = 33, 2, 32
    t = {k: torch.randn(n, n, h, d, device="cuda").bfloat16() for k in "qkvg"}
    t["bias"] = torch.randn(n, n, h, device="cuda").bfloat16()
    t["mask"] = torch.ones(n, n, dtype=torch.uint8, device="cuda")
    B.fwd(**t)
    t[which] = fault(t[which])
    with pytest.raises(error):
        B.fwd(**t)
