"""What a network holds between training steps: its activations, no workspace of the
backward pass."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import learned, synth  # noqa: E402
from gpu_util import log  # noqa: E402


def test_backward_keeps_no_workspace():
    log("case n 3000")
    G = learned.GraphBatch([synth.random_ksat(3000, 12600, 3, 1)], "cuda")
    net = learned.MPNN(learned.Params("cuda", seed=1))
    dx = torch.ones(G.Nv, device="cuda")
    net.forward(G, keep=True)
    held = torch.cuda.memory_allocated()
    net.backward(dx)
    assert torch.cuda.memory_allocated() == held
    grad = net.P.grad.clone()
    # another stream right after: its own workspace
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        net.forward(G, keep=True)
        net.backward(dx)
    torch.cuda.synchronize()
    assert torch.equal(net.P.grad, grad)
