"""The network against the single kernels around the numbers of rows up to which a
block gathers them together, for either side, and with long rows gathered 16 a wave."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import learned, synth  # noqa: E402
from gpu_util import log  # noqa: E402
from test_gpu_mpnn_net import single_kernels  # noqa: E402


@pytest.mark.parametrize("n,m", [(8192, 8193), (8193, 8192), (16384, 32768), (16384, 32767), (300, "long")])
def test_rows_around_the_lines(n, m):
    log(f"case n {n} m {m}")
    if m == "long":  # 8200 and more constraints of up to 40 literals, variables of some hundred occurrences
        inst = synth.mixed_small(n=n, seed=6, kmax=40, count=8300)
        assert inst.m > 8192
    else:
        inst = synth.random_ksat(n, m, 3, 9)
    G = learned.GraphBatch([inst], "cuda")
    net = learned.MPNN(learned.Params("cuda", seed=11))
    dx = torch.tensor(np.random.default_rng(12).standard_normal(G.Nv) / G.Nv, dtype=torch.float32, device="cuda")
    xhat = net.forward(G, keep=True)
    net.P.grad.fill_(float("nan"))
    net.backward(dx)
    ref_x, ref_g = single_kernels(net, G, dx)
    assert torch.equal(xhat, ref_x)
    for name, (o, shape) in net.P.offsets.items():  # as in test_network_equals_single_kernels
        a, b = (t[o:o + int(np.prod(shape))].double() for t in (net.P.grad, ref_g))
        assert torch.all((a - b).abs() <= 1e-5 * b.abs().max() + 1e-12), name
