"""The network's whole forward and backward pass against the single kernels run one
after another: the forward pass bit for bit, the gradients to the accuracy of the
split products.  Row counts around the 16- and 64-row tiles and the 256-row chunks,
variables without occurrences, no constraints at all."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import learned, synth  # noqa: E402
from gpu_util import log  # noqa: E402

H, F = learned.HID, learned.FEAT


def empty(*shape):
    return torch.empty(*shape, dtype=torch.float32, device="cuda")


def single_kernels(net, G, dxhat):
    """xhat and the flat gradient, one kernel per operation."""
    P, Nv, Nc, sc = net.P, G.Nv, G.Nc, learned.Scratch("cuda")
    Zv0, Hv, Zc0, Hc = empty(Nv, H), empty(Nv, H), empty(Nc, H), empty(Nc, H)
    learned.gemm(G.Fv, F, Nv, F, P.wb("Ev"), H, 0, P.w("ev"), Zv0, H, 0, Hv)
    learned.gemm(G.Fc, F, Nc, F, P.wb("Ec"), H, 0, P.w("ec"), Zc0, H, 0, Hc)
    kept = []
    for l in range(learned.LAYERS):
        Pm, Zc, Hc2, Qm, Zv, Hv2 = (empty(Nv, 2 * H), empty(Nc, H), empty(Nc, H), empty(Nc, 2 * H), empty(Nv, H),
                                    empty(Nv, H))
        learned.gemm(Hv, H, Nv, H, P.wb(f"Wpn_{l}"), 2 * H, 0, None, Pm, 2 * H)
        learned.gemm(Hc, H, Nc, H, P.wb(f"W1_{l}"), H, 0, P.w(f"bc_{l}"), Zc, H)
        learned.gather(G.cptr, G.cidx, G.cw, Nc, Pm, 2 * H, Zc, H, Hc2, 0)
        learned.gemm(Hc2, H, Nc, H, P.wb(f"Upn_{l}"), 2 * H, 0, None, Qm, 2 * H)
        learned.gemm(Hv, H, Nv, H, P.wb(f"W2_{l}"), H, 0, P.w(f"bv_{l}"), Zv, H)
        learned.gather(G.vptr, G.vidx, G.vw, Nv, Qm, 2 * H, Zv, H, Hv2, 0)
        kept.append((Hv, Hc, Zc, Hc2, Zv))
        Hv, Hc = Hv2, Hc2
    xhat = empty(Nv)
    learned.head_forward(Hv, Nv, P.w("wo"), P.w("bo"), xhat)
    grad = torch.zeros_like(P.grad)

    def g(name):
        o, shape = P.offsets[name]
        return grad[o:o + int(np.prod(shape))]

    dHv, dlogit, dHc = empty(Nv, H), empty(Nv), None
    learned.head_backward(xhat, dxhat, Nv, P.w("wo"), dHv, dlogit)
    o = P.offsets["wo"][0]
    learned.head_grad(Hv, dlogit, Nv, grad[o:o + H + 1], sc)
    for l in reversed(range(learned.LAYERS)):
        Hvl, Hcl, Zc, Hc2, Zv = kept[l]
        dZv, dHv_in, dQ, dZc, dHc_in, dP = (empty(Nv, H), empty(Nv, H), empty(Nc, 2 * H), empty(Nc, H), empty(Nc, H),
                                            empty(Nv, 2 * H))
        learned.relu_grad(dHv, Zv, dZv)
        learned.colsum(dZv, H, Nv, g(f"bv_{l}"), sc)
        learned.gemm_tn(dZv, H, Hvl, H, Nv, H, H, g(f"W2_{l}"), sc)
        learned.gemm(dZv, H, Nv, H, P.wb(f"W2_{l}"), H, 1, None, dHv_in, H)
        learned.gather(G.cptr, G.cidx, G.cw_t, Nc, dZv, H, dQ, 2 * H, None, 1)
        learned.gemm_tn(dQ, 2 * H, Hc2, H, Nc, 2 * H, H, g(f"Upn_{l}"), sc)
        beta = 0 if dHc is None else 1
        dHc = empty(Nc, H) if dHc is None else dHc
        learned.gemm(dQ, 2 * H, Nc, 2 * H, P.wb(f"Upn_{l}"), H, 1, None, dHc, H, beta)
        learned.relu_grad(dHc, Zc, dZc)
        learned.colsum(dZc, H, Nc, g(f"bc_{l}"), sc)
        learned.gemm_tn(dZc, H, Hcl, H, Nc, H, H, g(f"W1_{l}"), sc)
        learned.gemm(dZc, H, Nc, H, P.wb(f"W1_{l}"), H, 1, None, dHc_in, H)
        learned.gather(G.vptr, G.vidx, G.vw_t, Nv, dZc, H, dP, 2 * H, None, 1)
        learned.gemm_tn(dP, 2 * H, Hvl, H, Nv, 2 * H, H, g(f"Wpn_{l}"), sc)
        learned.gemm(dP, 2 * H, Nv, 2 * H, P.wb(f"Wpn_{l}"), H, 1, None, dHv_in, H, 1)
        dHv, dHc = dHv_in, dHc_in
    dZv0, dZc0 = empty(Nv, H), empty(Nc, H)
    learned.relu_grad(dHv, Zv0, dZv0)
    learned.relu_grad(dHc, Zc0, dZc0)
    learned.colsum(dZv0, H, Nv, g("ev"), sc)
    learned.colsum(dZc0, H, Nc, g("ec"), sc)
    learned.gemm_tn(dZv0, H, G.Fv, F, Nv, H, F, g("Ev"), sc)
    learned.gemm_tn(dZc0, H, G.Fc, F, Nc, H, F, g("Ec"), sc)
    return xhat, grad


def instances(case):
    if case[0] == "n":  # variables around the line where blocks share rows; degrees around 16 entries in flight
        return [synth.random_ksat(int(case[1:]), 6 * int(case[1:]), 3, 9)]
    if case == "longer":  # fewer constraints than variables: the constraints' rows are shared, some above 16 entries
        return [synth.mixed_small(n=400, seed=6, kmax=40, count=333)]
    if case == "one":
        return [synth.random_ksat(3, 1, 3, 1)]
    if case == "tiles":  # 63 variables, 65 constraints
        return [synth.random_ksat(63, 65, 3, 2)]
    if case == "isolated":  # most variables occur nowhere
        return [synth.random_ksat(257, 16, 3, 3)]
    if case == "types":
        return [synth.mixed_small(n=70, seed=4, kmax=40, count=255), synth.mixed_small(n=31, seed=5, kmax=5, count=17)]
    return [synth.c5_train(i) for i in range(3)] + [synth.c2_mixed(7, 300, 900, 90, 30)]


@pytest.mark.parametrize("case", ["one", "tiles", "isolated", "types", "several", "n16383", "n16384", "n16385", "longer"])
def test_network_equals_single_kernels(case):
    log(f"case {case}")
    G = learned.GraphBatch(instances(case), "cuda")
    net = learned.MPNN(learned.Params("cuda", seed=11))
    rng = np.random.default_rng(12)
    dx = torch.tensor(rng.standard_normal(G.Nv) / G.Nv, dtype=torch.float32, device="cuda")
    xhat = net.forward(G, keep=True)
    net.P.grad.fill_(float("nan"))  # every entry is written
    net.backward(dx)
    ref_x, ref_g = single_kernels(net, G, dx)
    assert torch.equal(xhat, ref_x)
    got, want = net.P.grad.double(), ref_g.double()
    # the same products in another order of summation: operands of 16 significant
    # bits, sums of float32 terms; 1e-5 of the largest entry of each tensor
    for name, (o, shape) in net.P.offsets.items():
        a, b = got[o:o + int(np.prod(shape))], want[o:o + int(np.prod(shape))]
        assert torch.all((a - b).abs() <= 1e-5 * b.abs().max() + 1e-12), name
    net.backward(dx)
    assert torch.equal(net.P.grad.double(), got)  # fixed order of summation


def test_no_constraints():
    inst = synth.Instance(5, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int8), np.zeros(0, np.int32))
    G = learned.GraphBatch([inst], "cuda")
    net = learned.MPNN(learned.Params("cuda", seed=1))
    xhat = net.forward(G, keep=True)
    net.P.grad.fill_(float("nan"))
    net.backward(torch.ones(5, device="cuda"))
    assert bool(torch.isfinite(xhat).all()) and bool(torch.isfinite(net.P.grad).all())
    for name in ("Ec", "ec", "W1_0", "Upn_2", "bc_1"):
        o, shape = net.P.offsets[name]
        assert bool((net.P.grad[o:o + int(np.prod(shape))] == 0).all())
