"""Which launches keep a small problem's codes in LDS: not those that would hold fewer
tiles on a CU for it.  More restarts than CUs, so that CUs run several tiles, side by
side or one after another."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_06656_amd import pcls, synth  # noqa: E402
from gpu_util import log  # noqa: E402


def state_bytes(n):
    """LDS of a tile of one restart without codes: x, gradient, objective slots, counters, flags."""
    return 8 * n + 16 + 2 * 64 * 8 + 4 * 96 + 8


@pytest.mark.parametrize("n,R,tile,block,in_lds,auto_block", [
    (200, 64, 0, 0, True, 1024), (200, 320, 0, 0, True, 512), (1000, 320, 0, 0, True, 512),
    (2000, 64, 0, 0, True, 1024), (2000, 320, 0, 0, False, 512), (2000, 320, 1, 512, False, 512),
    (1000, 320, 1, 256, True, 256), (1000, 768, 1, 256, False, 256), (2000, 640, 1, 1024, True, 1024)])
def test_rule_and_iterates(n, R, tile, block, in_lds, auto_block):
    log(f"case n {n} R {R} tile {tile} block {block}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus == 256  # the restart counts above are chosen for it
    prob = pcls.Problem.from_instance(synth.random_ksat(n, int(4.2 * n), 3, n))
    prob.set_launch(tile, block)
    info = prob.launch_info(R)
    assert info["tile_restarts"] == 1 and info["block_threads"] == auto_block
    assert (info["lds_bytes"] > state_bytes(n)) == in_lds
    X = prob.new_state(R)
    prob.init_restarts(X, R, 4)
    Y, Z = X.clone(), X.clone()
    tr = prob.step(X, R, 0.1, 12, trace=True)
    parts = torch.cat([prob.step(Y, R, 0.1, 4, trace=True) for _ in range(3)])
    assert torch.equal(tr, parts) and torch.equal(X[:, :R], Y[:, :R])
    prob.set_launch(2, 0)
    prob.step(Z, R, 0.1, 12)
    assert torch.equal(X[:, :R], Z[:, :R])
