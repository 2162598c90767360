"""GPU parity of the dense layers where their widths end inside a quad of
columns or a tile: one, two and three columns over, layers of one to three
neurons, either side of the 32- and 256-column rules, inputs of odd width, and
batches of a few rows.  Bounds, gradients, the network at x* and a short
optimisation against the FP64 oracle, over boxes and l2 balls.  Bar: 1e-4
guarded relative, as for the other parity tests."""
import numpy as np
import pytest

from oracle import batch as ob
from oracle import beta_crown as bc
from paper_2103_06624_amd import synth
from tests import test_gpu_conv_tiles as tiles

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

NETS = [
    [5, 3, 7, 10],
    [13, 17, 33, 31, 10],
    [31, 2, 1, 10],
    [66, 257, 30, 10],
    [9, 255, 261, 10],
]


@pytest.mark.parametrize("i", range(len(NETS)))
@pytest.mark.parametrize("n_dom", [1, 8])
def test_dense_widths(i, n_dom):
    from paper_2103_06624_amd.api import BoundProblem
    print("dense widths", NETS[i], n_dom, flush=True)
    rng = np.random.default_rng([78, i])
    net = synth.mlp(rng, NETS[i])
    x0 = rng.uniform(0, 1, size=(2, net.dims[0])).astype(np.float32)
    eps = 0.1
    xlo, xhi = synth.box(x0, eps)
    C = np.stack([synth.margin_spec(q, 10) for q in range(2)]).astype(np.float32)
    net64 = bc.dense_net(net.layers)
    # root bounds over the whole balls too: the box around x0, not clipped
    lo, up = bc.outward_f32(*ob.root_bounds_all(net64, x0 - np.float32(eps), x0 + np.float32(eps)))
    prop = (np.arange(n_dom) % 2).astype(np.int32)
    sp = synth.sample_splits(5 + i, net.dims, lo, up, prop, (0, 3))
    args = (sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    orc = ob.OracleProblem(net.layers, xlo, xhi, C, lo, up, *args, net64=net64)
    pb = BoundProblem(net.layers, xlo, xhi, C, lo, up, *args)
    tiles.check(orc, pb, (NETS[i], n_dom, "box"))
    pb.set_input_l2(x0, eps)
    orc.set_l2(x0, np.full(x0.shape[0], np.float32(eps)))
    tiles.check(orc, pb, (NETS[i], n_dom, "ball"))
    pb.close()
