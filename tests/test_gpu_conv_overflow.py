"""GPU test of the conv layers where A and the adjoint's pre-activations leave
float32 at neurons that multiply them by nothing: a neuron that is inactive, or
split to z < 0, contributes 0 (or beta), not 0 times infinity.  Two
convolutions whose weights from and into such neurons are 3e38, on register
tiles (where a layer has none, row-major) and on the row-major kernels alone,
against the FP64 oracle (where nothing overflows); 1e-4 guarded relative, as for
the other parity tests.  (The subdomain-major kernels multiply by coefficients
and are not asked for.)"""
import numpy as np
import pytest

from oracle import batch as ob
from oracle import beta_crown as bc
from paper_2103_06624_amd import synth
from tests import cases
from tests.cases import guarded_rel

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-4
BIG = np.float32(3e38)

NETS = [
    ((3, 16, 16), [(8, 4, 2, 1), (8, 3, 1, 1)]),
    ((3, 16, 16), [(8, 3, 1, 1), (16, 4, 2, 1)]),
    ((3, 11, 13), [(5, 3, 2, 1), (7, 3, 1, 0)]),
    ((3, 32, 32), [(8, 4, 2, 1), (8, 3, 1, 1)]),   # (tiles in both directions of both layers)
    ((3, 32, 32), [(16, 4, 2, 1), (5, 4, 2, 1)]),
]


def dev(a):
    return torch.from_numpy(np.asarray(a, np.float32)).cuda()


@pytest.mark.parametrize("i", range(len(NETS)))
@pytest.mark.parametrize("tiles", [0, 1])
def test_overflow_at_neurons_without_a_part(i, tiles):
    from paper_2103_06624_amd.api import BoundProblem
    shape, convs = NETS[i]
    print("overflow", NETS[i], tiles, flush=True)
    rng = np.random.default_rng([80, i])
    net = synth.cnn(rng, shape, convs, [16, 10])
    c1, c2 = net.layers[0], net.layers[1]
    # channel 0 of the first layer is inactive, channel 1 split to z < 0: both
    # feed the second layer by 3e38; channel 0 is fed by 3e38 as well, and so
    # is the inactive channel 0 of the second layer
    c2.weight[:, 0:2] = BIG
    c1.weight[0] = BIG
    c2.weight[0] = BIG
    n1 = int(np.prod(c1.out_shape)) // c1.out_shape[0]
    n2 = int(np.prod(c2.out_shape)) // c2.out_shape[0]
    d1, d2 = c1.d_out, c2.d_out
    P, n_dom = 2, 6
    nd = sum(net.dims[1:-1])
    kind = rng.integers(0, 3, size=(P, nd))
    kind[:, 0:n1] = 0
    kind[:, n1:2 * n1] = 2
    kind[:, d1:d1 + n2] = 0
    a, b = rng.uniform(0.2, 1.0, size=(2, P, nd)).astype(np.float32)
    lo = np.where(kind == 0, -a - b, np.where(kind == 1, a, -a)).astype(np.float32)
    up = np.where(kind == 0, -a, np.where(kind == 1, a + b, b)).astype(np.float32)
    x0 = rng.uniform(0, 1, size=(P, net.dims[0])).astype(np.float32)
    xlo, xhi = synth.box(x0, 4.0 / 255.0)
    C = np.stack([synth.margin_spec(q, 10) for q in range(P)]).astype(np.float32)
    prop = (np.arange(n_dom) % P).astype(np.int32)
    ptr = (np.arange(n_dom + 1) * n1).astype(np.int64)
    neuron = np.tile(np.arange(n1, 2 * n1), n_dom).astype(np.int32)
    args = (prop, ptr, np.ones(n_dom * n1, np.int32), neuron, -np.ones(n_dom * n1, np.int8))
    orc = ob.OracleProblem(net.layers, xlo, xhi, C, lo, up, *args, net64=bc.dense_net(net.layers))
    pb = BoundProblem(net.layers, xlo, xhi, C, lo, up, *args)
    pb.set_conv_variant(0)
    pb.set_conv_tiles(tiles)
    on = [pb.conv_tiles(j, d) for j in (1, 2) for d in (0, 1)]
    print("on tiles", on, flush=True)
    assert on == [tiles] * 4 or i < 3
    alpha, beta = cases.random_vars(orc, seed=3)
    ref = [orc.grad(d, alpha, beta) for d in range(n_dom)]
    lb_ref = np.stack([r[0] for r in ref])
    assert np.isfinite(lb_ref).all()
    assert guarded_rel(pb.eval(dev(alpha), dev(beta)).cpu().numpy(), lb_ref).max() <= TOL
    lb, ga, gb = (t.cpu().numpy() for t in pb.grad(dev(alpha), dev(beta)))
    assert guarded_rel(lb, lb_ref).max() <= TOL
    assert guarded_rel(ga, np.concatenate([r[1] for r in ref])).max() <= TOL
    assert guarded_rel(gb, np.concatenate([r[2].reshape(-1) for r in ref])).max() <= TOL
    a0, z0 = orc.default_alpha_flat(), np.zeros(orc.nnz * orc.m)
    best, _ = pb.optimize(dev(a0), dev(z0), iters=3)
    opt = np.stack([orc.optimize(d, a0, z0, bc.AdamConfig(iters=3))[0] for d in range(n_dom)])
    assert guarded_rel(best.cpu().numpy(), opt).max() <= TOL
    pb.close()
