"""Sound mode over l2 balls on batches of 512 rows and more, where several rows
share a workgroup: the row sums of A(0) x0 and of A(0)^2 by groups, on networks
whose first layer is a convolution and dense, a specification whose rows do not
fill the last group, and a layer whose three rows of planes take the whole 64 KB
of LDS that a group may; and subdomains of one, two, four and five rows, whose
groups are of one, two and three.  Every bound lies at or below the FP64 oracle's at the
same variables and within 1e-6 of it, as for boxes."""
import numpy as np
import pytest

from oracle import batch as ob
from oracle import beta_crown as bc
from paper_2103_06624_amd import synth
from tests.cases import guarded_rel, random_vars

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SOUND_TOL = 1e-6

# (input shape, convs (c_out, k, s, p), dense widths)
NETS = {
    "odd": ((3, 17, 19), [(5, 3, 2, 1), (6, 4, 1, 1)], [20, 9]),
    "full": ((2, 11, 19), [(10, 3, 1, 1), (10, 3, 1, 1)], [16, 11]),  # 3 rows of 10 planes of 13 x 21 doubles: 65,520 B
    "dense": (None, [], [40, 300, 31, 9]),
}


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()


@pytest.mark.parametrize("name", sorted(NETS))
@pytest.mark.parametrize("ball", [False, True])
def test_sound_balls(name, ball):
    from paper_2103_06624_amd.api import BoundProblem
    doms = 65
    print("sound balls", name, ball, flush=True)
    shape, convs, fcs = NETS[name]
    rng = np.random.default_rng([83, sorted(NETS).index(name)])
    net = synth.cnn(rng, shape, convs, fcs) if shape else synth.mlp(rng, fcs)
    x0 = rng.uniform(0.0, 1.0, size=(2, net.dims[0])).astype(np.float32)
    eps = np.float32(0.05 if shape else 0.2)
    xlo, xhi = (x0 - eps, x0 + eps)
    C = np.stack([synth.margin_spec(q, net.dims[-1]) for q in range(2)]).astype(np.float32)
    net64 = bc.dense_net(net.layers)
    lo, up = bc.outward_f32(*ob.root_bounds_all(net64, xlo, xhi))
    prop = (np.arange(doms) // 9 % 2).astype(np.int32)
    sp = synth.sample_splits(7, net.dims, lo, up, prop, (0, 6))
    args = (sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    orc = ob.OracleProblem(net.layers, xlo, xhi, C, lo, up, *args, net64=net64)
    pb = BoundProblem(net.layers, xlo, xhi, C, lo, up, *args)
    assert pb.n_rows >= 512
    if ball:
        pb.set_input_l2(x0, eps)
        orc.set_l2(x0, np.full(2, eps))
    alpha, beta = random_vars(orc, seed=13)
    pb.set_sound(1)
    lb = pb.eval(dev(alpha), dev(beta)).cpu().numpy()
    pick = [0, 1, 8, 9, 17, 18, 40, doms - 2, doms - 1]
    ref = np.stack([orc.eval(b, alpha, beta) for b in pick])
    print(name, "excess", float(np.maximum(lb[pick] - ref, 0).max()), "gap", float(guarded_rel(lb[pick], ref).max()), flush=True)
    assert (lb[pick] <= ref).all()
    assert guarded_rel(lb[pick], ref).max() <= SOUND_TOL
    pb.close()


@pytest.mark.parametrize("name", ["odd", "dense"])
@pytest.mark.parametrize("m", [1, 2, 4, 5])
def test_sound_few_rows(name, m):
    """Specifications of few rows."""
    from paper_2103_06624_amd.api import BoundProblem
    doms = 512 // m + 1
    print("sound rows", name, m, flush=True)
    shape, convs, fcs = NETS[name]
    fcs = fcs[:-1] + [m + 1]
    rng = np.random.default_rng([84, m])
    net = synth.cnn(rng, shape, convs, fcs) if shape else synth.mlp(rng, fcs)
    x0 = rng.uniform(0.0, 1.0, size=(2, net.dims[0])).astype(np.float32)
    eps = np.float32(0.05)
    C = np.stack([synth.margin_spec(q, m + 1) for q in range(2)]).astype(np.float32)
    net64 = bc.dense_net(net.layers)
    lo, up = bc.outward_f32(*ob.root_bounds_all(net64, x0 - eps, x0 + eps))
    prop = (np.arange(doms) // 9 % 2).astype(np.int32)
    sp = synth.sample_splits(7, net.dims, lo, up, prop, (0, 6))
    args = (sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    orc = ob.OracleProblem(net.layers, x0 - eps, x0 + eps, C, lo, up, *args, net64=net64)
    pb = BoundProblem(net.layers, x0 - eps, x0 + eps, C, lo, up, *args)
    assert pb.n_rows >= 512
    alpha, beta = random_vars(orc, seed=13)
    pb.set_sound(1)
    lb = pb.eval(dev(alpha), dev(beta)).cpu().numpy()
    pick = [0, 1, 8, 9, 17, 18, 40, doms - 2, doms - 1]
    ref = np.stack([orc.eval(b, alpha, beta) for b in pick])
    assert (lb[pick] <= ref).all()
    assert guarded_rel(lb[pick], ref).max() <= SOUND_TOL
    pb.close()
