"""Sound mode on batches of 512 rows and more, where several rows share a
workgroup: networks with channel counts that leave a group partly empty,
stride classes of other than 64 positions, a stride wider than its kernel
(positions no tap reaches), dense layers either side of 256 outputs, and
specifications whose rows do not fill the last group.
Every bound lies at or below the FP64 oracle's at the same variables, no
tolerance, and within SOUND_TOL of it (the float64 margin plus one float ulp,
relative to max(|bound|, 1)).
"""
import sys

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
    "odd": ((3, 17, 19), [(5, 3, 2, 1), (6, 4, 1, 1)], [20, 9]),       # 8 rows a subdomain
    "stride3": ((1, 24, 25), [(4, 2, 3, 0), (5, 3, 1, 1)], [16, 11]),  # 10 rows, 320 -> 16
}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()


@pytest.mark.parametrize("name", sorted(NETS))
@pytest.mark.parametrize("doms", [64, 65])
def test_sound_rows(name, doms):
    from paper_2103_06624_amd.api import BoundProblem
    say("sound rows", name, doms)
    in_shape, convs, fcs = NETS[name]
    wr, cr, sr = (np.random.default_rng(s) for s in np.random.SeedSequence(doms).spawn(3))
    net = synth.cnn(wr, in_shape, convs, fcs)
    x0 = cr.uniform(0.0, 1.0, size=(2, net.dims[0])).astype(np.float32)
    eps = 2.0 / 255.0
    lo_x, hi_x = synth.box(x0, eps)
    C = np.stack([synth.margin_spec(int(np.argmax(synth.forward(net, x))), net.dims[-1]) for x in x0]).astype(np.float32)
    wl = synth.Workload(name, net, lo_x, hi_x, x0, float(eps), C, np.array([33, doms - 33], np.int64), (1, 6),
                        int(sr.integers(0, 2**31 - 1)))
    net64 = bc.dense_net(wl.net.layers)
    lo, up = bc.outward_f32(*ob.root_bounds_all(net64, wl.x_lo, wl.x_hi))
    sp = synth.attach_splits(wl, lo, up)
    orc = ob.OracleProblem(wl.net.layers, wl.x_lo, wl.x_hi, wl.C, lo, up, sp.dom_prop, sp.split_ptr, sp.layer,
                           sp.neuron, sp.side, net64=net64)
    pb = BoundProblem.from_workload(wl, lo, up)
    alpha, beta = random_vars(orc, seed=13)
    pb.set_sound(1)
    lb = pb.eval(dev(alpha), dev(beta)).cpu().numpy()
    pick = [0, 1, 31, 32, 33, 47, doms - 2, doms - 1]
    ref = np.stack([orc.eval(b, alpha, beta) for b in pick])
    say(name, "excess", float(np.maximum(lb[pick] - ref, 0).max()), "gap", float(guarded_rel(lb[pick], ref).max()))
    assert (lb[pick] <= ref).all()
    assert guarded_rel(lb[pick], ref).max() <= SOUND_TOL
    pb.close()
