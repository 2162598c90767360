"""GPU parity of the conv kernels over K passes and over batches.

K passes: register tiles asked for on networks whose layers take one to seven
passes over K (one to six are compiled in, others looped) with one, two and four
row tiles per wave, in both directions.

Batches: enough subdomains that a workgroup walks several rows of a subdomain
and takes several units, with the property changing on the way, on register
tiles and on the subdomain-major kernels; a sample of subdomains (early, late,
either side of a change of property) is compared.

All against the FP64 oracle at 1e-4 guarded relative, as for the other parity
tests; sound bounds lie at or below it."""
import numpy as np
import pytest

from oracle import batch as ob
from oracle import beta_crown as bc
from paper_2103_06624_amd import synth
from tests import test_gpu_conv_tiles as tiles
from tests.cases import guarded_rel

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-4

# input (c, h, w), convolutions (c_out, k, s, p)
K_NETS = [
    ((1, 16, 16), [(5, 5, 1, 2), (8, 3, 1, 1), (16, 5, 2, 2)]),
    ((3, 32, 32), [(8, 4, 2, 1), (4, 3, 1, 0), (20, 4, 2, 1)]),
    ((4, 16, 16), [(16, 3, 1, 1), (16, 3, 1, 0), (8, 3, 1, 1)]),
    ((1, 28, 28), [(4, 5, 2, 2), (10, 2, 2, 0)]),
    ((2, 20, 20), [(8, 3, 1, 1), (24, 4, 2, 1), (6, 4, 2, 1)]),
    ((2, 20, 20), [(16, 2, 2, 0), (4, 3, 1, 1), (10, 5, 2, 2)]),
    ((4, 16, 16), [(16, 3, 2, 1), (12, 5, 2, 2), (6, 5, 1, 2)]),
    ((1, 28, 28), [(16, 4, 2, 1), (6, 4, 2, 1)]),
    ((1, 28, 28), [(8, 5, 2, 2), (16, 3, 1, 1)]),
    ((3, 32, 32), [(16, 5, 2, 2), (3, 3, 1, 0)]),
    ((3, 11, 13), [(5, 5, 1, 2), (16, 3, 1, 0)]),
    ((4, 16, 16), [(4, 3, 1, 1), (8, 4, 2, 1), (20, 5, 2, 2)]),
    ((4, 16, 16), [(20, 4, 2, 1), (8, 3, 1, 1)]),
    ((3, 32, 32), [(8, 4, 2, 1), (5, 3, 1, 1), (4, 4, 2, 1)]),
    ((4, 16, 16), [(6, 4, 2, 1), (8, 3, 1, 1)]),
    ((1, 28, 28), [(10, 5, 1, 2), (12, 3, 2, 1)]),
    ((3, 11, 13), [(16, 3, 1, 0), (10, 3, 1, 1), (16, 5, 2, 2)]),
    ((3, 32, 32), [(6, 2, 2, 0), (12, 3, 1, 0)]),
    ((3, 24, 24), [(10, 5, 1, 2), (10, 2, 2, 0), (8, 3, 1, 1)]),
    ((3, 24, 24), [(8, 3, 2, 1), (5, 3, 1, 0), (20, 3, 1, 1)]),
    ((2, 20, 20), [(12, 5, 2, 2), (10, 3, 2, 1), (32, 3, 2, 1)]),
    ((2, 16, 16), [(4, 3, 1, 0), (6, 3, 1, 0)]),
    ((2, 20, 20), [(4, 5, 1, 2), (3, 3, 2, 1)]),
    ((3, 20, 20), [(8, 5, 1, 2)]),
    ((1, 32, 32), [(4, 3, 1, 1), (8, 2, 2, 0)]),
    ((1, 28, 28), [(6, 4, 2, 1), (8, 3, 1, 1)]),
    ((1, 32, 32), [(4, 3, 1, 1), (10, 2, 2, 0)]),
    ((1, 28, 28), [(8, 3, 1, 1), (10, 2, 2, 0)]),
]

# rows staged by scalars and by float4s, outputs in pairs and not, one and two
# staged rows, first layers of stride 1 and 2, K passes compiled in and looped
BATCH_NETS = [
    ((3, 13, 17), [(6, 5, 2, 1), (9, 3, 1, 1)]),
    ((2, 16, 16), [(8, 3, 1, 1), (8, 3, 1, 1), (20, 3, 2, 1)]),
    ((3, 32, 32), [(8, 4, 2, 1), (16, 4, 2, 1)]),
    ((1, 9, 9), [(3, 3, 2, 1)]),
]
BATCH = 4200


def build(shape, convs, prop, seed, fc=20):
    """Network, properties (boxes inside balls of radius eps), splits."""
    from paper_2103_06624_amd.api import root_bounds
    rng = np.random.default_rng([81, seed])
    net = synth.cnn(rng, shape, convs, [fc, 10])
    P = int(prop.max()) + 1
    x0 = rng.uniform(0, 1, size=(P, net.dims[0])).astype(np.float32)
    eps = np.float32(4.0 / 255.0)
    xlo, xhi = synth.box(x0, eps)
    C = np.stack([synth.margin_spec(q, 10) for q in range(P)]).astype(np.float32)
    lo, up = root_bounds(net.layers, x0 - eps, x0 + eps)
    sp = synth.sample_splits(seed, net.dims, lo, up, prop, (0, 5))
    return net, x0, eps, (net.layers, xlo, xhi, C, lo, up), sp


def oracle(args, sp, pick, net64):
    """The oracle on the subdomains `pick` of the batch."""
    spans = [np.arange(sp.split_ptr[b], sp.split_ptr[b + 1]) for b in pick]
    t = np.concatenate(spans).astype(np.int64)
    ptr = np.concatenate([[0], np.cumsum([len(s) for s in spans])]).astype(np.int64)
    return ob.OracleProblem(*args, sp.dom_prop[pick], ptr, sp.layer[t], sp.neuron[t], sp.side[t], net64=net64), t


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("i", range(len(K_NETS)))
def test_k_passes(i):
    from paper_2103_06624_amd.api import BoundProblem
    shape, convs = K_NETS[i]
    prop = (np.arange(5) % 2).astype(np.int32)
    net, x0, eps, args, sp = build(shape, convs, prop, i)
    pb = BoundProblem(*args, sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    pb.set_conv_tiles(1)
    on = [(pb.conv_tiles(j + 1, 0), pb.conv_tiles(j + 1, 1)) for j in range(len(convs))]
    print("K passes", K_NETS[i], on, flush=True)
    orc, _ = oracle(args, sp, np.arange(5), bc.dense_net(net.layers))
    tiles.check(orc, pb, (K_NETS[i], "box"))
    pb.set_input_l2(x0, eps)
    orc.set_l2(x0, np.full(x0.shape[0], eps))
    tiles.check(orc, pb, (K_NETS[i], "ball"))
    pb.close()


def unit_rows(B, m, grid):
    """The rule of the subdomain-major kernels' work units (conv_unit_rows)."""
    cost = [(-(-B * -(-m // u) // grid) * (u + 1), -u) for u in range(1, min(m, 32) + 1)]
    return -min(cost)[1]


@pytest.mark.parametrize("i", range(len(BATCH_NETS)))
@pytest.mark.parametrize("kernel", ["default", "tiles", "variant 2", "variant 3"])
def test_many_subdomains(i, kernel):
    from paper_2103_06624_amd.api import BoundProblem
    # whatever fits on a CU (1 to 16 workgroups on 256 of them): several rows of
    # a subdomain in a unit, more units than workgroups
    for per in range(1, 17):
        mu = unit_rows(BATCH, 9, 256 * per)
        assert mu > 1 and BATCH * -(-9 // mu) > 256 * per, per
    shape, convs = BATCH_NETS[i]
    prop = (np.arange(BATCH) // 7 % 2).astype(np.int32)
    prop[BATCH // 3:BATCH // 2] = 1  # (a long run of one property, then changes again)
    net, x0, eps, args, sp = build(shape, convs, prop, 100 + i)
    pb = BoundProblem(*args, sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    pb.set_parts(1)
    if kernel.startswith("variant"):
        pb.set_conv_variant(int(kernel[-1]))
    elif kernel == "tiles":
        pb.set_conv_tiles(1)
    on = [(pb.conv_tiles(j + 1, 0), pb.conv_tiles(j + 1, 1)) for j in range(len(convs))]
    print("batch", BATCH_NETS[i], kernel, on, flush=True)
    rng = np.random.default_rng([82, i])
    pick = np.unique(np.concatenate([[0, 1, 6, 7, 8, BATCH // 3 - 1, BATCH // 3, BATCH // 2, BATCH - 8, BATCH - 7, BATCH - 1],
                                     rng.integers(0, BATCH, 5)]))
    orc, t = oracle(args, sp, pick, bc.dense_net(net.layers))
    m = orc.m
    uc = np.array([orc.unstable[int(p)].shape[0] for p in sp.dom_prop], np.int64) * m
    off = np.concatenate([[0], np.cumsum(uc)])
    assert off[-1] == pb.n_alpha
    ia = torch.from_numpy(np.concatenate([np.arange(off[b], off[b + 1]) for b in pick])).cuda()
    ib = torch.from_numpy((t[:, None] * m + np.arange(m)).reshape(-1)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(i)
    a = torch.rand(pb.n_alpha, device="cuda", generator=gen)
    b = torch.rand(pb.n_beta, device="cuda", generator=gen) * 0.5
    oa, obeta = a[ia].cpu().numpy().astype(np.float64), b[ib].cpu().numpy().astype(np.float64)

    def check(what):
        ref = [orc.grad(d, oa, obeta) for d in range(orc.B)]
        lb_ref = np.stack([r[0] for r in ref])
        assert guarded_rel(pb.eval(a, b)[pick].cpu().numpy(), lb_ref).max() <= TOL, what
        lb, ga, gb = pb.grad(a, b)
        assert guarded_rel(lb[pick].cpu().numpy(), lb_ref).max() <= TOL, what
        if orc.n_alpha:
            assert guarded_rel(ga[ia].cpu().numpy(), np.concatenate([r[1] for r in ref])).max() <= TOL, what
        if len(t):
            assert guarded_rel(gb[ib].cpu().numpy(), np.concatenate([r[2].reshape(-1) for r in ref])).max() <= TOL, what
        lbu, ub, _ = pb.upper(a, b)
        up_ref = np.stack([orc.upper(d, oa, obeta)[1] for d in range(orc.B)])
        assert guarded_rel(lbu[pick].cpu().numpy(), lb_ref).max() <= TOL, what
        assert guarded_rel(ub[pick].cpu().numpy(), up_ref).max() <= TOL, what
        a0, z0 = orc.default_alpha_flat(), np.zeros(orc.nnz * m)
        opt = np.stack([orc.optimize(d, a0, z0, bc.AdamConfig(iters=3))[0] for d in range(orc.B)])
        best, _ = pb.optimize(pb.alpha_init(), pb.zeros_beta(), iters=3)
        assert guarded_rel(best[pick].cpu().numpy(), opt).max() <= TOL, what
        return lb_ref, opt

    lb_ref, opt = check("box")
    pb.set_sound(1)
    lb = pb.eval(a, b)[pick].cpu().numpy()
    assert (lb <= lb_ref).all() and guarded_rel(lb, lb_ref).max() <= 1e-6
    # (the iterates are the float32 ones: the best of them by the bound with its margin)
    best, _ = pb.optimize(pb.alpha_init(), pb.zeros_beta(), iters=3)
    assert guarded_rel(best[pick].cpu().numpy(), opt).max() <= TOL
    pb.set_sound(0)
    pb.set_input_l2(x0, eps)
    orc.set_l2(x0, np.full(x0.shape[0], eps))
    check("ball")
    pb.close()
