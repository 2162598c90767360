"""GPU tests of which kernel a conv layer runs: every variant and the register
tiles can be asked for apart from one another, what a plan falls back to fits
its limits, and each choice meets the FP64 oracle (1e-4 guarded relative, as for
the other parity tests)."""
import pytest

from paper_2103_06624_amd import synth
from tests import test_gpu_conv_tiles as tiles

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def conv_layers(net):
    return [i + 1 for i, ly in enumerate(net.layers) if ly.kind == synth.CONV]


def problem(i, n_dom):
    from paper_2103_06624_amd.api import BoundProblem
    net, xlo, xhi, x0, eps, C, lo, up, args, orc = tiles.build(i, n_dom)
    return net, orc, BoundProblem(net.layers, xlo, xhi, C, lo, up, *args)


@pytest.mark.parametrize("i", range(len(tiles.NETS)))
def test_variants_and_tiles_are_chosen_apart(i):
    """A forced variant takes the register tiles off (variant 2 is the
    subdomain-major kernel itself); the tiles go on over any variant, in both
    directions of a first layer or in neither."""
    net, orc, pb = problem(i, 5)
    print("conv plans", tiles.NETS[i], flush=True)
    layers = conv_layers(net)
    on = lambda: [(pb.conv_tiles(j, 0), pb.conv_tiles(j, 1)) for j in layers]
    default = on()
    assert default[0][0] == default[0][1]
    for var in range(pb.num_conv_variants()):
        pb.set_conv_variant(var)
        ran = [(pb.conv_variant(j, 0), pb.conv_variant(j, 1)) for j in layers]
        if var < 2 or (i == 3 and var == 2):  # (where the variant runs every layer, or the first two)
            assert ran[:2] == [(var, var)] * len(ran[:2]), (var, ran)
            assert on()[:2] == [(0, 0)] * len(ran[:2]), (var, on())
        tiles.check(orc, pb, (tiles.NETS[i], "variant", var, ran))
    pb.set_conv_tiles(1)
    assert on()[0][0] == on()[0][1]
    assert all(a >= b for f, g in zip(on(), default) for a, b in zip(f, g))
    tiles.check(orc, pb, (tiles.NETS[i], "tiles", on()))
    pb.set_conv_variant(-1)
    pb.set_conv_tiles(0)
    assert not any(x for f in on() for x in f)
    tiles.check(orc, pb, (tiles.NETS[i], "no tiles"))
    pb.set_conv_tiles(-1)
    assert on() == default
    for bad in (-2, 2):
        with pytest.raises(Exception):
            pb.set_conv_tiles(bad)
    pb.autotune()
    assert on()[0][0] == on()[0][1]
    tiles.check(orc, pb, (tiles.NETS[i], "tuned", on()))
    pb.close()


def test_a_variant_past_the_lds_limit_is_not_taken():
    """A first layer of 96 channels on 8x8: register tiles exist for its
    back-substitution only, so neither direction runs on them, and the weights
    (24 KB) do not fit beside the row in 64 KB of LDS: the variants that would
    hold them there leave the layer its default."""
    from oracle import batch as ob
    from oracle import beta_crown as bc
    from paper_2103_06624_amd.api import BoundProblem
    import numpy as np
    rng = np.random.default_rng(79)
    net = synth.cnn(rng, (3, 16, 16), [(96, 4, 2, 1)], [16, 10])
    x0 = rng.uniform(0, 1, size=(1, net.dims[0])).astype(np.float32)
    eps = 2.0 / 255.0
    xlo, xhi = synth.box(x0, eps)
    C = synth.margin_spec(0, 10)[None].astype(np.float32)
    net64 = bc.dense_net(net.layers)
    # root bounds over the whole balls too: the box around x0, not clipped
    lo, up = bc.outward_f32(*ob.root_bounds_all(net64, x0 - np.float32(eps), x0 + np.float32(eps)))
    sp = synth.sample_splits(1, net.dims, lo, up, np.zeros(4, np.int32), (0, 5))
    args = (sp.dom_prop, sp.split_ptr, sp.layer, sp.neuron, sp.side)
    orc = ob.OracleProblem(net.layers, xlo, xhi, C, lo, up, *args, net64=net64)
    pb = BoundProblem(net.layers, xlo, xhi, C, lo, up, *args)
    default = [pb.conv_variant(1, d) for d in (0, 1)]
    print("96 channels: default", default, flush=True)
    assert [pb.conv_tiles(1, d) for d in (0, 1)] == [0, 0]
    for var in (0, 2):
        pb.set_conv_variant(var)
        assert pb.conv_variant(1, 0) == default[0], var
        tiles.check(orc, pb, ("96 channels", var))
    pb.close()
