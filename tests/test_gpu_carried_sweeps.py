"""Sweeps whose finalize the next red pass carries: a call of several sweeps ends
in the state, bit for bit, of as many calls of one sweep, each of which closes
with a finalize launch."""
import pytest

from tests import inputs

pytestmark = pytest.mark.gpu

# one record a pass or a few; about a wave's and a work-group's worth; a group
# of 1024 and one plane more; the most a pass may leave (2048) and one plane more;
# rows of tiles and of two halo sites; FP64 with the most LDS a launch shape may take
SHAPES = [((4, 2, 2), "periodic", (1, 2)), ((16, 16, 16), "antiperiodic", (4, 1)), ((32, 16, 63), "open", (1, 1)),
          ((32, 16, 65), "open", (1, 1)), ((32, 16, 257), "open", (1, 1)), ((64, 64, 128), "antiperiodic", (1, 1)),
          ((64, 64, 129), "open", (1, 1)), ((64, 64, 256), "periodic", (1, 1)), ((64, 64, 257), "open", (1, 1)),
          ((1024, 6, 5), "open", (1, 2)), ((512, 4, 6), "periodic", (2, 3)), ((340, 4, 6), "periodic", (4, 2))]


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("kind", ["plain", "masked", "deep"])
@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("shape,boundary,launch", SHAPES)
def test_calls_of_one_sweep_end_alike(H, shape, boundary, launch, precision, kind):
    kw = dict(inputs.random_params(shape[0] + shape[2]), precision=precision, seed=78, instance=2, init="random",
              boundary_z=boundary, bond_masks=kind == "masked")
    one, ones = H.Lattice(*shape, **kw), H.Lattice(*shape, **kw)
    if precision == 64 and 2 * (256 * launch[0] + shape[0]) * 24 > 65536:
        pytest.skip("a launch shape the interface refuses")
    for g in (one, ones):
        g.set_launch(*launch)
        if kind == "masked":
            g.set_bond_masks(inputs.random_bond_masks(shape, 0.3, 5))
        if kind == "deep":
            g.set_prefetch(2)
    for n, smp in ((7, False), (5, True), (2, True), (3, False), (4, True)):
        one.sweep(0.9, n, sample=smp)
        for _ in range(n):
            ones.sweep(0.9, 1, sample=smp)
        assert one.get_state() == ones.get_state(), (n, smp)
    a, b = one.observables(), ones.observables()
    assert a == b and a["status"] == H.OK


@pytest.mark.parametrize("theta0,T,ends", [(178, 1e9, 180), (3, 1e-9, 1)])
def test_cone_angle_clamps(H, theta0, T, ends):
    g = H.Lattice(32, 32, 8, precision=32, theta0_deg=theta0, init="aligned", seed=4)
    g.set_launch(1, 1)
    g.sweep(T, 6)
    assert g.observables()["theta_deg"] == ends
