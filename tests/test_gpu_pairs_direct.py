"""Constrained sweeps of small lattices (one thread per pair, no records):
spins and averages against the reference at the edges of the form, and a chain
that does not depend on how calls divide it."""
import numpy as np
import pytest

from tests import inputs

pytestmark = pytest.mark.gpu

# fewer pairs than a wave, one work-group and one pair more, cycle walking and none
# (a power of four sites per colour), the largest size and one row beyond it
SHAPES = [(4, 4, 2, "periodic"), (2, 6, 7, "open"), (16, 8, 8, "antiperiodic"), (16, 8, 10, "periodic"),
          (32, 32, 32, "periodic"), (64, 64, 64, "periodic"), (66, 64, 64, "antiperiodic")]


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("nx,ny,nz,boundary", SHAPES)
def test_fp64_matches_reference(H, nx, ny, nz, boundary, masked):
    from oracle import oracle as O
    kw = dict(inputs.random_params(nx + nz), seed=21, instance=2)
    eC = (0.6, 0.0, 0.8)
    S = inputs.tilted_spins(nx * ny * nz, 9, axis=eC)
    g = H.Lattice(nx, ny, nz, precision=64, boundary_z=boundary, bond_masks=masked, **kw)
    o = O.OracleLattice(nx, ny, nz, boundary_z=boundary, **kw)
    if masked:
        m = inputs.random_bond_masks((nx, ny, nz), 0.3, 5)
        g.set_bond_masks(m)
        o.set_bond_masks(m)
    g.set_spins(S)
    o.set_spins(S)
    for n, smp in ((2, False), (3, True)):
        g.constrained_sweep(0.7, eC, n, sample=smp)
        o.constrained_sweep(0.7, eC, n, sample=smp)
    assert np.max(np.abs(g.spins() - o.spins())) <= 1e-12
    a, b = g.observables(), o.observables(0.7)
    assert a["theta_deg"] == b["theta_deg"] and a["sweeps_done"] == 5 and a["torque_samples"] == 3
    for k in ("mean_m", "mean_E", "mean_Eanis"):
        assert np.allclose(a[k], b[k], rtol=1e-11, atol=1e-13), k
    assert np.allclose(a["mean_torque"], b["mean_torque"], rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("precision", [32, 64])
def test_calls_divide_a_chain_freely(H, precision):
    kw = dict(inputs.random_params(3), precision=precision, seed=5, init="aligned", init_dir=(0.6, 0.0, 0.8))
    one, split = H.Lattice(20, 18, 12, **kw), H.Lattice(20, 18, 12, **kw)
    for n, smp, parts in ((6, False, (1, 5)), (5, True, (2, 1, 2)), (4, False, (4,)), (3, True, (1, 1, 1))):
        one.constrained_sweep(0.6, (0.6, 0.0, 0.8), n, sample=smp)
        for p in parts:
            split.constrained_sweep(0.6, (0.6, 0.0, 0.8), p, sample=smp)
    assert one.get_state() == split.get_state()
