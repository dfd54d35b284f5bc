"""Sweeps of one launch (small lattices): spins, cone angle and counters equal
those of the colour passes, the chain does not depend on how calls divide it,
and the averages equal the reference's."""
import numpy as np
import pytest

from tests import inputs

pytestmark = pytest.mark.gpu

# two sites a row, the fewest planes, tiles that divide nothing evenly, one tile
# across a row of 512, rows and planes on the tile's own edges, the largest sizes
SHAPES = [(4, 2, 2, "periodic"), (4, 6, 2, "antiperiodic"), (6, 4, 3, "open"), (16, 16, 16, "periodic"),
          (10, 34, 22, "antiperiodic"), (1024, 2, 4, "periodic"), (34, 30, 41, "open"), (64, 64, 64, "periodic"),
          (92, 80, 80, "periodic")]


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("nx,ny,nz,boundary", SHAPES)
def test_equals_the_passes(H, nx, ny, nz, boundary, precision, masked):
    kw = dict(inputs.random_params(nx + nz), precision=precision, seed=77, instance=3, init="random",
              boundary_z=boundary, bond_masks=masked)
    lats = [H.Lattice(nx, ny, nz, **kw) for _ in range(3)]
    if masked:
        m = inputs.random_bond_masks((nx, ny, nz), 0.3, 5)
        for g in lats:
            g.set_bond_masks(m)
    one, split, passes = lats
    passes.set_launch(1, 2)
    calls = [(7, False), (6, True), (1, True), (4, False)]
    for n, smp in calls:
        one.sweep(0.9, n, sample=smp)
        passes.sweep(0.9, n, sample=smp)
        for part in ([1] * n if n < 5 else [2, n - 3, 1]):
            split.sweep(0.9, part, sample=smp)
    assert np.array_equal(one.spins(), passes.spins())
    assert one.get_state() == split.get_state()
    a, b = one.observables(), passes.observables()
    for k in ("theta_deg", "sweeps_done", "samples", "accepted_last"):
        assert a[k] == b[k], k
    # FP32: sums of a thread's few terms round in FP32 before they meet in FP64
    tol = 1e-6 if precision == 32 else 1e-13
    assert np.allclose(a["mean_m"] + [a["mean_E"], a["mean_Eanis"]], b["mean_m"] + [b["mean_E"], b["mean_Eanis"]],
                       rtol=0, atol=10 * tol)
    assert a["status"] == H.OK


def test_cone_angle_clamps(H):
    for theta0, T, ends in ((179, 1e9, 180), (2, 1e-9, 1)):
        g = H.Lattice(8, 8, 8, precision=64, theta0_deg=theta0, init="aligned", seed=4)
        g.sweep(T, 9)
        assert g.observables()["theta_deg"] == ends


def test_averages_match_reference(H):
    from oracle import oracle as O
    kw = dict(inputs.random_params(8), seed=99, instance=1, init="random")
    g, o = H.Lattice(12, 10, 14, precision=64, boundary_z="antiperiodic", **kw), O.OracleLattice(
        12, 10, 14, boundary_z="antiperiodic", **kw)
    for n, smp in ((5, False), (8, True)):
        g.sweep(0.7, n, sample=smp)
        o.sweep(0.7, n, sample=smp)
    a, b = g.observables(), o.observables(0.7)
    assert np.max(np.abs(g.spins() - o.spins())) <= 1e-12
    for k in ("mean_m", "mean_E", "mean_Eanis"):
        assert np.allclose(a[k], b[k], rtol=1e-11, atol=1e-13), k
    assert np.allclose(a["var_m"], b["var_m"], rtol=1e-7, atol=1e-14)
    assert a["theta_deg"] == b["theta_deg"]


def test_non_finite_is_reported(H):
    g = H.Lattice(8, 8, 8, precision=32, init="random", seed=4)
    S = g.spins()
    S[100] = np.nan
    g.set_spins(S)
    g.sweep(0.9, 2, sample=True)
    S[100] = (0.0, 0.0, 1.0)
    g.set_spins(S)
    assert g.observables(check=False)["status"] == H.ENUMERIC
