"""Which lattices take a launch per sweep: those whose tiles cost less than the
passes do.  Either way the spins, cone angle and counters are those of the
passes, and the chain does not depend on how calls divide it."""
import numpy as np
import pytest

from tests import inputs

pytestmark = pytest.mark.gpu

# (shape, boundary, precisions): rows of two sites, two and three planes, a
# lattice of odd thickness; tiles that divide nothing evenly; the longest rows
# that are taken at a small and at a larger size; one tile to a compute unit and
# (FP64) two, whose counts take two loads a thread; the most spins; 16 planes a tile
WHOLE = [((4, 32, 16), "periodic", (32, 64)), ((16, 8, 2), "antiperiodic", (32, 64)), ((4, 8, 2), "periodic", (64,)),
         ((16, 16, 3), "open", (32, 64)), ((34, 30, 41), "open", (32, 64)), ((326, 6, 4), "periodic", (32,)),
         ((326, 16, 16), "antiperiodic", (32,)), ((162, 10, 10), "periodic", (64,)), ((64, 64, 64), "periodic", (32, 64)),
         ((66, 66, 66), "antiperiodic", (64,)), ((92, 80, 80), "periodic", (32,)), ((8, 8, 8000), "open", (32,))]
# long rows, thin lattices of long rows, more spins or rows than the rule takes,
# too little scratch for a second copy
PASSES = [((272, 32, 64), "periodic", (32,)), ((320, 32, 32), "open", (32,)), ((240, 40, 30), "periodic", (32,)),
          ((200, 50, 50), "antiperiodic", (32,)), ((256, 256, 8), "periodic", (32,)), ((96, 64, 40), "periodic", (64,)),
          ((92, 82, 80), "periodic", (32,)), ((68, 68, 66), "periodic", (64,)), ((1024, 2, 4), "periodic", (32, 64)),
          ((4, 2, 2), "periodic", (32, 64)), ((2, 16, 16), "periodic", (32, 64)), ((16, 16, 1), "open", (32, 64))]
# sampled sweeps whole, unsampled ones in passes
SAMPLED = [((256, 32, 32), "open", (32,)), ((128, 68, 68), "antiperiodic", (32,))]
CASES = [(s, b, p, w) for cases, w in ((WHOLE, (True, True)), (PASSES, (False, False)), (SAMPLED, (False, True)))
         for s, b, ps in cases for p in ps]


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("shape,boundary,precision,whole", CASES)
def test_route_and_result(H, shape, boundary, precision, whole, masked):
    kw = dict(inputs.random_params(shape[0] + shape[2]), precision=precision, seed=79, instance=1, init="random",
              boundary_z=boundary, bond_masks=masked)
    one, split, passes = lats = [H.Lattice(*shape, **kw) for _ in range(3)]
    if masked:
        m = inputs.random_bond_masks(shape, 0.3, 5)
        for g in lats:
            g.set_bond_masks(m)
    passes.set_launch(1, 2)
    for n, smp in ((3, False), (4, True), (1, True)):
        one.set_timing(True)
        one.sweep(0.9, n, sample=smp)
        assert one.read_timing()["pass"]["count"] == (n if whole[smp] else 2 * n)
        one.set_timing(False)
        for part in [1] * n:
            split.sweep(0.9, part, sample=smp)
        passes.sweep(0.9, n, sample=smp)
    assert one.get_state() == split.get_state()
    assert np.array_equal(one.spins(), passes.spins())
    a, b = one.observables(), passes.observables()
    for k in ("theta_deg", "sweeps_done", "samples", "accepted_last"):
        assert a[k] == b[k], k
    # FP32: sums of a thread's few terms round in FP32 before they meet in FP64
    tol = 1e-5 if precision == 32 else 1e-12
    assert np.allclose(a["mean_m"] + [a["mean_E"]], b["mean_m"] + [b["mean_E"]], rtol=0, atol=tol)
