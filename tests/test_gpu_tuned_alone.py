"""A lattice whose launch shape the batch tuner set: swept alone it ends, bit for
bit, where the batch leaves it."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("precision", [32, 64])
def test_tuned_lattice_alone_equals_the_batch(H, precision):
    # small enough for a launch per sweep, were no shape set; and a larger one
    shapes, T = [(16, 16, 16), (34, 30, 18), (96, 88, 80)], [0.6, 0.9, 1.2]
    gs = [H.Lattice(*s, precision=precision, J=1.0, Ku=0.02, seed=5, instance=i, init="random")
          for i, s in enumerate(shapes)]
    B = H.Batch(gs)
    tuned = B.tune(T, trial_sweeps=1)
    assert [g.get_launch() for g in gs] == tuned
    begin = [g.get_state() for g in gs]
    for n, smp in ((3, False), (4, True)):
        B.sweep(T, n, sample=smp)
    end = [g.get_state() for g in gs]
    for g, t, s in zip(gs, T, begin):
        g.set_state(s)
        for n, smp in ((3, False), (4, True)):
            g.sweep(t, n, sample=smp)
    assert [g.get_state() == s for g, s in zip(gs, end)] == [True] * len(gs)
    B.close()
