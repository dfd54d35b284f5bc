"""The launch shape that a lattice of a batch takes where none was set, by its size
and the length of its rows: the lattice ends where it ends alone in that shape."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


# both sides of the lines in the number of spins; rows of 254, 256 and 260 colour sites
@pytest.mark.parametrize("shape,precision,default", [
    ((128, 128, 128), 32, (1, 4)), ((130, 128, 128), 32, (1, 8)), ((256, 256, 212), 32, (1, 8)),
    ((256, 256, 214), 32, (2, 16)), ((512, 20, 36), 32, (1, 4)), ((508, 20, 36), 64, (2, 8)),
    ((512, 20, 36), 64, (2, 16)), ((520, 20, 36), 64, (1, 8)), ((520, 20, 24), 64, (1, 4))])
def test_default_of_a_batch(H, shape, precision, default):
    kw = dict(precision=precision, J=1.0, Ku=0.02, seed=5, init="random")
    alone, inb = H.Lattice(*shape, **kw), H.Lattice(*shape, **kw)
    alone.set_launch(*default)
    other = H.Lattice(8, 8, 8, **dict(kw, instance=3))
    B = H.Batch([other, inb])
    for n, smp in [(1, False), (2, True)]:
        B.sweep(0.8, n, sample=smp)
        alone.sweep(0.8, n, sample=smp)
    same = alone.get_state() == inb.get_state()
    assert same
    B.close()
