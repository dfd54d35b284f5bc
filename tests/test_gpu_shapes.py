"""Default launch shapes: the spins are those of any other shape, the shapes
stay within one round of the device, and a lattice of a batch whose shape was
not set ends where it ends alone with the batch's default shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# around the lines of the rule: one slab per plane, 256-site blocks just full
# and just not, two sites per thread, the 16-plane cap, an odd open film, nx = 1024
SHAPES = [(2, 2, 2), (16, 16, 16), (34, 30, 18), (64, 64, 64), (66, 64, 64), (128, 128, 20), (320, 320, 12),
          (1024, 256, 6), (1024, 1024, 4)]


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2103_03517_amd as H
    assert torch.cuda.is_available(), "these tests need the GPU"
    H.lib()
    return H


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("shape", SHAPES)
def test_default_shape_gives_the_same_spins(H, shape, precision):
    kw = dict(precision=precision, J=1.0, Ku=0.02, Kc=-0.03, h=(0.01, 0.0, 0.02), seed=11, init="random")
    g, ref = H.Lattice(*shape, **kw), H.Lattice(*shape, **kw)
    spt, zc = g.get_launch()
    columns = -(-(shape[0] // 2 * shape[1]) // (256 * spt))
    slabs = -(-shape[2] // zc)
    assert zc <= 16 and (columns * slabs <= (1024 if precision == 32 else 512) or zc == min(16, shape[2]))
    ref.set_launch(1, 3)
    for lat in (g, ref):
        lat.sweep(0.9, 3, sample=True)
        lat.sweep(0.9, 2)
    assert np.array_equal(g.spins(), ref.spins())
    a, b = g.observables(), ref.observables()
    assert a["theta_deg"] == b["theta_deg"] and a["accepted_last"] == b["accepted_last"]
    assert np.allclose(a["mean_m"], b["mean_m"], rtol=0, atol=1e-6 if precision == 32 else 1e-13)


@pytest.mark.parametrize("shape,precision,default", [((16, 16, 16), 32, (1, 4)), ((64, 64, 64), 64, (1, 4)),
                                                     ((66, 64, 64), 64, (2, 8)), ((66, 64, 64), 32, (1, 4))])
def test_batch_default_shape(H, shape, precision, default):
    kw = dict(precision=precision, J=1.0, Ku=0.02, seed=5, init="random")
    alone, inb, other = H.Lattice(*shape, **kw), H.Lattice(*shape, **kw), H.Lattice(8, 8, 8, **dict(kw, instance=3))
    alone.set_launch(*default)
    B = H.Batch([other, inb])
    for n, smp in [(2, False), (3, True)]:
        B.sweep(0.8, n, sample=smp)
        alone.sweep(0.8, n, sample=smp)
    assert alone.get_state() == inb.get_state()
    B.close()


# one plane per thread, a ragged last slab, eight planes and more, thin
# lattices whose slabs share a work-group, one plane, several record groups
@pytest.mark.parametrize("shape,boundary", [((2, 2, 2), "periodic"), ((6, 4, 38), "antiperiodic"), ((2, 2, 2050), "periodic"),
                                            ((16, 18, 7), "open"), ((34, 10, 1), "open"), ((130, 128, 70), "antiperiodic"),
                                            ((256, 254, 190), "periodic")])
@pytest.mark.parametrize("precision", [32, 64])
def test_measurement_against_numpy(H, shape, boundary, precision):
    nx, ny, nz = shape
    kw = dict(J=1.1, Ku=0.03, eu=(0.2, -0.4, 0.9), Kc=-0.02, h=(0.01, 0.02, -0.015))
    g = H.Lattice(*shape, precision=precision, boundary_z=boundary, init="random", seed=7, **kw)
    o = g.observables()
    S = g.spins().reshape(nz, ny, nx, 3)
    e = np.asarray(kw["eu"]) / np.linalg.norm(kw["eu"])
    up = np.roll(S, -1, axis=0)
    up[-1] *= {"periodic": 1.0, "antiperiodic": -1.0, "open": 0.0}[boundary]
    ex = -kw["J"] * (S * (np.roll(S, -1, axis=2) + np.roll(S, -1, axis=1) + up)).sum()
    q = S ** 2
    un = -kw["Ku"] * ((S @ e) ** 2).sum()
    cu = kw["Kc"] * (q[..., 0] * q[..., 1] + q[..., 0] * q[..., 2] + q[..., 1] * q[..., 2]).sum()
    ze = -(S @ np.asarray(kw["h"])).sum()
    grad = 2 * kw["Ku"] * (S @ e)[..., None] * e - 2 * kw["Kc"] * S * (q.sum(-1, keepdims=True) - q)
    def total(v):       # pairwise sums: numpy adds a strided axis term after term
        return np.array([np.ascontiguousarray(v[..., i]).sum() for i in range(3)])

    tq = total(np.cross(S, grad))
    # each of N terms rounded a few times (unit roundoff u), errors of random sign, the sums in FP64
    tol = 40 * np.sqrt(g.n) * (2.0 ** -24 if precision == 32 else 2.0 ** -50)
    assert np.allclose(o["M"], total(S), rtol=0, atol=tol)
    assert np.allclose([o["E_exch"], o["E_uni"], o["E_cub"], o["E_zee"]], [ex, un, cu, ze], rtol=1e-7 if precision == 32 else 1e-14,
                       atol=tol)
    assert np.allclose(o["torque"], tq, rtol=0, atol=tol)
    B = H.Batch([H.Lattice(4, 4, 4, precision=precision, seed=2), g])
    b = B.observables()[1]
    assert all(b[k] == o[k] for k in b)
    B.close()


@pytest.mark.parametrize("shape", [(2, 2, 2), (6, 10, 4), (258, 2, 6), (64, 36, 30)])
@pytest.mark.parametrize("precision", [32, 64])
def test_spins_in_site_order(H, shape, precision):
    """Spins read back are the ones given, divided by their length as numpy
    does it in double precision and rounded to the lattice's; zero and
    non-finite vectors are kept."""
    n = shape[0] * shape[1] * shape[2]
    v = np.random.default_rng(n).normal(size=(n, 3)) * 3.0
    v[1], v[2], v[3, 1] = 0.0, (np.inf, 1.0, -2.0), np.nan
    n2 = (v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1]) + v[:, 2] * v[:, 2]
    with np.errstate(divide="ignore", invalid="ignore"):
        inv = np.where((n2 > 0) & np.isfinite(n2), 1.0 / np.sqrt(n2), 1.0)
    g = H.Lattice(*shape, precision=precision)
    g.set_spins(v)
    want = v * inv[:, None]
    if precision == 32:
        want = want.astype(np.float32).astype(np.float64)
    assert np.array_equal(g.spins(), want, equal_nan=True)
    # the component arrays at the head of the workspace: site 2k + p, colour (x + y + z) & 1
    rs, half = precision // 8, n // 2
    pitch = (half * rs + 255) // 256 * 256
    raw = g.workspace[:6 * pitch].cpu().numpy().view(np.float32 if rs == 4 else np.float64).reshape(6, -1)[:, :half]
    x, y, z = (i.T.reshape(-1) for i in np.indices(shape))
    for c in (0, 1):
        assert np.array_equal(raw[3 * c:3 * c + 3].T, want[(x + y + z) % 2 == c], equal_nan=True)


# rows above 256 colour sites (tiles): just above, a prime width, the widest; rows
# that a tile's height does not divide, one row of tiles, thin and thick slabs
@pytest.mark.parametrize("nx,ny,nz,boundary", [(514, 4, 2, "periodic"), (526, 18, 4, "antiperiodic"),
                                               (1024, 2, 6, "periodic"), (1024, 46, 5, "open"), (640, 34, 3, "open")])
@pytest.mark.parametrize("masked", [False, True])
def test_tiles_match_reference(H, nx, ny, nz, boundary, masked):
    from oracle import oracle as O
    from tests import inputs
    kw = dict(inputs.random_params(nx), seed=31, instance=4)
    S = inputs.random_unit_spins(nx * ny * nz, 12)
    o = O.OracleLattice(nx, ny, nz, boundary_z=boundary, **kw)
    m = inputs.random_bond_masks((nx, ny, nz), 0.3, 5)
    if masked:
        o.set_bond_masks(m)
    o.set_spins(S)
    accepted = [o.sweep(0.8, sample=True) for _ in range(3)][-1]
    ref = o.observables(0.8)
    for spt, zc, depth in [(1, 1, 1), (2, 3, 1), (4, 16, 1)] + ([] if masked else [(1, 2, 2), (2, 4, 2)]):
        g = H.Lattice(nx, ny, nz, precision=64, boundary_z=boundary, bond_masks=masked, **kw)
        if masked:
            g.set_bond_masks(m)
        g.set_spins(S)
        if 2 * (256 * spt + nx) * 24 > 65536:       # refused, as ever: the line of whole rows in LDS
            with pytest.raises(H.HmcError):
                g.set_launch(spt, zc)
            continue
        g.set_launch(spt, zc)
        g.set_prefetch(depth)
        g.sweep(0.8, 3, sample=True)
        assert np.max(np.abs(g.spins() - o.spins())) <= 1e-12, (spt, zc, depth)
        a = g.observables()
        assert a["accepted_last"] == accepted and a["theta_deg"] == ref["theta_deg"]
        for k in ("mean_m", "mean_E"):
            assert np.allclose(a[k], ref[k], rtol=1e-11, atol=1e-13), k


def test_tiles_in_a_batch_equal_tiles_alone(H):
    kw = dict(precision=32, J=1.0, Ku=0.02, Kc=0.01, seed=9, init="random")
    shapes = [((520, 6, 4), (4, 2)), ((1024, 10, 2), (1, 1)), ((12, 8, 6), (2, 3)), ((400, 6, 4), (1, 3))]
    alone, inb = ([H.Lattice(*sh, instance=i, **kw) for i, (sh, _) in enumerate(shapes)] for _ in range(2))
    for lats in (alone, inb):
        for g, (_, c) in zip(lats, shapes):
            g.set_launch(*c)
    B = H.Batch(inb)
    for n, smp in [(3, False), (4, True)]:
        B.sweep(0.8, n, sample=smp)
        for g in alone:
            g.sweep(0.8, n, sample=smp)
    for a, b in zip(alone, inb):
        assert a.get_state() == b.get_state()
    B.close()
