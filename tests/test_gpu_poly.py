"""The polynomial engine of ifl_filter (tile width left to the library)
against the FP64 oracle, at the sizes where its patches, slots, scale groups
and row widths change (needs MI355X).

Bars: the library's own, relative L2 <= 1e-11 in FP64: the residual is held
to a twentieth of rtol = 1e-12, and the system's smallest eigenvalue is that
of the mass."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle.solve import relative_l2

pytestmark = pytest.mark.gpu

TOL = 1e-11


@pytest.fixture(scope="module")
def ifl():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_07398_amd as m

    m.lib()
    return m


def _delaunay(n, seed=3):
    """Random points: rows of very different widths (up to 12 neighbours and
    beyond) and cells of very different sizes."""
    from scipy.spatial import Delaunay

    x = np.random.default_rng(seed).uniform(0.0, 30.0, (n, 2))
    return W.Mesh(coords=x, tris=Delaunay(x).simplices.astype(np.int32), geometry=W.GEOM_PLANAR, h=30.0 / n ** 0.5)


def _noise(n, seed):
    return np.random.default_rng(seed).normal(size=n)


def _sequence_ran(st, n_fields, n_scales):
    """The engine's iterations are the degree of a scale's polynomial, the
    same for every field."""
    it = np.array([s.iterations for s in st]).reshape(n_fields, n_scales)
    return bool(np.all(it == it[0])) and all(s.refinements == 0 for s in st)


@pytest.mark.parametrize("nx,ny,order,scales", [
    (3, 3, 1, 2), (32, 32, 1, 1), (33, 32, 1, 3), (64, 32, 2, 5), (64, 33, 1, 8), (64, 64, 2, 4),  # one patch
    (65, 64, 1, 16), (97, 61, 2, 3), (150, 149, 1, 17), (211, 160, 1, 2),                          # rings
])
def test_planar_sizes(ifl, nx, ny, order, scales):
    m = W.split_square(nx, jitter=0.2, ny=ny)
    fields = np.stack([_noise(nx * ny, 11 + f) for f in range(3)])
    ks = W.log_scales(1.0, scales, lam_max_cells=16.0)
    op = O.scalar_operator(m, order)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order)
    out, st = h.filter(fields, ks)
    assert _sequence_ran(st, 3, scales)
    for f in range(3):
        ref = O.filter_scalar(op, fields[f], ks)
        for j in range(scales):
            assert relative_l2(out[f, j], ref[j]) <= TOL, (f, j)
            assert st[f * scales + j].status == 0
    again, _ = h.filter(fields[1], ks)  # a field's result does not depend on its company
    assert np.array_equal(again[0], out[1])
    h.close()


@pytest.mark.parametrize("scales", [18, 20, 24, 32, 37])
def test_scale_groups(ifl, scales):
    """More than 16 scales: a full group and the next, of every width, are
    summed together; a third one by itself."""
    m = W.split_square(65, jitter=0.2, ny=64)
    field = _noise(65 * 64, 21)
    ks = W.log_scales(1.0, scales, lam_max_cells=16.0)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1)
    out, st = h.filter(field, ks)
    assert _sequence_ran(st, 1, scales)
    ref = O.filter_scalar(O.scalar_operator(m, 1), field, ks)
    for j in range(scales):
        assert relative_l2(out[0, j], ref[j]) <= TOL, j
    h.close()


@pytest.mark.parametrize("n", [60, 500, 2500])
def test_wide_and_uneven_rows(ifl, n):
    """Random Delaunay meshes: 8 to 12 neighbours a row; the widest, and
    those whose small cells would need too many products, stay with CG."""
    m = _delaunay(n)
    phi = _noise(n, 5)
    ks = W.log_scales(m.h, 3, lam_max_cells=8.0)
    ref = O.filter_scalar(O.scalar_operator(m, 1), phi, ks)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1)
    out, st = h.filter(phi, ks)
    for j in range(3):
        assert relative_l2(out[0, j], ref[j]) <= TOL and st[j].status == 0
    h.close()


@pytest.mark.parametrize("placement", ["cell", "vertex"])
@pytest.mark.parametrize("level,scales", [(2, 3), (3, 1), (4, 4), (5, 2)])
def test_vector_sizes(ifl, placement, level, scales):
    s = W.icosphere(level)
    wet = np.ones(s.n_vertices, np.uint8)
    wet[np.abs(s.coords[:, 2] / s.radius) > np.sin(np.radians(75))] = 0
    s = s.with_mask(wet)
    u = _noise(2 * s.n_triangles, 3).reshape(-1, 2)
    ks = W.log_scales(s.h, scales, lam_max_cells=12.0)
    if placement == "cell":
        h = ifl.prepare_mesh(s, ifl.IFL_CELL_VECTOR, 1)
        f = u.reshape(-1)
        ref = O.filter_vector(O.vector_operator(s, 1), u, ks)
    else:
        h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_VECTOR, 1)
        f = h.project_cells(u)
        ref = O.filter_vertex_vector(O.vertex_vector_operator(s, 1), u, ks)
    out, st = h.filter(np.stack([f, 2.0 * f]), ks)
    assert _sequence_ran(st, 2, scales)
    for j in range(scales):
        assert relative_l2(out[0, j], np.asarray(ref[j]).reshape(-1)) <= TOL
        assert np.array_equal(out[1, j], 2.0 * out[0, j])  # a power of two scales every step exactly
    h.close()


def test_limits_and_bad_input(ifl):
    """A cap below the degree leaves the call to CG and its status; a NaN
    leaves the outputs as they were; a zero field is a zero result."""
    import torch

    m = W.split_square(48, jitter=0.2)
    phi = _noise(48 * 48, 9)
    ks = W.log_scales(1.0, 3)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1, max_iter=5)
    _, st = h.filter(phi, ks[:1], raise_on_notconv=False)
    assert st[0].status == ifl.IFL_ENOTCONV and st[0].iterations == 5
    h.set_options(max_iter=20000)
    out, st = h.filter(np.stack([phi, 0.0 * phi]), ks)
    assert np.all(out[1] == 0.0) and all(x.iterations == 0 and x.status == 0 for x in st[3:])
    bad = phi.copy()
    bad[17] = np.nan
    for dev in (False, True):
        o = np.full((2, 3, phi.size), 7.0)
        f = np.stack([phi, bad])
        if dev:
            o, f = torch.from_numpy(o).cuda(), torch.from_numpy(f).cuda()
        with pytest.raises(ifl.IflError) as e:
            h.filter(f, ks, out=o)
        assert e.value.status == ifl.IFL_EINVAL and bool((o == 7.0).all())
    host, _ = h.filter(phi, ks)
    d = torch.zeros((1, 3, phi.size), dtype=torch.float64, device="cuda")
    h.filter(torch.from_numpy(phi).cuda(), ks, out=d)
    assert np.array_equal(d.cpu().numpy(), host)
    h.close()


@pytest.mark.parametrize("order,slots,scales", [(1, 4, 40), (2, 8, 19), (1, 64, 5)])
def test_served_in_several_sequences(ifl, order, slots, scales):
    """A request whose scales outgrow the worker's work space runs in several
    sequences: bitwise the fields of ifl_filter on the same handle; their
    energies up to the order of the sums (positive terms through trees of at
    most 32 additions: 64 u), and bitwise those of the same request without
    outputs."""
    s = W.icosphere(5)
    s = s.with_mask(W.land_mask(s, 0.3))
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, order, precision=ifl.IFL_MIXED)
    phi = _noise(s.n_vertices, 4)
    ks = W.log_scales(s.h, scales, lam_max_cells=20.0)[::-1].copy()
    out, st = h.filter(phi, ks)
    srv = ifl.Server(1 << 30, slots=slots)
    mid = srv.add(h)
    t, _ = srv.submit(mid, phi, ks)
    code, stats, o, _ = srv.wait(t, scales)
    assert code == 0 and np.array_equal(o, out[0])
    for x, y in zip(stats, st):
        assert abs(x.energy - y.energy) <= 64 * 2.0 ** -53 * y.energy
    t, _ = srv.submit(mid, phi, ks, spectrum_only=True)
    code, alone, _, _ = srv.wait(t, scales)
    assert code == 0 and [x.energy for x in alone] == [x.energy for x in stats]
    srv.close()
    h.close()
