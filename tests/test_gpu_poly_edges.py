"""The polynomial engine at the edges of what it takes: residuals at the
attainable accuracy, columns that fail their check, spectra with outliers,
served requests it declines (needs MI355X)."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O
import workloads as W
from oracle.solve import relative_l2

pytestmark = pytest.mark.gpu

TOL = 1e-11
U = 2.0 ** -53


@pytest.fixture(scope="module")
def ifl():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_07398_amd as m

    m.lib()
    return m


def _waves(m, noise=0.01):
    """A field far shorter than the filter scales below: its filtered part is
    small, and with it the accuracy that a residual can show."""
    lo, ext = m.coords.min(axis=0), np.ptp(m.coords, axis=0)
    x, y = 2.0 * np.pi * (m.coords[:, 0] - lo[0]) / ext[0], 2.0 * np.pi * (m.coords[:, 1] - lo[1]) / ext[1]
    return np.sin(3.0 * x) * np.cos(2.0 * y) + noise * np.random.default_rng(0).normal(size=len(x))


def _attainable(op, field, x, k, n):
    """8 u || |M phi| + |S| |x| || / ||M phi||, by rows, with |K| M^-1 |K| for
    |K M^-1 K| of order 2."""
    M = np.asarray(op.A)
    K = abs(sp.csr_matrix(op.K))
    kx = K @ np.abs(x)
    if n == 2:
        kx = K @ (kx / M)
    c = 0.5 / k ** (2 * n)
    return 8.0 * U * np.linalg.norm(M * np.abs(field) + M * np.abs(x) + c * kx) / np.linalg.norm(M * field)


@pytest.mark.parametrize("jitter", [0.2, 0.25, 0.3])
@pytest.mark.parametrize("cells", [64.0, 96.0])
def test_residual_at_the_attainable_accuracy(ifl, jitter, cells):
    """Converged means the tolerance or the attainable accuracy row by row: a
    mesh's smallest cells do not raise it for all rows. (1%: the sums' order
    and the 20 bits that the sizes of order 2 keep.)"""
    m = W.split_square(64, jitter=jitter)
    op = O.scalar_operator(m, 1)
    phi = _waves(m)
    k = 2.0 * np.pi / cells
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2)
    out, st = h.filter(phi, np.array([k]))
    assert st[0].status == 0
    assert st[0].rel_residual <= max(1e-12, 1.01 * _attainable(op, phi, out[0, 0], k, 2))
    h.close()


def test_fixed_width_handles_hold_no_patches(ifl):
    """The engine's patches are made with handles that leave the solver to the
    library, and otherwise by the first call that uses them (level 6: 40,962
    records of over 100 bytes)."""
    import torch

    s = W.icosphere(6)
    phi = np.random.default_rng(4).normal(size=s.n_vertices)
    ks = W.log_scales(s.h, 3, lam_max_cells=8.0)

    def held(**kw):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, 1, **kw)
        torch.cuda.synchronize()
        return h, before - torch.cuda.mem_get_info()[0]

    held()[0].close()  # the device's pools have grown
    h0, with_patches = held()
    ref, st0 = h0.filter(phi, ks)
    for kw in (dict(batch=8), dict(profile=1)):
        h, without = held(**kw)
        assert with_patches - without >= 4 << 20
        h.set_options(batch=0, profile=0)
        out, st = h.filter(phi, ks)
        assert np.array_equal(out, ref) and [x.iterations for x in st] == [x.iterations for x in st0]
        h.close()
    h0.close()


def _union_jack(n, jitter=0.1):
    """Periodic square of n x n cells (n even), the diagonals alternating: half
    of the vertices have 8 neighbours, half 4."""
    m = W.split_square(n, jitter=jitter)
    i, j = np.meshgrid(np.arange(n), np.arange(n), indexing="xy")
    a, b = (i + n * j).ravel(), ((i + 1) % n + n * j).ravel()
    d, c = (i + n * ((j + 1) % n)).ravel(), ((i + 1) % n + n * ((j + 1) % n)).ravel()
    even = ((i + j) % 2 == 0).ravel()
    t1 = np.where(even[:, None], np.stack([a, b, c], 1), np.stack([a, b, d], 1))
    t2 = np.where(even[:, None], np.stack([a, c, d], 1), np.stack([b, c, d], 1))
    return W.Mesh(coords=m.coords, tris=np.concatenate([t1, t2]).astype(np.int32), geometry=m.geometry, h=m.h,
                  period=m.period)


# On _waves of the 64 x 64 square, order 2 at 128 cells and more: the
# sequence's rounding (5e-11 of ||M phi||) stays above what FP64 can attain on
# a filtered field that small (5e-12), so the check sends the columns to CG.
FAILING = 2.0 * np.pi / np.array([128.0, 145.0, 165.0, 190.0])


def _counts(stats):
    return [(x.iterations, x.refinements, x.status) for x in stats]


def test_columns_that_fail_the_check_run_in_tiles(ifl):
    """All of a call's columns: bitwise the call of a handle that stays with CG
    (its launch events asked for), tile width and all."""
    m = W.split_square(64, jitter=0.2)
    fields = np.stack([_waves(m), 2.0 * _waves(m, 0.02), -_waves(m, 0.005)])
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2)
    cg = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2, profile=1)
    out, st = h.filter(fields, FAILING, raise_on_notconv=False)
    ref, rt = cg.filter(fields, FAILING, raise_on_notconv=False)
    assert all(x.refinements > 0 for x in rt)
    assert _counts(st) == _counts(rt)
    assert np.array_equal(out, ref)
    # some of them: the rest keep the engine's results, and those of all
    # fields, apart as their scales are, run in the tile of the whole call
    ks = np.concatenate([2.0 * np.pi / np.array([4.0]), FAILING[:1], 2.0 * np.pi / np.array([6.0, 8.0]), FAILING[1:2]])
    out, st = h.filter(fields, ks, raise_on_notconv=False)
    few, _ = h.filter(fields, ks[[0, 2, 3]])
    ref, rt = cg.filter(fields, ks, raise_on_notconv=False)
    assert np.array_equal(out[:, [0, 2, 3]], few) and np.array_equal(out[:, [1, 4]], ref[:, [1, 4]])
    assert [x.refinements > 0 for x in st] == 3 * [False, True, False, False, True]
    assert [x.iterations for x in st if x.refinements] == [rt[5 * f + j].iterations for f in range(3) for j in (1, 4)]
    up = np.sort(ks)
    _, st = h.filter(fields[0], up, raise_on_notconv=False)
    assert [x.refinements > 0 for x in st] == [True, True, False, False, False]
    assert list(h.spectrum(fields[0], up)[0]) == [x.energy for x in st]
    h.close()
    cg.close()


@pytest.mark.parametrize("device", [False, True])
def test_outputs_over_the_fields(ifl, device):
    """A call whose outputs take the place of its fields, with columns that
    pass the check and columns that do not: what it gives elsewhere."""
    import torch

    m = W.split_square(64, jitter=0.2)
    for n_fields, k in ((3, FAILING[0]), (3, 2.0 * np.pi / 8.0), (1, FAILING[1])):
        fields = np.stack([(1.0 + f) * _waves(m, 0.01 + 0.01 * f) for f in range(n_fields)])
        h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2)
        ref, rt = h.filter(fields, np.array([k]), raise_on_notconv=False)
        buf = torch.from_numpy(fields.copy()).cuda() if device else fields.copy()
        _, st = h.filter(buf, np.array([k]), out=buf.reshape(n_fields, 1, -1), raise_on_notconv=False)
        assert [x.status for x in st] == [x.status for x in rt]
        got = buf.cpu().numpy() if device else buf
        assert np.array_equal(got, ref[:, 0])
        h.close()


@pytest.mark.parametrize("nx,order,jitter,cells,sequence", [
    (64, 1, 0.2, 32.0, True), (64, 1, 0.2, 128.0, True), (64, 1, 0.2, 1000.0, False), (32, 1, 0.2, 2000.0, False),
    (64, 2, 0.2, 32.0, True), (64, 2, 0.3, 16.0, True), (64, 2, 0.3, 64.0, False), (256, 1, 0.2, 1000.0, False),
])
def test_scales_beyond_the_mesh_stay_with_cg(ifl, nx, order, jitter, cells, sequence):
    """Where CG has resolved every mode of the mesh long before the sequence
    ends, or rounding would fail the columns, the call is CG's alone: bitwise
    that of a handle whose launch events are asked for."""
    m = W.split_square(nx, jitter=jitter)
    phi, ks = _waves(m), np.array([2.0 * np.pi / cells])
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order)
    out, st = h.filter(phi, ks)
    assert (st[0].refinements == 0) == sequence
    h.set_options(profile=1)
    ref, rt = h.filter(phi, ks)
    if not sequence:
        assert np.array_equal(out, ref) and st[0].iterations == rt[0].iterations
    h.close()


def test_many_handles_share_a_work_space(ifl):
    """Handles used in turn hold one large work space (9 GB here) together, and
    give it back when they are closed."""
    import torch

    s = W.icosphere(8)
    s = s.with_mask(W.land_mask(s, 0.3))
    handles = [ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, 1) for _ in range(3)]
    L = s.n_vertices
    fields = torch.randn((8, L), dtype=torch.float64, generator=torch.Generator().manual_seed(2)).cuda()
    out = torch.zeros((8, 32, L), dtype=torch.float64, device="cuda")
    ks = W.log_scales(s.h, 32)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    start = free()
    handles[0].filter(fields, ks, out=out)
    one = start - free()
    assert 4 << 30 < one < 16 << 30
    first = out.clone()
    base = free()
    for h in handles[1:] + handles[:1]:
        h.filter(fields, ks, out=out)
        assert bool((out == first).all())
    assert base - free() < 1 << 30
    for h in handles:
        h.close()
    assert start - free() < out.numel() * 8 + (1 << 30)  # the clone, and change


def test_handles_on_several_threads(ifl):
    """Calls at the same time, each with a work space of its own."""
    import threading

    jobs = []
    for i, (nx, order, scales) in enumerate([(32, 1, 1), (64, 1, 8), (97, 2, 5), (150, 1, 17), (64, 2, 3)]):
        m = W.split_square(nx, jitter=0.2, ny=nx - 1)
        h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order)
        f = np.random.default_rng(i).normal(size=(1 + i % 3, nx * (nx - 1)))
        ks = W.log_scales(1.0, scales, lam_max_cells=16.0)
        jobs.append((h, f, ks, h.filter(f, ks)[0]))
    wrong = []

    def work(j):
        h, f, ks, ref = jobs[j]
        for _ in range(20):
            if not np.array_equal(h.filter(f, ks)[0], ref):
                wrong.append(j)

    threads = [threading.Thread(target=work, args=(j,)) for j in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for h, *_ in jobs:
        h.close()


def _serve(ifl, h, requests, slots=16, change=None):
    srv = ifl.Server(1 << 30, slots=slots)
    mid = srv.add(h)
    if change:
        h.set_options(**change)
    tickets = [srv.submit(mid, f, k) for f, k in requests]
    got = []
    for (t, _), (f, k) in zip(tickets, requests):
        code, st, out, _ = srv.wait(t, len(k))
        got.append((code, st, out))
    srv.close()
    return got


def _same(a, b):
    """Requests served alike: codes, iterations, replacements and bits."""
    for (ca, sa, oa), (cb, sb, ob) in zip(a, b):
        assert ca == cb
        assert _counts(sa) == _counts(sb)
        assert np.array_equal(oa, ob)


def test_served_requests_that_the_engine_declines_run_in_the_tile(ifl):
    """Among requests that it takes: bitwise those of a server of tiles, and the
    others those of the engine."""
    m = W.split_square(64, jitter=0.2)
    far = 2.0 * np.pi / np.array([1500.0, 1800.0, 2200.0])
    near = W.log_scales(1.0, 5, lam_max_cells=16.0)
    fields = [_waves(m, 0.01 * (1 + i)) for i in range(6)]
    mix = [(f, far if i in (1, 2, 4) else near) for i, f in enumerate(fields)]
    auto = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1)
    tile = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1, batch=16)
    got = _serve(ifl, auto, mix)
    _same([got[i] for i in (1, 2, 4)], _serve(ifl, tile, [mix[i] for i in (1, 2, 4)]))
    for i in (0, 3, 5):
        assert np.array_equal(got[i][2], auto.filter(fields[i], near)[0][0])
    # columns that miss the tolerance in the engine, beside columns that do not
    auto2 = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2)
    tile2 = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2, batch=16)
    ks = np.concatenate([2.0 * np.pi / np.array([4.0]), FAILING[:2], 2.0 * np.pi / np.array([6.0])])
    got = _serve(ifl, auto2, [(fields[0], ks), (fields[1], ks[[0, 3]])])
    ref = _serve(ifl, tile2, [(fields[0], ks)])
    assert [x.refinements > 0 for x in got[0][1]] == [False, True, True, False]
    assert np.array_equal(got[0][2][1:3], ref[0][2][1:3])
    assert [x.iterations for x in got[0][1][1:3]] == [x.iterations for x in ref[0][1][1:3]]
    assert np.array_equal(got[1][2], auto2.filter(fields[1], ks[[0, 3]])[0][0])
    # a mesh whose spectrum a few cells set is a tile's from the start
    m = W.split_square(64, jitter=0.35)
    wide = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1)
    wide_tile = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1, batch=16)
    reqs = [(_waves(m), near[:1]), (_waves(m), near[1:3])]
    _same(_serve(ifl, wide, reqs), _serve(ifl, wide_tile, reqs))
    for h in (auto, tile, auto2, tile2, wide, wide_tile):
        h.close()


def test_served_with_the_options_of_the_time_it_was_added(ifl):
    """Also requests that leave the engine for the tile, and one column at a
    time: the tolerance, precision and gamma of ifl_server_add."""
    m = W.split_square(64, jitter=0.2)
    far = 2.0 * np.pi / np.array([1500.0, 1800.0])
    change = dict(gamma=0.7, rtol=1e-6, max_iter=7, precision=ifl.IFL_MIXED)
    for order, kw in ((1, {}), (1, dict(batch=8)), (3, dict(solver=ifl.IFL_SOLVER_SHIFTED, max_iter=4000))):
        ks = far if order == 1 else 2.0 * np.pi / np.array([4.0, 6.0])
        h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order, **kw)
        ref = _serve(ifl, h, [(_waves(m), ks)])
        assert ref[0][0] == 0
        _same(_serve(ifl, h, [(_waves(m), ks)], change=change), ref)
        h.close()


def test_cancel_among_declined_requests(ifl):
    """Every request ends, done or cancelled, whichever way it was served."""
    m = W.split_square(64, jitter=0.2)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1)
    far = 2.0 * np.pi / np.array([1500.0, 1800.0, 2200.0])
    near = W.log_scales(1.0, 5, lam_max_cells=16.0)
    ref = {3: h.filter(_waves(m), far)[0][0], 5: h.filter(_waves(m), near)[0][0]}
    srv = ifl.Server(1 << 30, slots=4)
    mid = srv.add(h)
    for _ in range(3):
        ks = [far if i % 3 else near for i in range(24)]
        tickets = [srv.submit(mid, _waves(m), k)[0] for k in ks]
        srv.wait(tickets[0], len(ks[0]))
        srv.cancel()
        for t, k in zip(tickets[1:], ks[1:]):
            code, st, out, _ = srv.wait(t, len(k))
            assert code in (0, ifl.IFL_ECANCELED)
            if code == 0:
                assert relative_l2(out, ref[len(k)]) <= 1e-8
    code, _, out, _ = srv.wait(srv.submit(mid, _waves(m), near)[0], 5)
    assert code == 0 and np.array_equal(out, ref[5])
    srv.close()
    h.close()


def test_served_shifted_handle_holds_what_it_is_charged(ifl):
    """Order 2 with shifted solves on rows of 8 neighbours (no complex tile): the
    engine's work space alone, not the shifted solves' beside it."""
    import torch

    m = _union_jack(600)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 2, solver=ifl.IFL_SOLVER_SHIFTED)
    phi, ks = np.random.default_rng(1).normal(size=600 * 600), W.log_scales(1.0, 3, lam_max_cells=8.0)
    out, st = h.filter(phi, ks)
    assert all(x.refinements == 0 for x in st)
    srv = ifl.Server(1 << 30, slots=8)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    mid = srv.add(h)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= srv.query()["tiles"] + (8 << 20)
    code, _, got, _ = srv.wait(srv.submit(mid, phi, ks)[0], 3)
    assert code == 0 and np.array_equal(got, out[0])
    srv.close()
    h.close()


@pytest.mark.parametrize("order", [1, 2])
def test_constants_and_energies(ifl, order):
    """A constant is its own filtered field to a few roundings a step (c_0 .. c_m
    sum to 1 with alternating signs), and the energies of a field whose largest
    scale holds nearly all of it are exact to 2e-14 relative: truncation, a
    residual of 2e-14 (n = 2: 1e-14) at most, twice, where it is not 0."""
    s = W.icosphere(6)
    op = O.scalar_operator(s, order)
    ks = W.log_scales(s.h, 8, lam_max_cells=16.0)
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, order)
    out, st = h.filter(np.full(s.n_vertices, 3.0), ks)
    assert np.abs(out / 3.0 - 1.0).max() <= 4.0 * U * max(x.iterations for x in st)
    phi = s.coords[:, 2] / s.radius + 1e-3 * s.coords[:, 0] * s.coords[:, 1] / s.radius ** 2
    M = np.asarray(op.A)
    ref = np.array([0.5 * (M * x * x).sum() / M.sum() for x in O.filter_scalar(op, phi, ks)])
    e = h.spectrum(phi, ks)[0]
    assert np.abs(e / ref - 1.0).max() <= 4e-14
    h.close()


def _twelve(n):
    """Periodic triangular lattice of n x n vertices (n even), every triangle
    cut into six at its centre and its edges' midpoints: vertices of 12, 6 and
    4 neighbours, 6 n^2 of them in cells of one size."""
    x, ext = {}, np.array([float(n), n * np.sqrt(3.0) / 2.0])

    def vertex(p):
        q = np.mod(p, ext)
        q[np.isclose(q, ext, atol=1e-9)] = 0.0
        return x.setdefault((round(q[0], 6), round(q[1], 6)), len(x))

    tris = []
    for j in range(n):
        for i in range(n):
            o = np.array([i + 0.5 * (j % 2), j * np.sqrt(3.0) / 2.0])
            e, u = np.array([1.0, 0.0]), np.array([0.5, np.sqrt(3.0) / 2.0])
            for c in ([o, o + e, o + u], [o + e, o + e + u, o + u]):
                mid = vertex((c[0] + c[1] + c[2]) / 3.0)
                for a, b in ((0, 1), (1, 2), (2, 0)):
                    m = vertex(0.5 * (c[a] + c[b]))
                    tris += [[vertex(c[a]), m, mid], [m, vertex(c[b]), mid]]
    coords = np.array(sorted(x, key=x.get))
    return W.Mesh(coords=coords, tris=np.array(tris, np.int32), geometry=W.GEOM_PERIODIC, h=0.4, period=tuple(ext))


@pytest.mark.parametrize("kind,n,order", [
    ("8", 16, 1), ("8", 44, 2), ("8", 46, 1), ("8", 130, 2),      # one patch up to 2,048 units, rings
    ("12", 8, 1), ("12", 18, 2), ("12", 20, 1), ("12", 64, 1),
])
def test_rows_of_8_and_12_neighbours(ifl, kind, n, order):
    m = _union_jack(n) if kind == "8" else _twelve(n)
    L = len(m.coords)
    assert L == (n * n if kind == "8" else 6 * n * n)
    phi = np.random.default_rng(n).normal(size=(2, L))
    ks = W.log_scales(m.h, 5, lam_max_cells=12.0)
    op = O.scalar_operator(m, order)
    assert np.diff(sp.csr_matrix(op.K).indptr).max() == (9 if kind == "8" else 13)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order)
    out, st = h.filter(phi, ks)
    assert all(x.refinements == 0 for x in st)
    for f in range(2):
        ref = O.filter_scalar(op, phi[f], ks)
        assert max(relative_l2(out[f, j], ref[j]) for j in range(5)) <= TOL
    h.close()


@pytest.mark.parametrize("n", [16, 32, 34, 90])
def test_vertex_vectors_of_8_neighbours(ifl, n):
    """Turning blocks of 8 neighbours: one patch up to 1,024 units, rings."""
    m = _union_jack(n)
    u = np.random.default_rng(n).normal(size=(len(m.tris), 2))
    ks = W.log_scales(m.h, 3, lam_max_cells=10.0)
    ref = O.filter_vertex_vector(O.vertex_vector_operator(m, 1), u, ks)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_VECTOR, 1)
    out, st = h.filter(h.project_cells(u), ks)
    assert all(x.refinements == 0 for x in st)
    for j in range(3):
        assert relative_l2(out[0, j], np.asarray(ref[j]).reshape(-1)) <= TOL
    h.close()


@pytest.mark.parametrize("placement", ["voronoi", "circumcentre"])
@pytest.mark.parametrize("nx,order", [(24, 1), (24, 2), (70, 1), (70, 2)])
def test_other_placements_by_default(ifl, placement, nx, order):
    """Voronoi control volumes and cell scalars of acute triangles through the
    engine, in one patch and in rings."""
    m = W.split_square(nx, jitter=0.0)
    skew = m.coords - 0.5 * np.stack([m.coords[:, 1], np.zeros(nx * nx)], axis=1)
    m = W.Mesh(coords=skew * [1.0, np.sqrt(3.0) / 2.0], tris=m.tris, geometry=W.GEOM_PLANAR, h=1.0)
    tri = m.coords[m.tris]  # without the triangles across the seam
    inside = (np.ptp(tri[:, :, 0], axis=1) < 2.0) & (np.ptp(tri[:, :, 1], axis=1) < 2.0)
    m = W.Mesh(coords=m.coords, tris=m.tris[inside], geometry=W.GEOM_PLANAR, h=1.0)
    if placement == "voronoi":
        op, place, L = O.voronoi_operator(m, order), ifl.IFL_VORONOI_SCALAR, len(m.coords)
    else:
        op, place, L = O.circumcenter_operator(m, order), ifl.IFL_CIRCUMCENTER_SCALAR, len(m.tris)
    phi = np.random.default_rng(nx).normal(size=L)
    ks = W.log_scales(1.0, 4, lam_max_cells=8.0)
    ref = O.filter_scalar(op, phi, ks)
    h = ifl.prepare_mesh(m, place, order)
    out, st = h.filter(phi, ks)
    assert all(x.refinements == 0 for x in st)
    for j in range(4):
        assert relative_l2(out[0, j], ref[j]) <= TOL
    h.close()


def test_the_largest_mesh_by_default(ifl):
    """A level-9 call (2.6 million rows, 8 fields, more scales than a group) on
    the library's choice: each column's residual by ifl_apply, and a field's
    result not depending on its company."""
    import torch

    s = W.icosphere(9)
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, 1)
    g = torch.Generator().manual_seed(5)
    fields = torch.randn((8, s.n_vertices), dtype=torch.float64, generator=g).cuda()
    ks = W.log_scales(s.h, 18, lam_max_cells=24.0)
    out = torch.zeros((8, 18, s.n_vertices), dtype=torch.float64, device="cuda")
    _, st = h.filter(fields, ks, out=out)
    assert all(x.refinements == 0 and x.rel_residual <= 1e-12 for x in st)
    zero = torch.zeros(s.n_vertices, dtype=torch.float64, device="cuda")
    y, b = zero.clone(), zero.clone()
    h.apply(1e30, fields[3], y=b)  # c vanishes: M phi
    for j in (0, 9, 17):
        h.apply(float(ks[j]), out[3, j], y=y)
        assert float((y - b).norm() / b.norm()) <= 1e-12
    one = torch.zeros((1, 18, s.n_vertices), dtype=torch.float64, device="cuda")
    h.filter(fields[3].contiguous(), ks, out=one)
    assert bool((one[0] == out[3]).all())
    h.close()
