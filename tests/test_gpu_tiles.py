"""CG tiles of the library's own width, and served tiles, on handles that
stay with CG: launch events asked for (profile = 1), order 3, or a fixed width
(needs MI355X). Bars as for the other tiles: relative L2 1e-11 in FP64, 1e-9
mixed."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle.solve import relative_l2

pytestmark = pytest.mark.gpu

TOL = {0: 1e-11, 1: 1e-9}


@pytest.fixture(scope="module")
def ifl():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_07398_amd as m

    m.lib()
    return m


def _sphere(level):
    s = W.icosphere(level)
    return s.with_mask(W.land_mask(s, 0.3))


def _in_tiles(stats):
    """CG in tiles: whole chunks of 4 iterations, each with its replacement."""
    return all(x.iterations % 4 == 0 and 0 < x.refinements <= x.iterations // 4 + 1 for x in stats)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("order,kw", [(1, dict(profile=1)), (3, {})])
def test_tuned_width(ifl, order, kw, precision):
    s = _sphere(5)
    fields = np.stack([W.sphere_k3_field(s, 1001 + i, n_waves=256) for i in range(11)])
    ks = W.log_scales(s.h, 6, lam_max_cells=32.0 if order == 1 else 6.0)
    op = O.scalar_operator(s, order)
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, order, precision=precision, **kw)
    t = h.autotune()
    assert t["batch"] in (16, 32, 64)
    out, st = h.filter(fields, ks)
    assert _in_tiles(st) and np.array_equal(h.filter(fields, ks)[0], out)
    if order == 1:
        width = t["batch"]
        while width * 4 > len(st):
            width //= 2
        assert f", {width}, true" in h.profile_kernel()
    for f in (0, 10):
        ref = O.filter_scalar(op, fields[f], ks)
        assert max(relative_l2(out[f, j], ref[j]) for j in range(6)) <= TOL[precision]
    h.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_tail_moves_to_narrower_tiles(ifl, precision):
    """128 columns of very different lengths in the library's width (32, then 8,
    then 2 slots) against a tile of 32 that they do not leave, and the oracle."""
    s = _sphere(5)
    fields = np.stack([W.sphere_k3_field(s, 6000 + i, n_waves=128) for i in range(8)])
    ks = W.log_scales(s.h, 16)
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, 2, precision=precision, profile=1)
    out, st = h.filter(fields, ks)
    assert np.array_equal(h.filter(fields, ks)[0], out)
    h.set_options(batch=32)
    fixed, st_f = h.filter(fields, ks)
    its = [x.iterations for x in st]
    assert _in_tiles(st) and _in_tiles(st_f) and max(its) > 4 * min(its)
    op = O.scalar_operator(s, 2)
    for f in range(8):
        assert max(relative_l2(out[f, j], fixed[f, j]) for j in range(16)) <= TOL[precision]
    for f in (0, 7):
        ref = O.filter_scalar(op, fields[f], ks)
        assert max(relative_l2(out[f, j], ref[j]) for j in range(16)) <= TOL[precision]
    h.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_complex_tiles_of_the_librarys_width(ifl, precision):
    s = _sphere(5)
    fields = np.stack([W.sphere_k3_field(s, 700 + i, n_waves=64) for i in range(3)])
    ks = W.log_scales(s.h, 5)
    op = O.scalar_operator(s, 2)
    h = ifl.prepare_mesh(s, ifl.IFL_VERTEX_SCALAR, 2, precision=precision, solver=ifl.IFL_SOLVER_SHIFTED, profile=1)
    out, st = h.filter(fields, ks)
    assert _in_tiles(st)
    for f in range(3):
        ref = O.filter_scalar(op, fields[f], ks, method="shifted")
        assert max(relative_l2(out[f, j], ref[j]) for j in range(5)) <= TOL[precision]
    h.close()


def test_served_in_tiles(ifl):
    """Requests of three meshes joining tiles of 8 slots mid-flight: the oracle,
    bitwise the same alone, and bitwise with every kernel launched directly."""
    s, m = _sphere(5), W.split_square(64, jitter=0.2)
    meshes = [(s, 1), (s, 2), (m, 1)]
    rng = np.random.default_rng(7)
    reqs = []
    for r in range(24):
        mi = int(rng.integers(3))
        mesh = meshes[mi][0]
        ks = np.exp(np.sort(rng.uniform(np.log(np.pi / (8 * mesh.h)), np.log(np.pi / mesh.h), int(rng.integers(1, 7)))))
        field = W.sphere_k3_field(mesh, 5000 + r, n_waves=64) if mesh is s else W.planar_k3_field(mesh, 5000 + r)
        reqs.append((mi, field, ks))

    def serve(which, one_by_one=False, **kw):
        handles = [ifl.prepare_mesh(mesh, 0, n, precision=ifl.IFL_MIXED, batch=8, **kw) for mesh, n in meshes]
        srv = ifl.Server(4 << 30, slots=8)
        ids = [srv.add(h) for h in handles]
        got, open_ = {}, []
        for i in which:
            mi, field, ks = reqs[i]
            open_.append((i, srv.submit(ids[mi], field, ks)[0]))
            if one_by_one or i == which[-1]:
                for q, t in open_:
                    code, st, out, _ = srv.wait(t, len(reqs[q][2]))
                    assert code == 0 and _in_tiles(st)
                    got[q] = out.copy()
                open_ = []
        srv.close()
        for h in handles:
            h.close()
        return got

    together = serve(list(range(24)))
    alone = serve([0, 5, 11, 23], one_by_one=True)
    direct = serve([1, 5, 12, 23], graphs=0)
    for other in (alone, direct):
        for i, out in other.items():
            assert np.array_equal(out, together[i]), i
    ops = [O.scalar_operator(mesh, n) for mesh, n in meshes]
    for i in (0, 3, 7, 11, 15, 23):
        mi, field, ks = reqs[i]
        ref = O.filter_scalar(ops[mi], field, ks)
        assert max(relative_l2(together[i][j], ref[j]) for j in range(len(ks))) <= 1e-9
