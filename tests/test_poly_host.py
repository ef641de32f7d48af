"""Host side of the polynomial engine and of preparing a handle (CPU only):
what the library's C++ functions decide where no call reaches on its own, and
the prepare phase's limits."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O
import workloads as W

ifl = pytest.importorskip("paper_2404_07398_amd")

INF, NAN = float("inf"), float("nan")


def _function(name, restype, *argtypes):
    if not os.path.exists(ifl.LIB_PATH):
        pytest.skip("libifl.so not built")
    f = getattr(ifl.lib(), name)
    f.restype, f.argtypes = restype, argtypes
    return f


@pytest.mark.parametrize("res2,size2,bb,ok", [
    (1e-24, 1.0, 1.0, True), (1.1e-24, 1.0, 1.0, False),  # rtol = 1e-12
    (1e-24, 0.0, 0.0, False), (0.0, 0.0, 0.0, True),       # a zero field
    (7.8e-23, 1e8, 1.0, True), (7.9e-23, 1e8, 1.0, False),  # attainable: 8 u 1e4 = 8.9e-12
    (INF, INF, 1.0, False), (INF, 1.0, 1.0, False), (NAN, INF, 1.0, False),
    (1e-20, INF, 1.0, False), (1e-20, NAN, 1.0, False), (1e-25, INF, 1.0, True),
    (INF, INF, INF, True), (NAN, INF, INF, False),         # fields whose norm overflows
])
def test_columns_counted_as_converged(res2, size2, bb, ok):
    accepts = _function("_ZN3ifl12poly_acceptsEdddd", ctypes.c_bool, *[ctypes.c_double] * 4)
    assert accepts(res2, size2, bb, 1e-12) is ok


def test_prepare_of_a_vertex_with_very_many_neighbours():
    """A fan of 100,000 triangles in a shuffled numbering: its hub's row is
    sorted in n log n (a quadratic sort takes over 15 s, this 0.3)."""
    if not os.path.exists(ifl.LIB_PATH):
        pytest.skip("libifl.so not built")
    n = 100_000
    rim = np.random.default_rng(1).permutation(n) + 1
    a = 2.0 * np.pi * np.arange(n) / n
    xy = np.zeros((n + 1, 2))
    xy[rim] = 1000.0 * np.stack([np.cos(a), np.sin(a)], axis=1)
    tris = np.stack([np.zeros(n, np.int64), rim, np.roll(rim, -1)], axis=1).astype(np.int32)
    m = W.Mesh(coords=xy, tris=tris, geometry=W.GEOM_PLANAR, h=1.0)
    t0 = time.perf_counter()
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, 1, device=-1)
    assert time.perf_counter() - t0 < 6.0
    rp, col, val, mass, ent = h.export_operator()
    rows = np.diff(rp)
    assert rows.max() == n + 1 and np.all(np.diff(col[rp[rows.argmax()]:rp[rows.argmax() + 1]]) > 0)
    h.close()


@pytest.mark.parametrize("order", [2, 3])
def test_operator_products_with_rows_of_very_different_lengths(order):
    """K M^-1 K .. of a fan whose hub has 700 neighbours: the product's
    accumulator grows to its widest row."""
    if not os.path.exists(ifl.LIB_PATH):
        pytest.skip("libifl.so not built")
    n = 700
    rng = np.random.default_rng(2)
    rim = rng.permutation(n) + 1
    a = 2.0 * np.pi * np.arange(n) / n
    xy = np.zeros((n + 1, 2))
    xy[rim] = (10.0 + rng.uniform(-0.5, 0.5, n))[:, None] * np.stack([np.cos(a), np.sin(a)], axis=1)
    tris = np.stack([np.zeros(n, np.int64), rim, np.roll(rim, -1)], axis=1).astype(np.int32)
    m = W.Mesh(coords=xy, tris=tris, geometry=W.GEOM_PLANAR, h=1.0)
    h = ifl.prepare_mesh(m, ifl.IFL_VERTEX_SCALAR, order, device=-1)
    rp, col, val, mass, ent = h.export_operator()
    h.close()
    ref = O.scalar_operator(m, order)
    mine = sp.csr_matrix((val, col, rp), shape=(n + 1, n + 1)).toarray()
    want = ref.Kn.toarray()[np.ix_(ref.dof_of[ent], ref.dof_of[ent])]
    # each entry sums at most n products, at 2 (order - 1) roundings each way
    size = abs(want).max()
    assert np.abs(mine - want).max() <= 4 * order * n * 2.0 ** -53 * size
    for i in range(n + 1):
        assert np.all(np.diff(col[rp[i]:rp[i + 1]]) > 0)


def test_threads_that_cannot_be_started(tmp_path):
    """parallel_for with every allocation in turn refused: the work is done or
    std::bad_alloc arrives; the process does not end."""
    src = tmp_path / "t.cpp"
    src.write_text(r"""
#include "parallel.h"
#include <cstdio>
#include <cstdlib>
#include <new>
static thread_local long left = -1;
void* operator new(std::size_t n) {
  if (left >= 0 && left-- == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
int main() {
  int done = 0, thrown = 0;
  for (long refuse = 0; refuse < 40; ++refuse) {
    int hit[64] = {};
    try {
      left = refuse;
      ifl::parallel_for(64, [&](int64_t i) { hit[i] += 1; });
      left = -1;
      for (int h : hit) if (h != 1) return 2;
      ++done;
    } catch (const std::bad_alloc&) {
      left = -1;
      ++thrown;
    }
  }
  std::printf("%d %d\n", done, thrown);
  return done > 0 && thrown > 0 ? 0 : 3;
}
""")
    exe = tmp_path / "t"
    inc = os.path.join(os.path.dirname(ifl.LIB_PATH), "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe), "-pthread"], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0


def _lanczos(values, start, steps):
    v = start / np.linalg.norm(start)
    prev, b, alpha, beta = np.zeros_like(v), 0.0, [], []
    for _ in range(steps):
        w = values * v - b * prev
        a = w @ v
        w -= a * v
        b = np.linalg.norm(w)
        alpha.append(a)
        beta.append(b)
        prev, v = v, w / b
    return np.array(alpha), np.array(beta)


@pytest.mark.parametrize("steps,least", [(32, 2e-6), (64, 5e-7)])
@pytest.mark.parametrize("above", [0.0, 0.011, 0.02, 0.05, 0.3])
def test_upper_end_of_the_spectrum(steps, least, above):
    """One eigenvalue above a full band, and as little of its eigenvector in the
    start as the bound allows for: the bound covers it, a margin of 1% on the
    largest Ritz value does not always."""
    p = ctypes.POINTER(ctypes.c_double)
    bound = _function("_ZN3ifl14spectrum_boundEPKdS1_iid", ctypes.c_double, p, p, ctypes.c_int, ctypes.c_int,
                      ctypes.c_double)
    rng = np.random.default_rng(7)
    n = 200_000
    values = np.sort(rng.uniform(0.0, 1.0, n))
    start = rng.uniform(-1.0, 1.0, n)
    if above:
        values[-1] = 1.0 + above
        start[-1] = 1.01 * least * np.linalg.norm(start[:-1])
    alpha, beta = _lanczos(values, start, steps)
    ritz = np.linalg.eigvalsh(np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1))[-1]
    lam = bound(alpha.ctypes.data_as(p), beta.ctypes.data_as(p), steps, steps, least)
    assert lam >= max(values[-1], 1.01 * ritz * (1 - 1e-12))
    # no larger than Lanczos' own convergence allows: log(2 / least) growth at
    # acosh(1 + 2 x) a step above the band's end
    assert lam <= max(1.011 * ritz, (1.0 + np.log(4.0 * n / least) ** 2 / (4.0 * steps ** 2)) * max(ritz, 1.0))
    if above == 0.02 and steps == 32:
        assert 1.01 * ritz < values[-1]
    # an exhausted space: the Ritz value is an eigenvalue
    assert bound(alpha.ctypes.data_as(p), beta.ctypes.data_as(p), steps, steps - 1, least) == pytest.approx(1.01 * ritz)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("b", [0.01, 1.0, 30.0, 1e3, 1e5])
def test_polynomials(order, b):
    """p(x) against 1 / (1 + c x^n): 1 at x = 0, the residual within twice the
    tolerance of the degree on the spectrum, above it for a lower degree."""
    degree = _function("_ZN3ifl11poly_degreeEidddi", ctypes.c_int, ctypes.c_int, *[ctypes.c_double] * 3, ctypes.c_int)
    coefficients = _function("_ZN3ifl17poly_coefficientsEiddiPdi", None, ctypes.c_int, ctypes.c_double, ctypes.c_double,
                             ctypes.c_int, ctypes.POINTER(ctypes.c_double), ctypes.c_int)
    lam, tol = 3.7, 1e-9
    c = (b / lam) ** order
    m = degree(order, c, lam, tol, 100_000)
    out = np.zeros((m + 1, 2))
    coefficients(order, c, lam, m, out.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), 2)
    assert not out[:, 1].any()
    z = np.cos(np.linspace(0.0, np.pi, 4 * m + 201))
    x = 0.5 * lam * (z + 1.0)
    p = np.polynomial.chebyshev.chebval(z, out[:, 0])
    res = 1.0 - (1.0 + c * x ** order) * p
    # (the sum of m + 1 coefficients below 2 rounds to (m + 1) u, weighted)
    u = (m + 1) * 2.0 ** -52
    assert np.all(np.abs(res) <= 2.0 * tol + u * (1.0 + c * x ** order))
    assert abs(res[-1]) <= u
    assert m == 0 or degree(order, c, lam, tol, m - 1) == -1
