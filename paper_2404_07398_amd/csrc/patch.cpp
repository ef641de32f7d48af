// Host side of the polynomial engine: the first-order operator's rows cut
// into compact patches with halo rings, and the polynomial coefficients of a
// filter scale.
#include "poly.h"

#include "parallel.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <complex>

namespace ifl {

namespace {

// Unit graph of an operator: unit u's neighbours other than itself, in
// increasing order (a unit is a row, or the two rows of a vector dof).
struct UnitGraph {
  int64_t n = 0;
  std::vector<int64_t> ptr;
  std::vector<int32_t> adj;
};

UnitGraph unit_graph(int64_t n, int nc, const std::vector<int64_t>& rp, const std::vector<int32_t>& col) {
  UnitGraph g;
  g.n = n / nc;
  g.ptr.assign(g.n + 1, 0);
  const int64_t parts = pieces_of(g.n);
  std::vector<std::vector<int32_t>> adj(parts);
  parallel_for(parts, [&](int64_t p) {
    std::vector<int32_t>& a = adj[p];
    for (int64_t u = g.n * p / parts; u < g.n * (p + 1) / parts; ++u) {
      const size_t from = a.size();
      for (int64_t r = u * nc; r < (u + 1) * nc; ++r)
        for (int64_t e = rp[r]; e < rp[r + 1]; ++e)
          if (col[e] / nc != u) a.push_back(col[e] / nc);
      if (nc > 1) {
        std::sort(a.begin() + from, a.end());
        a.erase(std::unique(a.begin() + from, a.end()), a.end());
      }
      g.ptr[u + 1] = (int64_t)(a.size() - from);
    }
  });
  for (int64_t u = 0; u < g.n; ++u) g.ptr[u + 1] += g.ptr[u];
  g.adj.resize((size_t)g.ptr[g.n]);
  parallel_for(parts, [&](int64_t p) {
    std::copy(adj[p].begin(), adj[p].end(), g.adj.begin() + g.ptr[g.n * p / parts]);
  });
  return g;
}

// Recursive bisection of ord[b, e) into 'leaves' ranges of equal size: the
// range's units in breadth-first order from a peripheral unit, cut in
// proportion. 'mark' holds a number per unit that only the range it belongs
// to uses, so ranges are cut by different threads ('fork' levels of them).
void bisect(const UnitGraph& g, std::vector<int32_t>& ord, std::atomic<int32_t>* mark, int64_t b, int64_t e,
            int64_t leaves, int32_t node, int fork, std::vector<int64_t>* starts) {
  if (leaves <= 1) {
    starts->push_back(b);
    return;
  }
  const auto mo = std::memory_order_relaxed;
  std::vector<int32_t> queue((size_t)(e - b));
  for (int64_t i = b; i < e; ++i) mark[ord[i]].store(4 * node, mo);
  int32_t start = ord[b];
  for (int pass = 0; pass < 2; ++pass) {
    const int32_t from = 4 * node + pass, to = from + 1;
    size_t head = 0, tail = 0;
    int64_t next = b;
    int32_t seed = start;
    while (tail < queue.size()) {
      if (mark[seed].load(mo) == from) {
        mark[seed].store(to, mo);
        queue[tail++] = seed;
      }
      for (; head < tail; ++head) {
        const int32_t u = queue[head];
        for (int64_t k = g.ptr[u]; k < g.ptr[u + 1]; ++k) {
          const int32_t v = g.adj[k];
          if (mark[v].load(mo) == from) {
            mark[v].store(to, mo);
            queue[tail++] = v;
          }
        }
      }
      if (tail < queue.size()) seed = ord[next++];  // another component of the range
    }
    start = queue.back();
  }
  std::copy(queue.begin(), queue.end(), ord.begin() + b);
  std::vector<int32_t>().swap(queue);
  const int64_t left = leaves / 2, cut = b + (e - b) * left / leaves;
  if (fork > 0) {
    std::vector<int64_t> right;
    parallel_for(2, [&](int64_t h) {
      if (h == 0) bisect(g, ord, mark, b, cut, left, 2 * node, fork - 1, starts);
      else bisect(g, ord, mark, cut, e, leaves - left, 2 * node + 1, fork - 1, &right);
    });
    starts->insert(starts->end(), right.begin(), right.end());
    return;
  }
  bisect(g, ord, mark, b, cut, left, 2 * node, 0, starts);
  bisect(g, ord, mark, cut, e, leaves - left, 2 * node + 1, 0, starts);
}

}  // namespace

bool build_patches(const HostOperator& op, bool local_order, PatchPack* out) {
  const bool own = op.order >= 2;
  const std::vector<int64_t>& rp = own ? op.k1_row_ptr : op.row_ptr;
  const std::vector<int32_t>& col = own ? op.k1_col : op.col;
  const std::vector<double>& val = own ? op.k1_val : op.val;
  const int nc = op.n_components;
  if (rp.empty() || (nc != 1 && nc != 2) || op.n % nc) return false;
  for (double m : op.mass)
    if (!(m > 0.0)) return false;
  if (nc == 2)  // a unit is one entity's (east, north) pair
    for (int64_t i = 0; i < op.n; i += 2)
      if (op.entity[i] % 2 || op.entity[i + 1] != op.entity[i] + 1) return false;
  const UnitGraph g = unit_graph(op.n, nc, rp, col);
  int width = 0;
  for (int64_t u = 0; u < g.n; ++u) width = std::max(width, (int)(g.ptr[u + 1] - g.ptr[u]));
  PatchPack& pp = *out;
  pp = PatchPack();
  pp.units = g.n;
  pp.nc = nc;
  pp.width = width <= 3 ? 3 : (width <= 6 ? 6 : (width <= 8 ? 8 : (width <= 12 ? 12 : 0)));
  if (pp.width == 0 || (nc == 2 && pp.width > 8) || (nc == 1 && pp.width == 3)) {
    if (nc == 1 && pp.width == 3) pp.width = 6;
    else return false;
  }
  pp.block = nc * nc;
  if (nc == 1)  // a constant field is left as it is: the diagonal is minus the row's other entries
    for (int64_t r = 0; r < op.n; ++r) {
      double sum = 0.0, size = 0.0;
      for (int64_t e = rp[r]; e < rp[r + 1]; ++e) {
        sum += val[e];
        size += std::fabs(val[e]);
      }
      if (!(std::fabs(sum) <= 1e-14 * size)) return false;
    }
  if (nc == 2 && pp.width >= 6) {  // [[a, b], [-b, a]] blocks throughout?
    std::atomic<bool> turns{true};
    const int64_t parts = pieces_of(g.n);
    parallel_for(parts, [&](int64_t q) {
      for (int64_t u = g.n * q / parts; u < g.n * (q + 1) / parts && turns.load(); ++u) {
        // the two rows' entries as (column unit, same component, other component)
        const auto entry = [&](int64_t r, int32_t v, int cc) {
          const auto at = std::lower_bound(col.begin() + rp[r], col.begin() + rp[r + 1], 2 * v + cc);
          return at != col.begin() + rp[r + 1] && *at == 2 * v + cc ? val[at - col.begin()] : 0.0;
        };
        bool ok = op.mass[2 * u] == op.mass[2 * u + 1];
        for (int64_t r = 2 * u; ok && r < 2 * u + 2; ++r)
          for (int64_t e = rp[r]; ok && e < rp[r + 1]; ++e) {
            const int32_t v = col[e] / 2;
            const int c = (int)(r % 2), cc = col[e] % 2;
            const double twin = entry(2 * u + 1 - c, v, 1 - cc);
            ok = c == cc ? val[e] == twin : val[e] == -twin;
          }
        if (!ok) turns.store(false);
      }
    });
    if (!turns.load()) return false;
    pp.block = 2;
  }
  pp.single = g.n <= poly_single_units(pp.block);
  pp.cap = pp.single ? (int)g.n : poly_patch_units(nc, pp.width);
  pp.depth = pp.single ? 0 : poly_patch_depth(nc, pp.width);

  // the order: the parts of the rows' own locality order, each bisected
  std::vector<int32_t> ord((size_t)g.n);
  for (int64_t i = 0; i < g.n; ++i) ord[i] = (int32_t)i;
  std::vector<int64_t> leaf;
  if (pp.single) {
    leaf = {0, g.n};
  } else {
    // interior units of a patch: what a round patch of the capacity has left
    // inside its rings; on meshes that would not fill the chip a patch per CU,
    // with as many more rings as its capacity then holds
    const double side = std::sqrt((double)pp.cap);
    const double most = 0.92 * (side - 2.0 * pp.depth) * (side - 2.0 * pp.depth);
    const int64_t want =
        std::max<int64_t>(64, std::min<int64_t>(std::max<int64_t>(64, (int64_t)most), (g.n + 255) / 256));
    pp.depth = std::max(pp.depth, std::min(kPolyDepth, (int)(0.5 * (side - std::sqrt((double)want / 0.8)))));
    const int parts = local_order && g.n >= 32768 ? 8 : 1;
    std::vector<std::atomic<int32_t>> mark((size_t)g.n);
    for (int64_t i = 0; i < g.n; ++i) mark[i].store(0, std::memory_order_relaxed);
    std::vector<std::vector<int64_t>> starts(parts);
    parallel_for(parts, [&](int64_t p) {
      const int64_t b = g.n * p / parts, e = g.n * (p + 1) / parts;
      // tree nodes of part p are numbered from its own root
      bisect(g, ord, mark.data(), b, e, (e - b + want - 1) / want, parts == 1 ? 1 : 8 + (int32_t)p,
             parts == 1 ? 3 : 0, &starts[p]);
    });
    for (const auto& s : starts) leaf.insert(leaf.end(), s.begin(), s.end());
    leaf.push_back(g.n);
  }
  pp.order = std::move(ord);
  std::vector<int32_t> pos((size_t)g.n);
  for (int64_t i = 0; i < g.n; ++i) pos[pp.order[i]] = (int32_t)i;

  // rings of each patch, then its units' neighbours as local numbers; a
  // patch that outgrows the capacity is cut in two
  struct Local {
    int64_t begin, end;
    std::vector<int32_t> units;  // patch positions: interior, ring 1, ..
    std::vector<int32_t> ends;   // depth + 1
    std::vector<uint16_t> idx;   // records
  };
  const int64_t groups = std::min<int64_t>(16, (int64_t)leaf.size() - 1);
  std::vector<std::vector<Local>> made(groups);
  parallel_for(groups, [&](int64_t q) {
    std::vector<int32_t> loc((size_t)g.n, -1);
    const int64_t lb = (int64_t)(leaf.size() - 1) * q / groups, le = (int64_t)(leaf.size() - 1) * (q + 1) / groups;
    std::vector<std::pair<int64_t, int64_t>> todo;
    for (int64_t l = le - 1; l >= lb; --l) todo.push_back({leaf[l], leaf[l + 1]});
    while (!todo.empty()) {
      const auto [b, e] = todo.back();
      todo.pop_back();
      Local L{b, e, {}, {}, {}};
      for (int64_t i = b; i < e; ++i) {
        loc[i] = (int32_t)(i - b);
        L.units.push_back((int32_t)i);
      }
      L.ends.push_back((int32_t)L.units.size());
      bool fits = (int64_t)L.units.size() <= pp.cap;
      size_t from = 0;
      for (int d = 0; fits && d < pp.depth; ++d) {
        const size_t to = L.units.size();
        for (size_t i = from; i < to; ++i) {
          const int32_t u = pp.order[L.units[i]];
          for (int64_t k = g.ptr[u]; k < g.ptr[u + 1]; ++k) {
            const int32_t v = pos[g.adj[k]];
            if (loc[v] < 0) {
              loc[v] = 0;
              L.units.push_back(v);
            }
          }
        }
        // a ring in increasing position: its rows are read in runs
        std::sort(L.units.begin() + to, L.units.end());
        for (size_t i = to; i < L.units.size(); ++i) loc[L.units[i]] = (int32_t)i;
        from = to;
        L.ends.push_back((int32_t)L.units.size());
        fits = (int64_t)L.units.size() <= pp.cap;
      }
      if (!fits && e - b > 1) {
        for (int32_t u : L.units) loc[u] = -1;
        const int64_t mid = (b + e) / 2;
        todo.push_back({mid, e});
        todo.push_back({b, mid});
        continue;
      }
      const size_t rows = pp.depth ? (size_t)L.ends[pp.depth - 1] : L.units.size();
      const size_t rec = (size_t)poly_idx_record(pp.width);
      const uint32_t bytes = 8u * (uint32_t)nc;
      L.idx.assign(rows * rec, 0);
      for (size_t i = 0; fits && i < rows; ++i) {
        const int32_t u = pp.order[L.units[i]];
        size_t k = 0;
        for (int64_t a = g.ptr[u]; a < g.ptr[u + 1]; ++a, ++k)
          L.idx[i * rec + k] = (uint16_t)(bytes * (uint32_t)loc[pos[g.adj[a]]]);
        for (; k < rec; ++k) L.idx[i * rec + k] = (uint16_t)(bytes * (uint32_t)i);
      }
      for (int32_t u : L.units) loc[u] = -1;
      if (!fits) L.units.clear();  // one unit with more neighbours in its rings than the capacity
      made[q].push_back(std::move(L));
    }
  });
  for (const auto& m : made)
    for (const Local& L : m) {
      if (L.units.empty()) return false;
      PatchInfo info{};
      info.start = (int32_t)L.begin;
      info.halo = (int64_t)pp.halo.size();
      info.idx = (int64_t)pp.idx.size();
      for (int d = 0; d <= kPolyDepth; ++d) info.end[d] = L.ends[std::min(d, pp.depth)];
      pp.patches.push_back(info);
      pp.halo.insert(pp.halo.end(), L.units.begin() + L.ends[0], L.units.end());
      pp.idx.insert(pp.idx.end(), L.idx.begin(), L.idx.end());
    }

  pp.halo.push_back(0);  // a patch without halo units still reads one entry
  // M^-1 K by position, a record per unit, and the columns by position
  const int64_t U = g.n, bb = pp.block, rec = poly_val_record(pp.width, pp.block), crec = poly_col_record(pp.width);
  pp.val.assign((size_t)(U * rec), 0.0);
  pp.col.assign((size_t)(U * crec), 0);
  pp.mass.resize((size_t)(U * nc));
  const int64_t pieces = pieces_of(U);
  parallel_for(pieces, [&](int64_t q) {
    for (int64_t i = U * q / pieces; i < U * (q + 1) / pieces; ++i) {
      const int32_t u = pp.order[i];
      const int64_t a0 = g.ptr[u], a1 = g.ptr[u + 1];
      for (int64_t k = 0; k < crec; ++k) pp.col[i * crec + k] = k < a1 - a0 ? pos[g.adj[a0 + k]] : (int32_t)i;
      for (int c = 0; c < nc; ++c) {
        const int64_t r = (int64_t)u * nc + c;
        pp.mass[i * nc + c] = op.mass[r];
        const double im = 1.0 / op.mass[r];
        for (int64_t e = rp[r]; e < rp[r + 1]; ++e) {
          const int32_t v = col[e] / nc, cc = col[e] % nc;
          int64_t k = 0;
          if (v != u) k = 1 + std::lower_bound(g.adj.begin() + a0, g.adj.begin() + a1, v) - (g.adj.begin() + a0);
          if (bb == 1) {
            if (k) pp.val[i * rec + k - 1] = val[e] * im;
          } else if (bb == 4) pp.val[i * rec + k * bb + c * nc + cc] = val[e] * im;
          else if (c == 0) pp.val[i * rec + k * bb + cc] = val[e] * im;
        }
      }
    }
  });
  double mlo = pp.mass[0], mhi = pp.mass[0];
  for (double m : pp.mass) {
    mlo = std::min(mlo, m);
    mhi = std::max(mhi, m);
  }
  pp.mass_ratio = mhi / mlo;
  return true;
}

namespace {

// In extended precision: the coefficients of order 2 are read with the
// weight 1 + c lam^2, the condition number of the system.
using real = long double;

// One zero zr + i zi of 1 + c x^n in z (n = 2: the other is its conjugate),
// as z = (rho + 1 / rho) / 2, rho = exp(grow + i turn), grow > 0, and the
// residual of a degree, a_0 T_{m+1} (n = 1) or a_0 T_{m+1} + a_1 T_{m+2}
// (n = 2, real, from the real and imaginary part of its value 1 at the zero).
struct Residual {
  int n;
  real zr, zi, grow, turn;
  real a[2] = {0.0L, 0.0L};

  Residual(int order, double c, double lam) : n(order) {
    const real at = 2.0L / (real)lam * (n == 1 ? 1.0L / (real)c : 1.0L / std::sqrt((real)c));
    zr = n == 1 ? -1.0L - at : -1.0L;
    zi = n == 1 ? 0.0L : at;
    const std::complex<real> z(zr, zi);
    const std::complex<real> root = std::sqrt(z - (real)1) * std::sqrt(z + (real)1);
    std::complex<real> rho = z + root;
    if (std::abs(rho) < 1.0L) rho = z - root;
    grow = std::log(std::abs(rho));
    turn = std::arg(rho);
  }
  // T_k at the zero
  void cheb(int k, real* re, real* im) const {
    const real up = std::exp(k * grow), down = 1.0L / up;
    *re = 0.5L * (up + down) * std::cos(k * turn);
    *im = 0.5L * (up - down) * std::sin(k * turn);
  }
  // sets a for degree m; its size
  real solve(int m) {
    real r0, i0, r1, i1;
    cheb(m + 1, &r0, &i0);
    if (n == 1) {
      a[0] = 1.0L / r0;
      return std::abs(a[0]);
    }
    cheb(m + 2, &r1, &i1);
    const real det = r0 * i1 - r1 * i0;
    a[0] = i1 / det;
    a[1] = -i0 / det;
    return std::abs(a[0]) + std::abs(a[1]);
  }
  // its value at x = 0, z = -1, where T_k is 1 or -1
  real at_zero(int m) const { return m % 2 ? a[0] - a[1] : a[1] - a[0]; }
};

}  // namespace

int poly_degree(int order, double c, double lam, double tol, int max_degree) {
  if (order != 1 && order != 2) return -1;
  Residual r(order, c, lam);
  if (!(r.grow > 0.0L) || !std::isfinite((double)r.grow)) return -1;
  const double guess = std::log(2.0 / tol) / (double)r.grow;
  if (!(guess < 4.0 * max_degree + 64.0)) return -1;
  // n = 1: the size falls as 2 exp(-grow (m + 1)); n = 2: it swings about that
  int m = std::max(0, (int)guess - (order == 1 ? 2 : 8));
  while (m <= max_degree && !(r.solve(m) <= tol)) ++m;
  return m > max_degree ? -1 : m;
}

void poly_coefficients(int order, double c, double lam, int m, double* out, int stride) {
  Residual r(order, c, lam);
  r.solve(m);
  const int n = order;
  // s = (1 - R) / (z - z_0), from the highest term down (the growing
  // direction of the recurrence); p = s / (c (lam / 2)) for n = 1, and for
  // n = 2, 1 / |z - z_0|^2 = Im (1 / (z - z_0)) / Im z_0 gives p from Im s.
  // Scaled to p = 1 at x = 0: the largest scales, which hold most of a field's
  // energy, and constants come out exact, for a residual of twice the size
  // elsewhere
  const real lead = (n == 1 ? 1.0L / ((real)c * 0.5L * (real)lam)
                            : 1.0L / ((real)c * 0.25L * (real)lam * (real)lam * r.zi)) / (1.0L - r.at_zero(m));
  real sr = 0.0L, si = 0.0L, ur = 0.0L, ui = 0.0L;  // s_k, s_{k+1}
  for (int k = m + n; k >= 1; --k) {
    const real q = k > m ? -r.a[k - m - 1] : 0.0L;
    real nr = 2.0L * (q + r.zr * sr - r.zi * si) - ur, ni = 2.0L * (r.zr * si + r.zi * sr) - ui;
    if (k == 1) {
      nr *= 0.5L;
      ni *= 0.5L;
    }
    ur = sr;
    ui = si;
    sr = nr;
    si = ni;
    if (k - 1 <= m) out[(int64_t)(k - 1) * stride] = (double)((n == 1 ? sr : si) * lead);
  }
}

double spectrum_bound(const double* alpha, const double* beta, int m, int nb, double least) {
  // the largest eigenvalue of the tridiagonal by bisection
  double lo = alpha[0], hi = alpha[0];
  const int off = std::min(nb, m - 1);
  for (int i = 0; i < m; ++i) {
    const double r = (i > 0 && i - 1 < off ? std::fabs(beta[i - 1]) : 0.0) + (i < off ? std::fabs(beta[i]) : 0.0);
    lo = std::min(lo, alpha[i] - r);
    hi = std::max(hi, alpha[i] + r);
  }
  for (int it = 0; it < 100; ++it) {
    const double mid = 0.5 * (lo + hi);
    double q = 1.0;
    bool below = true;  // no eigenvalue above mid: all pivots of mid - T positive
    for (int i = 0; i < m && below; ++i) {
      q = mid - alpha[i] - (i > 0 && i - 1 < off ? beta[i - 1] * beta[i - 1] / q : 0.0);
      if (!(q > 0.0)) below = false;
    }
    (below ? hi : lo) = mid;
  }
  const double theta = hi;
  if (nb < m || !(theta > 0.0) || !(least > 0.0)) return 1.01 * theta;
  // log |p_m| above theta, where p_m increases
  const auto growth = [&](double x) {
    double p0 = 0.0, p1 = 1.0, log = 0.0;
    for (int j = 0; j < m; ++j) {
      const double p2 = ((x - alpha[j]) * p1 - (j > 0 ? beta[j - 1] * p0 : 0.0)) / beta[j];
      p0 = p1;
      p1 = p2;
      const double size = std::max(std::fabs(p0), std::fabs(p1));
      if (!(size > 0.0)) return -HUGE_VAL;
      p0 /= size;
      p1 /= size;
      log += std::log(size);
    }
    return log + std::log(std::fabs(p1));
  };
  double a = theta, b = 1.01 * theta;
  while (growth(b) < -std::log(least) && b < 16.0 * theta) {
    a = b;
    b += 0.5 * (b - theta) + 0.01 * theta;
  }
  for (int it = 0; it < 40 && b > 1.01 * theta; ++it) {
    const double mid = 0.5 * (a + b);
    (growth(mid) < -std::log(least) ? a : b) = mid;
  }
  return std::max(b, 1.01 * theta);
}

bool poly_accepts(double res2, double size2, double bb, double rtol) {
  if (!std::isfinite(bb)) return !std::isnan(res2);
  if (!std::isfinite(res2)) return false;
  const double floor = std::isfinite(size2) ? 8.0 * 1.1102230246251565e-16 * std::sqrt(size2) : 0.0;
  return std::sqrt(res2) <= std::max(rtol * std::sqrt(bb), floor);
}

}  // namespace ifl
