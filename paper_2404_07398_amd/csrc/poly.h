// The polynomial engine: all scales of a field from one Chebyshev sequence
// of the first-order operator (host and device declarations).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "internal.h"

namespace ifl {

// Rings of halo units around a patch, at most (16 rings make a call on 4,096
// to 30,000 units 2% faster than 12, and its patches a third larger).
constexpr int kPolyDepth = 12;

// Threads of a patch's workgroup and units per thread; what a patch holds.
constexpr int kPolyThreads = 512;
constexpr int kPolySingleThreads = 1024;
// (block: stored couplings of a neighbour block: 1, of two components 4 where a
// unit has at most 3 neighbours, as the cell vectors have, and 2 where every
// block is [[a, b], [-b, a]], as the vertex vectors' are)
constexpr int poly_slots(int nc, int width) { return nc == 1 && width <= 6 ? 4 : 2; }
constexpr int poly_patch_units(int nc, int width) { return nc == 1 ? kPolyThreads * poly_slots(nc, width) : 1024; }
constexpr int poly_single_units(int block) { return kPolySingleThreads * (block == 2 ? 1 : 2); }
// Rings of large meshes' patches (small ones take what their patches leave).
constexpr int poly_patch_depth(int nc, int width) { return nc == 1 && width <= 6 ? 8 : 4; }

// Records: a unit's own block and its neighbours' (doubles, whole 16-byte
// units; of a scalar the neighbours' alone, its row's sum being zero); its
// neighbours' LDS offsets in a patch (uint16_t, bytes of a buffer of units);
// its neighbours' positions.
constexpr int poly_val_record(int width, int block) {
  return block == 1 ? width : ((1 + width) * block + 1) / 2 * 2;
}
constexpr int poly_idx_record(int width) { return (width + 1) / 2 * 2; }
constexpr int poly_col_record(int width) { return (width + 3) / 4 * 4; }

struct PatchInfo {
  int32_t start;                // first interior position; the interior is contiguous
  int32_t end[kPolyDepth + 1];  // local units up to and with ring d
  int64_t halo;                 // first halo entry (the positions of local units end[0] ..)
  int64_t idx;                  // first entry of its rows' offset records (all units' but the last ring's)
};

// M^-1 K in the patches' own order of the units ("positions"). A unit is a
// row, or the two rows of a vector dof.
struct PatchPack {
  int64_t units = 0;
  int nc = 1;      // components of a unit
  int width = 6;   // neighbour entries per unit (padded with the unit itself, value 0)
  int block = 1;   // stored couplings of a block
  int cap = 0;     // units a patch may hold
  int depth = 0;   // rings
  bool single = false;          // one patch without rings holds the mesh
  double mass_ratio = 1.0;      // largest mass / smallest
  std::vector<int32_t> order;   // position -> unit of the operator
  std::vector<PatchInfo> patches;
  std::vector<int32_t> halo;
  std::vector<uint16_t> idx;
  std::vector<int32_t> col;
  std::vector<double> val;      // M^-1 K
  std::vector<double> mass;     // [units * nc]
};

// local_order: the rows are in the library's locality order. false (out
// unspecified): the engine does not take this operator (rows too wide, a mass
// that is not positive, or vectors of more than 3 neighbours whose blocks do
// not turn).
bool build_patches(const HostOperator& op, bool local_order, PatchPack* out);

// The polynomial p of one filter scale, p(z) = sum_k c_k T_k(z) on the
// spectrum [0, lam] of M^-1 K, z = 2 x / lam - 1, order 1 or 2: the residual
// 1 - (1 + c x^n) p is the combination of T_{m+1} .. T_{m+n} that is 1 at the n
// zeros of 1 + c x^n, but for a factor that makes it 0 at x = 0. poly_degree:
// the least m at which the combination stays within tol on [-1, 1] (and the
// residual within 2 tol), -1 if that is above max_degree or for another order.
int poly_degree(int order, double c, double lam, double tol, int max_degree);
// c_0 .. c_m of degree m to out[k * stride].
void poly_coefficients(int order, double c, double lam, int m, double* out, int stride);

// Upper end of the spectrum from the tridiagonal of m Lanczos steps: alpha[0 ..
// m), beta[0 .. nb), beta[j] coupling steps j and j + 1 (nb < m: the space was
// exhausted). The largest Ritz value lies below the largest eigenvalue, by
// more than a margin of 1% where an eigenvalue stands that far above the rest
// and the start vector has little of it. Of an eigenvalue x the next Lanczos
// vector has the part p_m(x) times the start's, p_m the polynomial of the
// recurrence, and no part exceeds 1: with a start's part of at least 'least'
// no eigenvalue lies above the x where p_m(x) = 1 / least (van Dorsselaer,
// Hochstenbach, van der Vorst, SIAM J. Matrix Anal. 22 (2000)). At least 1%
// above the Ritz value.
double spectrum_bound(const double* alpha, const double* beta, int m, int nb, double least);

// Whether a column with ||M phi - S x||^2 = res2, ||M phi||^2 = bb and terms of
// the residual of norm^2 size2 counts as converged: within rtol, or within what
// FP64 can tell, as CG has it. An overflowed sum proves nothing: a residual
// must be finite, and an infinite size2 raises no bar. Only where bb itself
// overflows (fields above 1e150, which CG returns unfiltered) is a column
// passed on any residual but NaN.
bool poly_accepts(double res2, double size2, double bb, double rtol);

// --------------------------------------------------------------- device side
struct PolyState;  // defined in poly.hip
struct PolyWork;

// Device copy of the patches and the bound on the spectrum, on the current
// device; *out stays NULL where the engine does not take the operator.
ifl_status poly_create(const HostOperator& op, bool local_order, hipStream_t s, PolyState** out);
void poly_destroy(PolyState* ps);

// Work space for calls on any handle; one call at a time. limit: bytes its
// large arrays take at most, allocated here (0: they grow with the calls).
ifl_status poly_work_create(size_t limit, PolyWork** out);
void poly_work_destroy(PolyWork* w);
// hipMalloc that gives the device's idle work spaces back and tries again where
// memory is short (the runtime's last error is cleared).
hipError_t device_malloc(void** p, size_t bytes);
// A work space without a limit for one call on ps, from those idle on its
// device; to be returned when nothing of the call is under way any more.
ifl_status poly_work_borrow(PolyState* ps, int32_t n_fields, int32_t n_scales, PolyWork** out);
void poly_work_return(PolyState* ps, PolyWork* w);
// Whether the engine should serve requests of a few scales in a work space of
// this size.
bool poly_work_takes(const PolyState* ps, size_t limit, int order);

struct PolyCall {
  int order = 1;
  bool shifted = false;  // what CG would solve: shifted first-order systems
  double gamma = 0.5, rtol = 1e-12;
  int max_iter = 20000;
  int32_t n_fields = 0, n_scales = 0;
  const double* fields = nullptr;  // n_fields x field_len
  bool fields_host = false;
  const double* k = nullptr;
  double* out = nullptr;           // n_fields x n_scales x field_len, or NULL
  bool out_host = false;
  ifl_solve_stats* stats = nullptr;
  double* energy = nullptr;
  hipStream_t stream = nullptr;
};

// Whether the engine should run the call: its scales' degrees are within
// max_iter, and its products with the operator are fewer than CG would need.
bool poly_takes(const PolyState* ps, const PolyCall& call);

// Filters every column; the numbers (field * n_scales + scale) of columns
// whose true residual misses the tolerance go to *failed (their outputs hold
// what was reached). IFL_ENOMEM, IFL_EUNSUPPORTED: nothing was written, and
// the work space is worth giving up.
ifl_status poly_filter(PolyState* ps, PolyWork* w, const PolyCall& call, std::vector<int64_t>* failed);
// Fields f0 .. f0 + n - 1 of w's last call, in the caller's numbering (0 where
// there is no row), to device memory.
ifl_status poly_fields(PolyState* ps, const PolyWork* w, int f0, int n, double* out, hipStream_t stream);
// Gives back what a work space without a limit holds, but for those fields.
void poly_work_trim(PolyWork* w);

}  // namespace ifl
