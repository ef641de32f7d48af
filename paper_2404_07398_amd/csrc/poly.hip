// The polynomial engine: every scale of a field from one sequence of products
// with the first-order operator.
//
// The filter of order n at scale factor c is f(A), f(x) = 1 / (1 + c x^n),
// of A = M^-1 K alone, so all scales (and both orders) of a field share the
// vectors t_k = T_k(2 A / lam - 1) phi of the Chebyshev recurrence
//   t_{k+1} = (4 / lam) A t_k - 2 t_k - t_{k-1},
// and a scale is the sum over k of its coefficients c_k times t_k. Where CG
// takes one product per scale and iteration, a field with S scales takes the
// products of its largest scale once; and the recurrence has no inner
// products, so nothing has to be known across the mesh between two steps.
// That is what the step kernel uses: a workgroup keeps a patch of the mesh
// with its rings of halo units in LDS and advances it several steps per
// launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <string>

#include "poly.h"

namespace ifl {

#define IFL_HIP(expr)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess)                                                                      \
      return fail(IFL_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));            \
  } while (0)

namespace {

constexpr int kXcd = 8;
constexpr int kRed = 256;       // threads of the row kernels
constexpr int kRedBlocks = 512; // blocks of the row kernels that write partial sums, at most
// Steps of the spectrum estimate, by launches and in one workgroup (the small
// meshes' bound is at most 2% above the estimate after 32 steps, the others'
// at most 0.2% after 64).
constexpr int kLanczos = 64, kLanczosSmall = 32;
constexpr int kMaxGroup = 16;   // scales summed together

// Without a limit: about 12 GB of the 288, which at level 9 hold 8 fields with
// 96 vectors of a sequence of 180 and 32 scales each (a patch's records are read
// once for them; 4 fields took 7% longer).
constexpr size_t kPolyBudget = (size_t)12 << 30;

struct PolyDev {
  const PatchInfo* info = nullptr;
  const int32_t* halo = nullptr;
  const uint16_t* idx = nullptr;
  const int32_t* col = nullptr;
  const double* val = nullptr;
  const double* mass = nullptr;
  const int32_t* entity = nullptr;  // caller index of each row
  const int32_t* row_of = nullptr;  // row of each caller index, -1: none
  int64_t units = 0, rows = 0, np = 0, field_len = 0;
  int npatch = 0;
};

template <int NC>
struct Unit;  // the NC components of a unit
template <>
struct Unit<1> {
  double v[1];
};
template <>
struct alignas(16) Unit<2> {
  double v[2];
};

// Coupling of component c of a unit to component d of the block's unit.
template <int NC, int BV>
__device__ __forceinline__ double coupling(const double* b, int c, int d) {
  if constexpr (BV == 2) return c == d ? b[0] : c == 0 ? b[1] : -b[1];
  else return b[c * NC + d];
}

// A store past the caches (see the launch for where it pays).
__device__ __forceinline__ void pass_by(const Unit<1>& t, Unit<1>* to) { __builtin_nontemporal_store(t.v[0], &to->v[0]); }
__device__ __forceinline__ void pass_by(const Unit<2>& t, Unit<2>* to) {
  typedef double Two __attribute__((ext_vector_type(2)));
  Two v = {t.v[0], t.v[1]};
  __builtin_nontemporal_store(v, reinterpret_cast<Two*>(to));
}

// A scalar's own entry, from its neighbours'.
template <int W>
__device__ __forceinline__ double minus_sum(const double* v) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) s -= v[k];
  return s;
}

// Slots of a thread that may hold interior units when the step kernel sums.
constexpr int sum_slots(int slots) { return slots < 2 ? slots : 2; }

// What a thread of the step kernel owns: its units' rows of (4 / lam) A, the
// neighbours' LDS offsets two to a register (kept packed: unpacked they cost
// the registers of a second resident workgroup), and the two latest vectors.
template <int NC, int W, int BV, int SLOTS, int ACC>
struct Rows {
  double val[SLOTS][W][BV], own[SLOTS][BV];
  uint32_t nb[SLOTS][(W + 1) / 2];
  Unit<NC> t[2][SLOTS];
  // sums of ACC scales, for the slots that hold interior units
  double acc[ACC ? sum_slots(SLOTS) : 1][ACC ? ACC : 1][NC];
};

// Coefficients, never written while a kernel runs: read through the scalar
// cache (a vector load would be waited for together with the steps' stores).
typedef const __attribute__((address_space(4))) double* Coef;

// One step for N of the thread's units from slot S on: the vector t[CUR] and
// the LDS buffer CUR hold t_k; t[1 - CUR] holds t_{k-1} and becomes t_{k+1}.
// All gathers are issued before the sums. Lanes past 'lim' compute on
// whatever is there and write nothing. coef: the new vector's coefficients.
template <int NC, int W, int BV, int SLOTS, int T, int ACC, bool PAST, int CUR, int N>
__device__ __forceinline__ void step_slots(Rows<NC, W, BV, SLOTS, ACC>& r, char* lds, int S, int tid, int lim, int inside,
                                           double half, Unit<NC>* out, Coef coef) {
  constexpr int BUF = T * SLOTS * (int)sizeof(Unit<NC>);
  Unit<NC> g[N][W];
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int k = 0; k < W; k += 2) {
      uint32_t two = r.nb[S + n][k / 2];
      asm volatile("" : "+v"(two));  // keeps the unpacking from being hoisted into registers of its own
      g[n][k] = *reinterpret_cast<const Unit<NC>*>(lds + CUR * BUF + (two & 0xffffu));
      if (k + 1 < W) g[n][k + 1 < W ? k + 1 : k] = *reinterpret_cast<const Unit<NC>*>(lds + CUR * BUF + (two >> 16));
    }
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int s = S + n, i = tid + s * T;
    double acc[NC], acc2[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      acc[c] = -r.t[1 - CUR][s].v[c];
      acc2[c] = 0.0;
#pragma unroll
      for (int d = 0; d < NC; ++d) acc2[c] += coupling<NC, BV>(r.own[s], c, d) * r.t[CUR][s].v[d];
#pragma unroll
      for (int k = 0; k < W; ++k)
#pragma unroll
        for (int d = 0; d < NC; ++d) {
          double& a = k % 2 == 0 ? acc[c] : acc2[c];
          a += coupling<NC, BV>(r.val[s][k], c, d) * g[n][k].v[d];
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) r.t[1 - CUR][s].v[c] = half * (acc[c] + acc2[c]);
    if (i < lim) *reinterpret_cast<Unit<NC>*>(lds + (1 - CUR) * BUF + i * (int)sizeof(Unit<NC>)) = r.t[1 - CUR][s];
    if (ACC && s < sum_slots(SLOTS)) {
#pragma unroll
      for (int a = 0; a < ACC; ++a)
#pragma unroll
        for (int c = 0; c < NC; ++c) r.acc[s < sum_slots(SLOTS) ? s : 0][a][c] += coef[a] * r.t[1 - CUR][s].v[c];
    }
    if ((ACC == 0 || out) && i < inside) {
      if constexpr (PAST) pass_by(r.t[1 - CUR][s], out + i);
      else out[i] = r.t[1 - CUR][s];
    }
  }
}

template <int NC, int W, int BV, int SLOTS, int T, int ACC, bool PAST, int CUR>
__device__ __forceinline__ void step_all(Rows<NC, W, BV, SLOTS, ACC>& r, char* lds, int tid, int lim, int inside,
                                         double half, Unit<NC>* out, Coef coef) {
  // first unit of this wavefront: the tests below are one scalar branch each
  const int wave = __builtin_amdgcn_readfirstlane(tid & ~63);
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
    if (wave + s * T < lim)
      step_slots<NC, W, BV, SLOTS, T, ACC, PAST, CUR, 1>(r, lds, s, tid, lim, inside, half, out, coef);
}

// 'steps' steps of the recurrence on one patch, field after field.
//
// A thread owns SLOTS units, kept in registers for all steps and fields; the
// neighbours' t_k come from LDS, t_{k+1} goes to the other buffer. Step j
// needs the rings up to steps - j only, a prefix of the local numbering. With
// one patch for the whole mesh (no rings) the steps are not limited.
//
// What bounds it: the memory system. A patch's records, halo list and first
// two vectors are read once per launch (about 2.7 local units per interior
// one at 8 rings), and its new interior vectors written; within the steps
// LDS gathers and FP64 FMAs take about as long as each other. Loads and
// stores must therefore never be waited for inside the steps, and two
// workgroups share a CU (128 registers) so that one loads while the other
// steps. Measured on one field of the 2.6 M-vertex sphere, per 8 steps: 319 us
// with the ring ends and the unpacked offsets in memory and the records read
// entry by entry, 150 us now with its one scale summed; of the 1.57 M-dof
// masked sphere 400 us for 4 fields, and 394 us now for 8 (822 MB written and
// 236 MB read, 2.7 TB/s): there its waves wait for LDS and memory in 46% of
// their cycles and for an issue slot in 36%, and bank conflicts of the gathers
// are 44% of LDS's busy cycles.
//
// prev == nullptr: the sequence starts (cur = t_0, the first step is halved).
// out: plane of the first new vector, the next ones 'plane' doubles on.
//
// ACC > 0 (calls of few scales): the kernel sums as it goes, x (rows x ACC)
// += coef[j][a] t, coef pointing at the coefficients of cur; then only the
// last two vectors are written (two planes at out), and no launch reads the
// sequence again: 16 ACC + 16 bytes a row and launch for 16 a row and step.
template <int NC, int W, int BV, int SLOTS, int T, int ACC, bool PAST>
__global__ __launch_bounds__(T, 4) void k_poly_steps(PolyDev m, const double* __restrict__ prev,
                                                     const double* __restrict__ cur, double* __restrict__ out,
                                                     int64_t plane, int n_fields, int steps, int ringed,
                                                     double scale, const double* __restrict__ coef,
                                                     double* __restrict__ x) {
  // consecutive patches on one XCD: their halos overlap in its L2
  const int per = (m.npatch + kXcd - 1) / kXcd;
  const int pid = (int)(blockIdx.x % kXcd) * per + (int)(blockIdx.x / kXcd);
  if (pid >= m.npatch || (int)(blockIdx.x / kXcd) >= per) return;
  __shared__ __align__(16) char lds[2 * T * SLOTS * sizeof(Unit<NC>)];
  const PatchInfo* p = m.info + pid;
  const int tid = threadIdx.x;
  // the ring ends, lane d of each wavefront holding ring d's: a step's limit
  // is read from there, since a load of it would wait for the stores before
  const int ends = p->end[min(tid & 63, kPolyDepth)];
  const int start = p->start, inside = p->end[0];
  const int loaded = p->end[ringed ? steps : 0];
  const int first_lim = p->end[ringed ? steps - 1 : 0];
  constexpr int VR = poly_val_record(W, BV), IR = poly_idx_record(W);
  Rows<NC, W, BV, SLOTS, ACC> r;
  int32_t at[SLOTS];
  // no branches between the loads, so that all are in flight together: units
  // past the last one read the first one's data
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int i = tid + s * T;
    const int h = i >= inside && i < loaded ? i - inside : 0;
    const int32_t q = ringed ? m.halo[p->halo + h] : 0;
    at[s] = i < loaded ? (i < inside ? start + i : q) : start;
  }
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int i = tid + s * T < first_lim ? tid + s * T : 0;
    const uint32_t* id = reinterpret_cast<const uint32_t*>(m.idx + p->idx + (int64_t)i * IR);
#pragma unroll
    for (int k = 0; k < (W + 1) / 2; ++k) r.nb[s][k] = id[k];
    const double* v = m.val + (int64_t)(tid + s * T < first_lim ? at[s] : start) * VR;
#pragma unroll
    for (int b = 0; b < BV; ++b)
      if (BV > 1) r.own[s][b] = v[b];
#pragma unroll
    for (int k = 0; k < W; ++k)
#pragma unroll
      for (int b = 0; b < BV; ++b) r.val[s][k][b] = v[(BV > 1 ? k + 1 : k) * BV + b];
  }
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    if (BV == 1) r.own[s][0] = minus_sum<W>(&r.val[s][0][0]);
#pragma unroll
    for (int b = 0; b < BV; ++b) r.own[s][b] = scale * r.own[s][b] - (b == 0 || b == 3 ? 2.0 : 0.0);
#pragma unroll
    for (int k = 0; k < W; ++k)
#pragma unroll
      for (int b = 0; b < BV; ++b) r.val[s][k][b] *= scale;
  }
  for (int f = blockIdx.y; f < n_fields; f += gridDim.y) {
    const Unit<NC>* cf = reinterpret_cast<const Unit<NC>*>(cur + (int64_t)f * m.np);
    const Unit<NC>* pf = reinterpret_cast<const Unit<NC>*>(prev + (int64_t)f * m.np);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) r.t[0][s] = cf[at[s]];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      if (prev) r.t[1][s] = pf[tid + s * T < first_lim ? at[s] : start];
      else
#pragma unroll
        for (int c = 0; c < NC; ++c) r.t[1][s].v[c] = 0.0;
    }
    if (ACC) {
#pragma unroll
      for (int s = 0; s < sum_slots(SLOTS); ++s) {
        const int i = tid + s * T < inside ? tid + s * T : 0;
        const double* xr = x + ((int64_t)f * m.np + (int64_t)(start + i) * NC) * ACC;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int a = 0; a < ACC; ++a) r.acc[s][a][c] = prev ? xr[c * ACC + a] : coef[a] * r.t[0][s].v[c];
      }
    }
    // the loads end here (vmcnt 0): waited for inside a step, they would be
    // waited for together with the stores of the steps before
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();  // the previous field's last step has been read
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (tid + s * T < loaded) reinterpret_cast<Unit<NC>*>(lds)[tid + s * T] = r.t[0][s];
    __syncthreads();
    Unit<NC>* of = reinterpret_cast<Unit<NC>*>(out + (int64_t)f * m.np) + start;
    const int64_t up = plane / NC;
    Coef cj = (Coef)(uintptr_t)(coef + ACC);
    for (int j = 1; j <= steps; j += 2, cj += 2 * ACC) {
      // the plane of step j: every step's own, or the last two's
      Unit<NC>* to = ACC == 0 ? of + (j - 1) * up : j >= steps - 1 ? of + (j - steps + 1) * up : nullptr;
      step_all<NC, W, BV, SLOTS, T, ACC, PAST, 0>(r, lds, tid, __builtin_amdgcn_readlane(ends, ringed ? steps - j : 0), inside,
                                        !prev && j == 1 ? 0.5 : 1.0, to, cj);
      __syncthreads();
      if (j == steps) break;
      to = ACC == 0 || j + 1 >= steps - 1 ? of + (ACC == 0 ? j : j - steps + 2) * up : nullptr;
      step_all<NC, W, BV, SLOTS, T, ACC, PAST, 1>(r, lds, tid, __builtin_amdgcn_readlane(ends, ringed ? steps - j - 1 : 0),
                                        inside, 1.0, to, cj + ACC);
      __syncthreads();
    }
    if (ACC) {
#pragma unroll
      for (int s = 0; s < sum_slots(SLOTS); ++s) {
        const int i = tid + s * T;
        double* xr = x + ((int64_t)f * m.np + (int64_t)(start + i) * NC) * ACC;
        if (i < inside)
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int a = 0; a < ACC; ++a) xr[c * ACC + a] = r.acc[s][a][c];
      }
    }
  }
}

// Block-wide sum of one value per thread in a fixed order (valid in thread 0).
template <int T>
__device__ __forceinline__ double block_total(double v, double* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if (threadIdx.x % 64 == 0) lds[threadIdx.x / 64] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < T / 64; ++w) t += lds[w];
  return t;
}

// Fields in the caller's numbering -> rows (grid.y = field), with ||M phi||^2
// by block; a NaN or Inf sets *bad to the call's number. Bound by HBM (the
// order is local: 16 level-9 fields 172 us, 3.1 TB/s).
__global__ __launch_bounds__(kRed) void k_poly_load(PolyDev m, const double* __restrict__ fields,
                                                    double* __restrict__ phi, double* __restrict__ part,
                                                    int* __restrict__ bad, int call) {
  __shared__ double lds[kRed / 64];
  const double* src = fields + (int64_t)blockIdx.y * m.field_len;
  double* dst = phi + (int64_t)blockIdx.y * m.np;
  double sum = 0.0;
  bool ok = true;
  for (int64_t r = (int64_t)blockIdx.x * kRed + threadIdx.x; r < m.np; r += (int64_t)gridDim.x * kRed) {
    double v = 0.0;
    if (r < m.rows) {
      v = src[m.entity[r]];
      ok = ok && isfinite(v);
      const double b = m.mass[r] * v;
      sum += b * b;
    }
    dst[r] = v;
  }
  if (!ok) *bad = call;
  const double t = block_total<kRed>(sum, lds);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
}

// x (rows x SC) = or += sum over k of coef[k][s] t_k, one thread per row
// (grid.y = field): each t_k is read once for SC scales, the coefficients
// come through the scalar cache. phi != nullptr: the sum starts with
// coef[0] phi, and coef + SC belongs to the first of the n planes. SB > 0:
// the next group's SB scales too, of at most n planes (nb of them), so that
// their vectors are read once for both (all stores come last: a store before
// the second loop would send its coefficients through vector loads). Bound by
// HBM: 5.2 TB/s over 8 level-9 fields x 16 scales, 4.2 TB/s x 32; 30 scales
// of 16 fields 10.3 ms, with the groups' vectors read apart 11.5 (two rows
// and 16-byte loads a thread: the same, and twice as long on small meshes).
template <int SC, int SB>
__global__ __launch_bounds__(kRed) void k_poly_sum(const double* __restrict__ phi, const double* __restrict__ t,
                                                   int64_t plane, int64_t np, int n,
                                                   const double* __restrict__ coef, double* __restrict__ x, int nb,
                                                   const double* __restrict__ coefb, double* __restrict__ xb) {
  const int64_t r = (int64_t)blockIdx.x * kRed + threadIdx.x;
  if (r >= np) return;
  const int64_t at = (int64_t)blockIdx.y * np + r;
  double acc[SC], accb[SB > 0 ? SB : 1];
  double* xr = x + at * SC;
  double* xbr = xb + at * SB;
  if (phi) {
    const double v = phi[at];
#pragma unroll
    for (int s = 0; s < SC; ++s) acc[s] = coef[s] * v;
#pragma unroll
    for (int s = 0; s < SB; ++s) accb[s] = coefb[s] * v;
    coef += SC;
    coefb += SB;
  } else {
#pragma unroll
    for (int s = 0; s < SC; ++s) acc[s] = xr[s];
#pragma unroll
    for (int s = 0; s < SB; ++s) accb[s] = xbr[s];
  }
  const double* tr = t + at;
  int k = 0;
  if constexpr (SB > 0) {
#pragma unroll 8
    for (; k < nb; ++k) {
      const double v = __builtin_nontemporal_load(tr + (int64_t)k * plane);
#pragma unroll
      for (int s = 0; s < SC; ++s) acc[s] += coef[(int64_t)k * SC + s] * v;
#pragma unroll
      for (int s = 0; s < SB; ++s) accb[s] += coefb[(int64_t)k * SB + s] * v;
    }
  }
#pragma unroll 16
  for (; k < n; ++k) {
    const double v = __builtin_nontemporal_load(tr + (int64_t)k * plane);
#pragma unroll
    for (int s = 0; s < SC; ++s) acc[s] += coef[(int64_t)k * SC + s] * v;
  }
#pragma unroll
  for (int s = 0; s < SC; ++s) xr[s] = acc[s];
#pragma unroll
  for (int s = 0; s < SB; ++s) xbr[s] = accb[s];
}

// Lanes of a row of SC scales, and a lane's scales.
constexpr int lane_scales(int sc) { return sc >= 2 ? 2 : 1; }

template <int V>
struct Lane;
template <>
struct Lane<1> {
  double v[1];
};
template <>
struct alignas(16) Lane<2> {
  double v[2];
};

// High words of a lane's doubles: magnitudes, of which 20 bits are plenty.
template <int V>
struct alignas(4 * V) LaneHigh {
  int v[V];
};

// The unit's product with A: y[c] = sum_j A_uj x_j, component c, for the
// lane's scales, and the sizes of its terms, mag[c] = sum_j |A_uj| s_j (MAG 1:
// s = |x|, MAG 2: what sizes holds). A unit's rows share their gathers.
template <int NC, int W, int BV, int SC, int MAG = 0>
__device__ __forceinline__ void unit_product(const PolyDev& m, const double* xf, int64_t u, int q,
                                             Lane<lane_scales(SC)> (&y)[NC],
                                             Lane<lane_scales(SC)> (*mag)[NC] = nullptr, const int* sizes = nullptr) {
  constexpr int V = lane_scales(SC);
  const Lane<V>* xt = reinterpret_cast<const Lane<V>*>(xf);
  const LaneHigh<V>* st = reinterpret_cast<const LaneHigh<V>*>(sizes);
  constexpr int LPR = SC / V, VR = poly_val_record(W, BV), CR = poly_col_record(W);
  int32_t col[CR];
#pragma unroll
  for (int k = 0; k < CR; k += 4) {
    const int4 q4 = *reinterpret_cast<const int4*>(m.col + u * CR + k);
    col[k] = q4.x;
    col[k + 1] = q4.y;
    col[k + 2] = q4.z;
    col[k + 3] = q4.w;
  }
  const double* a = m.val + u * VR;
  Lane<V> t[W + 1][NC];
  LaneHigh<V> h[MAG == 2 ? W + 1 : 1][NC];
#pragma unroll
  for (int k = 0; k <= W; ++k)
#pragma unroll
    for (int d = 0; d < NC; ++d) {
      const int64_t at = ((k == 0 ? u : (int64_t)col[k == 0 ? 0 : k - 1]) * NC + d) * LPR + q;
      t[k][d] = xt[at];
      if (MAG == 2) h[MAG == 2 ? k : 0][d] = st[at];
    }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      y[c].v[e] = 0.0;
      if (MAG) (*mag)[c].v[e] = 0.0;
    }
#pragma unroll
    for (int k = 0; k <= W; ++k)
#pragma unroll
      for (int d = 0; d < NC; ++d) {
        double v;
        if constexpr (BV == 1) v = k == 0 ? minus_sum<W>(a) : a[k == 0 ? 0 : k - 1];
        else v = coupling<NC, BV>(a + k * BV, c, d);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          y[c].v[e] += v * t[k][d].v[e];
          if (MAG)
            (*mag)[c].v[e] +=
                fabs(v) * (MAG == 2 ? __hiloint2double(h[MAG == 2 ? k : 0][d].v[e], 0) : fabs(t[k][d].v[e]));
        }
      }
  }
}

// y = A x and the high words of |A| |x| (grid.y = field), a lane's scales of
// one unit per thread.
template <int NC, int W, int BV, int SC>
__global__ __launch_bounds__(kRed) void k_poly_apply(PolyDev m, const double* __restrict__ x, double* __restrict__ y,
                                                     int* __restrict__ sizes) {
  constexpr int V = lane_scales(SC), LPR = SC / V;
  const int64_t g = (int64_t)blockIdx.x * kRed + threadIdx.x;
  const int64_t u = g / LPR;
  if (u >= m.units) return;
  const int64_t base = (int64_t)blockIdx.y * m.np * SC;
  const int q = (int)(g % LPR);
  Lane<V> v[NC], mag[NC];
  unit_product<NC, W, BV, SC, 1>(m, x + base, u, q, v, &mag);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    reinterpret_cast<Lane<V>*>(y + base)[(u * NC + c) * LPR + q] = v[c];
    LaneHigh<V> h;
#pragma unroll
    for (int e = 0; e < V; ++e) h.v[e] = __double2hiint(mag[c].v[e]);
    reinterpret_cast<LaneHigh<V>*>(sizes + base)[(u * NC + c) * LPR + q] = h;
  }
}

struct GroupScales {
  double c[kMaxGroup];      // scale factors
  int32_t column[kMaxGroup]; // index of the scale in the call's list, -1: padding
};

// FP64 true residual M (phi - x - c A z), z = x (order 1) or A x (order 2):
// block sums of its square, of the squared sizes of its terms row by row, M
// (|phi| + |x| + c |A| |z|) (the residual's rounding error is a small multiple
// of u times their norm; order 2, TWICE: |A| |x| for |z|, from sizes), and of
// M x^2 per scale. Bound by the gathers, which come from L2: a row and its
// neighbours, 128 bytes each of 16 scales (8 level-9 fields 1.08 ms, 11 TB/s
// of gathers, 1.7 TB/s of HBM).
template <int NC, int W, int BV, int SC, bool TWICE>
__global__ __launch_bounds__(kRed) void k_poly_check(PolyDev m, const double* __restrict__ phi,
                                                     const double* __restrict__ x, const double* __restrict__ z,
                                                     const int* __restrict__ sizes, GroupScales gs,
                                                     double* __restrict__ part) {
  constexpr int V = lane_scales(SC), LPR = SC / V;
  __shared__ double lds[kRed / 64][LPR][3 * V];
  const int64_t base = (int64_t)blockIdx.y * m.np * SC;
  const double* pf = phi + (int64_t)blockIdx.y * m.np;
  const int q = threadIdx.x % LPR;
  double sum[3 * V];
#pragma unroll
  for (int e = 0; e < 3 * V; ++e) sum[e] = 0.0;
  constexpr int UPB = kRed / LPR;
  for (int64_t u = (int64_t)blockIdx.x * UPB + threadIdx.x / LPR; u < m.units; u += (int64_t)gridDim.x * UPB) {
    Lane<V> y[NC], mag[NC];
    unit_product<NC, W, BV, SC, TWICE ? 2 : 1>(m, z + base, u, q, y, &mag, sizes + base);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int64_t r = u * NC + c;
      const Lane<V> xr = reinterpret_cast<const Lane<V>*>(x + base)[r * LPR + q];
      const double mr = m.mass[r], ph = pf[r];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const double res = mr * (ph - xr.v[e] - gs.c[q * V + e] * y[c].v[e]);
        const double size = mr * (fabs(ph) + fabs(xr.v[e]) + gs.c[q * V + e] * mag[c].v[e]);
        sum[e] += res * res;
        sum[V + e] += size * size;
        sum[2 * V + e] += mr * xr.v[e] * xr.v[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 3 * V; ++e) {
#pragma unroll
    for (int off = 32; off >= LPR; off >>= 1) sum[e] += __shfl_xor(sum[e], off, 64);
  }
  if (threadIdx.x % 64 < LPR)
#pragma unroll
    for (int e = 0; e < 3 * V; ++e) lds[threadIdx.x / 64][q][e] = sum[e];
  __syncthreads();
  if (threadIdx.x < LPR) {
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double t = 0.0;
        for (int w = 0; w < kRed / 64; ++w) t += lds[w][threadIdx.x][k * V + e];
        part[(((int64_t)blockIdx.y * SC + threadIdx.x * V + e) * 3 + k) * gridDim.x + blockIdx.x] = t;
      }
  }
}

// Sums of partials: block b of the first n writes the sum of its g partials
// to dst[b], the others theirs (g2 each) to dst2. dst is pinned host memory:
// no copy follows. bad_dst != nullptr: the flag goes there too.
__global__ __launch_bounds__(kRed) void k_poly_total(const double* __restrict__ part, int g, int n,
                                                     double* __restrict__ dst, const double* __restrict__ part2,
                                                     int g2, double* __restrict__ dst2, const int* __restrict__ bad,
                                                     int* __restrict__ bad_dst) {
  __shared__ double lds[kRed / 64];
  const bool first = (int)blockIdx.x < n;
  const int b = first ? blockIdx.x : blockIdx.x - n, len = first ? g : g2;
  const double* p = (first ? part : part2) + (int64_t)b * len;
  double s = 0.0;
  for (int i = threadIdx.x; i < len; i += kRed) s += p[i];
  const double t = block_total<kRed>(s, lds);
  if (threadIdx.x == 0) (first ? dst : dst2)[b] = t;
  if (bad_dst && blockIdx.x == 0 && threadIdx.x == 0) *bad_dst = *bad;
}

// x (rows x SC) -> the caller's numbering, a thread per caller entry
// (grid.y = field); entries without a row are 0. Nothing is written once a
// field was found bad. Bound by HBM and by the columns being written apart
// (8 level-9 fields x 16 scales 1.11 ms, 3.7 TB/s).
template <int SC>
__global__ __launch_bounds__(kRed) void k_poly_out(PolyDev m, const double* __restrict__ x, GroupScales gs,
                                                   int64_t field_stride, const int* __restrict__ bad, int call,
                                                   double* __restrict__ out) {
  if (*bad == call) return;
  const int64_t i = (int64_t)blockIdx.x * kRed + threadIdx.x;
  if (i >= m.field_len) return;
  const int32_t r = m.row_of[i];
  double v[SC];
  const double* xr = x + ((int64_t)blockIdx.y * m.np + (r < 0 ? 0 : r)) * SC;
#pragma unroll
  for (int s = 0; s < SC; ++s) v[s] = r < 0 ? 0.0 : xr[s];
  double* o = out + (int64_t)blockIdx.y * field_stride + i;
#pragma unroll
  for (int s = 0; s < SC; ++s)
    if (gs.column[s] >= 0) __builtin_nontemporal_store(v[s], o + gs.column[s] * m.field_len);
}

// ---- the spectrum's upper end: Lanczos on A in the M inner product ----
// u_j unnormalised, beta_j = ||u_{j+1}||_M; every block finishes the previous
// launch's sums in the same order, so nothing returns to the host.
__device__ __forceinline__ double partial_total(const double* part, int g, double* lds) {
  double s = 0.0;
  for (int i = threadIdx.x; i < g; i += kRed) s += part[i];
  return block_total<kRed>(s, lds);
}

// a start value of a row, by its place in the caller's numbering
__device__ __forceinline__ double lanczos_noise(const PolyDev& m, int64_t r) {
  uint64_t h = (uint64_t)m.entity[r] * 0x9E3779B97F4A7C15ull + 0xD1B54A32D192ED03ull;
  h ^= h >> 29;
  h *= 0xBF58476D1CE4E5B9ull;
  h ^= h >> 32;
  return (double)(int64_t)h * 1.0842021724855044e-19;
}

__global__ __launch_bounds__(kRed) void k_lanczos_start(PolyDev m, double* __restrict__ u, double* __restrict__ beta) {
  __shared__ double lds[kRed / 64];
  double sum = 0.0;
  for (int64_t r = (int64_t)blockIdx.x * kRed + threadIdx.x; r < m.rows; r += (int64_t)gridDim.x * kRed) {
    const double v = lanczos_noise(m, r);
    u[r] = v;
    sum += m.mass[r] * v * v;
  }
  const double t = block_total<kRed>(sum, lds);
  if (threadIdx.x == 0) beta[blockIdx.x] = t;
}

// w = A v - beta v_prev (v = u / b, v_prev = u_prev / b_prev, beta = b), (w, v)
template <int NC, int W, int BV>
__global__ __launch_bounds__(kRed) void k_lanczos_product(PolyDev m, const double* __restrict__ u,
                                                          const double* __restrict__ u_prev, double* __restrict__ w,
                                                          const double* __restrict__ beta,
                                                          const double* __restrict__ beta_prev,
                                                          double* __restrict__ alpha) {
  __shared__ double lds[kRed / 64];
  const double b = sqrt(partial_total(beta, gridDim.x, lds));
  const double bp = beta_prev ? sqrt(partial_total(beta_prev, gridDim.x, lds)) : 0.0;
  const double inv = b > 0.0 ? 1.0 / b : 0.0, invp = bp > 0.0 ? b / bp : 0.0;
  double sum = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kRed + threadIdx.x; i < m.units; i += (int64_t)gridDim.x * kRed) {
    Lane<1> v[NC];
    unit_product<NC, W, BV, 1>(m, u, i, 0, v);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int64_t r = i * NC + c;
      double y = inv * v[c].v[0];
      if (beta_prev) y -= invp * u_prev[r];
      w[r] = y;
      sum += m.mass[r] * y * u[r] * inv;
    }
  }
  const double t = block_total<kRed>(sum, lds);
  if (threadIdx.x == 0) alpha[blockIdx.x] = t;
}

// w -= alpha v; ||w||_M^2
__global__ __launch_bounds__(kRed) void k_lanczos_next(PolyDev m, const double* __restrict__ u, double* __restrict__ w,
                                                       const double* __restrict__ beta,
                                                       const double* __restrict__ alpha,
                                                       double* __restrict__ beta_next) {
  __shared__ double lds[kRed / 64];
  const double b = sqrt(partial_total(beta, gridDim.x, lds));
  const double a = partial_total(alpha, gridDim.x, lds);
  const double f = b > 0.0 ? a / b : 0.0;
  double sum = 0.0;
  for (int64_t r = (int64_t)blockIdx.x * kRed + threadIdx.x; r < m.rows; r += (int64_t)gridDim.x * kRed) {
    const double y = w[r] - f * u[r];
    w[r] = y;
    sum += m.mass[r] * y * y;
  }
  const double t = block_total<kRed>(sum, lds);
  if (threadIdx.x == 0) beta_next[blockIdx.x] = t;
}

// All of it in one workgroup, for meshes so small that the launches above
// would take longer (32 x 32 units: 0.45 ms in 65 launches). u: 3 vectors of
// np; beta[j], alpha[j] as the sums of those launches.
constexpr int kSmall = 1024;
template <int NC, int W, int BV>
__global__ __launch_bounds__(kSmall) void k_lanczos_small(PolyDev m, double* u, double* beta, double* alpha) {
  __shared__ double lds[kSmall / 64];
  double sum = 0.0;
  for (int64_t r = threadIdx.x; r < m.rows; r += kSmall) {
    u[r] = lanczos_noise(m, r);
    sum += m.mass[r] * u[r] * u[r];
  }
  double b2 = block_total<kSmall>(sum, lds), bp2 = 0.0;
  if (threadIdx.x == 0) beta[0] = b2;
  for (int j = 0; j < kLanczosSmall; ++j) {
    const double *cur = u + j % 3 * m.np, *prev = u + (j + 2) % 3 * m.np;
    double* next = u + (j + 1) % 3 * m.np;
    const double b = sqrt(b2), inv = b > 0.0 ? 1.0 / b : 0.0, invp = bp2 > 0.0 ? b / sqrt(bp2) : 0.0;
    sum = 0.0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < m.units; i += kSmall) {
      Lane<1> v[NC];
      unit_product<NC, W, BV, 1>(m, cur, i, 0, v);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int64_t r = i * NC + c;
        double y = inv * v[c].v[0];
        if (j) y -= invp * prev[r];
        next[r] = y;
        sum += m.mass[r] * y * cur[r] * inv;
      }
    }
    const double a = block_total<kSmall>(sum, lds), f = a * inv;
    if (threadIdx.x == 0) alpha[j] = a;
    sum = 0.0;
    __syncthreads();
    for (int64_t r = threadIdx.x; r < m.rows; r += kSmall) {
      const double y = next[r] - f * cur[r];
      next[r] = y;
      sum += m.mass[r] * y * y;
    }
    bp2 = b2;
    b2 = block_total<kSmall>(sum, lds);
    if (threadIdx.x == 0) beta[j + 1] = b2;
  }
}

}  // namespace

struct PolyState {
  int device = 0;
  PolyDev m;
  void* arrays = nullptr;  // the allocation that m's pointers are in
  int nc = 1, width = 6, block = 1, depth = 0;
  int largest[kPolyDepth + 1] = {};  // local units of the largest patch, up to and with ring d
  bool single = false;
  double lam = 0.0;         // upper end of the spectrum of A, with its margin
  double lam_typical = 0.0; // the same of a mesh whose rows were all like 95% of the rows
  double mass_ratio = 1.0, mass_sum = 0.0;
};

// Work space of one caller at a time, kept between calls. With a limit its
// large arrays live in one allocation of that size.
struct PolyWork {
  size_t limit = 0;         // bytes, 0: arrays grow as calls need them
  int device = 0;
  const PolyState* last = nullptr;  // whose call had it last
  double* arena = nullptr;
  double *phi = nullptr, *t = nullptr, *x = nullptr, *z = nullptr, *in = nullptr, *stage = nullptr;
  size_t phi_n = 0, t_n = 0, x_n = 0, z_n = 0, in_n = 0, stage_n = 0;
  double *part = nullptr, *norm = nullptr, *coef = nullptr;
  int* bad = nullptr;  // number of the last call with a non-finite field
  int call = 0;        // number of the running call
  size_t part_n = 0, norm_n = 0, coef_n = 0;
  double *host = nullptr, *host_coef = nullptr;  // pinned: totals and the bad flag; source of coef
  size_t host_n = 0, host_coef_n = 0;
};

namespace {

// The arrays of a PolyDev in one allocation, sent in one copy.
struct Upload {
  struct Item {
    const void** to;
    const void* from;
    size_t bytes, at;
  };
  std::vector<Item> items;
  size_t bytes = 0;
  template <typename T>
  void add(const T** to, const std::vector<T>& v) {
    items.push_back({(const void**)to, v.data(), v.size() * sizeof(T), bytes});
    bytes += (v.size() * sizeof(T) + 255) / 256 * 256;
  }
  ifl_status run(void** base) {
    if (device_malloc(base, std::max<size_t>(bytes, 256)) != hipSuccess) {
      *base = nullptr;
      return fail(IFL_ENOMEM, "hipMalloc failed for the patches");
    }
    if (bytes <= (size_t)4 << 20) {  // small: gathered on the host
      std::vector<char> all(bytes);
      for (const Item& i : items) std::memcpy(all.data() + i.at, i.from, i.bytes);
      IFL_HIP(hipMemcpy(*base, all.data(), bytes, hipMemcpyHostToDevice));
    } else {
      for (const Item& i : items)
        if (i.bytes) IFL_HIP(hipMemcpy((char*)*base + i.at, i.from, i.bytes, hipMemcpyHostToDevice));
    }
    for (const Item& i : items) *i.to = (char*)*base + i.at;
    return IFL_OK;
  }
};

ifl_status grow(double** p, size_t* have, size_t want) {
  if (*have >= want) return IFL_OK;
  if (*p) (void)hipFree(*p);
  *p = nullptr;
  *have = 0;
  if (device_malloc((void**)p, want * sizeof(double)) != hipSuccess) {
    *p = nullptr;
    return fail(IFL_ENOMEM, "hipMalloc failed for the polynomial engine's work space");
  }
  *have = want;
  return IFL_OK;
}

ifl_status grow_host(double** p, size_t* have, size_t want) {
  if (*have >= want) return IFL_OK;
  if (*p) (void)hipHostFree(*p);
  *p = nullptr;
  *have = 0;
  if (hipHostMalloc((void**)p, want * sizeof(double), hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
    return fail(IFL_ENOMEM, "hipHostMalloc failed for the polynomial engine's work space");
  }
  *have = want;
  return IFL_OK;
}

int red_blocks(int64_t items) { return (int)std::max<int64_t>(1, std::min<int64_t>(kRedBlocks, (items + kRed - 1) / kRed)); }

// One launch of the step kernel: where it reads and writes.
struct Steps {
  const double *prev, *cur;
  double* out;
  int64_t plane;
  int fields, steps;
  const double* coef = nullptr;  // with acc > 0
  double* x = nullptr;
  int acc = 0;
};

template <int NC, int W, int BV, int SLOTS, int T, int ACC, bool PAST>
void steps_acc(const PolyState* ps, const Steps& a, hipStream_t s) {
  const int per = (ps->m.npatch + kXcd - 1) / kXcd;
  // fields side by side only where the patches alone do not fill the chip:
  // a workgroup that walks the fields reads its rows of A once
  const int gy = std::min(a.fields, std::max(1, 1024 / std::max(1, ps->m.npatch)));
  k_poly_steps<NC, W, BV, SLOTS, T, ACC, PAST><<<dim3(per * kXcd, gy), T, 0, s>>>(
      ps->m, a.prev, a.cur, a.out, a.plane, a.fields, a.steps, ps->single ? 0 : 1, 4.0 / ps->lam, a.coef, a.x);
}

// The new vectors go past the caches where most of them are read only by the
// sums, much later, and would push the halos out of L2: several fields, or
// launches of 8 steps (of which the next launch reads the last two). Measured
// plain / past: 8 level-9 fields 440 / 394 us a launch, 8 vertex-vector
// fields 9.4 / 8.8 ms a call, 2 level-7 fields 0.48 / 0.45 ms; but one
// cell-vector field with 4 steps a launch 4.66 / 5.03 ms, and 64 x 64 units,
// whose sequence stays in L2, 207 / 216 us.
bool past_caches(const PolyState* ps, const Steps& a) {
  return (a.fields > 1 || a.steps >= 8) && (int64_t)a.fields * ps->m.np >= 1 << 17;
}

template <int NC, int W, int BV, int SLOTS, int T>
void steps_of(const PolyState* ps, const Steps& a, hipStream_t s) {
  switch (a.acc) {
    case 0:
      if (past_caches(ps, a)) steps_acc<NC, W, BV, SLOTS, T, 0, true>(ps, a, s);
      else steps_acc<NC, W, BV, SLOTS, T, 0, false>(ps, a, s);
      break;
    case 1: steps_acc<NC, W, BV, SLOTS, T, 1, true>(ps, a, s); break;
    case 2:
      if constexpr (SLOTS < 4) steps_acc<NC, W, BV, SLOTS, T, 2, true>(ps, a, s);
      break;
    default:
      if constexpr (NC == 1 && SLOTS < 4) steps_acc<NC, W, BV, SLOTS, T, 4, true>(ps, a, s);
      break;
  }
}

// The smallest workgroup and slot count that hold the patches' units.
void launch_steps(const PolyState* ps, const Steps& a, hipStream_t s) {
  const int L = ps->largest[ps->single ? 0 : a.steps];
  if (ps->nc == 1 && ps->width == 6) {
    if (ps->single && L <= 1024) steps_of<1, 6, 1, 1, kPolySingleThreads>(ps, a, s);
    else if (ps->single) steps_of<1, 6, 1, 2, kPolySingleThreads>(ps, a, s);
    else if (L <= 2 * kPolyThreads) steps_of<1, 6, 1, 2, kPolyThreads>(ps, a, s);
    else steps_of<1, 6, 1, 4, kPolyThreads>(ps, a, s);
  } else if (ps->nc == 1 && ps->width == 8) {
    if (ps->single) steps_of<1, 8, 1, 2, kPolySingleThreads>(ps, a, s);
    else steps_of<1, 8, 1, 2, kPolyThreads>(ps, a, s);
  } else if (ps->nc == 1) {
    if (ps->single) steps_of<1, 12, 1, 2, kPolySingleThreads>(ps, a, s);
    else steps_of<1, 12, 1, 2, kPolyThreads>(ps, a, s);
  } else if (ps->block == 2 && ps->width == 6) {
    if (L <= 512) steps_of<2, 6, 2, 1, 512>(ps, a, s);
    else steps_of<2, 6, 2, 2, 512>(ps, a, s);
  } else if (ps->block == 2) {
    steps_of<2, 8, 2, 1, 1024>(ps, a, s);
  } else if (L <= 1024) {
    steps_of<2, 3, 4, 2, 512>(ps, a, s);
  } else {
    steps_of<2, 3, 4, 2, 1024>(ps, a, s);
  }
}

// Whether the step kernel sums sc scales itself, by launches of 'steps' steps:
// every interior unit has to be in a slot with sums, and their registers have
// to be there. Kernels of 4 slots a thread are full: with 1 scale they spill
// 10 registers and still win (one field of the 2.6 M-vertex sphere: 171 us a
// launch, 150 with its stores past the caches, for 165 + 32 of the separate
// sum, 1.43 ms a call for 1.90), with 4 they lose (level 7: 23 us a launch for
// 15 + 2).
bool sums_itself(const PolyState* ps, int sc, int steps) {
  const bool full = !ps->single && ps->width == 6 && ps->nc == 1 && ps->largest[steps] > 2 * kPolyThreads;
  return sc <= (full ? 1 : ps->nc == 1 ? 4 : 2) &&
         (ps->nc == 2 || ps->single || ps->largest[0] <= 2 * kPolyThreads);
}

// A group's part in a launch of the sums: its scales, vectors, coefficients
// and sums.
struct SumOf {
  int sc = 0, n = 0;
  const double* coef = nullptr;
  double* x = nullptr;
};

template <int SC, int SB>
void sum_of(const double* phi, const double* t, int64_t plane, int64_t np, const SumOf& a, const SumOf& b, int F,
            hipStream_t s) {
  const dim3 g((unsigned)((np + kRed - 1) / kRed), (unsigned)F);
  k_poly_sum<SC, SB><<<g, kRed, 0, s>>>(phi, t, plane, np, a.n, a.coef, a.x, b.n, b.coef, b.x);
}

// One group, or a full one and the next (b.sc > 0, b.n <= a.n).
void launch_sum(const double* phi, const double* t, int64_t plane, int64_t np, const SumOf& a, const SumOf& b, int F,
                hipStream_t s) {
  static_assert(kMaxGroup == 16, "");
  if (b.sc == 0) {
    switch (a.sc) {
      case 1: sum_of<1, 0>(phi, t, plane, np, a, b, F, s); break;
      case 2: sum_of<2, 0>(phi, t, plane, np, a, b, F, s); break;
      case 4: sum_of<4, 0>(phi, t, plane, np, a, b, F, s); break;
      case 8: sum_of<8, 0>(phi, t, plane, np, a, b, F, s); break;
      default: sum_of<16, 0>(phi, t, plane, np, a, b, F, s); break;
    }
    return;
  }
  switch (b.sc) {
    case 1: sum_of<16, 1>(phi, t, plane, np, a, b, F, s); break;
    case 2: sum_of<16, 2>(phi, t, plane, np, a, b, F, s); break;
    case 4: sum_of<16, 4>(phi, t, plane, np, a, b, F, s); break;
    case 8: sum_of<16, 8>(phi, t, plane, np, a, b, F, s); break;
    default: sum_of<16, 16>(phi, t, plane, np, a, b, F, s); break;
  }
}

template <int NC, int W, int BV, int SC>
void check_of(const PolyState* ps, int order, const double* phi, const double* x, double* z, int* sizes,
              const GroupScales& gs, double* part, int G, int F, hipStream_t s) {
  constexpr int LPR = SC / lane_scales(SC);
  if (order == 2) {
    const dim3 g((unsigned)((ps->m.units * LPR + kRed - 1) / kRed), (unsigned)F);
    k_poly_apply<NC, W, BV, SC><<<g, kRed, 0, s>>>(ps->m, x, z, sizes);
    k_poly_check<NC, W, BV, SC, true><<<dim3(G, F), kRed, 0, s>>>(ps->m, phi, x, z, sizes, gs, part);
  } else {
    k_poly_check<NC, W, BV, SC, false><<<dim3(G, F), kRed, 0, s>>>(ps->m, phi, x, x, nullptr, gs, part);
  }
}

template <int NC, int W, int BV>
void check_scales(const PolyState* ps, int sc, int order, const double* phi, const double* x, double* z, int* sizes,
                  const GroupScales& gs, double* part, int G, int F, hipStream_t s) {
  switch (sc) {
    case 1: check_of<NC, W, BV, 1>(ps, order, phi, x, z, sizes, gs, part, G, F, s); break;
    case 2: check_of<NC, W, BV, 2>(ps, order, phi, x, z, sizes, gs, part, G, F, s); break;
    case 4: check_of<NC, W, BV, 4>(ps, order, phi, x, z, sizes, gs, part, G, F, s); break;
    case 8: check_of<NC, W, BV, 8>(ps, order, phi, x, z, sizes, gs, part, G, F, s); break;
    default: check_of<NC, W, BV, 16>(ps, order, phi, x, z, sizes, gs, part, G, F, s); break;
  }
}

// f with the operator's (components, entries a unit, couplings a block) as
// its template arguments
#define IFL_POLY_FORMS(f, ...)                                  \
  do {                                                          \
    if (ps->nc == 1) {                                          \
      if (ps->width == 6) f<1, 6, 1> __VA_ARGS__;               \
      else if (ps->width == 8) f<1, 8, 1> __VA_ARGS__;          \
      else f<1, 12, 1> __VA_ARGS__;                             \
    } else if (ps->block == 2) {                                \
      if (ps->width == 6) f<2, 6, 2> __VA_ARGS__;               \
      else f<2, 8, 2> __VA_ARGS__;                              \
    } else {                                                    \
      f<2, 3, 4> __VA_ARGS__;                                   \
    }                                                           \
  } while (0)

void launch_out(const PolyState* ps, const int* bad, int call, int sc, const double* x, const GroupScales& gs,
                int64_t field_stride, double* out, int F, hipStream_t s) {
  const dim3 g((unsigned)((ps->m.field_len + kRed - 1) / kRed), (unsigned)F);
  switch (sc) {
    case 1: k_poly_out<1><<<g, kRed, 0, s>>>(ps->m, x, gs, field_stride, bad, call, out); break;
    case 2: k_poly_out<2><<<g, kRed, 0, s>>>(ps->m, x, gs, field_stride, bad, call, out); break;
    case 4: k_poly_out<4><<<g, kRed, 0, s>>>(ps->m, x, gs, field_stride, bad, call, out); break;
    case 8: k_poly_out<8><<<g, kRed, 0, s>>>(ps->m, x, gs, field_stride, bad, call, out); break;
    default: k_poly_out<16><<<g, kRed, 0, s>>>(ps->m, x, gs, field_stride, bad, call, out); break;
  }
}

// lam from Lanczos; least: the part of the largest eigenvector that a start
// vector has, but for one in a thousand.
ifl_status estimate_spectrum(PolyState* ps, double least, hipStream_t s) {
  const PolyDev& m = ps->m;
  const bool small = m.rows <= 4096;
  const int G = small ? 1 : std::min(256, red_blocks(m.rows)), steps = small ? kLanczosSmall : kLanczos;
  const size_t nab = (size_t)(2 * steps + 1) * G;
  double* work = nullptr;  // three vectors, then the sums
  size_t have = 0;
  ifl_status st = grow(&work, &have, 3 * (size_t)m.np + nab);
  if (st != IFL_OK) return st;
  std::vector<double> parts(nab);
  double *u[3] = {work, work + m.np, work + 2 * m.np}, *beta = work + 3 * m.np;
  double* alpha = beta + (size_t)(steps + 1) * G;
  if (small) {
    IFL_POLY_FORMS(k_lanczos_small, <<<1, kSmall, 0, s>>>(m, work, beta, alpha));
  } else {
    k_lanczos_start<<<G, kRed, 0, s>>>(m, u[0], beta);
    for (int j = 0; j < steps; ++j) {
      double *cur = u[j % 3], *next = u[(j + 1) % 3], *prev = u[(j + 2) % 3];
      const double* bp = j ? beta + (size_t)(j - 1) * G : nullptr;
      IFL_POLY_FORMS(k_lanczos_product,
                     <<<G, kRed, 0, s>>>(m, cur, prev, next, beta + (size_t)j * G, bp, alpha + (size_t)j * G));
      k_lanczos_next<<<G, kRed, 0, s>>>(m, cur, next, beta + (size_t)j * G, alpha + (size_t)j * G,
                                        beta + (size_t)(j + 1) * G);
    }
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(parts.data(), beta, nab * sizeof(double), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(work);
  if (e != hipSuccess) return fail(IFL_EDEVICE, std::string("spectrum estimate: ") + hipGetErrorString(e));
  std::vector<double> a, b;  // alpha_0 .., and beta_1 ..
  double first = 0.0;
  for (int j = 0; j <= steps; ++j) {
    double bj = 0.0, aj = 0.0;
    for (int i = 0; i < G; ++i) bj += parts[(size_t)j * G + i];
    bj = std::sqrt(bj);
    if (j == 0) first = bj;
    // the space is exhausted (few rows): the eigenvalues so far are exact
    if (!(bj > 0.0) || (j > 0 && bj <= 1e-10 * std::fabs(a[0]))) break;
    if (j > 0) b.push_back(bj);
    if (j == steps) break;
    for (int i = 0; i < G; ++i) aj += parts[(size_t)(steps + 1 + j) * G + i];
    a.push_back(aj);
  }
  ps->lam = a.empty() || !(first > 0.0) ? 0.0 : spectrum_bound(a.data(), b.data(), (int)a.size(), (int)b.size(), least);
  return IFL_OK;
}

}  // namespace

static ifl_status create(const HostOperator& op, bool local_order, hipStream_t s, PolyState** out) {
  PatchPack pp;
  if (!build_patches(op, local_order, &pp)) return IFL_OK;
  PolyState* ps = new PolyState();
  *out = ps;
  IFL_HIP(hipGetDevice(&ps->device));
  ps->nc = pp.nc;
  ps->width = pp.width;
  ps->block = pp.block;
  ps->depth = pp.depth;
  for (const PatchInfo& p : pp.patches)
    for (int d = 0; d <= kPolyDepth; ++d) ps->largest[d] = std::max(ps->largest[d], p.end[d]);
  ps->single = pp.single;
  ps->mass_ratio = pp.mass_ratio;
  for (double a : op.mass) ps->mass_sum += a;
  PolyDev& m = ps->m;
  m.units = pp.units;
  m.rows = pp.units * pp.nc;
  m.np = (m.rows + 63) / 64 * 64;
  m.field_len = op.field_len;
  m.npatch = (int)pp.patches.size();
  std::vector<int32_t> entity((size_t)m.rows), row_of((size_t)op.field_len, -1);
  for (int64_t i = 0; i < pp.units; ++i)
    for (int c = 0; c < pp.nc; ++c) {
      const int64_t r = i * pp.nc + c;
      entity[r] = (int32_t)op.entity[(int64_t)pp.order[i] * pp.nc + c];
      row_of[entity[r]] = (int32_t)r;
    }
  Upload u;
  u.add(&m.info, pp.patches);
  u.add(&m.halo, pp.halo);
  u.add(&m.idx, pp.idx);
  u.add(&m.col, pp.col);
  u.add(&m.val, pp.val);
  u.add(&m.mass, pp.mass);
  u.add(&m.entity, entity);
  u.add(&m.row_of, row_of);
  ifl_status st = u.run(&ps->arrays);
  if (st != IFL_OK) return st;
  {
    std::vector<double> d((size_t)m.rows);
    const int rec = poly_val_record(pp.width, pp.block);
    for (int64_t r = 0; r < m.rows; ++r) {
      const double* v = &pp.val[(size_t)(r / pp.nc * rec)];
      if (pp.block == 1)
        for (int k = 0; k < pp.width; ++k) d[r] -= v[k];
      else
        d[r] = v[pp.block == 4 ? r % 2 * 3 : 0];
    }
    const size_t at = d.size() - 1 - d.size() / 20;
    std::nth_element(d.begin(), d.begin() + at, d.end());
    ps->lam_typical = 2.0 * d[at];
  }
  PolyWork* w = nullptr;  // the first call finds one made
  if ((st = poly_work_create(0, &w)) != IFL_OK) return st;
  poly_work_return(ps, w);
  // (the noise is uniform in the rows: the part is smallest in an eigenvector
  // of the row of least mass alone)
  return estimate_spectrum(ps, 1e-3 * std::sqrt(*std::min_element(op.mass.begin(), op.mass.end()) / ps->mass_sum), s);
}

ifl_status poly_create(const HostOperator& op, bool local_order, hipStream_t s, PolyState** out) {
  *out = nullptr;
  if (op.order < 1 || op.order > 2 || op.field_len > INT32_MAX) return IFL_OK;
  try {
    return create(op, local_order, s, out);
  } catch (const std::bad_alloc&) {
    return fail(IFL_ENOMEM, "out of host memory for the patches");
  }
}

void poly_work_trim(PolyWork* w) {
  for (auto [p, n] : {std::pair<double**, size_t*>{&w->t, &w->t_n}, {&w->x, &w->x_n}, {&w->z, &w->z_n},
                      {&w->in, &w->in_n}, {&w->stage, &w->stage_n}}) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    *n = 0;
  }
}

ifl_status poly_work_create(size_t limit, PolyWork** out) {
  PolyWork* w = new PolyWork();
  *out = w;
  w->limit = limit;
  (void)hipGetDevice(&w->device);
  size_t n = 0;
  ifl_status st = IFL_OK;
  if (limit) st = grow(&w->arena, &n, limit / sizeof(double));
  if (st == IFL_OK && (hipMalloc((void**)&w->bad, sizeof(int)) != hipSuccess ||
                       hipMemset(w->bad, 0, sizeof(int)) != hipSuccess || hipDeviceSynchronize() != hipSuccess)) {
    (void)hipGetLastError();
    st = fail(IFL_ENOMEM, "hipMalloc failed for the polynomial engine's work space");
  }
  if (st != IFL_OK) {
    poly_work_destroy(w);
    *out = nullptr;
  }
  return st;
}

void poly_work_destroy(PolyWork* w) {
  if (!w) return;
  if (!w->limit) {
    poly_work_trim(w);
    if (w->phi) (void)hipFree(w->phi);
  }
  void* ptrs[] = {w->arena, w->part, w->norm, w->coef, w->bad};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  if (w->host) (void)hipHostFree(w->host);
  if (w->host_coef) (void)hipHostFree(w->host_coef);
  delete w;
}

// Work spaces between calls, at most kIdle bytes of them on a device. A call
// takes the one of its handle's last call if that is large enough, else the
// smallest that is, so that many large handles used in turn hold one together
// (handles used at the same time grow one each).
namespace {

constexpr size_t kIdle = (size_t)16 << 30;
std::mutex g_idle_mu;
std::vector<PolyWork*> g_idle;  // least recently used first

size_t work_bytes(const PolyWork* w) {
  return sizeof(double) * (w->phi_n + w->t_n + w->x_n + w->z_n + w->in_n + w->stage_n + w->part_n + w->norm_n +
                           w->coef_n);
}

// Frees the idle work spaces that 'which' is true of; whether there were any.
template <typename F>
bool drop_idle(const F& which) {
  std::vector<PolyWork*> drop;
  {
    std::lock_guard<std::mutex> lk(g_idle_mu);
    const auto from = std::stable_partition(g_idle.begin(), g_idle.end(), [&](PolyWork* w) { return !which(w); });
    drop.assign(from, g_idle.end());
    g_idle.erase(from, g_idle.end());
  }
  for (PolyWork* w : drop) poly_work_destroy(w);
  return !drop.empty();
}

}  // namespace

ifl_status poly_work_borrow(PolyState* ps, int32_t n_fields, int32_t n_scales, PolyWork** out) {
  // half of what the call will need, roughly: a hundred vectors a field beside
  // its scales, within the budget
  const double need = 0.5 * std::min((double)kPolyBudget, 8.0 * ps->m.np * n_fields * (n_scales + 100.0));
  {
    std::lock_guard<std::mutex> lk(g_idle_mu);
    int own = -1, enough = -1;
    for (int i = 0; i < (int)g_idle.size(); ++i) {
      if (g_idle[i]->device != ps->device) continue;
      const size_t bytes = work_bytes(g_idle[i]);
      if (g_idle[i]->last == ps) own = i;
      if (bytes >= need && (enough < 0 || bytes < work_bytes(g_idle[enough]))) enough = i;
    }
    const int take = own >= 0 && (enough < 0 || work_bytes(g_idle[own]) >= need) ? own : enough;
    if (take >= 0) {
      *out = g_idle[take];
      g_idle.erase(g_idle.begin() + take);
      return IFL_OK;
    }
  }
  return poly_work_create(0, out);
}

void poly_work_return(PolyState* ps, PolyWork* w) {
  if (!w) return;
  w->last = ps;
  std::vector<PolyWork*> drop;
  {
    std::lock_guard<std::mutex> lk(g_idle_mu);
    try {
      drop.reserve(g_idle.size() + 1);
      g_idle.push_back(w);
    } catch (const std::bad_alloc&) {
      poly_work_destroy(w);
      return;
    }
    size_t bytes = 0;
    for (size_t i = g_idle.size(); i-- > 0;) {
      if (g_idle[i]->device != ps->device) continue;
      if (bytes + work_bytes(g_idle[i]) > kIdle) {
        drop.push_back(g_idle[i]);
        g_idle.erase(g_idle.begin() + (int64_t)i);
      } else {
        bytes += work_bytes(g_idle[i]);
      }
    }
  }
  for (PolyWork* d : drop) poly_work_destroy(d);
}

hipError_t device_malloc(void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) return e;
  (void)hipGetLastError();
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || !drop_idle([&](const PolyWork* w) { return w->device == device; }))
    return e;
  if ((e = hipMalloc(p, bytes)) != hipSuccess) (void)hipGetLastError();
  return e;
}

void poly_destroy(PolyState* ps) {
  if (!ps) return;
  if (ps->arrays) (void)hipFree(ps->arrays);
  drop_idle([&](const PolyWork* w) { return w->last == ps; });
  delete ps;
}

namespace {

// What the residual polynomial is kept within: a fiftieth of the tolerance, of
// order 2 a hundredth. CG, which overshoots it between its tests, leaves columns
// 1e-13 from an exact solution, but energies, which feel the large scales most,
// and columns of the shifted solves only 1e-14 to 4e-14. A twentieth (with a
// residual that was not 0 at the largest scales) left 2e-14 to 8e-14 of these,
// and of a spectrum's densities at level 8 7e-12 (n = 2 1e-10) for CG's 5e-12
// (1.3e-11); now 1e-14 to 3e-14, 2.5e-12 and 3e-12. It costs 3% of the products,
// and 9% where n = 2 reaches 32 cells: there the least degrees lie 30 apart.
// Less where the masses differ so much that the residual's norm can outgrow the
// polynomial's bound (their ratio's root, beyond the 4 that meshes with a
// coastline have without it).
double poly_tol(const PolyState* ps, const PolyCall& c) {
  return std::max(1e-15, (c.order == 1 ? 0.02 : 0.01) * c.rtol / std::max(1.0, 0.25 * std::sqrt(ps->mass_ratio)));
}

double scale_factor(const PolyCall& c, int32_t j) { return c.gamma / std::pow(c.k[j], 2.0 * c.order); }

// About how many products a scale needs with lam as the spectrum's end.
double steps_needed(int order, double c, double lam, double tol) {
  const double b = std::pow(c, 1.0 / order) * lam;
  return 0.5 * std::log(2.0 / tol) * std::sqrt(order == 1 ? 1.0 + b : 1.0 + 2.0 * b);
}

}  // namespace

bool poly_takes(const PolyState* ps, const PolyCall& c) {
  if (!ps || !(ps->lam > 0.0) || c.n_fields > 65535) return false;
  const double tol = poly_tol(ps, c), side = std::sqrt((double)ps->m.units);
  double most = 0.0, cg = 0.0, few = 0.0;
  bool rounds = false;
  for (int32_t j = 0; j < c.n_scales; ++j) {
    const double f = scale_factor(c, j);
    if (!(f > 0.0) || !std::isfinite(f)) return false;
    const double steps = steps_needed(c.order, f, ps->lam, tol), its = steps_needed(c.order, f, ps->lam_typical, tol);
    most = std::max(most, steps);
    cg += its;
    // where the scale outgrows the mesh CG has resolved its modes: order 1,
    // 1,000 cells, 212 iterations on 32 x 32, 382 on 64 x 64, 700 on 128 x 128,
    // 1,208 on 256 x 256; shifted systems of order 2, 250 cells, 280 and 488 on
    // the first two (K_2 itself takes thousands)
    few += c.order == 1 ? std::min(its, 6.5 * side) : c.shifted ? std::min(its, 9.0 * side) : its;
    // about the largest residual that rounding leaves, per ||M phi||: of smooth
    // fields whose filtered part is small (a sequence at the edge z = -1 loses
    // a digit for every one of its length, until the mesh's own lowest mode;
    // order 2 at 64 cells 4e-12, order 1 at 250 cells of 256 x 256 1.1e-12)
    const double u = 1.1102230246251565e-16;
    const double left = c.order == 1 ? u * std::min(0.017 * steps * steps, 0.08 * steps * side)
                                     : 0.12 * u * f * std::pow(ps->lam, 2.0);
    rounds = rounds || left > c.rtol;
  }
  // a step of the sequence costs less than half a CG iteration of one
  // column (2.6 M rows: 19 us for 90; 4,096 rows: 1 us for 12); lam exceeds
  // lam_typical where a few cells are much smaller than the rest, which CG
  // mostly does not feel and the sequence does
  if (!(most < 0.8 * c.max_iter && most <= 2.0 * cg + 8.0)) return false;
  // 64 x 64, one scale: 250 cells 1.3 ms for CG's 3.4, 1,000 cells 5.1 for 4.1
  if (most > 5.0 * few) return false;
  // where columns may have to be solved again by CG, only if the sequence
  // is short beside that (256 x 256, one scale: 250 cells 1.3 of 10 ms, 1,000
  // cells 6 of 19), and not where a few small cells set lam: the rounding
  // grows with lam, what CG's rule lets pass with the rows' own
  return !rounds || (most <= 2.0 * few && std::pow(ps->lam / ps->lam_typical, c.order) <= 7.0);
}

namespace {

// How a call goes through the work space: scales per sequence, vectors of
// the sequence kept at a time, steps of a launch (a launch must not write
// where the two vectors it starts from are), fields at a time, and outputs
// staged for the host at a time and field; false: not even one scale and one
// field fit.
struct Plan {
  int scales = 0, planes = 0, steps = 0, fields = 0, staged = 0;
};

int padded_scales(int n) {
  int p = n / kMaxGroup * kMaxGroup, r = 1;
  if (n % kMaxGroup == 0) return p;
  while (r < n % kMaxGroup) r *= 2;
  return p + r;
}

bool make_plan(const PolyState* ps, size_t limit, const PolyCall& c, int degree, Plan* out) {
  const PolyDev& m = ps->m;
  const size_t have = (limit ? limit : kPolyBudget) / sizeof(double);
  // 4: the two pairs of a sequence summed as it goes; 8: the sizes of a check of order 2
  const int least = std::max(c.order == 2 ? kMaxGroup / 2 : 4, std::min(degree, 16));
  const int F = c.n_fields;
  for (int sc = c.n_scales;; sc = (sc + 1) / 2) {
    const size_t group = (size_t)padded_scales(std::min(sc, kMaxGroup));
    const size_t rest = limit ? (size_t)F * m.np + (c.fields_host ? (size_t)F * m.field_len : 0) : 0;
    const size_t vecs = m.np * ((size_t)padded_scales(sc) + (c.order == 2 ? group : 0));
    // (with a limit also for energies alone: the grouping of the scales, and
    // with it the order of their sums, does not depend on the outputs)
    const size_t stage = limit || (c.out && c.out_host) ? (size_t)m.field_len : 0;
    const size_t avail = have > rest ? have - rest : 0;
    if (avail >= vecs + stage + least * (size_t)m.np || (!limit && sc == 1)) {
      out->staged = stage == 0 ? 0 : (int)std::min<size_t>(
          group, avail > vecs + least * (size_t)m.np ? (avail - vecs - least * (size_t)m.np) / stage : 1);
      const size_t field = vecs + out->staged * stage;
      const size_t left = avail > field ? (avail - field) / m.np : 0;
      out->scales = sc;
      // the whole sequence where it fits, so that its vectors are summed once
      // (the sums are read and written again after every part of it), for 8
      // fields if it does (they share a patch's records); fewer fields rather
      // than parts of less than 64 vectors
      const size_t share = avail / (size_t)std::min(F, 8);
      const size_t planes = share > field ? (share - field) / m.np : 0;
      out->planes = (int)std::max<size_t>(
          least, std::min<size_t>({left, (size_t)std::max(least, degree), std::max<size_t>(planes, 64)}));
      out->fields = (int)std::max<size_t>(
          1, std::min<size_t>((size_t)F, avail / (field + (size_t)out->planes * m.np)));
      // where the patches of all fields run one after another on a CU, more
      // rings than a large mesh's patch has cost more than the launches saved
      const bool many = (int64_t)m.npatch * std::min(F, out->fields) > 512;
      out->steps = ps->single ? out->planes : many ? std::min(ps->depth, 8) : ps->depth;
      if (!ps->single && out->planes < degree) {
        out->steps = std::min(out->steps, out->planes / 2);
        out->planes -= out->planes % out->steps;  // whole launches
      }
      return true;
    }
    if (sc == 1) return false;
  }
}

// A group of scales summed together, and where its totals are.
struct Group {
  int sc = 0, n = 0, degree = 0, pad0 = 0;  // scales padded to sc, real ones, largest degree, scales before
  GroupScales gs;
  size_t coef = 0;
};
struct Totals {
  Group g;
  int f0, nf;
  size_t at;
};

}  // namespace

bool poly_work_takes(const PolyState* ps, size_t limit, int order) {
  // (a few small cells that stretch the spectrum 16 times: the engine would
  // decline 4 scales of an octave each)
  if (!ps || !(ps->lam > 0.0) || ps->lam > 16.0 * ps->lam_typical) return false;
  // a request of 4 scales with its field and outputs in host memory, in one
  // sequence
  PolyCall c;
  double some = 0.0;
  c.order = order;
  c.n_fields = 1;
  c.n_scales = 4;
  c.fields_host = c.out_host = true;
  c.out = &some;
  Plan plan;
  return make_plan(ps, limit, c, 64, &plan) && plan.scales == 4;
}

static ifl_status run_call(PolyState* ps, PolyWork* w, const PolyCall& c, std::vector<int64_t>* failed) {
  const auto t0 = std::chrono::steady_clock::now();
  const PolyDev& m = ps->m;
  hipStream_t s = c.stream;
  failed->clear();
  const int S = c.n_scales, F = c.n_fields;
  const double tol = poly_tol(ps, c);
  // the scales' polynomials, largest degree first
  std::vector<int> deg((size_t)S), by((size_t)S);
  for (int j = 0; j < S; ++j) {
    deg[j] = poly_degree(c.order, scale_factor(c, j), ps->lam, tol, c.max_iter);
    by[j] = j;
    if (deg[j] < 0) return fail(IFL_EUNSUPPORTED, "a scale's polynomial exceeds max_iter");
  }
  std::stable_sort(by.begin(), by.end(), [&](int a, int b) { return deg[a] > deg[b]; });
  Plan plan;
  if (!make_plan(ps, w->limit, c, deg[by[0]], &plan))
    return fail(IFL_ENOMEM, "the work space holds no sequence of this mesh");
  const int FG = plan.fields, G = red_blocks(m.rows), GL = red_blocks(m.np);
  // sequences of up to plan.scales scales, each summed in groups
  std::vector<std::vector<Group>> seqs;
  size_t ncoef = 0, nsums = (size_t)F;
  for (int j = 0; j < S;) {
    std::vector<Group> groups;
    int pad = 0;
    for (const int end = std::min(S, j + plan.scales); j < end;) {
      Group g;
      g.n = std::min(kMaxGroup, end - j);
      g.sc = padded_scales(g.n);
      g.degree = deg[by[j]];
      g.pad0 = pad;
      g.coef = ncoef;
      for (int i = 0; i < kMaxGroup; ++i) {
        g.gs.column[i] = i < g.n ? by[j + i] : -1;
        g.gs.c[i] = i < g.n ? scale_factor(c, by[j + i]) : 0.0;
      }
      ncoef += (size_t)(g.degree + 1) * g.sc;
      nsums += (size_t)F * g.sc * 3;
      pad += g.sc;
      j += g.n;
      groups.push_back(g);
    }
    seqs.push_back(std::move(groups));
  }
  const size_t np = (size_t)m.np;
  const size_t group = (size_t)padded_scales(std::min(plan.scales, kMaxGroup));
  const size_t n_phi = F * np, n_t = (size_t)plan.planes * FG * np, n_x = (size_t)FG * padded_scales(plan.scales) * np;
  const size_t n_z = c.order == 2 ? (size_t)FG * group * np : 0;
  const size_t n_in = c.fields_host ? (size_t)F * m.field_len : 0;
  const size_t n_stage = (size_t)FG * plan.staged * m.field_len;
  ifl_status st;
  if (w->limit) {
    if ((n_phi + n_t + n_x + n_z + n_in + n_stage) * sizeof(double) > w->limit)
      return fail(IFL_ENOMEM, "the work space holds no sequence of this mesh");
    double* at = w->arena;
    for (auto [p, n] : {std::pair<double**, size_t>{&w->phi, n_phi}, {&w->t, n_t}, {&w->x, n_x}, {&w->z, n_z},
                        {&w->in, n_in}, {&w->stage, n_stage}}) {
      *p = at;
      at += n;
    }
  } else if ((st = grow(&w->phi, &w->phi_n, n_phi)) || (st = grow(&w->t, &w->t_n, n_t)) ||
             (st = grow(&w->x, &w->x_n, n_x)) || (st = grow(&w->z, &w->z_n, n_z)) ||
             (st = grow(&w->in, &w->in_n, n_in)) || (st = grow(&w->stage, &w->stage_n, n_stage))) {
    return st;
  }
  if ((st = grow(&w->part, &w->part_n, (size_t)FG * kMaxGroup * 3 * G)) ||
      (st = grow(&w->norm, &w->norm_n, (size_t)F * GL)) || (st = grow(&w->coef, &w->coef_n, ncoef)) ||
      (st = grow_host(&w->host, &w->host_n, nsums + 1)) ||
      (st = grow_host(&w->host_coef, &w->host_coef_n, ncoef)))
    return st;
  const int call = ++w->call;
  const double* fields = c.fields;
  if (c.fields_host) {
    IFL_HIP(hipMemcpyAsync(w->in, c.fields, n_in * sizeof(double), hipMemcpyHostToDevice, s));
    fields = w->in;
  }
  k_poly_load<<<dim3(GL, F), kRed, 0, s>>>(m, fields, w->phi, w->norm, w->bad, call);
  IFL_HIP(hipGetLastError());
  int* bad_host = reinterpret_cast<int*>(w->host + nsums);
  if (n_stage) {  // the copies to the host must not start on a bad field
    IFL_HIP(hipMemcpyAsync(bad_host, w->bad, sizeof(int), hipMemcpyDeviceToHost, s));
    IFL_HIP(hipStreamSynchronize(s));
    if (*bad_host == call) return fail(IFL_EINVAL, "field has a NaN or Inf at a wet entry");
  }
  // the coefficients are worked out when the first launches are under way
  bool sent = false;
  auto send_coefficients = [&]() -> ifl_status {
    if (sent) return IFL_OK;
    sent = true;
    for (const auto& groups : seqs)
      for (const Group& g : groups)
        for (int i = 0; i < g.sc; ++i) {
          double* to = w->host_coef + g.coef + i;
          const int d = i < g.n ? deg[g.gs.column[i]] : -1;
          if (d >= 0) poly_coefficients(c.order, g.gs.c[i], ps->lam, d, to, g.sc);
          for (int k = d + 1; k <= g.degree; ++k) to[(size_t)k * g.sc] = 0.0;
        }
    IFL_HIP(hipMemcpyAsync(w->coef, w->host_coef, ncoef * sizeof(double), hipMemcpyHostToDevice, s));
    return IFL_OK;
  };
  std::vector<Totals> totals;  // (no allocation once outputs may have been written)
  size_t sum_at = (size_t)F, n_groups = 0;
  for (const auto& groups : seqs) n_groups += groups.size();
  totals.reserve(n_groups * (size_t)((F + FG - 1) / FG));
  failed->reserve((size_t)S * F);
  for (int f0 = 0; f0 < F; f0 += FG) {
    const int nf = std::min(FG, F - f0);
    const int64_t plane = (int64_t)nf * m.np;
    const double* phi = w->phi + (int64_t)f0 * m.np;
    for (const auto& groups : seqs) {
      const int degree = groups[0].degree;
      const double *prev = nullptr, *cur = phi;
      const bool summing = degree > 0 && groups.size() == 1 && sums_itself(ps, groups[0].sc, plan.steps);
      if (summing && (st = send_coefficients()) != IFL_OK) return st;
      for (int k = 0, pair = 0; summing && k < degree; pair ^= 1) {
        const int d = std::min(plan.steps, degree - k);
        double* to = w->t + 2 * pair * plane;
        launch_steps(ps, {prev, cur, to, plane, nf, d, w->coef + groups[0].coef + (size_t)k * groups[0].sc, w->x,
                          groups[0].sc}, s);
        prev = d >= 2 ? to : cur;
        cur = to + plane;
        k += d;
      }
      for (int k0 = 0; !summing && (k0 < degree || k0 == 0);) {
        const int n = std::min(plan.planes, degree - k0);
        for (int j = 0; j < n;) {
          const int d = std::min(plan.steps, n - j);
          double* to = w->t + (int64_t)j * plane;
          launch_steps(ps, {prev, cur, to, plane, nf, d}, s);
          prev = d >= 2 ? to + (int64_t)(d - 2) * plane : cur;
          cur = to + (int64_t)(d - 1) * plane;
          j += d;
        }
        if ((st = send_coefficients()) != IFL_OK) return st;
        SumOf of[2];  // groups not launched yet: degrees fall from group to group
        for (const Group& g : groups) {
          const int ng = std::min(n, g.degree - k0);
          if (ng <= 0 && k0 > 0) break;
          SumOf& a = of[of[0].sc > 0];
          a = {g.sc, std::max(0, ng), w->coef + g.coef + (size_t)(k0 == 0 ? 0 : k0 + 1) * g.sc,
               w->x + (size_t)g.pad0 * nf * np};
          if (&a == of && &g != &groups.back()) continue;
          launch_sum(k0 == 0 ? phi : nullptr, w->t, plane, m.np, of[0], of[1], nf, s);
          of[0] = of[1] = SumOf();
        }
        if (of[0].sc > 0) launch_sum(k0 == 0 ? phi : nullptr, w->t, plane, m.np, of[0], of[1], nf, s);
        IFL_HIP(hipGetLastError());
        k0 += n;
        if (n == 0) break;
      }
      for (const Group& g : groups) {
        const double* x = w->x + (size_t)g.pad0 * nf * np;
        // (the sequence is done with: its space holds the sizes, half of g.sc vectors)
        IFL_POLY_FORMS(check_scales, (ps, g.sc, c.order, phi, x, w->z, reinterpret_cast<int*>(w->t), g.gs, w->part, G,
                                      nf, s));
        // with the call's last group go the norms of all its fields
        const bool last = f0 + nf == F && &g == &seqs.back().back();
        const int n = nf * g.sc * 3;
        k_poly_total<<<n + (last ? F : 0), kRed, 0, s>>>(w->part, G, n, w->host + sum_at, w->norm, GL, w->host, w->bad,
                                                         last ? bad_host : nullptr);
        totals.push_back({g, f0, nf, sum_at});
        sum_at += (size_t)nf * g.sc * 3;
        if (!c.out) continue;
        if (!n_stage) {
          launch_out(ps, w->bad, call, g.sc, x, g.gs, (int64_t)S * m.field_len, c.out + (int64_t)f0 * S * m.field_len, nf, s);
          continue;
        }
        // to the host through the staging: columns in the caller's order, so
        // that neighbouring scales leave in one copy
        int cols[kMaxGroup];
        std::copy(g.gs.column, g.gs.column + g.n, cols);
        std::sort(cols, cols + g.n);
        for (int q = 0; q < g.n; q += plan.staged) {
          const int qn = std::min(plan.staged, g.n - q);
          GroupScales some = g.gs;
          for (int i = 0; i < g.n; ++i) {
            const int at = (int)(std::lower_bound(cols, cols + g.n, g.gs.column[i]) - cols) - q;
            some.column[i] = at >= 0 && at < qn ? at : -1;
          }
          launch_out(ps, w->bad, call, g.sc, x, some, (int64_t)qn * m.field_len, w->stage, nf, s);
          for (int f = 0; f < nf; ++f)
            for (int i = q, e; i < q + qn; i = e) {
              for (e = i + 1; e < q + qn && cols[e] == cols[e - 1] + 1;) ++e;
              IFL_HIP(hipMemcpyAsync(c.out + ((int64_t)(f0 + f) * S + cols[i]) * m.field_len,
                                     w->stage + ((int64_t)f * qn + i - q) * m.field_len,
                                     sizeof(double) * (size_t)(e - i) * m.field_len, hipMemcpyDeviceToHost, s));
            }
        }
      }
      IFL_HIP(hipGetLastError());
    }
  }
  IFL_HIP(hipStreamSynchronize(s));
  if (*bad_host == call) return fail(IFL_EINVAL, "field has a NaN or Inf at a wet entry");
  const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  for (const Totals& t : totals)
    for (int f = 0; f < t.nf; ++f)
      for (int i = 0; i < t.g.n; ++i) {
        const double bb = w->host[t.f0 + f];
        const double* q = w->host + t.at + ((size_t)f * t.g.sc + i) * 3;
        const int64_t col = (int64_t)(t.f0 + f) * S + t.g.gs.column[i];
        const double res = std::sqrt(q[0]);
        if (!poly_accepts(q[0], q[1], bb, c.rtol)) failed->push_back(col);
        if (c.stats) {
          ifl_solve_stats& so = c.stats[col];
          so.iterations = bb > 0.0 ? deg[t.g.gs.column[i]] : 0;
          so.refinements = 0;
          so.status = IFL_OK;
          so.reserved = 0;
          so.rel_residual = bb > 0.0 ? res / std::sqrt(bb) : res;
          so.seconds = secs;
          so.energy = 0.5 * q[2] / ps->mass_sum;
        }
        if (c.energy) c.energy[col] = 0.5 * q[2] / ps->mass_sum;
      }
  std::sort(failed->begin(), failed->end());
  return IFL_OK;
}

ifl_status poly_filter(PolyState* ps, PolyWork* w, const PolyCall& c, std::vector<int64_t>* failed) {
  try {
    return run_call(ps, w, c, failed);
  } catch (const std::bad_alloc&) {
    (void)hipStreamSynchronize(c.stream);  // of what was launched before
    return fail(IFL_ENOMEM, "out of host memory for a call's scales");
  }
}

ifl_status poly_fields(PolyState* ps, const PolyWork* w, int f0, int n, double* out, hipStream_t stream) {
  GroupScales one{};
  launch_out(ps, w->bad, w->call, 1, w->phi + (int64_t)f0 * ps->m.np, one, ps->m.field_len, out, n, stream);
  IFL_HIP(hipGetLastError());
  return IFL_OK;
}

}  // namespace ifl
