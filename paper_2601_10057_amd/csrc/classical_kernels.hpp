// The classical MSAV scheme's Cahn-Hilliard solves (App. B remarks; the
// comparison system of Sec. 4), FP64: zeta x = b with the variable-coefficient
// zeta = alpha - lambda div(M_psi(phi*) grad) for the two right-hand sides of
// a step, g (explicit part) and L~ = div(M grad P~), by the conjugate gradient
// iteration preconditioned with alpha - lambda M_bar Delta_h (M_bar the mean of
// M_psi(phi*) over the cells), whose inverse is App. C's DCT solve.
//
// Both systems iterate in lock step in one set of launches; every scalar of
// the iteration lives in device memory, so the host enqueues a fixed number
// of iterations and the kernels of an iteration return at once when both
// systems have converged. A kernel reads that from a flag that no workgroup of
// its own launch writes, so that all waves of a workgroup take the same
// branch: k_cl_inv_rows, which makes the stopping test and sets done_all, goes
// by a copy of it from the start of the iteration. An iteration is four
// kernels:
//   k_cl_matvec       beta; p = z + beta p, q = zeta p; partial (p, q)
//   k_cl_update_rows  a; x += a p, r -= a q; partial |r|^2; the row DCT-II of
//                     both residuals as one complex line
//   k_col_solve       the preconditioner's column solve (step_kernels.hpp)
//   k_cl_inv_rows     the stopping test; the row DCT-III -> z; partial (r, z)
// On the grids where the scheme is used in comparisons the iteration is
// bound by launches and latency, not bytes: with the products, sums and
// scalars in kernels of their own it was ten launches of 2 to 16 us each
// (1024 x 512: 93 us an iteration, now 45; 1.75 -> 1.2 ms a step; 4096^2:
// 27.2 -> 25.1 ms). A kernel's partial sums
// are added by every workgroup of the kernel that needs them, in a fixed
// order (so runs repeat bit for bit), which costs each about 2 us; finished
// in the kernel itself by the workgroup that arrives last they cost 5 to 12
// (the wait for its stores, then the counter). Workgroup 0 keeps the scalars
// for the kernels after.
//
// Fields are row-major FP64 N x N; system s in {0: g, 1: L~} at field s * N^2.
#pragma once
#include "step_kernels.hpp"

namespace ccm {

constexpr int CL_THREADS = 256;
constexpr int CL_BLOCKS = 1024;     // grid of the pointwise kernels (grid-stride)
constexpr int CL_MAX_BLOCKS = 8192; // rows of partial sums (one per grid row at most)
constexpr int CL_PART_SUMS = 11;    // doubles per row of all partials (ClPart)

// Scalars of the two iterations.
struct PcgScalars {
  double alpha, lam, tol;          // zeta = alpha - lam div(M grad); stop at |r| <= tol |b|
  double bnorm2[2], bsum[2];       // |b|^2 and sum b per system
  double rz[2][2];                 // (r, z) of even and odd iterations' start
  double rnorm2[2];
  double shift[2];                 // mean correction added to x after the iteration
  double pl[2];                    // (P~, x_s) with the mean correction
  int iters[2];
  int done[2];
  int done_all;                    // set by k_cl_inv_rows, read by the other kernels
                                   //   (k_col_solve: MemberArgs::skip)
  int done_before;                 // done_all as the iteration began, for k_cl_inv_rows
};

// Partial sums of the iteration's kernels, one row per workgroup.
struct ClPart {
  double* rz;      // 2 per row: k_cl_inv_rows
  double* pq;      // 2: k_cl_matvec
  double* rr;      // 2: k_cl_update_rows
  double* sums;    // up to 5: |b|^2 and sum b; k_cl_gram
};

// The workgroup's sums of v to its row of part.
template <int NV, int NTHR>
__device__ __forceinline__ void cl_partial(double (&v)[NV], double* red, double* __restrict__ part) {
  block_sum<NV, NTHR>(v, red, threadIdx.x);
  if (threadIdx.x < NV) part[(size_t)blockIdx.x * NV + threadIdx.x] = red[threadIdx.x];
}

// Sums of `rows` rows of partials, for every thread of the workgroup.
template <int NV, int NTHR>
__device__ __forceinline__ void cl_gather(const double* __restrict__ part, int rows, double* red,
                                          double (&t)[NV]) {
#pragma unroll
  for (int q = 0; q < NV; ++q) t[q] = 0.0;
  for (int r = threadIdx.x; r < rows; r += NTHR) {
#pragma unroll
    for (int q = 0; q < NV; ++q) t[q] += part[(size_t)r * NV + q];
  }
  block_sum<NV, NTHR>(t, red, threadIdx.x);
#pragma unroll
  for (int q = 0; q < NV; ++q) t[q] = red[q];
  lds_sync();
}

// The stopping test of system s after an iteration that left |r|^2 = rr.
__device__ __forceinline__ void cl_test(PcgScalars* __restrict__ sc, const double (&rr)[2]) {
  for (int s = 0; s < 2; ++s) {
    if (sc->done[s]) continue;
    sc->rnorm2[s] = rr[s];
    sc->iters[s] += 1;
    if (rr[s] <= sc->tol * sc->tol * sc->bnorm2[s]) sc->done[s] = 1;
  }
  sc->done_all = sc->done[0] && sc->done[1];
}

// Iteration `it`: the next direction p_new = z + beta p_old (p_new = z at the
// first) and q = zeta p_new, with (p_new, q). zeta applies the five-point
// flux form with the face mobilities me (east face of each cell) and mn (north
// face); the wall faces carry no flux (Neumann, their mobilities are zero). A
// wave takes 64 columns by CL_ROWS rows: a lane keeps the rows above and below
// in registers, its neighbours along x are the adjacent lanes (the wave's end
// lanes load theirs), so that a direction value is formed once per cell and
// halo row instead of at each of five points (1024 x 512: 16 us, now 14 with
// the sums of beta in it).
constexpr int CL_ROWS = 4;
__global__ void __launch_bounds__(CL_THREADS)
k_cl_matvec(const double* __restrict__ z, const double* __restrict__ p_old,
            double* __restrict__ p_new, double* __restrict__ q, const double* __restrict__ me,
            const double* __restrict__ mn, int nx, int ny, double inv_h2,
            ClPart part, PcgScalars* __restrict__ sc, int it) {
  __shared__ double red[2 * (CL_THREADS / 64 + 1)];
  const int done = sc->done_all;
  if (blockIdx.x == 0 && threadIdx.x == 0) sc->done_before = done;
  if (done) return;
  const size_t n = (size_t)nx * ny;
  double rz[2], be[2] = {0.0, 0.0};
  cl_gather<2, CL_THREADS>(part.rz, ny, red, rz);
  const bool first = it == 0;
  for (int s = 0; s < 2; ++s) {
    if (!first && !sc->done[s]) be[s] = rz[s] / sc->rz[s][(it + 1) & 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->rz[s][it & 1] = rz[s];
  }
  const double alpha = sc->alpha, lam = sc->lam;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nseg = (nx + 63) / 64, units = nseg * (ny / CL_ROWS);
  double v[2] = {0.0, 0.0};
  for (int u = blockIdx.x * (CL_THREADS / 64) + wave; u < units;
       u += gridDim.x * (CL_THREADS / 64)) {
    const int i = u % nseg * 64 + lane, j0 = u / nseg * CL_ROWS;
    const bool in = i < nx;
    const bool edge_w = lane == 0 && i > 0, edge_e = lane == 63 && i + 1 < nx;
    // direction of system s at row j, column i + d (zero outside the grid,
    // where the mobility is zero too)
    auto dir = [&](int s, int j, int d) {
      const size_t k = s * n + (size_t)j * nx + i + d;
      return first ? z[k] : z[k] + be[s] * p_old[k];
    };
    double ps[2], pc[2], pn[2];
    double ms = 0.0;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      ps[s] = in && j0 > 0 ? dir(s, j0 - 1, 0) : 0.0;
      pc[s] = in ? dir(s, j0, 0) : 0.0;
    }
    if (in && j0 > 0) ms = mn[(size_t)(j0 - 1) * nx + i];
#pragma unroll
    for (int r = 0; r < CL_ROWS; ++r) {
      const int j = j0 + r;
      const size_t o = (size_t)j * nx + i;
      const double Me = in ? me[o] : 0.0, Mn = in ? mn[o] : 0.0;
      double Mw = lane_from_below(Me);
      if (lane == 0) Mw = edge_w ? me[o - 1] : 0.0;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        pn[s] = in && j + 1 < ny ? dir(s, j + 1, 0) : 0.0;
        double pw = lane_from_below(pc[s]), pe = lane_from_above(pc[s]);
        if (edge_w) pw = dir(s, j, -1);
        if (edge_e) pe = dir(s, j, 1);
        const double flux = Me * (pe - pc[s]) - Mw * (pc[s] - pw) + Mn * (pn[s] - pc[s]) -
                            ms * (pc[s] - ps[s]);
        const double qv = alpha * pc[s] - lam * flux * inv_h2;
        if (in) {
          p_new[s * n + o] = pc[s];
          q[s * n + o] = qv;
          v[s] += pc[s] * qv;
        }
        ps[s] = pc[s];
        pc[s] = pn[s];
      }
      ms = Mn;
    }
  }
  cl_partial<2, CL_THREADS>(v, red, part.pq);
}

// One row of both systems: x += a p, r -= a q for the systems still iterating
// with |r|^2, or (INIT) x = 0, r = b with |b|^2 and sum b; then the DCT-II of
// the residuals' row, r_0 + i r_1 as one complex line, into slots M_F and M_G
// of the strip-major intermediates.
template <int NX, bool INIT>
__global__ void __launch_bounds__(line_threads(NX))
k_cl_update_rows(const double* __restrict__ b, double* __restrict__ x, double* __restrict__ r,
                 const double* __restrict__ p, const double* __restrict__ q,
                 double* __restrict__ mid, int ny, ClPart part, int pq_rows,
                 const PcgScalars* __restrict__ sc, int it) {
  constexpr int NTHR = line_threads(NX), NV = INIT ? 4 : 2;
  constexpr int CPT = NX >= NTHR ? NX / NTHR : 1;
  constexpr int R = fft_radix<double>();
  using MAP = LdsMap<double, NX, SWZ_LINE>;
  using LS = LineSlots<NX, NTHR, R, MAP>;
  __shared__ cpx<double> buf[NX];
  const LdsLine<double> line(buf);
  __shared__ cpx<double> rtab[Roots<double, NX>::SIZE];
  __shared__ double red[NV * (NTHR / 64 + 1)];
  if (!INIT && sc->done_all) return;
  const int tid = threadIdx.x;
  const int j = xcd_remap(blockIdx.x, gridDim.x);
  const size_t n = (size_t)NX * ny;
  double a[2] = {0.0, 0.0};
  if constexpr (!INIT) {
    double pq[2];
    cl_gather<2, NTHR>(part.pq, pq_rows, red, pq);
#pragma unroll
    for (int s = 0; s < 2; ++s) a[s] = sc->done[s] ? 0.0 : sc->rz[s][it & 1] / pq[s];
  }
  Roots<double, NX> rt;
  rt.init(rtab, tid, NTHR);
  const LS sl(tid);
  double v[NV];
#pragma unroll
  for (int s = 0; s < NV; ++s) v[s] = 0.0;
  static_for<CPT>([&](auto iq) {
    constexpr int c = decltype(iq)::value;
    const int i = tid + c * NTHR;
    if (NX >= NTHR || i < NX) {
      double rv[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const size_t k = s * n + (size_t)j * NX + i;
        if constexpr (INIT) {
          rv[s] = b[k];
          x[k] = 0.0;
          v[2 + s] += rv[s];
        } else {
          x[k] += a[s] * p[k];
          rv[s] = r[k] - a[s] * q[k];
        }
        r[k] = rv[s];
        v[s] += rv[s] * rv[s];
      }
      line[sl.template mak<c>()] = {rv[0], rv[1]};
    }
  });
  lds_sync();
  fft_lines<double, NX, 1, NTHR, R, MAP>(line, rt, tid);
  const size_t SS = strip_stride(ny, 8), FSM = strip_field(NX, ny, 8);
  row_dct_pairs<double, NX, NTHR, MAP>(line, rt, tid,
                                       [&](int sp, double a0, double a1, double b0, double b1) {
    typedef double d2 __attribute__((ext_vector_type(2)));
    double* o = mid + (size_t)sp * SS + 2 * (size_t)j;
    *reinterpret_cast<d2*>(o + M_F * FSM) = d2{a0, a1};
    *reinterpret_cast<d2*>(o + M_G * FSM) = d2{b0, b1};
  });
  cl_partial<NV, NTHR>(v, red, INIT ? part.sums : part.rr);
}

// One row of the preconditioned residuals: DCT-III along x of the two solved
// fields as one complex line -> z, and (r, z). Workgroup 0 makes the stopping
// test of the update before (INIT: keeps |b|^2 and sum b instead); the others
// do not wait for it, and z of an iteration that has just converged is not
// used.
template <int NX, bool INIT>
__global__ void __launch_bounds__(line_threads(NX))
k_cl_inv_rows(const double* __restrict__ out, const double* __restrict__ r,
              double* __restrict__ z, int ny, ClPart part, PcgScalars* __restrict__ sc) {
  constexpr int NTHR = line_threads(NX);
  constexpr int CPT = NX >= NTHR ? NX / NTHR : 1;            // outputs per thread
  constexpr int UPT = NX / 2 >= NTHR ? NX / 2 / NTHR : 1;    // strips (and units) per thread
  constexpr int R = fft_radix<double>();
  using MAP = LdsMap<double, NX, SWZ_LINE>;
  using LS = LineSlots<NX, NTHR, R, MAP>;
  __shared__ cpx<double> buf[NX];
  const LdsLine<double> line(buf);
  __shared__ cpx<double> rtab[Roots<double, NX>::SIZE];
  __shared__ double red[(INIT ? 4 : 2) * (NTHR / 64 + 1)];
  if (!INIT && sc->done_before) return;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {                       // whole workgroup
    if constexpr (INIT) {
      double t[4];
      cl_gather<4, NTHR>(part.sums, ny, red, t);
      if (tid == 0) {
        for (int s = 0; s < 2; ++s) {
          sc->bnorm2[s] = t[s];
          sc->bsum[s] = t[2 + s];
          // a zero right-hand side is solved by x = 0
          sc->done[s] = t[s] > 0.0 ? 0 : 1;
        }
        sc->done_all = sc->done[0] && sc->done[1];
      }
    } else {
      double rr[2];
      cl_gather<2, NTHR>(part.rr, ny, red, rr);
      if (tid == 0) cl_test(sc, rr);
    }
  }
  const int j = xcd_remap(blockIdx.x, gridDim.x);
  const size_t n = (size_t)NX * ny, SS = strip_stride(ny, 8), FSM = strip_field(NX, ny, 8);
  Roots<double, NX> rt;
  rt.init(rtab, tid, NTHR);
  const LS sl(tid);
#pragma unroll
  for (int c = 0; c < UPT; ++c) {
    const int st = tid + c * NTHR;
    if (NX / 2 >= NTHR || st < NX / 2) {
      typedef double d2 __attribute__((ext_vector_type(2)));
      const double* o = out + (size_t)st * SS + 2 * (size_t)j;
      const d2 a = *reinterpret_cast<const d2*>(o), b = *reinterpret_cast<const d2*>(o + FSM);
      line[MAP::at(2 * st)] = {a[0], b[0]};
      line[MAP::at(2 * st + 1)] = {a[1], b[1]};
    }
  }
  lds_sync();
  static_for<UPT>([&](auto iq) {
    constexpr int c = decltype(iq)::value;
    const int u = tid + c * NTHR;
    if (NX / 2 >= NTHR || u < NX / 2) {
      const int pn = sl.template nat<c>(), pm = sl.template natm<c>();
      const cpx<double> xv = line[pn], xm = line[pm];
      cpx<double> Z, Zm;
      dct3_pair<double, NX>(rt, u, xv.re, xm.re, xv.im, xm.im, Z, Zm);
      line[pn] = Z;
      line[pm] = Zm;
    }
  });
  lds_sync();
  fft_lines<double, NX, 1, NTHR, R, MAP>(line, rt, tid);
  double v[2] = {0.0, 0.0};
  static_for<CPT>([&](auto iq) {
    constexpr int c = decltype(iq)::value;
    const int i = tid + c * NTHR;
    if (NX >= NTHR || i < NX) {
      const cpx<double> y = line[sl.template out<c>()];
      const size_t o = (size_t)j * NX + i;
      z[o] = y.re;
      z[n + o] = -y.im;
      v[0] += r[o] * y.re;
      v[1] += r[n + o] * -y.im;
    }
  });
  cl_partial<2, NTHR>(v, red, part.rz);
}

// The stopping test of the last allowed iteration (an error bit if it ends
// unconverged).
__global__ void __launch_bounds__(CL_THREADS)
k_cl_last(ClPart part, int rows, PcgScalars* __restrict__ sc, DevScalars* __restrict__ ds) {
  __shared__ double red[2 * (CL_THREADS / 64 + 1)];
  if (sc->done_all) return;
  double rr[2];
  cl_gather<2, CL_THREADS>(part.rr, rows, red, rr);
  if (threadIdx.x != 0) return;
  cl_test(sc, rr);
  if (!sc->done_all) ds->err |= ERR_PCG;
}

// Partial (P~, x_s), sum x_s and sum P~ for the mean correction.
constexpr int CL_GRAM_SUMS = 5;
__global__ void __launch_bounds__(CL_THREADS)
k_cl_gram(const double* __restrict__ P, const double* __restrict__ x, ClPart part, size_t n) {
  __shared__ double red[CL_GRAM_SUMS * (CL_THREADS / 64 + 1)];
  double v[CL_GRAM_SUMS] = {};
  for (size_t o = (size_t)blockIdx.x * CL_THREADS + threadIdx.x; o < n;
       o += (size_t)gridDim.x * CL_THREADS) {
    const double pv = P[o], xg = x[o], xl = x[n + o];
    v[0] += pv * xg;
    v[1] += pv * xl;
    v[2] += xg;
    v[3] += xl;
    v[4] += pv;
  }
  cl_partial<CL_GRAM_SUMS, CL_THREADS>(v, red, part.sums);
}

// The mean correction and (P~, x_s) for the 5x5 system, one workgroup. x_s +
// shift_s has the exact mean sum(b_s) / (alpha N^2): summing zeta x = b over
// the cells gives alpha sum x = sum b (the fluxes cancel).
__global__ void __launch_bounds__(CL_THREADS)
k_cl_final(ClPart part, int rows, PcgScalars* __restrict__ sc, DevScalars* __restrict__ ds,
           double cells) {
  __shared__ double red[CL_GRAM_SUMS * (CL_THREADS / 64 + 1)];
  double t[CL_GRAM_SUMS];
  cl_gather<CL_GRAM_SUMS, CL_THREADS>(part.sums, rows, red, t);
  if (threadIdx.x != 0) return;
  for (int s = 0; s < 2; ++s) {
    sc->shift[s] = (sc->bsum[s] / sc->alpha - t[2 + s]) / cells;
    sc->pl[s] = t[s] + sc->shift[s] * t[4];
    ds->cl[s] = sc->pl[s];
  }
}

// psi^{n+1} = (x_g + shift_g) + c (x_L + shift_L), c = the combination
// coefficient of L~ from the 5x5 solve (App. B Step 4 recovery).
__global__ void __launch_bounds__(CL_THREADS)
k_cl_combine(const double* __restrict__ x, const PcgScalars* __restrict__ sc,
             const double* __restrict__ coef, double* __restrict__ psi_new, size_t n) {
  const double c = coef[6];
  const double sg = sc->shift[0], sl = sc->shift[1];
  for (size_t o = (size_t)blockIdx.x * CL_THREADS + threadIdx.x; o < n;
       o += (size_t)gridDim.x * CL_THREADS)
    psi_new[o] = (x[o] + sg) + c * (x[n + o] + sl);
}

// The preconditioner's constants for this step, alpha - lambda M_bar Delta_h
// (M_bar = h^2 sum M_psi(phi*) / |Omega| from the stencil partials), into the
// solve table entry (chi group: C1 = alpha, C2 = lambda M_bar, C3 = 0; zeta
// group: alpha, lambda M_bar) and the iteration's scalars.
__global__ void __launch_bounds__(512)
k_cl_setup(const double* __restrict__ p1, int rows, MemberArgs* __restrict__ pre,
           PcgScalars* __restrict__ sc, double alpha, double lam, double tol, double cells) {
  constexpr int NV = (int)P1_NSUM;
  __shared__ double red[512 + NV];
  double t[NV];
  reduce_columns<NV, 512>(p1, rows, red, threadIdx.x, t);
  if (threadIdx.x != 0) return;
  const double m_bar = t[P1_MBAR] / cells;
  pre->k.C1 = alpha;
  pre->k.C2 = lam * m_bar;
  pre->k.C3 = 0.0;
  pre->k.alpha = alpha;
  pre->k.lam = lam * m_bar;
  sc->alpha = alpha;
  sc->lam = lam;
  sc->tol = tol;
  sc->iters[0] = sc->iters[1] = 0;
  sc->done[0] = sc->done[1] = sc->done_all = 0;
}

}  // namespace ccm
