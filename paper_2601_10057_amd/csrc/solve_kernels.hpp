// The fast direct solver of App. C on its own: chi^{-1} and zeta^{-1} of one
// real field, with the DCT (homogeneous Neumann boundaries) or the DST
// (homogeneous Dirichlet ones).
//   k_solve_rows  DCT-II along x, in FP64 of two rows as one complex line
//   k_solve_cols  per strip of two columns: DCT-II along y once, then for
//                 each operator the divide and the DCT-III along y
//   k_solve_inv   DCT-III along x of both results (the step's row inverse)
// The arguments are passed by value: no table upload and no wait for one.
//
// A DST-II is a DCT-II of the sign-alternated input read in reverse order:
// sum_i x_i sin(pi (N - k)(2 i + 1) / (2 N)) = sum_i (-1)^i x_i cos(pi k (2 i +
// 1) / (2 N)), so the Dirichlet solve reads and writes the rows times
// (-1)^(i + j) and re-indexes the eigenvalues.
#pragma once
#include "step_kernels.hpp"

namespace ccm {

// Eigenvalue tables that k_solve_rows forms on the device: none (they are
// there), Neumann (4/h^2) sin^2(pi k / (2 n)), or Dirichlet: (4/h^2) sin^2(pi
// (k + 1) / (2 n)) for DST index k, at DCT index N - 1 - k: (4/h^2) cos^2(pi k'
// / (2 n)).
enum SolveTables { TABLES_GIVEN = 0, TABLES_NEUMANN = 1, TABLES_DIRICHLET = 2 };

struct SolveArgs {
  gptr<const double> rhs;        // row-major
  gptr<void> mid;                // the x-transformed field, strip-major
  gptr<void> outc;               // the two y-solved fields, strip-major
  gptr<double> lamx;             // eigenvalue tables
  gptr<double> lamy;
  gptr<double> out_chi;          // row-major
  gptr<double> out_zeta;
  int nx, ny;
  int tables;                    // SolveTables
  int alt;                       // 1: rows read and written times (-1)^(i + j)
  double h;
  OpConst k;
};

// FP64: two real rows to a complex line (one row per line, half of each
// transform idle: 27 us at N = 2048, 24 us so; a solve at N = 4096 495 us, 457
// so), and a column pair's rows leave as one piece. The rounding errors of a
// line are relative to its larger row, which costs a solve up to 5% more error
// in the root mean square. FP32: one row to a line. With two, solves were off
// by up to 1.5 times as much (16 x 4096, Dirichlet; 0.3 to 4% elsewhere); one
// takes 80 us at N = 2048 in place of 73, and 357 at N = 4096 in place of 328.
template <typename TM> constexpr int solve_line_rows() { return sizeof(TM) == 8 ? 2 : 1; }
template <typename TM, int NX>
__global__ void __launch_bounds__(line_threads(NX)) k_solve_rows(SolveArgs a) {
  constexpr int ROWS = solve_line_rows<TM>();
  constexpr int NTHR = line_threads(NX);
  constexpr int CPT = NX >= NTHR ? NX / NTHR : 1;
  constexpr int R = fft_radix<TM>();
  using MAP = LdsMap<TM, NX, SWZ_LINE>;
  using LS = LineSlots<NX, NTHR, R, MAP>;
  __shared__ LinesLds<TM, NX, NX> L;
  const LdsLine<TM> line(L.line);
  const int tid = threadIdx.x;
  const int j = ROWS * xcd_remap(blockIdx.x, gridDim.x);
  if (a.tables != TABLES_GIVEN) {
    for (int e = blockIdx.x * NTHR + tid; e < NX + a.ny; e += gridDim.x * NTHR) {
      const bool x = e < NX;
      const int k = x ? e : e - NX, n = x ? NX : a.ny;
      const double t = (double)k / (2.0 * n);
      const double s = a.tables == TABLES_DIRICHLET ? cospi(t) : sinpi(t);
      (x ? a.lamx : a.lamy)[k] = 4.0 / (a.h * a.h) * s * s;
    }
  }
  Roots<TM, NX> rt;
  rt.init(L.rtab, tid, NTHR);
  const LS sl(tid);
  const auto src = a.rhs + (size_t)j * NX;
  static_for<CPT>([&](auto iq) {
    constexpr int q = decltype(iq)::value;
    const int i = tid + q * NTHR;
    if (NX >= NTHR || i < NX) {
      const double u = src[i], w = ROWS == 2 ? src[NX + i] : 0.0;
      const bool neg0 = a.alt & (i + j) & 1, neg1 = a.alt & (i + j + 1) & 1;
      line[sl.template mak<q>()] = {(TM)(neg0 ? -u : u), (TM)(neg1 ? -w : w)};
    }
  });
  lds_sync();
  fft_lines<TM, NX, 1, NTHR, R, MAP>(line, rt, tid);
  const size_t SS = strip_stride(a.ny, sizeof(TM));
  const auto mid = static_cast<gptr<TM>>(a.mid);
  row_dct_pairs<TM, NX, NTHR, MAP>(line, rt, tid, [&](int sp, TM a0, TM a1, TM b0, TM b1) {
    RowPiece<TM, ROWS> pc;
    pc.v[0] = a0;
    pc.v[1] = a1;
    if constexpr (ROWS == 2) {
      pc.v[2] = b0;
      pc.v[3] = b1;
    }
    store_piece<TM, ROWS>(mid + (size_t)sp * SS + 2 * (size_t)j, pc);
  });
}

// One strip: the forward transform is done once for both operators (by a
// workgroup per operator it is done and its input read twice: 66 us at N =
// 2048 in FP64, 52 us so). While the strips' threads do not fill the device
// the operators go to workgroups of their own (gridDim.y = 2), which halves
// the chain of transforms: a solve at 256 x 2048 takes 28.6 us against 32.4,
// at 512^2 19.5 against 21.0; at 1024^2 47.4 against 46.4, at 512 x 4096 64.8
// against 57.9.
inline bool solve_split(int nx, int ny) { return nx / 2 * line_threads(ny) <= 65536; }
template <typename TM, int NY>
__global__ void __launch_bounds__(line_threads(NY)) k_solve_cols(SolveArgs a) {
  constexpr int NTHR = line_threads(NY);
  constexpr int LPT = NY >= NTHR ? NY / NTHR : 1;            // elements per thread
  constexpr int UPT = NY / 2 >= NTHR ? NY / 2 / NTHR : 1;    // pair units per thread
  constexpr int R = fft_radix<TM>();
  using MAP = LdsMap<TM, NY, SWZ_LINE>;
  using LS = LineSlots<NY, NTHR, R, MAP>;
  __shared__ LinesLds<TM, NY, NY> L;
  const int tid = threadIdx.x;
  const int s = xcd_remap(blockIdx.x, gridDim.x);
  const size_t SS = strip_stride(NY, sizeof(TM)), FSM = strip_field(a.nx, NY, sizeof(TM));
  const LdsLine<TM> line(L.line);
  Roots<TM, NY> rt;
  rt.init(L.rtab, tid, NTHR);
  const LS sl(tid);
  const auto src = reinterpret_cast<gptr<const cpx<TM>>>(static_cast<gptr<const TM>>(
                       static_cast<gptr<const void>>(a.mid)) + (size_t)s * SS);
  static_for<LPT>([&](auto iq) {
    constexpr int q = decltype(iq)::value;
    const int i = tid + q * NTHR;
    if (NY >= NTHR || i < NY) line[sl.template mak<q>()] = gload<TM>(src + i);
  });
  lds_sync();
  fft_lines<TM, NY, 1, NTHR, R, MAP>(line, rt, tid);
  TM A[UPT], B[UPT], Am[UPT], Bm[UPT];
  static_for<UPT>([&](auto iq) {
    constexpr int q = decltype(iq)::value;
    const int u = tid + q * NTHR;
    if (NY / 2 >= NTHR || u < NY / 2)
      dct2_unit<TM, NY>(line, sl.template bin<q>(), sl.template binm<q>(), rt, u, A[q], B[q],
                        Am[q], Bm[q]);
  });
  const double lx0 = a.lamx[2 * s], lx1 = a.lamx[2 * s + 1];
#pragma unroll 1
  for (int op = blockIdx.y; op < 2; op += gridDim.y) {
    auto inv = [&](double ev) {
      return rcp64(op == 0 ? a.k.C1 + ev * (a.k.C2 + a.k.C3 * ev) : a.k.alpha + a.k.lam * ev);
    };
    // (slots formed anew: held across the loop they would spill on long lines)
    const int t = opaque_vgpr(tid);
    const LS sn(t);
    lds_sync();                  // the line's last reads
    static_for<UPT>([&](auto iq) {
      constexpr int q = decltype(iq)::value;
      const int u = t + q * NTHR;
      if (NY / 2 >= NTHR || u < NY / 2) {
        const double ly = a.lamy[u], lym = a.lamy[pair_mirror<NY>(u)];
        cpx<TM> Z, Zm;
        dct3_pair<TM, NY>(rt, u, (TM)((double)A[q] * inv(lx0 + ly)),
                          (TM)((double)Am[q] * inv(lx0 + lym)),
                          (TM)((double)B[q] * inv(lx1 + ly)),
                          (TM)((double)Bm[q] * inv(lx1 + lym)), Z, Zm);
        line[sn.template nat<q>()] = Z;
        line[sn.template natm<q>()] = Zm;
      }
    });
    lds_sync();
    fft_lines<TM, NY, 1, NTHR, R, MAP>(line, rt, t);
    const auto dst = reinterpret_cast<gptr<cpx<TM>>>(static_cast<gptr<TM>>(a.outc) + op * FSM +
                                                     (size_t)s * SS);
    static_for<LPT>([&](auto iq) {
      constexpr int q = decltype(iq)::value;
      const int i = t + q * NTHR;
      if (NY >= NTHR || i < NY) {
        const cpx<TM> y = line[sn.template out<q>()];
        gstore<TM>(dst + i, {y.re, -y.im});
      }
    });
  }
}

// Row inverse variants as in k_row_idct.
template <typename TM, int NX, int V>
__global__ void __launch_bounds__(row_idct_threads<TM>(NX, V),
                                  V == 0 && row_idct_threads<TM>(NX, V) == 512 ? 4 : 1)
k_solve_inv(SolveArgs a) {
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const auto out = static_cast<gptr<const TM>>(static_cast<gptr<const void>>(a.outc));
  if constexpr (V == 0) {
    __shared__ RowIdctBandLds<TM, NX> L;
    row_idct_band_body<TM, NX>(out, a.out_chi, a.out_zeta, a.ny, nullptr, nullptr, nullptr, blk, L,
                               threadIdx.x, a.alt);
  } else {
    __shared__ LinesLds<TM, NX, NX> L;
    row_idct_body<TM, NX, line_threads_v<TM>(NX, V)>(out, a.out_chi, a.out_zeta, a.ny, nullptr,
                                                     nullptr, nullptr, blk, L, threadIdx.x, a.alt);
  }
}

}  // namespace ccm
