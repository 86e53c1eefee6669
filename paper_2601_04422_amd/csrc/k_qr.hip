// QR preconditioning of the Jacobi SVD (Drmac and Veselic, "New fast and
// accurate Jacobi SVD algorithm", SIAM J. Matrix Anal. Appl. 29(4), 2008).
//
// The paper decomposes the merged two-site tensor with a Jacobi SVD on the GPU
// (Sec. IV.A, cusolverDnZgesvdj).  One-sided Jacobi applied to M directly
// needs many sweeps on these graded matrices; applied to R2^H from
//
//   M = Q1 R1      (m x n, m >= n, Householder)
//   R1^H = Q2 R2   (n x n, Householder; Q2 is not needed)
//
// it needs about half as many.  With R2^H = W S V^H (W from the Jacobi),
// M = (Q1 W) S (Q2 V)^H, so the left singular vectors are U = Q1 [W; 0] and
// no rotation has to be accumulated.
//
// Householder QR in the LAPACK convention: H = I - tau v v^H with v(0) = 1,
// H^H [alpha; x] = [beta; 0], beta real; a panel of QNB reflectors is
// I - V T V^H (compact WY, T upper triangular).  Everything is float64.
#include <algorithm>

#include "tnsim_internal.h"
#include "tn_complex.h"
#include "tn_buffer.h"
#include "tn_lanes.h"
#include "tn_fast.h"

namespace tn {

struct QrView {
  double2 *A;
  int ld, rows, cols;
};

// stage 0: M in Qm (m x n); stage 1: R1^H in X (n x n)
__device__ __forceinline__ QrView qr_view(const GateDesc &d, int stage) {
  if (stage == 0) return QrView{d.Qm, d.ldq, d.m, d.n};
  return QrView{d.X, d.ldx, d.n, d.n};
}

// T factors: those of the QNB-column panels of both stages, then those of
// the QG-column groups (QG / QNB panels each) of both stages.
__device__ __forceinline__ double2 *qr_tfac(const GateDesc &d, int stage, int panel) {
  const int np = d.colsPad / QNB;  // panels per stage
  return d.Tq + ((size_t)stage * np + panel) * (QNB * QNB);
}
__device__ __forceinline__ double2 *qr_tgrp(const GateDesc &d, int stage, int group) {
  const int np = d.colsPad / QNB, ngp = d.colsPad / QG;
  return d.Tq + (size_t)2 * np * (QNB * QNB) + ((size_t)stage * ngp + group) * (QG * QG);
}

// ---------------------------------------------------------------- panel

// Factor columns j0 .. j0+w-1 (rows j0 ..) of one gate's matrix: one
// workgroup per gate, the panel in registers (thread t holds panel rows
// t, t + THREADS, ...).  Writes R's panel rows, the reflectors below the
// diagonal and the panel's T factor.
//
// Gates with complex64 sites.  The order of every sum is fixed: over a
// thread's rows 512 apart, the halving tree of a wavefront, then the
// wavefronts in turn (rows that do not exist add zeros, so fewer threads or
// rows per thread change nothing).  The sites these gates write are rounded to
// float32, so another order would show in every later readout at 1e-8.  Two
// sums a column, the norm below the diagonal and then v^H a_p and v_p^H v;
// after each one barrier, and every wavefront computes what follows by itself.
// Bound by that chain (two reductions and barriers, a square root and three
// divisions a column).  Against four barriers and a thread that computes for
// all (one kernel for every height): 49 -> 12.4 us up to 256 rows, 49 -> 17.6 up
// to 512.
template <int THREADS, int RPT>
__global__ __launch_bounds__(THREADS) void k_qr_panel(const GateDesc *descs, int stage, int panel) {
  static_assert(RPT == 1 || THREADS == 512, "a thread's rows are 512 apart");
  const GateDesc &d = descs[blockIdx.x];
  if (!d.qr || d.storage == 0) return;
  const QrView q = qr_view(d, stage);
  const int j0 = panel * QNB;
  if (j0 >= q.cols) return;
  const int w = min(QNB, q.cols - j0);
  const int nr = q.rows - j0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int WAVES = THREADS / 64;
  __shared__ double rednorm[2][WAVES];          // by column parity
  __shared__ double reddot[2][WAVES][2 * QNB];
  __shared__ double2 top[2];                    // the diagonal entry

  double2 a[RPT][QNB];
#pragma unroll
  for (int i = 0; i < RPT; i++) {
    const int lr = tid + THREADS * i;
#pragma unroll
    for (int c = 0; c < QNB; c++)
      a[i][c] = (lr < nr && c < w) ? q.A[(size_t)(j0 + c) * q.ld + j0 + lr]
                                   : make_double2(0.0, 0.0);
  }
  double2 trow[QNB];  // thread t < 8: row t of T
#pragma unroll
  for (int c = 0; c < QNB; c++) trow[c] = make_double2(0.0, 0.0);

#pragma unroll
  for (int c = 0; c < QNB; c++) {
    if (c >= w) break;
    // ||x||^2 below the diagonal of column c
    double xn = 0.0;
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const int lr = tid + THREADS * i;
      if (lr > c) xn += cabs2(a[i][c]);
    }
    xn = wave_total(xn);
    if (tid == c) top[c & 1] = a[0][c];
    if (lane == 0) rednorm[c & 1][wave] = xn;
    __syncthreads();
    double x2 = 0.0;
#pragma unroll
    for (int v = 0; v < WAVES; v++) x2 += rednorm[c & 1][v];
    const double2 al = top[c & 1];
    double2 tau = make_double2(0.0, 0.0), scale = tau;
    double beta = al.x;
    if (!(x2 == 0.0 && al.y == 0.0)) {  // else already triangular: H = I
      beta = -copysign(sqrt(cabs2(al) + x2), al.x);
      tau = make_double2((beta - al.x) / beta, -al.y / beta);
      const double2 dn = make_double2(al.x - beta, al.y);  // alpha - beta
      const double inv = 1.0 / cabs2(dn);
      scale = make_double2(dn.x * inv, -dn.y * inv);  // 1 / (alpha - beta)
    }
    as_loaded(tau);
    as_loaded(scale);
    // reflector below the diagonal, beta on it; vr = v at this thread's rows
    double2 vr[RPT];
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const int lr = tid + THREADS * i;
      if (lr > c) {
        a[i][c] = cmul(a[i][c], scale);
        vr[i] = a[i][c];
      } else if (lr == c) {
        a[i][c] = make_double2(beta, 0.0);
        vr[i] = make_double2(1.0, 0.0);
      } else {
        vr[i] = make_double2(0.0, 0.0);
      }
    }
    // one reduction for both: s_p = v^H a_p (p > c, to update the panel) and
    // g_p = v_p^H v (p < c, for the T factor)
    double part[2 * QNB];
#pragma unroll
    for (int p = 0; p < QNB; p++) {
      double2 acc = make_double2(0.0, 0.0);
      if (p != c && p < w) {
#pragma unroll
        for (int i = 0; i < RPT; i++) {
          if (p > c)
            cfmac(acc, vr[i], a[i][p]);  // conj(v) a_p
          else
            cfmac(acc, a[i][p], vr[i]);  // conj(v_p) v (rows >= c, where v_p is stored)
        }
      }
      part[2 * p] = acc.x;
      part[2 * p + 1] = acc.y;
    }
    const double mine = wave_sums<2 * QNB, true>(part);  // lane l: value l / 4
    if ((lane & 3) == 0) reddot[c & 1][wave][lane >> 2] = mine;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int v = 0; v < WAVES; v++) tot += reddot[c & 1][v][lane & 15];
    // a_p <- a_p - conj(tau) v s_p for the later panel columns;
    // T(0:c, c) = -tau T(0:c, 0:c) g(0:c), T(c, c) = tau
    const double2 ctau = cconj(tau);
    double2 tc = make_double2(0.0, 0.0);
#pragma unroll
    for (int p = 0; p < QNB; p++) {
      if (p == c || p >= w) continue;
      const double2 sp = make_double2(lane_value(tot, 2 * p), lane_value(tot, 2 * p + 1));
      if (p > c) {
        const double2 f = cmul(ctau, sp);
#pragma unroll
        for (int i = 0; i < RPT; i++) a[i][p] = csub(a[i][p], cmul(vr[i], f));
      } else {
        const double2 t = trow[p];
        tc.x += fma(t.x, sp.x, -(t.y * sp.y));
        tc.y += fma(t.y, sp.x, t.x * sp.y);
      }
    }
    trow[c] = tid < c ? make_double2(fma(tau.y, tc.y, -(tau.x * tc.x)),
                                     fma(-tau.y, tc.x, -(tau.x * tc.y)))
                      : (tid == c ? tau : make_double2(0.0, 0.0));
  }
#pragma unroll
  for (int i = 0; i < RPT; i++) {
    const int lr = tid + THREADS * i;
    if (lr < nr) {
#pragma unroll
      for (int c = 0; c < QNB; c++)
        if (c < w) q.A[(size_t)(j0 + c) * q.ld + j0 + lr] = a[i][c];
    }
  }
  double2 *T = qr_tfac(d, stage, panel);
  if (tid < QNB) {
#pragma unroll
    for (int c = 0; c < QNB; c++) T[tid * QNB + c] = trow[c];
  }
}

// The same panel with one reduction and one barrier per column (gates with
// complex128 sites; the order of the sums differs from k_qr_panel's, and
// complex64 handles keep theirs, see GateDesc::fullOrder).  The products
// conj(x) a_p of the column below its diagonal with every panel column come
// out of one transposed sum (wave_sums), the norm among them; reflector,
// update factors and T follow from them in every wavefront by itself:
//   v = [1; scale x],  v^H a_p = a_p(c) + conj(scale) x^H a_p      (p > c)
//   v_p^H v = conj(v_p(c)) + scale conj(x^H v_p)                   (p < c)
// RPT rows per thread, chosen with the threads by the rows that are left.
// Bound by the column's chain (sum, barrier, square root and two reciprocals):
// a panel takes 24 instead of 51 us at 2048 rows, 12 instead of 49 at 256
// (k_qr_panel: four barriers and 96 lane exchanges a column).
template <int THREADS, int RPT>
__global__ __launch_bounds__(THREADS) void k_qr_panel1(const GateDesc *descs, int stage,
                                                          int panel) {
  const GateDesc &d = descs[blockIdx.x];
  if (!d.qr || d.storage != 0) return;
  const QrView q = qr_view(d, stage);
  const int j0 = panel * QNB;
  if (j0 >= q.cols) return;
  const int w = min(QNB, q.cols - j0);
  const int nr = q.rows - j0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int WAVES = THREADS / 64;
  __shared__ double red[2][WAVES][2 * QNB];  // by column parity
  __shared__ double2 top[2][QNB];               // row c of the panel
  double2 a[RPT][QNB];
#pragma unroll
  for (int i = 0; i < RPT; i++) {
    const int lr = tid + THREADS * i;
#pragma unroll
    for (int c = 0; c < QNB; c++)
      a[i][c] = (lr < nr && c < w) ? q.A[(size_t)(j0 + c) * q.ld + j0 + lr]
                                   : make_double2(0.0, 0.0);
  }
  double2 trow[QNB];  // thread t < 8: row t of T
#pragma unroll
  for (int c = 0; c < QNB; c++) trow[c] = make_double2(0.0, 0.0);
#pragma unroll
  for (int c = 0; c < QNB; c++) {
    if (c >= w) break;
    double s[2 * QNB];
#pragma unroll
    for (int p = 0; p < QNB; p++) {
      double2 g = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < RPT; i++) {
        const bool below = i > 0 || tid > c;
        const double2 x = below ? a[i][c] : make_double2(0.0, 0.0);
        if (p == c)
          g.x = fma(x.x, x.x, fma(x.y, x.y, g.x));
        else
          cfmac(g, x, a[i][p]);
      }
      s[2 * p] = g.x;
      s[2 * p + 1] = g.y;
    }
    const double mine = wave_sums<2 * QNB>(s);  // lane l: value l / 4
    if ((lane & 3) == 0) red[c & 1][wave][lane >> 2] = mine;
    if (tid == c) {
#pragma unroll
      for (int p = 0; p < QNB; p++) top[c & 1][p] = a[0][p];
    }
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int v = 0; v < WAVES; v++) tot += red[c & 1][v][lane & 15];
    const double x2 = lane_value(tot, 2 * c);
    const double2 al = top[c & 1][c];
    double2 tau = make_double2(0.0, 0.0), scale = tau;
    double beta = al.x;
    if (!(x2 == 0.0 && al.y == 0.0)) {  // else already triangular: H = I
      const double n2 = cabs2(al) + x2;
      double rb, inv;  // 1 / beta, 1 / |alpha - beta|^2
      double2 dn;      // alpha - beta
      if (n2 > 0x1p-900 && n2 < 0x1p900) {  // (uniform) the short chains hold
        const double r = fast_rsqrt(n2);
        beta = -copysign(fast_sqrt(n2), al.x);
        rb = -copysign(r, al.x);
        dn = make_double2(al.x - beta, al.y);
        inv = fast_rcp(cabs2(dn));
      } else {
        beta = -copysign(sqrt(n2), al.x);
        rb = 1.0 / beta;
        dn = make_double2(al.x - beta, al.y);
        inv = 1.0 / cabs2(dn);
      }
      tau = make_double2((beta - al.x) * rb, -al.y * rb);
      scale = make_double2(dn.x * inv, -dn.y * inv);  // 1 / (alpha - beta)
    }
    const double2 ctau = cconj(tau);
    double2 tc = make_double2(0.0, 0.0);  // sum over p < c of T(t, p) v_p^H v
    double2 v[RPT];
#pragma unroll
    for (int i = 0; i < RPT; i++) {
      const bool below = i > 0 || tid > c, diag = i == 0 && tid == c;
      v[i] = below ? cmul(a[i][c], scale) : make_double2(diag ? 1.0 : 0.0, 0.0);
      if (below) a[i][c] = v[i];
      if (diag) a[i][c] = make_double2(beta, 0.0);
    }
#pragma unroll
    for (int p = 0; p < QNB; p++) {
      if (p == c || p >= w) continue;
      const double2 g = make_double2(lane_value(tot, 2 * p), lane_value(tot, 2 * p + 1));
      const double2 t = top[c & 1][p];
      if (p > c) {  // a_p <- a_p - conj(tau) (v^H a_p) v
        const double2 f = cmul(ctau, cadd(t, cmulc(scale, g)));
#pragma unroll
        for (int i = 0; i < RPT; i++) a[i][p] = csub(a[i][p], cmul(v[i], f));
      } else {
        tc = cadd(tc, cmul(trow[p], cadd(cconj(t), cmul(scale, cconj(g)))));
      }
    }
    // T(0:c, c) = -tau T(0:c, 0:c) (V^H v)(0:c), T(c, c) = tau
    trow[c] = tid < c ? cmul(make_double2(-tau.x, -tau.y), tc)
                      : (tid == c ? tau : make_double2(0.0, 0.0));
  }
#pragma unroll
  for (int i = 0; i < RPT; i++) {
    const int lr = tid + THREADS * i;
    if (lr < nr) {
#pragma unroll
      for (int c = 0; c < QNB; c++)
        if (c < w) q.A[(size_t)(j0 + c) * q.ld + j0 + lr] = a[i][c];
    }
  }
  double2 *T = qr_tfac(d, stage, panel);
  if (tid < QNB) {
#pragma unroll
    for (int c = 0; c < QNB; c++) T[tid * QNB + c] = trow[c];
  }
}

void launch_qr_panel(hipStream_t st, const GateDesc *d, int ng, int stage, int panel, int max_rows,
                     bool c128, bool c64) {
  if (ng <= 0) return;
  const int left = max_rows - panel * QNB;
  using std::integral_constant;
  auto run1 = [&](auto threads, auto rpt) {
    constexpr int T = decltype(threads)::value, R = decltype(rpt)::value;
    hipLaunchKernelGGL((k_qr_panel1<T, R>), dim3(ng), dim3(T), 0, st, d, stage, panel);
  };
  auto run = [&](auto threads, auto rpt) {
    constexpr int T = decltype(threads)::value, R = decltype(rpt)::value;
    hipLaunchKernelGGL((k_qr_panel<T, R>), dim3(ng), dim3(T), 0, st, d, stage, panel);
  };
  if (left <= 256) {
    if (c128) run1(integral_constant<int, 256>(), integral_constant<int, 1>());
    if (c64) run(integral_constant<int, 256>(), integral_constant<int, 1>());
  } else if (left <= 512) {
    if (c128) run1(integral_constant<int, 256>(), integral_constant<int, 2>());
    if (c64) run(integral_constant<int, 512>(), integral_constant<int, 1>());
  } else if (left <= 1024) {
    if (c128) run1(integral_constant<int, 512>(), integral_constant<int, 2>());
    if (c64) run(integral_constant<int, 512>(), integral_constant<int, 2>());
  } else {
    if (c128) run1(integral_constant<int, 512>(), integral_constant<int, 4>());
    if (c64) run(integral_constant<int, 512>(), integral_constant<int, 4>());
  }
}

// ---------------------------------------------------------------- block update

constexpr int QU_ROWS = 64;  // rows per LDS chunk

// Apply a block reflector of NB Householder vectors to COLS target columns per
// workgroup: B = A(j0:, first:last) <- (I - V T V^H)^H B, the columns after the
// block up to col_end.  S = V^H B over all rows, Y = T^H S, B -= V Y; V is staged
// in LDS, the next rows loaded meanwhile.
template <int NB, int COLS, int NT>
__device__ void qr_block_update(const GateDesc &d, const QrView q, int j0, const double2 *T,
                                int col_end) {
  static_assert((NB * COLS) % NT == 0 && NT % QU_ROWS == 0, "whole entries per thread");
  constexpr int EPT = NB * COLS / NT;
  if (j0 >= q.cols) return;
  const int w = min(NB, q.cols - j0);
  const int ldb = q.ld, rows = q.rows, ncols = min(col_end, q.cols) - j0 - w;
  double2 *B = q.A + (size_t)(j0 + w) * ldb;
  const int c0 = blockIdx.x * COLS;
  if (c0 >= ncols) return;
  const int nc = min(COLS, ncols - c0);
  B += (size_t)c0 * ldb;
  const double2 *V = q.A + (size_t)j0 * q.ld;  // reflector p: column p, from row j0 + p

  __shared__ double2 Vs[QU_ROWS][NB + 1];
  __shared__ double2 Bs[QU_ROWS][COLS + 1];
  __shared__ double2 S[NB][COLS];
  __shared__ double2 Y[NB][COLS];
  __shared__ double2 Tl[NB][NB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < NB * NB; e += NT) Tl[e / NB][e % NB] = T[e];

  // rows r0 .. r0+63 of V: 1 on the diagonal, stored below; and of B.  All loads
  // of a chunk are under way before the first is waited for.
  constexpr int VPT = QU_ROWS * NB / NT, BPT = QU_ROWS * COLS / NT;
  auto get_v = [&](double2 (&x)[VPT], int r0) {
#pragma unroll
    for (int k = 0; k < VPT; k++) {
      const int e = tid + NT * k, p = e / QU_ROWS, gr = r0 + e % QU_ROWS;
      x[k] = p < w && gr < rows && gr > j0 + p ? V[(size_t)p * q.ld + gr]
                                               : make_double2(gr == j0 + p && p < w ? 1.0 : 0.0, 0.0);
    }
  };
  auto get_b = [&](double2 (&x)[BPT], int r0) {
#pragma unroll
    for (int k = 0; k < BPT; k++) {
      const int e = tid + NT * k, cc = e / QU_ROWS, gr = r0 + e % QU_ROWS;
      x[k] = gr < rows && cc < nc ? B[(size_t)cc * ldb + gr] : make_double2(0.0, 0.0);
    }
  };
  auto put_v = [&](const double2 (&x)[VPT]) {
#pragma unroll
    for (int k = 0; k < VPT; k++) {
      const int e = tid + NT * k;
      Vs[e % QU_ROWS][e / QU_ROWS] = x[k];
    }
  };

  // phase 1: S = V^H B
  double2 sacc[EPT];
#pragma unroll
  for (int e = 0; e < EPT; e++) sacc[e] = make_double2(0.0, 0.0);
  double2 vx[VPT], bx[BPT];
  get_v(vx, j0);
  get_b(bx, j0);
  for (int r0 = j0; r0 < rows; r0 += QU_ROWS) {
    put_v(vx);
#pragma unroll
    for (int k = 0; k < BPT; k++) {
      const int e = tid + NT * k;
      Bs[e % QU_ROWS][e / QU_ROWS] = bx[k];
    }
    __syncthreads();
    get_v(vx, r0 + QU_ROWS);  // the next chunk (zeros past the end)
    get_b(bx, r0 + QU_ROWS);
#pragma unroll
    for (int e = 0; e < EPT; e++) {
      const int id = tid + NT * e, p = id / COLS, cc = id % COLS;
#pragma unroll 8
      for (int r = 0; r < QU_ROWS; r++) cfmac(sacc[e], Vs[r][p], Bs[r][cc]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int id = tid + NT * e;
    S[id / COLS][id % COLS] = sacc[e];
  }
  __syncthreads();
  // phase 2: Y = T^H S
#pragma unroll
  for (int e = 0; e < EPT; e++) {
    const int id = tid + NT * e, p = id / COLS, cc = id % COLS;
    double2 y = make_double2(0.0, 0.0);
    for (int l = 0; l < NB; l++) {
      const double2 t = cconj(Tl[l][p]);
      y = cadd(y, cmul(t, S[l][cc]));
    }
    Y[p][cc] = y;
  }
  __syncthreads();
  // phase 3: B -= V Y; lanes along rows
  const int rl = tid % QU_ROWS, cg = tid / QU_ROWS;  // 64 rows x column groups
  get_v(vx, j0);
  get_b(bx, j0);  // entry k: column cg + NT / QU_ROWS k of row rl
  for (int r0 = j0; r0 < rows; r0 += QU_ROWS) {
    put_v(vx);
    double2 old[BPT];
#pragma unroll
    for (int k = 0; k < BPT; k++) old[k] = bx[k];
    __syncthreads();
    get_v(vx, r0 + QU_ROWS);
    get_b(bx, r0 + QU_ROWS);
    const int r = r0 + rl;
#pragma unroll
    for (int k = 0; k < BPT; k++) {
      const int cc = cg + NT / QU_ROWS * k;
      if (r < rows && cc < nc) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll
        for (int p = 0; p < NB; p++) cfma(acc, Vs[rl][p], Y[p][cc]);
        B[(size_t)cc * ldb + r] = csub(old[k], acc);
      }
    }
    __syncthreads();
  }
}

constexpr int QU_COLS = 32;  // target columns per workgroup, panel updates

// One panel's reflectors on the columns after it up to col_end (inside its
// group while the group is being factored).
__global__ __launch_bounds__(QNB * QU_COLS) void k_qr_update(const GateDesc *descs, int stage, int panel,
                                                   int col_end) {
  const GateDesc &d = descs[blockIdx.y];
  if (!d.qr || d.storage == 0) return;
  qr_block_update<QNB, QU_COLS, QNB * QU_COLS>(d, qr_view(d, stage), panel * QNB, qr_tfac(d, stage, panel),
                                col_end);
}

// The same for gates with complex128 sites: QU1_COLS columns per workgroup,
// rows dealt to the threads, the 8 x 4 products V^H B in registers and summed
// over the workgroup once.  77 -> 17 us at 2048 rows, 14 -> 7.5 at 256 (one workgroup took all
// columns of the group, its dot products serial over the rows in LDS).
constexpr int QU1_COLS = 4;
__global__ __launch_bounds__(256) void k_qr_update1(const GateDesc *descs, int stage, int panel,
                                                    int col_end) {
  const GateDesc &d = descs[blockIdx.y];
  if (!d.qr || d.storage != 0) return;
  const QrView q = qr_view(d, stage);
  const int j0 = panel * QNB;
  if (j0 >= q.cols) return;
  const int w = min(QNB, q.cols - j0), rows = q.rows;
  const int ncols = min(col_end, q.cols) - j0 - w;
  const int c0 = blockIdx.x * QU1_COLS;
  if (c0 >= ncols) return;
  const int nc = min(QU1_COLS, ncols - c0);
  const double2 *V = q.A + (size_t)j0 * q.ld;
  double2 *B = q.A + (size_t)(j0 + w + c0) * q.ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto vget = [&](int r, int p) {  // reflector p: 1 on its diagonal, stored below
    const int dr = r - (j0 + p);
    return p < w && dr > 0 ? V[(size_t)p * q.ld + r]
                           : make_double2(p < w && dr == 0 ? 1.0 : 0.0, 0.0);
  };
  double s[2 * QNB * QU1_COLS];
#pragma unroll
  for (int e = 0; e < 2 * QNB * QU1_COLS; e++) s[e] = 0.0;
  for (int r = j0 + tid; r < rows; r += 256) {
    double2 v[QNB], b[QU1_COLS];
#pragma unroll
    for (int p = 0; p < QNB; p++) v[p] = vget(r, p);
#pragma unroll
    for (int c = 0; c < QU1_COLS; c++)
      b[c] = c < nc ? B[(size_t)c * q.ld + r] : make_double2(0.0, 0.0);
#pragma unroll
    for (int p = 0; p < QNB; p++)
#pragma unroll
      for (int c = 0; c < QU1_COLS; c++) {
        double2 g = make_double2(s[2 * (p * QU1_COLS + c)], s[2 * (p * QU1_COLS + c) + 1]);
        cfmac(g, v[p], b[c]);
        s[2 * (p * QU1_COLS + c)] = g.x;
        s[2 * (p * QU1_COLS + c) + 1] = g.y;
      }
  }
  __shared__ double red[4][2 * QNB * QU1_COLS];
  __shared__ double2 Y[QNB][QU1_COLS];
  red[wave][lane] = wave_sums<2 * QNB * QU1_COLS>(s);
  __syncthreads();
  if (tid < QNB * QU1_COLS) {  // Y = T^H S
    const int p = tid / QU1_COLS, c = tid % QU1_COLS;
    const double2 *T = qr_tfac(d, stage, panel);
    double2 y = make_double2(0.0, 0.0);
    for (int l = 0; l <= p; l++) {
      const int e = 2 * (l * QU1_COLS + c);
      const double2 sum = make_double2(red[0][e] + red[1][e] + red[2][e] + red[3][e],
                                       red[0][e + 1] + red[1][e + 1] + red[2][e + 1] + red[3][e + 1]);
      y = cadd(y, cmulc(T[l * QNB + p], sum));
    }
    Y[p][c] = y;
  }
  __syncthreads();
  double2 y[QNB][QU1_COLS];
#pragma unroll
  for (int p = 0; p < QNB; p++)
#pragma unroll
    for (int c = 0; c < QU1_COLS; c++) y[p][c] = Y[p][c];
  for (int r = j0 + tid; r < rows; r += 256) {
    double2 v[QNB];
#pragma unroll
    for (int p = 0; p < QNB; p++) v[p] = vget(r, p);
#pragma unroll
    for (int c = 0; c < QU1_COLS; c++)
      if (c < nc) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll
        for (int p = 0; p < QNB; p++) cfma(acc, v[p], y[p][c]);
        double2 *bp = B + (size_t)c * q.ld + r;
        *bp = csub(*bp, acc);
      }
  }
}

void launch_qr_update(hipStream_t st, const GateDesc *d, int ng, int stage, int panel,
                      int col_end, int max_cols, bool c128, bool c64) {
  if (ng <= 0 || max_cols <= 0) return;
  if (c64)
    hipLaunchKernelGGL(k_qr_update, dim3((max_cols + QU_COLS - 1) / QU_COLS, ng),
                       dim3(QNB * QU_COLS), 0, st, d, stage, panel, col_end);
  if (c128)
    hipLaunchKernelGGL(k_qr_update1, dim3((max_cols + QU1_COLS - 1) / QU1_COLS, ng), dim3(256), 0,
                       st, d, stage, panel, col_end);
}

// ------------------------------------------------ group update on matrix cores
//
// A group's QG reflectors on everything after the group (apply = 0), or on U
// (apply = 1, stage-0 groups in reverse order), in three launches so that the
// rows are spread over workgroups as well as the columns:
//   k_qrg_s : partial S = V^H B over a chunk of QR_RC rows      (per chunk)
//   k_qrg_y : Y = op(T) sum_chunks S                           (per column tile)
//   k_qrg_b : B -= V Y over a chunk of rows                     (per chunk)
// Partial sums and Y go to a scratch buffer that is idle at that time (U while
// factoring, the Jacobi matrix once its columns have been gathered into U).
// Fixed summation order: results do not depend on scheduling.

typedef double qd4_t __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64: lane l supplies A[l%16][l/16] and B[l/16][l%16];
// result entry v of lane l is D[l/16 + 4v][l%16].
__device__ __forceinline__ qd4_t qmfma(double a, double b, qd4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int QGT = 32;     // target columns per workgroup

struct QrTarget {
  double2 *B;     // first target column
  int ldb, rows;  // rows of B (all of them; the reflectors start at row j0)
  int ncols;      // target columns
  double2 *scr;   // scratch: partial S then Y, QG rows of ldS each
  int ldS;
};

__device__ __forceinline__ QrTarget qr_target(const GateDesc &d, const QrView &q, int j0, int w,
                                              int apply) {
  QrTarget t;
  t.ldS = d.colsPad;
  if (apply) {
    t.B = d.U;
    t.ldb = d.ldu;
    t.rows = d.m;
    t.ncols = d.sc->k;
    t.scr = d.X;
  } else {
    t.B = q.A + (size_t)(j0 + w) * q.ld;
    t.ldb = q.ld;
    t.rows = q.rows;
    t.ncols = q.cols - j0 - w;
    t.scr = d.U;
  }
  return t;
}

// reflector p of the group at absolute row r: 1 on its diagonal, stored below
__device__ __forceinline__ double2 qr_vget(const QrView &q, int j0, int w, int r, int p) {
  if (p >= w || r >= q.rows) return make_double2(0.0, 0.0);
  const int dr = r - (j0 + p);
  if (dr < 0) return make_double2(0.0, 0.0);
  if (dr == 0) return make_double2(1.0, 0.0);
  return q.A[(size_t)(j0 + p) * q.ld + r];
}

__global__ __launch_bounds__(256) void k_qrg_s(const GateDesc *descs, int stage, int group,
                                               int apply, int gram_tile) {
  const GateDesc &d = descs[blockIdx.z];
  if (!d.qr) return;
  const int stg = apply ? 0 : stage;
  const QrView q = qr_view(d, stg);
  const int j0 = group * QG;
  if (j0 >= q.cols) return;
  const int w = min(QG, q.cols - j0);
  const QrTarget t = qr_target(d, q, j0, w, apply);
  // while factoring a gate with complex128 sites, the first column tile of
  // the launch is V itself: V^H V, from which k_qrg_y solves for T's product
  const bool gram = gram_tile && blockIdx.x == 0;
  if (gram && d.storage != 0) return;
  const int c0 = ((int)blockIdx.x - gram_tile) * QGT;
  const int rbeg = j0 + blockIdx.y * QR_RC;
  if ((!gram && c0 >= t.ncols) || rbeg >= t.rows) return;
  const int rend = min(t.rows, rbeg + QR_RC);
  __shared__ double2 Vs[32][QG + 1];
  __shared__ double2 Bs[32][QGT + 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, lg = lane >> 4;
  const int tp = (wave >> 1) * 16, tc = (wave & 1) * 16;  // this wave's 16x16 tile of S
  qd4_t accR = {0.0, 0.0, 0.0, 0.0}, accI = {0.0, 0.0, 0.0, 0.0};
  // Rows come in chunks of 32, each thread holding 4 elements of V and 4 of
  // B per chunk.  Two chunks are in flight ahead of the one being
  // multiplied: buffer loads (counted apart from the LDS accesses), never
  // skipped, and masked only when written to LDS.
  static_assert(32 * QG == 4 * 256 && 32 * QGT == 4 * 256, "four elements per thread");
  const BufRes rA = make_res(q.A, q.ld * q.cols);
  const BufRes rB = gram ? rA : make_res(t.B, t.ldb * t.ncols);
  const int ldb = gram ? q.ld : t.ldb, cb = gram ? j0 : c0;
  auto load = [&](int r0, double2 *vv, double2 *bb) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int e = tid + 256 * k, r = e % 32, p = e / 32;
      vv[k] = bload(rA, (j0 + p) * q.ld + r0 + r);
      bb[k] = bload(rB, (cb + p) * ldb + r0 + r);
    }
  };
  auto to_lds = [&](int r0, const double2 *vv, const double2 *bb) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int e = tid + 256 * k, r = e % 32, p = e / 32;
      const int rr = r0 + r, dr = rr - (j0 + p);  // reflector p: 1 on its diagonal, stored below
      const bool in = rr < rend;
      Vs[r][p] = (in && p < w && dr > 0) ? vv[k] : make_double2(in && p < w && dr == 0 ? 1.0 : 0.0, 0.0);
      Bs[r][p] = gram ? Vs[r][p] : (in && c0 + p < t.ncols) ? bb[k] : make_double2(0.0, 0.0);
    }
  };
  auto chunk = [&]() {
#pragma unroll
    for (int kk = 0; kk < 32; kk += 4) {
      const double2 a = Vs[kk + lg][tp + l16];  // S = conj(V)^T B
      const double2 b = Bs[kk + lg][tc + l16];
      accR = qmfma(a.x, b.x, accR);
      accR = qmfma(a.y, b.y, accR);
      accI = qmfma(a.x, b.y, accI);
      accI = qmfma(-a.y, b.x, accI);
    }
  };
  const int nchunk = (rend - rbeg + 31) / 32;
  double2 va[4], ba[4], vb[4], bb[4];
  load(rbeg, va, ba);
  load(rbeg + 32, vb, bb);
  for (int c = 0; c < nchunk; c += 2) {  // an odd last chunk is followed by an all-zero one
    const int r0 = rbeg + 32 * c;
    to_lds(r0, va, ba);
    __syncthreads();
    load(r0 + 64, va, ba);
    chunk();
    __syncthreads();
    to_lds(r0 + 32, vb, bb);
    __syncthreads();
    load(r0 + 96, vb, bb);
    chunk();
    __syncthreads();
  }
  double2 *Sp = t.scr + (size_t)blockIdx.y * QG * t.ldS;
#pragma unroll
  for (int v = 0; v < 4; v++) {
    const int p = tp + lg + 4 * v, c = c0 + tc + l16;
    // V^H V goes to the last QG columns of the scratch rows: a full group has
    // at most ldS - QG columns after it, a narrower (last) one has none
    if (gram)
      Sp[(size_t)p * t.ldS + t.ldS - QG + tc + l16] = make_double2(accR[v], accI[v]);
    else if (c < t.ncols)
      Sp[(size_t)p * t.ldS + c] = make_double2(accR[v], accI[v]);
  }
}

__global__ __launch_bounds__(256) void k_qrg_y(const GateDesc *descs, int stage, int group,
                                               int apply) {
  const GateDesc &d = descs[blockIdx.y];
  if (!d.qr) return;
  const int stg = apply ? 0 : stage;
  const QrView q = qr_view(d, stg);
  const int j0 = group * QG;
  if (j0 >= q.cols) return;
  const int w = min(QG, q.cols - j0);
  const QrTarget t = qr_target(d, q, j0, w, apply);
  const int c0 = blockIdx.x * QGT;
  const bool solve = d.storage == 0;
  // the first workgroup also keeps V^H V and tau for U = Q1 [W; 0]
  if (c0 >= t.ncols && !(solve && !apply && blockIdx.x == 0)) return;
  const int nch = (t.rows - j0 + QR_RC - 1) / QR_RC;
  __shared__ double2 S[QG][QGT + 1];
  __shared__ double2 Tl[QG][QG + 1];
  double2 *T = qr_tgrp(d, stg, group);
  const int tid = threadIdx.x;
  for (int e = tid; e < QG * QGT; e += 256) {
    const int p = e / QGT, cc = e % QGT, c = c0 + cc;
    double2 sum = make_double2(0.0, 0.0);
    if (c < t.ncols)
      for (int ch = 0; ch < nch; ch++)
        sum = cadd(sum, t.scr[((size_t)ch * QG + p) * t.ldS + c]);
    S[p][cc] = sum;
  }
  for (int e = tid; e < QG * QG; e += 256) {
    const int p = e / QG, l = e % QG;
    if (solve && !apply) {  // T of the panels on the diagonal, V^H V above
      double2 g = make_double2(0.0, 0.0);
      if (p / QNB == l / QNB) {
        if (j0 + p < q.cols) g = qr_tfac(d, stg, (j0 + p) / QNB)[(p % QNB) * QNB + l % QNB];
      } else if (p < l) {
        for (int ch = 0; ch < nch; ch++)
          g = cadd(g, t.scr[((size_t)ch * QG + p) * t.ldS + t.ldS - QG + l]);
      }
      Tl[p][l] = g;
      if (blockIdx.x == 0) T[e] = g;
    } else {
      Tl[p][l] = T[e];
    }
  }
  __syncthreads();
  double2 *Yg = t.scr + (size_t)nch * QG * t.ldS;  // after the partials
  if (solve) {
    // T^-1 is block upper triangular with the panels' T_b^-1 on the diagonal
    // and V_a^H V_b above, so Y = op(T) S is a block substitution over the
    // four panels: Y_b = op(T_b) S_b, then Y_b is taken out of the panels
    // after it (T^H: ascending) or before it (T: descending).  Thread (cc,
    // part) has column cc and row `part` of each panel.
    const int cc = tid % QGT, part = tid / QGT, nb = (w + QNB - 1) / QNB;
    static_assert(256 / QGT == QNB, "a row of the panel per thread");
    for (int k = 0; k < nb; k++) {
      const int o = QNB * (apply ? nb - 1 - k : k);
      double2 y = make_double2(0.0, 0.0);
#pragma unroll
      for (int l = 0; l < QNB; l++)  // T_b is upper triangular
        y = cadd(y, cmul(apply ? Tl[o + part][o + l] : cconj(Tl[o + l][o + part]), S[o + l][cc]));
      __syncthreads();
      S[o + part][cc] = y;
      __syncthreads();
      for (int r = apply ? part : o + QNB + part; r < (apply ? o : QG); r += QNB) {
        double2 x = S[r][cc];
#pragma unroll
        for (int l = 0; l < QNB; l++)
          x = csub(x, cmul(apply ? Tl[r][o + l] : cconj(Tl[o + l][r]), S[o + l][cc]));
        S[r][cc] = x;
      }
      __syncthreads();
    }
    for (int e = tid; e < QG * QGT; e += 256) {
      const int p = e / QGT, c = c0 + e % QGT;
      if (c < t.ncols) Yg[(size_t)p * t.ldS + c] = S[p][e % QGT];
    }
    return;
  }
  for (int e = tid; e < QG * QGT; e += 256) {
    const int p = e / QGT, cc = e % QGT, c = c0 + cc;
    double2 y = make_double2(0.0, 0.0);
    for (int l = 0; l < QG; l++) {
      const double2 tv = apply ? Tl[p][l] : cconj(Tl[l][p]);  // T or T^H
      y = cadd(y, cmul(tv, S[l][cc]));
    }
    if (c < t.ncols) Yg[(size_t)p * t.ldS + c] = y;
  }
}

__global__ __launch_bounds__(256) void k_qrg_b(const GateDesc *descs, int stage, int group,
                                               int apply) {
  const GateDesc &d = descs[blockIdx.z];
  if (!d.qr) return;
  const int stg = apply ? 0 : stage;
  const QrView q = qr_view(d, stg);
  const int j0 = group * QG;
  if (j0 >= q.cols) return;
  const int w = min(QG, q.cols - j0);
  const QrTarget t = qr_target(d, q, j0, w, apply);
  const int c0 = blockIdx.x * QGT;
  const int rbeg = j0 + blockIdx.y * QR_RC;
  if (c0 >= t.ncols || rbeg >= t.rows) return;
  const int rend = min(t.rows, rbeg + QR_RC);
  const int nch = (t.rows - j0 + QR_RC - 1) / QR_RC;
  __shared__ double2 Ys[QG][QGT + 1];
  const double2 *Yg = t.scr + (size_t)nch * QG * t.ldS;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, lg = lane >> 4;
  for (int e = tid; e < QG * QGT; e += 256) {
    const int p = e / QGT, cc = e % QGT;
    Ys[p][cc] = (c0 + cc < t.ncols) ? Yg[(size_t)p * t.ldS + c0 + cc] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  // (V Y)^T = Y^T V^T: tiles of 16 target columns x 16 rows; the wave's tiles
  // are column tile (wave & 1) and every other row tile of the chunk
  // the next tile's V and B entries are loaded while the current tile is
  // multiplied (row tiles of one wave never overlap those of another)
  const int tc = (wave & 1) * 16;
  // Buffer loads and stores (counted apart from the LDS reads of Y), never
  // skipped: what lies past the chunk is masked when used, stores past it
  // are dropped by their offset.  Row tiles of one wave never overlap those
  // of another; the next tile's V and B are loaded while the current tile
  // is multiplied, into the other of two register sets.
  const BufRes rA = make_res(q.A, q.ld * q.cols);
  const BufRes rB = make_res(t.B, t.ldb * t.ncols);
  auto load = [&](int rt, double2 *vv, double2 *bb) {
    const int r = rt + l16;
#pragma unroll
    for (int k = 0; k < QG / 4; k++) vv[k] = bload(rA, (j0 + 4 * k + lg) * q.ld + r);  // V^T[k][row]
#pragma unroll
    for (int v = 0; v < 4; v++) bb[v] = bload(rB, (c0 + tc + lg + 4 * v) * t.ldb + r);
  };
  auto tile = [&](int rt, const double2 *vv, const double2 *bb) {
    const int r = rt + l16;
    qd4_t accR = {0.0, 0.0, 0.0, 0.0}, accI = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < QG / 4; k++) {
      const int p = 4 * k + lg, dr = r - (j0 + p);  // reflector p: 1 on its diagonal, stored below
      const bool ok = r < rend && p < w;
      const double2 b = (ok && dr > 0) ? vv[k] : make_double2(ok && dr == 0 ? 1.0 : 0.0, 0.0);
      const double2 a = Ys[4 * k + lg][tc + l16];  // Y^T[col][k]
      accR = qmfma(a.x, b.x, accR);
      accR = qmfma(-a.y, b.y, accR);
      accI = qmfma(a.x, b.y, accI);
      accI = qmfma(a.y, b.x, accI);
    }
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int c = c0 + tc + lg + 4 * v;
      const bool ok = r < rend && c < t.ncols;
      bstore_bytes(rB, ok ? (c * t.ldb + r) * 16 : BUF_DROP,
                   make_double2(bb[v].x - accR[v], bb[v].y - accI[v]));
    }
  };
  const int rt0 = rbeg + (wave >> 1) * 16;
  const int ntile = rt0 < rend ? (rend - rt0 + 31) / 32 : 0;
  double2 va[QG / 4], ba[4], vb[QG / 4], bb[4];
  load(rt0, va, ba);
  for (int i = 0; i < ntile; i += 2) {  // an odd last tile is followed by one past the chunk
    const int rt = rt0 + 32 * i;
    load(rt + 32, vb, bb);
    tile(rt, va, ba);
    load(rt + 64, va, ba);
    tile(rt + 32, vb, bb);
  }
}

void launch_qr_update_group(hipStream_t st, const GateDesc *d, int ng, int stage, int group,
                            int apply, int max_cols, int max_rows, bool c128) {
  if (ng <= 0 || max_rows <= group * QG) return;
  const int gram = c128 && !apply;  // V^H V of every group, also the last
  if (max_cols <= 0 && !gram) return;
  const int ct = max_cols > 0 ? (max_cols + QGT - 1) / QGT : 0;
  const int rc = (max_rows - group * QG + QR_RC - 1) / QR_RC;
  hipLaunchKernelGGL(k_qrg_s, dim3(ct + gram, rc, ng), dim3(256), 0, st, d, stage, group, apply,
                     gram);
  hipLaunchKernelGGL(k_qrg_y, dim3(std::max(ct, 1), ng), dim3(256), 0, st, d, stage, group, apply);
  if (ct)
    hipLaunchKernelGGL(k_qrg_b, dim3(ct, rc, ng), dim3(256), 0, st, d, stage, group, apply);
}

// T factor of a group of QG reflectors (compact WY, forward, columnwise):
// T(i, i) = tau_i (from the panels' factors), T(0:i, i) = -tau_i T(0:i, 0:i)
// (V(:, 0:i)^H v_i), with the Gram V^H V summed over the group's rows in turn.
// Gates with complex64 sites only; complex128 ones take V^H V from k_qrg_s.
//
// The Gram's columns first, QT_COLS per workgroup, one entry above the diagonal
// per thread, into the place of T, the next rows' loads under way during the
// sums; then T, row t in the registers of thread t (no barriers: G's column i
// is the same for every row).  Bound by the chains of both.  One workgroup that
// took the Gram, with loads and sums in turn, and a barrier per column of T:
// 62 us at 512 rows, 51 at 256; now 16.3 + 16.6 and 13.5 + 16.6.
constexpr int QT_COLS = 4;
__global__ __launch_bounds__(QG * QT_COLS) void k_qr_tgram(const GateDesc *descs, int stage,
                                                           int group) {
  constexpr int NT = QG * QT_COLS;
  const GateDesc &d = descs[blockIdx.y];
  if (!d.qr || d.storage == 0) return;
  const QrView q = qr_view(d, stage);
  const int j0 = group * QG, l0 = blockIdx.x * QT_COLS;
  if (j0 + l0 >= q.cols) return;
  const int nv = min(l0 + QT_COLS, q.cols - j0);  // reflectors that count here
  const double2 *V = q.A + (size_t)j0 * q.ld;
  __shared__ double2 Vs[QU_ROWS][QG + 1];
  const int tid = threadIdx.x, p = tid / QT_COLS, l = l0 + tid % QT_COLS;
  double2 acc = make_double2(0.0, 0.0);
  constexpr int VPT = QU_ROWS * QG / NT;
  double2 x[VPT];
  auto get = [&](int r0) {
#pragma unroll
    for (int k = 0; k < VPT; k++) {
      const int e = tid + NT * k, c = e / QU_ROWS, gr = r0 + e % QU_ROWS;
      x[k] = c < nv && gr < q.rows && gr > j0 + c
                 ? V[(size_t)c * q.ld + gr]
                 : make_double2(gr == j0 + c && c < nv ? 1.0 : 0.0, 0.0);
    }
  };
  get(j0 + l0);
  for (int r0 = j0 + l0; r0 < q.rows; r0 += QU_ROWS) {  // v_l starts at row l
#pragma unroll
    for (int k = 0; k < VPT; k++) {
      const int e = tid + NT * k;
      Vs[e % QU_ROWS][e / QU_ROWS] = x[k];
    }
    __syncthreads();
    get(r0 + QU_ROWS);
    if (p < l && l < nv) {
#pragma unroll 8
      for (int r = 0; r < QU_ROWS; r++) cfmac(acc, Vs[r][p], Vs[r][l]);
    }
    __syncthreads();
  }
  if (p < l && l < nv) qr_tgrp(d, stage, group)[p * QG + l] = acc;
}

__global__ __launch_bounds__(64) void k_qr_tgroup(const GateDesc *descs, int stage, int group) {
  const GateDesc &d = descs[blockIdx.x];
  if (!d.qr || d.storage == 0) return;
  const QrView q = qr_view(d, stage);
  const int j0 = group * QG;
  if (j0 >= q.cols) return;
  const int w = min(QG, q.cols - j0);
  double2 *Tg = qr_tgrp(d, stage, group);
  __shared__ double2 G[QG][QG];
  __shared__ double2 taus[QG];
  const int tid = threadIdx.x;
  double2 g[QG * QG / 64];
#pragma unroll
  for (int k = 0; k < QG * QG / 64; k++) {  // (what lies on and below the diagonal is not used)
    const int p = (tid + 64 * k) / QG, l = tid % QG;
    g[k] = p < l && l < w ? Tg[tid + 64 * k] : make_double2(0.0, 0.0);
  }
  if (tid < QG)
    taus[tid] = tid < w ? qr_tfac(d, stage, (j0 + tid) / QNB)[(tid % QNB) * (QNB + 1)]
                        : make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < QG * QG / 64; k++) (&G[0][0])[tid + 64 * k] = g[k];
  __syncthreads();
  if (tid >= QG) return;
  double2 T[QG];  // row tid
#pragma unroll
  for (int i = 0; i < QG; i++) {
    const double2 tau = taus[i];
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int l = 0; l < i; l++) {  // (T(tid, l) = 0 before the diagonal)
      const double2 t = T[l], x = G[l][i];
      s.x += fma(t.x, x.x, -(t.y * x.y));
      s.y += fma(t.y, x.x, t.x * x.y);
    }
    const bool before = tid < i, at = tid == i;
    T[i].x = before ? fma(tau.y, s.y, -(tau.x * s.x)) : (at ? tau.x : 0.0);
    T[i].y = before ? fma(-tau.y, s.x, -(tau.x * s.y)) : (at ? tau.y : 0.0);
  }
#pragma unroll
  for (int i = 0; i < QG; i++) Tg[tid * QG + i] = T[i];
}

void launch_qr_tgroup(hipStream_t st, const GateDesc *d, int ng, int stage, int group) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_qr_tgram, dim3(QG / QT_COLS, ng), dim3(QG * QT_COLS), 0, st, d, stage,
                     group);
  hipLaunchKernelGGL(k_qr_tgroup, dim3(ng), dim3(64), 0, st, d, stage, group);
}

// ---------------------------------------------------------------- triangular transposes

constexpr int QT = 32;

// X (n x n) = R1^H: lower triangle conj(R1)^T, upper triangle zero.  R1 is
// the upper triangle of Qm.  grid: (tiles of X rows, tiles of X columns, gate)
__global__ __launch_bounds__(256) void k_qr_r1h(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.z];
  if (!d.qr) return;
  const int n = d.n;
  const int i0 = blockIdx.x * QT, jc0 = blockIdx.y * QT;  // X rows i, X columns j
  if (i0 >= n || jc0 >= n) return;
  __shared__ double2 t[QT][QT + 1];
  const int tid = threadIdx.x;
  // X(i, j) = conj(R1(j, i)) = conj(Qm[i * ldq + j]) for i >= j
  for (int e = tid; e < QT * QT; e += 256) {
    const int jj = e % QT, ii = e / QT;  // read along j (rows of Qm column i)
    const int i = i0 + ii, j = jc0 + jj;
    t[ii][jj] = (i < n && j < n && i >= j) ? cconj(d.Qm[(size_t)i * d.ldq + j])
                                           : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int e = tid; e < QT * QT; e += 256) {
    const int ii = e % QT, jj = e / QT;  // write along i (rows of X column j)
    const int i = i0 + ii, j = jc0 + jj;
    if (i < n && j < n) d.X[(size_t)j * d.ldx + i] = t[ii][jj];
  }
}

void launch_qr_r1h(hipStream_t st, const GateDesc *d, int ng, int max_n) {
  if (ng <= 0 || max_n <= 0) return;
  const int nt = (max_n + QT - 1) / QT;
  hipLaunchKernelGGL(k_qr_r1h, dim3(nt, nt, ng), dim3(256), 0, st, d);
}

// In place in X: R2 (upper triangle, reflectors below) -> R2^H (lower
// triangle, zero above).  The workgroup of tile pair (I, J), I <= J, reads
// the upper tile (I, J) and writes tiles (J, I) and (I, J); nothing else
// touches them.
__global__ __launch_bounds__(256) void k_qr_r2h(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.z];
  if (!d.qr) return;
  const int n = d.n;
  const int I = blockIdx.x, J = blockIdx.y;
  if (I > J || I * QT >= n || J * QT >= n) return;
  __shared__ double2 t[QT][QT + 1];  // t[r][c] = R2(I*QT + r, J*QT + c)
  const int tid = threadIdx.x;
  for (int e = tid; e < QT * QT; e += 256) {
    const int r = e % QT, c = e / QT;
    const int gr = I * QT + r, gc = J * QT + c;
    t[r][c] = (gr < n && gc < n && gr <= gc) ? d.X[(size_t)gc * d.ldx + gr]
                                             : make_double2(0.0, 0.0);
  }
  __syncthreads();
  // X(J*QT + c, I*QT + r) = conj(R2(I*QT + r, J*QT + c)); upper entries cleared
  for (int e = tid; e < QT * QT; e += 256) {
    const int c = e % QT, r = e / QT;  // along the rows c of column I*QT + r
    const int gi = J * QT + c, gj = I * QT + r;
    if (gi < n && gj < n) d.X[(size_t)gj * d.ldx + gi] = cconj(t[r][c]);
  }
  for (int e = tid; e < QT * QT; e += 256) {
    const int r = e % QT, c = e / QT;
    const int gr = I * QT + r, gc = J * QT + c;
    if (gr < n && gc < n && gr < gc) d.X[(size_t)gc * d.ldx + gr] = make_double2(0.0, 0.0);
  }
}

void launch_qr_r2h(hipStream_t st, const GateDesc *d, int ng, int max_n) {
  if (ng <= 0 || max_n <= 0) return;
  const int nt = (max_n + QT - 1) / QT;
  hipLaunchKernelGGL(k_qr_r2h, dim3(nt, nt, ng), dim3(256), 0, st, d);
}

// ---------------------------------------------------------------- U = [W_k; 0]

// Column j of U: the kept Jacobi column perm[j] divided by its norm (rows
// 0..n-1), zero below.  grid: (row tiles of 64, kept columns, gate)
__global__ __launch_bounds__(64) void k_qr_gather(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.z];
  if (!d.qr) return;
  const int j = blockIdx.y;
  if (j >= d.sc->k) return;
  const int r = blockIdx.x * 64 + threadIdx.x;
  if (r >= d.m) return;
  const int col = d.perm[j];
  const double inv = 1.0 / sqrt(d.sig2[col]);
  d.U[(size_t)j * d.ldu + r] =
      r < d.n ? cscale(d.X[(size_t)col * d.ldx + r], inv) : make_double2(0.0, 0.0);
}

void launch_qr_gather(hipStream_t st, const GateDesc *d, int ng, int max_m, int max_k) {
  if (ng <= 0 || max_m <= 0 || max_k <= 0) return;
  hipLaunchKernelGGL(k_qr_gather, dim3((max_m + 63) / 64, max_k, ng), dim3(64), 0, st, d);
}

}  // namespace tn
