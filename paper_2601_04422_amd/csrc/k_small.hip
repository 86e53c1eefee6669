// Two-qubit gates whose Jacobi matrix fits in the LDS of one workgroup:
// merge, gate, weight (Sec. III.A, IV.A) and the whole one-sided Jacobi SVD in
// one launch, one workgroup per gate.
//
// The block Jacobi (k_jacobi.hip) takes about 140 us per sweep on such a
// matrix, nearly all of it launches, the host's convergence test and one pair
// solve of 63 rounds, whatever the size; a circuit of 10 qubits spent 97% of
// its time there.  Here the columns of X (X = M, or M^H when M is wide or the
// caller needs the full left basis, then with J's rows appended below) lie in
// LDS, and a round rotates all disjoint pairs of the circle method on `cols`
// columns, 16 lanes per pair: x^H y by row rotations, the rotation, both
// columns written back, one barrier.  Squared norms are kept with the columns
// and computed afresh at the start of every sweep, so the last sweep, which
// rotates nothing, tests against exact norms.
//
// Bound by the chain of a round (LDS read, 16-lane sum, rotation parameters,
// LDS write, barrier).  Ten layers of a 10-qubit circuit: 8.7 -> 2.2 ms; one
// gate at chi = 24 with its readout: 2.2 -> 1.2 ms; loss and gradient of a
// 14-qubit ansatz: 75 -> 31 ms.
#include "tnsim_internal.h"
#include "tn_complex.h"
#include "tn_lanes.h"
#include "tn_fast.h"

#include <cfloat>
#include <type_traits>

namespace tn {

// Rows of a column in LDS: whole rows of 16 lanes, one of the counts that
// small_sweeps is unrolled for.
__host__ __device__ __forceinline__ int small_ld(int tot) {
  const int nt = (tot + 15) / 16;
  return 16 * (nt <= 4 ? nt : nt <= 6 ? 6 : nt <= 8 ? 8 : SMALL_ROWS / 16);
}

// sum over the 16 lanes of a row, in every lane
__device__ __forceinline__ double row_sum(double x) {
  x += row_next<8>(x);
  x += row_next<4>(x);
  x += row_next<2>(x);
  return x + row_next<1>(x);
}

// Sweeps over the columns of X (rows of the dot products, then J's rows, NT
// rows of 16 lanes in all) until one rotates nothing; returns whether the last
// sweep still rotated, with the sweeps taken in `sweep`.  RARE: rotations are
// counted in `nrot`, and one from an infinite radicand vanishes, as 2 / inf
// does (so that the gate ends in E_NOCONV).  Both cost every gate 3 % (75.0 ->
// 77.5 us a launch in ten layers of a 10-qubit circuit), so that the sweeps of
// gates that need neither are compiled without them.
template <int NT, int GROUPS, bool RARE>
__device__ __forceinline__ int small_sweeps(double2 *X, double *nrm, int &rotated, int rows,
                                            int cols, int maxSweeps, double tol2, double small,
                                            int &sweep, unsigned &nrot) {
  constexpr int ld = 16 * NT;
  const int tid = threadIdx.x, l = tid & 15, grp = tid >> 4;
  const int P = (cols + 1) & ~1;  // players of the circle method
  int rot = 1;
  sweep = 0;
  while (rot && sweep < maxSweeps) {
    sweep++;
    // squared norms afresh
    for (int c = grp; c < cols; c += GROUPS) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < NT; i++)
        if (16 * i + l < rows) s += cabs2(X[c * ld + 16 * i + l]);
      s = row_sum(s);
      if (l == 0) nrm[c] = s;
    }
    if (tid == 0) rotated = 0;
    __syncthreads();
    // pair grp of round r: (r, P - 1) for grp = 0, (r + grp, r - grp) mod P - 1 otherwise
    int pu = grp, pd = grp ? P - 1 - grp : 0;
    for (int r = 0; r < P - 1; r++) {
      const int o = grp ? pd : P - 1;
      const int p = min(pu, o), q = max(pu, o);
      pu = pu + 1 == P - 1 ? 0 : pu + 1;
      pd = pd + 1 == P - 1 ? 0 : pd + 1;
      if (grp < P / 2 && q < cols) {  // an odd column sits out
        double2 *xp = X + p * ld + l, *yp = X + q * ld + l;
        const double a = nrm[p], b = nrm[q];
        double2 x[NT], y[NT];
#pragma unroll
        for (int i = 0; i < NT; i++) {
          x[i] = xp[16 * i];
          y[i] = yp[16 * i];
        }
        double2 g = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < NT; i++)
          if (16 * i + l < rows) cfmac(g, x[i], y[i]);
        g = make_double2(row_sum(g.x), row_sum(g.y));
        const double h = cabs2(g);
        if (a > small && b > small && h > tol2 * a * b) {
          // as in the pair solve: w = 2 sign(delta) / (|delta| + sqrt(delta^2
          // + 4h)), cosine 1 / sqrt(1 + w^2 h), s e^{i phi} = c w g
          const double delta = b - a, s2 = fma(delta, delta, 4.0 * h);
          double w = copysign(2.0 * fast_rcp(fabs(delta) + s2 * fast_rsqrt(s2)), delta);
          if (RARE && !(s2 <= DBL_MAX)) w = 0.0;
          const double wh = w * h, c = fast_rsqrt(fma(w, wh, 1.0)), cw = c * w;
          const double2 se = make_double2(cw * g.x, cw * g.y), sec = cconj(se);
#pragma unroll
          for (int i = 0; i < NT; i++) {
            xp[16 * i] = csub(cscale(x[i], c), cmul(sec, y[i]));
            yp[16 * i] = cadd(cmul(se, x[i]), cscale(y[i], c));
          }
          if (RARE) nrot++;
          if (l == 0) {
            nrm[p] = a - wh;
            nrm[q] = b + wh;
            rotated = 1;
          }
        }
      }
      __syncthreads();
    }
    rot = rotated;
    __syncthreads();  // every thread reads before it is cleared
  }
  return rot;
}

template <int THREADS, int ELEMS, int CLASS>
__global__ __launch_bounds__(THREADS) void k_small(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.x];
  if (d.small != CLASS) return;
  __shared__ double2 X[ELEMS];       // column c, row r at c * ld + r
  __shared__ double nrm[64];         // squared column norms
  __shared__ int rotated;
  const int tid = threadIdx.x, l = tid & 15, grp = tid >> 4;
  constexpr int GROUPS = THREADS / 16;
  const int m = d.m, n = d.n, chiL = d.chiL, chiM = d.chiM, chiR = d.chiR;
  const int rows = d.rows, cols = d.cols, tot = rows + (d.trans ? m : 0);
  const int ld = small_ld(tot);

  // theta' (kept for the write-back) and X
  for (int e = tid; e < cols * ld; e += THREADS) {
    const int r = e % ld, c = e / ld;
    if (r >= rows) X[e] = make_double2(d.trans && r - rows == c ? 1.0 : 0.0, 0.0);
  }
  const double2 *A0 = (const double2 *)d.A0, *A1 = (const double2 *)d.A1;
  double2 *T = (double2 *)d.T;
  for (int task = tid; task < chiL * chiR; task += THREADS) {
    const int a = task / chiR, c = task - a * chiR;
    const double2 *p0 = A0 + (size_t)a * 2 * chiM, *q0 = A1 + c;
    double2 v[4];
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int b = 0; b < chiM; b++) {
      const double2 x0 = p0[b], x1 = p0[chiM + b];
      const double2 y0 = q0[(size_t)b * 2 * chiR], y1 = q0[(size_t)b * 2 * chiR + chiR];
      cfma(v[0], x0, y0);
      cfma(v[1], x0, y1);
      cfma(v[2], x1, y0);
      cfma(v[3], x1, y1);
    }
    const double w = d.lamR ? d.lamR[c] : 1.0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      double2 o = make_double2(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < 4; j++) cfma(o, d.g[e * 4 + j], v[j]);
      const int r = 2 * a + (e >> 1), t = e & 1;
      T[(size_t)r * n + t * chiR + c] = o;
      if (!d.trans)
        X[(2 * c + t) * ld + r] = cscale(o, w);  // columns in the order (c, t), as the merge
      else
        X[r * ld + t * chiR + c] = cscale(cconj(o), w);
    }
  }
  __syncthreads();

  // ||X||_F^2 for the rounding-noise rule, every thread the same sum
  for (int c = grp; c < cols; c += GROUPS) {
    double v = 0.0;
    for (int r = l; r < rows; r += 16) v += cabs2(X[c * ld + r]);
    v = row_sum(v);
    if (l == 0) nrm[c] = v;
  }
  __syncthreads();
  double fro2 = 0.0;
  for (int c = 0; c < cols; c++) fro2 += nrm[c];
  __syncthreads();
  const double eps_r = rows * 0x1p-53, small = fro2 * eps_r * eps_r, tol2 = d.tol * d.tol;
  int sweep = 0, rot = 0;
  unsigned nrot = 0;  // rotations of this group of lanes (profiling)
  auto sweeps = [&](auto rare) {
    auto run = [&](auto nt) {
      rot = small_sweeps<decltype(nt)::value, GROUPS, decltype(rare)::value>(
          X, nrm, rotated, rows, cols, d.maxSweeps, tol2, small, sweep, nrot);
    };
    switch (ld / 16) {
      case 1: run(std::integral_constant<int, 1>()); break;
      case 2: run(std::integral_constant<int, 2>()); break;
      case 3: run(std::integral_constant<int, 3>()); break;
      case 4: run(std::integral_constant<int, 4>()); break;
      case 5:
      case 6: run(std::integral_constant<int, 6>()); break;
      case 7:
      case 8: run(std::integral_constant<int, 8>()); break;
      default: run(std::integral_constant<int, SMALL_ROWS / 16>()); break;
    }
  };
  // (norms below 2^510 have finite squares)
  if (__builtin_amdgcn_readfirstlane(d.ctr || !(fro2 < 0x1p510)))
    sweeps(std::true_type());
  else
    sweeps(std::false_type());
  // left vectors and squared norms where the truncation and the write-back
  // (and the adjoint) look for them
  for (int e = tid; e < cols * ld; e += THREADS) {
    const int r = e % ld, c = e / ld;
    if (!d.trans && r < rows) d.X[(size_t)c * d.ldx + r] = X[e];
    if (d.trans && r >= rows && r < tot) d.J[(size_t)c * d.ldj + r - rows] = X[e];
  }
  for (int c = tid; c < cols; c += THREADS) d.sig2[c] = nrm[c];
  // 8 flops a row for the dot product of every pair of columns, 32 a row (J's
  // included) for a rotation of two columns
  if (d.ctr && l == 0) {
    const unsigned dots = tid == 0 ? sweep * (cols * (cols - 1) / 2) : 0;
    atomicAdd(&d.ctr[CTR_SMALL_FLOP], 8ull * dots * rows + 32ull * nrot * tot);
  }
  if (tid == 0) {
    d.sc->fro2 = fro2;
    d.sc->rot = rot;  // 1: not converged
    d.sc->active = 0;
    d.sc->sweeps = sweep;
    d.sc->k = 0;
  }
}

// Class of a gate: 0 (block Jacobi), or the k_small variant that holds it.
// X takes `cols` columns of its rows (and J's) in LDS; the first variant
// leaves room for four workgroups on a CU.
int small_class(int rows, int cols, int jrows) {
  const int tot = rows + jrows, ld = small_ld(tot);
  if (tot > SMALL_ROWS || cols > 64) return 0;
  if (cols <= 32 && cols * ld <= SMALL_ELEMS_1) return 1;
  return cols * ld <= SMALL_ELEMS_2 ? 2 : 0;
}

void launch_small(hipStream_t st, const GateDesc *d, int ng, bool class1, bool class2) {
  if (ng <= 0) return;
  if (class1)
    hipLaunchKernelGGL((k_small<256, SMALL_ELEMS_1, 1>), dim3(ng), dim3(256), 0, st, d);
  if (class2)
    hipLaunchKernelGGL((k_small<512, SMALL_ELEMS_2, 2>), dim3(ng), dim3(512), 0, st, d);
}

}  // namespace tn
