// Truncated SVD of M by block one-sided Jacobi in float64.
//
// The paper decomposes the merged two-site tensor with a Jacobi SVD on the
// GPU (Sec. IV.A, cusolverDnZgesvdj).  Here the columns of X (X = M, or M^H
// when M is wide, with J accumulating the left vectors) are split into
// blocks of 32.  A sweep runs the round-robin tournament over the blocks; in
// one round every block is paired with one other block, and for every pair:
//
//   k_gram_mfma2, k_gram_cross : G = X_IJ^H X_IJ (64x64 Hermitian), split over
//                  row chunks; whole, or only the block between I and J;
//   k_eig, k_eig_full : G = V D V^H by cyclic two-sided Jacobi; a pair whose
//                  columns are already orthogonal to tolerance is left alone;
//   k_rot_cols, k_rot_mfma3 : X_IJ <- X_IJ V (and J_IJ <- J_IJ V).
//
// Matrices of up to 64 columns that fit in LDS take k_small instead.  All pairs
// of all gates of a batch run in the same launches.  The sweep ends the rounds;
// a gate converges after a sweep in which no pair rotated.  Then k_colnorm gives
// sigma_j^2 = ||x_j||^2 and k_trunc sorts them and applies the truncation rule.

#include <cfloat>

#include "tnsim_internal.h"
#include "tn_complex.h"
#include "tn_buffer.h"
#include "tn_lanes.h"
#include "tn_fast.h"

namespace tn {

// A column whose squared norm is below (rows * 2^-53)^2 ||X||_F^2 is rounding
// noise (far under the truncation's numerical-zero floor); pairs holding one
// are not rotated.
__device__ __forceinline__ double small_norm2(const GateDesc &d) {
  const double r = d.rows * 0x1p-53;
  return d.sc->fro2 * r * r;
}

// Round-robin tournament: pair k of round r over P players (P even).
__device__ __forceinline__ void rr_pair(int r, int k, int P, int &p, int &q) {
  if (k == 0) {
    p = P - 1;
    q = r;
  } else {
    p = (r + k) % (P - 1);
    q = (r - k + (P - 1)) % (P - 1);
  }
  if (p > q) {
    int t = p;
    p = q;
    q = t;
  }
}

__device__ __forceinline__ int pair_col(int I, int J, int p) {
  return p < BW ? I * BW + p : J * BW + (p - BW);
}

// A block pair that tested orthogonal and whose two blocks have not been
// rotated since has the same Gram matrix as then, so it would test orthogonal
// again: its Gram and pair solve are skipped (the result is unchanged).
__device__ __forceinline__ bool pair_known_orthogonal(const GateDesc &d, int I, int J) {
  if (!d.blkVer) return false;
  const int2 s = d.pairSeen[I * d.nblk + J];
  return s.x == d.blkVer[I] && s.y == d.blkVer[J];
}

// ---------------------------------------------------------------- setup

// Zero X's padding columns; J = identity (trans gates).
__global__ void k_setup_slots(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.y];
  if (d.small) return;
  int col = blockIdx.x;
  if (col < d.colsPad && col >= d.cols) {
    for (int r = threadIdx.x; r < d.ldx; r += blockDim.x)
      d.X[(size_t)col * d.ldx + r] = make_double2(0.0, 0.0);
  }
  if (d.trans && col < d.colsPad) {
    for (int r = threadIdx.x; r < d.ldj; r += blockDim.x)
      d.J[(size_t)col * d.ldj + r] = make_double2(r == col ? 1.0 : 0.0, 0.0);
  }
}

void launch_setup_slots(hipStream_t st, const GateDesc *d, int ng, int max_cols_pad, int) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_setup_slots, dim3(max_cols_pad, ng), dim3(256), 0, st, d);
}

// sigma_j^2 = ||x_j||^2, one wavefront per column.
__global__ __launch_bounds__(256) void k_colnorm(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.y];
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int col = blockIdx.x * 4 + wave;
  if (d.small || col >= d.colsPad) return;
  const double2 *x = d.X + (size_t)col * d.ldx;
  double s = 0.0;
  for (int r = lane; r < d.rows; r += 64) s += cabs2(x[r]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) d.sig2[col] = s;
}

void launch_colnorm(hipStream_t st, const GateDesc *d, int ng, int max_cols) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_colnorm, dim3((max_cols + 3) / 4, ng), dim3(256), 0, st, d);
}

// ||X||_F^2 in a fixed order; all gates start active; no block pair is known
// orthogonal yet.
__global__ void k_gate_init(const GateDesc *descs) {
  const GateDesc &d = descs[blockIdx.x];
  if (d.small) return;
  if (d.blkVer) {
    for (int b = threadIdx.x; b < d.nblk; b += blockDim.x) d.blkVer[b] = 0;
    for (int e = threadIdx.x; e < d.nblk * d.nblk; e += blockDim.x)
      d.pairSeen[e] = make_int2(-1, -1);
  }
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int j = 0; j < d.cols; j++) s += d.sig2[j];
    d.sc->fro2 = s;
    d.sc->rot = 1;
    d.sc->active = 1;
    d.sc->k = 0;
  }
}

void launch_gate_init(hipStream_t st, const GateDesc *d, int ng) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_gate_init, dim3(ng), dim3(64), 0, st, d);
}

// A gate keeps sweeping only if some pair rotated in the previous sweep.
__global__ void k_begin_sweep(const GateDesc *descs, int ng) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ng) return;
  SlotScalars *sc = descs[g].sc;
  sc->active = sc->rot;
  sc->rot = 0;
}

void launch_begin_sweep(hipStream_t st, const GateDesc *d, int ng) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_begin_sweep, dim3((ng + 63) / 64), dim3(64), 0, st, d, ng);
}

// ---------------------------------------------------------------- Gram of a column pair

typedef double d4_t __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4f64 operand layout (lane l = 0..63): A[l%16][l/16],
// B[l/16][l%16]; result entry v of lane l is D[l/16 + 4v][l%16] (rows
// strided by 4, unlike the float32 16x16 results).

__device__ __forceinline__ d4_t mfma64(double a, double b, d4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Pair Gram on float64 matrix cores (v_mfma_f64_16x16x4), without LDS
// staging.  G is Hermitian, so only its 10 upper 16x16 tiles are computed (the
// pair solve mirrors the lower triangle).  In one k-step (4 rows) lane l reads
// row 4 s + l/16 of the pair's columns 16 t + l%16 (t = 0..3): that is both
// the A operand (conjugated) and the B operand of v_mfma_f64_16x16x4 for
// every tile.  Each complex product conj(x) y takes three real products
// (Gauss): with x = a + ib, y = c + id, P1 = a c, P2 = b d,
// P3 = (a - b)(c + d), conj(x) y = (P1 + P2) + i (P3 - P1 + P2).  Waves 0
// and 1 compute tiles 0-4, which use all four column groups, waves 2 and 3
// tiles 5-9, which use groups 1-3 (15 MFMAs per k-step either way); the two
// waves of a set take alternate 16-row tiles, and their partial Grams are
// summed in LDS in a fixed order at the end.
constexpr int GT_A[10] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};
constexpr int GT_B[10] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};

template <int SET>
__device__ __forceinline__ void gram_tiles(BufRes rI, BufRes rJ, int ld, int rbeg, int rend,
                                           int half, int l16, int lg, d4_t (&p1)[5],
                                           d4_t (&p2)[5], d4_t (&p3)[5]) {
  constexpr int U0 = SET * 5, T0 = SET;  // tiles U0..U0+4 use column groups T0..3
  // loads of the 16-lane column groups T0..3 for one k-step (4 rows): buffer
  // loads (columns 16 t + l%16 of the pair, block I for t < 2), never
  // skipped (a row past the chunk reads what lies there, or zero past the
  // block, and is zeroed when used), so that the loads in flight are counted
  // exactly
  auto load_step = [&](double2 *x, int r) {
#pragma unroll
    for (int t = T0; t < 4; t++) x[t] = bload(t < 2 ? rI : rJ, (16 * (t & 1) + l16) * ld + r);
  };
  auto mfma_step = [&](const double2 *xin, int r) {
    // the step's own operands only: nothing of a later step is hoisted here
    // (its loads are still in flight)
    __builtin_amdgcn_sched_barrier(0);
    double2 x[4];
#pragma unroll
    for (int t = T0; t < 4; t++) x[t] = r < rend ? xin[t] : make_double2(0.0, 0.0);
    double dm[4], sp[4];  // a - b of the A operand, c + d of the B operand
#pragma unroll
    for (int t = T0; t < 4; t++) {
      dm[t] = x[t].x - x[t].y;
      sp[t] = x[t].x + x[t].y;
    }
#pragma unroll
    for (int u = 0; u < 5; u++) {
      const int ta = GT_A[U0 + u], tb = GT_B[U0 + u];
      const double2 a = x[ta], b = x[tb];  // G_pq += conj(x_rp) x_rq
      p1[u] = mfma64(a.x, b.x, p1[u]);
      p2[u] = mfma64(a.y, b.y, p2[u]);
      p3[u] = mfma64(dm[ta], sp[tb], p3[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the wavefront's k-steps: 16-row tiles base, base + 32, ... (the other
  // wavefront of the set takes the tiles in between), 4 steps per tile;
  // loads run three steps ahead of the products
  const int base = rbeg + half * 16;
  const int nstep = base < rend ? (rend - base + 31) / 32 * 4 : 0;
  auto row_of = [&](int n) { return base + 32 * (n >> 2) + 4 * (n & 3) + lg; };
  if (nstep == 0) return;
  double2 x0[4], x1[4], x2[4], x3[4];
  load_step(x0, row_of(0));
  load_step(x1, row_of(1));
  load_step(x2, row_of(2));
  for (int n = 0; n < nstep; n += 4) {
    load_step(x3, row_of(n + 3));
    mfma_step(x0, row_of(n));
    load_step(x0, row_of(n + 4));
    mfma_step(x1, row_of(n + 1));
    load_step(x1, row_of(n + 5));
    mfma_step(x2, row_of(n + 2));
    load_step(x2, row_of(n + 6));
    mfma_step(x3, row_of(n + 3));
  }
}

__global__ __launch_bounds__(256, 2) void k_gram_mfma2(const GateDesc *descs, int round,
                                                       int ksplit) {
  const GateDesc &d = descs[blockIdx.y];
  const int pairIdx = blockIdx.x / ksplit, kc = blockIdx.x % ksplit;
  if (!d.sc->active || round >= d.nblk - 1 || pairIdx >= d.nblk / 2) return;
  if (round > 0 && !d.fullOrder) return;  // k_gram_cross
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  if (pair_known_orthogonal(d, I, J)) return;
  int chunk = (d.rows + ksplit - 1) / ksplit;
  chunk = (chunk + 15) / 16 * 16;
  const int rbeg = kc * chunk;
  const int rend = min(d.rows, rbeg + chunk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int l16 = lane & 15, lg = lane >> 4;
  const int ld = d.ldx;
  const BufRes rI = make_res(d.X + (size_t)I * BW * ld, BW * ld);
  const BufRes rJ = make_res(d.X + (size_t)J * BW * ld, BW * ld);
  d4_t p1[5], p2[5], p3[5];
#pragma unroll
  for (int u = 0; u < 5; u++) {
    p1[u] = d4_t{0.0, 0.0, 0.0, 0.0};
    p2[u] = d4_t{0.0, 0.0, 0.0, 0.0};
    p3[u] = d4_t{0.0, 0.0, 0.0, 0.0};
  }
  const int set = wave >> 1, half = wave & 1;
  if (set == 0)
    gram_tiles<0>(rI, rJ, ld, rbeg, rend, half, l16, lg, p1, p2, p3);
  else
    gram_tiles<1>(rI, rJ, ld, rbeg, rend, half, l16, lg, p1, p2, p3);
  // sum of the two wavefronts of each set, the first one's partial first
  __shared__ double red[10][4][64][2];
  for (int h = 0; h < 2; h++) {
    if (half == h) {
#pragma unroll
      for (int u = 0; u < 5; u++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const double gr = p1[u][v] + p2[u][v], gi = p3[u][v] - p1[u][v] + p2[u][v];
          double *o = red[set * 5 + u][v][lane];
          if (h == 0) {
            o[0] = gr;
            o[1] = gi;
          } else {
            o[0] += gr;
            o[1] += gi;
          }
        }
    }
    __syncthreads();
  }
  if (tid == 0 && d.ctr && rend > rbeg) {
    atomicAdd(&d.ctr[CTR_GRAM_FLOP], 8ull * (rend - rbeg) * (PW * (PW + 1) / 2));
    atomicAdd(&d.ctr[CTR_GRAM_BYTE], 16ull * (rend - rbeg) * PW + 16ull * PW * PW);
  }
  double2 *G = d.Gp + ((size_t)kc * d.gpStride + pairIdx) * (PW * PW);
  for (int e = tid; e < 10 * 4 * 64; e += 256) {
    const int u = e / 256, v = (e / 64) % 4, l = e % 64;
    const int p = GT_A[u] * 16 + (l >> 4) + 4 * v, q = GT_B[u] * 16 + (l & 15);
    G[p * PW + q] = make_double2(red[u][v][l][0], red[u][v][l][1]);
  }
}

// The cross block G_IJ = X_I^H X_J alone (rounds after a sweep's first: the
// pair solves hand the blocks' own Grams on, see k_eig).  Four 16x16 tiles,
// (column groups 0, 1 of block I) x (2, 3: block J); every wavefront holds
// all four and takes each fourth 16-row tile, so that a k-step's four loads
// feed twelve MFMAs; the four partials are added in LDS in a fixed order.
// Reading X bounds it: 16 x 64 bytes per row against 12 MFMAs per 4 rows,
// so the loads run three k-steps ahead.
__global__ __launch_bounds__(256, 2) void k_gram_cross(const GateDesc *descs, int round,
                                                       int ksplit) {
  const GateDesc &d = descs[blockIdx.y];
  const int pairIdx = blockIdx.x / ksplit, kc = blockIdx.x % ksplit;
  if (d.fullOrder || !d.sc->active || round >= d.nblk - 1 || pairIdx >= d.nblk / 2) return;
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  if (pair_known_orthogonal(d, I, J)) return;
  int chunk = (d.rows + ksplit - 1) / ksplit;
  chunk = (chunk + 15) / 16 * 16;
  const int rbeg = kc * chunk;
  const int rend = min(d.rows, rbeg + chunk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int l16 = lane & 15, lg = lane >> 4;
  const int ld = d.ldx;
  const BufRes rI = make_res(d.X + (size_t)I * BW * ld, BW * ld);
  const BufRes rJ = make_res(d.X + (size_t)J * BW * ld, BW * ld);
  d4_t p1[4], p2[4], p3[4];  // tile u: column groups (u >> 1, 2 + (u & 1))
#pragma unroll
  for (int u = 0; u < 4; u++) {
    p1[u] = d4_t{0.0, 0.0, 0.0, 0.0};
    p2[u] = d4_t{0.0, 0.0, 0.0, 0.0};
    p3[u] = d4_t{0.0, 0.0, 0.0, 0.0};
  }
  auto load_step = [&](double2 *x, int r) {
#pragma unroll
    for (int t = 0; t < 4; t++) x[t] = bload(t < 2 ? rI : rJ, (16 * (t & 1) + l16) * ld + r);
  };
  auto mfma_step = [&](const double2 *xin, int r) {
    __builtin_amdgcn_sched_barrier(0);  // later steps' loads stay in flight
    double2 x[4];
#pragma unroll
    for (int t = 0; t < 4; t++) x[t] = r < rend ? xin[t] : make_double2(0.0, 0.0);
    double dm[2], sp[2];  // a - b of the A operands, c + d of the B operands
#pragma unroll
    for (int t = 0; t < 2; t++) {
      dm[t] = x[t].x - x[t].y;
      sp[t] = x[2 + t].x + x[2 + t].y;
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const double2 a = x[u >> 1], b = x[2 + (u & 1)];
      p1[u] = mfma64(a.x, b.x, p1[u]);
      p2[u] = mfma64(a.y, b.y, p2[u]);
      p3[u] = mfma64(dm[u >> 1], sp[u & 1], p3[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int base = rbeg + wave * 16;
  const int nstep = base < rend ? (rend - base + 63) / 64 * 4 : 0;
  auto row_of = [&](int n) { return base + 64 * (n >> 2) + 4 * (n & 3) + lg; };
  if (nstep) {
    double2 x0[4], x1[4], x2[4], x3[4];
    load_step(x0, row_of(0));
    load_step(x1, row_of(1));
    load_step(x2, row_of(2));
    for (int n = 0; n < nstep; n += 4) {
      load_step(x3, row_of(n + 3));
      mfma_step(x0, row_of(n));
      load_step(x0, row_of(n + 4));
      mfma_step(x1, row_of(n + 1));
      load_step(x1, row_of(n + 5));
      mfma_step(x2, row_of(n + 2));
      load_step(x2, row_of(n + 6));
      mfma_step(x3, row_of(n + 3));
    }
  }
  __shared__ double2 red[4][4][64];
  for (int w = 0; w < 4; w++) {
    if (wave == w) {
#pragma unroll
      for (int u = 0; u < 4; u++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
          const double gr = p1[u][v] + p2[u][v], gi = p3[u][v] - p1[u][v] + p2[u][v];
          double2 *o = &red[u][v][lane];
          *o = w == 0 ? make_double2(gr, gi) : make_double2(o->x + gr, o->y + gi);
        }
    }
    __syncthreads();
  }
  if (tid == 0 && d.ctr && rend > rbeg) {
    atomicAdd(&d.ctr[CTR_GRAM_FLOP], 8ull * (rend - rbeg) * (BW * BW));
    atomicAdd(&d.ctr[CTR_GRAM_BYTE], 16ull * (rend - rbeg) * PW + 16ull * BW * BW);
  }
  double2 *G = d.Gp + ((size_t)kc * d.gpStride + pairIdx) * (PW * PW);
  for (int e = tid; e < BW * BW; e += 256) {
    const int p = e / BW, q = e % BW;  // tile entry v of lane l: row l / 16 + 4 v, column l % 16
    const int u = (p >> 4) * 2 + (q >> 4), v = (p & 15) >> 2, l = (p & 3) * 16 + (q & 15);
    G[p * PW + BW + q] = red[u][v][l];
  }
}

// ---------------------------------------------------------------- 64x64 Hermitian Jacobi

constexpr int LDG = PW + 1;

// The upper triangle of a pair's Gram, put(r, c, G(r, c)) for r <= c, by
// THREADS threads.  In a sweep's first round everything comes from the Gram
// partials; later only the cross block does, and the blocks' own Grams are as
// their last pair solves left them (a sweep that rotates nothing has seen all
// of them computed afresh, so convergence is decided on fresh Grams).  Four
// entries at a time, so that the loads of the K-split's partials overlap (one
// entry at a time, 16 partials took longer than the solve's rounds).
template <int THREADS, class F>
__device__ __forceinline__ void pair_gram(const GateDesc &d, int I, int J, int round, int pairIdx,
                                          int ksplit, F put) {
  const int tid = threadIdx.x;
  const size_t step = (size_t)d.gpStride * (PW * PW);
  const double2 *G = d.Gp + (size_t)pairIdx * (PW * PW);
  auto sums = [&](const int (&o)[4], double2 (&x)[4]) {
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = G[o[k]];
#pragma unroll 4
    for (int kc = 1; kc < ksplit; kc++)
#pragma unroll
      for (int k = 0; k < 4; k++) x[k] = cadd(x[k], G[kc * step + o[k]]);
  };
  if (round == 0) {
    for (int e0 = tid; e0 < PW * PW; e0 += 4 * THREADS) {
      int o[4];
      double2 x[4];
#pragma unroll
      for (int k = 0; k < 4; k++) {  // entries below the diagonal: any other is read and dropped
        const int e = e0 + k * THREADS;
        o[k] = e / PW <= e % PW ? e : 0;
      }
      sums(o, x);
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int e = e0 + k * THREADS;
        if (e / PW <= e % PW) put(e / PW, e % PW, x[k]);
      }
    }
    return;
  }
  static_assert(BW * BW % THREADS == 0 && PW * PW % (4 * THREADS) == 0, "whole entries per thread");
  constexpr int CE = BW * BW / THREADS;  // entries of a 32x32 block per thread
  double2 dI[CE], dJ[CE];
#pragma unroll
  for (int k = 0; k < CE; k++) {
    const int e = tid + k * THREADS, o = e / BW * PW + e % BW;
    dI[k] = d.Dg[(size_t)I * (PW * PW) + o];
    dJ[k] = d.Dg[(size_t)J * (PW * PW) + o];
  }
  int o[4];
  double2 x[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int e = tid + (k % CE) * THREADS;
    o[k] = e / BW * PW + BW + e % BW;
  }
  sums(o, x);
#pragma unroll
  for (int k = 0; k < CE; k++) {
    const int e = tid + k * THREADS, r = e / BW, c = e % BW;
    put(r, BW + c, x[k]);
    if (r <= c) {
      put(r, c, dI[k]);
      put(BW + r, BW + c, dJ[k]);
    }
  }
}

// Pair solve: cyclic two-sided Jacobi on the pair Gram G (64x64 Hermitian)
// with the rotations accumulated in V.
//
// Passes.  A pass takes one bit b of the column number and pairs every column
// x whose bit b is 0 (32 of them, the p columns) with every column whose bit b
// is 1 (the q columns): two half-passes (v = 0, 1) of 16 rounds, each round 32
// disjoint rotations.  Slot s = 16 g + l (g = 0, 1; l = 0 .. 15) holds the
// p column with index 16 g + l, and in round r the q column with index
// 16 (g ^ v) + (l + r) mod 16 (indices count the columns with that bit).  Bit
// 5 pairs block I with block J; bits 4 .. 0 pair columns inside each block.
// Every solve makes the pass of bit 5.  The passes inside the blocks are
// spread over a sweep: one of them in every fourth round of the tournament,
// or, when the sweep has few rounds, several in one round, so that each pair
// of columns meets at least once per sweep.  Measured sweep counts on the
// merged matrices equal those of a solve that takes all 2016 pairs every time
// (N = 128, 256, 512: 7, 8, 9), at 1.25 passes of 32 rounds instead of 63.
//
// Layout.  G's off-diagonal 2x2 blocks (p, q of slot i) x (p, q of slot j)
// lie in the registers of wavefronts 0 .. 3, two per thread: inside a group of
// 16 slots the block (l, l + delta) for delta = 1 .. 8 (delta = 8 twice, as
// each other's adjoint), across the groups (slot l, slot 16 + l + delta) for
// delta = 0 .. 15; lane l of a row of 16 lanes holds slot l's, a row holds two
// neighbouring deltas.  Between rounds the q columns move on by one slot, so
// with entries a = G(p_i, p_j), b = G(p_i, q_j), c = G(q_i, p_j),
// e = G(q_i, q_j): a stays, b comes from delta + 1, c from lane l + 1 and
// delta - 1, e from lane l + 1.  Those are register moves and row rotations
// (DPP); only one b and one c per thread cross rows, through LDS.  V is in the
// registers of wavefronts 4 .. 7, EIG_VROWS rows of one slot's two columns per
// thread.  LDS carries the rotation parameters, the row crossings, and G
// between half-passes (upper triangle, 32 KB).
//
// Rotations without square-root scaling: with V = V~ S and G = S G~ S, S
// diagonal, x_p' = x_p - alpha x_q and x_q' = x_q + beta x_p (unscaled
// columns), 4 multiply-adds per complex entry instead of 6; the squared
// scales s^2 <- s^2 cos^2 (cos^2 >= 1/2) are multiplied in after 16 rounds.
// The threads that hold delta = 1 hold the next round's couplings
// b = G(p_l, q_{l+1}), so they compute the next rotations as soon as their
// first block is updated, while the other wavefronts update the rest: one
// barrier a round.
//
// A solve whose couplings all pass the test returns before the first pass.
// Bound by the chain of a round (parameters through LDS, first block, next
// parameters, barrier: about 2000 clocks with rotations, 700 without), not by
// the vector units, so G and V go to wavefronts of their own: one wavefront of
// each per SIMD in place of one that does both in turn, and a V wavefront
// never waits for the parameters.  The relayouts between half-passes cost 8000
// clocks each; with 162 registers (one workgroup per CU) they do not spill, with
// 128 (two) they do, which is worth it only when every CU has two (EIG_PACKED).
// Per launch, 256 threads that hold both / 512 with 128 registers / with 162:
// chi 300 (10 pairs) 41.5 / 34.8 / 31.5 us, chi 128 (layers of 4 .. 56 pairs)
// 57 / 48.1 / 43.5, chi 1024 (288 .. 384 pairs at once) 46.2 / 45.8 / 40.9;
// 1600 pairs at once (two layers of a 100-qubit circuit) - / 219 / 257 ms.
constexpr int EIG_THREADS = 512;  // wavefronts 0 .. 3 hold G, 4 .. 7 hold V
// solves in a launch from which two workgroups share a CU (256 CUs)
constexpr int EIG_PACKED = 512;
constexpr int EIG_ROWS = 16;      // rows of 16 lanes that hold G
constexpr int EIG_VROWS = PW / 8; // rows of V held by each half-wavefront
constexpr int EIG_EVERY = 4;  // tournament rounds between passes inside the blocks
constexpr int EIG_UPPER = PW / 2 * (PW + 1);

// Bits of the passes a solve makes in a round of a sweep of nr >= 3 rounds.
__device__ __forceinline__ int eig_bits(int round, int nr) {
  int bits = 32;
  if (round % EIG_EVERY == 0) {
    const int k = round / EIG_EVERY, ns = (nr + EIG_EVERY - 1) / EIG_EVERY;
    for (int t = 0; t < 5; t++)
      if (ns >= 5 ? t == k % 5 : t % ns == k) bits |= 16 >> t;
  }
  return bits;
}

// x with bit value v inserted at position b; x without bit b.
__device__ __forceinline__ int bit_ins(int x, int b, int v) {
  return ((x >> b) << (b + 1)) | (v << b) | (x & ((1 << b) - 1));
}
__device__ __forceinline__ int bit_del(int x, int b) {
  return ((x >> (b + 1)) << b) | (x & ((1 << b) - 1));
}

// Place of entry (a, b), a < b, of the strict upper triangle: the rows from 32
// on turned round into the free halves of rows 31 .. 0.
__device__ __forceinline__ int gpack(int a, int b) {
  const int m = a & (PW / 2) ? PW - 1 : 0;
  return (a ^ m) * (PW + 1) + (b ^ m);
}

__device__ __forceinline__ double2 gget(const double2 *Gs, int a, int b) {
  const double2 x = Gs[gpack(min(a, b), max(a, b))];
  return make_double2(x.x, a < b ? x.y : -x.y);
}
__device__ __forceinline__ void gput(double2 *Gs, int a, int b, double2 x) {
  Gs[gpack(min(a, b), max(a, b))] = make_double2(x.x, a < b ? x.y : -x.y);
}

// x - a y and x + a y
__device__ __forceinline__ double2 cfms(double2 x, double2 a, double2 y) {
  return make_double2(fma(a.y, y.y, fma(-a.x, y.x, x.x)), fma(-a.y, y.x, fma(-a.x, y.y, x.y)));
}
__device__ __forceinline__ double2 cfmad(double2 x, double2 a, double2 y) {
  return make_double2(fma(-a.y, y.y, fma(a.x, y.x, x.x)), fma(a.y, y.x, fma(a.x, y.y, x.y)));
}

// One 2x2 block of G between two slots.
struct GBlk {
  double2 a, b, c, e;
};

// B <- R_i^H B R_j with R = [[1, beta], [-alpha, 1]].
__device__ __forceinline__ void blk_rotate(GBlk &B, double2 ali, double2 bei, double2 alj,
                                           double2 bej) {
  const double2 a = cfms(B.a, alj, B.b), b = cfmad(B.b, bej, B.a);
  const double2 c = cfms(B.c, alj, B.e), e = cfmad(B.e, bej, B.c);
  const double2 ai = cconj(ali), bi = cconj(bei);
  B.a = cfms(a, ai, c);
  B.c = cfmad(c, bi, a);
  B.b = cfms(b, ai, e);
  B.e = cfmad(e, bi, b);
}

struct EigShared {
  double2 Gs[EIG_UPPER];        // strict upper triangle of G, between half-passes
  double dg[PW];                // diagonal of G
  double sca[2][PW / 2];        // scales of the p and q columns of each slot
  double2 prm[2][2][PW / 2];    // alpha, beta of each slot, by round parity
  double2 xb[2][EIG_ROWS][16];  // b entries that cross rows, by round parity
  double2 xc[2][EIG_ROWS][16];  // c entries
  int anyr[2];                  // some rotation in the round held by that buffer
  int sweep_rot;                // some rotation in the current inner sweep
};

// A solve's walk over its half-passes; the wavefronts that hold G and those
// that hold V take the same steps and meet the same barriers.
struct EigWalk {
  int b, v;  // bit and half of the current half-pass
  int t;
  __device__ __forceinline__ bool next(int bits) {  // bits 4 .. 0, then 5; two halves each
    while (++t < 12) {
      b = t < 10 ? 4 - (t >> 1) : 5;
      v = t & 1;
      if ((bits >> b) & 1) return true;
    }
    return false;
  }
};

// Wavefronts 0 .. 3: G's blocks and, in the first one (W0), the rotations.
template <bool W0>
__device__ __forceinline__ int eig_solve_g(const GateDesc &d, EigShared &S, int bits, double tol2,
                                           double small, unsigned &nrot) {
  const int tid = threadIdx.x;
  const int l = tid & 15, rho = tid >> 4, gpar = rho & 1, u = rho >> 1;
  const bool intra = u < 4;        // wavefronts 0, 1; the others: across the groups
  const bool param = W0 && u == 0; // delta = 1: holds the next couplings
  const int del = intra ? 2 * u + 1 : 2 * (rho - 8);  // first of this thread's two deltas
  // slots of this thread's blocks: si x sj0, si x sj1
  const int si = intra ? 16 * gpar + l : l;
  const int gj = intra ? 16 * gpar : 16;
  const int sj0 = gj + ((l + del) & 15), sj1 = gj + ((l + del + 1) & 15);
  // rows that b and c come from (the rows of delta + 2 and delta - 2)
  const int rb = intra ? (u < 3 ? rho + 2 : rho) : 8 + ((rho - 7) & 7);
  const int rc = intra ? (u > 0 ? rho - 2 : rho) : 8 + ((rho - 1) & 7);
  int first_rot = 0;
  for (int sweep = 0; sweep < d.innerSweeps; sweep++) {
    if (tid == 0) S.sweep_rot = 0;
    EigWalk at{0, 0, -1};
    while (at.next(bits)) {
      const int b = at.b, vx = at.v << 4;
      const int pi = bit_ins(si, b, 0), qi = bit_ins(si ^ vx, b, 1);
      const int pj0 = bit_ins(sj0, b, 0), qj0 = bit_ins(sj0 ^ vx, b, 1);
      const int pj1 = bit_ins(sj1, b, 0), qj1 = bit_ins(sj1 ^ vx, b, 1);
      GBlk B0, B1;
      B0.a = gget(S.Gs, pi, pj0);
      B0.b = gget(S.Gs, pi, qj0);
      B0.c = gget(S.Gs, qi, pj0);
      B0.e = gget(S.Gs, qi, qj0);
      B1.a = gget(S.Gs, pi, pj1);
      B1.b = gget(S.Gs, pi, qj1);
      B1.c = gget(S.Gs, qi, pj1);
      B1.e = gget(S.Gs, qi, qj1);
      // parameter threads (slot si): diagonal entries, squared scales, the
      // coupling of the slot's pair, and what it is after its rotation
      double dp = 0.0, dq = 0.0, s2p = 1.0, s2q = 1.0;
      double2 gc = make_double2(0.0, 0.0), gres = gc;
      if (param) {
        dp = S.dg[pi];
        dq = S.dg[qi];
        gc = gget(S.Gs, pi, qi);
      }
      // Rotations into buffer w.  With true diagonal entries x, y, coupling
      // g = s_p s_q g~, h = |g|^2 and delta = y - x, the rotation that zeroes
      // g has w = 2 sign(delta) / (|delta| + sqrt(delta^2 + 4h)), tangent
      // w |g|, cos^2 = 1 / (1 + w^2 h); the new diagonal is (x - w h,
      // y + w h).  On the unscaled columns alpha = w conj(g~) s_q^2, beta =
      // w g~ s_p^2.  The whole first wavefront computes and the parameter
      // threads' results count, without branches per thread, so that the
      // chain overlaps the update of the second block; a round in which no
      // coupling acts leaves after the test (three rounds of four are so).
      auto params = [&](int w, bool live) {
        const double h = s2p * s2q * cabs2(gc);
        const bool act = live && param && dp > small && dq > small && h > tol2 * dp * dq;
        const unsigned long long m = __ballot(act);
        if (tid == 0) S.anyr[w] = m != 0ull;
        gres = gc;
        if (!m) return;
        if (tid == 0) S.sweep_rot = 1;
        const double delta = dq - dp, s2 = fma(delta, delta, 4.0 * h);
        // (an infinite s2 gives no rotation, as 2 / inf does, and so E_NOCONV)
        const double tw = copysign(
            s2 <= DBL_MAX ? 2.0 * fast_rcp(fabs(delta) + fast_sqrt(s2)) : 0.0, delta);
        const double wq = act ? tw * s2q : 0.0, wp = act ? tw * s2p : 0.0;
        if (param) {
          S.prm[w][0][si] = make_double2(wq * gc.x, -wq * gc.y);
          S.prm[w][1][si] = make_double2(wp * gc.x, wp * gc.y);
        }
        const double wh = tw * h, c2 = fast_rcp(fma(tw, wh, 1.0));
        gres = act ? make_double2(0.0, 0.0) : gc;
        dp = act ? dp - wh : dp;
        dq = act ? dq + wh : dq;
        s2p = act ? s2p * c2 : s2p;
        s2q = act ? s2q * c2 : s2q;
        nrot += act;
      };
      if (W0) params(0, true);
      __syncthreads();
#pragma nounroll
      for (int r = 0; r < 16; r++) {
        const int w = r & 1;
        double2 cg = make_double2(0.0, 0.0);
        if (S.anyr[w]) {
          const double2 ali = S.prm[w][0][si], bei = S.prm[w][1][si];
          const double2 al0 = S.prm[w][0][sj0], be0 = S.prm[w][1][sj0];
          const double2 al1 = S.prm[w][0][sj1], be1 = S.prm[w][1][sj1];
          blk_rotate(B0, ali, bei, al0, be0);
          S.xb[w][rho][l] = B0.b;
          if (W0) {  // next round's couplings and q columns
            cg = cconj(row_next<1>(gres));
            gc = B0.b;
            dq = row_next<1>(dq);
            s2q = row_next<1>(s2q);
            params(w ^ 1, r < 15);
          }
          blk_rotate(B1, ali, bei, al1, be1);
          S.xc[w][rho][l] = B1.c;
        } else {
          S.xb[w][rho][l] = B0.b;
          S.xc[w][rho][l] = B1.c;
          if (W0) {
            cg = cconj(row_next<1>(gres));
            gc = B0.b;
            dq = row_next<1>(dq);
            s2q = row_next<1>(s2q);
            params(w ^ 1, r < 15);
          }
        }
        // the q columns move on by one slot
        const double2 c8 = cconj(row_next<9>(B0.c));  // delta = 8: b from the adjoint of c at 7
        const double2 c1 = row_next<1>(B0.c);
        B0.b = B1.b;
        B1.c = c1;
        B0.e = row_next<1>(B0.e);
        B1.e = row_next<1>(B1.e);
        __syncthreads();
        B1.b = S.xb[w][rb][l];
        B0.c = S.xc[w][rc][(l + 1) & 15];
        if (intra && u == 3) B1.b = c8;
        if (param) B0.c = cg;
      }
      // back to LDS with the scales multiplied in
      if (param) {
        const double fp = fast_sqrt(s2p), fq = fast_sqrt(s2q);
        S.sca[0][si] = fp;
        S.sca[1][si] = fq;
        S.dg[pi] = dp;
        S.dg[qi] = dq;
        gput(S.Gs, pi, qi, cscale(gc, fp * fq));
      }
      __syncthreads();
      const double fpi = S.sca[0][si], fqi = S.sca[1][si];
      {
        const double fp = S.sca[0][sj0], fq = S.sca[1][sj0];
        gput(S.Gs, pi, pj0, cscale(B0.a, fpi * fp));
        gput(S.Gs, pi, qj0, cscale(B0.b, fpi * fq));
        gput(S.Gs, qi, pj0, cscale(B0.c, fqi * fp));
        gput(S.Gs, qi, qj0, cscale(B0.e, fqi * fq));
      }
      if (!(intra && u == 3 && l >= 8)) {  // delta = 8 is held twice
        const double fp = S.sca[0][sj1], fq = S.sca[1][sj1];
        gput(S.Gs, pi, pj1, cscale(B1.a, fpi * fp));
        gput(S.Gs, pi, qj1, cscale(B1.b, fpi * fq));
        gput(S.Gs, qi, pj1, cscale(B1.c, fqi * fp));
        gput(S.Gs, qi, qj1, cscale(B1.e, fqi * fq));
      }
      __syncthreads();
    }
    const int cont = S.sweep_rot;  // every thread reads before anyone clears it
    if (sweep == 0) first_rot = cont;
    __syncthreads();
    if (!cont) break;
  }
  return first_rot;
}

// Wavefronts 4 .. 7: V, EIG_VROWS rows of one slot's two columns per thread.
__device__ __forceinline__ int eig_solve_v(const GateDesc &d, EigShared &S, int bits, double2 *V) {
  const int lane = threadIdx.x & 63, sv = lane & 31;
  const int vrow0 = ((threadIdx.x >> 5) - 8) * EIG_VROWS;
  double2 vp[EIG_VROWS], vq[EIG_VROWS];
  int lb = __ffs(bits) - 1, lv = 0;  // labelling of V's columns (bit, half-pass): any to start
  {
    const int cp = bit_ins(sv, lb, 0), cq = bit_ins(sv, lb, 1);
#pragma unroll
    for (int h = 0; h < EIG_VROWS; h++) {
      vp[h] = make_double2(vrow0 + h == cp ? 1.0 : 0.0, 0.0);
      vq[h] = make_double2(vrow0 + h == cq ? 1.0 : 0.0, 0.0);
    }
  }
  int first_rot = 0;
  for (int sweep = 0; sweep < d.innerSweeps; sweep++) {
    EigWalk at{0, 0, -1};
    while (at.next(bits)) {
      const int b = at.b, v = at.v;
      // V's columns to this half-pass's slots
      if (b == lb) {
        if (v != lv) {
#pragma unroll
          for (int h = 0; h < EIG_VROWS; h++)
            vq[h] = swap_rows(vq[h]);
        }
      } else {
        const int cp = bit_ins(sv, b, 0), cq = bit_ins(sv ^ (v << 4), b, 1);
        const bool pq = (cp >> lb) & 1, qq = (cq >> lb) & 1;  // held as a q column until now
        const int ps = (lane & 32) | (bit_del(cp, lb) ^ (pq ? lv << 4 : 0));
        const int qs = (lane & 32) | (bit_del(cq, lb) ^ (qq ? lv << 4 : 0));
#pragma unroll
        for (int h = 0; h < EIG_VROWS; h++) {
          __builtin_amdgcn_sched_barrier(0);  // one row's permutes at a time (registers)
          const double px = __shfl(vp[h].x, ps, 64), py = __shfl(vp[h].y, ps, 64);
          const double qx = __shfl(vq[h].x, ps, 64), qy = __shfl(vq[h].y, ps, 64);
          const double rx = __shfl(vp[h].x, qs, 64), ry = __shfl(vp[h].y, qs, 64);
          const double tx = __shfl(vq[h].x, qs, 64), ty = __shfl(vq[h].y, qs, 64);
          vp[h] = make_double2(pq ? qx : px, pq ? qy : py);
          vq[h] = make_double2(qq ? tx : rx, qq ? ty : ry);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      lb = b;
      lv = v;
      __syncthreads();
#pragma nounroll
      for (int r = 0; r < 16; r++) {
        const int w = r & 1;
        if (S.anyr[w]) {
          const double2 al = S.prm[w][0][sv], be = S.prm[w][1][sv];
#pragma unroll
          for (int h = 0; h < EIG_VROWS; h++) {
            const double2 x = cfms(vp[h], al, vq[h]);
            vq[h] = cfmad(vq[h], be, vp[h]);
            vp[h] = x;
          }
        }
#pragma unroll
        for (int h = 0; h < EIG_VROWS; h++) vq[h] = row_next<1>(vq[h]);
        __syncthreads();
      }
      __syncthreads();  // the scales
      const double fp = S.sca[0][sv], fq = S.sca[1][sv];
#pragma unroll
      for (int h = 0; h < EIG_VROWS; h++) {
        vp[h] = cscale(vp[h], fp);
        vq[h] = cscale(vq[h], fq);
      }
      __syncthreads();
    }
    const int cont = S.sweep_rot;
    if (sweep == 0) first_rot = cont;
    __syncthreads();
    if (!cont) break;
  }
  if (first_rot) {
    const int cp = bit_ins(sv, lb, 0), cq = bit_ins(sv ^ (lv << 4), lb, 1);
#pragma unroll
    for (int h = 0; h < EIG_VROWS; h++) {
      V[(vrow0 + h) * PW + cp] = vp[h];
      V[(vrow0 + h) * PW + cq] = vq[h];
    }
  }
  return first_rot;
}

template <int WAVES>
__global__ __launch_bounds__(EIG_THREADS, WAVES) void k_eig(const GateDesc *descs, int round,
                                                        int ksplit) {
  const GateDesc &d = descs[blockIdx.y];
  const int pairIdx = blockIdx.x;
  if (d.fullOrder || !d.sc->active || round >= d.nblk - 1 || pairIdx >= d.nblk / 2) return;
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  if (pair_known_orthogonal(d, I, J)) {
    if (threadIdx.x == 0) d.pairFlag[pairIdx] = 0;
    return;
  }
  __shared__ EigShared S;
  const int tid = threadIdx.x;
  const double tol2 = d.tol * d.tol;
  const double small = small_norm2(d);
  unsigned nrot = 0;  // rotations computed by this thread (profiling)
  const int bits = eig_bits(round, d.nblk - 1);
  pair_gram<EIG_THREADS>(d, I, J, round, pairIdx, ksplit, [&](int r, int c, double2 x) {
    if (r < c)
      S.Gs[gpack(r, c)] = x;
    else
      S.dg[r] = x.x;
  });
  __syncthreads();
  // does any pair of this solve's passes need a rotation?
  int need = 0;
  for (int e = tid; e < PW * PW; e += EIG_THREADS) {
    const int r = e / PW, c = e % PW;
    if (r < c && ((r ^ c) & bits)) {
      const double a = S.dg[r], b = S.dg[c];
      need |= a > small && b > small && cabs2(S.Gs[gpack(r, c)]) > tol2 * a * b;
    }
  }
  int rotated = 0;
  if (__syncthreads_or(need)) {
    double2 *V = d.V + (size_t)pairIdx * (PW * PW);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave == 0)
      rotated = eig_solve_g<true>(d, S, bits, tol2, small, nrot);
    else if (wave < 4)
      rotated = eig_solve_g<false>(d, S, bits, tol2, small, nrot);
    else
      rotated = eig_solve_v(d, S, bits, V);
  }
  if (d.ctr && tid < 64) {
    // fold the per-thread counts of the first wavefront, one atomic per pair
    unsigned v = nrot;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (tid == 0 && v) atomicAdd(&d.ctr[CTR_EIG_ROT], (unsigned long long)v);
  }
  if (round == 0 || rotated) {  // the blocks' own Grams for the later rounds
    for (int e = tid; e < 2 * BW * BW; e += EIG_THREADS) {
      const int blk = e / (BW * BW), r = (e / BW) % BW, c = e % BW, o = blk * BW;
      if (r <= c)
        d.Dg[(size_t)(blk ? J : I) * (PW * PW) + r * PW + c] =
            r < c ? S.Gs[gpack(o + r, o + c)] : make_double2(S.dg[o + r], 0.0);
    }
  }
  if (tid == 0) {
    // An unrotated solve means the pair was already orthogonal.
    d.pairFlag[pairIdx] = rotated;
    if (rotated) atomicOr(&d.sc->rot, 1);
    if (d.blkVer) {  // only this workgroup touches blocks I and J during the round
      if (rotated) {
        d.blkVer[I] += 1;
        d.blkVer[J] += 1;
      } else {
        d.pairSeen[I * d.nblk + J] = make_int2(d.blkVer[I], d.blkVer[J]);
      }
    }
  }
}

constexpr int EIGF_THREADS = 512;  // 8 wavefronts
// rows of V held by each row of 16 lanes of the wavefronts 1, 2, 3, 5, 6, 7
constexpr int EIGF_VROWS = (PW + 23) / 24;
constexpr int EIGF_OFFD = (PW / 2) * (PW / 2 - 1) / 2;  // off-diagonal 2x2 blocks (i < j)

// Order of the 2016 column pairs of a pair solve (columns 0-31 from block I,
// 32-63 from block J).  Rounds 0-31 pair the blocks: slot k pairs column k
// with column 32 + (k + r) mod 32.  Rounds 32-62 pair columns inside each
// block by the circle method on 32 (round r' = r - 32; slots 0-15 block I,
// 16-31 block J, s = k mod 16): s = 0 pairs 31 with r', s >= 1 pairs
// (r' + s) mod 31 with (r' - s) mod 31.  After the first outer sweep a
// block's own columns enter a pair solve mutually orthogonal (its last pair
// solve made them so), so in the later sweeps the rounds inside the blocks
// often rotate nothing and cost only their rotation test.  Neighbouring
// slots hold neighbouring columns (distinct LDS banks of row * 65 + column).
__device__ __forceinline__ void eigf_pair(int r, int k, int &p, int &q) {
  constexpr int H = PW / 2;
  if (r < H) {
    p = k;
    q = H + ((k + r) & (H - 1));
    return;
  }
  const int rr = r - H, off = k >= H / 2 ? H : 0, s = k & (H / 2 - 1);
  if (s == 0) {
    p = H - 1;
    q = rr;
  } else {
    p = rr + s;
    if (p >= H - 1) p -= H - 1;
    q = rr - s;
    if (q < 0) q += H - 1;
  }
  p += off;
  q += off;
}

// Off-diagonal entry (a, b), a != b, of the Hermitian pair Gram: only the
// upper triangle is stored, entry (a, b) at min(a, b) * 65 + max(a, b).
__device__ __forceinline__ int gslot(int a, int b) { return a < b ? a * LDG + b : b * LDG + a; }

// Pair solve over all 2016 column pairs (gates with fullOrder set).
// Cyclic two-sided Jacobi on the pair Gram G (64x64 Hermitian, in LDS) with
// the rotations accumulated in V.  A round applies the 32 disjoint rotations
// of the tournament at once: G <- R^H G R, V <- V R.  G keeps its upper
// triangle only (the diagonal in a separate array): the 496 off-diagonal
// 2x2 blocks (rows of pair i x columns of pair j, i < j) are updated by one
// thread each, and the 2x2 diagonal block of a rotating pair takes its
// exact values (new diagonal entries, zero coupling) when the rotation is
// computed.  At most `inner_sweeps` sweeps; the outer sweeps finish what a
// capped inner solve leaves.
//
// V lies in registers, by slots of the tournament: a row of 16 lanes holds
// EIGF_VROWS rows of V, lane l the p and q columns of slots l and 16 + l.  The
// columns move between neighbouring slots from round to round, by row
// rotations (DPP): between the blocks slot k takes the q column of slot k + 1
// (mod 32); inside a block the columns r' + s move down and r' - s up by one
// slot around the fixed column 31.  So V needs no LDS, which holds G and the
// rotation parameters (69 KB).
//
// A round takes two barriers: G's blocks on all wavefronts, then the next
// rotations in the first one (into the other parameter buffer) while six
// others rotate V and move its columns; one if it rotates nothing.  The
// wavefronts 0 and 4, which share a SIMD, hold no rows of V, so that nothing
// delays the parameters' chain.  Bound by that chain (1200 of 3200 clocks a
// round) and by G's blocks through LDS (1300).  With eight wavefronts that
// took the partners' entries of V by lane permutes (LDS) after the parameters,
// a round was 4400 clocks: 124 -> 95 us for 64 pairs, one inner sweep; with V
// in wavefronts 4 .. 7 99 us, with V rotated beside G 104.  136 registers, one
// solve per CU: limited to 128 for two it spills, and batches of 60 to 500
// solves took 3 % longer; above EIG_PACKED two share a CU, as for k_eig (one
// layer of four 80-qubit handles at chi = 256, 1280 solves in a launch: 220 us
// a launch against 283 over its sweeps, 379 against 460 where all rotate).
template <int WAVES>
__global__ __launch_bounds__(EIGF_THREADS, WAVES) void k_eig_full(const GateDesc *descs, int round, int ksplit) {
  const GateDesc &d = descs[blockIdx.y];
  const int pairIdx = blockIdx.x;
  if (!d.fullOrder || !d.sc->active || round >= d.nblk - 1 || pairIdx >= d.nblk / 2)
    return;
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  if (pair_known_orthogonal(d, I, J)) {
    if (threadIdx.x == 0) d.pairFlag[pairIdx] = 0;
    return;
  }
  __shared__ double2 Gs[PW * LDG];
  __shared__ double dg[PW];           // diagonal of G
  __shared__ double rc[2][PW / 2];    // cos
  __shared__ double2 rse[2][PW / 2];  // s * e^{i phi}
  __shared__ int anyr[2];  // some rotation in the round held by that buffer
  __shared__ int sweep_rot, first_rot;
  const int tid = threadIdx.x;
  const double tol2 = d.tol * d.tol;
  const double small = small_norm2(d);
  unsigned nrot_local = 0;  // rotations applied by this thread (profiling)

  pair_gram<EIGF_THREADS>(d, I, J, 0, pairIdx, ksplit, [&](int r, int c, double2 x) {
    if (r < c)
      Gs[r * LDG + c] = x;
    else
      dg[r] = x.x;
  });
  // rows of V (those from PW on do not exist), P and Q columns of slots l + 16 u
  constexpr int H = PW / 2;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool hasV = wave & 3;
  const int l = tid & 15, vrow0 = (((tid >> 4) & 3) + 4 * (wave - 1 - (wave > 4))) * EIGF_VROWS;
  const bool at0 = l == 0, at15 = l == 15;
  double2 P[EIGF_VROWS][2], Q[EIGF_VROWS][2];
#pragma unroll
  for (int h = 0; h < EIGF_VROWS; h++)
#pragma unroll
    for (int u = 0; u < 2; u++) {
      P[h][u] = make_double2(vrow0 + h == l + 16 * u ? 1.0 : 0.0, 0.0);
      Q[h][u] = make_double2(vrow0 + h == H + l + 16 * u ? 1.0 : 0.0, 0.0);
    }
  if (tid == 0) first_rot = 0;
  __syncthreads();

  // Rotations of round r into buffer b, from the current G (first wavefront
  // only: lanes < 32 hold one pair each, the ballot gives the round's flag).
  // With delta = b - a and h = |g|^2 for the pair's 2x2 block [[a, g],
  // [conj g, b]], the rotation that zeroes g has tangent t = w |g|,
  // w = 2 sign(delta) / (|delta| + sqrt(delta^2 + 4h)), cosine
  // c = 1 / sqrt(1 + w^2 h), s e^{i phi} = c w g, and the new diagonal is
  // (a - w h, b + w h).  The pair's own block is set to those values here:
  // no other thread reads or writes it until the round is applied.
  auto params = [&](int r, int b) {
    int act = 0;
    if (tid < PW / 2) {
      int p, q;
      eigf_pair(r, tid, p, q);
      const double a = dg[p], bb = dg[q];
      const int gs = gslot(p, q);
      const double2 g = p < q ? Gs[gs] : cconj(Gs[gs]);
      const double h = cabs2(g);
      double c = 1.0;
      double2 se = make_double2(0.0, 0.0);
      if (a > small && bb > small && h > tol2 * a * bb) {
        act = 1;
        const double delta = bb - a;
        const double w = (delta >= 0.0 ? 2.0 : -2.0) / (fabs(delta) + sqrt(delta * delta + 4.0 * h));
        c = 1.0 / sqrt(1.0 + w * w * h);
        const double cw = c * w;
        se = make_double2(cw * g.x, cw * g.y);
        dg[p] = a - w * h;
        dg[q] = bb + w * h;
        Gs[gs] = make_double2(0.0, 0.0);
        nrot_local++;
      }
      rc[b][tid] = c;
      rse[b][tid] = se;
    }
    const unsigned long long m = __ballot(act);
    if (tid == 0) anyr[b] = m != 0ull;
  };

  // this thread's off-diagonal block: the upper triangle of 32 x 32 pair
  // indices folded into 16 rows of 31 (row a with row 31 - a)
  int bi = 0, bj = 1;
  if (tid < EIGF_OFFD) {
    const int a = tid / (H - 1), col = tid - (H - 1) * a;
    if (col < H - 1 - a) {
      bi = a;
      bj = a + 1 + col;
    } else {
      bi = H - 1 - a;
      bj = col + 1;
    }
  }
  // entry (x, y) of G at its place in the upper triangle; its value or, from
  // below the diagonal, the conjugate
  auto place = [](int x, int y) { return min(x, y) * LDG + max(x, y); };
  auto flip = [](double2 v, bool f) { return make_double2(v.x, f ? -v.y : v.y); };
  // R = [[c, s e^{i phi}], [-s e^{-i phi}, c]] on columns (p, q); block (row
  // pair i, column pair j): B <- R_i^H B R_j.  A pair that does not rotate has
  // c = 1, s = 0, which leaves its entries exactly as they are, so every block
  // is updated without branches.  The fused multiply-adds are written out:
  // what complex64 gates store depends on how these round.
  auto rotate_block = [&](int b, int o00, int o01, int o10, int o11, bool f00, bool f01, bool f10,
                          bool f11) {
    const double2 b00 = flip(Gs[o00], f00), b01 = flip(Gs[o01], f01), b10 = flip(Gs[o10], f10),
                  b11 = flip(Gs[o11], f11);
    double2 n00, n01, n10, n11;
    {  // columns: [x_p x_q] R_j
      const double c = rc[b][bj];
      const double2 e = rse[b][bj];
      n00.x = fma(b00.x, c, -fma(b01.x, e.x, b01.y * e.y));
      n00.y = fma(b00.y, c, -fma(b01.y, e.x, -(b01.x * e.y)));
      n01.x = fma(b01.x, c, fma(b00.x, e.x, -(b00.y * e.y)));
      n01.y = fma(b01.y, c, fma(b00.y, e.x, b00.x * e.y));
      n10.x = fma(b10.x, c, -fma(b11.x, e.x, b11.y * e.y));
      n10.y = fma(b10.y, c, -fma(b11.y, e.x, -(b11.x * e.y)));
      n11.x = fma(b11.x, c, fma(b10.x, e.x, -(b10.y * e.y)));
      n11.y = fma(b11.y, c, fma(b10.y, e.x, b10.x * e.y));
    }
    {  // rows: R_i^H [row_p; row_q]
      const double c = rc[b][bi];
      const double2 e = rse[b][bi];
      Gs[o00] = flip(make_double2(fma(c, n00.x, -fma(e.x, n10.x, -(e.y * n10.y))),
                                  fma(c, n00.y, -fma(e.x, n10.y, e.y * n10.x))), f00);
      Gs[o01] = flip(make_double2(fma(c, n01.x, -fma(e.x, n11.x, -(e.y * n11.y))),
                                  fma(c, n01.y, -fma(e.x, n11.y, e.y * n11.x))), f01);
      Gs[o10] = flip(make_double2(fma(c, n10.x, fma(e.x, n00.x, e.y * n00.y)),
                                  fma(c, n10.y, fma(e.x, n00.y, -(e.y * n00.x)))), f10);
      Gs[o11] = flip(make_double2(fma(c, n11.x, fma(e.x, n01.x, e.y * n01.y)),
                                  fma(c, n11.y, fma(e.x, n01.y, -(e.y * n01.x)))), f11);
    }
  };
  // V <- V R on this thread's slots: new x_p = c x_p - conj(e) x_q, new x_q =
  // e x_p + c x_q
  auto rotate_v = [&](int b) {
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const double c = rc[b][l + 16 * u];
      const double2 e = rse[b][l + 16 * u];
#pragma unroll
      for (int h = 0; h < EIGF_VROWS; h++) {
        const double2 x = P[h][u], y = Q[h][u];
        P[h][u] = make_double2(fma(c, x.x, fma(-e.x, y.x, -(e.y * y.y))),
                               fma(c, x.y, fma(e.y, y.x, -e.x * y.y)));
        Q[h][u] = make_double2(fma(c, y.x, fma(e.x, x.x, -(e.y * x.y))),
                               fma(c, y.y, fma(e.y, x.x, e.x * x.y)));
      }
    }
  };
  auto sel = [](bool c, double2 x, double2 y) {
    return make_double2(c ? x.x : y.x, c ? x.y : y.y);
  };

  for (int sweep = 0; sweep < d.innerSweeps; sweep++) {
    if (tid == 0) sweep_rot = 0;
    if (tid < 64) params(0, 0);
    __syncthreads();
#pragma nounroll
    for (int r = 0; r < H; r++) {  // between the blocks
      const int b = r & 1;
      const bool any = anyr[b] != 0;
      if (any) {
        if (tid < EIGF_OFFD) {
          const int qi = H + ((bi + r) & (H - 1)), qj = H + ((bj + r) & (H - 1));
          rotate_block(b, bi * LDG + bj, bi * LDG + qj, bj * LDG + qi, place(qi, qj), false, false,
                       true, qi > qj);
        }
        __syncthreads();  // G after round r
        if (tid == 0) sweep_rot = 1;
      }
      // (a round without rotations leaves G as it was, and the next rotations
      // go to the other buffer)
      if (tid < 64) params(r + 1, b ^ 1);
      if (hasV) {
        if (any) rotate_v(b);
#pragma unroll
        for (int h = 0; h < EIGF_VROWS; h++) {  // slot k takes the q column of slot k + 1
          const double2 x = row_next<1>(Q[h][0]), y = row_next<1>(Q[h][1]);
          Q[h][0] = sel(at15, y, x);
          Q[h][1] = sel(at15, x, y);
        }
      }
      __syncthreads();  // V after round r; rotations of round r + 1 ready
    }
    // P holds block I and Q block J again, column l + 16 u; to the slots of the
    // rounds inside the blocks (u = block, slot l): s = 0 pairs 31 with 0, s >= 1
    // pairs s with 31 - s
    if (hasV) {
#pragma unroll
      for (int h = 0; h < EIGF_VROWS; h++) {
        const double2 i0 = P[h][0], i1 = row_mirror(P[h][1]), j0 = Q[h][0],
                      j1 = row_mirror(Q[h][1]);
        P[h][0] = sel(at0, i1, i0);
        Q[h][0] = sel(at0, i0, i1);
        P[h][1] = sel(at0, j1, j0);
        Q[h][1] = sel(at0, j0, j1);
      }
    }
    // this thread's columns there, p and q of slot bi and of slot bj (slot 0's
    // p stays, the others move on by one modulo 31)
    const int si = bi & (H / 2 - 1), sj = bj & (H / 2 - 1);
    const int oi = bi & (H / 2) ? H : 0, oj = bj & (H / 2) ? H : 0;
    int ip = si ? si : H - 1, iq = si ? H - 1 - si : 0;
    int jp = sj ? sj : H - 1, jq = sj ? H - 1 - sj : 0;
    auto next = [](int x) { return x + 1 == H - 1 ? 0 : x + 1; };
#pragma nounroll
    for (int r = H; r < PW - 1; r++) {  // inside the blocks
      const int b = r & 1;
      const bool any = anyr[b] != 0;
      if (any) {
        if (tid < EIGF_OFFD) {
          const int pi = ip + oi, qi = iq + oi, pj = jp + oj, qj = jq + oj;
          rotate_block(b, place(pi, pj), place(pi, qj), place(qi, pj), place(qi, qj), pi > pj,
                       pi > qj, qi > pj, qi > qj);
        }
        __syncthreads();
        if (tid == 0) sweep_rot = 1;
      }
      ip = si ? next(ip) : ip;
      jp = sj ? next(jp) : jp;
      iq = next(iq);
      jq = next(jq);
      if (tid < 64 && r + 1 < PW - 1) params(r + 1, b ^ 1);
      if (hasV) {
        if (any) rotate_v(b);
        // p columns move down by one slot, q columns up, around slot 0's p
#pragma unroll
        for (int h = 0; h < EIGF_VROWS; h++)
#pragma unroll
          for (int u = 0; u < 2; u++) {
            const double2 x = row_next<1>(P[h][u]), y = row_next<15>(Q[h][u]);
            P[h][u] = sel(at0, P[h][u], sel(at15, Q[h][u], x));
            Q[h][u] = sel(at0, x, y);
          }
      }
      __syncthreads();
    }
    if (hasV) {
#pragma unroll
      for (int h = 0; h < EIGF_VROWS; h++) {  // and back
        const double2 i0 = sel(at0, Q[h][0], P[h][0]), i1 = sel(at0, P[h][0], Q[h][0]);
        const double2 j0 = sel(at0, Q[h][1], P[h][1]), j1 = sel(at0, P[h][1], Q[h][1]);
        P[h][0] = i0;
        P[h][1] = row_mirror(i1);
        Q[h][0] = j0;
        Q[h][1] = row_mirror(j1);
      }
    }
    const int cont = sweep_rot;  // every thread reads before anyone clears it
    if (sweep == 0 && tid == 0) first_rot = cont;
    __syncthreads();
    if (!cont) break;
  }
  if (d.ctr && tid < 64) {
    // fold the per-thread counts of the first wavefront, one atomic per pair
    unsigned v = nrot_local;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (tid == 0 && v) atomicAdd(&d.ctr[CTR_EIG_ROT], (unsigned long long)v);
  }
  // An unrotated first sweep means the pair was already orthogonal.
  if (tid == 0) {
    d.pairFlag[pairIdx] = first_rot;
    if (first_rot) atomicOr(&d.sc->rot, 1);
    if (d.blkVer) {  // only this workgroup touches blocks I and J during the round
      if (first_rot) {
        d.blkVer[I] += 1;
        d.blkVer[J] += 1;
      } else {
        d.pairSeen[I * d.nblk + J] = make_int2(d.blkVer[I], d.blkVer[J]);
      }
    }
  }
  if (first_rot) {
    double2 *V = d.V + (size_t)pairIdx * (PW * PW);
    if (hasV) {
#pragma unroll
      for (int h = 0; h < EIGF_VROWS; h++)
#pragma unroll
        for (int u = 0; u < 2; u++)
          if (vrow0 + h < PW) {
            V[(vrow0 + h) * PW + l + 16 * u] = P[h][u];
            V[(vrow0 + h) * PW + H + l + 16 * u] = Q[h][u];
          }
    }
  }
}

void launch_eig(hipStream_t st, const GateDesc *d, int ng, int round, int max_pairs, int ksplit,
                bool cross, bool full) {
  if (ng <= 0) return;
  const bool packed = (long long)max_pairs * ng > EIG_PACKED;
  if (cross)
    hipLaunchKernelGGL(packed ? k_eig<4> : k_eig<2>, dim3(max_pairs, ng), dim3(EIG_THREADS), 0, st,
                       d, round, ksplit);
  if (full)
    hipLaunchKernelGGL(packed ? k_eig_full<4> : k_eig_full<2>, dim3(max_pairs, ng),
                       dim3(EIGF_THREADS), 0, st, d, round, ksplit);
}

// ---------------------------------------------------------------- apply a pair rotation

// Pair rotation on float64 matrix cores, as the transposed product (X V)^T = V^T X^T, so that
// the X operand of v_mfma_f64_16x16x4 (B: 16 lanes = 16 consecutive rows of
// one column) and the result (16 lanes = 16 consecutive rows of one column)
// are both contiguous 256-byte segments.  A wavefront owns whole 16-row tiles
// (all 64 columns), so it overwrites exactly the rows it read and needs no
// barrier; two workgroups per CU hide the load latency.  Each complex product
// takes three real products (Gauss): with v = a + ib and x = c + id,
// P1 = a c, P2 = b d, P3 = (a + b)(c + d), v x = (P1 - P2) + i (P3 - P1 - P2).
__global__ __launch_bounds__(256, 2) void k_rot_mfma3(const GateDesc *descs, int round) {
  const GateDesc &d = descs[blockIdx.y];
  if (!d.sc->active || round >= d.nblk - 1) return;
  const int npairs = d.nblk / 2;
  const int RRW = d.rotRows;
  const int xchunks = (d.rows + RRW - 1) / RRW;
  const int jchunks = d.trans ? (d.m + RRW - 1) / RRW : 0;
  const int per = xchunks + jchunks;
  const int pairIdx = blockIdx.x / per, chunk = blockIdx.x % per;
  if (pairIdx >= npairs) return;
  if (!d.pairFlag[pairIdx]) return;
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  double2 *base;
  int ld, nrows, r0;
  if (chunk < xchunks) {
    base = d.X;
    ld = d.ldx;
    nrows = d.rows;
    r0 = chunk * RRW;
  } else {
    base = d.J;
    ld = d.ldj;
    nrows = d.m;
    r0 = (chunk - xchunks) * RRW;
  }
  const int r1 = min(nrows, r0 + RRW);
  __shared__ double2 Vs[PW * LDG];  // [k][col]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int l16 = lane & 15, lg = lane >> 4;
  const double2 *V = d.V + (size_t)pairIdx * (PW * PW);
  for (int e = tid; e < PW * PW; e += 256) Vs[(e / PW) * LDG + e % PW] = V[e];
  if (tid == 0 && d.ctr) {
    unsigned long long nr = (unsigned long long)(r1 - r0);
    atomicAdd(&d.ctr[CTR_ROT_FLOP], 8ull * nr * PW * PW);
    atomicAdd(&d.ctr[CTR_ROT_BYTE], 32ull * nr * PW + 16ull * PW * PW);
  }
  __syncthreads();
  // The lane's column for k-step s is pair column 4 s + lg (block I for
  // s < 8).  Buffer loads and stores (one resource per block of 32 padded columns, a
  // 32-bit element offset per access): one register per address, counted
  // on the vector memory counter only.  Tile q of the wavefront covers rows
  // r0 + 16 (wave + 4 q) ..; a tile past the chunk uses an empty resource
  // (loads read zero, stores are dropped), so every wavefront runs an even
  // number of tiles with no branch around loads or stores, and the loads in
  // flight are counted exactly: the products of a tile wait only for that
  // tile's data while the next tile's block I is still on its way.  Columns
  // are padded to whole 16-row tiles and chunks are whole tiles, so rows
  // past the matrix land in the column's padding (never read).  (A wavefront
  // with an odd number of tiles leaves before the empty one's products.)
  const BufRes rI = make_res(base + (size_t)I * BW * ld, BW * ld);
  const BufRes rJ = make_res(base + (size_t)J * BW * ld, BW * ld);
  const BufRes rZ = make_res(base, 0);
  const int ntile = (r1 - r0 + 15) / 16;
  const int mytiles = wave < ntile ? (ntile - wave + 3) / 4 : 0;
  auto tile_row = [&](int q) { return r0 + 16 * (wave + 4 * q); };
  // k-steps 0..7 read block I, 8..15 block J
  auto load_half = [&](double2 *xv, int half, int q) {
    const int rt = tile_row(q);
    const BufRes r = rt < r1 ? (half ? rJ : rI) : rZ;
    const int lo = lg * ld + rt + l16;
#pragma unroll
    for (int s = 0; s < BW / 4; s++) xv[s] = bload(r, lo + 4 * s * ld);
  };
  // one 16-row tile: block I from xi, block J from xj
  auto tile = [&](const double2 *xi, const double2 *xj, int q) {
    d4_t p1[4], p2[4], p3[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      p1[t] = d4_t{0.0, 0.0, 0.0, 0.0};
      p2[t] = d4_t{0.0, 0.0, 0.0, 0.0};
      p3[t] = d4_t{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int s = 0; s < PW / 4; s++) {
      const double2 b = s < BW / 4 ? xi[s] : xj[s - BW / 4];  // X^T[k][row]
      const double bs = b.x + b.y;
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const double2 a = Vs[(4 * s + lg) * LDG + t * 16 + l16];  // V^T[col][k]
        p1[t] = mfma64(a.x, b.x, p1[t]);
        p2[t] = mfma64(a.y, b.y, p2[t]);
        p3[t] = mfma64(a.x + a.y, bs, p3[t]);
      }
      __builtin_amdgcn_sched_barrier(0);  // keep each step's V reads in that step
    }
    // Loads and stores share the vector memory counter, and a load issued
    // before a store can only be waited for with the store: so the next
    // tile's block I (issued at this tile's start, long arrived) is waited
    // for here, before this tile's stores.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    // output column t * 16 + lg + 4 v of the pair: block I for t < 2
    const int rt = tile_row(q);
    const bool live = rt < r1;
    const BufRes oI = live ? rI : rZ, oJ = live ? rJ : rZ;
    const int lo = lg * ld + rt + l16;
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
      for (int v = 0; v < 4; v++)
        bstore(t < 2 ? oI : oJ, lo + (16 * (t & 1) + 4 * v) * ld,
               make_double2(p1[t][v] - p2[t][v], p3[t][v] - p1[t][v] - p2[t][v]));
  };
  // Two block-I buffers take turns (no register copies between tiles).
  double2 xi0[BW / 4], xi1[BW / 4], xj[BW / 4];
  load_half(xi0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop starts with block I in hand
  for (int q = 0; q < mytiles; q += 2) {
    load_half(xj, 1, q);
    load_half(xi1, 0, q + 1);
    tile(xi0, xj, q);
    if (q + 1 >= mytiles) break;
    load_half(xj, 1, q + 1);
    load_half(xi0, 0, q + 2);
    tile(xi1, xj, q + 1);
  }
}

// The same rotation with the columns of the result split over the wavefronts:
// each computes 16 of the 64 columns of every tile of its workgroup, its
// columns of V in registers.  All four read a tile's X, so a barrier stands
// between reading and overwriting it.  The products and their order are those
// above, so the results are the same to the bit.
// A tile's 192 matrix instructions take one SIMD 12000 clocks (5 us), which a
// launch with fewer tiles than SIMDs cannot hide; here they take a quarter of
// that.  chi 90 (3 pairs x 12 tiles) 13.8 -> 5.3 us, chi 300 (10 x 38) 18.3 ->
// 9.5, chi 128 (up to 56 x 16) 25 -> 11.6, chi 256 in a batch of many gates 46 ->
// 45 us, bound by the matrix cores there.
__global__ __launch_bounds__(256, 2) void k_rot_cols(const GateDesc *descs, int round) {
  const GateDesc &d = descs[blockIdx.y];
  if (!d.sc->active || round >= d.nblk - 1) return;
  const int npairs = d.nblk / 2;
  const int RRW = d.rotRows;
  const int xchunks = (d.rows + RRW - 1) / RRW;
  const int jchunks = d.trans ? (d.m + RRW - 1) / RRW : 0;
  const int per = xchunks + jchunks;
  const int pairIdx = blockIdx.x / per, chunk = blockIdx.x % per;
  if (pairIdx >= npairs) return;
  if (!d.pairFlag[pairIdx]) return;
  int I, J;
  rr_pair(round, pairIdx, d.nblk, I, J);
  const bool inX = chunk < xchunks;
  double2 *base = inX ? d.X : d.J;
  const int ld = inX ? d.ldx : d.ldj, nrows = inX ? d.rows : d.m;
  const int r0 = (inX ? chunk : chunk - xchunks) * RRW;
  const int r1 = min(nrows, r0 + RRW);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (scalar)
  const int l16 = lane & 15, lg = lane >> 4;
  if (tid == 0 && d.ctr) {
    unsigned long long nr = (unsigned long long)(r1 - r0);
    atomicAdd(&d.ctr[CTR_ROT_FLOP], 8ull * nr * PW * PW);
    atomicAdd(&d.ctr[CTR_ROT_BYTE], 32ull * nr * PW + 16ull * PW * PW);
  }
  const BufRes rI = make_res(base + (size_t)I * BW * ld, BW * ld);
  const BufRes rJ = make_res(base + (size_t)J * BW * ld, BW * ld);
  const BufRes rZ = make_res(base, 0);
  const double2 *V = d.V + (size_t)pairIdx * (PW * PW) + lg * PW + 16 * wave + l16;
  double2 a[PW / 4], x0[PW / 4], x1[PW / 4];  // lane: column l16 of V, row l16 of X; k = 4 s + lg
  // a tile past the chunk reads zeros (and is not used)
  auto load = [&](double2 *x, int rt) {
    const BufRes bI = rt < r1 ? rI : rZ, bJ = rt < r1 ? rJ : rZ;
    const int lo = lg * ld + rt + l16;
#pragma unroll
    for (int s = 0; s < PW / 4; s++)
      x[s] = bload(s < BW / 4 ? bI : bJ, lo + 4 * (s % (BW / 4)) * ld);
  };
  auto tile = [&](const double2 *x, int rt) {
    d4_t p1{0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
#pragma unroll
    for (int s = 0; s < PW / 4; s++) {
      p1 = mfma64(a[s].x, x[s].x, p1);
      p2 = mfma64(a[s].y, x[s].y, p2);
      p3 = mfma64(a[s].x + a[s].y, x[s].x + x[s].y, p3);
    }
    __syncthreads();
    const BufRes out = wave < 2 ? rI : rJ;
    const int lo = (16 * (wave & 1) + lg) * ld + rt + l16;
#pragma unroll
    for (int v = 0; v < 4; v++)
      bstore(out, lo + 4 * v * ld,
             make_double2(p1[v] - p2[v], p3[v] - p1[v] - p2[v]));
  };
#pragma unroll
  for (int s = 0; s < PW / 4; s++) a[s] = V[4 * s * PW];
  load(x0, r0);
  for (int rt = r0; rt < r1; rt += 32) {
    load(x1, rt + 16);
    tile(x0, rt);
    if (rt + 16 >= r1) break;
    load(x0, rt + 32);
    tile(x1, rt + 16);
  }
}

void launch_gram(hipStream_t st, const GateDesc *d, int ng, int round, int max_pairs, int ksplit,
                 bool cross, bool full) {
  if (ng <= 0) return;
  if (round == 0 || full)
    hipLaunchKernelGGL(k_gram_mfma2, dim3(max_pairs * ksplit, ng), dim3(256), 0, st, d, round,
                       ksplit);
  if (round > 0 && cross)
    hipLaunchKernelGGL(k_gram_cross, dim3(max_pairs * ksplit, ng), dim3(256), 0, st, d, round,
                       ksplit);
}

// Copy every gate's scalars into one array (one device-to-host copy per sweep).
__global__ void k_gather_sc(const GateDesc *descs, int ng, SlotScalars *out) {
  int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < ng) out[g] = *descs[g].sc;
}

void launch_gather_sc(hipStream_t st, const GateDesc *d, int ng, SlotScalars *out) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_gather_sc, dim3((ng + 63) / 64), dim3(64), 0, st, d, ng, out);
}

void launch_rot(hipStream_t st, const GateDesc *d, int ng, int round, int max_pairs,
                int max_rows, int max_m, int rot_rows, bool cols) {
  if (ng <= 0) return;
  const int per = (max_rows + rot_rows - 1) / rot_rows + (max_m + rot_rows - 1) / rot_rows;
  if (cols)
    hipLaunchKernelGGL(k_rot_cols, dim3(max_pairs * per, ng), dim3(256), 0, st, d, round);
  else
    hipLaunchKernelGGL(k_rot_mfma3, dim3(max_pairs * per, ng), dim3(256), 0, st, d, round);
}

// ---------------------------------------------------------------- sort + truncate

constexpr int SORT_MAX = 4096;

// If some gate of the launch has not converged (k_small), none is cut: the
// call then fails and its sites and Schmidt weights keep their values.
__global__ __launch_bounds__(256) void k_trunc(const GateDesc *descs, int ng) {
  const GateDesc &d = descs[blockIdx.x];
  int failed = 0;
  for (int g = threadIdx.x; g < ng; g += 256) failed |= descs[g].small && descs[g].sc->rot;
  if (__syncthreads_or(failed)) return;
  __shared__ double key[SORT_MAX];
  __shared__ int idx[SORT_MAX];
  __shared__ double tail[SORT_MAX + 1];
  __shared__ int s_k;
  __shared__ double s_N;
  const int tid = threadIdx.x;
  int P = 1;
  while (P < d.cols) P <<= 1;
  for (int j = tid; j < P; j += 256) {
    key[j] = j < d.cols ? d.sig2[j] : -1.0;
    idx[j] = j;
  }
  __syncthreads();
  // bitonic sort: descending key, ascending index on ties
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int j = tid; j < P; j += 256) {
        int l = j ^ stride;
        if (l > j) {
          bool up = ((j & size) == 0);  // this block sorted "descending-first"
          double kj = key[j], kl = key[l];
          int ij = idx[j], il = idx[l];
          bool j_first = (kj > kl) || (kj == kl && ij < il);
          bool swap = up ? !j_first : j_first;
          if (swap) {
            key[j] = kl;
            key[l] = kj;
            idx[j] = il;
            idx[l] = ij;
          }
        }
      }
      __syncthreads();
    }
  }
  if (tid == 0) {
    const int cnt = d.cols;
    double W = 0.0;
    for (int j = 0; j < cnt; j++) W += key[j];
    double floor2 = (double)d.m * 0x1p-53 * key[0];
    int nz = 0;
    for (int j = 0; j < cnt; j++) nz += key[j] > floor2;
    if (nz < 1) nz = 1;
    tail[cnt] = 0.0;
    for (int k = cnt - 1; k >= 0; k--) tail[k] = tail[k + 1] + key[k];
    const double cutoff = d.cutoff;
    int kc = cnt;
    for (int k = 1; k <= cnt; k++)
      if (tail[k] <= cutoff * W) {
        kc = k;
        break;
      }
    int k = kc;
    if (k > nz) k = nz;
    if (k > d.chiMax) k = d.chiMax;
    if (k < 1) k = 1;
    double head = 0.0;
    for (int j = 0; j < k; j++) head += key[j];
    double N = sqrt(head);
    if (!(N > 0.0)) N = 1.0;
    d.sc->k = k;
    d.sc->N = N;
    d.sc->W = W;
    d.sc->eps = W > 0.0 ? tail[k] / W : 0.0;
    d.sc->nz = nz;
    d.dimsDev[d.i + 1] = k;
    s_k = k;
    s_N = N;
  }
  __syncthreads();
  for (int j = tid; j < s_k; j += 256) {
    d.lamOut[j] = sqrt(key[j]) / s_N;
    d.perm[j] = idx[j];
  }
}

void launch_trunc(hipStream_t st, const GateDesc *d, int ng) {
  if (ng <= 0) return;
  hipLaunchKernelGGL(k_trunc, dim3(ng), dim3(256), 0, st, d, ng);
}

}  // namespace tn
