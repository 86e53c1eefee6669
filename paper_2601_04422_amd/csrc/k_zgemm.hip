// Complex float64 GEMM on the FP64 matrix cores: C = op(A) B.
//
// A complex product is four real products (C_re += A_re B_re - A_im B_im,
// C_im += A_re B_im + A_im B_re), each a v_mfma_f64_16x16x4f64.  A workgroup
// computes a 32 x 32 tile of C, and its NW wavefronts split K between them,
// each with all 2 x 2 MFMA tiles.  Operands go from memory straight into the
// matrix-core layout (16 lanes along a row of B or along A's rows), two
// k-steps ahead of the products, so the K loop has no barrier; the NW partial
// tiles are added in LDS in wavefront order, so results do not depend on
// scheduling.  Operands are read in their storage precision (complex64 sites
// are widened on load); C is complex128.
//
// Why this split: with 64 x 64 tiles (16 or 32 of them at a bond of 256, each
// a chain of K / 16 staged steps of 2 us) most CUs stood idle.  Three
// expectations, an overlap, a norm and four amplitudes at chi = 500, n = 28:
// 35.5 -> 9.1 ms; 1000 shots at chi = 256, n = 48: 8.7 -> 3.85 ms.  Large
// products of the transfer chains gain nothing from larger tiles either (the
// four wavefronts' loads of a tile meet in L1 and L2): an expectation value at
// chi = 1024 5.8 -> 5.7 ms, at 2048 42.0 -> 41.3 (65 TFLOP/s), 2048 shots at 1024
// 8.5 -> 7.8.  Products over very many columns do: see k_zgemm_cols.
// Bound by the matrix cores: their rate when the chip is full, the chain of
// K / (4 NW) steps of 16 products when it is not.
#include <algorithm>

#include "tnsim_internal.h"
#include "tn_complex.h"

namespace tn {

typedef double zd4_t __attribute__((ext_vector_type(4)));

// lane l supplies A[l%16][l/16] and B[l/16][l%16]; entry v of the result is
// D[l/16 + 4v][l%16]
__device__ __forceinline__ zd4_t zmfma(double a, double b, zd4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int ZT = 32;

// AK: A(i,k) = A[i*sa + k], else A[k*sa + i]; AC: use conj(A).
// BK: B(k,j) = B[j*sb + k], else B[k*sb + j].
// CM: C(i,j) = C[j*sc + i], else C[i*sc + j].
// blockIdx.z: batch index.
// GA (gathered columns): output columns *g.clo .. *g.chi - 1 (device
// values; the grid covers at most N of them), column j reads column
// g.bmap[j] of B and is scaled by g.cscale[j]; tiles from column *g.asplit
// on read A + g.za.
template <class TA, class TB, bool AK, bool AC, bool BK, bool CM, bool GA, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_zgemm(ZgemmArgs g) {
  int N = g.N, j0 = blockIdx.x * ZT, A_off_tile = 0;
  if (GA) {
    const int lo = *g.clo;
    N = *g.chi;
    j0 += lo;
    if (g.asplit && j0 >= *g.asplit) A_off_tile = 1;
  } else if (g.mcount) {
    N = min(N, g.mult * *g.mcount);
  }
  const int i0 = blockIdx.y * ZT;
  if (j0 >= N) return;
  const int M = g.M, K = g.K, z = blockIdx.z;
  const TA *A = (const TA *)g.A + (z + A_off_tile) * g.za;
  const TB *B = (const TB *)g.B + z * g.zb;
  double2 *C = g.C + z * g.zc;
  const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, lg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  // this wavefront's part of K, in whole k-steps of 4
  const int kc = ((K + NW - 1) / NW + 3) / 4 * 4;
  const int kb = w * kc, ke = min(K, kb + kc);
  // rows of A and columns of B past the matrix repeat the last one (their
  // products are not stored)
  const TA *pa[2];
  const TB *pb[2];
#pragma unroll
  for (int x = 0; x < 2; x++) {
    const int gi = min(i0 + 16 * x + l16, M - 1);
    pa[x] = AK ? A + (long long)gi * g.sa : A + gi;
    const int gj = min(j0 + 16 * x + l16, N - 1);
    const long long bj = GA ? (long long)g.bmap[gj] : gj;
    pb[x] = BK ? B + bj * g.sb : B + bj;
  }
  constexpr int D = 2;  // k-steps loaded together (32 products, longer than a load from L2)
  double2 a[2][D][2], b[2][D][2];
  auto load = [&](int k0, double2 (&ra)[D][2], double2 (&rb)[D][2]) {
#pragma unroll
    for (int s = 0; s < D; s++) {
      const int k = k0 + 4 * s + lg;
      const long long kk = min(k, K - 1);
      const bool in = k < ke;
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const double2 va = cload(AK ? pa[x] + kk : pa[x] + kk * g.sa);
        const double2 vb = cload(BK ? pb[x] + kk : pb[x] + kk * g.sb);
        ra[s][x] = in ? va : make_double2(0.0, 0.0);
        rb[s][x] = in ? vb : make_double2(0.0, 0.0);
      }
    }
  };
  zd4_t cr[2][2], ci[2][2];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++) {
      cr[x][y] = zd4_t{0.0, 0.0, 0.0, 0.0};
      ci[x][y] = zd4_t{0.0, 0.0, 0.0, 0.0};
    }
  auto mul = [&](const double2 (&ra)[D][2], const double2 (&rb)[D][2]) {
#pragma unroll
    for (int s = 0; s < D; s++) {
      double2 av[2];
#pragma unroll
      for (int x = 0; x < 2; x++) av[x] = AC ? cconj(ra[s][x]) : ra[s][x];
#pragma unroll
      for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) {
          cr[x][y] = zmfma(av[x].x, rb[s][y].x, cr[x][y]);
          ci[x][y] = zmfma(av[x].x, rb[s][y].y, ci[x][y]);
        }
#pragma unroll
      for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) {
          cr[x][y] = zmfma(-av[x].y, rb[s][y].y, cr[x][y]);
          ci[x][y] = zmfma(av[x].y, rb[s][y].x, ci[x][y]);
        }
    }
  };
  if (kb < ke) {
    load(kb, a[0], b[0]);
    for (int k0 = kb; k0 < ke; k0 += 8 * D) {  // past the end: zeros
      load(k0 + 4 * D, a[1], b[1]);
      mul(a[0], b[0]);
      load(k0 + 8 * D, a[0], b[0]);
      mul(a[1], b[1]);
    }
  }
  __shared__ double2 part[NW][ZT][ZT + 1];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++)
#pragma unroll
      for (int v = 0; v < 4; v++)
        part[w][16 * x + lg + 4 * v][16 * y + l16] = make_double2(cr[x][y][v], ci[x][y][v]);
  __syncthreads();
#pragma unroll
  for (int e = t; e < ZT * ZT; e += 64 * NW) {
    const int il = CM ? e % ZT : e / ZT, jl = CM ? e / ZT : e % ZT;  // along C's rows in memory
    const int i = i0 + il, j = j0 + jl;
    if (i >= M || j >= N) continue;
    double2 c = part[0][il][jl];
#pragma unroll
    for (int q = 1; q < NW; q++) c = cadd(c, part[q][il][jl]);
    if (GA) c = cscale(c, g.cscale[j]);
    C[CM ? (long long)j * g.sc + i : (long long)i * g.sc + j] = c;
  }
}

// The same for the columns of many shots (A k-contiguous, B and C
// column-major): 64 x 64 tiles, each wavefront a 32 x 32 quarter, K advances 16
// at a time through LDS with the next step's loads issued before the current
// step's products.  A tile's four wavefronts share what they load, and the tiles
// of an XCD are a contiguous run along A's rows, so that those rows stay in its
// L2: 2048 x 32768 x 1024 7.9 ms (69 TFLOP/s) against 9.7 in 32 x 32 tiles, 512 x
// 32768 x 256 545 us against 587, 128 x 32768 x 64 52 against 66.  Bound by the
// matrix cores.
constexpr int ZW = 64, ZWK = 16;
template <class TA, class TB, bool GA>
__global__ __launch_bounds__(256, 4) void k_zgemm_cols(ZgemmArgs g) {
  // workgroup L runs on XCD L % 8
  const int nx = gridDim.x, ntile = gridDim.x * gridDim.y;
  const int L = blockIdx.x + nx * blockIdx.y, xcd = L & 7, slot = L >> 3;
  const int per = ntile >> 3, extra = ntile & 7;
  const int t_lin = xcd * per + min(xcd, extra) + slot;
  const int tx = t_lin % nx, ty = t_lin / nx;
  int N = g.N, j0 = tx * ZW, A_off_tile = 0;
  if (GA) {
    const int lo = *g.clo;
    N = *g.chi;
    j0 += lo;
    if (g.asplit && j0 >= *g.asplit) A_off_tile = 1;
  } else if (g.mcount) {
    N = min(N, g.mult * *g.mcount);
  }
  const int i0 = ty * ZW;
  if (j0 >= N) return;
  const int M = g.M, K = g.K, z = blockIdx.z;
  const TA *A = (const TA *)g.A + (z + A_off_tile) * g.za;
  const TB *B = (const TB *)g.B + z * g.zb;
  double2 *C = g.C + z * g.zc;
  __shared__ double2 As[ZWK][ZW], Bs[ZWK][ZW];
  const int t = threadIdx.x;
  // this thread's share of a K step: 4 elements of a row of A and of a column of B
  const int row = t >> 2, k4 = (t & 3) * 4, gi = i0 + row, gj = j0 + row;
  const TA *pa = A + (long long)min(gi, M - 1) * g.sa;
  const TB *pb = B + (GA ? (long long)g.bmap[min(gj, N - 1)] : min(gj, N - 1)) * g.sb;
  double2 ra[4], rb[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int gk = k0 + k4 + q;
      ra[q] = gi < M && gk < K ? cload(pa + gk) : make_double2(0.0, 0.0);
      rb[q] = gj < N && gk < K ? cload(pb + gk) : make_double2(0.0, 0.0);
    }
  };
  const int w = t >> 6, lane = t & 63, l16 = lane & 15, lg = lane >> 4;
  const int wm = (w & 1) * 32, wn = (w >> 1) * 32;
  zd4_t cr[2][2], ci[2][2];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++) {
      cr[x][y] = zd4_t{0.0, 0.0, 0.0, 0.0};
      ci[x][y] = zd4_t{0.0, 0.0, 0.0, 0.0};
    }
  load(0);
  for (int k0 = 0; k0 < K; k0 += ZWK) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      As[k4 + q][row] = ra[q];
      Bs[k4 + q][row] = rb[q];
    }
    __syncthreads();
    if (k0 + ZWK < K) load(k0 + ZWK);
#pragma unroll
    for (int kk = 0; kk < ZWK; kk += 4) {
      double2 a[2], b[2];
#pragma unroll
      for (int x = 0; x < 2; x++) {
        a[x] = As[kk + lg][wm + 16 * x + l16];
        b[x] = Bs[kk + lg][wn + 16 * x + l16];
      }
#pragma unroll
      for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) {
          cr[x][y] = zmfma(a[x].x, b[y].x, cr[x][y]);
          cr[x][y] = zmfma(-a[x].y, b[y].y, cr[x][y]);
          ci[x][y] = zmfma(a[x].x, b[y].y, ci[x][y]);
          ci[x][y] = zmfma(a[x].y, b[y].x, ci[x][y]);
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int y = 0; y < 2; y++) {
      const int j = j0 + wn + 16 * y + l16;
      if (j >= N) continue;
      const double sc = GA ? g.cscale[j] : 1.0;
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int i = i0 + wm + 16 * x + lg + 4 * v;
        if (i < M) C[(long long)j * g.sc + i] = make_double2(sc * cr[x][y][v], sc * ci[x][y][v]);
      }
    }
}

// Whether the 64 x 64 tiles are the better ones.  They need about four of them
// for every row of K, up to the 1024 that the chip holds at once, and past that a
// last round of tiles that is not nearly empty; K of up to 16 leaves the 32 x 32
// kernel's wavefronts without work.  us in 32 x 32 / 64 x 64 tiles: K = 32, 128
// tiles 6.5 / 9.1, 256 tiles 10.1 / 9.7; K = 128, 376 tiles 38 / 45, 512 tiles 49 /
// 46; K = 256, 376 tiles 61 / 79, 1024 tiles 152 / 146; K = 384, 1128 tiles 247 / 267,
// 1536 tiles 329 / 312; K = 16, 64 tiles 6.0 / 5.4.
static bool zgemm_cols(const ZgemmArgs &g) {
  const long long tiles = (long long)((g.M + ZW - 1) / ZW) * ((g.N + ZW - 1) / ZW) * g.batch;
  const long long rounds = (tiles + 1023) / 1024;
  return g.K <= 16 || (tiles >= std::max(180, std::min(4 * g.K, 1024)) &&
                       (rounds == 1 || 10 * tiles >= 7 * 1024 * rounds));
}

// f(TA(), TB()) with the operands' element types
template <class F>
static void zgemm_types(int a_storage, int b_storage, F f) {
  if (a_storage == 0 && b_storage == 0)
    f(double2(), double2());
  else if (a_storage == 0)
    f(double2(), float2());
  else if (b_storage == 0)
    f(float2(), double2());
  else
    f(float2(), float2());
}

template <bool AK, bool AC, bool BK, bool CM, bool GA = false>
static void zgemm_dispatch(hipStream_t st, const ZgemmArgs &g, int a_storage, int b_storage) {
  static_assert(!CM || (AK && !AC && BK), "column-major products take k_zgemm_cols");
  const dim3 grid((g.N + ZT - 1) / ZT, (g.M + ZT - 1) / ZT, g.batch);
  // fewer tiles than CUs and a K to split: twice the wavefronts on each
  const bool few = (size_t)grid.x * grid.y * grid.z <= 256 && g.K >= 64;
  zgemm_types(a_storage, b_storage, [&](auto ta, auto tb) {
    using TA = decltype(ta);
    using TB = decltype(tb);
    if constexpr (CM) {
      if (zgemm_cols(g)) {
        hipLaunchKernelGGL((k_zgemm_cols<TA, TB, GA>),
                           dim3((g.N + ZW - 1) / ZW, (g.M + ZW - 1) / ZW, g.batch), dim3(256), 0,
                           st, g);
        return;
      }
    }
    if (few)
      hipLaunchKernelGGL((k_zgemm<TA, TB, AK, AC, BK, CM, GA, 8>), grid, dim3(512), 0, st, g);
    else
      hipLaunchKernelGGL((k_zgemm<TA, TB, AK, AC, BK, CM, GA, 4>), grid, dim3(256), 0, st, g);
  });
}

void launch_zgemm(hipStream_t st, ZgemmKind kind, const ZgemmArgs &g, int a_storage,
                  int b_storage) {
  if (g.M <= 0 || g.N <= 0) return;
  switch (kind) {
    case ZGEMM_NN_ROW:  // C = A B, A k-contiguous, B and C row-major
      zgemm_dispatch<true, false, false, false>(st, g, a_storage, b_storage);
      break;
    case ZGEMM_CN_ROW:  // C = A^H B, A stored K x M row-major, B and C row-major
      zgemm_dispatch<false, true, false, false>(st, g, a_storage, b_storage);
      break;
    case ZGEMM_NN_COL:  // C = A B, A k-contiguous, B and C column-major
      zgemm_dispatch<true, false, true, true>(st, g, a_storage, b_storage);
      break;
    case ZGEMM_NN_COL_GATHER:  // the same on gathered, scaled columns
      if (g.clo && g.chi && g.bmap && g.cscale)
        zgemm_dispatch<true, false, true, true, true>(st, g, a_storage, b_storage);
      break;
  }
}

}  // namespace tn
