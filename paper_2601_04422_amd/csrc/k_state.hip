// State kernels: |0...0> initialisation, one-qubit gates, storage conversion.
#include <algorithm>

#include "tnsim_internal.h"
#include "tn_complex.h"

namespace tn {

// |0...0>: every site (1,2,1) = (1, 0), every bond weight (1)   (Sec. IV.A)
__global__ void k_init_state(void *const *sites, int n, int storage, double *const *lams, int nb) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) {
    if (storage == 0) {
      double2 *a = (double2 *)sites[q];
      a[0] = make_double2(1.0, 0.0);
      a[1] = make_double2(0.0, 0.0);
    } else {
      float2 *a = (float2 *)sites[q];
      a[0] = make_float2(1.0f, 0.0f);
      a[1] = make_float2(0.0f, 0.0f);
    }
  }
  if (q < nb) lams[q][0] = 1.0;
}

void launch_init_state(hipStream_t st, void *const *sites, int n, int storage,
                       double *const *lams, int nb) {
  int m = n > nb ? n : nb;
  hipLaunchKernelGGL(k_init_state, dim3((m + 255) / 256), dim3(256), 0, st, sites, n, storage,
                     lams, nb);
}

__global__ void k_fill_zero(uint4 *p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

// Zero a 16-byte aligned region whose size is a multiple of 16 (a kernel, so
// that the call may sit inside a captured graph).
void launch_fill_zero(hipStream_t st, void *p, size_t bytes) {
  size_t n16 = bytes / 16;
  if (!n16) return;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st, (uint4 *)p, n16);
}

// One-qubit gates of a layer: A'[a,s',b] = sum_s U[s',s] A[a,s,b]  (eq. 3).
// grid.y = gate, grid.x covers the chiL*chiR (a,b) pairs of the largest site.
template <class S>
__device__ void apply_1q_body(const Gate1Desc &d, int e) {
  S *A = (S *)d.A;
  int a = e / d.chiR, b = e - a * d.chiR;
  size_t i0 = ((size_t)a * 2) * d.chiR + b, i1 = i0 + d.chiR;
  double2 x0 = cload(A + i0), x1 = cload(A + i1);
  // the fused multiply-adds written out, so that every kernel rounds alike
  auto mul = [](double2 u, double2 x) {
    return make_double2(fma(u.x, x.x, -(u.y * x.y)), fma(u.x, x.y, u.y * x.x));
  };
  double2 y0 = cadd(mul(d.u[0], x0), mul(d.u[1], x1));
  double2 y1 = cadd(mul(d.u[2], x0), mul(d.u[3], x1));
  cstore(A + i0, y0);
  cstore(A + i1, y1);
}

__global__ void k_apply_1q(const Gate1Desc *descs) {
  const Gate1Desc &d = descs[blockIdx.y];
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d.chiL * d.chiR) return;
  if (d.storage == 0)
    apply_1q_body<double2>(d, e);
  else
    apply_1q_body<float2>(d, e);
}

void launch_apply_1q(hipStream_t st, const Gate1Desc *d, int ng, int max_elems) {
  if (ng <= 0 || max_elems <= 0) return;
  hipLaunchKernelGGL(k_apply_1q, dim3((max_elems + 255) / 256, ng), dim3(256), 0, st, d);
}

// Descriptors as kernel arguments, 1 or GATE1_ARGS per launch (the arguments
// of a kernel are limited to 4 KB): no staging buffer, no copy to the device
// and no wait for the buffer, 12 us of a 1-qubit layer.
constexpr int GATE1_ARGS = 32;
template <int N>
struct Gate1Args {
  Gate1Desc d[N];
};

template <int N>
__global__ void k_apply_1q_args(const Gate1Args<N> args) {
  const Gate1Desc &d = args.d[N == 1 ? 0 : blockIdx.y];
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d.chiL * d.chiR) return;
  if (d.storage == 0)
    apply_1q_body<double2>(d, e);
  else
    apply_1q_body<float2>(d, e);
}

void launch_apply_1q_args(hipStream_t st, const Gate1Desc *d, int ng, int max_elems) {
  if (ng <= 0 || max_elems <= 0) return;
  if (ng == 1) {
    hipLaunchKernelGGL(k_apply_1q_args<1>, dim3((max_elems + 255) / 256), dim3(256), 0, st,
                       Gate1Args<1>{d[0]});
    return;
  }
  for (int g = 0; g < ng; g += GATE1_ARGS) {
    const int cnt = std::min(GATE1_ARGS, ng - g);
    Gate1Args<GATE1_ARGS> a{};
    std::copy(d + g, d + g + cnt, a.d);
    hipLaunchKernelGGL(k_apply_1q_args<GATE1_ARGS>, dim3((max_elems + 255) / 256, cnt), dim3(256),
                       0, st, a);
  }
}

// Copies inside device memory, up to COPY_ARGS per launch (blockIdx.y).  Each
// copy on its own took 2 us and a gap of 3; what a gradient records of a gate
// at chi = 64 is six of them, a checkpoint two per site.
constexpr int COPY_ARGS = 32;
struct CopyArgs {
  CopyItem c[COPY_ARGS];
};

__global__ __launch_bounds__(256) void k_copy_list(const CopyArgs args) {
  const CopyItem &c = args.c[blockIdx.y];
  const uint64_t *src = (const uint64_t *)c.src;
  uint64_t *dst = (uint64_t *)c.dst;
  const size_t total = (size_t)c.words * c.rows, stride = (size_t)gridDim.x * blockDim.x;
  size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c.rows == 1) {
    for (; e < total; e += stride) dst[e] = src[e];
  } else {
    for (; e < total; e += stride) {
      const size_t r = e / c.words, w = e - r * c.words;
      dst[r * c.dpitch + w] = src[r * c.spitch + w];
    }
  }
}

void launch_copy_list(hipStream_t st, const CopyItem *items, int n) {
  for (int g = 0; g < n; g += COPY_ARGS) {
    const int cnt = std::min(COPY_ARGS, n - g);
    CopyArgs a{};
    std::copy(items + g, items + g + cnt, a.c);
    size_t most = 0;
    for (int i = 0; i < cnt; i++) most = std::max(most, (size_t)a.c[i].words * a.c[i].rows);
    if (!most) continue;
    const size_t blocks = std::min<size_t>((most + 255) / 256, 2048);
    hipLaunchKernelGGL(k_copy_list, dim3((unsigned)blocks, cnt), dim3(256), 0, st, a);
  }
}

__global__ void k_convert(const void *src, int ss, void *dst, int ds, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    double2 v = ss == 0 ? ((const double2 *)src)[i] : f2d(((const float2 *)src)[i]);
    if (ds == 0)
      ((double2 *)dst)[i] = v;
    else
      ((float2 *)dst)[i] = d2f(v);
  }
}

void launch_convert(hipStream_t st, const void *src, int ss, void *dst, int ds, size_t count) {
  if (!count) return;
  size_t blocks = (count + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_convert, dim3((unsigned)blocks), dim3(256), 0, st, src, ss, dst, ds, count);
}

// A state copied in one launch, blockIdx.y = site (and the bond right of it).
// Two launches or copies per site took 3-5 us of host time each: 0.7 ms for 64
// sites, more than the bytes of any state up to chi = 400.
__global__ __launch_bounds__(256) void k_copy_state(int n, const int *dims, void *const *src,
                                                    int ss, void *const *dst, int ds,
                                                    double *const *lam_src,
                                                    double *const *lam_dst) {
  const int q = blockIdx.y;
  const size_t cnt = (size_t)dims[q] * 2 * dims[q + 1];
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  if (ss == ds && ss == 0) {
    const double2 *a = (const double2 *)src[q];
    double2 *b = (double2 *)dst[q];
    for (size_t i = i0; i < cnt; i += stride) b[i] = a[i];
  } else {
    for (size_t i = i0; i < cnt; i += stride) {
      const double2 v = ss == 0 ? ((const double2 *)src[q])[i] : f2d(((const float2 *)src[q])[i]);
      if (ds == 0)
        ((double2 *)dst[q])[i] = v;
      else
        ((float2 *)dst[q])[i] = d2f(v);
    }
  }
  if (q + 1 < n)
    for (size_t i = i0; i < (size_t)dims[q + 1]; i += stride) lam_dst[q][i] = lam_src[q][i];
}

void launch_copy_state(hipStream_t st, int n, const int *dims, void *const *src, int src_storage,
                       void *const *dst, int dst_storage, double *const *lam_src,
                       double *const *lam_dst, size_t most) {
  // four elements per thread of the largest site, at most 64 K threads a site
  const size_t blocks = std::min<size_t>((most + 1023) / 1024, 256);
  for (int q = 0; q < n; q += 65535) {  // grid.y limit
    const int k = std::min(n - q, 65535);
    hipLaunchKernelGGL(k_copy_state, dim3((unsigned)blocks, k), dim3(256), 0, st, n - q, dims + q,
                       src + q, src_storage, dst + q, dst_storage, lam_src + q, lam_dst + q);
  }
}

// Bond propagation (Sec. III.A, non-local gates): one site of the window
// with the gate's operator bond r (rg terms) merged into its bonds.  `old`
// holds the site as it was (complex128, chiL x 2 x chiR); `out` receives
//   role 0 (left site):   out[l, s', r chiR + c]        = sum_x X_r[s',x] old[l,x,c]
//   role 1 (in between):  out[r chiL + l, s, r chiR + c] = old[l,s,c]
//   role 2 (right site):  out[r chiL + l, s', c]        = sum_y Y_r[s',y] old[l,y,c]
// (other entries of a role-1 site, r != r', are zero).  F holds rg 2x2
// factors, row-major.  One thread per output entry.
template <class S>
__global__ void k_prop_merge(const double2 *old, S *out, int chiL, int chiR, int rg, int role,
                             Mat4x4 F) {
  const int nL = role == 0 ? chiL : rg * chiL, nR = role == 2 ? chiR : rg * chiR;
  const size_t total = (size_t)nL * 2 * nR;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x) {
    const int ri = (int)(e % nR), sp = (int)((e / nR) % 2), li = (int)(e / ((size_t)2 * nR));
    double2 v = make_double2(0.0, 0.0);
    if (role == 1) {
      const int r = li / chiL, l = li % chiL, r2 = ri / chiR, c = ri % chiR;
      if (r == r2) v = old[((size_t)l * 2 + sp) * chiR + c];
    } else {
      const int r = role == 0 ? ri / chiR : li / chiL;
      const int l = role == 0 ? li : li % chiL, c = role == 0 ? ri % chiR : ri;
      const double2 *f = F.v[r];
      v = cadd(cmul(f[2 * sp], old[((size_t)l * 2) * chiR + c]),
               cmul(f[2 * sp + 1], old[((size_t)l * 2 + 1) * chiR + c]));
    }
    cstore(out + e, v);
  }
}

void launch_prop_merge(hipStream_t st, const double2 *old, void *out, int storage, int chiL,
                       int chiR, int rg, int role, const Mat4x4 &F) {
  const size_t total = (size_t)(role == 0 ? chiL : rg * chiL) * 2 * (role == 2 ? chiR : rg * chiR);
  size_t blocks = (total + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (storage == 0)
    hipLaunchKernelGGL(k_prop_merge<double2>, dim3((unsigned)blocks), dim3(256), 0, st, old,
                       (double2 *)out, chiL, chiR, rg, role, F);
  else
    hipLaunchKernelGGL(k_prop_merge<float2>, dim3((unsigned)blocks), dim3(256), 0, st, old,
                       (float2 *)out, chiL, chiR, rg, role, F);
}

// Small results to the host: one workgroup writes them to pinned memory and
// then raises a flag there that the host polls.  Bound by launch and flag
// latency: 7.2 us from call to data for up to 4 KB, against 11.6 us for an
// asynchronous copy and a stream synchronisation.
__global__ __launch_bounds__(256) void k_fetch(uint64_t *host, const uint64_t *dev, int words,
                                               uint32_t *flag, uint32_t value) {
  for (int e = threadIdx.x; e < words; e += 256) host[e] = dev[e];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_fetch(hipStream_t st, void *host, const void *dev, size_t bytes, uint32_t *flag,
                  uint32_t value) {
  hipLaunchKernelGGL(k_fetch, dim3(1), dim3(256), 0, st, (uint64_t *)host, (const uint64_t *)dev,
                     (int)(bytes / 8), flag, value);
}

__global__ void k_put(double2 *dst, double2 value) { *dst = value; }

void launch_put(hipStream_t st, double2 *dst, double2 value) {
  hipLaunchKernelGGL(k_put, dim3(1), dim3(1), 0, st, dst, value);
}

}  // namespace tn
