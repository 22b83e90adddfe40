// Algorithm 1 (Delta-Gauss-Chebyshev coefficients) for all sweep points at once.
//
// mu_l(t) = (2 - delta_l0) / (2 N_theta) * Re sum_{j<2N_theta} exp(-i 2 pi j l / 2N_theta) g_j,
// g_j = g_sigma(t - x(cos theta_j)), theta_j = j pi / N_theta   (Eq. mucoef2 discretised),
// by a fast Fourier transform per sweep point.
#include <algorithm>

#include "ssm_kernels.h"

namespace ssm {
namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));

// The transform.  N = N_theta is a power of two, and g is even in j (cos theta_{2N-j} =
// cos theta_j), so only N + 1 values are evaluated.  The 2N real values h_j are taken as N
// complex ones z_m = h_{2m} + i h_{2m+1}, transformed in LDS by self-sorting (Stockham)
// passes of radix 8, and at the end 4 or 2, a thread holding its inputs in registers
// between the two barriers of a pass; then, with Z_l = a + ib and Z_{N-l} = c + id,
//   Re sum_j h_j e^{-i pi j l / N} = ((a + c) + cos(pi l/N) (b + d) - sin(pi l/N) (a - c)) / 2.
// Twiddles and the cos theta_j come from one table cos(pi m / N), m < N/2, in LDS; a
// butterfly looks up the first, second and fourth power of its root and multiplies them up
// to the others.  Element i of z sits at i ^ ((i >> 3) & 7): a radix-8 pass writes elements
// 8 j + r from lane j, which unswizzled all fall in the same banks.
//
// What bounds it: LDS traffic, about 2 log_8 N passes over 16 N bytes per point, and the
// N + 1 exponentials.  A workgroup keeps its table for several points (as many workgroups
// as fit on the 256 CUs), and the points of one XCD are consecutive, so that the 8-byte
// entries of a table row that neighbouring points write meet in that XCD's L2.
// Measured: 81 us for 2000 points of degree 2000 (48 MB written), against 8040 us for the
// direct cosine sums over the same LDS tables, which read 2 N_theta values per coefficient;
// 25 us for 1000 points of degree 1000, 113 us for 1000 of degree 4000.
__device__ __forceinline__ int fft_at(int i) { return i ^ ((i >> 3) & 7); }

// cos(pi m / N) for 0 <= m < 2N from the table of m < N/2
__device__ __forceinline__ double cos_at(const double* tab, int n, int m) {
  m = m > n ? 2 * n - m : m;  // cos(2 pi - x)
  const bool neg = 2 * m > n;
  m = neg ? n - m : m;
  const double v = 2 * m == n ? 0.0 : tab[m];
  return neg ? -v : v;
}

// e^{-2 pi i t / N}, 0 <= t < N
__device__ __forceinline__ f64x2 root_at(const double* tab, int n, int t) {
  const int m = 2 * t;                            // angle pi m / N
  const int q = m >= n / 2 ? m - n / 2 : n / 2 - m;  // sin x = cos(x - pi/2)
  return (f64x2){cos_at(tab, n, m), -cos_at(tab, n, q)};
}

__device__ __forceinline__ f64x2 cmul(f64x2 a, f64x2 b) {
  return (f64x2){a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// forward transforms of 2, 4 and 8 values, in place, results in natural order
__device__ __forceinline__ void dft2(f64x2& a, f64x2& b) {
  const f64x2 t = a - b;
  a = a + b;
  b = t;
}
__device__ __forceinline__ f64x2 mul_mi(f64x2 a) { return (f64x2){a.y, -a.x}; }  // times -i
__device__ __forceinline__ void dft4(f64x2& a, f64x2& b, f64x2& c, f64x2& d) {
  dft2(a, c);
  dft2(b, d);
  d = mul_mi(d);
  dft2(a, b);
  dft2(c, d);
  const f64x2 t = b;  // order a, c, b, d -> a, b, c, d
  b = c;
  c = t;
}
template <int R>
__device__ __forceinline__ void dft(f64x2 (&v)[R]) {
  if constexpr (R == 2) {
    dft2(v[0], v[1]);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
  } else {
    constexpr double h = 0.70710678118654752440;
    f64x2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft4(e[0], e[1], e[2], e[3]);
    dft4(o[0], o[1], o[2], o[3]);
    o[1] = (f64x2){h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};
    o[2] = mul_mi(o[2]);
    o[3] = (f64x2){h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = e[r] + o[r];
      v[r + 4] = e[r] - o[r];
    }
  }
}

// One pass of radix R over z (ns: product of the radices before it).  A thread takes the
// 8 / R butterflies tid, tid + TH, ..., where TH >= N / 8.
template <int R>
__device__ __forceinline__ void fft_pass(f64x2* z, const double* tab, int n, int ns) {
  constexpr int B = 8 / R;
  const int nb = n / R;
  f64x2 v[B][R];
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const int j = threadIdx.x + u * blockDim.x;
    if (j >= nb) continue;
#pragma unroll
    for (int r = 0; r < R; ++r) v[u][r] = z[fft_at(j + r * nb)];
    const int k = j & (ns - 1);
    if (ns > 1) {
      const int step = k * (n / (ns * R));  // root of index r is e^{-2 pi i r step / N}, r step < N
      f64x2 w[R];
      w[1] = root_at(tab, n, step);
      if constexpr (R >= 4) {
        w[2] = root_at(tab, n, 2 * step);
        w[3] = cmul(w[1], w[2]);
      }
      if constexpr (R == 8) {
        w[4] = root_at(tab, n, 4 * step);
        w[5] = cmul(w[4], w[1]);
        w[6] = cmul(w[4], w[2]);
        w[7] = cmul(w[4], w[3]);
      }
#pragma unroll
      for (int r = 1; r < R; ++r) v[u][r] = cmul(v[u][r], w[r]);
    }
    dft<R>(v[u]);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const int j = threadIdx.x + u * blockDim.x;
    if (j >= nb) continue;
    const int k = j & (ns - 1);
    const int o = (j - k) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) z[fft_at(o + r * ns)] = v[u][r];
  }
  __syncthreads();
}

__global__ void __launch_bounds__(1024) dgc_coefficients_kernel(double c0, double hw, double sigma, double inv_norm,
                                                                const double* __restrict__ t, int nt, int per_xcd,
                                                                int degree, int n, double* __restrict__ c,
                                                                float* __restrict__ c32, int64_t ldc) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  f64x2* z = (f64x2*)lds;        // n complex values
  double* zs = lds;              // the same as 2n doubles
  double* tab = lds + 2 * n;     // n / 2
  for (int m = threadIdx.x; m < n / 2; m += blockDim.x) tab[m] = cospi((double)m / (double)n);
  const double inv2s2 = 1.0 / (2.0 * sigma * sigma);
  const int first = (int)(blockIdx.x & 7) * per_xcd;
  const int last = min(first + per_xcd, nt);
  for (int i = first + (int)(blockIdx.x >> 3); i < last; i += (int)(gridDim.x >> 3)) {
    const double ti = t[i];
    __syncthreads();  // the table is written; the last point's z is read
    for (int j = threadIdx.x; j <= n; j += blockDim.x) {
      const double s = ti - (c0 + hw * cos_at(tab, n, j));
      const double g = inv_norm * exp(-s * s * inv2s2);
      // h_j and h_{2n-j}: even j are real parts, odd j imaginary parts
      const int part = j & 1;
      zs[2 * fft_at(j >> 1) + part] = g;
      const int jm = 2 * n - j;
      if (j > 0) zs[2 * fft_at(jm >> 1) + part] = g;
    }
    __syncthreads();
    int ns = 1;
    for (; ns * 8 <= n; ns *= 8) fft_pass<8>(z, tab, n, ns);
    if (ns * 4 == n) fft_pass<4>(z, tab, n, ns);
    if (ns * 2 == n) fft_pass<2>(z, tab, n, ns);
    for (int l = threadIdx.x; l <= degree; l += blockDim.x) {
      const f64x2 zl = z[fft_at(l)], zc = z[fft_at((n - l) & (n - 1))];
      const double cs = cos_at(tab, n, l), sn = cos_at(tab, n, n / 2 >= l ? n / 2 - l : l - n / 2);
      const double re = 0.5 * ((zl.x + zc.x) + (cs * (zl.y + zc.y) - sn * (zl.x - zc.x)));
      const double mu = re / (double)(2 * n) * (l == 0 ? 1.0 : 2.0);
      c[(int64_t)l * ldc + i] = mu;
      if (c32) c32[(int64_t)l * ldc + i] = (float)mu;
    }
  }
}

// Proposition 1: nu_l(t_i), l = 0..2h, of the square of sum_{k<=h} mu_k(t_i) T_k.  With
// T_p T_q = (T_{p+q} + T_{|p-q|}) / 2 over ordered pairs (p, q),
//   nu_l = 1/2 sum_{p+q=l} mu_p mu_q + 1/2 sum_{|p-q|=l} mu_p mu_q,
// the second sum being sum_p mu_p^2 for l = 0 and 2 sum_p mu_p mu_{p+l} otherwise: the
// exact coefficients (the quadrature the proposition names gives the same numbers for
// N_theta > 2h).  One lane per (l, column); columns nt..ldn-1 are written as 0.
__global__ void __launch_bounds__(256) square_coefficients_kernel(const double* __restrict__ mu, int64_t ldc,
                                                                  int nt, int h, int64_t ldn,
                                                                  double* __restrict__ nu) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int m1 = 2 * h + 1;
  if (idx >= (int64_t)m1 * ldn) return;
  const int l = (int)(idx / ldn);
  const int i = (int)(idx - (int64_t)l * ldn);
  if (i >= nt) {
    nu[idx] = 0.0;
    return;
  }
  double conv = 0.0;  // p + q = l
  const int p_lo = l > h ? l - h : 0;
  const int p_hi = l < h ? l : h;
  for (int p = p_lo; p <= p_hi; ++p) conv += mu[(int64_t)p * ldc + i] * mu[(int64_t)(l - p) * ldc + i];
  double diff = 0.0;  // |p - q| = l
  for (int p = 0; p + l <= h; ++p) diff += mu[(int64_t)p * ldc + i] * mu[(int64_t)(p + l) * ldc + i];
  if (l > 0) diff *= 2.0;
  nu[idx] = 0.5 * (conv + diff);
}

}  // namespace

hipError_t launch_square_coefficients(const double* mu, int64_t ldc, int nt, int h, double* nu, int64_t ldn,
                                      hipStream_t stream) {
  const int64_t total = (int64_t)(2 * h + 1) * ldn;
  hipLaunchKernelGGL(square_coefficients_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, mu, ldc,
                     nt, h, ldn, nu);
  return hipGetLastError();
}

namespace {

// mun[i] = sqrt(sum_l c[l][i]^2): 16 points per workgroup, 64 groups of 16 lanes taking every
// 64th degree, summed in a fixed order (deterministic).  With 64 points and four waves a
// workgroup, 500 points left 8 workgroups of 250 dependent steps: 74 us at 1001 degrees.
__global__ void __launch_bounds__(1024) coefficient_norms_kernel(const double* __restrict__ c, int64_t ldc, int nt,
                                                                 int m1, double* __restrict__ mun) {
  __shared__ double part[64][17];
  const int lane = threadIdx.x & 15, q = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + lane;
  double acc = 0.0;
  if (i < nt) {
#pragma unroll 4
    for (int l = q; l < m1; l += 64) {
      const double v = c[(int64_t)l * ldc + i];
      acc += v * v;
    }
  }
  part[q][lane] = acc;
  __syncthreads();
  for (int s = 32; s > 0; s >>= 1) {
    if (q < s) part[q][lane] += part[q + s][lane];
    __syncthreads();
  }
  if (q == 0 && i < nt) mun[i] = sqrt(part[0][lane]);
}

// kmax[l] = max_i |c[l][i]|: one workgroup per degree
__global__ void __launch_bounds__(256) coefficient_row_max_kernel(const double* __restrict__ c, int64_t ldc, int nt,
                                                                  double* __restrict__ kmax) {
  __shared__ double red[256];
  const double* row = c + (int64_t)blockIdx.x * ldc;
  double m = 0.0;
  for (int i = threadIdx.x; i < nt; i += 256) m = fmax(m, fabs(row[i]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) kmax[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) rounding_floor_kernel(const double* __restrict__ mun, int nt, double eta,
                                                             const double* __restrict__ w_sumsq, double inv_sqrt_e,
                                                             double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nt) out[i] = eta * mun[i] * (w_sumsq[0] * inv_sqrt_e);
}

}  // namespace

hipError_t launch_coefficient_norms(const double* c, int64_t ldc, int nt, int m1, double* mun, hipStream_t stream) {
  hipLaunchKernelGGL(coefficient_norms_kernel, dim3((unsigned)((nt + 15) / 16)), dim3(1024), 0, stream, c, ldc, nt, m1,
                     mun);
  return hipGetLastError();
}

hipError_t launch_coefficient_row_max(const double* c, int64_t ldc, int nt, int m1, double* kmax,
                                      hipStream_t stream) {
  hipLaunchKernelGGL(coefficient_row_max_kernel, dim3((unsigned)m1), dim3(256), 0, stream, c, ldc, nt, kmax);
  return hipGetLastError();
}

hipError_t launch_rounding_floor(const double* mun, int nt, double eta, const double* w_sumsq, double inv_sqrt_e,
                                 double* floor_out, hipStream_t stream) {
  hipLaunchKernelGGL(rounding_floor_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, stream, mun, nt, eta,
                     w_sumsq, inv_sqrt_e, floor_out);
  return hipGetLastError();
}

hipError_t launch_coefficients(double c0, double hw, double sigma, double inv_norm, const double* t, int nt,
                               int degree, int n_theta, double* c, float* c32, int64_t ldc,
                               hipStream_t stream) {
  // z (n_theta complex) and the table of n_theta / 2 cosines: 160 KB, a CU's whole LDS, at the
  // largest degrees (n_theta = 8192)
  const size_t lds = (size_t)n_theta * 20;
  if (n_theta < 4 || (n_theta & (n_theta - 1)) || lds > 160 * 1024 || 2 * (degree + 1) > n_theta)
    return hipErrorInvalidValue;
  hipError_t err = hipFuncSetAttribute((const void*)dgc_coefficients_kernel,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (err != hipSuccess) return err;
  const int th = std::max(64, n_theta / 8);
  // workgroups that are resident at once (at most 2048 threads and 160 KB of LDS a CU), at
  // most one per point
  const int per_cu = std::min<int>(2048 / th, (int)(160 * 1024 / lds));
  const int per_xcd = (nt + 7) / 8;
  const int grid = 8 * std::min(per_xcd, 32 * per_cu);
  hipLaunchKernelGGL(dgc_coefficients_kernel, dim3(grid), dim3(th), lds, stream, c0, hw, sigma, inv_norm, t, nt,
                     per_xcd, degree, n_theta, c, c32, ldc);
  return hipGetLastError();
}

}  // namespace ssm
