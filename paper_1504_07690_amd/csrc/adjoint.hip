// Kernels of the adjoint of the estimate L = sum_i phibar_i phi~(t_i) with respect to
// the stored values of A (the hot path run backwards; not part of the paper).
//
//   Zbar_i = W Kbar_W,i + 2 Z_i Kbar_Z,i            (from K_W = sym(W^T Z), K_Z = Z^T Z)
//   Ybar_k = sum_i mu_k(t_i) Zbar_i                  (transposed sweep: the sweep kernels
//                                                    with the coefficient table transposed)
//   Lambda_k = Ybar_k + 2 A~ Lambda_{k+1} - Lambda_{k+2}   (the recurrence kernel)
//   abar_e += alpha c_k Lambda_k[r_e] . Y_{k-1}[c_e],  c_1 = 1, c_k = 2 (k >= 2)
#include <algorithm>

#include "ssm_kernels.h"

namespace ssm {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Zbar, in place over Z: one workgroup per (sweep point, run of rows).  The
// stack [Kbar_W; 2 Kbar_Z] sits in LDS as FP64 (two 16T x 16T halves); each wave takes 16
// rows at a time and multiplies [W | Z] (16 x 2 N_v) by it on
// v_mfma_f64_16x16x4_f64, T = N_v/16 output blocks per wave.  A wave reads only
// the rows it writes, and writes them after its last read of them.
// ---------------------------------------------------------------------------
// What bounds it: the FP64 MFMAs: 1.15 ms at the rate of a large product for 100 points of N = 32768,
// N_v = 80 in FP32, which took 1.81 ms with one wave a SIMD and 4096 rows a workgroup and take 1.6:
// two waves a SIMD, one's stores and conversions behind the other's MFMAs, where the registers hold
// it, and rows dealt so that no CU waits for a last round (zbar_rows).
template <int T, typename In>
constexpr int zbar_threads() {
  return T <= (sizeof(In) == 4 ? 5 : 4) ? 512 : 256;
}

template <int T, typename In>
__global__ void __launch_bounds__((zbar_threads<T, In>())) zbar_kernel(int64_t n, int nv, int64_t rows_per_block,
                                                                       const In* __restrict__ w, In* __restrict__ z,
                                                                       const double* __restrict__ kw_bar,
                                                                       const double* __restrict__ kz_bar) {
  constexpr int TH = zbar_threads<T, In>();
  // [Kbar_W; 2 Kbar_Z] as two NP x NP halves (rows and columns past N_v zero), so that
  // the contraction index q < 2 NP needs no bounds test
  extern __shared__ double kb[];
  constexpr int NP = 16 * T;
  constexpr int KQ = 2 * NP / 4;  // contraction steps of four
  const int i = blockIdx.y;
  const int64_t nn = (int64_t)nv * nv;
  const double* kwb = kw_bar + i * nn;
  const double* kzb = kz_bar + i * nn;
  // stack fill: eight loads in flight per thread before their LDS stores
  constexpr int total = 2 * NP * NP;
  for (int base = threadIdx.x; base < total; base += 8 * TH) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = base + TH * u;
      const int r = idx / NP, c = idx % NP;
      const int hr = r < NP ? r : r - NP;  // row inside its half
      double x = 0.0;
      if (idx < total && c < nv && hr < nv) x = (r < NP) ? kwb[(int64_t)hr * nv + c] : 2.0 * kzb[(int64_t)hr * nv + c];
      v[u] = x;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (base + TH * u < total) kb[base + TH * u] = v[u];
  }
  __syncthreads();
  In* zi = z + (int64_t)i * n * nv;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r_end = (r_begin + rows_per_block < n) ? r_begin + rows_per_block : n;
  // the 16 x 2 NP slab of [W | Z] for rows r0 .. r0+15: A[m = lane%16][k = 4 s + lane/16];
  // indices are clamped into the arrays (rows past the range, columns past N_v), and the
  // values they bring meet zero stack rows or feed rows that are not stored
  auto load_slab = [&](int64_t r0, In (&av)[KQ]) {
    int64_t row = r0 + (lane & 15);
    row = row < r_end ? row : r_end - 1;
    const In* wr = w + row * nv;
    const In* zr = zi + row * nv;
#pragma unroll
    for (int s = 0; s < KQ; ++s) {
      const int q = 4 * s + (lane >> 4);
      const int c = (q < NP ? q : q - NP);
      const int cc = c < nv ? c : nv - 1;
      av[s] = (q < NP) ? wr[cc] : zr[cc];
    }
  };
  In cur[KQ], nxt[KQ];
  int64_t r0 = r_begin + 16 * wave;
  if (r0 < r_end) load_slab(r0, cur);
  for (; r0 < r_end; r0 += TH / 4) {
    // the next slab's loads are in flight behind this slab's MFMAs
    if (r0 + TH / 4 < r_end) load_slab(r0 + TH / 4, nxt);
    f64x4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    // the stack operands of step s + 1 are read from LDS behind the MFMAs of step s
    const double* kbl = kb + (lane >> 4) * NP + (lane & 15);
    double bcur[T], bnxt[T];
#pragma unroll
    for (int t = 0; t < T; ++t) bcur[t] = kbl[16 * t];
#pragma unroll
    for (int s = 0; s < KQ; ++s) {
      if (s + 1 < KQ) {
#pragma unroll
        for (int t = 0; t < T; ++t) bnxt[t] = kbl[4 * (s + 1) * NP + 16 * t];
      }
      const double a = (double)cur[s];
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bcur[t], acc[t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < T; ++t) bcur[t] = bnxt[t];
    }
    // result register r of lane l holds D[l/16 + 4r][l%16]; every read of these
    // rows by this wave is complete (the MFMA results depend on all of them)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int col = 16 * t + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t orow = r0 + (lane >> 4) + 4 * r;
        if (orow < r_end && col < nv) zi[orow * nv + col] = (In)acc[t][r];
      }
    }
#pragma unroll
    for (int s = 0; s < KQ; ++s) cur[s] = nxt[s];
  }
}

// N_v above 96: the stack does not fit in LDS; the same MFMA walk reads [Kbar_W;
// 2 Kbar_Z] through the cache (one point's stack is shared by all its row blocks),
// and the 16 x 2 N_v slab is loaded eight k-steps at a time.
template <int T, typename In>
__global__ void __launch_bounds__(256) zbar_big_kernel(int64_t n, int nv, int64_t rows_per_block,
                                                       const In* __restrict__ w,
                                                       In* __restrict__ z, const double* __restrict__ kw_bar,
                                                       const double* __restrict__ kz_bar) {
  constexpr int NP = 16 * T;
  constexpr int KQ = 2 * NP / 4;
  const int i = blockIdx.y;
  const int64_t nn = (int64_t)nv * nv;
  const double* kwb = kw_bar + i * nn;
  const double* kzb = kz_bar + i * nn;
  In* zi = z + (int64_t)i * n * nv;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r_end = (r_begin + rows_per_block < n) ? r_begin + rows_per_block : n;
  for (int64_t r0 = r_begin + 16 * wave; r0 < r_end; r0 += 64) {
    const int64_t row = r0 + (lane & 15);
    const bool rok = row < r_end;
    f64x4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    for (int s0 = 0; s0 < KQ; s0 += 8) {
      In av[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = 4 * (s0 + u) + (lane >> 4);
        In v = (In)0;
        if (rok && q < 2 * nv) v = (q < nv) ? w[row * nv + q] : zi[row * nv + (q - nv)];
        av[u] = v;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = 4 * (s0 + u) + (lane >> 4);
        const double a = (double)av[u];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const int c = 16 * t + (lane & 15);
          double bv = 0.0;
          if (c < nv && q < 2 * nv) bv = (q < nv) ? kwb[(int64_t)q * nv + c] : 2.0 * kzb[(int64_t)(q - nv) * nv + c];
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv, acc[t], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int col = 16 * t + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t orow = r0 + (lane >> 4) + 4 * r;
        if (orow < r_end && col < nv) zi[orow * nv + col] = (In)acc[t][r];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// One step of the reverse recurrence fused with the gradient on the pattern:
//
//   out = Lambda_k = a (A x) + b x + c xprev + d,   x = Lambda_{k+1}, xprev =
//         Lambda_{k+2}, d = Ybar_k, (a, b, c) = (2 alpha, 2 beta, -1);
//         x == NULL gives out = d (k = M), xprev == NULL drops the c term;
//   abar[p] += coef * Lambda_k[r] . y[c_p] for the stored entries p of row r,
//         y = Y_{k-1}, in FP64.
//
// A row of N_v values is held by L = N_v/4 lanes, 4 values each (16 bytes in FP32, 32 in FP64); a
// wave holds R = min(64/L, 16) whole rows side by side, so that a gather's lanes read whole
// cache lines (eight lanes a row in passes read parts of more lines, and stalled on lines in flight).
// Each CSR entry of the wave's rows is loaded once, by one lane, and reaches the row's lanes
// through LDS: eight entries a row at a time.  The lanes' partial dot products of those go
// through LDS too: H lanes sum one (row, entry) over the row's L lanes.  (Summed by permutes,
// each entry's six steps of two permutes bounded the kernel.)
// Rows go to XCDs in contiguous ranges, as in the forward recurrence, and a lattice's rows are
// visited in the same tiled order.
// What bounds it: up to the gradient's part, the blocks that it moves (14.7 us of the 21 at N = 32768,
// N_v = 80 in FP32, 52 MB a step with Y's 10); then the exact products, 36 conversions and 32 FP64
// operations a lane, and their sums through LDS.
// Measured per step, FP32 (FP64), permutes and per-lane entries before: N = 32768 lattice, N_v = 80
// 28.9 to 21.0 us (47 to 33); N = 22500, N_v = 40 12.8 to 7.7; N = 262144, N_v = 80 173 to 139;
// a random graph of 20000 rows and 17 entries a row, N_v = 80 43.6 to 36.4.
// ---------------------------------------------------------------------------
constexpr int RV_ROWS = 16;
constexpr int RV_LD = 65;  // lanes of one entry's partial sums, padded: the sums' reads spread over the banks

template <typename T>
struct ReverseShared {
  double part[8 * RV_LD];
  T vals[8 * RV_ROWS];
  uint32_t cols[8 * RV_ROWS];
};

__device__ __forceinline__ void reverse_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// BUF: blocks below 2 GiB, gathered through buffer resources: a 32-bit offset an entry instead of
// a 64-bit address, and the padding's offset is past the block, which reads as zero unasked.
template <typename T, typename V, bool BUF>
__global__ void __launch_bounds__(256, !BUF ? 1 : sizeof(T) == 4 ? 4 : 3)
    reverse_step_kernel(int64_t n, int L, int R, int H, int64_t nblocks, int64_t per_xcd,
                        const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                        const T* __restrict__ val, T a, T b, T c, const V* __restrict__ x,
                        const V* __restrict__ xprev, const V* __restrict__ d, V* __restrict__ out,
                        const V* __restrict__ y, double coef, double* __restrict__ abar, int keep,
                        TileOrder order) {
  __shared__ ReverseShared<T> shared[4];
  const int64_t lblock = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lblock >= nblocks) return;  // uniform over the workgroup
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ReverseShared<T>& sh = shared[wave];
  const int lane = threadIdx.x & 63;
  const int g = lane / L;
  const int q = lane - g * L;
  const int64_t rho = (lblock * 4 + wave) * R + g;
  const bool active = g < R && rho < n;
  const int64_t rs = !active ? 0 : order.nx ? (int64_t)order.row((uint32_t)rho) : rho;  // idle lanes read row 0
  const int p0 = row_ptr[rs];
  const int len = active ? row_ptr[rs + 1] - p0 : 0;
  const bool longer = __any(len > 8);  // uniform over the wave, like every loop below
  const uint32_t bytes = BUF ? (uint32_t)(n * L * sizeof(V)) : 0;
  const int slots = 8 * R;

  // entries j .. j + 7 of the wave's rows: to LDS, then each row's eight to its lanes
  uint32_t cols[8];  // BUF: the rows' byte offsets
  T vals[8];
  auto load_entries = [&](int j) {
    reverse_sync();
    for (int s0 = 0; s0 < slots; s0 += 64) {
      const int s = s0 + lane, src = (s >> 3) * L;
      const int pg = __shfl(p0, src), lg = __shfl(len, src), e = j + (s & 7);
      if (s < slots) {
        const bool ok = e < lg;
        const uint32_t col = ok ? (uint32_t)col_idx[pg + e] : 0u;
        sh.cols[s] = !BUF ? col : ok ? col * (uint32_t)(L * sizeof(V)) : 0x80000000u;
        sh.vals[s] = ok ? val[pg + e] : (T)0;
      }
    }
    reverse_sync();
    const int s = 8 * (g < R ? g : 0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      cols[u] = BUF && !active ? 0x80000000u : sh.cols[s + u];
      vals[u] = sh.vals[s + u];
    }
  };
  // their rows' pieces in a block; padded slots issue no gather
  auto gather = [&](const V* block, int j, V (&v)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if constexpr (BUF) {
        if (u >= 5 && !__any(j + u < len)) {  // no row of the wave has a sixth, seventh, eighth entry
          v[u] = (V)(T)0;
          continue;
        }
        const auto r = __builtin_amdgcn_make_buffer_rsrc((void*)block, (short)0, bytes, 0x00020000);
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 w[sizeof(V) / 16];
#pragma unroll
        for (int h = 0; h < (int)sizeof(V) / 16; ++h)
          w[h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                               r, (int)(cols[u] + (uint32_t)sizeof(V) * q + 16 * h), 0, 0));
        __builtin_memcpy(&v[u], w, sizeof(V));
      } else {
        v[u] = (V)(T)0;
        if (j + u < len) v[u] = block[(int64_t)cols[u] * L + q];
      }
    }
  };

  // the sums that this lane's group of H forms: (row, entry j + (o & 7)) o = lane / H, ...
  const int hl = lane & (H - 1), per_round = 64 / H;
  double g0[2] = {};  // what they are added to, for j = 0, loaded ahead of the gathers
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int o = lane / H + r * per_round, src = (o >> 3) * L & 63;
    const int pg = __shfl(p0, src), lg = __shfl(len, src);
    if (o < slots && hl == 0 && (o & 7) < lg) g0[r] = abar[pg + (o & 7)];
  }

  load_entries(0);
  const int64_t own = rs * L + q;
  V res = (V)(T)0, xp = (V)(T)0, xo = (V)(T)0;
  if (active) {
    // Lambda_{k+2} and Ybar_k are read for the last time: streamed with non-temporal hints
    res = __builtin_nontemporal_load(&d[own]);
    if (xprev) xp = __builtin_nontemporal_load(&xprev[own]);
    if (x) xo = x[own];
  }
  if (x) {
    V acc = (V)(T)0;
    V v[8];
    gather(x, 0, v);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __builtin_elementwise_fma((V)vals[u], v[u], acc);
    if (longer) {
#pragma unroll 1
      for (int j = 8; __any(j < len); j += 8) {
        load_entries(j);
        gather(x, j, v);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_elementwise_fma((V)vals[u], v[u], acc);
      }
      load_entries(0);
    }
    // the product with x, then one FMA with the larger a acc, as in the recurrence: left to the compiler's
    // contraction it rounds a acc by itself, which costs a step in FP32 4.37e-8 of error for 4.15e-8
    V t;
    {
#pragma clang fp contract(off)
      t = b * xo;
    }
    t = __builtin_elementwise_fma((V)a, acc, t);
    if (xprev) t = __builtin_elementwise_fma((V)c, xp, t);
    res = t + res;
  }
  if (active) {
    if (keep)
      out[own] = res;
    else
      __builtin_nontemporal_store(res, &out[own]);
  }
#pragma unroll 1
  for (int j = 0; __any(j < len); j += 8) {
    if (j > 0) load_entries(j);
    V v[8];
    gather(y, j, v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      double t = (double)res.x * (double)v[u].x;
      t += (double)res.y * (double)v[u].y;
      t += (double)res.z * (double)v[u].z;
      t += (double)res.w * (double)v[u].w;
      sh.part[u * RV_LD + lane] = t;
    }
    reverse_sync();
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int o = lane / H + r * per_round;
      if (r * per_round >= slots) break;  // uniform
      const int src = (o >> 3) * L & 63;
      const int pg = __shfl(p0, src), lg = __shfl(len, src), e = j + (o & 7);
      const bool ok = o < slots && e < lg;
      double t = 0.0;
      if (ok) {
        const double* part = sh.part + (o & 7) * RV_LD + src;
        for (int i = hl; i < L; i += H) t += part[i];
      }
      for (int m = H >> 1; m > 0; m >>= 1) t += __shfl_xor(t, m);
      if (ok && hl == 0) {
        double* to = &abar[pg + e];
        *to = (j == 0 ? g0[r] : *to) + coef * t;
      }
    }
    reverse_sync();
  }
}

// ct[i*ldct + k] = c[k*ldc + i] (FP64 and FP32 copies), zero padded to ldct
__global__ void __launch_bounds__(256) transpose_coefficients_kernel(const double* __restrict__ c, int64_t ldc, int nt,
                                                                     int m1, double* __restrict__ ct64,
                                                                     float* __restrict__ ct32, int64_t ldct) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)nt * ldct) return;
  const int i = (int)(gid / ldct);
  const int k = (int)(gid - (int64_t)i * ldct);
  const double v = k < m1 ? c[(int64_t)k * ldc + i] : 0.0;
  if (ct64) ct64[gid] = v;
  if (ct32) ct32[gid] = (float)v;
}

// Rows per workgroup of `step` rows a turn, at most 4096: of the multiples of step the one whose
// workgroups, one a CU at a time, end first, counting what each spends before its rows (the
// stack's fill, the last rows' stores) as `before` rows.
int64_t zbar_rows(int64_t n, int ntb, int step, int before) {
  int64_t best = step, least = INT64_MAX;
  for (int64_t r = step; r <= 4096; r += step) {
    const int64_t groups = (n + r - 1) / r * ntb;
    const int64_t cost = (groups + 255) / 256 * (r + before);
    if (cost < least) {
      least = cost;
      best = r;
    }
  }
  return best;
}

template <int T>
hipError_t launch_zbar_big(int is_f32, int64_t n, int nv, int ntb, const void* w, void* z, const double* kwb,
                           const double* kzb, hipStream_t stream) {
  constexpr int64_t rows = 256;  // no stack to fill: as many workgroups as hide each other's loads
  dim3 grid((unsigned)((n + rows - 1) / rows), ntb);
  if (is_f32)
    hipLaunchKernelGGL((zbar_big_kernel<T, float>), grid, dim3(256), 0, stream, n, nv, rows, (const float*)w,
                       (float*)z, kwb, kzb);
  else
    hipLaunchKernelGGL((zbar_big_kernel<T, double>), grid, dim3(256), 0, stream, n, nv, rows, (const double*)w,
                       (double*)z, kwb, kzb);
  return hipGetLastError();
}

template <int T, typename In>
hipError_t launch_zbar_in(int64_t n, int nv, int ntb, const In* w, In* z, const double* kwb, const double* kzb,
                          hipStream_t stream) {
  constexpr int TH = zbar_threads<T, In>();
  const size_t lds = (size_t)2 * (16 * T) * (16 * T) * sizeof(double);
  const int64_t rows = zbar_rows(n, ntb, TH / 4, 64);
  hipError_t err = hipFuncSetAttribute((const void*)zbar_kernel<T, In>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((zbar_kernel<T, In>), dim3((unsigned)((n + rows - 1) / rows), ntb), dim3(TH), lds, stream, n, nv,
                     rows, w, z, kwb, kzb);
  return hipGetLastError();
}

template <int T>
hipError_t launch_zbar_t(int is_f32, int64_t n, int nv, int ntb, const void* w, void* z, const double* kwb,
                         const double* kzb, hipStream_t stream) {
  return is_f32 ? launch_zbar_in<T, float>(n, nv, ntb, (const float*)w, (float*)z, kwb, kzb, stream)
                : launch_zbar_in<T, double>(n, nv, ntb, (const double*)w, (double*)z, kwb, kzb, stream);
}

// Split tables of the transposed sweep: rows k, columns the sweep points i,
// chi[k*ldk + i] = bf16(c[k][i]), clo = bf16(c[k][i] - chi), each rounded once from
// the FP64 value (ties to even); zero padding up to ldk.
__global__ void __launch_bounds__(256) split_rows_kernel(const double* __restrict__ c, int64_t ldc, int nt, int m1,
                                                         __bf16* __restrict__ chi, __bf16* __restrict__ clo,
                                                         int64_t ldk) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)m1 * ldk) return;
  const int k = (int)(gid / ldk);
  const int i = (int)(gid - (int64_t)k * ldk);
  __bf16 hi = (__bf16)0.f, lo = (__bf16)0.f;
  if (i < nt) {
    const double v = c[(int64_t)k * ldc + i];
    hi = (__bf16)v;
    lo = (__bf16)(v - (double)hi);
  }
  chi[gid] = hi;
  clo[gid] = lo;
}

}  // namespace

hipError_t launch_split_rows(const double* c, int64_t ldc, int nt, int m1, __bf16* chi, __bf16* clo, int64_t ldk,
                             hipStream_t stream) {
  const int64_t total = (int64_t)m1 * ldk;
  hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, c, ldc, nt, m1,
                     chi, clo, ldk);
  return hipGetLastError();
}

hipError_t launch_zbar(int is_f32, int64_t n, int nv, int ntb, const void* w, void* z, const double* kw_bar,
                       const double* kz_bar, hipStream_t stream) {
  switch ((nv + 15) / 16) {
    case 1: return launch_zbar_t<1>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 2: return launch_zbar_t<2>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 3: return launch_zbar_t<3>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 4: return launch_zbar_t<4>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 5: return launch_zbar_t<5>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 6: return launch_zbar_t<6>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 7: case 8: return launch_zbar_big<8>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 9: case 10: case 11: case 12: return launch_zbar_big<12>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    case 13: case 14: case 15: case 16: return launch_zbar_big<16>(is_f32, n, nv, ntb, w, z, kw_bar, kz_bar, stream);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, typename V>
hipError_t launch_reverse_t(int64_t n, int nv, const int32_t* row_ptr, const int32_t* col_idx, const T* val, T a, T b,
                            T c, const T* x, const T* xprev, const T* d, T* out, const T* y, double coef,
                            double* abar, const RowOrder& o, hipStream_t stream) {
  const int L = nv / 4;
  if (L < 1 || L > 64 || nv % 4) return hipErrorInvalidValue;
  const int R = std::min(64 / L, RV_ROWS);
  int H = 1;  // lanes that sum one (row, entry): 8 R groups of H, in one round up to 8 rows
  while (16 * R * H <= 64) H *= 2;
  const int64_t rows_per_block = 4 * (int64_t)R;
  const int64_t nblocks = (n + rows_per_block - 1) / rows_per_block;
  const int64_t per_xcd = (nblocks + 7) / 8;
  if (per_xcd * 8 > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (o.nx > 0 &&
      !(o.tx > 0 && o.ty > 0 && o.nx % o.tx == 0 && o.ny % o.ty == 0 && (int64_t)o.nx * o.ny * o.nz == n))
    return hipErrorInvalidValue;
  // Lambda_k is next gathered by the following step, from the last-level cache if a step's five
  // blocks leave it there: stored normally up to 64 MiB (33 MB: 56.3 us a step against 59.4 stored
  // non-temporally; 84 MB: 144 against 142)
  const int keep = n * L * (int64_t)sizeof(V) <= ((int64_t)64 << 20);
  const auto fn = n * L * (int64_t)sizeof(V) < ((int64_t)1 << 31) ? reverse_step_kernel<T, V, true>
                                                                  : reverse_step_kernel<T, V, false>;
  hipLaunchKernelGGL(fn, dim3((unsigned)(per_xcd * 8)), dim3(256), 0, stream, n, L, R, H, nblocks, per_xcd, row_ptr,
                     col_idx, val, a, b, c, (const V*)x, (const V*)xprev, (const V*)d, (V*)out, (const V*)y, coef, abar,
                     keep, o.nx > 0 ? TileOrder(o) : TileOrder());
  return hipGetLastError();
}

hipError_t launch_transpose_coefficients(const double* c, int64_t ldc, int nt, int m1, double* ct64, float* ct32,
                                         int64_t ldct, hipStream_t stream) {
  const int64_t total = (int64_t)nt * ldct;
  hipLaunchKernelGGL(transpose_coefficients_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, c,
                     ldc, nt, m1, ct64, ct32, ldct);
  return hipGetLastError();
}

hipError_t launch_reverse_step_f64(int64_t n, int nv, const int32_t* row_ptr, const int32_t* col_idx,
                                   const double* val, double a, double b, double c, const double* x,
                                   const double* xprev, const double* d, double* out, const double* y, double coef,
                                   double* abar, hipStream_t stream, const RowOrder& order) {
  return launch_reverse_t<double, f64x4>(n, nv, row_ptr, col_idx, val, a, b, c, x, xprev, d, out, y, coef, abar,
                                         order, stream);
}

hipError_t launch_reverse_step_f32(int64_t n, int nv, const int32_t* row_ptr, const int32_t* col_idx,
                                   const float* val, float a, float b, float c, const float* x, const float* xprev,
                                   const float* d, float* out, const float* y, double coef, double* abar,
                                   hipStream_t stream, const RowOrder& order) {
  return launch_reverse_t<float, f32x4>(n, nv, row_ptr, col_idx, val, a, b, c, x, xprev, d, out, y, coef, abar,
                                        order, stream);
}

}  // namespace ssm
