// Gram matrices of the sweep (Eq. tracelr; Algorithm 5, step 13):
//
//   K_W(t_i) = W^T Z_i (symmetric),   K_Z(t_i) = Z_i^T Z_i,     Z_i, W: N x N_v
//
// in FP64 on v_mfma_f64_16x16x4_f64.  FP32 inputs are widened to FP64 exactly, so
// every product is exact and only the FP64 sums round.  W^T Z_i = W^T g(t_i I - A~) W is
// symmetric in exact arithmetic, so only its upper 16x16 blocks W_a^T Z_b (a <= b) are
// formed: a diagonal block is averaged with its transpose and the lower blocks mirror
// the upper ones.  This is one symmetric completion of the computed W^T Z; (W^T Z +
// Z^T W)/2 is another, with the same value in exact arithmetic and one more product.
//
// Work split.  N_v <= 96: a wave keeps every upper 16x16 block (a <= b) of Z^T Z and of W^T Z
// of one point in registers.  Above, the block grid is cut into tiles of 4 x 4 blocks (ti <= tj)
// and a wave keeps one tile's (the upper ten of a diagonal tile: with all sixteen a quarter of
// the matrix work at N_v = 128 went into blocks that are never read).  The pairs (tile, point)
// are items of n rows each.  Every item is cut into 4 nseg parts, what the caller's scratch holds,
// one per wave.  Where whole rounds of the waves resident on the 1024 SIMDs would leave the last one
// rather empty (125 points in 9 segments of 4 waves are 4.4 rounds of 1024, 12% idle), the items, laid
// end to end, are cut into equal shares instead, one per resident wave.  A wave walks its rows eight
// at a time (two MFMA steps of four rows) and writes its partial blocks to scratch; a second kernel
// adds the partials of an item in order and completes the symmetric matrices (deterministic).
//
// Rounding.  A matrix that is the sum of many chains of MFMAs is off in proportion to the chains' length:
// each by its length's root, with as many fewer to average (rms of the diagonal of W^T Z at N = 262144,
// N_v = 80: parts of 7282 rows 1.9e-15, shares of 32000 rows as one chain 9.2e-15).  So a share is summed
// in runs no longer than a part, each a chain of its own, which are added in the wave's partial: 1.8e-15.
//
// What bounds it: the FP64 matrix cores.  Operands come straight from memory, two steps ahead of
// the MFMAs that consume them: lane l reads column 16a + l%16 of row r + l/16 for each column
// block a, for Z_i and W (a 4-row slab is contiguous).
// Measured (FP32 blocks, N = 262144, with the reduction; before: a workgroup per point and segment, all
// sixteen blocks of diagonal tiles): N_v = 80, 125 points 9.25 to 7.99 ms; N_v = 128, 151 points 34.0 to
// 26.3 ms (49 TFLOP/s on 2 N N_v^2 a point, of 72.7 for the library's square product); N_v = 256,
// 20 points 19.2 to 12.7 ms.
#include <algorithm>

#include "ssm_kernels.h"

namespace ssm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int GR_WAVES = 4;   // waves per workgroup, and scratch slots per segment
constexpr int GT_B = 4;       // blocks per side of a tile (N_v above 96)
constexpr int GR_ROWS = 8;    // rows per unit of work

// The items of one kind (nz tiles x ntb points, item it = z ntb + i) and the waves that share
// them.  parts > 0: every item in `parts` equal pieces, one per wave; else wave w takes q units
// (GR_ROWS rows), and one more if w < rem, of the items' units laid end to end, in runs.
struct GramShare {
  int64_t units;  // per item
  int64_t items, q, rem;
  int64_t seg;
  int64_t run;  // rows of one chain of sums at most (a multiple of GR_ROWS)
  int waves, parts;

  // first row of piece k, or the row past its last (end = 1)
  __host__ __device__ int64_t part_begin(int k, int64_t n, int end = 0) const {
    const int64_t s0 = k / GR_WAVES * seg, s1 = s0 + seg < n ? s0 + seg : n;
    const int64_t q = ((s1 - s0 + GR_WAVES - 1) / GR_WAVES + 3) / 4 * 4;
    const int64_t r = s0 + (k % GR_WAVES + end) * q;
    return r < s1 ? r : s1;
  }
  __host__ __device__ int64_t start(int64_t w) const { return w * q + (w < rem ? w : rem); }
  // the wave that holds unit u of the line
  __host__ __device__ int64_t owner(int64_t u) const {
    const int64_t b = rem * (q + 1);
    return u < b ? u / (q + 1) : rem + (u - b) / q;
  }
  __host__ __device__ int slots(int64_t it) const {
    return parts ? parts : (int)(owner((it + 1) * units - 1) - owner(it * units) + 1);
  }
};

struct GramPlan {
  GramShare diag, off;  // N_v <= 96: one diagonal tile holding every block
  int64_t n;
  int ntb, ntile;       // points, tiles per side
};

// Operand loads are buffer loads over the wave's own rows: the resource's byte range
// ends at the last row of the piece, and the hardware returns 0 for reads past it, so
// the rows of the last partial step arrive as zeros with no clamping, masking or
// branching.  Columns 16a + l%16 >= N_v of a row inside the range read the next row;
// they only feed output entries that are never stored.  Unpredicated loads whose
// values are used as loaded let the compiler count them: waiting for the oldest
// buffer does not also wait for the prefetch just issued.
template <typename In>
__device__ __forceinline__ In buffer_load(__amdgpu_buffer_rsrc_t r, int byte_off);
template <>
__device__ __forceinline__ float buffer_load<float>(__amdgpu_buffer_rsrc_t r, int byte_off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0));
}
template <>
__device__ __forceinline__ double buffer_load<double>(__amdgpu_buffer_rsrc_t r, int byte_off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, 0));
}

constexpr int kBufferWord3 = 0x00020000;  // raw 32-bit buffer access (gfx9 family)

// The blocks a wave keeps: A columns ca .. ca + TA - 1 of Z and W against TB columns of Z from
// cb; UPPER: TA = TB and ca = cb, blocks a <= b only (and one set of Z columns).
template <int TA, int TB, bool UPPER>
struct GramShape {
  static constexpr int NP = UPPER ? TA * (TA + 1) / 2 : TA * TB;
  static __device__ constexpr int index(int a, int b) { return UPPER ? a * TA - a * (a - 1) / 2 + (b - a) : a * TB + b; }
};

template <int TA, int TB, bool UPPER, typename In>
__device__ __forceinline__ void gram_rows(const In* __restrict__ z, const In* __restrict__ w, int64_t r_begin,
                                          int rows, int nv, int ca, int cb,
                                          f64x4 (&acc_zz)[GramShape<TA, TB, UPPER>::NP],
                                          f64x4 (&acc_wz)[GramShape<TA, TB, UPPER>::NP]) {
  using G = GramShape<TA, TB, UPPER>;
  const int lane = threadIdx.x & 63;
  const int es = (int)sizeof(In);
  int off_a[TA], off_b[TB];
#pragma unroll
  for (int a = 0; a < TA; ++a) off_a[a] = ((lane >> 4) * nv + 16 * (ca + a) + (lane & 15)) * es;
#pragma unroll
  for (int b = 0; b < TB; ++b) off_b[b] = ((lane >> 4) * nv + 16 * (cb + b) + (lane & 15)) * es;
  struct Raw {
    In za[TA], wa[TA], zb[TB];
  };
  const __amdgpu_buffer_rsrc_t rz =
      __builtin_amdgcn_make_buffer_rsrc((void*)(z + r_begin * nv), (short)0, rows * nv * es, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc((void*)(w + r_begin * nv), (short)0, rows * nv * es, kBufferWord3);
  auto load = [&](Raw& r, int row) {
    const int base = row * nv * es;
#pragma unroll
    for (int a = 0; a < TA; ++a) {
      r.za[a] = buffer_load<In>(rz, base + off_a[a]);
      r.wa[a] = buffer_load<In>(rw, base + off_a[a]);
    }
    if constexpr (!UPPER) {
#pragma unroll
      for (int b = 0; b < TB; ++b) r.zb[b] = buffer_load<In>(rz, base + off_b[b]);
    }
  };
  struct Op {
    double za[TA], wa[TA], zb[TB];
  };
  auto widen = [&](Op& o, const Raw& r) {
#pragma unroll
    for (int a = 0; a < TA; ++a) {
      o.za[a] = (double)r.za[a];
      o.wa[a] = (double)r.wa[a];
    }
#pragma unroll
    for (int b = 0; b < TB; ++b) o.zb[b] = UPPER ? o.za[b] : (double)r.zb[b];
  };
  auto multiply_zz = [&](const Op& o) {
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int b = UPPER ? a : 0; b < TB; ++b) {
        const int p = G::index(a, b);
        acc_zz[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.za[a], o.zb[b], acc_zz[p], 0, 0, 0);
      }
  };
  auto multiply_wz = [&](const Op& o) {
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
      for (int b = UPPER ? a : 0; b < TB; ++b) {
        const int p = G::index(a, b);
        acc_wz[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.wa[a], o.zb[b], acc_wz[p], 0, 0, 0);
      }
  };
  // A step widens its rows, refills their buffer with the rows two steps ahead and runs its
  // MFMAs; scheduling barriers keep steps apart, so that their operands need not be live
  // together.  At T = 5 (one wave per SIMD, registers to spare) the next step's rows are widened
  // between the two halves of this step's MFMAs instead, 3% faster (8.33 to 8.07 ms at N =
  // 262144, N_v = 80, 125 points); elsewhere that was 0-2% slower, and spilled at T = 6.
  constexpr bool AHEAD = TA == 5;
  Raw r0, r1;
  load(r0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load(r1, 4);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (AHEAD) {
    Op c0, c1;
    widen(c0, r0);
    load(r0, 8);
    __builtin_amdgcn_sched_barrier(0);
    auto step = [&](const Op& cur, Op& nxt, Raw& raw, int row) {
      multiply_zz(cur);
      widen(nxt, raw);
      load(raw, row);
      __builtin_amdgcn_sched_barrier(0);
      multiply_wz(cur);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma clang loop unroll(disable)
    for (int rr = 0; rr < rows; rr += 8) {
      step(c0, c1, r1, rr + 12);
      step(c1, c0, r0, rr + 16);
    }
  } else {
    auto step = [&](Raw& raw, int row) {
      Op o;
      widen(o, raw);
      load(raw, row);
      multiply_zz(o);
      multiply_wz(o);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma clang loop unroll(disable)
    for (int rr = 0; rr < rows; rr += 8) {
      step(r0, rr + 8);
      step(r1, rr + 12);
    }
  }
}

// The blocks into a partial, or (ADD and add) onto what the same lanes stored there before.  Entries past
// N_v go to an offset past the resource's range: the hardware reads 0 there and drops the store.
template <int TA, int TB, bool UPPER, bool ADD>
__device__ __forceinline__ void gram_store(double* __restrict__ pz, int nv, int ca, int cb, bool add,
                                           const f64x4 (&acc_zz)[GramShape<TA, TB, UPPER>::NP],
                                           const f64x4 (&acc_wz)[GramShape<TA, TB, UPPER>::NP]) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63;
  int cols = nv;  // opaque: the bounds tests are made here, not kept in registers over the row loop
  asm volatile("" : "+s"(cols));
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)pz, (short)0, 16 * cols * cols, kBufferWord3);
  const int to_w = 8 * cols * cols;
  // the lane's entry r of block p; FP64 result layout: D[l/16 + 4r][l%16]
  auto offset = [&](int p, int r) {
    int a = 0, b = p;
    if constexpr (UPPER) {
      while (b >= TA - a) b -= TA - a++;
      b += a;
    } else {
      a = p / TB;
      b = p % TB;
    }
    const int row = 16 * (ca + a) + (lane >> 4) + 4 * r, col = 16 * (cb + b) + (lane & 15);
    return row < cols && col < cols ? 8 * (row * cols + col) : (int)0x80000000;
  };
  // a group of blocks at a time: the loads of its old values are in flight together
  constexpr int NP = GramShape<TA, TB, UPPER>::NP, G = !ADD ? 1 : NP == 15 ? 5 : NP >= 6 ? 2 : 1;
#pragma unroll
  for (int p0 = 0; p0 < NP; p0 += G) {
    double z[G][4] = {}, w[G][4] = {};
    if (ADD && add) {  // uniform
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (p0 + g < NP) {
            const int off = offset(p0 + g, r);
            z[g][r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rp, off, 0, 0));
            w[g][r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rp, off, to_w, 0));
          }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (p0 + g < NP) {
        f64x4 az = acc_zz[p0 + g], aw = acc_wz[p0 + g];
        // five blocks a side fill the accumulation registers, and stay there until their turn
        if constexpr (ADD && NP == 15) asm volatile("" : "+a"(az), "+a"(aw));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int off = offset(p0 + g, r);
          const double vz = ADD ? z[g][r] + az[r] : az[r], vw = ADD ? w[g][r] + aw[r] : aw[r];
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, vz), rp, off, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, vw), rp, off, to_w, 0);
        }
      }
    __builtin_amdgcn_sched_barrier(0);  // group by group: their offsets and old values need not be live together
  }
}

// A wave's part of the items of one kind.  locate(zt, ca, cb) gives the first columns of tile zt.
template <int TA, int TB, bool UPPER, bool EVEN, typename In, typename F>
__device__ __forceinline__ void gram_share(const GramShare& sh, int64_t wv, int64_t n, int ntb, int nv,
                                           const In* __restrict__ w, int64_t w_stride, const In* __restrict__ z,
                                           int64_t z_stride, double* __restrict__ part, F locate) {
  using G = GramShape<TA, TB, UPPER>;
  const int64_t nn = (int64_t)nv * nv;
  int64_t it, r0, left;  // item, first row in it, rows left to do
  const int64_t item = sh.units * GR_ROWS;  // rows of an item, the last unit filled up
  if (!EVEN || sh.parts) {
    it = wv / sh.parts;
    const int k = (int)(wv - it * sh.parts);
    r0 = sh.part_begin(k, n);
    left = sh.part_begin(k, n, 1) - r0;
  } else {
    const int64_t s0 = sh.start(wv);
    it = s0 / sh.units;
    r0 = (s0 - it * sh.units) * GR_ROWS;
    left = (sh.start(wv + 1) - s0) * GR_ROWS;
  }
  bool add = false;  // an item's later runs are added onto its first
#pragma unroll 1
  do {  // a run: a chain of sums of its own
    int64_t take = left < item - r0 ? left : item - r0;
    if (EVEN && take > sh.run) take = sh.run;
    const int zt = (int)(it / ntb);
    const int i = (int)(it - (int64_t)zt * ntb);
    const int64_t slot = !EVEN || sh.parts ? wv - it * sh.parts : wv - sh.owner(it * sh.units);
    int ca, cb;
    locate(zt, ca, cb);
    const int64_t r1 = r0 + take < n ? r0 + take : n;
    f64x4 acc_zz[G::NP], acc_wz[G::NP];
#pragma unroll
    for (int p = 0; p < G::NP; ++p) {
      acc_zz[p] = (f64x4){0.0, 0.0, 0.0, 0.0};
      acc_wz[p] = (f64x4){0.0, 0.0, 0.0, 0.0};
    }
    gram_rows<TA, TB, UPPER, In>(z + (int64_t)i * z_stride, w + (int64_t)i * w_stride, r0, (int)(r1 - r0), nv, ca, cb,
                                 acc_zz, acc_wz);
    gram_store<TA, TB, UPPER, EVEN>(part + (slot * ntb + i) * 2 * nn, nv, ca, cb, add, acc_zz, acc_wz);
    left -= take;
    r0 += take;
    add = r0 < item;
    if (!add) {
      ++it;
      r0 = 0;
    }
  } while (EVEN && left > 0);
}

// T >= 1: one tile of T x T blocks (upper); T = 0: 4 x 4-block tiles
// Even shares where the blocks leave registers for the partials they are added onto: at six blocks a side
// the row loop spilled (N = 100000, N_v = 96, 64 points in FP64: 5.0 ms, in parts 3.0).  Tiles are so many
// items that parts are not far from whole rounds (N = 200000, N_v = 256, 40 points: 23.5 ms, in parts 18.6).
template <int T>
constexpr bool gram_even() {
  return T >= 1 && T <= 5;
}

template <int T>
constexpr int gram_occupancy() {  // waves per SIMD (16 T (T + 1) accumulator registers, or 256)
  return T == 0 || T >= 5 ? 1 : T == 4 ? 2 : T == 3 ? 3 : T == 2 ? 5 : 8;
}

template <int T, typename In>
__global__ void __launch_bounds__(64 * GR_WAVES, (gram_occupancy<T>()))
    gram_kernel(GramPlan pl, int nv, const In* __restrict__ w, int64_t w_stride, const In* __restrict__ z,
                int64_t z_stride, double* __restrict__ part) {
  const int64_t wv = (int64_t)blockIdx.x * GR_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int D = T ? T : GT_B;
  if (wv < pl.diag.waves) {  // uniform over the wave; the kernel has no barrier
    gram_share<D, D, true, gram_even<T>(), In>(pl.diag, wv, pl.n, pl.ntb, nv, w, w_stride, z, z_stride, part,
                                               [](int zt, int& ca, int& cb) { ca = cb = GT_B * zt; });
  } else if (T == 0 && wv < pl.diag.waves + pl.off.waves) {
    const int side = pl.ntile;
    if constexpr (T == 0)
      gram_share<GT_B, GT_B, false, false, In>(pl.off, wv - pl.diag.waves, pl.n, pl.ntb, nv, w, w_stride, z, z_stride,
                                               part, [side](int zt, int& ca, int& cb) {
                                                 int ti = 0;  // tiles (ti, tj), ti < tj, row by row
                                                 while (zt >= side - 1 - ti) zt -= side - 1 - ti++;
                                                 ca = GT_B * ti;
                                                 cb = GT_B * (ti + 1 + zt);
                                               });
  }
}

// K(i) from its items' partials, added in order: a workgroup per 16 x 16 block (a <= b) of a point, an
// entry per lane, which stores a diagonal block's average with its transpose, or the block and, through
// LDS, its mirror.
// What bounds it: reading the partials, GR_LOAD of each kind in flight a lane (N = 4096, N_v = 80, 200
// points, 24 partials each: 0.3 GB).  A lane per entry of the whole matrices, which branched on the
// block's kind before its loads, read most entries twice, those of the lower blocks N_v apart.
// Measured, FP32 blocks: that case 520 to 76 us (before the branch 298), N = 1000, N_v = 80, 200 points
// 220 to 26 (136), N = 200000, N_v = 256, 12 points 3600 to 318 (3600), N = 20000, N_v = 4, 16 points
// 82 to 20.
constexpr int GR_LOAD = 8;

__global__ void __launch_bounds__(256) gram_reduce_kernel(GramPlan pl, int nv, const double* __restrict__ part,
                                                          double* __restrict__ k_w, double* __restrict__ k_z) {
  __shared__ double tz[16][17], tw[16][17];
  const int side = (nv + 15) / 16, pairs = side * (side + 1) / 2;
  const int i = (int)(blockIdx.x / (unsigned)pairs);
  int b = (int)blockIdx.x - i * pairs, a = 0;
  while (b >= side - a) b -= side - a++;
  b += a;
  const int64_t nn = (int64_t)nv * nv;
  const int ti = pl.ntile ? a / GT_B : 0, tj = pl.ntile ? b / GT_B : 0;
  const int zt = ti * (pl.ntile - 1) - ti * (ti - 1) / 2 + (tj - ti - 1);
  const int ns = ti == tj ? pl.diag.slots((int64_t)ti * pl.ntb + i) : pl.off.slots((int64_t)zt * pl.ntb + i);
  const int y = threadIdx.x >> 4, x = threadIdx.x & 15;
  const int r = 16 * a + y, c = 16 * b + x;
  const bool in = r < nv && c < nv;
  double sz = 0.0, sw = 0.0;
  if (in) {
    const double* p = part + (int64_t)i * 2 * nn + r * nv + c;
    const int64_t step = (int64_t)pl.ntb * 2 * nn;
    for (int s = 0; s < ns; s += GR_LOAD) {
      double vz[GR_LOAD], vw[GR_LOAD];
#pragma unroll
      for (int u = 0; u < GR_LOAD; ++u) {
        const double* q = p + (s + u < ns ? s + u : ns - 1) * step;
        vz[u] = q[0];
        vw[u] = q[nn];
      }
#pragma unroll
      for (int u = 0; u < GR_LOAD; ++u) {
        if (s + u < ns) {
          sz += vz[u];
          sw += vw[u];
        }
      }
    }
  }
  tz[y][x] = sz;
  tw[y][x] = sw;
  __syncthreads();
  double* oz = k_z + i * nn;
  double* ow = k_w + i * nn;
  if (a == b) {
    if (in) {
      oz[r * nv + c] = 0.5 * (sz + tz[x][y]);
      ow[r * nv + c] = 0.5 * (sw + tw[x][y]);
    }
    return;
  }
  if (in) {
    oz[r * nv + c] = sz;
    ow[r * nv + c] = sw;
  }
  const int rm = 16 * b + y, cm = 16 * a + x;
  if (rm < nv && cm < nv) {
    oz[rm * nv + cm] = tz[x][y];
    ow[rm * nv + cm] = tw[x][y];
  }
}

// `waves` equal shares of the items in runs of at most `part` rows, if an item's partials (at most its
// units over a wave's, and one) fit `slots` and a run's rows fit `max_rows`
bool share_evenly(GramShare& sh, int64_t waves, int slots, int64_t part, int64_t max_rows) {
  const int64_t total = sh.items * sh.units;
  if (total < waves) return false;
  sh.parts = 0;
  sh.waves = (int)waves;
  sh.q = total / waves;
  sh.rem = total % waves;
  sh.run = part / GR_ROWS * GR_ROWS;
  return (sh.units + sh.q - 1) / sh.q + 1 <= slots && sh.run <= max_rows;
}

// every item in its scratch's slots: segments of `seg` rows of GR_WAVES parts
bool share_parts(GramShare& sh, int64_t n, int64_t seg, int64_t max_rows) {
  const int64_t parts = (n + seg - 1) / seg * GR_WAVES;
  if (sh.items * parts > 0x3FFFFFFF) return false;
  sh.seg = seg;
  sh.parts = (int)parts;
  sh.waves = (int)(sh.items * parts);
  sh.run = seg / GR_WAVES;
  return sh.run <= max_rows;
}

template <int T>
hipError_t launch_t(int is_f32, GramPlan& pl, int nv, int nseg, const void* w, int64_t ws, const void* z, int64_t zs,
                    double* scratch, hipStream_t stream) {
  const int slots = nseg * GR_WAVES;
  // a wave's rows, with the prefetch's overrun, must be addressable by 32-bit byte offsets
  const int64_t max_rows = (((int64_t)1 << 31) - 1) / ((int64_t)nv * (is_f32 ? 4 : 8)) - 16;
  const int64_t resident = 1024 * (int64_t)gram_occupancy<T>();
  // rows of a segment, of which a part is a quarter
  int64_t seg = (pl.n + nseg - 1) / nseg;
  seg = (seg + 4 * GR_WAVES - 1) / (4 * GR_WAVES) * (4 * GR_WAVES);
  GramShare& d = pl.diag;
  if (!share_parts(d, pl.n, seg, max_rows) || (pl.off.items && !share_parts(pl.off, pl.n, seg, max_rows)))
    return hipErrorInvalidValue;
  // Even shares instead where the parts' last round of resident waves would leave 1% and more of the
  // waves' time idle, and parts are long beside the stores and loads of a run's end (1024 rows, a
  // quarter of a millisecond at N_v = 80).  N_v = 80: N = 262144, 125 points (14% idle) 8.95 ms in parts,
  // 7.97 in even shares; N = 110592, 500 points (2.4%) 13.7, 13.4.
  const int64_t idle = (d.waves + resident - 1) / resident * resident - d.waves;
  if (gram_even<T>() && seg / GR_WAVES >= 1024 && d.waves > resident && 100 * idle >= d.waves) {
    GramShare even = d;
    if (share_evenly(even, resident, slots, seg / GR_WAVES, max_rows)) d = even;
  }
  const int64_t waves = (int64_t)pl.diag.waves + pl.off.waves;
  const dim3 grid((unsigned)((waves + GR_WAVES - 1) / GR_WAVES)), block(64 * GR_WAVES);
  if (is_f32)
    hipLaunchKernelGGL((gram_kernel<T, float>), grid, block, 0, stream, pl, nv, (const float*)w, ws, (const float*)z,
                       zs, scratch);
  else
    hipLaunchKernelGGL((gram_kernel<T, double>), grid, block, 0, stream, pl, nv, (const double*)w, ws,
                       (const double*)z, zs, scratch);
  return hipGetLastError();
}

// Point i reads W at w + i * ws and Z at z + i * zs (elements).
hipError_t launch_strided(int is_f32, int64_t n, int nv, int ntb, const void* w, int64_t ws, const void* z,
                          int64_t zs, double* k_w, double* k_z, int nseg, double* scratch, hipStream_t stream) {
  const int t = (nv + 15) / 16;
  if (t > 16) return hipErrorInvalidValue;
  GramPlan pl{};
  pl.n = n;
  pl.ntb = ntb;
  pl.ntile = t <= 6 ? 0 : (t + GT_B - 1) / GT_B;
  pl.diag.units = pl.off.units = (n + GR_ROWS - 1) / GR_ROWS;
  pl.diag.items = (int64_t)ntb * std::max(1, pl.ntile);
  pl.off.items = (int64_t)ntb * (pl.ntile * (pl.ntile - 1) / 2);
  hipError_t err;
  switch (pl.ntile ? 0 : t) {
    case 1: err = launch_t<1>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    case 2: err = launch_t<2>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    case 3: err = launch_t<3>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    case 4: err = launch_t<4>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    case 5: err = launch_t<5>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    case 6: err = launch_t<6>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream); break;
    default: err = launch_t<0>(is_f32, pl, nv, nseg, w, ws, z, zs, scratch, stream);
  }
  if (err != hipSuccess) return err;
  const int64_t blocks = (int64_t)ntb * (t * (t + 1) / 2);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, pl, nv, scratch, k_w, k_z);
  return hipGetLastError();
}

}  // namespace

int gram_scratch_slots(int nseg) { return nseg * GR_WAVES; }

hipError_t launch_gram(int is_f32, int64_t n, int nv, int ntb, const void* w, const void* z, double* k_w,
                       double* k_z, int nseg, double* scratch, hipStream_t stream) {
  return launch_strided(is_f32, n, nv, ntb, w, 0, z, n * nv, k_w, k_z, nseg, scratch, stream);
}

hipError_t launch_gram_pairs(int is_f32, int64_t n, int nv, int npairs, const void* y_hi, const void* y_lo,
                             int64_t stride, double* k_w, double* k_z, int nseg, double* scratch,
                             hipStream_t stream) {
  return launch_strided(is_f32, n, nv, npairs, y_hi, stride, y_lo, stride, k_w, k_z, nseg, scratch, stream);
}

}  // namespace ssm
