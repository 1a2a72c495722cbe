// Line transforms of the spectral readouts as matrix products on the FP64 matrix units.
//
// The spectral derivative and the Fourier transform of a line of n points are products with a
// fixed n x n matrix.  Sixteen lines make it a contraction for v_mfma_f64_16x16x4: any length,
// one barrier between load and product, no bit reversal.  Each line is folded first into its
// even and odd part about point 0 (e_m = z_m + z_{n-m}, o_m = z_m - z_{n-m}), which maps even to
// odd and back under the derivative and separates cosines from sines: half the operations, and
// results j and n - j come out of the same two products.
//
// Derivative of one line: n^2 / 2 multiply-adds, i.e. n flops per point against 16 to 32 bytes of
// traffic; at the 70 TFLOP/s that chained products reach here and 5 TB/s the two meet near
// n = 300.  Measured (us): lengths that are no power of two, which were direct sums, 192^3 500 per
// component and axis -> 150 per axis of three components (products 63, traffic 68); its eps sums
// (45) ride along.  Powers of two up to 128, which were LDS transforms: 128^3 54 per axis -> 45 and
// no eps pass (18), 32^3 nine launches of 5 -> three of 7.  At 256 points the products lose
// (1.43 against 1.20 ms for the readout of 256^3), at 512 the register transform is faster still.
// Spectrum: only the kappa_x >= 0 half of the modes is formed; 192^3 nine passes of 3780 ->
// 133 + 141 + 167 (x, y, z, three components each); 128^3 likewise.
#include <algorithm>
#include <cmath>

#include "cnsf_impl.h"
#include "diag_common.h"
#include "lines.h"

namespace cnsf {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int LT = 256;            // threads per block of the derivative: four waves
constexpr int LG = 16;             // lines per group
constexpr int LROW = LG + 1;       // LDS row of one point: sixteen lines and a pad

__host__ __device__ inline int half_rows(int n) { return (n / 2 + 1 + 7) / 8 * 8; }   // m = 0 .. n/2, pairs of k-steps

// First point of line l along an axis of a box with rows of nx points.
__device__ inline uint32_t line_first(uint32_t l, int axis, uint32_t nx, uint32_t nxy) {
  if (axis == 0) return l * nx;
  if (axis == 1) return (l / nx) * nxy + (l % nx);
  return l;
}

// Groups of one block, XCD-contiguous: gridDim.x is a multiple of 8.
__device__ inline void group_range(uint32_t groups, uint32_t& begin, uint32_t& end, uint32_t& step) {
  const uint32_t x = blockIdx.x & 7u, per = (groups + 7u) / 8u;
  begin = x * per + (blockIdx.x >> 3);
  end = min(groups, (x + 1u) * per);
  step = gridDim.x >> 3;
}

// d_a of the component blockIdx.y along one axis, times its sign, into or onto its accumulator;
// a component that completes its field (eps >= 0) adds mu field^2 to this block's partial
// instead.  Along x the operands change places, so that the lanes of a result row run along x.
template <bool XAX>
__global__ void __launch_bounds__(LT, 4) k_deriv_lines(const double* __restrict__ fields_in, double* __restrict__ fields,
                                                    const LineDeriv ld, DiagPartial* __restrict__ partials) {
  extern __shared__ double lsh[];
  const int n = (int)ld.n, H = n / 2, K = half_rows(n);
  const bool even = (n & 1) == 0;
  const int rows = even ? H : H + 1, JT = (rows + 15) / 16;   // row n/2 of an even length is summed apart
  double* E = lsh;                      // E[m * LROW + line]
  double* O = E + K * LROW;
  double* dt = O + K * LROW;            // d(i - K) / 2
  double* red = dt + (2 * K + JT * 16 + 1);
  const LineComp lc = ld.c[blockIdx.y];
  const double* u = fields_in + lc.in;
  double* acc = fields + lc.out;
  const double* mu = fields_in + ld.mu;
  const uint32_t ngroups = (ld.nlines + LG - 1) / LG;
  uint32_t gb, ge, gs;
  group_range(ngroups, gb, ge, gs);
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  double esum = 0.0;
  if (gb < ge) {
    // d(m) = (pi / L) (-1)^m cot(pi m / n) for even n, csc for odd; d(0) = 0.  Odd in m, period n.
    for (int i = tid; i < 2 * K + JT * 16 + 1; i += LT) {
      const int m = ((i - K) % n + n) % n;
      double s, c;
      sincospi((double)m / (double)n, &s, &c);
      dt[i] = m == 0 ? 0.0 : 0.25 * ld.kscale * ((m & 1) ? -1.0 : 1.0) * (even ? (2 * m == n ? 0.0 : c / s) : 1.0 / s);
    }
    for (int i = (H + 1) * LROW + tid; i < K * LROW; i += LT) E[i] = O[i] = 0.0;   // rows past n/2
  }
  for (uint32_t grp = gb; grp < ge; grp += gs) {
    const uint32_t l0 = grp * LG;
    __syncthreads();   // table and pads in; the last group's rows consumed
    // eight loads in flight per thread; lines past the last one repeat it (columns do not mix)
    if constexpr (XAX) {
      const double* z[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) z[q] = u + (uint64_t)min(l0 + 4 * wave + q, ld.nlines - 1) * n;
      for (int m = lane; m <= H; m += 64) {
        const int mm = m == 0 || 2 * m == n ? -1 : n - m;
        double a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[q] = z[q][m];
          b[q] = z[q][mm < 0 ? m : mm];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          E[m * LROW + 4 * wave + q] = mm < 0 ? a[q] : a[q] + b[q];
          O[m * LROW + 4 * wave + q] = mm < 0 ? 0.0 : a[q] - b[q];
        }
      }
    } else {
      const double* z = u + line_first(min(l0 + l16, ld.nlines - 1), ld.axis, ld.nx, ld.nxy);
      for (int m0 = tid >> 4; m0 <= H; m0 += 4 * (LT / 16)) {
        double a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = min(m0 + q * (LT / 16), H);
          a[q] = z[(uint64_t)m * ld.stride];
          b[q] = z[(uint64_t)(m == 0 ? 0 : n - m) * ld.stride];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = min(m0 + q * (LT / 16), H);   // the last rows may be written twice, alike
          const bool self = m == 0 || 2 * m == n;
          E[m * LROW + l16] = self ? a[q] : a[q] + b[q];
          O[m * LROW + l16] = self ? 0.0 : a[q] - b[q];
        }
      }
    }
    __syncthreads();
    // one result: stored, added to the accumulator's value `old`, or summed into eps
    auto put = [&](uint32_t a, double v, double old, double m) {
      v *= lc.sign;
      if (!lc.init) v = old + v;
      if (lc.eps >= 0) esum += m * v * v;
      else acc[a] = v;
    };
    // which wave starts with tile 0 changes from block to block: the same SIMD would get the odd tiles
    for (int t = (wave + (int)blockIdx.x) & 3; t < JT; t += LT / 64) {
      const int j0 = 16 * t;
      f64x4 P = {0.0, 0.0, 0.0, 0.0}, R = {0.0, 0.0, 0.0, 0.0};
      // where the tile's results go, and what is there: in flight during the product
      uint32_t at[8];
      double old[8], mv[8];
      bool on[8];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 4 * v + lq;
        const int j = j0 + (XAX ? l16 : row);
        const uint32_t l = l0 + (XAX ? row : l16);
        const bool in = j < rows && l < ld.nlines;
        const uint32_t b = in ? line_first(l, ld.axis, ld.nx, ld.nxy) : 0;
        at[v] = in ? b + (uint32_t)j * ld.stride : 0;
        at[4 + v] = in && j > 0 ? b + (uint32_t)(n - j) * ld.stride : 0;
        on[v] = in;
        on[4 + v] = in && j > 0;
      }
      if (!lc.init)
#pragma unroll
        for (int v = 0; v < 8; ++v) old[v] = acc[at[v]];
      if (lc.eps >= 0)
#pragma unroll
        for (int v = 0; v < 8; ++v) mv[v] = mu[at[v]];
      const double* d1 = dt + K + j0 + l16 - lq;
      const double* d2 = dt + K + j0 + l16 + lq;
      const double *e = E + lq * LROW + l16, *o = O + lq * LROW + l16;
      // two k-steps at a time (the compiler does not unroll loops with matrix instructions)
      if constexpr (XAX) {
        for (int m = 0; m < K; m += 8) {
#pragma unroll
          for (int q = 0; q < 8; q += 4) {
            const double c1 = d1[-(m + q)], c2 = d2[m + q];
            P = __builtin_amdgcn_mfma_f64_16x16x4f64(e[(m + q) * LROW], c1 + c2, P, 0, 0, 0);
            R = __builtin_amdgcn_mfma_f64_16x16x4f64(o[(m + q) * LROW], c1 - c2, R, 0, 0, 0);
          }
        }
      } else {
        for (int m = 0; m < K; m += 8) {
#pragma unroll
          for (int q = 0; q < 8; q += 4) {
            const double c1 = d1[-(m + q)], c2 = d2[m + q];
            P = __builtin_amdgcn_mfma_f64_16x16x4f64(c1 + c2, e[(m + q) * LROW], P, 0, 0, 0);
            R = __builtin_amdgcn_mfma_f64_16x16x4f64(c1 - c2, o[(m + q) * LROW], R, 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (on[v]) put(at[v], P[v] + R[v], old[v], mv[v]);
        if (on[4 + v]) put(at[4 + v], R[v] - P[v], old[4 + v], mv[4 + v]);
      }
    }
    if (even) {
      // point n/2: sum_m o_m d(n/2 - m), sixteen partial sums per line
      double s = 0.0;
      for (int m = 1 + (tid >> 4); m < H; m += LT / 16) s += O[m * LROW + l16] * dt[K + H - m];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (lane < 16) red[wave * 16 + lane] = s;
      __syncthreads();
      if (tid < LG && l0 + tid < ld.nlines) {
        const double r = 2.0 * (((red[tid] + red[16 + tid]) + red[32 + tid]) + red[48 + tid]);
        const uint32_t a = line_first(l0 + tid, ld.axis, ld.nx, ld.nxy) + (uint32_t)H * ld.stride;
        put(a, r, lc.init ? 0.0 : acc[a], lc.eps >= 0 ? mu[a] : 0.0);
      }
    }
  }
  if (lc.eps >= 0) {
    esum = wave_sum(esum);
    __syncthreads();
    if (lane == 0) red[wave] = esum;
    __syncthreads();
    if (tid == 0) {
      const double s = ((red[0] + red[1]) + red[2]) + red[3];
      for (uint32_t b = blockIdx.x; b < LINE_PARTIALS; b += gridDim.x) {   // the others of the quarter stay neutral
        DiagPartial& P = partials[lc.eps * LINE_PARTIALS + b];
        const double v = b == blockIdx.x ? s : 0.0;
        if (ld.full) {
          DiagPartial p;
          part_zero(p);
          P = p;
        }
        P.eps_s = lc.eps_d ? 0.0 : v;
        P.eps_d = lc.eps_d ? v : 0.0;
      }
    }
  }
}

bool deriv_lines_serves(uint32_t n) {
  const bool pow2 = (n & (n - 1)) == 0;
  return pow2 ? n <= 128 : n <= 1024;
}

// Blocks along x of a grid with `ny` more: one round of the CUs' slots, every block the same
// number of groups (1536 blocks on 1280 slots took 1.3 times as long as 1152).
static uint32_t line_blocks(uint32_t nlines, size_t lds, int threads, uint32_t ny, uint32_t most) {
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const uint32_t per_cu = std::max(1u, std::min((uint32_t)(163840 / std::max<size_t>(lds, 1)), 1024u / (uint32_t)threads));
  const uint32_t slots = std::max(8u, std::min(most, (uint32_t)cus * per_cu / ny) / 8u * 8u);
  const uint32_t groups = (nlines + LG - 1) / LG, each = (groups + slots - 1) / slots;
  return std::min(slots, ((groups + each - 1) / each + 7u) / 8u * 8u);
}

hipError_t launch_deriv_lines(const LineDeriv& ld, double* fields, DiagPartial* partials, hipStream_t s) {
  const int n = (int)ld.n, K = half_rows(n), rows = n % 2 ? n / 2 + 1 : n / 2, JT = (rows + 15) / 16;
  const size_t lds = ((size_t)2 * K * LROW + 2 * K + JT * 16 + 1 + 64) * sizeof(double);
  const void* k = ld.axis == 0 ? (const void*)k_deriv_lines<true> : (const void*)k_deriv_lines<false>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid(line_blocks(ld.nlines, lds, LT, 3, LINE_PARTIALS), 3);
  if (ld.axis == 0)
    hipLaunchKernelGGL(k_deriv_lines<true>, grid, dim3(LT), lds, s, (const double*)fields, fields, ld, partials);
  else
    hipLaunchKernelGGL(k_deriv_lines<false>, grid, dim3(LT), lds, s, (const double*)fields, fields, ld, partials);
  return hipGetLastError();
}

// ------------------------------------------------------------------ shell spectrum
// Forward transform along one axis.  Axis x: a real line to its n/2 + 1 independent modes
// (X_{n-k} is the conjugate of X_k), so the arrays of the y and z passes have rows of nxh =
// nx/2 + 1 complex points; axis y in place; axis z adds |X|^2 escale of the three components
// to the energy instead.  blockIdx.y: the component (x, y).
template <int AXIS>
__global__ void __launch_bounds__(AXIS == 0 ? 256 : 512) k_dft_lines(const double* __restrict__ real_in, double2* __restrict__ data,
                                                  double* __restrict__ energy, const LineDft ld) {
  extern __shared__ double lsh[];
  const int n = (int)ld.n, H = n / 2, K = half_rows(n);
  const int JT = (H + 1 + 15) / 16;
  constexpr int PARTS = AXIS == 0 ? 2 : 4;
  constexpr int LT = AXIS == 0 ? 256 : 512;   // four parts fill twice the LDS: more waves to a block instead of blocks
  double* F = lsh;                        // even real, odd real (even imaginary, odd imaginary): F[p][m * LROW + line]
  double2* cs = (double2*)(lsh + ((PARTS * K * LROW + 1) & ~1));   // exp(i 2 pi m / n)
  const int FS = K * LROW;
  const uint32_t ngroups = (ld.nlines + LG - 1) / LG;
  uint32_t gb, ge, gs;
  group_range(ngroups, gb, ge, gs);
  if (gb >= ge) return;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  for (int m = tid; m < n; m += LT) {
    double s, c;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    cs[m] = make_double2(c, s);
  }
  for (int i = (H + 1) * LROW + tid; i < K * LROW; i += LT)
#pragma unroll
    for (int p = 0; p < PARTS; ++p) F[p * FS + i] = 0.0;
  for (uint32_t grp = gb; grp < ge; grp += gs) {
    const uint32_t l0 = grp * LG;
    for (int c = AXIS == 2 ? 0 : (int)blockIdx.y; c < (AXIS == 2 ? 3 : (int)blockIdx.y + 1); ++c) {
      const double* in = real_in + (uint64_t)c * ld.real_size;
      double2* dat = data + (uint64_t)c * ld.size;
      __syncthreads();
      if constexpr (AXIS == 0) {
        const double* z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) z[q] = in + (uint64_t)min(l0 + 4 * wave + q, ld.nlines - 1) * n;
        for (int m = lane; m <= H; m += 64) {
          const int mm = m == 0 || 2 * m == n ? -1 : n - m;
          double a[4], b[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            a[q] = z[q][m];
            b[q] = z[q][mm < 0 ? m : mm];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            F[m * LROW + 4 * wave + q] = mm < 0 ? a[q] : a[q] + b[q];
            F[FS + m * LROW + 4 * wave + q] = mm < 0 ? 0.0 : a[q] - b[q];
          }
        }
      } else {
        const double2* z = dat + line_first(min(l0 + l16, ld.nlines - 1), AXIS, ld.nxh, ld.plane);
        for (int m0 = tid >> 4; m0 <= H; m0 += 4 * (LT / 16)) {
          double2 a[4], b[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = min(m0 + q * (LT / 16), H);
            a[q] = z[(uint64_t)m * ld.stride];
            b[q] = z[(uint64_t)(m == 0 ? 0 : n - m) * ld.stride];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = min(m0 + q * (LT / 16), H);   // the last rows may be written twice, alike
            const bool self = m == 0 || 2 * m == n;
            double* f = F + m * LROW + l16;
            f[0] = self ? a[q].x : a[q].x + b[q].x;
            f[FS] = self ? 0.0 : a[q].x - b[q].x;
            f[2 * FS] = self ? a[q].y : a[q].y + b[q].y;
            f[3 * FS] = self ? 0.0 : a[q].y - b[q].y;
          }
        }
      }
      __syncthreads();
      for (int t = (wave + (int)blockIdx.x) & (LT / 64 - 1); t < JT; t += LT / 64) {
        const int j0 = 16 * t;
        // coefficient exp(i 2 pi j m / n) of j = j0 + l16, m = 4 step + lq
        const uint32_t j = (uint32_t)(j0 + l16) % (uint32_t)n;
        uint32_t idx = (j * (uint32_t)lq) % (uint32_t)n;
        const uint32_t step = (4u * j) % (uint32_t)n;
        f64x4 A[PARTS];
#pragma unroll
        for (int p = 0; p < PARTS; ++p) A[p] = {0.0, 0.0, 0.0, 0.0};
        const double* f = F + lq * LROW + l16;
        for (int m = 0; m < K; m += 8) {
#pragma unroll
          for (int q = 0; q < 8; q += 4) {
            const double2 w = cs[idx];
            idx += step;
            idx -= idx >= (uint32_t)n ? (uint32_t)n : 0u;
#pragma unroll
            for (int p = 0; p < PARTS; ++p) {
              const double v = f[p * FS + (m + q) * LROW], k = (p & 1) ? w.y : w.x;
              if constexpr (AXIS == 0) A[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, k, A[p], 0, 0, 0);
              else A[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(k, v, A[p], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 4 * v + lq;
          const int jj = j0 + (AXIS == 0 ? l16 : row);
          const uint32_t l = l0 + (AXIS == 0 ? row : l16);
          if (jj > H || l >= ld.nlines) continue;
          if constexpr (AXIS == 0) {
            dat[(uint64_t)l * ld.nxh + jj] = make_double2(A[0][v], -A[1][v]);
          } else {
            const uint64_t b = line_first(l, AXIS, ld.nxh, ld.plane);
            const double2 X = make_double2(A[0][v] + A[3][v], A[2][v] - A[1][v]);
            const double2 Y = make_double2(A[0][v] - A[3][v], A[2][v] + A[1][v]);   // mode n - j
            const uint64_t ax = b + (uint64_t)jj * ld.stride, ay = b + (uint64_t)(n - jj) * ld.stride;
            const bool two = jj > 0 && 2 * jj != n;
            if constexpr (AXIS == 1) {
              dat[ax] = X;
              if (two) dat[ay] = Y;
            } else {
              const double ex = (X.x * X.x + X.y * X.y) * ld.escale, ey = (Y.x * Y.x + Y.y * Y.y) * ld.escale;
              energy[ax] = c ? energy[ax] + ex : ex;
              if (two) energy[ay] = c ? energy[ay] + ey : ey;
            }
          }
        }
      }
    }
  }
}

bool dft_lines_serves(uint32_t n) { return n >= 6 && n < 512; }

hipError_t launch_dft_lines(uint32_t n, double* fields, hipStream_t s) {
  const uint64_t N = (uint64_t)n * n * n;
  const uint32_t nxh = n / 2 + 1;
  const int K = half_rows((int)n);
  for (int a = 0; a < 3; ++a) {
    LineDft ld{};
    ld.n = n;
    ld.nxh = nxh;
    ld.plane = nxh * n;
    ld.stride = a == 1 ? nxh : nxh * n;
    ld.nlines = a == 0 ? n * n : nxh * n;
    ld.real_size = N;
    ld.size = (uint64_t)nxh * n * n;
    ld.escale = 0.5 / ((double)N * (double)N);
    const int parts = a == 0 ? 2 : 4;
    const size_t lds = ((size_t)((parts * K * LROW + 1) & ~1) + 2 * (size_t)n) * sizeof(double);
    const int threads = a == 0 ? 256 : 512;
    const uint32_t ny = a == 2 ? 1 : 3, blocks = line_blocks(ld.nlines, lds, threads, ny, 1u << 20);
    const void* k = a == 0 ? (const void*)k_dft_lines<0> : a == 1 ? (const void*)k_dft_lines<1> : (const void*)k_dft_lines<2>;
    if (lds > 65536) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    double2* data = (double2*)(fields + 4 * N);
    const dim3 grid(blocks, ny);
    if (a == 0) hipLaunchKernelGGL(k_dft_lines<0>, grid, dim3(threads), lds, s, (const double*)fields, data, fields, ld);
    else if (a == 1) hipLaunchKernelGGL(k_dft_lines<1>, grid, dim3(threads), lds, s, (const double*)fields, data, fields, ld);
    else hipLaunchKernelGGL(k_dft_lines<2>, grid, dim3(threads), lds, s, (const double*)fields, data, fields, ld);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace cnsf
