// Several updates per launch for thin lattices (shock tubes, Couette channels, columns).
//
// A lattice of a few thousand cells leaves the chip idle: an update is one launch whose time is the
// latency of one cell (load 98 values, collide, store) plus the gap to the next launch, 5 to 7 us
// whatever the size.  Here a block of 256 threads holds a window of whole y-z cross-sections in
// registers, one cell per thread, and advances it `steps` times, links between neighbours going
// through LDS, before it stores its middle planes: one plane at either end of the window becomes
// stale per update, so neighbouring windows overlap by 2 steps planes and compute those twice, on
// compute units that would idle otherwise.  No block waits for another.  Windows read what their
// neighbours would overwrite, so a launch writes a second array and the next one comes back; a
// lattice that fits one window needs neither and makes all its updates in one launch.
// Stored values pass through the storage format after every update and the ends act as in the
// single update, so the results are the same bit for bit; launches make even numbers of updates,
// because an equilibrium end enters 16-bit storage rounded only every second update.
//
// Measured on MI355X (us per update, single updates in a replayed graph -> windows): FP32 16 x 4 x 4
// (one window) 4.9 -> 2.2, Sod 256 x 4 x 4 5.0 -> 3.6, Becker 1024 x 4 x 4 6.3 -> 4.3, 1024 x 1 x 1 4.7 ->
// 2.3; FP16 Sod 256 7.8 -> 4.0.  What bounds it: an update is 2.2 to 2.65 us of one wave per SIMD (750 vector
// instructions at 4 cycles, 168 LDS accesses, two barriers), a launch with its loads and stores
// 5.3 us and more (Sod: 15.9 us with four updates, 21.2 with six).
#include <algorithm>

#include "cnsf_impl.h"
#include "launch.h"

namespace cnsf {

constexpr int TUBE_THREADS = 256;

// No-slip link, rounded to FP32: fused with the conversion to 16 bits that follows (v_fma_mixlo_f16
// rounds once) one value in ten thousand would differ from the single update's.
__device__ inline float wall_link(int k, float v, int s, const Geom& g, const Phys& ph, const WallCell& w) {
  float r = noslip_link(k, v, s, g, ph, w);
  asm volatile("" : "+v"(r));
  return r;
}

template <int ST, bool SC>
__device__ inline typename Store<ST>::T tube_code(const Codec& cd, int k, float v) {
  if (ST != 0 && SC) v *= cd.inv_scale[k];
  return Store<ST>::enc(v);
}
template <int ST, bool SC>
__device__ inline float tube_value(const Codec& cd, int k, typename Store<ST>::T c) {
  float v = Store<ST>::dec(c);
  if (ST != 0 && SC) v *= cd.scale[k];
  return v;
}

// Window of `xw` planes (xw * ny * nz <= 256), of which the block stores planes
// [blockIdx.x * keep, + keep); xw == nx: the whole lattice (one block, src may be dst).
template <int ST, int BC, bool SC>
__global__ void __launch_bounds__(TUBE_THREADS, 1)
k_tube(const typename Store<ST>::T* src, typename Store<ST>::T* dst, const Geom g, const Phys ph, const Codec cd,
       int xw, int keep, int steps) {
  using T = typename Store<ST>::T;
  __shared__ T link[6 * NC * TUBE_THREADS];   // outgoing links of every thread's cell
  const int nx = (int)g.nx, ny = (int)g.ny, nz = (int)g.nz;
  const int tid = (int)threadIdx.x, yz = tid / xw, xi = tid % xw;
  const bool live = yz < ny * nz, whole = xw == nx;
  const int x0 = (int)blockIdx.x * keep;
  int xs = whole ? 0 : x0 - steps;                       // first plane of the window
  if (BC != 0 && !whole) xs = max(0, min(xs, nx - xw));  // the ends of the lattice need no overlap
  int x = xs + xi;
  if (BC == 0) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
  const uint32_t cell = live ? (uint32_t)x + (uint32_t)nx * (uint32_t)yz : 0u;
  const bool first = BC != 0 && x == 0, last = BC != 0 && x == nx - 1;
  // threads whose links arrive here (a stale end of the window reads itself)
  int from[6];
  {
    const int y = yz % ny, z = yz / ny;
    const bool wrap = BC == 0 && whole;
    from[0] = xi > 0 ? tid - 1 : (wrap ? tid + xw - 1 : tid);
    from[1] = xi < xw - 1 ? tid + 1 : (wrap ? tid - (xw - 1) : tid);
    from[2] = y > 0 ? tid - xw : tid + (ny - 1) * xw;
    from[3] = y < ny - 1 ? tid + xw : tid - (ny - 1) * xw;
    from[4] = z > 0 ? tid - ny * xw : tid + (nz - 1) * ny * xw;
    from[5] = z < nz - 1 ? tid + ny * xw : tid - (nz - 1) * ny * xw;
    if (!live)
#pragma unroll
      for (int i = 0; i < 6; ++i) from[i] = tid;
  }
  float f[NC][NV];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const __amdgpu_buffer_rsrc_t rs = component_rsrc<ST>(src, g, k);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float v = buf_load<ST>(rs, slot_offset<ST>(g, i, cell));
      if (ST != 0 && SC) v *= cd.scale[k];
      f[k][i] = v;
    }
  }
  for (int s = 0; s < steps; ++s) {
    WallCell wc{};
    update_cell(f, cd, ph, nullptr, BC == 3 ? &wc : nullptr);
    float end[NC];   // the link that enters through an end, from what the cell sent there
    if constexpr (BC != 0) {
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        float v = first ? f[k][2] : f[k][1];
        if (BC == 3) v = wall_link(k, v, first ? 0 : 1, g, ph, wc);
        if (BC == 2) v = first ? g.dev_left[k] : g.dev_right[k];
        if (BC == 2 && (s & 1) == 0) {
          end[k] = v;   // enters unrounded after the first, third, ... update
        } else {
          v = tube_value<ST, SC>(cd, k, tube_code<ST, SC>(cd, k, v));
          end[k] = BC == 1 && x_odd(k) ? -v : v;
        }
      }
      // one plane between two ends: its other link
      if (nx == 1) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          float v = f[k][1];
          if (BC == 3) v = wall_link(k, v, 1, g, ph, wc);
          if (BC == 2) v = g.dev_right[k];
          if (!(BC == 2 && (s & 1) == 0)) {
            v = tube_value<ST, SC>(cd, k, tube_code<ST, SC>(cd, k, v));
            if (BC == 1 && x_odd(k)) v = -v;
          }
          f[k][1] = v;   // kept here: no neighbour takes it
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      f[k][0] = tube_value<ST, SC>(cd, k, tube_code<ST, SC>(cd, k, f[k][0]));
#pragma unroll
      for (int i = 0; i < 6; ++i) link[(i * NC + k) * TUBE_THREADS + tid] = tube_code<ST, SC>(cd, k, f[k][i + 1]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const float other = f[k][1];
#pragma unroll
      for (int i = 0; i < 6; ++i)
        f[k][i + 1] = tube_value<ST, SC>(cd, k, link[(i * NC + k) * TUBE_THREADS + from[i]]);
      if constexpr (BC != 0) {
        if (last) f[k][2] = nx == 1 ? other : end[k];
        if (first) f[k][1] = end[k];
      }
    }
    __syncthreads();   // the links are consumed
  }
  if (!live || x < x0 || x >= x0 + keep || (BC == 0 && !whole && (xi < steps || xi >= xw - steps))) return;
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const __amdgpu_buffer_rsrc_t rs = component_rsrc<ST>(dst, g, k);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float v = f[k][i];
      if (ST != 0 && SC) v *= cd.inv_scale[k];
      // a value that went through the storage format comes back to its code; fused with the conversion to FP16 the
      // product gains + 0, and a negative zero (an update's underflow) would lose its sign
      if (ST == 1 && SC) asm volatile("" : "+v"(v));
      buf_store<ST>(rs, slot_offset<ST>(g, i, cell), v);
    }
  }
}

// Windows of a lattice: planes a window holds, and the even number of updates per launch that is fastest, if
// that beats single updates.  A launch of s updates takes (us, within 10% over cross-sections of 1 to 32 cells,
// 64 to 3000 planes) 8.0 + 2.03 s + 0.27 per MB read and written, 16-bit 8.0 + 2.45 s + 0.45; single updates take
// 4.0 + 0.095 per thousand cells, 16-bit 4.6 + 0.043.  Measured (us per update, windows / single): FP32 4 x 4
// cross-sections of 64, 256, 1024 and 3000 planes 3.2 / 4.0, 3.7 / 4.3, 4.4 / 5.4 and, left, 10.9 / 8.7; left too
// FP32 5 x 4 4.8 / 4.3 and 4 x 6 5.2 / 4.4 of 256 planes, FP16 4 x 6 of 256 and 1024 5.3 / 4.7 and 9.6 / 5.5.
bool tube_plan(const Geom& g, int storage, int cus, TubePlan* out) {
  const uint32_t cross = g.ny * g.nz;
  if (cross > TUBE_THREADS / 4u) return false;
  const int most = TUBE_THREADS / (int)cross, nx = (int)g.nx;
  if (nx <= most) {
    *out = TubePlan{nx, 1 << 20, 4, 0.0};
    return true;
  }
  const bool fp32 = storage == 0;
  // Short calls: windows go out and come back, two launches (us per call among others, windows / single, the
  // worst of FP32 and 16-bit, walls and periodic): 4 updates of 1024 x 1 x 1 18.8 / 20.2, 3000 x 2 x 2 22.8 / 22.0,
  // but 1024 x 4 x 2 23.5 / 19.9 and 1024 x 4 x 4 32.4 / 22.3.  From 6 on the queue tells: 1024 x 4 x 4 36.7 / 33.2
  // among others, but with a readout after it, as most calls of a few updates have, 101 / 143 (64 x 4 x 4
  // 58 / 110; 4 updates 54 / 54).
  const int least = most >= 64 ? 4 : 6;
  const double cell_mb = NP * (fp32 ? 4e-6 : 2e-6);
  double best = 1e300;
  for (int s = 2; 2 * s < most && s <= 64; s += 2) {
    const int keep = most - 2 * s, blocks = (nx + keep - 1) / keep, rounds = (blocks + cus - 1) / cus;
    const double mb = cell_mb * ((double)blocks * TUBE_THREADS + g.ncells);
    const double t = (rounds * (8.0 + (fp32 ? 2.03 : 2.45) * s) + (fp32 ? 0.27 : 0.45) * mb) / s;
    if (t < best) {
      best = t;
      *out = TubePlan{most, s, least, 0.0};
    }
  }
  out->gain = (fp32 ? 4.0 + 9.5e-5 * g.ncells : 4.6 + 4.3e-5 * g.ncells) - best;
  return out->gain > 0.0;
}

template <int ST, int BC, bool SC>
static hipError_t launch_tube_t(const void* src, void* dst, const Geom& g, const Phys& ph, const Codec& cd, int xw,
                                int steps, hipStream_t s) {
  using T = typename Store<ST>::T;
  const int nx = (int)g.nx, keep = xw == nx ? nx : xw - 2 * steps;
  hipLaunchKernelGGL((k_tube<ST, BC, SC>), dim3((nx + keep - 1) / keep), dim3(TUBE_THREADS), 0, s, (const T*)src, (T*)dst,
                     g, ph, cd, xw, keep, steps);
  return hipGetLastError();
}

hipError_t launch_tube(int storage, const void* src, void* dst, const Geom& g, const Phys& ph, const Codec& cd, int xw,
                       int steps, hipStream_t s) {
  if (steps < 2 || (steps & 1) || (xw != (int)g.nx && 2 * steps >= xw)) return hipErrorInvalidValue;
  const bool sc = cd.scaled != 0;
#define CNSF_CASE(ST, BC, SC) \
  if (storage == ST && g.bc_x == BC && sc == SC) return launch_tube_t<ST, BC, SC>(src, dst, g, ph, cd, xw, steps, s);
  CNSF_CASE(0, 0, false) CNSF_CASE(0, 1, false) CNSF_CASE(0, 2, false) CNSF_CASE(0, 3, false)
  CNSF_CASE(1, 0, false) CNSF_CASE(1, 1, false) CNSF_CASE(1, 2, false) CNSF_CASE(1, 3, false)
  CNSF_CASE(2, 0, false) CNSF_CASE(2, 1, false) CNSF_CASE(2, 2, false) CNSF_CASE(2, 3, false)
  CNSF_CASE(1, 0, true) CNSF_CASE(1, 1, true) CNSF_CASE(1, 2, true) CNSF_CASE(1, 3, true)
  CNSF_CASE(2, 0, true) CNSF_CASE(2, 1, true) CNSF_CASE(2, 2, true) CNSF_CASE(2, 3, true)
#undef CNSF_CASE
  return hipErrorInvalidValue;
}

}  // namespace cnsf
