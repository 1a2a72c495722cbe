// Two updates in one pass over memory, for periodic lattices at an even time level.
//
// The single update moves every population through HBM twice per step (784 bytes per FP32 cell)
// and is bound by that.  Here a block advances a column of the lattice by two steps while its
// populations are on the chip: it walks a tile of columns plane by plane along z, collides plane
// z of level t (the columns around the tile too: D3Q7 needs the four faces, no corners), hands
// the links on through LDS (x and y) and per-thread storage (z), collides plane z - 1 of level
// t + 1 from them and streams the result into the neighbours' slots, i.e. level t + 2 in the
// layout of an even level.  Stored values pass through the storage format between the two
// steps, so the result is that of two single updates bit for bit.
//
// A pass reads and writes other memory (neighbouring tiles read what a tile would overwrite):
//  * the whole lattice into a second array of its size and back in the next pass, or
//  * for large lattices, slab by slab into the place `split` planes further down, the first
//    planes into a workspace of `split` planes: slab s overwrites planes that slab s - 1 was the
//    last to read.  The next pass goes the other way, from the top, and brings every plane home.
// Passes therefore come in pairs, four updates, and between calls the array is as it always is.
// The periodic end in z is the one place where order matters: the plane that the last slab
// reads across the end is copied aside first, and the links that the first slab sends across it
// are parked until their plane is free.
//
// Tile.  At most 256 columns: 64 x 4 (or whole rows of up to 96 cells) take four waves, and up to 192
// ring columns two or three more; 6 or 7 waves of up to 256 registers and 91 (FP32: 154) KiB of LDS
// are one block per CU.  Every x-row of a tile also touches the 128-byte lines of its two ring
// cells, which are whole lines of the neighbouring tiles: they are cheap only while both blocks
// are at the same plane and the line is in their XCD's L2 (tiles of one XCD are a contiguous
// patch).  Tiles of 64 x 4 fetch less than 32 x 8, and non-temporal stores, which keep the written planes from
// pushing those lines out, less again: 512^3 FP32 fetches 1.45 to 1.61 times the array per pass (by the
// allocation; FP16 1.18 times).
// The next plane's loads are issued before the second collision: 14.5 -> 13.9 ms per update
// (same array), 16-bit 10.9 -> 8.4.
// Measured on MI355X per update, single updates -> pairs: 512^3 FP32 17.5 -> 10.9 ms on a fast
// array, 20.8 -> 13.7 ms on a plain one; FP16 10.5 -> 8.0 ms (plain); 256^3 FP32 2.61 -> 1.54 ms,
// FP16 1.28 -> 0.94 ms; 128^3 FP32 0.337 -> 0.194 ms.  What bounds it now: FP32 the fetch above
// (vector units busy 29% of a pass at 256^3), 16-bit the vector units (58%: 7 + 4 wave collisions per 256
// cells, three of them on the fullest SIMD).
#include <algorithm>
#include <type_traits>

#include "cnsf_impl.h"
#include "launch.h"

namespace cnsf {

constexpr int PNI = 256;          // interior threads: tiles of at most as many columns
constexpr int PNR = 192;          // ring threads at most

// Ring columns of tiles of tx x ty: a tile as wide as the lattice has its neighbours along x inside.
__host__ __device__ inline int ring_columns(int tx, int ty, int nx) { return 2 * tx + (tx == nx ? 0 : 2 * ty); }

// Where a level of the lattice is stored: planes z < split in `scr` (cell index as in the
// lattice), the others in `arr`, split planes further down than in the lattice.
template <typename T>
struct Place {
  T *arr, *scr;
  uint64_t cs_arr, cs_scr;   // elements between component regions
  int split;
};

template <typename T>
__device__ inline void plane_of(const Place<T>& p, int z, uint32_t nxy, T*& base, uint64_t& cs, uint32_t& cell0) {
  if (z < p.split) {
    base = p.scr;
    cs = p.cs_scr;
    cell0 = (uint32_t)z * nxy;
  } else {
    base = p.arr;
    cs = p.cs_arr;
    cell0 = (uint32_t)(z - p.split) * nxy;
  }
}

template <typename T>
__device__ inline __amdgpu_buffer_rsrc_t region_rsrc(T* base, uint64_t cs, int k) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (uint64_t)k * cs), (short)0, (int)(uint32_t)(cs * sizeof(T)),
                                           BUF_WORD3);
}

// The stored code as it is (16-bit codes are decoded only when they are needed: a conversion
// right after the load would wait for it).
template <int ST>
__device__ inline typename Store<ST>::T load_code(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (ST == 0) {
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
  } else {
    return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
  }
}

template <int ST, bool NT>
__device__ inline void store_pop(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
  constexpr int AUX = NT ? 2 : 0;   // 2: non-temporal
  if constexpr (ST == 0) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, (int)off, 0, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b16((short)Store<ST>::enc(v), r, (int)off, 0, AUX);
  }
}

// What a store to the array and a load from it do to a shifted population.
template <int ST, bool SC>
__device__ inline typename Store<ST>::T encode(const Codec& cd, int k, float v) {
  if (ST != 0 && SC) v *= cd.inv_scale[k];
  return Store<ST>::enc(v);
}
template <int ST, bool SC>
__device__ inline float decode(const Codec& cd, int k, typename Store<ST>::T c) {
  float v = Store<ST>::dec(c);
  if (ST != 0 && SC) v *= cd.scale[k];
  return v;
}

// LDS of a block: links along x and y of the last two planes collided, by destination cell, and
// links kept by their own thread: rest links (the last RB planes, by z mod RB) and +z links (the
// last UB planes, by z mod UB).  16-bit links leave room to store a plane's own while the older ones
// are still needed; FP32 links wait in registers until those are consumed.
template <int ST>
struct PairLds {
  using T = typename Store<ST>::T;
  static constexpr bool EARLY = ST != 0;
  static constexpr int RB = EARLY ? 2 : 1, UB = EARLY ? 3 : 2;
  T xl[2][NC * 4 * PNI];
  T zl[NC * (RB + UB) * PNI];
};

// One block: planes [za, zb) of the tile at (x0, y0) of tiles tx x ty, za - 1 and zb being read too.
// Plane wrap_z (one past an end) is read from `wrap`, the links to plane over_z are written to `over`.
template <int ST, bool SC, bool NT>
__device__ inline void pair_block(PairLds<ST>& sh, const Place<typename Store<ST>::T> src,
                                  const Place<typename Store<ST>::T> dst, const Geom& g, const Phys& ph, const Codec& cd,
                                  int za, int zb, int x0, int y0, int tx, int ty,
                                  const typename Store<ST>::T* __restrict__ wrap, int wrap_z,
                                  typename Store<ST>::T* __restrict__ over, int over_z) {
  using T = typename Store<ST>::T;
  constexpr int NI = PNI, PF = ST == 0 ? 5 : 7;   // components fetched ahead: as many as fit 256 VGPRs
  constexpr bool EARLY = PairLds<ST>::EARLY;
  constexpr int RB = PairLds<ST>::RB, UB = PairLds<ST>::UB;
  auto& xl = sh.xl;
  auto& zl = sh.zl;
  const int w = min(tx, (int)g.nx - x0), h = min(ty, (int)g.ny - y0);
  const bool row = tx == (int)g.nx;   // whole rows: the links along x stay in the tile

  const int tid = (int)threadIdx.x;
  const bool inner = __builtin_amdgcn_readfirstlane(tid) < NI;
  int lx, ly, rdir = 0, rdst = 0;   // tile coordinates; ring threads: link they hand in and its destination
  bool live;
  if (inner) {
    lx = tid % tx;
    ly = tid / tx;
    live = lx < w && ly < h;
  } else {
    const int r = tid - NI;
    if (r < tx) { lx = r; ly = -1; rdir = 2; rdst = r; live = r < w; }
    else if (r < 2 * tx) { lx = r - tx; ly = h; rdir = 3; rdst = (h - 1) * tx + lx; live = lx < w; }
    else if (r < 2 * tx + ty) { lx = -1; ly = r - 2 * tx; rdir = 0; rdst = ly * tx; live = ly < h; }
    else { lx = w; ly = r - 2 * tx - ty; rdir = 1; rdst = ly * tx + w - 1; live = ly < h; }
    if (r >= ring_columns(tx, ty, (int)g.nx)) live = false;
  }
  int gx = x0 + lx, gy = y0 + ly;
  gx = gx < 0 ? gx + (int)g.nx : (gx >= (int)g.nx ? gx - (int)g.nx : gx);
  gy = gy < 0 ? gy + (int)g.ny : (gy >= (int)g.ny ? gy - (int)g.ny : gy);
  const uint32_t cxy = live ? (uint32_t)gy * g.nx + (uint32_t)gx : 0u;
  // in-plane neighbours of the interior column
  const uint32_t rowx = cxy - (uint32_t)gx;
  const uint32_t cxp = gx == (int)g.nx - 1 ? rowx : cxy + 1u, cxm = gx == 0 ? cxy + (g.nx - 1u) : cxy - 1u;
  const uint32_t cyp = gy == (int)g.ny - 1 ? (uint32_t)gx : cxy + g.nx;
  const uint32_t cym = gy == 0 ? cxy + (g.nxy - g.nx) : cxy - g.nx;
  const int xp = lx + 1 < w ? 1 : 1 - w, xm = lx > 0 ? -1 : w - 1;   // threads of the neighbours along x
  constexpr uint32_t DEAD = 0xFFFF0000u;   // beyond every region: loads give 0, stores are dropped

  T c[NC][NV];   // stored codes of the next plane, in flight
  const T* lbase;
  uint64_t lcs;
  uint32_t lo;
  auto aim = [&](int z) {   // where plane z of level t is
    if (z == wrap_z) {
      lbase = wrap;
      lcs = (uint64_t)NV * ((g.nxy + SLOT_GROUP - 1) / SLOT_GROUP * SLOT_GROUP);
      lo = slot_offset<ST>(g, 0, cxy);
    } else {
      T* b;
      uint32_t c0;
      plane_of(src, z < 0 ? z + (int)g.nz : (z >= (int)g.nz ? z - (int)g.nz : z), g.nxy, b, lcs, c0);
      lbase = b;
      lo = slot_offset<ST>(g, 0, c0 + cxy);
    }
    lo = live ? lo : DEAD;
  };
  auto fetch = [&](auto K0, auto K1) {
#pragma unroll
    for (int k = decltype(K0)::value; k < decltype(K1)::value; ++k) {
      const __amdgpu_buffer_rsrc_t rs = region_rsrc(lbase, lcs, k);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        c[k][i] = load_code<ST>(rs, lo + (uint32_t)(i * SLOT_GROUP * sizeof(T)));
      }
    }
  };
  aim(za - 1);
  fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, PF>{});

  for (int z = za - 1; z <= zb; ++z) {
    const bool links = z >= za && z < zb;   // the plane's x and y links are needed
    fetch(std::integral_constant<int, PF>{}, std::integral_constant<int, NC>{});
    float f[NC][NV];
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int i = 0; i < NV; ++i) f[k][i] = decode<ST, SC>(cd, k, c[k][i]);
    update_cell(f, cd, ph);
    T* const Z = zl + tid;
    const int rw = (z & 1) % RB, uw = RB + (z + UB) % UB;   // where plane z's own links go
    const int rr = ((z - 1) & 1) % RB, ur = RB + (z + 2 * UB - 2) % UB;   // plane z - 1's rest, z - 2's +z links
    T fm[NC], r0[NC], up[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      r0[k] = encode<ST, SC>(cd, k, f[k][0]);
      up[k] = encode<ST, SC>(cd, k, f[k][5]);
      fm[k] = encode<ST, SC>(cd, k, f[k][6]);
    }
    if (EARLY && inner) {
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        Z[(k * (RB + UB) + rw) * NI] = r0[k];
        Z[(k * (RB + UB) + uw) * NI] = up[k];
      }
    }
    T* xw = xl[z & 1];
    if (links) {
      if (inner) {
        T* X = xw + tid;
        if (live && (lx + 1 < w || row))
#pragma unroll
          for (int k = 0; k < NC; ++k) X[(k * 4 + 0) * NI + xp] = encode<ST, SC>(cd, k, f[k][1]);
        if (live && (lx > 0 || row))
#pragma unroll
          for (int k = 0; k < NC; ++k) X[(k * 4 + 1) * NI + xm] = encode<ST, SC>(cd, k, f[k][2]);
        if (live && ly + 1 < h)
#pragma unroll
          for (int k = 0; k < NC; ++k) X[(k * 4 + 2) * NI + tx] = encode<ST, SC>(cd, k, f[k][3]);
        if (live && ly > 0)
#pragma unroll
          for (int k = 0; k < NC; ++k) X[(k * 4 + 3) * NI - tx] = encode<ST, SC>(cd, k, f[k][4]);
      } else if (live) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          const float v = rdir == 0 ? f[k][1] : (rdir == 1 ? f[k][2] : (rdir == 2 ? f[k][3] : f[k][4]));
          xw[(k * 4 + rdir) * NI + rdst] = encode<ST, SC>(cd, k, v);
        }
      }
    }
    asm volatile("" ::: "memory");
    if (z < zb) {
      aim(z + 1);
      fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, PF>{});
    }
    asm volatile("" ::: "memory");
    // second update of plane z - 1: its links along z are in registers, along x and y in LDS
    if (z > za && inner) {
      const T* X = xl[(z - 1) & 1] + tid;
      auto load = [&](int k, float e[NV]) {
        e[0] = decode<ST, SC>(cd, k, Z[(k * (RB + UB) + rr) * NI]);
#pragma unroll
        for (int i = 1; i < 5; ++i) e[i] = decode<ST, SC>(cd, k, X[(k * 4 + i - 1) * NI]);
        e[5] = decode<ST, SC>(cd, k, Z[(k * (RB + UB) + ur) * NI]);
        e[6] = decode<ST, SC>(cd, k, fm[k]);
      };
      float dQ[NC], Q[NC], omega;
      DevPrim P;
      {
        float e[NC][NV];
#pragma unroll
        for (int k = 0; k < NC; ++k) load(k, e[k]);
        omega = cell_state(e, cd, ph, dQ, Q, P);
      }
      asm volatile("" ::: "memory");   // the links are read again below instead of being held
      // streamed into the neighbours' slots (level t + 2)
      T* base[3];
      uint64_t cs[3];
      uint32_t o[NV], d0;
      const int zp = z - 1;
      plane_of(dst, zp, g.nxy, base[0], cs[0], d0);
      o[0] = slot_offset<ST>(g, 0, d0 + cxy);
      o[1] = slot_offset<ST>(g, 1, d0 + cxp);
      o[2] = slot_offset<ST>(g, 2, d0 + cxm);
      o[3] = slot_offset<ST>(g, 3, d0 + cyp);
      o[4] = slot_offset<ST>(g, 4, d0 + cym);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int zn = zp + (j == 0 ? 1 : -1);
        if (zn == over_z) {
          // the plane across the periodic end, parked until its place is free
          base[1 + j] = over;
          cs[1 + j] = (g.nxy + SLOT_GROUP - 1) / SLOT_GROUP * SLOT_GROUP;
          o[5 + j] = cxy * (uint32_t)sizeof(T);
        } else {
          plane_of(dst, zn < 0 ? zn + (int)g.nz : (zn >= (int)g.nz ? zn - (int)g.nz : zn), g.nxy, base[1 + j], cs[1 + j], d0);
          o[5 + j] = slot_offset<ST>(g, 5 + j, d0 + cxy);
        }
      }
#pragma unroll
      for (int i = 0; i < NV; ++i) o[i] = live ? o[i] : DEAD;
      auto finish = [&](auto K) {
        constexpr int k = decltype(K)::value;
        float e[NV];
        load(k, e);
        collide_dev<k>(e, dQ, Q, P, ph, omega);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int j = i < 5 ? 0 : i - 4;
          if (ST != 0 && SC) e[i] *= cd.inv_scale[k];
          store_pop<ST, NT>(region_rsrc(base[j], cs[j], k), o[i], e[i]);
        }
      };
      finish(std::integral_constant<int, 0>{});
      finish(std::integral_constant<int, 1>{});
      finish(std::integral_constant<int, 2>{});
      finish(std::integral_constant<int, 3>{});
      finish(std::integral_constant<int, 4>{});
      finish(std::integral_constant<int, 5>{});
      finish(std::integral_constant<int, 6>{});
      finish(std::integral_constant<int, 7>{});
      finish(std::integral_constant<int, 8>{});
      finish(std::integral_constant<int, 9>{});
      finish(std::integral_constant<int, 10>{});
      finish(std::integral_constant<int, 11>{});
      finish(std::integral_constant<int, 12>{});
      finish(std::integral_constant<int, 13>{});
    }
    if (!EARLY && inner) {
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        Z[(k * (RB + UB) + rw) * NI] = r0[k];
        Z[(k * (RB + UB) + uw) * NI] = up[k];
      }
    }
    __syncthreads();   // the links of plane z are in, those of plane z - 1 consumed
  }
}

// Position of block b among nb when XCD j takes a contiguous span of them.
__device__ inline uint32_t xcd_span(uint32_t b, uint32_t nb) {
  const uint32_t per = nb / 8u, rem = nb % 8u, j = b & 7u;
  return j * per + (j < rem ? j : rem) + (b >> 3);
}

// A launch: planes [z_lo, z_hi), `chunk` per block; tiles of one chunk after the other.
template <int ST, bool SC, bool NT>
__global__ void __launch_bounds__(PNI + PNR, 2)
k_pair(const Place<typename Store<ST>::T> src, const Place<typename Store<ST>::T> dst, const Geom g, const Phys ph,
       const Codec cd, int z_lo, int z_hi, int chunk, int tx, int ty, int ntx, int ncol,
       const typename Store<ST>::T* __restrict__ wrap, int wrap_z, typename Store<ST>::T* __restrict__ over, int over_z) {
  __shared__ PairLds<ST> sh;
  const uint32_t t = xcd_span(blockIdx.x, gridDim.x);
  const int ch = (int)(t / (uint32_t)ncol), col = (int)(t % (uint32_t)ncol), za = z_lo + ch * chunk;
  pair_block<ST, SC, NT>(sh, src, dst, g, ph, cd, za, min(z_hi, za + chunk), (col % ntx) * tx, (col / ntx) * ty, tx, ty,
                         wrap, wrap_z, over, over_z);
}

// Position of block b when runs of 32 consecutive tiles, one per CU of an XCD, are dealt to the XCDs in
// turn: a batch's tiles differ in cost, and whole spans would leave XCDs idle.
__device__ inline uint32_t xcd_deal(uint32_t b, uint32_t nb) {
  return b < nb / 256u * 256u ? b / 256u * 256u + (b & 7u) * 32u + ((b >> 3) & 31u) : b;
}

// All members of a batch: from each member's array to its place in the second one, or back.
template <int ST, bool SC>
__global__ void __launch_bounds__(PNI + PNR, 2)
k_pair_batch(typename Store<ST>::T* __restrict__ home, typename Store<ST>::T* __restrict__ second,
             const Member* __restrict__ members, const PairMember* __restrict__ pm,
             const uint16_t* __restrict__ block_member, int back) {
  using T = typename Store<ST>::T;
  __shared__ PairLds<ST> sh;
  const uint32_t t = xcd_deal(blockIdx.x, gridDim.x);
  const uint32_t m = __builtin_amdgcn_readfirstlane(block_member[t]);
  const Member& M = members[m];
  const PairMember& P = pm[m];
  const Geom g = M.g;
  const int q = (int)(t - P.block0), ch = q / P.ncol, col = q % P.ncol, za = ch * P.chunk;
  T* const a = home + M.pop_offset;
  T* const b = second + P.offset;
  const Place<T> at_home{a, b, g.cstride, P.cstride, 0}, moved{a, b, g.cstride, P.cstride, (int)g.nz};
  pair_block<ST, SC, false>(sh, back ? moved : at_home, back ? at_home : moved, g, M.ph, M.cd, za,
                            min((int)g.nz, za + P.chunk), (col % P.ntx) * P.tx, (col / P.ntx) * P.ty, P.tx, P.ty,
                            (const T*)nullptr, -1000000, (T*)nullptr, -1000000);
}

// One plane's stored populations, copied aside (98 slots; groups as in the lattice, cell 0 first).
template <typename T>
__global__ void __launch_bounds__(256) k_plane_save(const T* __restrict__ base, uint64_t cs, uint32_t cell0, uint32_t nxy,
                                                    T* __restrict__ out, uint64_t ocs) {
  const uint32_t c = blockIdx.x * 256u + threadIdx.x;
  if (c >= nxy) return;
  const uint32_t k = blockIdx.y;
#pragma unroll
  for (int i = 0; i < NV; ++i) out[k * ocs + slot_index(i, c)] = base[k * cs + slot_index(i, cell0 + c)];
}

// The parked links of one direction, put into their plane.
template <typename T>
__global__ void __launch_bounds__(256) k_plane_put(const T* __restrict__ in, uint64_t ics, uint32_t nxy, int slot,
                                                   T* __restrict__ base, uint64_t cs, uint32_t cell0) {
  const uint32_t c = blockIdx.x * 256u + threadIdx.x;
  if (c >= nxy) return;
  const uint32_t k = blockIdx.y;
  base[k * cs + slot_index(slot, cell0 + c)] = in[k * ics + c];
}

static uint64_t groups(uint64_t n) { return (n + SLOT_GROUP - 1) / SLOT_GROUP * SLOT_GROUP; }

size_t pair_workspace_bytes(const Geom& g, int storage, int split) {
  const size_t e = storage == 0 ? 4 : 2;
  size_t n = (size_t)NP * groups((uint64_t)split * g.nxy);
  if (split < (int)g.nz) n += (size_t)(NP + NC) * groups(g.nxy);   // the wrapped plane and the parked links
  return n * e;
}

// Rows of a tile of tx columns, 0 if there is no such tile: whole rows up to 96 cells, else tiles that
// start on line boundaries (equal cuts lose: 112^3 FP32 56-wide 196 us per update, 64-wide 154; 320^3
// 54-wide 5.7 ms, 64-wide 3.4).
static int tile_rows(int tx, int nx, int ny) {
  if (tx > 96 || (tx == 64 && nx < 64)) return 0;
  int ty = std::min(PNI / tx, ny);
  while (ty > 1 && ring_columns(tx, ty, nx) > PNR) --ty;
  if (ring_columns(tx, ty, nx) > PNR) return 0;
  const int n = (ny + ty - 1) / ty;
  return (ny + n - 1) / n;
}

static double plane_us(int storage, int nx, double columns, bool cached) {
  const double fill = columns / PNI;
  const int row = nx * (storage == 0 ? 4 : 2);
  if (storage == 0) return cached ? 7.5 : 11.0 * (0.2 + 0.8 * fill) + (row % 128 ? 2.5 : 0.0);
  return row % 128 ? 7.3 * (0.5 + 0.5 * fill) + (row % 32 ? 2.0 : 1.0) : 7.3;
}

// How to cut a lattice, and whether two updates in one pass are faster than two single ones.
// A launch takes rounds x (planes per block + 3) plane times: rounds are its blocks over the CUs,
// a block reads one plane more at either end and needs about one plane time to start.  Measured
// plane times (us, TGV boxes of 32^3 to 512^3): FP32 11.0 with full tiles and rows of whole
// 128-byte lines (9.6-11.2), shorter as fewer of the tile's columns exist, about 2.5 more with
// rows of partial lines, 6.6-8.2 when the lattice fits the 256 MB last-level cache; 16-bit 7.3
// (7.0-7.4) and one or two more with rows of partial lines.  Single updates (ns per cell): FP32
// 0.155 (0.12 in cache), 16-bit 0.077 (0.063).  Pairs must win by 5%.  Taken (us per update, single
// / pairs): FP32 64^3 31 / 23, 80^3 62 / 49, 96^3 132 / 79, 100^3 173 / 133, 128^3 336 / 188, 150^3
// 578 / 470; 16-bit 128^3 163 / 123, 192^3 552 / 450, 240^3 1118 / 972.  Left: FP32 48^3 and 16-bit
// 64^3 (equal), 16-bit 96^3 55 / 73, 200^3 647 / 713.
bool pair_plan(const Geom& g, int storage, size_t budget, int cus, PairPlan* out) {
  if (g.bc_x != 0) return false;
  const size_t e = storage == 0 ? 4 : 2;
  if (g.cstride * e > 0xFFFF0000ull) return false;   // dead lanes use offsets from there on
  const int nz = (int)g.nz, nx = (int)g.nx, ny = (int)g.ny;
  int m = 1;   // planes that hold whole slot groups
  while (m < (int)SLOT_GROUP && (uint64_t)m * g.nxy % SLOT_GROUP) m *= 2;
  const bool cached = (double)NP * e * g.ncells <= 256e6;
  double best = 1e300;
  for (const int tx : {nx, 64}) {
    const int ty = tile_rows(tx, nx, ny);
    if (!ty) continue;
    const int ntx = (nx + tx - 1) / tx, ncol = ntx * ((ny + ty - 1) / ty);
    const double plane = plane_us(storage, nx, (double)g.nxy / ncol, cached);
    auto consider = [&](int split, int slab) {
      if (pair_workspace_bytes(g, storage, split) > budget) return;
      const int nslab = (nz + slab - 1) / slab;
      for (int c = 1; c <= std::min(slab, 64); ++c) {
        const int h = (slab + c - 1) / c;
        const int rounds = (ncol * ((slab + h - 1) / h) + cus - 1) / cus;
        const double t = (double)nslab * rounds * (h + 3) * plane;
        if (t < best) {
          best = t;
          *out = PairPlan{split, slab, h, tx, ty, 0.0};
        }
      }
    };
    consider(nz, nz);
    for (int n = 2; n * 4 <= nz && nz / n >= 4; ++n) {
      const int slab = (nz + n - 1) / n, split = (slab + 2 + m - 1) / m * m;
      if (split + 2 <= nz) consider(split, slab);
    }
  }
  const double cell = storage == 0 ? (cached ? 0.12 : 0.155) : (cached ? 0.063 : 0.077);
  out->gain = 1e-3 * cell * g.ncells - 0.5 * best;
  return 1.05 * best < 2e-3 * cell * g.ncells;
}

template <int ST, bool SC>
static hipError_t launch_pair_t(void* pop, void* ws, const Geom& g, const Phys& ph, const Codec& cd, const PairPlan& pl,
                                bool back, hipStream_t s, bool* torn) {
  using T = typename Store<ST>::T;
  const bool whole = pl.split >= (int)g.nz;
  const uint64_t cs_scr = (uint64_t)NV * groups((uint64_t)pl.split * g.nxy);
  T* scr = (T*)ws;
  T* wrap = scr + NC * cs_scr;
  T* over = wrap + (uint64_t)NP * groups(g.nxy);
  const Place<T> home{(T*)pop, scr, g.cstride, cs_scr, 0}, moved{(T*)pop, scr, g.cstride, cs_scr, pl.split};
  const Place<T> src = back ? moved : home, dst = back ? home : moved;
  // non-temporal stores from arrays of 32 GB on: 512^3 FP32 10.9 ms per update against 12.8 with
  // ordinary ones, 384^3 and 320^3 the same with both, rows of partial lines and 16-bit codes slower
  // (100^3 164 against 133 us, 256^3 FP16 1057 against 955): the partial lines no longer meet in L2
  const bool nt = (double)NP * sizeof(T) * g.ncells >= 32e9;
  const int nz = (int)g.nz, none = -1000000;
  const int wrap_z = whole ? none : (back ? -1 : nz), over_z = whole ? none : (back ? nz : -1);
  auto cell = [&](const Place<T>& p, int z, T*& b, uint64_t& cs) {
    b = z < p.split ? p.scr : p.arr;
    cs = z < p.split ? p.cs_scr : p.cs_arr;
    return (uint32_t)(z < p.split ? z : z - p.split) * g.nxy;
  };
  const dim3 pg((g.nxy + 255) / 256, NC);
  // slabs: the array is no longer the level of the forward pass's start once its second slab has run (the first
  // one writes the workspace only)
  bool moving = !whole && back;
  hipError_t e = hipSuccess;
  auto refused = [&] {
    e = hipGetLastError();
    if (e != hipSuccess) *torn = moving;
    return e != hipSuccess;
  };
  if (!whole) {
    T* b;
    uint64_t cs;
    const uint32_t c0 = cell(src, back ? nz - 1 : 0, b, cs);
    hipLaunchKernelGGL(k_plane_save<T>, pg, dim3(256), 0, s, (const T*)b, cs, c0, g.nxy, wrap, (uint64_t)NV * groups(g.nxy));
    if (refused()) return e;
  }
  const int ntx = ((int)g.nx + pl.tx - 1) / pl.tx, ncol = ntx * (((int)g.ny + pl.ty - 1) / pl.ty);
  const int threads = PNI + (ring_columns(pl.tx, pl.ty, (int)g.nx) + 63) / 64 * 64;
  auto kernel = k_pair<ST, SC, false>;
  if constexpr (ST == 0)
    if (nt) kernel = k_pair<ST, SC, true>;
  const int nslab = (nz + pl.slab - 1) / pl.slab;
  for (int j = 0; j < nslab; ++j) {
    const int q = back ? nslab - 1 - j : j;
    const int z0 = q * pl.slab, z1 = std::min(nz, z0 + pl.slab);
    const int nch = (z1 - z0 + pl.chunk - 1) / pl.chunk;
    hipLaunchKernelGGL(kernel, dim3(ncol * nch), dim3(threads), 0, s, src, dst, g, ph, cd, z0, z1, pl.chunk, pl.tx,
                       pl.ty, ntx, ncol, (const T*)wrap, wrap_z, over, over_z);
    if (refused()) return e;
    moving = !whole && (back || j > 0);
  }
  if (!whole) {
    T* b;
    uint64_t cs;
    const uint32_t c0 = cell(dst, back ? 0 : nz - 1, b, cs);
    hipLaunchKernelGGL(k_plane_put<T>, pg, dim3(256), 0, s, (const T*)over, groups(g.nxy), g.nxy, back ? 5 : 6, b, cs, c0);
    if (refused()) return e;
  }
  return e;
}

hipError_t launch_pair(int storage, void* pop, void* ws, const Geom& g, const Phys& ph, const Codec& cd,
                       const PairPlan& pl, bool back, hipStream_t s, bool* torn) {
  const bool sc = cd.scaled != 0;
  *torn = false;
  if (storage == 0) return launch_pair_t<0, false>(pop, ws, g, ph, cd, pl, back, s, torn);
  if (storage == 1)
    return (sc ? launch_pair_t<1, true> : launch_pair_t<1, false>)(pop, ws, g, ph, cd, pl, back, s, torn);
  return (sc ? launch_pair_t<2, true> : launch_pair_t<2, false>)(pop, ws, g, ph, cd, pl, back, s, torn);
}

// Tiles of every member for blocks of about `height` planes; the blocks' total time and that of the
// longest one (us), 0 total if some member has no tile.
static double batch_cut(const Member* m, int n, int storage, int height, PairMember* out, uint32_t* blocks, int* threads,
                        double* longest) {
  double total = 0.0;
  uint64_t off = 0;
  *blocks = 0;
  *threads = 0;
  *longest = 0.0;
  for (int j = 0; j < n; ++j) {
    const Geom& g = m[j].g;
    const int nx = (int)g.nx, ny = (int)g.ny, nz = (int)g.nz;
    if (nz < 4) return 0.0;   // a block's planes wrap around the end once
    PairMember& P = out[j];
    const int c = std::max(1, (nz + height / 2) / height);
    P.chunk = (nz + c - 1) / c;
    const int nch = (nz + P.chunk - 1) / P.chunk;
    double best = 1e300, block = 0.0;
    for (const int tx : {nx, 64}) {
      const int ty = tile_rows(tx, nx, ny);
      if (!ty) continue;
      const int ntx = (nx + tx - 1) / tx, ncol = ntx * ((ny + ty - 1) / ty);
      const double us = plane_us(storage, nx, (double)g.nxy / ncol, false) * (P.chunk + 3);
      if (us * ncol < best) {
        best = us * ncol;
        block = us;
        P.tx = tx;
        P.ty = ty;
        P.ntx = ntx;
        P.ncol = ncol;
      }
    }
    if (best > 1e299) return 0.0;
    P.block0 = *blocks;
    P.offset = off;
    P.cstride = (uint64_t)NV * groups(g.ncells);
    off += (uint64_t)NC * P.cstride;
    *blocks += (uint32_t)(P.ncol * nch);
    *threads = std::max(*threads, PNI + (ring_columns(P.tx, P.ty, nx) + 63) / 64 * 64);
    total += best * nch;
    *longest = std::max(*longest, block);
  }
  return total;
}

// Cut of a batch and whether pairs are the faster way.  Higher blocks read fewer planes twice, lower
// ones end closer together: a pass takes the blocks' time over all CUs (0.77 of it FP32, 0.85 16-bit:
// the plane times are those of a lattice alone, where every CU is at the same step) and 0.8 of the
// longest block's.  Single updates (ns per cell): FP32 0.155, 16-bit 0.08.  Measured, single / pairs in
// ms per update (64 members of 32^3 to 96^3, heights 12 / 16 / 24 / 32 / 48): FP32 3.85 / 2.02, 1.98,
// 2.04, 2.01, 2.12; FP16 1.87 / 1.68, 1.61, 1.68, 1.64, 1.74; 64 of 64^3 FP16 1.30 / 1.02, 0.99, 0.98,
// 0.96, 0.94.  Few members: 8 of mixed sizes FP16 0.16 / 0.15, BF16 0.29 / 0.29 and three BF16 0.17 /
// 0.20 are left to single updates.
bool pair_batch_plan(const Member* m, int n, int storage, int cus, PairMember* out, uint32_t* blocks, int* threads,
                     uint64_t* elements, double* gain) {
  double best = 1e300, cells = 0.0, longest = 0.0;
  int height = 0;
  for (const int h : {12, 16, 24, 32, 48}) {
    const double total = batch_cut(m, n, storage, h, out, blocks, threads, &longest);
    if (total == 0.0) return false;
    const double t = (storage == 0 ? 0.77 : 0.85) * total / cus + 0.8 * longest;
    if (t < best) {
      best = t;
      height = h;
    }
  }
  batch_cut(m, n, storage, height, out, blocks, threads, &longest);
  *elements = out[n - 1].offset + NC * out[n - 1].cstride;
  for (int j = 0; j < n; ++j) cells += m[j].g.ncells;
  *gain = 1e-3 * (storage == 0 ? 0.155 : 0.08) * cells - 0.5 * best;
  return *gain > 0.0;
}

hipError_t launch_pair_batch(int storage, bool scaled, void* home, void* second, const Member* members,
                             const PairMember* pm, const uint16_t* block_member, uint32_t blocks, int threads, bool back,
                             hipStream_t s) {
#define CNSF_CASE(ST, SC, T)                                                                                        \
  if (storage == ST && scaled == SC) {                                                                              \
    hipLaunchKernelGGL((k_pair_batch<ST, SC>), dim3(blocks), dim3(threads), 0, s, (T*)home, (T*)second, members, pm, \
                       block_member, back ? 1 : 0);                                                                 \
    return hipGetLastError();                                                                                       \
  }
  CNSF_CASE(0, false, float)
  CNSF_CASE(1, false, uint16_t)
  CNSF_CASE(2, false, uint16_t)
  CNSF_CASE(1, true, uint16_t)
  CNSF_CASE(2, true, uint16_t)
#undef CNSF_CASE
  return hipErrorInvalidValue;
}

}  // namespace cnsf
