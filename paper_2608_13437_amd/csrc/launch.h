// Host-side launchers of the cnsf kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>

#include "cnsf_impl.h"

namespace cnsf {

// Launch shape of the update: threads per block (<= 256), cells per tile (a
// multiple of block), blocks in a persistent grid (0: one block per tile) and
// the XCD-contiguous tile remap.
struct Launch {
  int block = 256;
  int tile = 1024;
  int grid = 0;
  int remap = 1;
};
// Shape measured best on MI355X for each storage type (512^3 Taylor-Green).
Launch default_launch(int storage);
// Shape in which a lattice of ncells is launched on `cus` compute units unless its caller set one.
Launch lattice_launch(int storage, uint64_t ncells, int cus);

hipError_t launch_update(int storage, void* pop, const Geom& g, const Phys& ph, const Codec& cd, int parity,
                         const Launch& lc, hipStream_t s);
hipError_t launch_init(int storage, void* pop, const double* Q, const Geom& g, const PhysD& ph, const Codec& cd,
                       uint32_t cell0, uint32_t nslab, int* bad, bool primitive, hipStream_t s);
hipError_t launch_primitives(int storage, const void* pop, double* out, const Geom& g, const Codec& cd, const PhysD& ph,
                             int parity, uint32_t cell0, uint32_t nslab, hipStream_t s);
hipError_t launch_moments(int storage, const void* pop, double* out, const Geom& g, const Codec& cd, int parity,
                          uint32_t cell0, uint32_t nslab, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);

// What making a workspace costs a call (us; first call with / without: 256 x 4 x 4 FP32, 1.6 MB, from the runtime's
// pool, 37 / 35; 1024 x 4 x 4, 6.4 MB, 70 / 40; 64^3, 103 MB, 320 / 208; 4.5 GB 1.5 ms).
inline double ws_cost(size_t bytes) {
  const double mb = 1e-6 * (double)bytes;
  return (mb < 2.0 ? 2.0 : mb < 24.0 ? 5.0 + 4.0 * mb : 100.0) + 0.3 * mb;
}

// Two updates in one pass (pair.hip): planes of the workspace, planes per launch, planes per block,
// columns of a tile along x and y.
struct PairPlan {
  int split = 0, slab = 0, chunk = 0, tx = 0, ty = 0;
  double gain = 0.0;   // us per update over single updates, by the plan's times
};
// The plan of a lattice with at most `budget` workspace bytes on `cus` compute units; false if
// single updates are at least as fast or the lattice is not served.
bool pair_plan(const Geom& g, int storage, size_t budget, int cus, PairPlan* out);
size_t pair_workspace_bytes(const Geom& g, int storage, int split);
// One pass of a lattice at an even level: forward from the array to the shifted place, or back.  If a launch is
// refused the array holds the level from which the last forward pass began, unless *torn is set: slabs had begun
// to overwrite it.
hipError_t launch_pair(int storage, void* pop, void* ws, const Geom& g, const Phys& ph, const Codec& cd,
                       const PairPlan& pl, bool back, hipStream_t s, bool* torn);

// One member of a batch in the device table, and its cut for paired passes (second array: member
// after member, each laid out like a lattice of its own).
struct Member {
  Geom g;
  Phys ph;
  Codec cd;
  uint64_t pop_offset;  // elements from the batch base
  uint32_t tile0;       // first tile of this member
  uint32_t ntiles;
};
struct PairMember {
  uint32_t block0;
  int tx, ty, ntx, ncol, chunk;
  uint64_t offset, cstride;
};
// `gain`: us per update over single updates, by the plan's times.
bool pair_batch_plan(const Member* m, int n, int storage, int cus, PairMember* out, uint32_t* blocks, int* threads,
                     uint64_t* elements, double* gain);
hipError_t launch_pair_batch(int storage, bool scaled, void* home, void* second, const Member* members,
                             const PairMember* pm, const uint16_t* block_member, uint32_t blocks, int threads, bool back,
                             hipStream_t s);

// Several updates per launch for thin lattices (tube.hip): planes of a window and the even number
// of updates per launch; calls of fewer than `least` updates are faster as single ones.  A window as
// long as the lattice takes any number, in place.
struct TubePlan {
  int xw = 0, steps = 0, least = 4;
  double gain = 0.0;   // us per update over single updates, by the plan's times
};
bool tube_plan(const Geom& g, int storage, int cus, TubePlan* out);
// `steps` (even) updates of a lattice at an even level, from src to dst (both laid out as the array).
hipError_t launch_tube(int storage, const void* src, void* dst, const Geom& g, const Phys& ph, const Codec& cd, int xw,
                       int steps, hipStream_t s);

// Diagnostics: FP64 sums and the spectral dissipation averages.
struct DiagPartial {
  double mass, mx, my, mz, energy, ek2;  // ek2 = sum rho |u|^2
  double min_rho, min_p;
  double sensor, nonfinite;
  double eps_s, eps_d;                   // sums of mu |curl u|^2 and mu (div u)^2
};
constexpr int DIAG_BLOCKS = 2048;
// The update of one time level that also reduces that level's Eq. (7) sums:
// one DiagPartial per block (update_blocks of them) and, if fields is given,
// u, v, w, mu into fields.
uint32_t update_blocks(const Geom& g, const Launch& lc);
hipError_t launch_update_diag(int storage, void* pop, const Geom& g, const Phys& ph, const Codec& cd, int parity,
                              const Launch& lc, const PhysD& phd, DiagPartial* partials, double* fields,
                              hipStream_t s);
hipError_t launch_diag_sums(int storage, const void* pop, const Geom& g, const Phys& ph, const PhysD& phd,
                            const Codec& cd, int parity, DiagPartial* partials, double* fields, hipStream_t s);
// u, v, w of a periodic lattice into fields (3 * ncells doubles), in the
// arithmetic of launch_diag_sums, reading only the rho and rho u populations.
hipError_t launch_velocity(int storage, const void* pop, const Geom& g, const Codec& cd, int parity, double* fields,
                           hipStream_t s);
// fields: u, v, w, mu (4 * ncells doubles), then div, wx, wy, wz (4 * ncells).
// Spectral eps sums of the u, v, w, mu fields into DIAG_BLOCKS partials: only
// their eps fields, or (full) whole partials with the other fields neutral.
hipError_t launch_spectral(const Geom& g, double dx, double* fields, DiagPartial* partials, bool full,
                           hipStream_t s);
// Total of the partials into out[0], in two levels when there are many (chunks reduced into tmp, at most ntmp
// of them, by many blocks; tmp may be NULL), and of a second set, unless that is NULL, into out[1].  out may be
// host memory that the device can write.
hipError_t launch_diag_final(const DiagPartial* partials, int nparts, DiagPartial* tmp, int ntmp,
                             const DiagPartial* second, int nsecond, DiagPartial* out, hipStream_t s);
// Shell spectrum of the velocity held in fields (u, v, w: the first 3 * ncells
// doubles, written by launch_velocity), which it overwrites; uses fields[4 ncells, 8 ncells) as
// workspace and partial (SHELL_PARTS * nz * spectrum_shells(nx) doubles).  Writes nout
// values to E (zero beyond the shell count).  Cubic periodic lattices only.
constexpr uint32_t SHELL_PARTS = 4;
uint32_t spectrum_shells(uint32_t n);
hipError_t launch_spectrum(const Geom& g, double* fields, double* partial, double* E, uint32_t nout, hipStream_t s);

}  // namespace cnsf
