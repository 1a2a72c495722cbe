// Line transforms as FP64 matrix products (lines.hip): spectral derivatives and the spectrum's
// Fourier transforms.
#pragma once

#include <hip/hip_runtime.h>

#include "launch.h"

namespace cnsf {

// One component of a derivative launch: offsets (doubles) of its field and accumulator, and what
// becomes of the result: stored (init) or added; eps >= 0: its field is complete, and mu field^2
// goes into the partials of quarter eps instead.
constexpr uint32_t LINE_PARTIALS = DIAG_BLOCKS / 4;
struct LineComp {
  uint64_t in, out;
  double sign;
  int init, eps, eps_d;
};
struct LineDeriv {
  uint32_t n, stride, nlines, nx, nxy;
  int axis, full;       // full: eps partials are written whole, their other fields neutral
  uint64_t mu;          // offset of mu
  double kscale;        // 2 pi / (n dx)
  LineComp c[3];
};
// Whether the product is the faster way for lines of n points (or the only one in LDS).
bool deriv_lines_serves(uint32_t n);
hipError_t launch_deriv_lines(const LineDeriv& ld, double* fields, DiagPartial* partials, hipStream_t s);

struct LineDft {
  uint32_t n, nxh, plane, stride, nlines;
  uint64_t real_size, size;   // points of a real component, of a complex one
  double escale;
};
bool dft_lines_serves(uint32_t n);
// Modes of u, v, w (fields[0, 3 n^3)) of an n^3 box with kappa_x >= 0 and the sum over the
// components of |X|^2 / (2 n^6) of each, into fields as rows of n/2 + 1; workspace fields[4 n^3, 8 n^3).
hipError_t launch_dft_lines(uint32_t n, double* fields, hipStream_t s);

}  // namespace cnsf
