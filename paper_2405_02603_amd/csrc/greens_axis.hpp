// greens_axis.hpp -- the potential's precompute in three axis passes (greens_axis.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace fsp {

// One axis pass.  Inputs and outputs are float64 arrays with rows (axis 2) of
// pitch p2; the axes keep their order and the contracted one shrinks to n + 1.
struct AxisArgs {
  const double* image;  // matrix image of this axis (green_axis_image)
  const double* x;      // axes 1 and 2: the last pass's result
  double* y;            // axes 0 and 1: result
  void* octant;         // axis 2: the stored octant, [k1][k2 tile][k0][tile]
  int n;                // grid points along the contracted axis
  int N;                // columns: axis 0 d1 p2, axis 1 (n0 + 1) p2, axis 2 (n0 + 1)(n1 + 1)
  int d1, p2;           // inputs along axis 1 (2 n1 + 1, or n1 + 1), pitch of axis 2
  int n0, n1, n2;
  int tile, f64;
  double scale;
  double f[3];          // axis 0: frequency step (or spacing) of each axis
  double half_turns, at_zero;  // Vico-Greengard: L / (2 pi), L^2 / 2
  double g0;                   // Hockney-Eastwood: the value at the origin
  int periodic;         // axis 0, Hockney-Eastwood: bit a, axis a takes its nearest image's offset
};

size_t green_axis_image_elems(int n);
hipError_t green_axis_image(double* out, int n, bool vico, hipStream_t s);
hipError_t green_axis(const AxisArgs& a, bool vico, int axis, hipStream_t s);

}  // namespace fsp
