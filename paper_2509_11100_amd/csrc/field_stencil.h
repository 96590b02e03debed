// Stencils of the implicit field solve, shared by the field kernels and the
// GMRES kernels: the curl of a cube of values.
//
// Both curls use one stencil shape: the difference along d averaged over the
// transverse corners of a 2x2(x2) cube.  Nodes -> centre of cell (i,j,k)
// reads the cube of nodes starting at (i,j,k); centres -> node (i,j,k) reads
// the cube of cells starting at (i-1,j-1,k-1).  That makes C_CN the exact
// transpose of C_NC on the periodic grid.
#pragma once

#include "relsim_internal.h"

namespace relsim {
namespace {

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Cube of 2^DIM values of the three components starting at (i0, j0, k0).
template <int DIM>
__device__ __forceinline__ void load_cube(const KParams &kp, const double *__restrict__ F, int i0, int j0, int k0,
                                          double c[3][8]) {
  const size_t N = (size_t)kp.ncells;
  const int x0 = wrapi(i0, kp.nx), x1 = wrapi(i0 + 1, kp.nx);
  const int y0 = wrapi(j0, kp.ny), y1 = wrapi(j0 + 1, kp.ny);
  const int z0 = DIM == 3 ? wrapi(k0, kp.nz) : 0, z1 = DIM == 3 ? wrapi(k0 + 1, kp.nz) : 0;
#pragma unroll
  for (int a = 0; a < (DIM == 3 ? 8 : 4); ++a) {
    const size_t id = (size_t)((a & 1) ? x1 : x0) +
                      (size_t)kp.nx * ((size_t)((a & 2) ? y1 : y0) + (size_t)kp.ny * ((a & 4) ? z1 : z0));
    c[0][a] = F[id];
    c[1][a] = F[N + id];
    c[2][a] = F[2 * N + id];
  }
}

// curl of the cube: (dy Fz - dz Fy, dz Fx - dx Fz, dx Fy - dy Fx)
template <int DIM>
__device__ __forceinline__ void cube_curl(const KParams &kp, const double c[3][8], double out[3]) {
  const double ax = kp.inv_dx / (DIM == 3 ? 4.0 : 2.0);
  const double ay = kp.inv_dy / (DIM == 3 ? 4.0 : 2.0);
  const double az = kp.inv_dz / 4.0;
  double d[3][3];  // d[comp][dim]
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if constexpr (DIM == 2) {
      d[q][0] = ax * ((c[q][1] - c[q][0]) + (c[q][3] - c[q][2]));
      d[q][1] = ay * ((c[q][2] - c[q][0]) + (c[q][3] - c[q][1]));
      d[q][2] = 0.0;
    } else {
      d[q][0] = ax * ((c[q][1] - c[q][0]) + (c[q][3] - c[q][2]) + (c[q][5] - c[q][4]) + (c[q][7] - c[q][6]));
      d[q][1] = ay * ((c[q][2] - c[q][0]) + (c[q][3] - c[q][1]) + (c[q][6] - c[q][4]) + (c[q][7] - c[q][5]));
      d[q][2] = az * ((c[q][4] - c[q][0]) + (c[q][5] - c[q][1]) + (c[q][6] - c[q][2]) + (c[q][7] - c[q][3]));
    }
  }
  out[0] = d[2][1] - d[1][2];
  out[1] = d[0][2] - d[2][0];
  out[2] = d[1][0] - d[0][1];
}

}  // namespace
}  // namespace relsim
