// Stencils of the implicit field solve, shared by the field kernels and the
// GMRES kernels: the curl of a cube of values and the mass-matrix product.
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

__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb >> 3;
  if (b >= (q << 3)) return b;
  return (b & 7) * q + (b >> 3);
}

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

// Linear index of node (i + dx, j + dy, k + dz), periodic.
template <int DIM>
__device__ __forceinline__ size_t node_at(const KParams &kp, int i, int j, int k, int dx, int dy, int dz) {
  return (size_t)wrapi(i + dx, kp.nx) +
         (size_t)kp.nx * ((size_t)wrapi(j + dy, kp.ny) + (size_t)kp.ny * (DIM == 3 ? wrapi(k + dz, kp.nz) : 0));
}

// (M x)_g, or (M^T x)_g with TR (each 3x3 block transposed), from the stored
// half of the blocks: slot h of node g couples x at g + delta(h), and for
// h > 0 the same slot of node g - delta(h) couples x at g - delta(h)
// (M_{g,g-delta} = M_{g-delta,g}).  MT is M's storage type (double, or
// float on request in mixed precision); the products and sums are FP64.
template <int DIM, bool TR, typename MT>
__device__ __forceinline__ void apply_M(const KParams &kp, const MT *__restrict__ M,
                                        const double *__restrict__ x, int g, int i, int j, int k, double mx[3]) {
  constexpr int NSLOT = m_slots<DIM>(), CEN = m_centre<DIM>();
  const size_t N = (size_t)kp.ncells;
#pragma unroll
  for (int h = 0; h < NSLOT; ++h) {
    const int off = CEN + h;
    const int dx = off % 3 - 1, dy = (off / 3) % 3 - 1, dz = DIM == 3 ? off / 9 - 1 : 0;
#pragma unroll
    for (int side = 0; side < (h ? 2 : 1); ++side) {
      // side 0: own block times x at g + delta; side 1: the neighbour's
      // block times x at g - delta
      const size_t id = side ? node_at<DIM>(kp, i, j, k, -dx, -dy, -dz) : node_at<DIM>(kp, i, j, k, dx, dy, dz);
      const double x0 = x[id], x1 = x[N + id], x2 = x[2 * N + id];
      const MT *Mo = M + (size_t)h * 9 * N + (side ? id : (size_t)g);
      double m[9];
#pragma unroll
      for (int q = 0; q < 9; ++q) m[q] = (double)Mo[q * N];
      if constexpr (!TR) {
        mx[0] += m[0] * x0 + m[1] * x1 + m[2] * x2;
        mx[1] += m[3] * x0 + m[4] * x1 + m[5] * x2;
        mx[2] += m[6] * x0 + m[7] * x1 + m[8] * x2;
      } else {
        mx[0] += m[0] * x0 + m[3] * x1 + m[6] * x2;
        mx[1] += m[1] * x0 + m[4] * x1 + m[7] * x2;
        mx[2] += m[2] * x0 + m[5] * x1 + m[8] * x2;
      }
    }
  }
}

}  // namespace
}  // namespace relsim
