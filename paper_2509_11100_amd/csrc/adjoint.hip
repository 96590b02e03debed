// Hand-written adjoint (reverse mode) of one step, FP64 only.
//
// Forward step of one particle (S1, S2, S6), positions in physical units:
//   B_p = sum_c W_c(x) B^n_c, gbar = gamma(u), b = beta B_p/(gbar c),
//   alpha(b) = (I - [b]x + b b^T)/(1 + b^2), E_p = sum_g W_g(x) E_th_g,
//   z = u + beta E_p, ubar = alpha z, u' = 2 ubar - u, x' = x + dt u'/gamma(u').
// The deposit (S3) enters the linearised objective only through
//   Jbar = Jhat + M E_th = V^-1 sum_p w q W_g ubar_p / gbar_p,
// so its adjoint is, per particle, the derivative of
//   Phi_p = K_p mu_p^T alpha (u + beta E_p),  K_p = -4 pi th dt w q / (V gbar),
// with mu = A^-T lambda_{E_th} gathered at the particle: two node gathers and
// one outer product per particle, no 9 x 9 x offset scatter.
// Gradients of the CIC weights are piecewise constant (one-sided at a node,
// taken from the particle's own cell).
//
// Grid adjoints.  All particles of a cell add to the cell's 2^dim nodes (E_th)
// and to the 3^dim centres around it (B), so a group of G lanes takes a cell,
// each lane sums its particles' contributions in registers (a centre's weight
// is a product over the dimensions of max(1/2 - f, 0), max(f - 1/2, 0) or what
// they leave of 1), the group adds its lanes through LDS once per cell and
// writes the cell's sums, and a second kernel adds the sums of the cells
// around each grid point to the caller's arrays in a fixed order: no atomics,
// and the results are deterministic.
#include <type_traits>

#include "relsim_internal.h"

namespace relsim {
namespace {

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// The cell of lane group grp of the block, its particles [beg, end) and the
// first one of its second species.
struct AdjCell {
  int cell, c[3], beg, second, end;
  bool valid;
};

template <int DIM, int G>
__device__ __forceinline__ AdjCell adj_cell(const KParams &kp, const int32_t *__restrict__ bin_start, int grp) {
  AdjCell a;
  const int id = (int)blockIdx.x * (64 / G) + grp;
  a.valid = id < kp.ncells;
  a.cell = a.valid ? id : kp.ncells - 1;
  a.c[0] = a.cell % kp.nx;
  a.c[1] = (a.cell / kp.nx) % kp.ny;
  a.c[2] = DIM == 3 ? a.cell / (kp.nx * kp.ny) : 0;
  a.beg = bin_start[a.cell * kp.nspecies];
  a.second = bin_start[a.cell * kp.nspecies + 1];  // the cell's end with one species
  a.end = a.valid ? bin_start[(a.cell + 1) * kp.nspecies] : a.beg;
  return a;
}

struct D3 {
  double x, y, z;
};

// The cell's fields in LDS, staged by its group: B at the 3^DIM centres
// around it (x fastest) and node values at its 2^DIM corners.
template <int DIM>
struct AdjFields {
  static constexpr int NC = DIM == 3 ? 27 : 9, NN = 1 << DIM;
};

template <int DIM, int G>
__device__ __forceinline__ void stage_points(const KParams &kp, const AdjCell &a, const double *__restrict__ F,
                                             bool centres, int gl, D3 *out) {
  const size_t N = (size_t)kp.ncells;
  const int np = centres ? AdjFields<DIM>::NC : AdjFields<DIM>::NN;
  for (int t = gl; t < np; t += G) {
    const int ox = centres ? t % 3 - 1 : t & 1;
    const int oy = centres ? (t / 3) % 3 - 1 : (t >> 1) & 1;
    const int oz = DIM == 3 ? (centres ? t / 9 - 1 : t >> 2) : 0;
    const int id = wrapi(a.c[0] + ox, kp.nx) +
                   kp.nx * (wrapi(a.c[1] + oy, kp.ny) + kp.ny * (DIM == 3 ? wrapi(a.c[2] + oz, kp.nz) : 0));
    out[t] = D3{F[id], F[N + id], F[2 * N + id]};
  }
}

// One particle's state and its order in the other array.
struct PRec {
  double f[3], u[3], w;
  int q;
};

template <int DIM>
__device__ __forceinline__ PRec load_particle(const double *__restrict__ xy, const double *__restrict__ uw,
                                              const int32_t *__restrict__ new_index, int p) {
  PRec r;
  if constexpr (DIM == 3) {
    // one 8-value record per particle at xy: (off_x, off_y, off_z, 0, u_x, u_y, u_z, w)
    const V4<double> *const R = reinterpret_cast<const V4<double> *>(xy) + 2 * (size_t)p;
    const V4<double> a = R[0], b = R[1];
    r.f[0] = a.x, r.f[1] = a.y, r.f[2] = a.z;
    r.u[0] = b.x, r.u[1] = b.y, r.u[2] = b.z, r.w = b.w;
  } else {
    const V2<double> a = reinterpret_cast<const V2<double> *>(xy)[p];
    const V4<double> b = reinterpret_cast<const V4<double> *>(uw)[p];
    r.f[0] = a.x, r.f[1] = a.y, r.f[2] = 0.0;
    r.u[0] = b.x, r.u[1] = b.y, r.u[2] = b.z, r.w = b.w;
  }
  r.q = new_index ? new_index[p] : p;
  return r;
}

// CIC weights of the 2^DIM points around a particle whose fractional
// distances from the lowest one are g, and the field there: F_p = sum wt F.
template <int DIM>
__device__ __forceinline__ void corner_weights(const double g[3], double wt[1 << DIM]) {
#pragma unroll
  for (int a = 0; a < (1 << DIM); ++a) {
    wt[a] = ((a & 1) ? g[0] : 1.0 - g[0]) * ((a & 2) ? g[1] : 1.0 - g[1]);
    if constexpr (DIM == 3) wt[a] *= (a & 4) ? g[2] : 1.0 - g[2];
  }
}

template <int DIM>
__device__ __forceinline__ void gather(const D3 *F, const int st[3], const double wt[1 << DIM], double out[3]) {
  out[0] = out[1] = out[2] = 0.0;
#pragma unroll
  for (int a = 0; a < (1 << DIM); ++a) {
    const D3 v = F[(a & 1) * st[0] + ((a >> 1) & 1) * st[1] + (DIM == 3 ? (a >> 2) * st[2] : 0)];
    out[0] += wt[a] * v.x;
    out[1] += wt[a] * v.y;
    out[2] += wt[a] * v.z;
  }
}

// lx[d] += d/dx_d of sum_a wt_a e_a (wt the corner weights at g)
template <int DIM>
__device__ __forceinline__ void add_gradient(const KParams &kp, const double g[3], const double e[1 << DIM],
                                             double lx[3]) {
  const double inv[3] = {kp.inv_dx, kp.inv_dy, kp.inv_dz};
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < (1 << DIM); ++a) {
      if ((a >> d) & 1) continue;
      double w = 1.0;
#pragma unroll
      for (int o = 0; o < DIM; ++o)
        if (o != d) w *= ((a >> o) & 1) ? g[o] : 1.0 - g[o];
      s += w * (e[a | (1 << d)] - e[a]);
    }
    lx[d] += inv[d] * s;
  }
}

// e_a = F_a . v at the corners
template <int DIM>
__device__ __forceinline__ void corner_dots(const D3 *F, const int st[3], const double v[3], double e[1 << DIM]) {
#pragma unroll
  for (int a = 0; a < (1 << DIM); ++a) {
    const D3 x = F[(a & 1) * st[0] + ((a >> 1) & 1) * st[1] + (DIM == 3 ? (a >> 2) * st[2] : 0)];
    e[a] += x.x * v[0] + x.y * v[1] + x.z * v[2];
  }
}

// The centres' lower corner and fractions of a particle at f: pointer into
// the staged 3^DIM block.
template <int DIM>
__device__ __forceinline__ const D3 *centre_corner(const D3 *B, const double f[3], double g[3]) {
  int at = 0, stride = 1;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const bool hi = f[d] >= 0.5;
    g[d] = hi ? f[d] - 0.5 : f[d] + 0.5;
    at += hi ? stride : 0;
    stride *= 3;
  }
  return B + at;
}

// acc[3 t + k] += (weight of centre t) v[k] over the 3^DIM centres
template <int DIM>
__device__ __forceinline__ void add_centres(const double f[3], const double v[3], double *acc) {
  double w[3][3];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    w[d][0] = fmax(0.5 - f[d], 0.0);
    w[d][2] = fmax(f[d] - 0.5, 0.0);
    w[d][1] = 1.0 - w[d][0] - w[d][2];
  }
#pragma unroll
  for (int t = 0; t < (DIM == 3 ? 27 : 9); ++t) {
    double wt = w[0][t % 3] * w[1][(t / 3) % 3];
    if constexpr (DIM == 3) wt *= w[2][t / 9];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[3 * t + k] += wt * v[k];
  }
}

// The group's sums of acc over its lanes (through LDS, kChunk at a time, in
// lane order) into sums[m ncells + cell].
constexpr int kChunk = 32;
constexpr double kAdjRounds = 4.0;
template <int NACC, int G>
__device__ __forceinline__ void put_sums(const double (&acc)[NACC], const AdjCell &a, int ncells, double *red,
                                         double *__restrict__ sums) {
  const int lane = threadIdx.x, grp = lane / G, gl = lane % G;
#pragma unroll
  for (int c0 = 0; c0 < NACC; c0 += kChunk) {
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (c0 + k < NACC) red[lane * (kChunk + 1) + k] = acc[c0 + k];
    __syncthreads();
    const int kend = NACC - c0 < kChunk ? NACC - c0 : kChunk;
    for (int k = gl; k < kend; k += G) {
      double s = 0.0;
#pragma unroll 8
      for (int j = 0; j < G; ++j) s += red[(grp * G + j) * (kChunk + 1) + k];
      if (a.valid) sums[(size_t)(c0 + k) * ncells + a.cell] = s;
    }
    __syncthreads();
  }
}

// lE (NE = 3 2^DIM sums per cell, or none) and lB (3^{DIM+1} sums) += the
// sums of the cells around each node and centre.
template <int DIM, bool HASE>
__global__ __launch_bounds__(256) void k_adj_gather(KParams kp, const double *__restrict__ sums,
                                                    double *__restrict__ lE, double *__restrict__ lB) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g >= kp.ncells) return;
  constexpr int NN = 1 << DIM, NC = DIM == 3 ? 27 : 9;
  const size_t N = (size_t)kp.ncells;
  const int i = g % kp.nx, j = (g / kp.nx) % kp.ny, k = DIM == 3 ? g / (kp.nx * kp.ny) : 0;
  auto cell = [&](int ox, int oy, int oz) {
    return (size_t)wrapi(i - ox, kp.nx) +
           (size_t)kp.nx * (wrapi(j - oy, kp.ny) + (size_t)kp.ny * (DIM == 3 ? wrapi(k - oz, kp.nz) : 0));
  };
  if constexpr (HASE) {
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < NN; ++a) {
      const size_t c = cell(a & 1, (a >> 1) & 1, a >> 2);
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q] += sums[(size_t)(3 * a + q) * N + c];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) lE[q * N + g] += s[q];
  }
  const double *const sb = sums + (HASE ? (size_t)(3 * NN) * N : 0);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < NC; ++t) {
    const size_t c = cell(t % 3 - 1, (t / 3) % 3 - 1, DIM == 3 ? t / 9 - 1 : 0);
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q] += sb[(size_t)(3 * t + q) * N + c];
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) lB[q * N + g] += s[q];
}

// alpha(b); returns 1 / (1 + b^2)
__device__ __forceinline__ double alpha_of(const double b[3], double a[9]) {
  const double inv = 1.0 / (1.0 + b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
  a[0] = (1.0 + b[0] * b[0]) * inv;
  a[1] = (b[2] + b[0] * b[1]) * inv;
  a[2] = (b[0] * b[2] - b[1]) * inv;
  a[3] = (b[0] * b[1] - b[2]) * inv;
  a[4] = (1.0 + b[1] * b[1]) * inv;
  a[5] = (b[0] + b[1] * b[2]) * inv;
  a[6] = (b[1] + b[0] * b[2]) * inv;
  a[7] = (b[1] * b[2] - b[0]) * inv;
  a[8] = (1.0 + b[2] * b[2]) * inv;
  return inv;
}

// d(l^T alpha(b) z)/db, with inv = 1 / (1 + b^2) and phi = l^T alpha z:
// (l x z + l (z.b) + z (l.b) - 2 phi b) / (1 + b^2)
__device__ __forceinline__ void alpha_vjp(const double b[3], double inv, const double l[3], const double z[3],
                                          double phi, double lb[3]) {
  const double zb = z[0] * b[0] + z[1] * b[1] + z[2] * b[2];
  const double lbd = l[0] * b[0] + l[1] * b[1] + l[2] * b[2];
  const double p2 = 2.0 * phi;
  lb[0] = (l[1] * z[2] - l[2] * z[1] + l[0] * zb + z[0] * lbd - p2 * b[0]) * inv;
  lb[1] = (l[2] * z[0] - l[0] * z[2] + l[1] * zb + z[1] * lbd - p2 * b[1]) * inv;
  lb[2] = (l[0] * z[1] - l[1] * z[0] + l[2] * zb + z[2] * lbd - p2 * b[2]) * inv;
}

// Charge and beta of particle p of the cell (ac.second: the first particle
// of species 1; further species look their bounds up).
__device__ __forceinline__ void species(const KParams &kp, const int32_t *__restrict__ bin_start, const AdjCell &a,
                                        int p, double &q, double &beta) {
  const bool s1 = p >= a.second;
  q = s1 ? kp.q[1] : kp.q[0];
  beta = s1 ? kp.beta[1] : kp.beta[0];
  for (int s = 2; s < kp.nspecies; ++s)
    if (p >= bin_start[a.cell * kp.nspecies + s]) {
      q = kp.q[s];
      beta = kp.beta[s];
    }
}

// Both kernels need about 130 bytes per particle and take 95 to 101 and 75 to 80
// us for the 2.1M particles of the 256 x 128 sheet.  Counted, with the cells' sums,
// they move 0.42 and 0.32 GB, 4.4 and 4.3 TB/s, with the VALU busy 0.30 and 0.35
// of the time: they run at the memory's rate (59 and 57 us for the bytes needed
// at the copy rate; with the lanes summed by wave butterflies per particle and
// added by atomics they took 445 and 305 us).  In 2D they hold 39 and 27 sums
// per lane and fit two waves per SIMD without spilling; forcing three spills
// (1865 us for the step instead of 1350), and so does loading the next
// round's particle ahead.  In 3D (105 and 81 sums) one wave fits.
template <int DIM, int G>
__global__ __launch_bounds__(64, DIM == 2 ? 2 : 1) void k_push_adjoint(KParams kp, AdjInPtrs in, int n, const double *__restrict__ Eth,
                                                     const double *__restrict__ B,
                                                     const int32_t *__restrict__ new_index,
                                                     const double *__restrict__ lx_in,
                                                     const double *__restrict__ lu_in, double *__restrict__ lx_out,
                                                     double *__restrict__ lu_out, double *__restrict__ sums) {
  constexpr int NC = AdjFields<DIM>::NC, NN = AdjFields<DIM>::NN;
  __shared__ double red[64 * (kChunk + 1)];
  __shared__ D3 Bsh[64 / G][NC], Esh[64 / G][NN];
  const int lane = threadIdx.x, grp = lane / G, gl = lane % G;
  const AdjCell ac = adj_cell<DIM, G>(kp, in.bin_start, grp);
  stage_points<DIM, G>(kp, ac, B, true, gl, Bsh[grp]);
  stage_points<DIM, G>(kp, ac, Eth, false, gl, Esh[grp]);
  __syncthreads();
  const int sc[3] = {1, 3, 9}, sn[3] = {1, 2, 4};
  double acc[3 * (NN + NC)];
#pragma unroll
  for (int m = 0; m < 3 * (NN + NC); ++m) acc[m] = 0.0;
  int p = ac.beg + gl;
  for (; p < ac.end; p += G) {
    const PRec st = load_particle<DIM>(in.xy, in.uw, new_index, p);
    // incoming cotangents (new order -> this particle)
    double lxp[3] = {0, 0, 0}, lun[3];
#pragma unroll
    for (int d = 0; d < DIM; ++d) lxp[d] = lx_in[(size_t)d * n + st.q];
#pragma unroll
    for (int k = 0; k < 3; ++k) lun[k] = lu_in[(size_t)k * n + st.q];
    double qs, beta;
    species(kp, in.bin_start, ac, p, qs, beta);
    double gc[3], wc[NN], wn[NN], Bp[3], Ep[3];
    const D3 *const Bc = centre_corner<DIM>(Bsh[grp], st.f, gc);
    corner_weights<DIM>(gc, wc);
    corner_weights<DIM>(st.f, wn);
    gather<DIM>(Bc, sc, wc, Bp);
    gather<DIM>(Esh[grp], sn, wn, Ep);
    const double *u = st.u;
    const double igb = kp.nonrel ? 1.0 : 1.0 / sqrt(1.0 + (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) * kp.inv_c2);
    const double kb = beta * igb * kp.inv_c;
    const double b[3] = {kb * Bp[0], kb * Bp[1], kb * Bp[2]};
    double a[9];
    const double inv = alpha_of(b, a);
    const double z[3] = {u[0] + beta * Ep[0], u[1] + beta * Ep[1], u[2] + beta * Ep[2]};
    double ub[3], un[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ub[i] = a[3 * i] * z[0] + a[3 * i + 1] * z[1] + a[3 * i + 2] * z[2];
      un[i] = 2.0 * ub[i] - u[i];
    }
    const double ign = kp.nonrel ? 1.0 : 1.0 / sqrt(1.0 + (un[0] * un[0] + un[1] * un[1] + un[2] * un[2]) * kp.inv_c2);
    // x' = x + dt u'/gamma(u'):  d(u/gamma)/du = (I - u u^T/(c^2 gamma^2))/gamma
    {
      double ulx = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) ulx += un[d] * lxp[d];
      const double r = kp.nonrel ? 0.0 : ulx * ign * ign * kp.inv_c2;
#pragma unroll
      for (int k = 0; k < 3; ++k) lun[k] += kp.dt * ign * ((k < DIM ? lxp[k] : 0.0) - un[k] * r);
    }
    // u' = 2 ubar - u, ubar = alpha z
    const double lub[3] = {2.0 * lun[0], 2.0 * lun[1], 2.0 * lun[2]};
    const double phi = lub[0] * ub[0] + lub[1] * ub[1] + lub[2] * ub[2];
    double lu[3], lz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      lz[j] = a[j] * lub[0] + a[3 + j] * lub[1] + a[6 + j] * lub[2];
      lu[j] = lz[j] - lun[j];
    }
    const double lEp[3] = {beta * lz[0], beta * lz[1], beta * lz[2]};
    double lx[3] = {lxp[0], lxp[1], lxp[2]};
    double e[NN];
#pragma unroll
    for (int c = 0; c < NN; ++c) e[c] = 0.0;
    corner_dots<DIM>(Esh[grp], sn, lEp, e);
    add_gradient<DIM>(kp, st.f, e, lx);
#pragma unroll
    for (int c = 0; c < NN; ++c)
#pragma unroll
      for (int k = 0; k < 3; ++k) acc[3 * c + k] += wn[c] * lEp[k];
    // alpha(b(B_p, gbar))
    double lb[3];
    alpha_vjp(b, inv, lub, z, phi, lb);
    const double lBp[3] = {kb * lb[0], kb * lb[1], kb * lb[2]};
    if (!kp.nonrel) {
      const double lgb = -(b[0] * lb[0] + b[1] * lb[1] + b[2] * lb[2]) * igb * igb * kp.inv_c2;
#pragma unroll
      for (int k = 0; k < 3; ++k) lu[k] += lgb * u[k];
    }
#pragma unroll
    for (int c = 0; c < NN; ++c) e[c] = 0.0;
    corner_dots<DIM>(Bc, sc, lBp, e);
    add_gradient<DIM>(kp, gc, e, lx);
    add_centres<DIM>(st.f, lBp, acc + 3 * NN);
#pragma unroll
    for (int d = 0; d < DIM; ++d) lx_out[(size_t)d * n + p] = lx[d];
#pragma unroll
    for (int k = 0; k < 3; ++k) lu_out[(size_t)k * n + p] = lu[k];
  }
  put_sums<3 * (NN + NC), G>(acc, ac, kp.ncells, red, sums);
}

template <int DIM, int G>
__global__ __launch_bounds__(64, DIM == 2 ? 2 : 1) void k_deposit_adjoint(KParams kp, AdjInPtrs in, int n,
                                                        const double *__restrict__ B,
                                                        const double *__restrict__ Eth,
                                                        const double *__restrict__ mu, double *__restrict__ lx_out,
                                                        double *__restrict__ lu_out, double *__restrict__ sums) {
  constexpr int NC = AdjFields<DIM>::NC, NN = AdjFields<DIM>::NN;
  __shared__ double red[64 * (kChunk + 1)];
  __shared__ D3 Bsh[64 / G][NC], Esh[64 / G][NN], Msh[64 / G][NN];
  const int lane = threadIdx.x, grp = lane / G, gl = lane % G;
  const AdjCell ac = adj_cell<DIM, G>(kp, in.bin_start, grp);
  stage_points<DIM, G>(kp, ac, B, true, gl, Bsh[grp]);
  stage_points<DIM, G>(kp, ac, Eth, false, gl, Esh[grp]);
  stage_points<DIM, G>(kp, ac, mu, false, gl, Msh[grp]);
  __syncthreads();
  const int sc[3] = {1, 3, 9}, sn[3] = {1, 2, 4};
  double acc[3 * NC];
#pragma unroll
  for (int m = 0; m < 3 * NC; ++m) acc[m] = 0.0;
  int p = ac.beg + gl;
  for (; p < ac.end; p += G) {
    const PRec st = load_particle<DIM>(in.xy, in.uw, nullptr, p);
    double lx[3] = {0, 0, 0}, lu[3];
#pragma unroll
    for (int d = 0; d < DIM; ++d) lx[d] = lx_out[(size_t)d * n + p];
#pragma unroll
    for (int k = 0; k < 3; ++k) lu[k] = lu_out[(size_t)k * n + p];
    double qs, beta;
    species(kp, in.bin_start, ac, p, qs, beta);
    double gc[3], wc[NN], wn[NN], Bp[3], Ep[3], mp[3];
    const D3 *const Bc = centre_corner<DIM>(Bsh[grp], st.f, gc);
    corner_weights<DIM>(gc, wc);
    corner_weights<DIM>(st.f, wn);
    gather<DIM>(Bc, sc, wc, Bp);
    gather<DIM>(Esh[grp], sn, wn, Ep);
    gather<DIM>(Msh[grp], sn, wn, mp);
    const double *u = st.u;
    const double igb = kp.nonrel ? 1.0 : 1.0 / sqrt(1.0 + (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) * kp.inv_c2);
    const double kb = beta * igb * kp.inv_c;
    const double b[3] = {kb * Bp[0], kb * Bp[1], kb * Bp[2]};
    double a[9];
    const double inv = alpha_of(b, a);
    const double z[3] = {u[0] + beta * Ep[0], u[1] + beta * Ep[1], u[2] + beta * Ep[2]};
    double ub[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) ub[i] = a[3 * i] * z[0] + a[3 * i + 1] * z[1] + a[3 * i + 2] * z[2];
    const double K = -4.0 * M_PI * kp.theta * kp.dt * kp.inv_V * st.w * qs * igb;
    const double phi = K * (mp[0] * ub[0] + mp[1] * ub[1] + mp[2] * ub[2]);
    // d/d mu_p and d/d z
    const double lmp[3] = {K * ub[0], K * ub[1], K * ub[2]};
    double lz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      lz[j] = K * (a[j] * mp[0] + a[3 + j] * mp[1] + a[6 + j] * mp[2]);
      lu[j] += lz[j];
    }
    const double lEp[3] = {beta * lz[0], beta * lz[1], beta * lz[2]};
    double e[NN];
#pragma unroll
    for (int c = 0; c < NN; ++c) e[c] = 0.0;
    corner_dots<DIM>(Esh[grp], sn, lEp, e);
    corner_dots<DIM>(Msh[grp], sn, lmp, e);
    add_gradient<DIM>(kp, st.f, e, lx);
    // d/d alpha = K mu_p z^T
    const double l[3] = {K * mp[0], K * mp[1], K * mp[2]};
    double lb[3];
    alpha_vjp(b, inv, l, z, phi, lb);
    const double lBp[3] = {kb * lb[0], kb * lb[1], kb * lb[2]};
    if (!kp.nonrel) {
      // gbar enters through b and through K
      const double lgb = -(b[0] * lb[0] + b[1] * lb[1] + b[2] * lb[2] + phi) * igb * igb * kp.inv_c2;
#pragma unroll
      for (int k = 0; k < 3; ++k) lu[k] += lgb * u[k];
    }
#pragma unroll
    for (int c = 0; c < NN; ++c) e[c] = 0.0;
    corner_dots<DIM>(Bc, sc, lBp, e);
    add_gradient<DIM>(kp, gc, e, lx);
    add_centres<DIM>(st.f, lBp, acc);
#pragma unroll
    for (int d = 0; d < DIM; ++d) lx_out[(size_t)d * n + p] = lx[d];
#pragma unroll
    for (int k = 0; k < 3; ++k) lu_out[(size_t)k * n + p] = lu[k];
  }
  put_sums<3 * NC, G>(acc, ac, kp.ncells, red, sums);
}

// Calls f<G> for the group width: kAdjRounds rounds per cell at the mean
// occupancy, at least 8 lanes, wider on small grids until the launch has 1024
// waves.  On the 256 x 128 sheet (64 particles per cell), 8 rounds of 8 lanes,
// 4 of 16 and 2 of 32 take 1370, 1350 and 1346 us for a step forward and
// backward.
template <typename F>
void with_group(const KParams &kp, int n, F &&f) {
  const double mean = (double)n / kp.ncells;
  int g = 8;
  while (g < 64 && (2.0 * g * kAdjRounds <= mean || (double)kp.ncells * g < 1024.0 * 64.0)) g *= 2;
  switch (g) {
    case 8: return f(std::integral_constant<int, 8>());
    case 16: return f(std::integral_constant<int, 16>());
    case 32: return f(std::integral_constant<int, 32>());
    default: return f(std::integral_constant<int, 64>());
  }
}

template <int DIM>
void push_adjoint(const KParams &kp, const AdjInPtrs &in, int n, const double *Eth, const double *B,
                  const int32_t *new_index, const double *lx_in, const double *lu_in, double *lx_out, double *lu_out,
                  double *lEth, double *lB, double *sums, hipStream_t st) {
  with_group(kp, n, [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    const int nb = (kp.ncells + 64 / G - 1) / (64 / G);
    hipLaunchKernelGGL((k_push_adjoint<DIM, G>), dim3(nb), dim3(64), 0, st, kp, in, n, Eth, B, new_index, lx_in,
                       lu_in, lx_out, lu_out, sums);
  });
  hipLaunchKernelGGL((k_adj_gather<DIM, true>), dim3((kp.ncells + 255) / 256), dim3(256), 0, st, kp, sums, lEth, lB);
}

template <int DIM>
void deposit_adjoint(const KParams &kp, const AdjInPtrs &in, int n, const double *B, const double *Eth,
                     const double *mu, double *lx_out, double *lu_out, double *lB, double *sums, hipStream_t st) {
  with_group(kp, n, [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    const int nb = (kp.ncells + 64 / G - 1) / (64 / G);
    hipLaunchKernelGGL((k_deposit_adjoint<DIM, G>), dim3(nb), dim3(64), 0, st, kp, in, n, B, Eth, mu, lx_out,
                       lu_out, sums);
  });
  hipLaunchKernelGGL((k_adj_gather<DIM, false>), dim3((kp.ncells + 255) / 256), dim3(256), 0, st, kp, sums, nullptr,
                     lB);
}

}  // namespace

void launch_push_adjoint(const KParams &kp, const AdjInPtrs &in, int n, const double *Eth, const double *B,
                         const int32_t *new_index, const double *lx_in, const double *lu_in, double *lx_out,
                         double *lu_out, double *lEth, double *lB, double *sums, hipStream_t st) {
  if (n <= 0) return;
  if (kp.dim == 2)
    push_adjoint<2>(kp, in, n, Eth, B, new_index, lx_in, lu_in, lx_out, lu_out, lEth, lB, sums, st);
  else
    push_adjoint<3>(kp, in, n, Eth, B, new_index, lx_in, lu_in, lx_out, lu_out, lEth, lB, sums, st);
}

void launch_deposit_adjoint(const KParams &kp, const AdjInPtrs &in, int n, const double *B, const double *Eth,
                            const double *mu, double *lx_out, double *lu_out, double *lB, double *sums,
                            hipStream_t st) {
  if (n <= 0) return;
  if (kp.dim == 2)
    deposit_adjoint<2>(kp, in, n, B, Eth, mu, lx_out, lu_out, lB, sums, st);
  else
    deposit_adjoint<3>(kp, in, n, B, Eth, mu, lx_out, lu_out, lB, sums, st);
}

}  // namespace relsim
