// Restarted GMRES of the implicit field solve (S4-S5 and the transposed
// solve of the adjoint), FP64.
//
// The Krylov iteration runs on the device without the host: the Hessenberg
// columns, the Givens rotations, the stopping test and the triangular solve
// are computed by the kernels that need them, and the host enqueues the steps
// it expects and reads the state once at the end (api.hip).
//
// Orthogonalisation: classical Gram-Schmidt twice, with the second pass of a
// vector delayed until the operator has been applied to it (Bielich, Langou,
// Thomas, Swirydowicz, Yamazaki and Boman, "Low-synch Gram-Schmidt with
// delayed reorthogonalization for Krylov solvers", 2022).  Column j starts
// from w~ = w / |w|, the candidate for v_j after one pass against V =
// (v_0 .. v_{j-1}):
//   k_gm_apply  u = A w~, and the sums s = V^T w~, z = V^T u, w~.u
//   k_gm_ortho  v_j = (w~ - V s) / nu, nu^2 = 1 - |s|^2 (the second pass),
//               z_j = v_j.u = (w~.u - s.z) / nu, and the next candidate
//               w = (u - V z - z_j v_j) / nu, with the sum w.w.
// A V s lies in the span of v_0 .. v_j, so the next candidate needs no other
// vector; the Hessenberg column is (z - H s) / nu, and the column before gets
// the second pass's correction s |w|.  Each step reads the basis twice and
// takes two kernels (a third, k_gm_dots, has the sums of columns past the 16th
// in 2D and the 8th in 3D), where two plain passes read it three times in three
// kernels.
//
// Each kernel starts by summing the block partial sums that the one before
// it left: a dependent kernel costs 2.6 us on this device, a separate
// reduction kernel 4.3 us, and the host round trip that each step used to end
// with 15 us.  A grid-wide barrier inside one persistent kernel would cost
// more than a kernel: 3.1 us over 32 blocks, 4.8 over 64, 11.6 over 256.  Sums
// are taken in a fixed order (per thread, wave, block, then block by block),
// so a solve is deterministic.
#include <climits>
#include <cmath>

#include "field_stencil.h"

namespace relsim {
namespace {

constexpr int TB = kGmThreads;
constexpr int NW = TB / 64;

// Block b's groups of TB nodes: group first, first + step, ... below last.
// Each XCD (blocks are dispatched to the 8 XCDs round robin) works through
// one contiguous band of the grid, its blocks side by side: a node reads the
// mass-matrix blocks of the rows below it, which are then in the same L2.
struct Groups {
  int first, last, step;
};
__device__ __forceinline__ Groups block_groups(int ng) {
  const int nb = (int)gridDim.x, b = (int)blockIdx.x;
  if (nb == ng) {
    const int first = xcd_bands(b, nb);
    return {first, first + 1, 1};
  }
  if (nb & 7) return {b, ng, nb};
  const int band = (ng + 7) >> 3, x = b & 7;
  const int lo = x * band;
  return {lo + (b >> 3), lo + band < ng ? lo + band : ng, nb >> 3};
}

// Node of thread t in group grp, or -1: in 2D TB consecutive nodes, in 3D
// TB / 64 chunks of the strip order.
template <int DIM>
__device__ __forceinline__ int group_node(const KParams &kp, int grp, int &i, int &j, int &k) {
  if constexpr (DIM == 2) {
    const int g = grp * TB + (int)threadIdx.x;
    j = g / kp.nx;
    i = g - j * kp.nx;
    k = 0;
    return g < kp.ncells ? g : -1;
  } else {
    return strip_node(kp.nx, kp.ny, kp.nz, grp * NW + (int)(threadIdx.x >> 6), (int)(threadIdx.x & 63), i, j, k);
  }
}
__host__ __device__ inline int node_groups(const KParams &kp) {
  return kp.dim == 2 ? (kp.ncells + TB - 1) / TB : grid_node_blocks(kp.nx, kp.ny, kp.nz);
}

// Sum of acc[q] (q < nv) over the block into P[q * gridDim.x + block].
template <int NV, int NW = kGmThreads / 64>
__device__ __forceinline__ void put_partials(const double (&acc)[NV], int nv, double *lds, double *__restrict__ P) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    if (q < nv) {
      double v = acc[q];
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
      if (lane == 0) lds[wid * NV + q] = v;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nv; q += 64 * NW) {
    double s = lds[q];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += lds[w * NV + q];
    P[(size_t)q * gridDim.x + blockIdx.x] = s;
  }
}

// out[q] (LDS) = the sum over the blocks of partials P[q][.], q < nv; every
// block forms the same sums.  Ends with a barrier.
template <int NW = kGmThreads / 64>
__device__ __forceinline__ void get_sums(const double *__restrict__ P, int nparts, int nv, double *out) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int q = wid; q < nv; q += NW) {
    const double *const p = P + (size_t)q * nparts;
    double v = 0.0;
#pragma unroll 4
    for (int b = lane; b < nparts; b += 64) v += p[b];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) out[q] = v;
  }
  __syncthreads();
}

// Whether the kernels of column j have nothing to do: the solve has ended,
// or its cycle ended with an earlier column.  A block that starts after block
// 0 of its own kernel has recorded an end would come to the same end, and one
// that started before decides from entries that block 0 leaves alone in that
// kernel.  One thread of a block reads the state for all of it, so that the
// block stays together.
__device__ __forceinline__ bool arnoldi_off(const GmState *st, int j) {
  return st->code != 0 || st->done != 0 || (st->end_at >= 0 && st->end_at < j);
}
// The same for the kernels after the Arnoldi steps (update, residual).
__device__ __forceinline__ bool tail_off(const GmState *st) {
  return st->code != 0 || st->done != 0 || st->end_at < 0;
}

// Adds the 3x3 block m, or its transpose, times x to y.
template <bool TR>
__device__ __forceinline__ void add_block(const double m[9], const double x[3], double y[3]) {
  if constexpr (!TR) {
    y[0] += m[0] * x[0] + m[1] * x[1] + m[2] * x[2];
    y[1] += m[3] * x[0] + m[4] * x[1] + m[5] * x[2];
    y[2] += m[6] * x[0] + m[7] * x[1] + m[8] * x[2];
  } else {
    y[0] += m[0] * x[0] + m[3] * x[1] + m[6] * x[2];
    y[1] += m[1] * x[0] + m[4] * x[1] + m[7] * x[2];
    y[2] += m[2] * x[0] + m[5] * x[1] + m[8] * x[2];
  }
}
template <typename MT>
__device__ __forceinline__ void load_block(const MT *__restrict__ M, size_t N, double m[9]) {
#pragma unroll
  for (int e = 0; e < 9; ++e) m[e] = (double)M[e * N];
}

// (A x)_g or (A^T x)_g in 2D: the 3 x 3 nodes around g hold all that the curl
// of the curl and the mass matrix read, and the curl is formed again for each
// of the 4 cells around g.
template <bool TR, typename MT>
__device__ __forceinline__ void apply_node(const KParams &kp, const MT *__restrict__ M, const double *__restrict__ x,
                                           int g, int i, int j, double xc[3], double out[3]) {
  const size_t N = (size_t)kp.ncells;
  const double a = kp.c * kp.theta * kp.dt;
  const double b = 4.0 * M_PI * kp.theta * kp.dt;
  double mx[3] = {0.0, 0.0, 0.0}, cc[3];
  {
    int id[9];
    double x9[3][9];
    const int im = wrapi(i - 1, kp.nx), ip = wrapi(i + 1, kp.nx);
    const int jm = kp.nx * wrapi(j - 1, kp.ny), jp = kp.nx * wrapi(j + 1, kp.ny), j0 = kp.nx * j;
    id[0] = im + jm, id[1] = i + jm, id[2] = ip + jm;
    id[3] = im + j0, id[4] = g, id[5] = ip + j0;
    id[6] = im + jp, id[7] = i + jp, id[8] = ip + jp;
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) x9[c][q] = x[c * N + id[q]];
#pragma unroll
    for (int h = 0; h < 5; ++h) {
#pragma unroll
      for (int side = 0; side < (h ? 2 : 1); ++side) {
        // side 0: own block times x at g + delta; side 1: the block of node
        // g - delta times x there
        const int q = side ? 4 - h : 4 + h;
        const MT *Mo = M + (size_t)h * 9 * N + (side ? id[q] : g);
        double m[9];
        load_block<MT>(Mo, N, m);
        const double xq[3] = {x9[0][q], x9[1][q], x9[2][q]};
        add_block<TR>(m, xq, mx);
      }
    }
    double tc[3][8];
#pragma unroll
    for (int cell = 0; cell < 4; ++cell) {
      double c[3][8], r[3];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int q = (cell & 1) + (n & 1) + 3 * ((cell >> 1) + (n >> 1));
#pragma unroll
        for (int s = 0; s < 3; ++s) c[s][n] = x9[s][q];
      }
      cube_curl<2>(kp, c, r);
#pragma unroll
      for (int s = 0; s < 3; ++s) tc[s][cell] = r[s];
    }
    cube_curl<2>(kp, tc, cc);
#pragma unroll
    for (int c = 0; c < 3; ++c) xc[c] = x9[c][4];
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) out[q] = xc[q] + a * a * cc[q] + b * mx[q];
}


// ---------------------------------------------------------------------------
// The operator in 3D: a march over z with every stored block read once.
//
// A node's 14 blocks couple it to 13 nodes ahead of it, and 13 nodes behind it
// hold the blocks that couple it to them.  Gathering those again from memory
// made the operator read 1.5 times the stored blocks (6.5 GB on the 256 x 128
// x 128 grid, 1.35 ms and 0.08 ms for the curl, at the memory's rate).  Here a
// block of waves owns a tile of w x ty nodes and marches over lz planes: lane
// and wave are a node's x and y, and a block read once gives both products, M
// x_{g+d} for its own node and M x_g for node g + d.  The latter goes to its
// lane by a lane shift, to its row through LDS and to the next plane in
// registers.  Nodes around the tile whose blocks reach into it are done again
// by the tile: a lane on either side of the row, a wave before (6 of 14
// blocks) and a wave behind (3) and the plane before the first (9).  The curl
// of the curl comes along: t = C_NC x of the wave's cells, shifted and passed
// the same way.  Counted for k_gm_residual, which also reads b and writes r: 6.1
// GB, 1.25 ms (4.9 TB/s); the product alone 1.18 ms; tiles of 2, 6, 8, 10 and
// 14 rows took 14.9, 14.2, 14.3, 14.3 and 15.2 ms for the whole solve (the
// last ones spill), and loading the next plane's first blocks ahead of the
// exchange 14.2.  The blocks are loaded a row (of three) ahead of their use:
// on smaller grids, where the caches hold part of M, a wave's loads in flight
// count (128 x 64 x 64, M in FP32: 1.84 -> 1.45 ms; gathering, 1.66 ms).
// ---------------------------------------------------------------------------
constexpr int kRows3 = 6;             // most rows of a tile
constexpr int NW3 = kRows3 + 2;       // waves: the rows and one on either side
constexpr int TB3 = 64 * NW3;

// Tiles of w x ty x lz nodes (plan_tiles3), the last ones along y and z
// possibly smaller.
struct Tiles3 {
  int w, ty, lz, ntx, nty, ntz;
  __host__ __device__ explicit Tiles3(const KParams &kp) : w(kp.t3x), ty(kp.t3y), lz(kp.t3z) {
    ntx = (kp.nx + w - 1) / w;
    nty = (kp.ny + ty - 1) / ty;
    ntz = (kp.nz + lz - 1) / lz;
  }
  __host__ __device__ int count() const { return ntx * nty * ntz; }
};

struct D3 {
  double x, y, z;
};
struct Planes3 {
  D3 a[NW3][64], b[NW3][64], c[NW3][64], t[NW3][64];
};

__device__ __forceinline__ D3 d3(const double v[3]) { return D3{v[0], v[1], v[2]}; }

// v of the lane to the left (x - 1) or right (x + 1)
template <bool RIGHT>
__device__ __forceinline__ double beside(double v) {
  constexpr int ctrl = RIGHT ? 0x130 : 0x138;  // DPP wave_shl:1, wave_shr:1
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// x of the node at dx, seen from this lane
template <int DX>
__device__ __forceinline__ void at_dx(const double v[3], double out[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) out[q] = DX == 0 ? v[q] : (DX > 0 ? beside<true>(v[q]) : beside<false>(v[q]));
}
// sum += c moved to the lane at dx
template <int DX>
__device__ __forceinline__ void send_dx(const double c[3], double sum[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) sum[q] += DX == 0 ? c[q] : (DX > 0 ? beside<false>(c[q]) : beside<true>(c[q]));
}

// Block m at DX of the lane's node (x = x_g): with GATHER its product with the
// x at DX (of the row and plane given, xr) is added to y, with SEND its
// product with x_g to sum at DX.
template <bool TR, int DX, bool GATHER, bool SEND>
__device__ __forceinline__ void use_block(const double m[9], const double x[3], const double xr[3], double y[3],
                                          double sum[3]) {
  if constexpr (GATHER) {
    double v[3];
    at_dx<DX>(xr, v);
    add_block<TR>(m, v, y);
  }
  if constexpr (SEND) {
    double c[3] = {0.0, 0.0, 0.0};
    add_block<TR>(m, x, c);
    send_dx<DX>(c, sum);
  }
}
// NB consecutive blocks from slot h on, loaded; three of them, at dx = -1, 0, 1
// of one row, used
template <int NB, typename MT>
__device__ __forceinline__ void load_row(const MT *__restrict__ M, size_t N, int h, int g, MT m[27]) {
#pragma unroll
  for (int e = 0; e < 9 * NB; ++e) m[e] = M[((size_t)h * 9 + e) * N + g];
}
template <typename MT>
__device__ __forceinline__ void as_double(const MT *m, double d[9]) {
#pragma unroll
  for (int e = 0; e < 9; ++e) d[e] = (double)m[e];
}
template <bool TR, bool GATHER, bool SEND, typename MT>
__device__ __forceinline__ void use_row(const MT m[27], const double x[3], const double xr[3], double y[3],
                                        double sum[3]) {
  double d[9];
  as_double(m, d);
  use_block<TR, -1, GATHER, SEND>(d, x, xr, y, sum);
  as_double(m + 9, d);
  use_block<TR, 0, GATHER, SEND>(d, x, xr, y, sum);
  as_double(m + 18, d);
  use_block<TR, 1, GATHER, SEND>(d, x, xr, y, sum);
}

// Barrier for the LDS exchange only: loads of the next planes stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Calls out(g, x_g, (A x)_g) for every node of the block's tiles, in the
// lanes and waves that own them, and before that pre(g), before the loads of
// the node's plane (also for the lanes beside).
template <bool TR, typename MT, typename P, typename F>
__device__ __forceinline__ void march3(const KParams &kp, const MT *__restrict__ M, const double *__restrict__ x,
                                       Planes3 &sh, P &&pre, F &&out) {
  const size_t N = (size_t)kp.ncells;
  const int lane = threadIdx.x & 63, rw = threadIdx.x >> 6;
  const Tiles3 tl(kp);
  const double a = kp.c * kp.theta * kp.dt;
  const double b = 4.0 * M_PI * kp.theta * kp.dt;
  const Groups gr = block_groups(tl.count());
  for (int tile = gr.first; tile < gr.last; tile += gr.step) {
    const int t1 = tile / tl.ntx, t2 = t1 / tl.nty;
    const int i0 = (tile - t1 * tl.ntx) * tl.w, j0 = (t1 - t2 * tl.nty) * tl.ty, k0 = t2 * tl.lz;
    const int w = tl.w < kp.nx - i0 ? tl.w : kp.nx - i0;
    const int rows = tl.ty < kp.ny - j0 ? tl.ty : kp.ny - j0;
    const int planes = tl.lz < kp.nz - k0 ? tl.lz : kp.nz - k0;
    // lanes past the right neighbour repeat it (their products reach no owned lane)
    const int i = wrapi(i0 - 1 + (lane < w + 1 ? lane : w + 1), kp.nx);
    const bool before = rw == 0, own = rw >= 1 && rw <= rows, behind = rw == rows + 1;
    const bool active = rw <= rows + 1;
    const int j = active ? wrapi(j0 - 1 + rw, kp.ny) : 0;
    const int row = i + kp.nx * j, up = i + kp.nx * wrapi(j + 1, kp.ny), down = i + kp.nx * wrapi(j - 1, kp.ny);
    const int nxy = kp.nx * kp.ny;
    int k = wrapi(k0 - 1, kp.nz);
    double x0[3], xp[3], carry[3] = {0, 0, 0}, t0[3] = {0, 0, 0}, tm0[3] = {0, 0, 0};
    auto load = [&](int plane, int at, double v[3]) {
      const size_t id = (size_t)plane * nxy + at;
#pragma unroll
      for (int q = 0; q < 3; ++q) v[q] = x[q * N + id];
    };
    load(k, row, x0);
    load(k, up, xp);
    for (int s = -1; s < planes; ++s) {
      const int kn = k + 1 == kp.nz ? 0 : k + 1;
      const int g = k * nxy + row;
      double nm[3], n0[3], np[3], y[3], s0[3], sA[3], sB[3], sC[3], t[3];
      load(kn, down, nm);
      load(kn, row, n0);
      load(kn, up, np);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        y[q] = carry[q];
        s0[q] = sA[q] = sB[q] = sC[q] = 0.0;
      }
      // rows of blocks in two buffers, one loaded while the other is used
      MT ma[27], mb[27];
      if (own) {
        if (s >= 0) {
          double d[9];
          pre(g);
          load_row<2>(M, N, 0, g, ma);
          load_row<3>(M, N, 2, g, mb);
          as_double(ma, d);
          add_block<TR>(d, x0, y);
          as_double(ma + 9, d);
          use_block<TR, 1, true, true>(d, x0, x0, y, y);
          load_row<3>(M, N, 5, g, ma);
          use_row<TR, true, true>(mb, x0, xp, y, sA);
          load_row<3>(M, N, 8, g, mb);
          use_row<TR, true, true>(ma, x0, nm, y, sB);
          load_row<3>(M, N, 11, g, ma);
          use_row<TR, true, true>(mb, x0, n0, y, s0);
          use_row<TR, true, true>(ma, x0, np, y, sC);
        } else {
          load_row<3>(M, N, 5, g, ma);
          load_row<3>(M, N, 8, g, mb);
          use_row<TR, false, true>(ma, x0, nm, y, sB);
          load_row<3>(M, N, 11, g, ma);
          use_row<TR, false, true>(mb, x0, n0, y, s0);
          use_row<TR, false, true>(ma, x0, np, y, sC);
        }
      } else if (before) {
        load_row<3>(M, N, 11, g, ma);
        if (s >= 0) {
          load_row<3>(M, N, 2, g, mb);
          use_row<TR, false, true>(mb, x0, xp, y, sA);
        }
        use_row<TR, false, true>(ma, x0, np, y, sC);
      } else if (behind) {
        load_row<3>(M, N, 5, g, ma);
        use_row<TR, false, true>(ma, x0, nm, y, sB);
      }
      if (own || before) {
        double c[3][8];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const double v[4] = {x0[q], xp[q], n0[q], np[q]};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            c[q][2 * r] = v[r];
            c[q][2 * r + 1] = beside<true>(v[r]);
          }
        }
        cube_curl<3>(kp, c, t);
        sh.a[rw][lane] = d3(sA);
        sh.c[rw][lane] = d3(sC);
        sh.t[rw][lane] = d3(t);
      }
      if (own || behind) sh.b[rw][lane] = d3(sB);
      lds_barrier();
      if (own) {
        const D3 va = sh.a[rw - 1][lane], vc = sh.c[rw - 1][lane], vb = sh.b[rw + 1][lane], vt = sh.t[rw - 1][lane];
        y[0] += va.x, y[1] += va.y, y[2] += va.z;
        carry[0] = s0[0] + vc.x + vb.x;
        carry[1] = s0[1] + vc.y + vb.y;
        carry[2] = s0[2] + vc.z + vb.z;
        const double tm[3] = {vt.x, vt.y, vt.z};
        double c[3][8], cc[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const double v[4] = {tm0[q], t0[q], tm[q], t[q]};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            c[q][2 * r] = beside<false>(v[r]);
            c[q][2 * r + 1] = v[r];
          }
        }
        cube_curl<3>(kp, c, cc);
        if (s >= 0 && lane >= 1 && lane <= w) {
          double r[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) r[q] = x0[q] + a * a * cc[q] + b * y[q];
          out(g, x0, r);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          t0[q] = t[q];
          tm0[q] = tm[q];
        }
      }
      lds_barrier();
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        x0[q] = n0[q];
        xp[q] = np[q];
      }
      k = kn;
    }
  }
}

// Calls pre(g), then out(g, x_g, (A x)_g) for the nodes of the block's share of
// the grid.
template <int DIM>
struct Shared {};
template <>
struct Shared<3> {
  Planes3 p;
};
struct NoPre {
  __device__ void operator()(int) const {}
};
template <int DIM, bool TR, typename MT, typename P, typename F>
__device__ __forceinline__ void apply_all(const KParams &kp, const MT *__restrict__ M, const double *__restrict__ x,
                                          Shared<DIM> &sh, P &&pre, F &&out) {
  if constexpr (DIM == 3) {
    march3<TR, MT>(kp, M, x, sh.p, pre, out);
  } else {
    const Groups gr = block_groups(node_groups(kp));
    for (int grp = gr.first; grp < gr.last; grp += gr.step) {
      int i, j, k;
      const int g = group_node<2>(kp, grp, i, j, k);
      if (g < 0) continue;
      double xc[3], y[3];
      pre(g);
      apply_node<TR, MT>(kp, M, x, g, i, j, xc, y);
      out(g, xc, y);
    }
  }
}
// Threads and waves of the kernels that apply the operator.
template <int DIM>
constexpr int kOpThreads = DIM == 3 ? TB3 : TB;
template <int DIM>
constexpr int kOpWaves = DIM == 3 ? NW3 : NW;

// y = A x or A^T x (relsim_apply_A, relsim_apply_AT)
template <int DIM, bool TR, typename MT>
__global__ __launch_bounds__(kOpThreads<DIM>, DIM == 3 ? NW3 / 4 : 1) void k_apply(KParams kp, const MT *__restrict__ M,
                                                           const double *__restrict__ x, double *__restrict__ y) {
  __shared__ Shared<DIM> sh;
  const size_t N = (size_t)kp.ncells;
  apply_all<DIM, TR, MT>(kp, M, x, sh, NoPre(), [&](int g, const double *, const double *r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) y[c * N + g] = r[c];
  });
}

__device__ __forceinline__ void init_state(const GmBuf &gm, int code) {
  GmState *st = gm.st;
  st->code = code;
  st->done = 0;
  st->end_at = -1;
  st->total_it = 0;
  st->cycle = 0;
  st->rel = 0.0;
}

// The vectors' rows are padded to an even length for 16-byte access; the pad
// stays 0.
__device__ __forceinline__ void zero_pads(const GmBuf &gm) {
  if (gm.ld == gm.n3) return;
  for (int q = threadIdx.x; q <= gm.m; q += TB) gm.V[(size_t)q * gm.ld + gm.n3] = 0.0;
  if (threadIdx.x == 0) gm.r[gm.n3] = 0.0;
}

// Start of the forward solve: b = E^n + c th dt C_CN B^n - 4 pi th dt Jhat,
// x = x0, and the partial sums of b.b.  Does nothing, and stops the kernels
// that follow, when an earlier call left an error flag.
template <int DIM>
__global__ __launch_bounds__(TB) void k_gm_rhs(KParams kp, GmBuf gm, const double *En, const double *Bn,
                                               const double *J, const double *x0, double *x,
                                               const int32_t *__restrict__ flags) {
  __shared__ double lds[NW];
  const bool refused = *flags != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) init_state(gm, refused ? kGmRefused : 0);
  if (refused) return;
  if (blockIdx.x == 0) zero_pads(gm);
  const size_t N = (size_t)kp.ncells;
  const double a = kp.c * kp.theta * kp.dt;
  const double b = 4.0 * M_PI * kp.theta * kp.dt;
  double acc[1] = {0.0};
  const Groups gr = block_groups(node_groups(kp));
  for (int grp = gr.first; grp < gr.last; grp += gr.step) {
    int i, j, k;
    const int g = group_node<DIM>(kp, grp, i, j, k);
    if (g < 0) continue;
    double c[3][8], cc[3];
    load_cube<DIM>(kp, Bn, i - 1, j - 1, k - 1, c);
    cube_curl<DIM>(kp, c, cc);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double bq = En[q * N + g] + a * cc[q] - b * J[q * N + g];
      gm.b[q * N + g] = bq;
      if (x != x0) x[q * N + g] = x0[q * N + g];
      acc[0] += bq * bq;
    }
  }
  put_partials<1>(acc, 1, lds, gm.p3);
}

// Start of the transposed solve: b = l_th + l_E1 / theta - c dt C_CN l_B1
// (C_NC^T = C_CN), x = 0, r = b, and the partial sums as above.
template <int DIM>
__global__ __launch_bounds__(TB) void k_gm_adj_start(KParams kp, GmBuf gm, const double *__restrict__ lth,
                                                     const double *__restrict__ lE1, const double *__restrict__ lB1,
                                                     double *__restrict__ x, const int32_t *__restrict__ flags) {
  __shared__ double lds[NW * 2];
  const bool refused = *flags != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) init_state(gm, refused ? kGmRefused : 0);
  if (refused) return;
  if (blockIdx.x == 0) zero_pads(gm);
  const size_t N = (size_t)kp.ncells;
  const double cdt = kp.c * kp.dt;
  double acc[2] = {0.0, 0.0};
  const Groups gr = block_groups(node_groups(kp));
  for (int grp = gr.first; grp < gr.last; grp += gr.step) {
    int i, j, k;
    const int g = group_node<DIM>(kp, grp, i, j, k);
    if (g < 0) continue;
    double c[3][8], cc[3];
    load_cube<DIM>(kp, lB1, i - 1, j - 1, k - 1, c);
    cube_curl<DIM>(kp, c, cc);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double bq = lth[q * N + g] + lE1[q * N + g] / kp.theta - cdt * cc[q];
      gm.b[q * N + g] = bq;
      gm.r[q * N + g] = bq;
      x[q * N + g] = 0.0;
      acc[0] += bq * bq;
    }
  }
  acc[1] = acc[0];
  put_partials<2>(acc, 2, lds, gm.p3);
}

// The cycle ends with column k, whose vector's norm is hn: its last rotation.
// One thread.  Blocks of the same kernel may still read a and g[k] to come to
// the same end, so the rotated entry of row k goes into a place of its own.
__device__ __forceinline__ void end_cycle(GmState *st, int k, double hn) {
  const double a = st->a, den = hypot(a, hn);
  st->R[(size_t)k * (kMaxRestart + 1) + k] = den;
  st->g_end = st->g[k] * (den > 0 ? a / den : 1.0);
  st->end_at = k;
}

// Basis vectors are taken kQ at a time, all loads of a group before their
// use (past the last vector a group repeats it, with results not used).
constexpr int kQ = 4;

// First half of column j: u = A w~ into V[j + 1], w~ = w / |w| with w in
// V[j], and the partial sums of w~.u, and with NV (at least j) also of V^T w~
// and V^T u.  The norm of w, summed here, first tells whether column j - 1 was
// the cycle's last (its residual is |g| |w| / hypot(a, |w|)).  FIRST (j = 0): w
// is the residual r, whose norm (and in the solve's first cycle the right-hand
// side's) is summed here.
template <int DIM, bool TR, typename MT, int NV, bool FIRST>
__global__ __launch_bounds__(kOpThreads<DIM>, DIM == 3 ? NW3 / 4 : 2) void k_gm_apply(
    KParams kp, GmBuf gm, const MT *__restrict__ M, int j, int cycle0) {
  constexpr int NW = kOpWaves<DIM>;
  __shared__ double lds[NW * (2 * NV + 1)];
  __shared__ Shared<DIM> sh;
  __shared__ bool off;
  GmState *const st = gm.st;
  if (threadIdx.x == 0) off = arnoldi_off(st, j);
  const size_t N = (size_t)kp.ncells;
  const bool head = blockIdx.x == 0 && threadIdx.x == 0;
  double wn;
  if constexpr (FIRST) {
    get_sums<NW>(gm.p3, gm.na, 2, lds);
    if (off) return;
    wn = sqrt(lds[1]);
    const double bnorm = cycle0 ? sqrt(lds[0]) : st->bnorm;
    const double tol = gm.rtol * bnorm;
    const int code = (cycle0 && !isfinite(bnorm)) ? kGmBadRhs : (!isfinite(wn) ? kGmBadResidual : 0);
    const bool conv = cycle0 && wn <= tol;
    if (head) {
      if (cycle0) {  // later cycles read bnorm here
        st->bnorm = bnorm;
        st->tol = tol;
      }
      st->rel = bnorm > 0 ? wn / bnorm : 0.0;
      st->g[0] = wn;
      st->wn = wn;
      if (code)
        st->code = code;
      else if (conv)
        st->done = kGmAtStart;
    }
    if (code || conv) return;
  } else {
    get_sums<NW>(gm.p2, gm.no, 1, lds);
    if (off) return;
    wn = sqrt(lds[0]);
    const double den = hypot(st->a, wn);
    const double est = den > 0 ? fabs(st->g[j - 1]) * (wn / den) : 0.0;
    const bool bad = !isfinite(wn);
    const bool last = est <= st->tol || wn == 0.0 || j == gm.m || st->total_it >= gm.maxit;
    if (head) {
      if (bad)
        st->code = kGmBadVector;
      else if (last)
        end_cycle(st, j - 1, wn);
      else
        st->wn = wn;
    }
    if (bad || last) return;
  }
  const double inv = 1.0 / wn;
  __syncthreads();
  const double *const x = FIRST ? gm.r : gm.V + (size_t)j * gm.ld;
  double *const u = gm.V + (size_t)(j + 1) * gm.ld;
  // w~.u, then s, then z
  double acc[2 * NV + 1];
#pragma unroll
  for (int q = 0; q <= 2 * NV; ++q) acc[q] = 0.0;
  apply_all<DIM, TR, MT>(kp, M, x, sh, NoPre(), [&](int g, const double *xg, const double *r) {
    double w[3], y[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      w[c] = inv * xg[c];
      y[c] = inv * r[c];
      u[c * N + g] = y[c];
      acc[0] += w[c] * y[c];
    }
    if constexpr (NV > 0) {
#pragma unroll
      for (int q0 = 0; q0 < NV; q0 += kQ) {
        if (q0 < j) {
          double v[kQ][3];
#pragma unroll
          for (int q = 0; q < kQ; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[q][c] = gm.V[(size_t)min(q0 + q, j - 1) * gm.ld + c * N + g];
#pragma unroll
          for (int q = 0; q < kQ; ++q) {
            acc[1 + q0 + q] += v[q][0] * w[0] + v[q][1] * w[1] + v[q][2] * w[2];
            acc[1 + NV + q0 + q] += v[q][0] * y[0] + v[q][1] * y[1] + v[q][2] * y[2];
          }
        }
      }
    }
  });
  // partial sums: w~.u, s_0 .. s_{j-1}, z_0 .. z_{j-1}
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q <= 2 * NV; ++q) {
    const int k = q <= NV ? q : q - NV;  // 1 + vector
    if (k <= j) {
      double v = acc[q];
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
      if (lane == 0) lds[wid * (2 * NV + 1) + (q <= NV ? q : j + k)] = v;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q <= (NV > 0 ? 2 * j : 0); q += 64 * NW) {
    double s = lds[q];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += lds[w * (2 * NV + 1) + q];
    gm.p1[(size_t)q * gridDim.x + blockIdx.x] = s;
  }
}

struct alignas(16) D2 {
  double x, y;
};

// The sums s = V^T w~ and z = V^T u of a column too long for the registers that
// the operator leaves (gm_apply): kDots vectors at a time, over the same blocks
// as the operator's, so that the partial sums lie where its own would.
constexpr int kDots = 16, kDotThreads = 512;
__global__ __launch_bounds__(kDotThreads) void k_gm_dots(GmBuf gm, int j) {
  constexpr int NW = kDotThreads / 64;
  __shared__ double lds[NW][2 * kDots];
  __shared__ bool off;
  const GmState *const st = gm.st;
  if (threadIdx.x == 0) off = arnoldi_off(st, j);
  __syncthreads();
  if (off) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const double inv = 1.0 / st->wn;
  const size_t n2 = gm.ld >> 1, ld2 = gm.ld >> 1;
  const D2 *const V = reinterpret_cast<const D2 *>(gm.V);
  for (int q0 = 0; q0 < j; q0 += kDots) {
    double acc[2 * kDots];
#pragma unroll
    for (int q = 0; q < 2 * kDots; ++q) acc[q] = 0.0;
    for (size_t i = (size_t)blockIdx.x * kDotThreads + threadIdx.x; i < n2; i += (size_t)gridDim.x * kDotThreads) {
      const D2 w = V[(size_t)j * ld2 + i], u = V[(size_t)(j + 1) * ld2 + i];
#pragma unroll
      for (int q1 = 0; q1 < kDots; q1 += 2 * kQ) {
        if (q0 + q1 < j) {
          D2 v[2 * kQ];
#pragma unroll
          for (int q = 0; q < 2 * kQ; ++q) v[q] = V[(size_t)min(q0 + q1 + q, j - 1) * ld2 + i];
#pragma unroll
          for (int q = 0; q < 2 * kQ; ++q) {
            acc[q1 + q] += v[q].x * w.x + v[q].y * w.y;
            acc[kDots + q1 + q] += v[q].x * u.x + v[q].y * u.y;
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 2 * kDots; ++q) {
      if (q0 + q % kDots < j) {
        double v = acc[q];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) lds[wid][q] = v;
      }
    }
    __syncthreads();
    const int q = threadIdx.x;
    if (q < 2 * kDots && q0 + q % kDots < j) {
      double s = lds[0][q];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += lds[w][q];
      const int at = 1 + q0 + (q < kDots ? q : j + q - kDots);
      gm.p1[(size_t)at * gridDim.x + blockIdx.x] = q < kDots ? inv * s : s;
    }
    __syncthreads();
  }
}

// Column j of the Hessenberg matrix and the rotations (one wave): s, z and
// z_j as in k_gm_ortho, hh: room for 2 (kMaxRestart + 1) values in LDS.
// Column j - 1 takes the correction of its vector's second pass and its final
// rotation; column j is rotated by all of them, its last entry kept in a until
// the norm of the next candidate is known.
__device__ void hessenberg_column(const GmBuf &gm, int j, const double *s, const double *z, double zj, double nu,
                                  double *hh) {
  constexpr int LD = kMaxRestart + 1;
  GmState *const st = gm.st;
  const int lane = threadIdx.x & 63;
  double *const prev = hh, *const cur = hh + LD;  // the two columns
  const double wn = st->wn;
  for (int k = lane; k <= j; k += 64) {
    if (j > 0) {
      const double h = k < j ? st->H[(size_t)(j - 1) * LD + k] + s[k] * wn : nu * wn;
      st->H[(size_t)(j - 1) * LD + k] = h;
      prev[k] = h;
    }
    double c = k < j ? z[k] : zj;
    for (int i = k > 0 ? k - 1 : 0; i + 1 < j; ++i) c -= st->H[(size_t)i * LD + k] * s[i];
    if (j > 0) c -= prev[k] * s[j - 1];
    c /= nu;
    st->H[(size_t)j * LD + k] = c;
    cur[k] = c;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane != 0) return;
  double a = prev[0], b = cur[0];
  for (int k = 0; k + 1 < j; ++k) {
    const double c = st->cs[k], sn = st->sn[k];
    const double p = prev[k + 1], q = cur[k + 1];
    st->R[(size_t)(j - 1) * LD + k] = c * a + sn * p;
    a = -sn * a + c * p;
    st->R[(size_t)j * LD + k] = c * b + sn * q;
    b = -sn * b + c * q;
  }
  if (j > 0) {
    const double hn = prev[j], den = hypot(a, hn);
    const double c = den > 0 ? a / den : 1.0, sn = den > 0 ? hn / den : 0.0;
    st->R[(size_t)(j - 1) * LD + j - 1] = den;
    st->cs[j - 1] = c;
    st->sn[j - 1] = sn;
    const double g = st->g[j - 1];
    st->g[j - 1] = c * g;
    st->g[j] = -sn * g;
    const double q = cur[j];
    st->R[(size_t)j * LD + j - 1] = c * b + sn * q;
    b = -sn * b + c * q;
  }
  st->a = b;
  ++st->total_it;
}

// Second half of column j: v_j into V[j], the next candidate into V[j + 1],
// and the partial sums of its square.  When nu^2 has cancelled (at most 1e-4:
// the candidate lay in the span of the basis) the cycle ends with the column
// before.
__global__ __launch_bounds__(TB) void k_gm_ortho(GmBuf gm, int j) {
  __shared__ double sums[2 * kMaxRestart + 1], s[kMaxRestart], z[kMaxRestart], hh[2 * (kMaxRestart + 1)], lds[NW];
  __shared__ bool off;
  GmState *const st = gm.st;
  if (threadIdx.x == 0) off = arnoldi_off(st, j);
  get_sums(gm.p1, gm.na, 2 * j + 1, sums);
  if (off) return;
  const int jq = (j + kQ - 1) / kQ * kQ;
  for (int q = threadIdx.x; q < jq; q += TB) {
    s[q] = q < j ? sums[1 + q] : 0.0;
    z[q] = q < j ? sums[1 + j + q] : 0.0;
  }
  __syncthreads();
  double ss = 0.0, sz = 0.0;
  for (int q = 0; q < j; ++q) {
    ss += s[q] * s[q];
    sz += s[q] * z[q];
  }
  const double nu2 = 1.0 - ss;
  const double wn = st->wn;
  if (j > 0 && !(nu2 > 1e-4)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) end_cycle(st, j - 1, wn);
    return;
  }
  const double nu = sqrt(nu2);
  const double zj = (sums[0] - sz) / nu;
  if (blockIdx.x == 0 && threadIdx.x >= TB - 64) hessenberg_column(gm, j, s, z, zj, nu, hh);
  const double inv = 1.0 / wn, inu = 1.0 / nu;
  const size_t n2 = gm.ld >> 1, ld2 = gm.ld >> 1;
  D2 *const V = reinterpret_cast<D2 *>(gm.V);
  const D2 *const wv = j == 0 ? reinterpret_cast<const D2 *>(gm.r) : V + (size_t)j * ld2;
  double acc[1] = {0.0};
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n2; i += (size_t)gridDim.x * TB) {
    D2 w = wv[i], u = V[(size_t)(j + 1) * ld2 + i];
    w.x *= inv;
    w.y *= inv;
    for (int q0 = 0; q0 < j; q0 += kQ) {
      D2 v[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[q] = V[(size_t)min(q0 + q, j - 1) * ld2 + i];
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const double sq = s[q0 + q], zq = z[q0 + q];
        w.x -= sq * v[q].x;
        w.y -= sq * v[q].y;
        u.x -= zq * v[q].x;
        u.y -= zq * v[q].y;
      }
    }
    w.x *= inu;
    w.y *= inu;
    u.x = (u.x - zj * w.x) * inu;
    u.y = (u.y - zj * w.y) * inu;
    V[(size_t)j * ld2 + i] = w;
    V[(size_t)(j + 1) * ld2 + i] = u;
    acc[0] += u.x * u.x + u.y * u.y;
  }
  put_partials<1>(acc, 1, lds, gm.p2);
}

// End of a cycle of n columns: y = R^-1 g (upper triangular, a column at a
// time over the lanes of one wave) and x += V y.
__global__ __launch_bounds__(TB) void k_gm_update(GmBuf gm, double *__restrict__ x) {
  __shared__ double y[kMaxRestart];
  __shared__ bool off;
  const GmState *const st = gm.st;
  if (threadIdx.x == 0) off = tail_off(st);
  __syncthreads();
  if (off) return;
  const int n = st->end_at + 1;
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;  // n <= 64: one row per lane
    double g = lane < n - 1 ? st->g[lane] : (lane == n - 1 ? st->g_end : 0.0);
    for (int k = n - 1; k >= 0; --k) {
      const double *const col = st->R + (size_t)k * (kMaxRestart + 1);
      const double d = col[k], gk = __shfl(g, k);
      const double yk = d != 0.0 ? gk / d : 0.0;
      if (lane == k) y[k] = yk;
      if (lane < k) g -= col[lane] * yk;
    }
  }
  __syncthreads();
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < gm.n3; i += (size_t)gridDim.x * TB) {
    double xi = x[i];
#pragma unroll 8
    for (int q = 0; q < n; ++q) xi += y[q] * gm.V[(size_t)q * gm.ld + i];
    x[i] = xi;
  }
}

// r = b - A x and the partial sums of r.r (beside those of b.b), at the
// start or after a cycle
template <int DIM, bool TR, typename MT>
__global__ __launch_bounds__(kOpThreads<DIM>, DIM == 3 ? NW3 / 4 : 1) void k_gm_residual(KParams kp, GmBuf gm, const MT *__restrict__ M,
                                                                 const double *__restrict__ x, int start) {
  __shared__ double lds[kOpWaves<DIM>];
  __shared__ Shared<DIM> sh;
  __shared__ bool off;
  if (threadIdx.x == 0) off = start ? gm.st->code != 0 : tail_off(gm.st);
  __syncthreads();
  if (off) return;
  const size_t N = (size_t)kp.ncells;
  double acc[1] = {0.0}, bg[3];
  auto pre = [&](int g) {
#pragma unroll
    for (int q = 0; q < 3; ++q) bg[q] = gm.b[q * N + g];
  };
  apply_all<DIM, TR, MT>(kp, M, x, sh, pre, [&](int g, const double *, const double *y) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double rq = bg[q] - y[q];
      gm.r[q * N + g] = rq;
      acc[0] += rq * rq;
    }
  });
  put_partials<1, kOpWaves<DIM>>(acc, 1, lds, gm.p3 + gridDim.x);
}

// The true residual's test.  True when the solve has ended (converged, at
// the start or now, or at its iteration limit) and the caller's update is
// due; else a new cycle starts.  Every block takes the same decision; block
// 0 records it.
__device__ __forceinline__ bool solve_ended(const GmBuf &gm) {
  __shared__ double rr[1];
  __shared__ int how;  // 0: nothing to do; 1: ended at the start; 2: to be tested
  GmState *const st = gm.st;
  if (threadIdx.x == 0) how = st->code != 0 ? 0 : (st->done == kGmAtStart ? 1 : (st->end_at < 0 ? 0 : 2));
  get_sums(gm.p3 + gm.na, gm.na, 1, rr);
  if (how < 2) return how == 1;
  const double beta = sqrt(rr[0]);
  const double bnorm = st->bnorm;
  const bool bad = !isfinite(beta);
  const bool conv = beta <= st->tol;
  const bool ended = !bad && (conv || st->total_it >= gm.maxit);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->rel = bnorm > 0 ? beta / bnorm : 0.0;
    if (bad)
      st->code = kGmBadResidual;
    else if (ended)
      st->done = conv ? kGmConverged : kGmAtLimit;
    else {
      st->end_at = -1;
      ++st->cycle;
    }
  }
  return ended;
}

// End of the forward solve: the test, then B^{n+1} = B^n - c dt C_NC E_th and
// E^{n+1} = (E_th - (1 - th) E^n) / th.
template <int DIM>
__global__ __launch_bounds__(TB) void k_gm_finish(KParams kp, GmBuf gm, const double *En, const double *Bn,
                                                  const double *__restrict__ Eth, double *En1, double *Bn1) {
  if (!solve_ended(gm)) return;
  const size_t N = (size_t)kp.ncells;
  const double th = kp.theta;
  const Groups gr = block_groups(node_groups(kp));
  for (int grp = gr.first; grp < gr.last; grp += gr.step) {
    int i, j, k;
    const int g = group_node<DIM>(kp, grp, i, j, k);
    if (g < 0) continue;
    double c[3][8], cc[3];
    load_cube<DIM>(kp, Eth, i, j, k, c);
    cube_curl<DIM>(kp, c, cc);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      Bn1[q * N + g] = Bn[q * N + g] - kp.c * kp.dt * cc[q];
      En1[q * N + g] = (Eth[q * N + g] - (1.0 - th) * En[q * N + g]) / th;
    }
  }
}

// End of the transposed solve: the test, then l_En += -(1 - th)/th l_E1 + mu
// and l_Bn += l_B1 + c th dt C_NC mu (C_CN^T = C_NC).
template <int DIM>
__global__ __launch_bounds__(TB) void k_gm_adj_finish(KParams kp, GmBuf gm, const double *lE1, const double *lB1,
                                                      const double *__restrict__ mu, double *lEn, double *lBn) {
  if (!solve_ended(gm)) return;
  const size_t N = (size_t)kp.ncells;
  const double th = kp.theta, ctdt = kp.c * kp.theta * kp.dt;
  const Groups gr = block_groups(node_groups(kp));
  for (int grp = gr.first; grp < gr.last; grp += gr.step) {
    int i, j, k;
    const int g = group_node<DIM>(kp, grp, i, j, k);
    if (g < 0) continue;
    double c[3][8], cc[3];
    load_cube<DIM>(kp, mu, i, j, k, c);
    cube_curl<DIM>(kp, c, cc);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      lEn[q * N + g] += -(1.0 - th) / th * lE1[q * N + g] + mu[q * N + g];
      lBn[q * N + g] += lB1[q * N + g] + ctdt * cc[q];
    }
  }
}


// KERNEL(DIM, TR, MT) for the solve's dimension, transposition and M's type
#define RELSIM_GM_MASS(KERNEL)                                   \
  do {                                                           \
    if (kp.dim == 2) {                                           \
      if (transpose) {                                           \
        if (mass_fp32) KERNEL(2, true, float);                   \
        else KERNEL(2, true, double);                            \
      } else {                                                   \
        if (mass_fp32) KERNEL(2, false, float);                  \
        else KERNEL(2, false, double);                           \
      }                                                          \
    } else {                                                     \
      if (transpose) {                                           \
        if (mass_fp32) KERNEL(3, true, float);                   \
        else KERNEL(3, true, double);                            \
      } else {                                                   \
        if (mass_fp32) KERNEL(3, false, float);                  \
        else KERNEL(3, false, double);                           \
      }                                                          \
    }                                                            \
  } while (0)

// The operator sums a column's dots along the way while the sums fit beside it in
// the registers: 16 vectors in 2D (12 registers spilled with M in FP64, none in
// FP32), 8 in 3D.  Past that k_gm_dots sums them all from a second read of w~ and
// u.  Before that the operator had variants of 16 (3D), 32 and 64 vectors that
// spilled up to 638 registers; ms for 14 and 25 steps of 30 and 60 of 64, then and
// now: 256 x 128 x 128 26.2, 53.4, 214 and 25.3, 47.8, 151; 64 x 48 x 40 0.98,
// 2.31, 12.7 and 0.94, 1.92, 7.0; 625 x 625 1.15, 2.91, 13.3 and 1.15, 2.71, 12.2.
template <int DIM, bool TR, typename MT>
void gm_apply(const KParams &kp, const GmBuf &gm, const void *Mv, int j, bool cycle0, int nb, hipStream_t st) {
  const MT *M = static_cast<const MT *>(Mv);
#define RELSIM_GM_APPLY(NV, FIRST)                                                                                  \
  hipLaunchKernelGGL((k_gm_apply<DIM, TR, MT, NV, FIRST>), dim3(nb), dim3(kOpThreads<DIM>), 0, st, kp, gm, M, j,    \
                     cycle0 ? 1 : 0)
  if (j == 0)
    RELSIM_GM_APPLY(0, true);
  else if (j <= 8)
    RELSIM_GM_APPLY(8, false);
  else if (DIM == 2 && j <= 16)
    RELSIM_GM_APPLY(DIM == 2 ? 16 : 8, false);
  else {
    RELSIM_GM_APPLY(0, false);
    // the call after the last column only finds the cycle's end
    if (j < gm.m) hipLaunchKernelGGL(k_gm_dots, dim3(nb), dim3(kDotThreads), 0, st, gm, j);
  }
#undef RELSIM_GM_APPLY
}

void gm_residual(const KParams &kp, const GmBuf &gm, int mass_fp32, bool transpose, const void *M, const double *x,
                 bool start, hipStream_t st) {
#define RELSIM_RES(DIM, TR, MT)                                                                                       \
  hipLaunchKernelGGL((k_gm_residual<DIM, TR, MT>), dim3(gm.na), dim3(kOpThreads<DIM>), 0, st, kp, gm,                 \
                     static_cast<const MT *>(M), x, start ? 1 : 0)
  RELSIM_GM_MASS(RELSIM_RES);
#undef RELSIM_RES
}

}  // namespace

void launch_apply(const KParams &kp, int mass_fp32, bool transpose, const void *M, const double *x, double *y,
                  hipStream_t st) {
  const int nb = kp.dim == 2 ? node_groups(kp) : Tiles3(kp).count();
#define RELSIM_APPLY(DIM, TR, MT)                                                                        \
  hipLaunchKernelGGL((k_apply<DIM, TR, MT>), dim3(nb), dim3(kOpThreads<DIM>), 0, st, kp,                 \
                     static_cast<const MT *>(M), x, y)
  RELSIM_GM_MASS(RELSIM_APPLY);
#undef RELSIM_APPLY
}

// Tile extents of the 3D operator: rows of at most 62 nodes (a lane on either
// side is the neighbour's), and the ty <= kRows3 rows and lz planes for which
// the tiles read least, each with 9 of the 14 blocks of a row and of a plane
// of its neighbours, while the tiles, one to a CU at a time, keep 85 % of the
// 256 CUs busy; fewer busy CUs count against them in proportion.  Solve, us, M in
// FP64, with 70, 85 and 95 %: 64 x 48 x 40 639, 588 and 579, 96 x 47 x 33 628, 650
// and 676, 128 x 64 x 64 2291, 2094 and 2106, 120 x 100 x 90 3980, 3773 and 3772,
// 256 x 128 x 128 14820, 14880 and 13690.  The width of a row is not weighed: one
// of 64 nodes takes two tiles of 32 in 34 of the 64 lanes, one of 16 nodes 18.
void plan_tiles3(KParams &kp) {
  const int ntx = (kp.nx + 61) / 62;
  kp.t3x = (kp.nx + ntx - 1) / ntx;
  kp.t3y = kp.t3z = 0;
  double best = 0.0;
  for (int ty = kRows3 < kp.ny ? kRows3 : kp.ny; ty >= 1; --ty)
    for (int lz = kp.nz; lz >= 1; --lz) {
      const double tiles = (double)ntx * ((kp.ny + ty - 1) / ty) * ((kp.nz + lz - 1) / lz);
      const double busy = tiles / (256.0 * ceil(tiles / 256.0)) / 0.85;
      const double cost = tiles * (ty + 9.0 / 14.0) * (lz + 9.0 / 14.0) / (busy < 1.0 ? busy : 1.0);
      if (kp.t3z == 0 || cost < best) {
        best = cost;
        kp.t3y = ty;
        kp.t3z = lz;
      }
    }
}

void gm_blocks(const KParams &kp, GmBuf &gm) {
  if (kp.dim == 3) {
    const int nt = Tiles3(kp).count();
    gm.na = nt < kGmTileBlocks ? nt : kGmTileBlocks;
  } else {
    const int ng = node_groups(kp);
    gm.na = ng < kGmNodeBlocks ? ng : kGmNodeBlocks;
  }
  const size_t nv = (gm.ld / 2 + TB - 1) / TB;
  gm.no = nv < (size_t)kGmVecBlocks ? (int)nv : kGmVecBlocks;
}

void launch_gm_start(const KParams &kp, const GmBuf &gm, int mass_fp32, const void *M, const double *En,
                     const double *Bn, const double *J, const double *x0, double *x, const int32_t *flags,
                     hipStream_t st) {
  const int nb = gm.na;
  if (kp.dim == 2)
    hipLaunchKernelGGL(k_gm_rhs<2>, dim3(nb), dim3(TB), 0, st, kp, gm, En, Bn, J, x0, x, flags);
  else
    hipLaunchKernelGGL(k_gm_rhs<3>, dim3(nb), dim3(TB), 0, st, kp, gm, En, Bn, J, x0, x, flags);
  gm_residual(kp, gm, mass_fp32, false, M, x, true, st);
}

void launch_gm_adj_start(const KParams &kp, const GmBuf &gm, const double *lth, const double *lE1, const double *lB1,
                         double *x, const int32_t *flags, hipStream_t st) {
  const int nb = gm.na;
  if (kp.dim == 2)
    hipLaunchKernelGGL(k_gm_adj_start<2>, dim3(nb), dim3(TB), 0, st, kp, gm, lth, lE1, lB1, x, flags);
  else
    hipLaunchKernelGGL(k_gm_adj_start<3>, dim3(nb), dim3(TB), 0, st, kp, gm, lth, lE1, lB1, x, flags);
}

void launch_gm_apply(const KParams &kp, const GmBuf &gm, int mass_fp32, bool transpose, const void *M, int j,
                     bool cycle0, hipStream_t st) {
  const int nb = gm.na;
#define RELSIM_STEP(DIM, TR, MT) gm_apply<DIM, TR, MT>(kp, gm, M, j, cycle0, nb, st)
  RELSIM_GM_MASS(RELSIM_STEP);
#undef RELSIM_STEP
}

void launch_gm_ortho(const GmBuf &gm, int j, hipStream_t st) {
  hipLaunchKernelGGL(k_gm_ortho, dim3(gm.no), dim3(TB), 0, st, gm, j);
}

void launch_gm_update(const GmBuf &gm, double *x, hipStream_t st) {
  hipLaunchKernelGGL(k_gm_update, dim3(gm.no), dim3(TB), 0, st, gm, x);
}

void launch_gm_residual(const KParams &kp, const GmBuf &gm, int mass_fp32, bool transpose, const void *M,
                        const double *x, hipStream_t st) {
  gm_residual(kp, gm, mass_fp32, transpose, M, x, false, st);
}

void launch_gm_finish(const KParams &kp, const GmBuf &gm, const double *En, const double *Bn, const double *Eth,
                      double *En1, double *Bn1, hipStream_t st) {
  const int nb = node_groups(kp);
  if (kp.dim == 2)
    hipLaunchKernelGGL(k_gm_finish<2>, dim3(nb), dim3(TB), 0, st, kp, gm, En, Bn, Eth, En1, Bn1);
  else
    hipLaunchKernelGGL(k_gm_finish<3>, dim3(nb), dim3(TB), 0, st, kp, gm, En, Bn, Eth, En1, Bn1);
}

void launch_gm_adj_finish(const KParams &kp, const GmBuf &gm, const double *lE1, const double *lB1, const double *mu,
                          double *lEn, double *lBn, hipStream_t st) {
  const int nb = node_groups(kp);
  if (kp.dim == 2)
    hipLaunchKernelGGL(k_gm_adj_finish<2>, dim3(nb), dim3(TB), 0, st, kp, gm, lE1, lB1, mu, lEn, lBn);
  else
    hipLaunchKernelGGL(k_gm_adj_finish<3>, dim3(nb), dim3(TB), 0, st, kp, gm, lE1, lB1, mu, lEn, lBn);
}

}  // namespace relsim
