// Grid kernels, all FP64: the discrete curls (see field_stencil.h) and the
// fixed-order reductions of the energies.
#include "field_stencil.h"

namespace relsim {
namespace {

template <int DIM>
__global__ __launch_bounds__(256) void k_curl(KParams kp, const double *__restrict__ in, double *__restrict__ out,
                                              int shift) {
  int i, j, k;
  const int g = strip_node(kp.nx, kp.ny, kp.nz, xcd_bands(blockIdx.x, gridDim.x) * 4 + (int)(threadIdx.x >> 6),
                           (int)(threadIdx.x & 63), i, j, k);
  if (g < 0) return;
  double c[3][8], r[3];
  load_cube<DIM>(kp, in, i - shift, j - shift, k - shift, c);
  cube_curl<DIM>(kp, c, r);
  const size_t N = (size_t)kp.ncells;
  out[g] = r[0];
  out[N + g] = r[1];
  out[2 * N + g] = r[2];
}

// ---- fixed-order reductions ----
__device__ __forceinline__ double block_sum_256(double v, double *lds) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  if (lane == 0) lds[wid] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (lds[0] + lds[1]) + (lds[2] + lds[3]);
  __syncthreads();
  return r;
}

// res[kv] = the sum over b of partials[b * nvec + kv], one block per kv.
__global__ __launch_bounds__(256) void k_reduce_partials(const double *__restrict__ partials, int nparts, int nvec,
                                                         double *__restrict__ res) {
  __shared__ double lds[4];
  const int kv = blockIdx.x;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nparts; b += 256) acc += partials[(size_t)b * nvec + kv];
  const double s = block_sum_256(acc, lds);
  if (threadIdx.x == 0) res[kv] = s;
}

// Sums of consecutive chunks of a long array of partial sums, one block per
// chunk, in a fixed order.
__global__ __launch_bounds__(256) void k_reduce_chunks(const double *__restrict__ in, int n, int chunk,
                                                       double *__restrict__ out) {
  __shared__ double lds[4];
  const int b0 = blockIdx.x * chunk;
  const int b1 = b0 + chunk < n ? b0 + chunk : n;
  double acc = 0.0;
  for (int i = b0 + threadIdx.x; i < b1; i += 256) acc += in[i];
  const double s = block_sum_256(acc, lds);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_sumsq(const double *__restrict__ x, size_t n, double *__restrict__ partials) {
  __shared__ double lds[4];
  const size_t chunk = (n + gridDim.x - 1) / gridDim.x;
  const size_t beg = (size_t)blockIdx.x * chunk;
  const size_t end = beg + chunk < n ? beg + chunk : n;
  double acc = 0.0;
  for (size_t i = beg + threadIdx.x; i < end; i += 256) acc += x[i] * x[i];
  const double s = block_sum_256(acc, lds);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// blocks of the per-node kernels (strip node order)
inline int node_blocks(const KParams &kp) { return grid_node_blocks(kp.nx, kp.ny, kp.nz); }

}  // namespace

void launch_curl(const KParams &kp, const double *in, double *out, int to_centres, hipStream_t st) {
  const int shift = to_centres ? 0 : 1;
  if (kp.dim == 2)
    hipLaunchKernelGGL(k_curl<2>, dim3(node_blocks(kp)), dim3(256), 0, st, kp, in, out, shift);
  else
    hipLaunchKernelGGL(k_curl<3>, dim3(node_blocks(kp)), dim3(256), 0, st, kp, in, out, shift);
}

void launch_sumsq_partials(const double *x, size_t n, double *partials, hipStream_t st) {
  hipLaunchKernelGGL(k_sumsq, dim3(kRedBlocks), dim3(256), 0, st, x, n, partials);
}

void launch_reduce_partials(const double *partials, int nparts, int nvec, double *res, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_partials, dim3(nvec), dim3(256), 0, st, partials, nparts, nvec, res);
}

void launch_reduce_long(const double *in, int n, double *tmp, double *res, hipStream_t st) {
  const int chunk = (n + kRedBlocks - 1) / kRedBlocks;
  hipLaunchKernelGGL(k_reduce_chunks, dim3(kRedBlocks), dim3(256), 0, st, in, n, chunk > 0 ? chunk : 1, tmp);
  hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(256), 0, st, tmp, kRedBlocks, 1, res);
}

}  // namespace relsim
