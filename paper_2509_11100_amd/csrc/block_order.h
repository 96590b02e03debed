// Which work item a workgroup takes.  Consecutive workgroups are dispatched to
// the 8 XCDs round robin, and items next to each other (cells, segments,
// nodes) share lines of memory, so an XCD, with its L2, should get runs of
// consecutive items.
#pragma once

namespace relsim {

// One run per XCD, the last nb % 8 items as they come.
__host__ __device__ inline int xcd_bands(int b, int nb) {
  const int q = nb >> 3;
  if (b >= (q << 3)) return b;
  return (b & 7) * q + (b >> 3);
}

// Runs of `chunk` items going round the XCDs, so that a band of the grid that
// holds more particles than the rest is spread over all XCDs.  What is left
// after the last whole round of 8 chunks (all of it, on a small grid) is cut
// into one run per XCD.
__host__ __device__ inline int xcd_chunks(int b, int nb, int chunk) {
  const int round = chunk << 3, full = nb / round * round;
  if (b >= full) return full + xcd_bands(b - full, nb - full);
  const int i = b >> 3, c = i / chunk;
  return (c * 8 + (b & 7)) * chunk + (i - c * chunk);
}

// The 2D deposit's blocks of 64 / G cells.  One run per XCD leaves most of the
// particles of a sheet with crowded rows to a few XCDs, so on larger grids an
// XCD takes 512 cells (4 tiles of 16 x 8, whole rows of the stored moments) at a
// time: deposit and assembly, us, one run per XCD and in chunks, mixed, 625 x
// 625 reconnection sheet 282 and 264 (FP64 515 and 454; chunks of 1024 and
// 2048 cells, mixed: 280, 322), 1000 x 64 cells of it 129 and 96, 512 x 256
// evenly filled 96 and 94.  On small grids a chunk is a large part of the grid
// and its ends count: 120 x 120 cells of the reconnection sheet 97 and 101, 100
// x 77 evenly filled 24.4 and 25.4, 200 x 102 31.8 and 32.4.
constexpr int kDepositBands = 49152;  // cells up to which each XCD takes one run
__host__ __device__ inline int deposit_block(int b, int nb, int G, int ncells) {
  return ncells <= kDepositBands ? xcd_bands(b, nb) : xcd_chunks(b, nb, 8 * G);
}

// Extent of equal tiles of about `cap` that cover n places: n / cap rounded
// down or up tiles, whichever reaches less far past n, with at most `most`
// places in one.
__host__ __device__ inline int even_tile(int n, int cap, int most) {
  const int hi = (n + cap - 1) / cap, lo = n / cap > 0 ? n / cap : 1;
  const int eh = (n + hi - 1) / hi, el = (n + lo - 1) / lo;
  return el <= most && el * lo < eh * hi ? el : eh;
}

// Segments of a row that the push passes' tiles hold side by side, of rows of
// nseg segments of C cells: in 2D tiles of about 16 cells, in 3D one segment.
// A tile's width that does not divide the row leaves places without cells,
// each of them a wave: 40 x 96 x 96 cells, whose rows are 5 segments of 8, lost
// 24 of 280 us of the scatter with two side by side.
__host__ __device__ inline int tile_segments(int dim, int nseg, int C) {
  const int cap = dim == 2 && C < 16 ? 16 / C : 1;
  return even_tile(nseg, cap, 2 * cap);
}

}  // namespace relsim
