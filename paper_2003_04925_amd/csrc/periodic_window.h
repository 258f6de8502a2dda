// CiC of a block's particles onto a periodic 64-bit fixed-point grid (the output density, the
// mass mesh of the periodic tCOLA run), privatised in LDS.
#pragma once

#include "common.h"
#include "kernels.h"
#include "particle_common.h"

namespace scola {
namespace {

__device__ __forceinline__ int wrap_node(int i, int n) {
  if (i >= 0 && i < n) return i;
  i %= n;
  return i < 0 ? i + n : i;
}

// Cells of particles at u that the block's packed extent can hold (common cell indices lie in
// [-16383, 16383]); others, and non-finite positions, work on global memory.
__device__ __forceinline__ bool periodic_cell(bool active, const double (&u)[3], int (&j0)[3],
                                              double (&f)[3]) {
  constexpr double kFar = 16000.0;
  bool in = active;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double fl = floor(u[c]);
    f[c] = u[c] - fl;
    j0[c] = (int)fl;
    in = in && u[c] > -kFar && u[c] < kFar;
  }
  return in;
}

// Adds the 2^40 units of every active particle at u (grid cells, any range) to the periodic
// n^3 grid.  The particles of a block are one Lagrangian brick, so they share nodes: the block
// accumulates in an LDS window over its cells (when that holds at most kWindow nodes) and
// flushes it with one atomic per touched node, neighbouring lanes on neighbouring nodes.
// Eight global 64-bit atomics per particle instead ran at 29 per nanosecond wherever they
// landed and bounded every kernel that used them.  Integer sums: every form gives the same
// result.  win: kWindow words, 16-byte aligned, last used before a barrier.  Called by all
// threads of the block.
__device__ __forceinline__ void periodic_deposit_block(unsigned long long* __restrict__ grid,
                                                       int n, bool active, const double (&u)[3],
                                                       unsigned long long* win, int* bounds) {
  int j0[3];
  double f[3];
  const bool in = periodic_cell(active, u, j0, f);
  long long w[8];
  split_weights<long long, double>(f[0], f[1], f[2], 1ll << 40, w);
  {
    uint4* const w4 = reinterpret_cast<uint4*>(win);
#pragma unroll
    for (int k = 0; k < kWindow * 8 / 16 / kBlock; ++k)
      w4[threadIdx.x + kBlock * k] = make_uint4(0u, 0u, 0u, 0u);
  }
  const CellRange cr = block_cells(in, j0, bounds);   // its barrier also ends the clearing
  const int wx = cr.hi[0] - cr.lo[0] + 2, wy = cr.hi[1] - cr.lo[1] + 2,
            wz = cr.hi[2] - cr.lo[2] + 2, wyz = wy * wz;
  const bool use_lds = cr.any && wx <= kWindow && wyz <= kWindow && wx * wyz <= kWindow;
  if (active && !(in && use_lds)) {
    // fmod: any finite position wraps as the reals do
#pragma unroll
    for (int c = 0; c < 3; ++c) j0[c] = wrap_node((int)fmod(floor(u[c]), (double)n), n);
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (w[c] != 0)
        atomicAdd(grid + ((int64_t)wrap_node(j0[0] + ((c >> 2) & 1), n) * n +
                          wrap_node(j0[1] + ((c >> 1) & 1), n)) * n +
                      wrap_node(j0[2] + (c & 1), n), (unsigned long long)w[c]);
  }
  if (!use_lds) return;
  if (in) {
    unsigned long long* const p =
        win + ((j0[0] - cr.lo[0]) * wyz + (j0[1] - cr.lo[1]) * wz + (j0[2] - cr.lo[2]));
#pragma unroll
    for (int c = 0; c < 8; ++c)
      atomicAdd(p + ((c >> 2) & 1) * wyz + ((c >> 1) & 1) * wz + (c & 1),
                (unsigned long long)w[c]);
  }
  __syncthreads();
  // each thread takes a (y, z) column of the window and walks it along x
  const float inv_wz = 1.0f / (float)wz;
  const int x0 = wrap_node(cr.lo[0], n);
  for (int pos = threadIdx.x; pos < wyz; pos += kBlock) {
    const int y = (int)(((float)pos + 0.5f) * inv_wz), z = pos - y * wz;
    unsigned long long* const col =
        grid + ((int64_t)wrap_node(cr.lo[1] + y, n) * n + wrap_node(cr.lo[2] + z, n));
    int xw = x0;
    for (int x = 0; x < wx; ++x) {
      const unsigned long long v = win[pos + x * wyz];
      if (v != 0) atomicAdd(col + (int64_t)xw * n * n, v);
      if (++xw == n) xw = 0;
    }
  }
}

// A position in cells taken into [0, n): fmod's result, without its loop where it is the
// identity.
__device__ __forceinline__ double wrap_position(double x, double n) {
  if (x >= 0.0 && x < n) return x;
  x = fmod(x, n);
  return x < 0 ? x + n : x;
}

}  // namespace
}  // namespace scola
