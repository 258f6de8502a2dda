// FP64 set-up kernels of the boxes: Psi1 / Psi2 at the box particles and the LEP boundary
// potential Phi_BC^0, from the Lagrangian potentials phi1 / phi2 on the periodic LPT grid
// (kernels_fft.hip).
//
// Paper: Sec. 3.3 (C.1-C.3: exact Psi in the box, Phi_BCs interpolated from the LPT grid to
// the PM grid), Sec. 3 (finite differences of order 2, 4 or 6: ng = 1, 2, 3 neighbours per
// side; Sec. 4 runs order 2).
#include "common.h"
#include "kernels.h"
#include "particle_common.h"

namespace scola {

namespace {

// C.1-C.2: Psi1 = D phi1 and Psi2 = D phi2 at every box particle, differenced in FP64 and
// stored in the plan precision (FP32 plans keep the paper's single-precision particle record);
// also the operator L- (x_res = p_res = 0).  One block per brick.
//
// LPT grid of N = Np nodes per side (k_extract_psi): the nodes coincide with the particles, no
// interpolation.  The brick's nodes and the stencils' reach are staged in LDS (all loads in
// flight at once; N is a power of two, so the periodic index is a mask).  Bound by memory: 48
// bytes stored per particle in FP32 and about 40 read.  The stores are streams as large as
// the evolution's state, so they bypass the caches, where neighbouring bricks find each
// other's nodes; an XCD takes runs of four of them (kXcdRuns) in large plans: for the 80 million particles of
// the mixed 256^3 tiling 1.48 ms before, 1.65 with cached stores, 1.57 with single bricks dealt
// out over the XCDs, 1.17 with a contiguous range for each, 1.12 so.
template <typename T, int NG>
__global__ void __launch_bounds__(kBlock)
k_extract_psi(const TileDesc* __restrict__ tiles, BlockMap m, const double* __restrict__ phi1,
              const double* __restrict__ phi2, T* __restrict__ psi1, T* __restrict__ psi2,
              T* __restrict__ xres, T* __restrict__ pres, int N, int64_t P) {
  const int L = logical_block(m);
  if (L >= m.count) return;
  constexpr int W = 8 + 2 * NG, WX = 4 + 2 * NG;   // the brick's sites and the stencils' reach
  __shared__ double win[2][WX * W * W];
  const TileDesc t = tiles[m.tile[L]];
  const int brick = m.local[L], nb = t.M >> 3;
  const int ox = t.origin[0] + brick / (nb * nb) * 4 - NG,
            oy = t.origin[1] + (brick / nb) % nb * 8 - NG, oz = t.origin[2] + brick % nb * 8 - NG;
  const int mask = N - 1;
  constexpr int kEach = (WX * W * W + kBlock - 1) / kBlock;
  double v1[kEach], v2[kEach];
#pragma unroll
  for (int q = 0; q < kEach; ++q) {
    const int e = min((int)threadIdx.x + q * kBlock, WX * W * W - 1);
    const int x = e / (W * W), y = e / W % W, z = e % W;
    const unsigned g =
        (unsigned)((((ox + x) & mask) * N + ((oy + y) & mask)) * N + ((oz + z) & mask));
    v1[q] = phi1[g];
    v2[q] = phi2[g];
  }
#pragma unroll
  for (int q = 0; q < kEach; ++q) {
    const int e = min((int)threadIdx.x + q * kBlock, WX * W * W - 1);
    win[0][e] = v1[q];
    win[1][e] = v2[q];
  }
  __syncthreads();
  const int w = threadIdx.x;
  const int at = (((w >> 6) + NG) * W + ((w >> 3) & 7) + NG) * W + (w & 7) + NG;
  double s1[3] = {0.0, 0.0, 0.0}, s2[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 1; q <= NG; ++q) {
    const int d[3] = {q * W * W, q * W, q};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double d1 = win[0][at + d[c]] - win[0][at - d[c]];
      const double d2 = win[1][at + d[c]] - win[1][at - d[c]];
      if constexpr (NG == 1) {
        s1[c] = 0.5 * d1;
        s2[c] = 0.5 * d2;
      } else {
        s1[c] += first_difference_weight(NG, q) * d1;
        s2[c] += first_difference_weight(NG, q) * d2;
      }
    }
  }
  const int64_t p = t.p_off + (int64_t)brick * kBlock + w;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    __builtin_nontemporal_store((T)s1[c], psi1 + c * P + p);
    __builtin_nontemporal_store((T)s2[c], psi2 + c * P + p);
    __builtin_nontemporal_store(T(0), xres + c * P + p);
    __builtin_nontemporal_store(T(0), pres + c * P + p);
  }
}

// N < Np (Np / N a power of two): LPT node m sits at the centre (m + 1/2) Np / N of its cell;
// the gradient at the 8 nodes around the particle's LPT coordinate u = (g + 1/2) N / Np - 1/2
// is interpolated by CiC and converted from LPT-grid cells to lattice cells (x Np / N).  A
// brick's particles share few nodes (at most 6 x 6 x 4 and the stencil's reach, as N / Np <=
// 1/2), which the block stages in LDS; along its own axis the gradient and the interpolation
// are one stencil of 2 NG + 2 nodes.  (With 96 global loads per particle at 8 corners it took
// 0.99 ms for 16.8 million particles on an LPT grid of 64^3, now 0.25.)
template <typename T, int NG>
__global__ void __launch_bounds__(kBlock)
k_interpolate_psi(const TileDesc* __restrict__ tiles, BlockMap m, const double* __restrict__ phi1,
                  const double* __restrict__ phi2, T* __restrict__ psi1, T* __restrict__ psi2,
                  T* __restrict__ xres, T* __restrict__ pres, int N, int64_t P, int Np) {
  // nodes of a brick per axis: floor(u) spans at most 5 values over 8 sites and 3 over 4, one
  // more for the upper corner, NG more on each side
  constexpr int W = 6 + 2 * NG, WX = 4 + 2 * NG;
  __shared__ double win[2][WX * W * W];
  const int L = logical_block(m);
  if (L >= m.count) return;
  const TileDesc t = tiles[m.tile[L]];
  const int brick = m.local[L], nb = t.M >> 3;
  const double r = (double)N / (double)Np;
  const int g0[3] = {t.origin[0] + brick / (nb * nb) * 4, t.origin[1] + (brick / nb) % nb * 8,
                     t.origin[2] + brick % nb * 8};
  int o[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) o[c] = (int)floor(((double)g0[c] + 0.5) * r - 0.5) - NG;
  for (int e = threadIdx.x; e < WX * W * W; e += kBlock) {
    const int x = e / (W * W), y = (e / W) % W, z = e % W;
    const int64_t a = ((int64_t)((o[0] + x) & (N - 1)) * N + ((o[1] + y) & (N - 1))) * N +
                      ((o[2] + z) & (N - 1));
    win[0][e] = phi1[a];
    win[1][e] = phi2[a];
  }
  __syncthreads();
  const int w = threadIdx.x;
  const int g[3] = {g0[0] + (w >> 6), g0[1] + ((w >> 3) & 7), g0[2] + (w & 7)};
  int b[3];
  double wt[3][2], h[3][2 * NG + 2];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double u = ((double)g[c] + 0.5) * r - 0.5, fl = floor(u);
    b[c] = (int)fl - NG - o[c];
    wt[c][1] = u - fl;
    wt[c][0] = 1.0 - wt[c][1];
#pragma unroll
    for (int q = 0; q < 2 * NG + 2; ++q) h[c][q] = 0.0;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int q = 1; q <= NG; ++q) {
        h[c][NG + d + q] += wt[c][d] * first_difference_weight(NG, q);
        h[c][NG + d - q] -= wt[c][d] * first_difference_weight(NG, q);
      }
  }
  const int base = (b[0] * W + b[1]) * W + b[2];
  const int64_t p = t.p_off + (int64_t)brick * kBlock + w;
  const double scale = (double)Np / (double)N;
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const double* const s = win[f] + base;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < 2 * NG + 2; ++q) {
          v[0] += wt[1][d] * wt[2][e] * h[0][q] * s[(q * W + NG + d) * W + NG + e];
          v[1] += wt[0][d] * wt[2][e] * h[1][q] * s[((NG + d) * W + q) * W + NG + e];
          v[2] += wt[0][d] * wt[1][e] * h[2][q] * s[((NG + d) * W + NG + e) * W + q];
        }
    T* const out = f ? psi2 : psi1;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      __builtin_nontemporal_store((T)(scale * v[c]), out + c * P + p);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    __builtin_nontemporal_store(T(0), xres + c * P + p);
    __builtin_nontemporal_store(T(0), pres + c * P + p);
  }
}

// C.3: Phi_BC^0 at the padded PM nodes j in [-ng, M+ng]^3 outside [1, M-1]^3: trilinear
// interpolation of phi1 at the PM node, i.e. with N = Np the mean of the 8 LPT nodes around
// it (PM nodes sit half a cell from the LPT nodes).  Interior entries are set to zero.  One
// block per x plane of a box; on interior planes the zeros are stored first and the border's
// nodes then taken one per thread, so that a block waits for its loads three times instead of
// once per row and column (mixed 256^3 tiling: 0.51 ms, now 0.26).
__global__ void __launch_bounds__(kBlock)
k_boundary_potential(const TileDesc* __restrict__ tiles, const double* __restrict__ phi1,
                     double* __restrict__ bc0, int N, int ng, int Np) {
  const TileDesc t = tiles[blockIdx.y];
  const int M = t.M, Mp = M + 1 + 2 * ng, mask = N - 1;
  if ((int)blockIdx.x >= Mp) return;
  const int a = (int)blockIdx.x - ng;
  const bool ain = a >= 1 && a <= M - 1;
  double* const out = bc0 + t.h_off + (int64_t)blockIdx.x * Mp * Mp;
  auto node = [&](int x, int y, int z) {
    return phi1[(unsigned)(((x & mask) * N + (y & mask)) * N + (z & mask))];
  };
  const double r = (double)N / (double)Np;
  auto value = [&](int b, int c) {
    double v = 0.0;
    if (N != Np) {
      // LPT grid coarser than the lattice: CiC at the node's LPT coordinate X N / Np - 1/2,
      // converted from LPT-grid cells^2 to lattice cells^2
      const int X[3] = {t.origin[0] + a, t.origin[1] + b, t.origin[2] + c};
      int m0[3];
      double w[3][2];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double u = (double)X[d] * r - 0.5;
        const double fl = floor(u);
        m0[d] = (int)fl;
        w[d][1] = u - fl;
        w[d][0] = 1.0 - w[d][1];
      }
#pragma unroll
      for (int cn = 0; cn < 8; ++cn) {
        const int dx = (cn >> 2) & 1, dy = (cn >> 1) & 1, dz = cn & 1;
        v += w[0][dx] * w[1][dy] * w[2][dz] * node(m0[0] + dx, m0[1] + dy, m0[2] + dz);
      }
      return v * (((double)Np / (double)N) * ((double)Np / (double)N));
    }
    const int gx = t.origin[0] + a, gy = t.origin[1] + b, gz = t.origin[2] + c;
#pragma unroll
    for (int dx = -1; dx <= 0; ++dx)
#pragma unroll
      for (int dy = -1; dy <= 0; ++dy)
#pragma unroll
        for (int dz = -1; dz <= 0; ++dz) v += node(gx + dx, gy + dy, gz + dz);
    return v * 0.125;
  };
  // row and column by a reciprocal (exact: fewer than 2^15 nodes)
  const float inv = 1.0f / (float)Mp;
  if (!ain) {
#pragma unroll 2
    for (int e = threadIdx.x; e < Mp * Mp; e += kBlock) {
      const int row = (int)(((float)e + 0.5f) * inv);
      out[e] = value(row - ng, e - row * Mp - ng);
    }
    return;
  }
#pragma unroll 4
  for (int e = threadIdx.x; e < Mp * Mp; e += kBlock) {
    const int row = (int)(((float)e + 0.5f) * inv);
    const int b = row - ng, c = e - row * Mp - ng;
    if (b >= 1 && b <= M - 1 && c >= 1 && c <= M - 1) out[e] = 0.0;
  }
  // border element i: the W / 2 first and last rows whole, then the W / 2 first and last
  // columns of the rows in between
  const int W = 2 * (ng + 1), border = Mp * Mp - (M - 1) * (M - 1);
#pragma unroll 2
  for (int i = threadIdx.x; i < border; i += kBlock) {
    int row, col;
    if (i < W * Mp) {
      const int q = (int)(((float)i + 0.5f) * inv);
      row = q <= ng ? q : M - 1 + q;
      col = i - q * Mp;
    } else {
      const int k = i - W * Mp, q = k / W, c = k - q * W;
      row = ng + 1 + q;
      col = c <= ng ? c : M - 1 + c;
    }
    out[row * Mp + col] = value(row - ng, col - ng);
  }
}

template <typename T, int NG>
void launch_psi(const BoxSetupArgs& a, T* xres, T* pres, hipStream_t s) {
  BlockMap m;
  m.tile = a.blk_tile;
  m.local = a.blk_first;
  m.count = a.n_blocks;
  if (a.N == a.Np && a.n_blocks > kRunBricks) m.xcd_remap = kXcdRuns;
  const dim3 grid(padded_grid(m)), block(kBlock);
  if (a.N == a.Np)
    hipLaunchKernelGGL((k_extract_psi<T, NG>), grid, block, 0, s, a.tiles, m, a.phi1, a.phi2,
                       static_cast<T*>(a.psi1), static_cast<T*>(a.psi2), xres, pres, a.N, a.P);
  else
    hipLaunchKernelGGL((k_interpolate_psi<T, NG>), grid, block, 0, s, a.tiles, m, a.phi1, a.phi2,
                       static_cast<T*>(a.psi1), static_cast<T*>(a.psi2), xres, pres, a.N, a.P,
                       a.Np);
}

}  // namespace

template <typename T>
hipError_t launch_setup_boxes(const BoxSetupArgs& a, T* xres, T* pres, hipStream_t s) {
  if (a.n_blocks > 0) {
    switch (a.ng) {
      case 1: launch_psi<T, 1>(a, xres, pres, s); break;
      case 2: launch_psi<T, 2>(a, xres, pres, s); break;
      case 3: launch_psi<T, 3>(a, xres, pres, s); break;
      default: return hipErrorInvalidValue;
    }
  }
  hipLaunchKernelGGL(k_boundary_potential, dim3(a.max_M + 1 + 2 * a.ng, a.n_tiles), dim3(kBlock),
                     0, s, a.tiles, a.phi1, a.bc0, a.N, a.ng, a.Np);
  return hipGetLastError();
}

template hipError_t launch_setup_boxes<float>(const BoxSetupArgs&, float*, float*, hipStream_t);
template hipError_t launch_setup_boxes<double>(const BoxSetupArgs&, double*, double*,
                                               hipStream_t);

}  // namespace scola
