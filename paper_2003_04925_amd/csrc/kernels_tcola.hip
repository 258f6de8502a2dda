// Monolithic periodic tCOLA (Sec. 2.2, App. A eqs. drift-cola and kick-tcola, App. B): the
// whole box of N^3 particles evolved at once with a periodic PM grid of N^3 nodes, so no
// tiling approximation is made.  It is the reference the sCOLA boxes are compared with
// (Sec. 4.2) and the source of the true density and potential of the consistency tests
// (Sec. 4.3).
//
// The operators are those of the boxes without the box cut: CiC deposit onto the periodic
// node grid (nodes at integer positions, one per lattice cell, global mean density one
// particle per cell), the Poisson equation solved in Fourier space with the symbol of the
// finite-difference Laplacian of the plan's order (-4 sum sin^2(k/2) at order 2, zero mode
// removed), the central-difference gradient of the same order and CiC interpolation, then
// the same COLA kick and drift.  Particles are in lattice order; every
// position is formed in FP64 as in the box kernels; deposits are 64-bit fixed point (2^40
// units per particle), exact and order independent.  The Poisson solve is the FP64 periodic
// one of kernels_fft.hip.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "particle_common.h"
#include "particle_step.h"
#include "periodic_window.h"

namespace scola {

namespace {

__device__ __forceinline__ int pwrap(int i, int N) { return i & (N - 1); }   // N: power of 2

// Psi1 = D phi1, Psi2 = D phi2 (order-2 central differences) at every lattice site, and
// the operator L- (x_res = p_res = 0).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_tcola_setup(TcolaArgs<T> a, const double* phi1,
                                                        const double* phi2) {
  const int N = a.N;
  const int64_t n3 = (int64_t)N * N * N;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n3) return;
  const int x = (int)(p / ((int64_t)N * N)), y = (int)((p / N) % N), z = (int)(p % N);
  auto at = [&](const double* f, int i, int j, int k) {
    return f[((int64_t)pwrap(i, N) * N + pwrap(j, N)) * N + pwrap(k, N)];
  };
  T* s1 = const_cast<T*>(a.psi1);
  T* s2 = const_cast<T*>(a.psi2);
  double g1[3] = {0.0, 0.0, 0.0}, g2[3] = {0.0, 0.0, 0.0};
  for (int k = 1; k <= a.ng; ++k) {
    const double c = first_difference_weight(a.ng, k);
    g1[0] += c * (at(phi1, x + k, y, z) - at(phi1, x - k, y, z));
    g1[1] += c * (at(phi1, x, y + k, z) - at(phi1, x, y - k, z));
    g1[2] += c * (at(phi1, x, y, z + k) - at(phi1, x, y, z - k));
    g2[0] += c * (at(phi2, x + k, y, z) - at(phi2, x - k, y, z));
    g2[1] += c * (at(phi2, x, y + k, z) - at(phi2, x, y - k, z));
    g2[2] += c * (at(phi2, x, y, z + k) - at(phi2, x, y, z - k));
  }
  for (int c = 0; c < 3; ++c) {
    s1[c * n3 + p] = (T)g1[c];
    s2[c * n3 + p] = (T)g2[c];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    a.xres[c * n3 + p] = T(0);
    a.pres[c * n3 + p] = T(0);
  }
}

// The lattice site and array index of this thread: a block is a brick of 4 x 8 x 8 sites, so
// that its particles share mesh nodes (the arrays are in lattice order: rows of 8 values).  Each
// XCD takes a contiguous range of bricks (N >= 16, whose bricks divide evenly): the four bricks
// that share the arrays' 128-byte lines and the mesh nodes of neighbours then meet in one L2
// (particle step of 128^3: 100 us with bricks dealt to the XCDs in turn, 67 so).
__device__ __forceinline__ int64_t tcola_site(int N, int (&idx)[3]) {
  const int nb = N >> 3, w = threadIdx.x;
  int b = blockIdx.x;
  if ((gridDim.x & 7) == 0) b = (b & 7) * (int)(gridDim.x >> 3) + (b >> 3);
  idx[0] = b / (nb * nb) * 4 + (w >> 6);
  idx[1] = b / nb % nb * 8 + ((w >> 3) & 7);
  idx[2] = b % nb * 8 + (w & 7);
  return ((int64_t)idx[0] * N + idx[1]) * N + idx[2];
}

// Central-difference gradient (order 2 NG) of the periodic potential at the 8 CiC corners,
// interpolated with the CiC weights, for the particles of a block: the nodes of the block's
// stencils are staged in an LDS window sized to them (when it holds at most kWindow), else
// read from global memory.  Called by all threads of the block.
template <typename T, int NG>
__device__ __forceinline__ void tcola_force(const T* __restrict__ phi, int N,
                                            const double (&u)[3], T* win, int* bounds, T (&g)[3]) {
  int j0[3];
  double f[3];
  const bool in = periodic_cell(true, u, j0, f);
  const T fr[3] = {(T)f[0], (T)f[1], (T)f[2]};
  const int zero[3] = {0, 0, 0};   // every corner carries its weight: nodes 0 and 1 of [0, 1]
  const CellRange cr = block_cells(in, j0, bounds);
  const int ox = cr.lo[0] - NG, oy = cr.lo[1] - NG, oz = cr.lo[2] - NG;
  const int wx = cr.hi[0] - cr.lo[0] + 2 + 2 * NG, wy = cr.hi[1] - cr.lo[1] + 2 + 2 * NG,
            wz = cr.hi[2] - cr.lo[2] + 2 + 2 * NG, wyz = wy * wz;
  const bool use_lds = cr.any && wx <= kWindow && wyz <= kWindow && wx * wyz <= kWindow;
  if (use_lds) {
    const float inv_wz = 1.0f / (float)wz;
    for (int pos = threadIdx.x; pos < wyz; pos += kBlock) {
      const int y = (int)(((float)pos + 0.5f) * inv_wz), z = pos - y * wz;
      const T* const col = phi + (pwrap(oy + y, N) * N + pwrap(oz + z, N));
#pragma unroll 8
      for (int x = 0; x < wx; ++x)
        win[pos + x * wyz] = col[(int64_t)pwrap(ox + x, N) * N * N];
    }
  }
  __syncthreads();
  auto gather = [&](auto at) {
    if constexpr (NG == 1)
      gather_force<T>(1, zero, fr, at, g);
    else
      gather_force_wide<T, NG>(1, zero, fr, at, g);
  };
  if (in && use_lds) {
    const T* const p = win + ((j0[0] - cr.lo[0]) * wyz + (j0[1] - cr.lo[1]) * wz +
                              (j0[2] - cr.lo[2]));
    gather([&](int kx, int ky, int kz) { return p[kx * wyz + ky * wz + kz]; });
  } else {
    gather([&](int kx, int ky, int kz) {
      return phi[((int64_t)pwrap(j0[0] - NG + kx, N) * N + pwrap(j0[1] - NG + ky, N)) * N +
                 pwrap(j0[2] - NG + kz, N)];
    });
  }
  __syncthreads();   // the window and `bounds` are free again
}

// One particle pass: (MODE kInit) L- and the deposit of the LPT positions; (kStep,
// kStepNoDeposit) force at u = q - D1 Psi1 + D2 Psi2 + x_res, kick, drift and (kStep) the
// deposit of the new positions; (kFinalKick) the last half kick and L+.  One LDS window per
// block serves the potential and then the mass: with one thread per site in lattice order,
// 32 reads of the potential and 8 atomics per particle in global memory, a step of 128^3
// particles took 0.35 ms, now 0.067.
template <typename T, int MODE, int NG>
__global__ void __launch_bounds__(kBlock) k_tcola_particles(TcolaArgs<T> a) {
  __shared__ __align__(16) unsigned long long win[kWindow];
  __shared__ int bounds[kCellScratch];
  const int N = a.N;
  const int64_t n3 = (int64_t)N * N * N;
  int idx[3];
  const int64_t p = tcola_site(N, idx);
  const StepScalars sc = a.sc;
  double s1[3], s2[3], u[3];
  T xr[3], pr[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    s1[c] = a.psi1[c * n3 + p];
    s2[c] = a.psi2[c * n3 + p];
    xr[c] = MODE == kInit ? T(0) : a.xres[c * n3 + p];
    pr[c] = MODE == kInit ? T(0) : a.pres[c * n3 + p];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (MODE == kInit) {
      a.xres[c * n3 + p] = T(0);
      a.pres[c * n3 + p] = T(0);
    }
    u[c] = lpt_base(idx[c] + 0.5, sc.D1, s1[c], sc.D2, s2[c]) + (double)xr[c];
  }
  if constexpr (MODE != kInit) {
    T g[3];
    tcola_force<T, NG>(a.phi, N, u, reinterpret_cast<T*>(win), bounds, g);
    const double d2 = sc.D2 - sc.D1 * sc.D1;
#pragma unroll
    for (int c = 0; c < 3; ++c) pr[c] += (T)sc.beta * (g[c] - (T)(sc.D1 * s1[c] - d2 * s2[c]));
    if (MODE == kFinalKick) {
#pragma unroll
      for (int c = 0; c < 3; ++c) a.pres[c * n3 + p] = pr[c] + (T)(sc.c1 * s1[c] + sc.c2 * s2[c]);
      return;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      xr[c] += (T)sc.alpha * pr[c];
      a.xres[c * n3 + p] = xr[c];
      a.pres[c * n3 + p] = pr[c];
    }
    if (MODE == kStepNoDeposit) return;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      u[c] = lpt_base(idx[c] + 0.5, sc.D1n, s1[c], sc.D2n, s2[c]) + (double)xr[c];
  }
  // periodic CiC deposit, 2^40 units per particle
  periodic_deposit_block(a.rho, N, true, u, win, bounds);
}

// Final positions (Mpc/h in [0, L)) and momenta at the lattice index, and the periodic CiC of
// all particles on the N_out^3 output grid (2^40 units per particle).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_tcola_output(TcolaArgs<T> a, T* pos, T* mom,
                                                         unsigned long long* grid, int N_out,
                                                         double cell, double L) {
  __shared__ __align__(16) unsigned long long win[kWindow];
  __shared__ int bounds[kCellScratch];
  const int N = a.N;
  const int64_t n3 = (int64_t)N * N * N;
  int idx[3];
  const int64_t p = tcola_site(N, idx);
  const double s = (double)N_out / (double)N;
  double uo[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double ug = lpt_base(idx[c] + 0.5, a.sc.D1, a.psi1[c * n3 + p], a.sc.D2,
                               a.psi2[c * n3 + p]) + (double)a.xres[c * n3 + p];
    if (pos) {
      T xl = (T)(wrap_position(ug, (double)N) * cell);
      if (xl >= (T)L) xl = T(0);
      pos[c * n3 + p] = xl;
    }
    if (mom) mom[c * n3 + p] = (T)((double)a.pres[c * n3 + p] * cell);
    uo[c] = ug * s;
  }
  if (grid) periodic_deposit_block(grid, N_out, true, uo, win, bounds);
}

template <typename T>
__global__ void k_tcola_density_out(const unsigned long long* __restrict__ grid, T* out,
                                    int64_t n, double scale) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (T)((double)(long long)grid[i] * kFixedInv * scale - 1.0);
}

inline unsigned blocks_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

template <typename T>
hipError_t launch_tcola_setup(const TcolaArgs<T>& a, const double* phi1, const double* phi2,
                              hipStream_t s) {
  const int64_t n3 = (int64_t)a.N * a.N * a.N;
  hipLaunchKernelGGL(k_tcola_setup<T>, dim3(blocks_of(n3)), dim3(kBlock), 0, s, a, phi1, phi2);
  return hipGetLastError();
}

template <typename T, int NG>
hipError_t launch_tcola_particles_ng(const TcolaArgs<T>& a, int mode, hipStream_t s) {
  const dim3 grid((unsigned)((int64_t)a.N * a.N * a.N / kBlock)), block(kBlock);
  switch (mode) {
    case kStep: hipLaunchKernelGGL((k_tcola_particles<T, kStep, NG>), grid, block, 0, s, a); break;
    case kStepNoDeposit:
      hipLaunchKernelGGL((k_tcola_particles<T, kStepNoDeposit, NG>), grid, block, 0, s, a);
      break;
    case kFinalKick:
      hipLaunchKernelGGL((k_tcola_particles<T, kFinalKick, NG>), grid, block, 0, s, a);
      break;
    case kInit:   // no force: one kernel for every order
      hipLaunchKernelGGL((k_tcola_particles<T, kInit, 1>), grid, block, 0, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tcola_particles(const TcolaArgs<T>& a, int mode, hipStream_t s) {
  switch (a.ng) {
    case 1: return launch_tcola_particles_ng<T, 1>(a, mode, s);
    case 2: return launch_tcola_particles_ng<T, 2>(a, mode, s);
    case 3: return launch_tcola_particles_ng<T, 3>(a, mode, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_tcola_output(const TcolaArgs<T>& a, T* pos, T* mom, unsigned long long* grid,
                               T* density, int N_out, double cell, double L, hipStream_t s) {
  const int64_t n3 = (int64_t)a.N * a.N * a.N;
  const int64_t no3 = (int64_t)N_out * N_out * N_out;
  if (density) {
    hipError_t e = launch_zero_u64(grid, no3, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_tcola_output<T>, dim3((unsigned)(n3 / kBlock)), dim3(kBlock), 0, s, a, pos, mom,
                     density ? grid : nullptr, N_out, cell, L);
  if (density) {
    const double r = (double)N_out / (double)a.N;
    hipLaunchKernelGGL(k_tcola_density_out<T>, dim3(blocks_of(no3)), dim3(kBlock), 0, s, grid,
                       density, no3, r * r * r);
  }
  return hipGetLastError();
}

#define SCOLA_TCOLA_INSTANTIATE(T)                                                         \
  template hipError_t launch_tcola_setup<T>(const TcolaArgs<T>&, const double*,             \
                                            const double*, hipStream_t);                    \
  template hipError_t launch_tcola_particles<T>(const TcolaArgs<T>&, int, hipStream_t);     \
  template hipError_t launch_tcola_output<T>(const TcolaArgs<T>&, T*, T*, unsigned long long*, \
                                             T*, int, double, double, hipStream_t);
SCOLA_TCOLA_INSTANTIATE(float)
SCOLA_TCOLA_INSTANTIATE(double)
#undef SCOLA_TCOLA_INSTANTIATE

}  // namespace scola
