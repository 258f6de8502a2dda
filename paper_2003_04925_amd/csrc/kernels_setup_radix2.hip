// Lagrangian potentials by complex radix-2 transforms, for FP32 plans with the reverse mode
// only (do_setup decides).  The fused transforms of kernels_fft.hip are 4 to 5 times as fast, as
// accurate and as reproducible, but they round phi differently in the last bits (1e-15 and 2e-15
// of the maximum of phi1 and phi2).  Some tens of the FP32 displacements then round the other
// way, and where such a particle lies on a cell face, at which the gradient of the CiC weights
// has a kink, the returned gradient changes by more than it does from one run to the next: over
// 120 noise fields of 64^3 and 128^3 particles and 20 or 24 steps, by up to 1e-6 of its norm and
// 2.2e-6 of its largest entry, against 4e-7 and 1e-7 between two runs (its distance from an FP64
// run is 2.9e-5).  Neither is nearer the truth; these transforms keep the gradients of such plans
// where they were to within their run-to-run differences, for 0.7 ms of the 35 ms of a forward
// and reverse pass.  A plan without checkpoints takes the fused ones, so that its FP32 results
// can differ from these in their rounding.
#include "common.h"
#include "kernels.h"

namespace scola {

namespace {

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ inline int wrap(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

// Batched complex FFT (FP64, power-of-two length n) along one axis of an n^3 array held as
// [outer][n][inner].  Each block transforms `lines` lines staged in LDS with a radix-2
// Stockham pass per stage.  sign = -1 forward, +1 inverse (unnormalised).
__global__ void __launch_bounds__(kBlock) k_fft_axis(double2* __restrict__ data, int n,
                                                      int64_t inner, int lines, double sign) {
  extern __shared__ double2 lds[];
  double2* buf0 = lds;
  double2* buf1 = lds + (size_t)lines * n;
  const int64_t total_lines = (int64_t)n * n;       // n^3 / n
  const int64_t first = (int64_t)blockIdx.x * lines;
  const int tid = threadIdx.x;
  const int count = lines * n;
  // element e of the block -> (line b, position i) with coalesced global addresses
  auto address = [&](int e, int& b, int& i) -> int64_t {
    if (inner == 1) {
      b = e / n;
      i = e % n;
      return (first + b) * n + i;
    }
    b = e % lines;
    i = e / lines;
    const int64_t line = first + b;
    const int64_t o = line / inner, c = line % inner;
    return o * n * inner + (int64_t)i * inner + c;
  };
  for (int e = tid; e < count; e += blockDim.x) {
    int b, i;
    const int64_t a = address(e, b, i);
    if (first + b < total_lines) buf0[b * n + i] = data[a];
  }
  __syncthreads();
  double2* src = buf0;
  double2* dst = buf1;
  const int half = n / 2;
  for (int ns = 1; ns < n; ns <<= 1) {
    for (int e = tid; e < lines * half; e += blockDim.x) {
      const int b = e / half, j = e % half;
      const int k = j & (ns - 1);
      double s, c;
      sincospi(sign * (double)k / (double)ns, &s, &c);
      const double2 x0 = src[b * n + j];
      const double2 x1 = cmul(src[b * n + j + half], make_double2(c, s));
      const int o = b * n + ((j - k) << 1) + k;
      dst[o] = make_double2(x0.x + x1.x, x0.y + x1.y);
      dst[o + ns] = make_double2(x0.x - x1.x, x0.y - x1.y);
    }
    __syncthreads();
    double2* t = src;
    src = dst;
    dst = t;
  }
  for (int e = tid; e < count; e += blockDim.x) {
    int b, i;
    const int64_t a = address(e, b, i);
    if (first + b < total_lines) data[a] = src[b * n + i];
  }
}

__global__ void k_real_to_complex(const double* __restrict__ in, double2* __restrict__ out,
                                  int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = make_double2(in[i], 0.0);
}

__global__ void k_take_real(const double2* __restrict__ in, double* __restrict__ out,
                            double scale, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i].x * scale;
}

__device__ inline int signed_mode(int i, int N) { return i < N / 2 ? i : i - N; }

// Symbol of the order-2 Laplacian, one-cell spacing: -4 sum sin^2(pi m / N).
__device__ inline double fda2_symbol(int mx, int my, int mz, int N) {
  double sx = sinpi((double)mx / N), sy = sinpi((double)my / N), sz = sinpi((double)mz / N);
  return -4.0 * (sx * sx + sy * sy + sz * sz);
}

// A.1 + A.2 (first order): multiply FFT(w) by sqrt(P(k, a_i) N^3 / L^3) and divide by the
// FDA Laplacian symbol; the zero mode is set to zero.
__global__ void k_ic_filter(double2* __restrict__ c, int N, double L, double amplitude,
                            double ns, double Om, double Ob, double h, double Tcmb,
                            double growth2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n3 = (int64_t)N * N * N;
  if (i >= n3) return;
  const int ix = (int)(i / ((int64_t)N * N)), iy = (int)((i / N) % N), iz = (int)(i % N);
  const int mx = signed_mode(ix, N), my = signed_mode(iy, N), mz = signed_mode(iz, N);
  if (mx == 0 && my == 0 && mz == 0) {
    c[i] = make_double2(0.0, 0.0);
    return;
  }
  const double kf = 2.0 * M_PI / L;
  const double k = kf * sqrt((double)mx * mx + (double)my * my + (double)mz * mz);
  const double T = eh_nowiggle_transfer(k, Om, Ob, h, Tcmb);
  const double P = amplitude * pow(k, ns) * T * T * growth2;
  const double f = sqrt(P * (double)N * N * N / (L * L * L)) / fda2_symbol(mx, my, mz, N);
  c[i] = make_double2(c[i].x * f, c[i].y * f);
}

// Division by the FDA Laplacian symbol (A.2, second order), zero mode to zero.
__global__ void k_inverse_laplacian(double2* __restrict__ c, int N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n3 = (int64_t)N * N * N;
  if (i >= n3) return;
  const int ix = (int)(i / ((int64_t)N * N)), iy = (int)((i / N) % N), iz = (int)(i % N);
  const int mx = signed_mode(ix, N), my = signed_mode(iy, N), mz = signed_mode(iz, N);
  if (mx == 0 && my == 0 && mz == 0) {
    c[i] = make_double2(0.0, 0.0);
    return;
  }
  const double inv = 1.0 / fda2_symbol(mx, my, mz, N);
  c[i] = make_double2(c[i].x * inv, c[i].y * inv);
}

// Second-order source sum_{i>j} [phi_,ii phi_,jj - phi_,ij^2] with phi_,ij = D_i D_j phi,
// D the central difference (wide stencils), periodic; written as complex
// input of the next FFT.
__global__ void k_second_order_source(const double* __restrict__ phi, double2* __restrict__ out,
                                      int N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n3 = (int64_t)N * N * N;
  if (i >= n3) return;
  const int x = (int)(i / ((int64_t)N * N)), y = (int)((i / N) % N), z = (int)(i % N);
  auto P = [&](int dx, int dy, int dz) {
    return phi[((int64_t)wrap(x + dx, N) * N + wrap(y + dy, N)) * N + wrap(z + dz, N)];
  };
  const double c0 = P(0, 0, 0);
  const double xx = 0.25 * (P(2, 0, 0) - 2.0 * c0 + P(-2, 0, 0));
  const double yy = 0.25 * (P(0, 2, 0) - 2.0 * c0 + P(0, -2, 0));
  const double zz = 0.25 * (P(0, 0, 2) - 2.0 * c0 + P(0, 0, -2));
  const double xy = 0.25 * (P(1, 1, 0) - P(1, -1, 0) - P(-1, 1, 0) + P(-1, -1, 0));
  const double xz = 0.25 * (P(1, 0, 1) - P(1, 0, -1) - P(-1, 0, 1) + P(-1, 0, -1));
  const double yz = 0.25 * (P(0, 1, 1) - P(0, 1, -1) - P(0, -1, 1) + P(0, -1, -1));
  const double s = yy * xx - xy * xy + zz * xx - xz * xz + zz * yy - yz * yz;
  out[i] = make_double2(s, 0.0);
}

inline unsigned grid1(int64_t n, int b = kBlock) { return (unsigned)((n + b - 1) / b); }

hipError_t fft3d(double2* c, int N, double sign, hipStream_t s) {
  const int lines = N >= 1024 ? 1 : 1024 / N;     // 32 KiB of LDS per block
  const size_t lds = (size_t)2 * lines * N * sizeof(double2);
  const int64_t total_lines = (int64_t)N * N;
  const unsigned blocks = (unsigned)((total_lines + lines - 1) / lines);
  const int64_t inners[3] = {(int64_t)N * N, N, 1};   // axes x, y, z
  for (int ax = 0; ax < 3; ++ax) {
    hipLaunchKernelGGL(k_fft_axis, dim3(blocks), dim3(kBlock), lds, s, c, N,
                       inners[ax], lines, sign);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_setup_potentials_radix2(const SetupArgs& a, hipStream_t s) {
  const int N = a.tables.N;
  const int64_t n3 = (int64_t)N * N * N;
  hipLaunchKernelGGL(k_real_to_complex, dim3(grid1(n3)), dim3(kBlock), 0, s, a.white_noise,
                     a.cbuf, n3);
  hipError_t e = fft3d(a.cbuf, N, -1.0, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ic_filter, dim3(grid1(n3)), dim3(kBlock), 0, s, a.cbuf, N, a.L,
                     a.amplitude, a.ns, a.Om, a.Ob, a.h, a.Tcmb, a.growth2);
  if ((e = fft3d(a.cbuf, N, +1.0, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_take_real, dim3(grid1(n3)), dim3(kBlock), 0, s, a.cbuf, a.phi1,
                     1.0 / (double)n3, n3);
  hipLaunchKernelGGL(k_second_order_source, dim3(grid1(n3)), dim3(kBlock), 0, s, a.phi1,
                     a.cbuf, N);
  if ((e = fft3d(a.cbuf, N, -1.0, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_inverse_laplacian, dim3(grid1(n3)), dim3(kBlock), 0, s, a.cbuf, N);
  if ((e = fft3d(a.cbuf, N, +1.0, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_take_real, dim3(grid1(n3)), dim3(kBlock), 0, s, a.cbuf, a.phi2,
                     1.0 / (double)n3, n3);
  return hipGetLastError();
}

}  // namespace scola
