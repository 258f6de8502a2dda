// In-register FFT of one line of N = 2^p complex FP64 points held by N / 8 threads (Stockham
// radix 8, the last stage 4 or 2 where p is no multiple of 3): the building block of the
// periodic solves in kernels_fft.hip.
#pragma once

#include <hip/hip_runtime.h>

namespace scola {
namespace {

__device__ __forceinline__ double2 z_add(double2 a, double2 b) {
  return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 z_sub(double2 a, double2 b) {
  return make_double2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ double2 z_mul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a times S i, S = -1 or +1
template <int S>
__device__ __forceinline__ double2 z_times_i(double2 a) {
  return S < 0 ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}

// Threads of a line and elements of a thread: thread j holds elements j + m T, m < E, before
// and after the transform.
template <int N>
struct FftLine {
  static constexpr int E = N < 8 ? N : 8;
  static constexpr int T = N / E;
};

// DFT of R = 2, 4, 8 values with W = exp(S 2 pi i / R), natural order.
template <int R, int S>
__device__ __forceinline__ void z_dft(double2 (&x)[R]) {
  if constexpr (R == 2) {
    const double2 a = x[0], b = x[1];
    x[0] = z_add(a, b);
    x[1] = z_sub(a, b);
  } else if constexpr (R == 4) {
    const double2 t0 = z_add(x[0], x[2]), t1 = z_sub(x[0], x[2]);
    const double2 t2 = z_add(x[1], x[3]), t3 = z_times_i<S>(z_sub(x[1], x[3]));
    x[0] = z_add(t0, t2);
    x[1] = z_add(t1, t3);
    x[2] = z_sub(t0, t2);
    x[3] = z_sub(t1, t3);
  } else {
    static_assert(R == 8, "radix");
    double2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    z_dft<4, S>(e);
    z_dft<4, S>(o);
    constexpr double h = 0.70710678118654752440;
    constexpr double s = (double)S;
    o[1] = make_double2(h * (o[1].x - s * o[1].y), h * (o[1].y + s * o[1].x));
    o[2] = z_times_i<S>(o[2]);
    o[3] = make_double2(h * (-o[3].x - s * o[3].y), h * (s * o[3].x - o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = z_add(e[k], o[k]);
      x[k + 4] = z_sub(e[k], o[k]);
    }
  }
}

// exp(S 2 pi i m / NT) from the table tw of exp(-2 pi i m / NT), m < NT.
template <int S>
__device__ __forceinline__ double2 z_twiddle(const double2* __restrict__ tw, int m) {
  const double2 w = tw[m];
  return S < 0 ? w : make_double2(w.x, -w.y);
}

// The stages from sub-transform length Ns on.  Between stages the line's values pass through
// LDS at pos(i), i < N (a barrier on each side; the caller's own use of that LDS ended at a
// barrier).  The twiddles W^k, W^2k, W^4k of a radix-8 butterfly are read from the table and
// the other four formed as one product of two of them.
template <int N, int NT, int S, int Ns, typename Pos>
__device__ __forceinline__ void fft_stages(double2 (&x)[FftLine<N>::E], int j,
                                           const double2* __restrict__ tw, double2* lds,
                                           Pos pos) {
  constexpr int E = FftLine<N>::E, T = FftLine<N>::T;
  constexpr int R = N / Ns >= 8 ? 8 : N / Ns, B = E / R;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    double2 y[R];
#pragma unroll
    for (int q = 0; q < R; ++q) y[q] = x[b + q * B];
    if constexpr (Ns > 1) {
      const int k = (j + b * T) & (Ns - 1);
      constexpr int step = NT / (Ns * R);
      double2 w[R];
      w[1] = z_twiddle<S>(tw, k * step);
      if constexpr (R >= 4) {
        w[2] = z_twiddle<S>(tw, 2 * k * step);
        w[3] = z_mul(w[1], w[2]);
      }
      if constexpr (R == 8) {
        w[4] = z_twiddle<S>(tw, 4 * k * step);
        w[5] = z_mul(w[1], w[4]);
        w[6] = z_mul(w[2], w[4]);
        w[7] = z_mul(w[3], w[4]);
      }
#pragma unroll
      for (int q = 1; q < R; ++q) y[q] = z_mul(y[q], w[q]);
    }
    z_dft<R, S>(y);
#pragma unroll
    for (int q = 0; q < R; ++q) x[b + q * B] = y[q];
  }
  if constexpr (Ns * R < N) {
    if constexpr (Ns > 1) __syncthreads();
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int jb = j + b * T, k = jb & (Ns - 1);
#pragma unroll
      for (int q = 0; q < R; ++q) lds[pos((jb - k) * R + k + q * Ns)] = x[b + q * B];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = lds[pos(j + m * T)];
    fft_stages<N, NT, S, Ns * R>(x, j, tw, lds, pos);
  }
}

// Unnormalised FFT of a line, exponent sign S; tw: exp(-2 pi i m / NT), m < NT, N | NT.
// Called by all threads of the block; the LDS may be reused only after a barrier.
template <int N, int NT, int S, typename Pos>
__device__ __forceinline__ void fft_line(double2 (&x)[FftLine<N>::E], int j,
                                         const double2* __restrict__ tw, double2* lds, Pos pos) {
  fft_stages<N, NT, S, 1>(x, j, tw, lds, pos);
}

}  // namespace
}  // namespace scola
