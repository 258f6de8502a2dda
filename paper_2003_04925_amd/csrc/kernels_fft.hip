// Periodic solves on an N^3 grid (N a power of two, 8 to 1024, FP64): out = F^-1 f F in, with
// real input and output and a real symmetric filter f (the initial spectrum over the FDA
// Laplacian's symbol, or 1 / symbol).  They serve the set-up (Sec. 3.1, A.1-A.2), its reverse
// mode and the Poisson solve of the periodic tCOLA run.
//
// What bounds them is memory: one axis of a half spectrum is read and written per pass.  So
// the transform is real to complex (half the data of a complex one), the x axis is
// transformed forward, filtered and transformed back while its lines are in registers, and
// the field is formed and taken up by the first and last pass themselves (LoadOp, StoreOp):
// five passes in all,
//   z: field -> half spectrum along z (N / 2 complex points per line and an untangling step);
//   y: forward;  x: forward, filter, inverse;  y: inverse;  z: half spectrum -> field,
// where the radix-2 complex form took six passes of twice the data plus four more for the
// filter, the conversions and the source: on 256^3 a solve took 2.2 ms, on 128^3 0.26 ms.
// The half spectrum lies in the caller's N^3 complex scratch as rows of `pitch` values, so
// that every tile of columns starts on a cache line.  The filter of a mode depends on its
// |m|^2, an integer: the initial spectrum is tabulated over it once per plan (its power and
// logarithms, evaluated per mode, cost 0.59 ms on 256^3).
#include "common.h"
#include "fft_lines.h"
#include "kernels.h"

namespace scola {

namespace {

// Row pitch of the half spectrum (N / 2 + 1 values used, at most N).
template <int N>
constexpr int half_pitch() {
  return N >= 16 ? N / 2 + 8 : 8;
}
// Columns of a block in the y and x passes (128 bytes of each row; half for N = 1024, whose
// tile would exceed 64 KB of LDS).
template <int N>
constexpr int col_tile() {
  return N <= 512 ? 8 : 4;
}
// Lines of a block in the z passes: 256 threads, or 64 for small grids, which then have
// enough blocks.
template <int N>
constexpr int z_lines() {
  return (N >= 128 ? 256 : 64) / FftLine<N / 2>::T;
}
// LDS position of value i of a z line (its first stage writes at a stride of 8 values, which
// the shift turns into distinct banks) and the line's pitch (N / 2 + 1 values).
__device__ __forceinline__ int z_pos(int i) { return i + (i >> 3); }
template <int H>
constexpr int z_pitch() {
  return H + H / 8 + 1;
}

template <int N, typename Load>
__global__ void __launch_bounds__(z_lines<N>() * FftLine<N / 2>::T)
k_solve_z_forward(Load load, double2* __restrict__ c, const double2* __restrict__ tw) {
  constexpr int H = N / 2, E = FftLine<H>::E, T = FftLine<H>::T, C = z_lines<N>();
  __shared__ double2 lds[C * z_pitch<H>()];
  const int j = threadIdx.x % T, l = threadIdx.x / T;
  const int line = blockIdx.x * C + l;
  double2* const mine = lds + l * z_pitch<H>();
  double2 v[E];
#pragma unroll
  for (int m = 0; m < E; ++m)
    v[m] = line < N * N ? load.template pair<N>(line / N, line % N, 2 * (j + m * T))
                        : make_double2(0.0, 0.0);
  fft_line<H, N, -1>(v, j, tw, mine, z_pos);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < E; ++m) mine[z_pos(j + m * T)] = v[m];
  __syncthreads();
  if (line >= N * N) return;
  // even and odd samples separated: X_k = (Z_k + conj Z_(H-k)) / 2 - i W_N^k (Z_k - conj
  // Z_(H-k)) / 2, and X_H = Re Z_0 - Im Z_0
  double2* const out = c + (int64_t)line * half_pitch<N>();
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int k = j + m * T;
    const double2 a = v[m], b = mine[z_pos((H - k) & (H - 1))], w = tw[k];
    const double2 e = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    const double2 d = make_double2(0.5 * (a.x - b.x), 0.5 * (a.y + b.y));
    out[k] = z_add(e, z_mul(d, make_double2(w.y, -w.x)));
    if (k == 0) out[H] = make_double2(a.x - a.y, 0.0);
  }
}

template <int N, typename Store>
__global__ void __launch_bounds__(z_lines<N>() * FftLine<N / 2>::T)
k_solve_z_inverse(Store store, const double2* __restrict__ c, const double2* __restrict__ tw) {
  constexpr int H = N / 2, E = FftLine<H>::E, T = FftLine<H>::T, C = z_lines<N>();
  __shared__ double2 lds[C * z_pitch<H>()];
  const int j = threadIdx.x % T, l = threadIdx.x / T;
  const int line = blockIdx.x * C + l;
  const bool in = line < N * N;
  double2* const mine = lds + l * z_pitch<H>();
  const double2* const src = c + (int64_t)(in ? line : 0) * half_pitch<N>();
  double2 v[E];
#pragma unroll
  for (int m = 0; m < E; ++m) v[m] = src[j + m * T];
#pragma unroll
  for (int m = 0; m < E; ++m) mine[z_pos(j + m * T)] = v[m];
  if (j == 0) mine[z_pos(H)] = src[H];
  __syncthreads();
  // Z_k = (X_k + conj X_(H-k)) + i W_N^-k (X_k - conj X_(H-k))
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int k = j + m * T;
    const double2 a = v[m], b = mine[z_pos(H - k)], w = tw[k];
    const double2 e = make_double2(a.x + b.x, a.y - b.y);
    const double2 d = make_double2(a.x - b.x, a.y + b.y);
    v[m] = z_add(e, z_mul(d, make_double2(w.y, w.x)));
  }
  __syncthreads();
  fft_line<H, N, +1>(v, j, tw, mine, z_pos);
  if (!in) return;
#pragma unroll
  for (int m = 0; m < E; ++m)
    store.template pair<N>(line / N, line % N, 2 * (j + m * T), v[m]);
}

template <int N, int S>
__global__ void __launch_bounds__(col_tile<N>() * FftLine<N>::T)
k_solve_y(double2* __restrict__ c, const double2* __restrict__ tw) {
  constexpr int H = N / 2, E = FftLine<N>::E, T = FftLine<N>::T, C = col_tile<N>();
  constexpr int tiles = (H + C) / C, pitch = half_pitch<N>();
  __shared__ double2 lds[N * C];
  const int cc = threadIdx.x % C, j = threadIdx.x / C;
  const int x = blockIdx.x / tiles, col = (blockIdx.x % tiles) * C + cc;
  double2* const base = c + (int64_t)x * N * pitch + col;
  const bool in = col <= H;
  double2 v[E];
#pragma unroll
  for (int m = 0; m < E; ++m)
    v[m] = in ? base[(int64_t)(j + m * T) * pitch] : make_double2(0.0, 0.0);
  fft_line<N, N, S>(v, j, tw, lds, [cc](int i) { return i * C + cc; });
  if (!in) return;
#pragma unroll
  for (int m = 0; m < E; ++m) base[(int64_t)(j + m * T) * pitch] = v[m];
}

// x axis: forward, filter, inverse.  IC: the initial spectrum's table over |m|^2 divided by
// the Laplacian's symbol (A.1, A.2 first order); else the inverse Laplacian.  Both carry the
// transforms' 1 / N^3; the zero mode is set to zero.
template <int N, bool IC>
__global__ void __launch_bounds__(col_tile<N>() * FftLine<N>::T)
k_solve_x(double2* __restrict__ c, PeriodicTables t) {
  constexpr int H = N / 2, E = FftLine<N>::E, T = FftLine<N>::T, C = col_tile<N>();
  constexpr int tiles = (H + C) / C, pitch = half_pitch<N>();
  __shared__ double2 lds[N * C];
  const int cc = threadIdx.x % C, j = threadIdx.x / C;
  const int y = blockIdx.x / tiles, col = (blockIdx.x % tiles) * C + cc;
  double2* const base = c + (int64_t)y * pitch + col;
  constexpr int64_t stride = (int64_t)N * pitch;
  const bool in = col <= H;
  double2 v[E];
#pragma unroll
  for (int m = 0; m < E; ++m)
    v[m] = in ? base[(j + m * T) * stride] : make_double2(0.0, 0.0);
  auto pos = [cc](int i) { return i * C + cc; };
  fft_line<N, N, -1>(v, j, t.tw, lds, pos);
  const int my = y < H ? y : y - N, mz = in ? col : 0;
  const double syz = t.symbol[y] + t.symbol[mz];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int kx = j + m * T, mx = kx < H ? kx : kx - N;
    const int m2 = mx * mx + my * my + mz * mz;
    const double num = IC ? t.spectrum[m2] : 1.0 / ((double)N * N * N);
    const double f = m2 == 0 ? 0.0 : num / (t.symbol[kx] + syz);
    v[m] = make_double2(v[m].x * f, v[m].y * f);
  }
  __syncthreads();
  fft_line<N, N, +1>(v, j, t.tw, lds, pos);
  if (!in) return;
#pragma unroll
  for (int m = 0; m < E; ++m) base[(j + m * T) * stride] = v[m];
}

// Per plan: exp(-2 pi i m / N), the per-axis symbol of the FDA Laplacian of order 2 ng
// (sum_k a_k (2 cos(2 pi k m / N) - 2), i.e. -4 sin^2(pi m / N) at order 2), and over |m|^2
// the initial amplitude sqrt(P(k, a_i) N^3 / L^3) / N^3 (A.1).
__global__ void k_periodic_tables(double2* tw, double* symbol, double* spectrum, int64_t n_spectrum,
                                  int N, double L, double amplitude, double ns, double Om, double Ob,
                                  double h, double Tcmb, double growth2, int ng) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) {
    double s, c;
    sincospi(2.0 * (double)i / N, &s, &c);
    tw[i] = make_double2(c, -s);
    double sum = 0.0;
    for (int k = 1; k <= ng; ++k) {
      // 2 cos(t) - 2 = -4 sin^2(t / 2)
      const double sh = sinpi((double)((k * i) % (2 * N)) / N);
      sum += second_difference_weight(ng, k) * (-4.0 * sh * sh);
    }
    symbol[i] = sum;
  }
  if (i < n_spectrum) {
    const double k = 2.0 * M_PI / L * sqrt((double)i);
    double f = 0.0;
    if (i > 0) {
      const double T = eh_nowiggle_transfer(k, Om, Ob, h, Tcmb);
      const double P = amplitude * pow(k, ns) * T * T * growth2;
      const double n3 = (double)N * N * N;
      f = sqrt(P * n3 / (L * L * L)) / n3;
    }
    spectrum[i] = f;
  }
}

template <int N, typename Load, typename Store>
hipError_t solve_n(const PeriodicTables& t, double2* c, const Load& load, const Store& store,
                   bool initial_spectrum, hipStream_t s) {
  constexpr int C = z_lines<N>(), tiles = (N / 2 + col_tile<N>()) / col_tile<N>();
  const dim3 zg((N * N + C - 1) / C), zb(C * FftLine<N / 2>::T);
  const dim3 cg(N * tiles), cb(col_tile<N>() * FftLine<N>::T);
  hipLaunchKernelGGL((k_solve_z_forward<N, Load>), zg, zb, 0, s, load, c, t.tw);
  hipLaunchKernelGGL((k_solve_y<N, -1>), cg, cb, 0, s, c, t.tw);
  if (initial_spectrum)
    hipLaunchKernelGGL((k_solve_x<N, true>), cg, cb, 0, s, c, t);
  else
    hipLaunchKernelGGL((k_solve_x<N, false>), cg, cb, 0, s, c, t);
  hipLaunchKernelGGL((k_solve_y<N, +1>), cg, cb, 0, s, c, t.tw);
  hipLaunchKernelGGL((k_solve_z_inverse<N, Store>), zg, zb, 0, s, store, c, t.tw);
  return hipGetLastError();
}

template <typename Load, typename Store>
hipError_t solve(const PeriodicTables& t, double2* c, const Load& load, const Store& store,
                 bool initial_spectrum, hipStream_t s) {
  switch (t.N) {
    case 8: return solve_n<8>(t, c, load, store, initial_spectrum, s);
    case 16: return solve_n<16>(t, c, load, store, initial_spectrum, s);
    case 32: return solve_n<32>(t, c, load, store, initial_spectrum, s);
    case 64: return solve_n<64>(t, c, load, store, initial_spectrum, s);
    case 128: return solve_n<128>(t, c, load, store, initial_spectrum, s);
    case 256: return solve_n<256>(t, c, load, store, initial_spectrum, s);
    case 512: return solve_n<512>(t, c, load, store, initial_spectrum, s);
    case 1024: return solve_n<1024>(t, c, load, store, initial_spectrum, s);
    default: return hipErrorInvalidValue;
  }
}

// --- what the first pass reads and the last one writes: the values at (x, y, z), (x, y, z+1),
// z even (callers' arrays need only their type's alignment) ------------------------------------

struct LoadReal {
  const double* in;
  template <int N>
  __device__ double2 pair(int x, int y, int z) const {
    const double* p = in + ((int64_t)x * N + y) * N + z;
    return make_double2(p[0], p[1]);
  }
};

struct StoreReal {
  double* out;
  template <int N>
  __device__ void pair(int x, int y, int z, double2 v) const {
    double* p = out + ((int64_t)x * N + y) * N + z;
    p[0] = v.x;
    p[1] = v.y;
  }
};

// Second-order source sum_{i>j} [phi_,ii phi_,jj - phi_,ij^2] with phi_,ij = D_i D_j phi,
// D the central difference of order 2 ng (wide stencils), periodic.
struct LoadSource {
  const double* phi;
  int ng;
  // orders 4 and 6 at one node
  template <int N>
  __device__ double point(int x, int y, int z) const {
    auto P = [&](int dx, int dy, int dz) {
      return phi[((int64_t)((x + dx) & (N - 1)) * N + ((y + dy) & (N - 1))) * N +
                 ((z + dz) & (N - 1))];
    };
    // D_i (D_j phi) = sum_k c_k sum_l c_l [phi(+k e_i + l e_j) - phi(+k e_i - l e_j)
    //                                      - phi(-k e_i + l e_j) + phi(-k e_i - l e_j)]
    double d[3][3];
    for (int a = 0; a < 3; ++a)
      for (int b = a; b < 3; ++b) {
        double acc = 0.0;
        for (int k = 1; k <= ng; ++k)
          for (int l = 1; l <= ng; ++l) {
            double t = 0.0;
            for (int sk = -1; sk <= 1; sk += 2)
              for (int sl = -1; sl <= 1; sl += 2) {
                int o[3] = {0, 0, 0};
                o[a] += sk * k;
                o[b] += sl * l;
                t += sk * sl * P(o[0], o[1], o[2]);
              }
            acc += first_difference_weight(ng, k) * first_difference_weight(ng, l) * t;
          }
        d[a][b] = d[b][a] = acc;
      }
    return d[1][1] * d[0][0] - d[0][1] * d[0][1] + d[2][2] * d[0][0] - d[0][2] * d[0][2] +
           d[2][2] * d[1][1] - d[1][2] * d[1][2];
  }
  // Order 2 at the nodes (x, y, z) and (x, y, z + 1), z even: the 38 nodes that the two share
  // in part, as 15 pairs and 8 single ones (256^3: 208 us node by node, now 136).
  template <int N>
  __device__ double2 pair(int x, int y, int z) const {
    if (ng > 1) return make_double2(point<N>(x, y, z), point<N>(x, y, z + 1));
    auto row = [&](int dx, int dy) {
      return phi + ((int64_t)((x + dx) & (N - 1)) * N + ((y + dy) & (N - 1))) * N;
    };
    auto two = [&](int dx, int dy, int dz) {
      return *reinterpret_cast<const double2*>(row(dx, dy) + ((z + dz) & (N - 1)));
    };
    const double2 c = two(0, 0, 0), cm = two(0, 0, -2), cp = two(0, 0, 2);
    const double2 x2 = two(2, 0, 0), xm2 = two(-2, 0, 0), y2 = two(0, 2, 0), ym2 = two(0, -2, 0);
    const double2 pp = two(1, 1, 0), pm = two(1, -1, 0), mp = two(-1, 1, 0), mm = two(-1, -1, 0);
    // rows one step along x or y: the nodes z - 1 .. z + 2
    double r[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double* const q = row(i == 0 ? 1 : i == 1 ? -1 : 0, i == 2 ? 1 : i == 3 ? -1 : 0);
      const double2 v = *reinterpret_cast<const double2*>(q + z);
      r[i][0] = q[(z - 1) & (N - 1)];
      r[i][1] = v.x;
      r[i][2] = v.y;
      r[i][3] = q[(z + 2) & (N - 1)];
    }
    auto source = [](double c0, double xp, double xm, double yp, double ym, double zp, double zm,
                     double app, double apm, double amp, double amm, const double* rxp,
                     const double* rxm, const double* ryp, const double* rym) {
      const double xx = 0.25 * (xp - 2.0 * c0 + xm);
      const double yy = 0.25 * (yp - 2.0 * c0 + ym);
      const double zz = 0.25 * (zp - 2.0 * c0 + zm);
      const double xy = 0.25 * (app - apm - amp + amm);
      const double xz = 0.25 * (rxp[2] - rxp[0] - rxm[2] + rxm[0]);
      const double yz = 0.25 * (ryp[2] - ryp[0] - rym[2] + rym[0]);
      return yy * xx - xy * xy + zz * xx - xz * xz + zz * yy - yz * yz;
    };
    return make_double2(source(c.x, x2.x, xm2.x, y2.x, ym2.x, cp.x, cm.x, pp.x, pm.x, mp.x, mm.x,
                               r[0], r[1], r[2], r[3]),
                        source(c.y, x2.y, xm2.y, y2.y, ym2.y, cp.y, cm.y, pp.y, pm.y, mp.y, mm.y,
                               r[0] + 1, r[1] + 1, r[2] + 1, r[3] + 1));
  }
};

// tCOLA's mass mesh -> delta = mass - 1 (one particle per cell); the mesh is cleared for the
// next deposit and delta optionally recorded.
template <typename T>
struct LoadMass {
  unsigned long long* rho;
  T* record;
  template <int N>
  __device__ double2 pair(int x, int y, int z) const {
    const int64_t i = ((int64_t)x * N + y) * N + z;
    const double2 d = make_double2((double)(long long)rho[i] * kFixedInv - 1.0,
                                   (double)(long long)rho[i + 1] * kFixedInv - 1.0);
    rho[i] = rho[i + 1] = 0ull;
    if (record) {
      record[i] = (T)d.x;
      record[i + 1] = (T)d.y;
    }
    return d;
  }
};

template <typename T>
struct StorePotential {
  T* phi;
  T* record;
  template <int N>
  __device__ void pair(int x, int y, int z, double2 v) const {
    const int64_t i = ((int64_t)x * N + y) * N + z;
    phi[i] = (T)v.x;
    phi[i + 1] = (T)v.y;
    if (record) {
      record[i] = (T)v.x;
      record[i + 1] = (T)v.y;
    }
  }
};

// Transpose of Psi = D phi (central difference, periodic): D^T f (q) = (f(q-e) - f(q+e)) / 2.
// lam_phi1 += D^T lam_Psi1; the second-order part D^T lam_Psi2 is the field.
struct LoadPsiTranspose {
  const double* g;          // lam_Psi1, lam_Psi2: six N^3 fields
  double* lam_phi1;
  template <int N>
  __device__ double2 pair(int x, int y, int z) const {
    constexpr int64_t N3 = (int64_t)N * N * N;
    auto at = [&](int c, int zz, int dx, int dy, int dz) {
      return g[c * N3 + ((int64_t)((x + dx) & (N - 1)) * N + ((y + dy) & (N - 1))) * N +
               ((zz + dz) & (N - 1))];
    };
    auto part = [&](int c, int zz) {
      return 0.5 * (at(c, zz, -1, 0, 0) - at(c, zz, 1, 0, 0) + at(c + 1, zz, 0, -1, 0) -
                    at(c + 1, zz, 0, 1, 0) + at(c + 2, zz, 0, 0, -1) - at(c + 2, zz, 0, 0, 1));
    };
    double* const lam = lam_phi1 + ((int64_t)x * N + y) * N + z;
    lam[0] += part(0, z);
    lam[1] += part(0, z + 1);
    return make_double2(part(3, z), part(3, z + 1));
  }
};

}  // namespace

size_t periodic_table_bytes(int N) {
  return (size_t)N * (sizeof(double2) + sizeof(double)) + spectrum_entries(N) * sizeof(double);
}

hipError_t launch_periodic_tables(void* buf, int N, const SetupArgs& a, PeriodicTables* out,
                                  hipStream_t s) {
  double2* tw = static_cast<double2*>(buf);
  double* symbol = reinterpret_cast<double*>(tw + N);
  double* spectrum = symbol + N;
  const int64_t n = (int64_t)spectrum_entries(N), m = n > N ? n : N;
  hipLaunchKernelGGL(k_periodic_tables, dim3((unsigned)((m + kBlock - 1) / kBlock)), dim3(kBlock),
                     0, s, tw, symbol, spectrum, n, N, a.L, a.amplitude, a.ns, a.Om, a.Ob, a.h,
                     a.Tcmb, a.growth2, a.ng);
  out->tw = tw;
  out->symbol = symbol;
  out->spectrum = spectrum;
  out->N = N;
  return hipGetLastError();
}

hipError_t launch_setup_potentials(const SetupArgs& a, hipStream_t s) {
  hipError_t e = solve(a.tables, a.cbuf, LoadReal{a.white_noise}, StoreReal{a.phi1}, true, s);
  if (e != hipSuccess) return e;
  return solve(a.tables, a.cbuf, LoadSource{a.phi1, a.ng}, StoreReal{a.phi2}, false, s);
}

hipError_t launch_adj_phi_from_psi(const SetupArgs& a, const double* lam_psig, double* lam_phi1,
                                   double* lam_s, hipStream_t s) {
  return solve(a.tables, a.cbuf, LoadPsiTranspose{lam_psig, lam_phi1}, StoreReal{lam_s}, false, s);
}

hipError_t launch_adj_white_noise(const SetupArgs& a, const double* lam_phi1, double* grad_w,
                                  hipStream_t s) {
  return solve(a.tables, a.cbuf, LoadReal{lam_phi1}, StoreReal{grad_w}, true, s);
}

template <typename T>
hipError_t launch_tcola_poisson(const TcolaArgs<T>& a, const PeriodicTables& t, double2* cbuf,
                                T* phi, T* rec_delta, T* rec_phi, hipStream_t s) {
  return solve(t, cbuf, LoadMass<T>{a.rho, rec_delta}, StorePotential<T>{phi, rec_phi}, false, s);
}

template hipError_t launch_tcola_poisson<float>(const TcolaArgs<float>&, const PeriodicTables&,
                                                double2*, float*, float*, float*, hipStream_t);
template hipError_t launch_tcola_poisson<double>(const TcolaArgs<double>&, const PeriodicTables&,
                                                 double2*, double*, double*, double*, hipStream_t);

}  // namespace scola
