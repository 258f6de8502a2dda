// Dirichlet Poisson solve of every sCOLA box by type-I discrete sine transforms (App. C).
//
// A box of M particles per side has n = M - 1 interior PM nodes per side.  Three passes
// over the (n)^3 mesh of every box, all boxes in one launch each:
//   P1  per x-plane: fixed-point mass -> delta, delta' = delta - Delta Phi_BCs (App. C.1),
//       forward DST-I along z then y, in LDS;
//   P2  per chunk of consecutive x pencils of the box's n^2 (64 in FP32 plans, 32 in FP64):
//       forward DST-I along x, division by the FDA eigenvalue sum times the inverse
//       normalisation 8/M^3 (App. C.2, eq. Poisson_sine_space), inverse DST-I along x;
//   P3  per x-plane: inverse DST-I along y then z, and the potential written to the padded
//       node grid [-g, M+g]^3 with the shell filled from Phi_BCs (Sec. 3.4.2); g = 1, 2, 3
//       ghost layers at finite-difference order 2, 4, 6 (Sec. 3), where delta' also takes
//       the wide stencil's reach into the g Dirichlet layers (App. C.1).
//
// FP32 plans form every DST-I as a product with the sine matrix on the matrix cores
// (dst_mfma.h: split FP16 operands, FP32 accumulation); FP64 plans use the real-data sine
// transform through a half-length complex FFT on a quarter wavefront (poisson_passes.h).
// Within an evolution, P3 leaves each plane's boundary-source perimeter terms in its
// consumed work plane for the next solve's P1 (MeshArgs::bc_handoff).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "particle_common.h"
#include "poisson_passes.h"

namespace scola {

namespace {

// Waves per SIMD the FP32 passes are compiled for: their matrix-core transforms leave them
// latency-bound, so boxes up to 64^3 ask for full occupancy (at most 64 registers a lane), and
// so does the first pass of 80^3 at order 2 (16 boxes: 125 -> 107 us).  The other passes of
// larger boxes would spill (first pass of 96^3, 512 boxes: 1324 -> 1716 us, pencils 965 ->
// 1344), so they and FP64 plans take what their registers allow.  The 64^3 reverse passes and
// the passes of 64^3 and 48^3 at orders 4 and 6 need a few more registers than 64: they take 7
// waves (72 registers) rather than spill to scratch.
template <typename T, int R, bool ADJ = false, int NG = 1>
constexpr int pass_waves() {
  if (!std::is_same<T, float>::value) return 1;
  if ((R == 4 && (ADJ || NG > 1)) || (R == 3 && NG > 1)) return 7;
  return R <= 4 ? 8 : 1;
}
template <typename T, int R, bool ADJ, int NG>
constexpr int first_pass_waves() {
  return std::is_same<T, float>::value && R == 5 && NG == 1 ? 8 : pass_waves<T, R, ADJ, NG>();
}

// Threads of a block.  The FP32 passes above 64^3 have more 16-row tiles of the sine matrix than
// a block of 256 has waves: with 512, each wave has one tile, half the values in flight per
// thread and so fewer registers, and more waves fit a CU.  With 256 and 512 threads, us for 64
// boxes: first pass of 96^3 228 and 195, of 112^3 455 and 347, of 128^3 577 and 462; pencils of
// 80^3 107 and 95, 96^3 159 and 141, 112^3 256 and 235; third pass of 80^3 105 and 106, 112^3 337
// and 276, 128^3 453 and 367; reverse third pass of 80^3 to 128^3 146, 222, 411, 539 and 129,
// 197, 324, 481.  The third pass of 96^3, whose six tiles leave two of eight waves idle in the
// products, takes the same time either way (64 boxes 159 and 153, 512 boxes 1046 and 1059).  The
// pencils of 128^3, whose eight tiles four waves share evenly, are faster with 256 where they
// fill the chip (64 boxes 360 and 392, 8 boxes 55 and 56; one box, a block per CU, 16 and 14).
// 64 R threads, where no wave is idle, were slower (96^3, 512 boxes: 1522, 1049 and 1244): six or
// seven waves do not spread evenly over the four SIMDs.
template <typename T, int R>
constexpr int pass_threads() {
  return std::is_same<T, float>::value && R >= 5 ? 512 : kBlock;
}
// of the pencil pass in launches of more than kFewChunks chunks (8 boxes of 128^3 have 2024)
constexpr int kFewChunks = 2048;
template <typename T, int R>
constexpr int many_pencils_threads() {
  return R == 8 ? kBlock : pass_threads<T, R>();
}

template <typename T, int R, bool ADJ, int NG>
__global__ void __launch_bounds__((pass_threads<T, R>()))
__attribute__((amdgpu_waves_per_eu(first_pass_waves<T, R, ADJ, NG>())))
k_poisson_p1(MeshArgs<T> a, BlockMap m) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = logical_block(m);
  if (L < m.count) poisson_p1_block<T, R, ADJ, NG, pass_threads<T, R>()>(a, m, L, smem);
}

template <typename T, int R, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(pass_waves<T, R>())))
k_poisson_p2(MeshArgs<T> a, BlockMap m) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = logical_block(m);
  if (L < m.count) poisson_p2_block<T, R, NT>(a, m, L, smem);
}

template <typename T, int R, bool ADJ, int NG>
__global__ void __launch_bounds__((pass_threads<T, R>()))
__attribute__((amdgpu_waves_per_eu(pass_waves<T, R, ADJ, NG>())))
k_poisson_p3(MeshArgs<T> a, BlockMap m) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = logical_block(m);
  if (L < m.count) poisson_p3_block<T, R, ADJ, NG, pass_threads<T, R>()>(a, m, L, smem);
}

}  // namespace

// Dynamic LDS of each pass for boxes of M nodes: FP64 plans the 2M twiddles, then P1 the
// (M-1)^2 plane, P2 the M eigenvalues and an (M-1) x 33 pencil tile, P3 the plane and the
// perimeter terms it hands on; FP32 plans the block-maximum slots, then the plane region
// (the plane or the split lines aliasing it, whose tail beyond the plane holds P3's
// perimeter terms before the transform), P2 the eigenvalues and the chunk's split lines
// aliased by its output tile.  P3 holds the padded plane's border in registers.  Sized per M
// and per pass, so small boxes keep more blocks per CU.
template <typename T>
size_t poisson_lds_bytes(int M, int pass, int ng) {
  (void)ng;
  const size_t n = (size_t)M - 1, tw = 2 * (size_t)M * sizeof(cx<T>);
  // P3: the perimeter terms it hands to the next solve's P1, 8-byte aligned behind the plane
  const size_t terms = 8 + 4 * (n - 1) * sizeof(double);
  if (std::is_same<T, float>::value) {
    // matrix-core transforms: block-maximum slots, then the plane region (the plane or the
    // split lines that alias it); P2: the eigenvalues, then the split lines of the chunk's
    // columns aliased by the output tile
    const int R = M / 16;
    const size_t head = R >= 5 ? mfma_head<512>() : mfma_head<kBlock>();   // of any block size
    const size_t region = std::max(n * n * sizeof(float), mfma_split_bytes(R));
    if (pass == 1 || pass == 3) return head + region;
    const size_t lines =
        (size_t)kPencilChunkMfma * (32 * ((R + 1) / 2) + 8) * 2 * sizeof(_Float16);
    return head + (size_t)M * sizeof(float) +
           std::max(n * (kPencilChunkMfma + 1) * sizeof(float), lines);
  }
  if (pass == 1) return tw + n * n * sizeof(T);
  if (pass == 2) return tw + ((size_t)M + n * (kPencilChunk + 1)) * sizeof(T);
  return tw + n * n * sizeof(T) + terms;
}

namespace {

template <typename T, int R, bool ADJ, int NG>
hipError_t launch_poisson_R(const MeshArgs<T>& a, const BlockMap& p1, const BlockMap& p2,
                            const BlockMap& p3, hipStream_t s) {
  const size_t l1 = poisson_lds_bytes<T>(16 * R, 1, NG), l2 = poisson_lds_bytes<T>(16 * R, 2, NG),
               l3 = poisson_lds_bytes<T>(16 * R, 3, NG);
  constexpr int kNT = pass_threads<T, R>(), kMany = many_pencils_threads<T, R>();
  if (l1 > 65536 || l2 > 65536 || l3 > 65536) {
    // allow more than 64 KiB of dynamic LDS (160 KiB on gfx950): a function attribute of
    // each device, set once per device
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? (1ull << dev) : 0ull;
    if (!bit || !(done.load() & bit)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_poisson_p1<T, R, ADJ, NG>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)l1);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_poisson_p2<T, R, kNT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)l2);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_poisson_p2<T, R, kMany>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)l2);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_poisson_p3<T, R, ADJ, NG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)l3);
      if (e != hipSuccess) return e;
      done.fetch_or(bit);
    }
  }
  const dim3 block(kNT);
  if (p1.count > 0)
    hipLaunchKernelGGL((k_poisson_p1<T, R, ADJ, NG>), dim3(padded_grid(p1)), block, l1, s, a, p1);
  if (p2.count > kFewChunks)
    hipLaunchKernelGGL((k_poisson_p2<T, R, kMany>), dim3(padded_grid(p2)), dim3(kMany), l2, s, a,
                       p2);
  else if (p2.count > 0)
    hipLaunchKernelGGL((k_poisson_p2<T, R, kNT>), dim3(padded_grid(p2)), block, l2, s, a, p2);
  if (p3.count > 0)
    hipLaunchKernelGGL((k_poisson_p3<T, R, ADJ, NG>), dim3(padded_grid(p3)), block, l3, s, a, p3);
  return hipGetLastError();
}

template <typename T, int R>
hipError_t launch_poisson_RA(const MeshArgs<T>& a, const BlockMap& p1, const BlockMap& p2,
                             const BlockMap& p3, hipStream_t s, bool adjoint) {
  if (adjoint) {
    // the reverse passes exist for order 2 only (the plan refuses the others)
    if (a.ng != 1) return hipErrorInvalidValue;
    return launch_poisson_R<T, R, true, 1>(a, p1, p2, p3, s);
  }
  switch (a.ng) {
    case 1: return launch_poisson_R<T, R, false, 1>(a, p1, p2, p3, s);
    case 2: return launch_poisson_R<T, R, false, 2>(a, p1, p2, p3, s);
    case 3: return launch_poisson_R<T, R, false, 3>(a, p1, p2, p3, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <typename T>
hipError_t launch_poisson(const MeshArgs<T>& a, int M, const BlockMap& p1, const BlockMap& p2,
                          const BlockMap& p3, hipStream_t s, bool adjoint) {
  switch (M) {
    case 16: return launch_poisson_RA<T, 1>(a, p1, p2, p3, s, adjoint);
    case 32: return launch_poisson_RA<T, 2>(a, p1, p2, p3, s, adjoint);
    case 48: return launch_poisson_RA<T, 3>(a, p1, p2, p3, s, adjoint);
    case 64: return launch_poisson_RA<T, 4>(a, p1, p2, p3, s, adjoint);
    case 80: return launch_poisson_RA<T, 5>(a, p1, p2, p3, s, adjoint);
    case 96: return launch_poisson_RA<T, 6>(a, p1, p2, p3, s, adjoint);
    case 112: return launch_poisson_RA<T, 7>(a, p1, p2, p3, s, adjoint);
    case 128: return launch_poisson_RA<T, 8>(a, p1, p2, p3, s, adjoint);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_poisson<float>(const MeshArgs<float>&, int, const BlockMap&,
                                          const BlockMap&, const BlockMap&, hipStream_t, bool);
template hipError_t launch_poisson<double>(const MeshArgs<double>&, int, const BlockMap&,
                                           const BlockMap&, const BlockMap&, hipStream_t, bool);
template size_t poisson_lds_bytes<float>(int, int, int);
template size_t poisson_lds_bytes<double>(int, int, int);

}  // namespace scola
