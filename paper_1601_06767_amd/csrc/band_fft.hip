// Band -> real space: u_n(r) = sum_G c_n(G) exp(iG.r) on the transform grid, the
// wavefunctions whose products form the matrix element of Eq. (chi0).
//
// The coefficients live on a sphere of half-width rw (W = 2 rw + 1 frequencies per
// axis), so each axis is transformed from its W nonzero frequencies only, by the folded sums
// of fold.h: four real sums over the folded frequencies give the four points of a quad
// (about W / 2 complex by real FMAs per point).
//
//   k_band_ab (one workgroup per band and n1): the x3 lines of the n1 slab,
//     t3[j2][p3] in LDS, then the x2 lines -> tB[j1][p2][p3];
//   k_band_c: the x1 lines -> u[x1][p2][p3].
// x2 and x3 are stored in quad order (p = 4 j + t) so that the pair kernel reads whole quads;
// rows of x3 are padded to an odd number of 16-byte units (Geom::row).
#include <algorithm>

#include "common.h"
#include "fold.h"
#include "internal.h"

namespace gw {

namespace {

__device__ __forceinline__ int slot_band(const int32_t* band_idx, int band0, int nvalid, int nrows, int slot) {
  int idx = band0 + slot;
  if (idx >= nvalid) idx = nvalid - 1;
  const int band = band_idx ? band_idx[idx] : idx;
  return band < 0 ? 0 : (band >= nrows ? nrows - 1 : band);   // never read outside the coefficient rows
}

template <typename V> __device__ __forceinline__ double2 widen(V x) { return double2{(double)x.x, (double)x.y}; }
template <typename T> __device__ __forceinline__ cx<T> narrow(double2 x) { return cx<T>{T(x.x), T(x.y)}; }

// Sums of the float32 bands: those of x3 (with the float32 factors) and of x1, which memory bounds, in float64,
// those of x2 in float32.  The rounding of three float32 passes made about half of a pair density's error (rms
// of the norm, 24^3 1.8e-7 -> 1.6e-7, 48^3 2.1 -> 1.7, 72^3 1.9 -> 1.5, 128^3 2.2 -> 1.8; 128^3 in 32 bands: x3 and
// x2 112 -> 134 us, x1 88 -> 92; with float64 factors from memory x3 and x2 210 us, 1.62e-7 for 1.64e-7 at 96^3).
constexpr int kBandAbThreads = 512;
constexpr int kBq = 4;   // quads per thread: the four share one pass over the line's frequencies

// One workgroup per (band slot, j1).  tab[n][j]: the factors (cos, sin)(n j theta), quad 0 as fold.h;
// in LDS beside the slab when both fit (TL).  Where the LDS has room for them (CL), the slab's coefficients are
// gathered into it first, all at once: a thread that sums a line would wait for two dependent loads per
// frequency (72^3: float64, 56 bands 52 us, 58 before; float32, 4000 bands with the x1 pass 4.0 ms, 5.3 before).
template <typename T, bool TL, bool CL>
__global__ __launch_bounds__(kBandAbThreads) void k_band_ab(const double2* __restrict__ coef, int npw,
                                                            const int32_t* __restrict__ band_idx, int band0,
                                                            int nvalid, int nrows, const int32_t* __restrict__ wf_map,
                                                            int rw, int nt, int row, const cx<T>* __restrict__ gtab,
                                                            cx<T>* __restrict__ tB) {
  using V = cx<T>;
  extern __shared__ __align__(16) unsigned char s_raw[];
  const int W = 2 * rw + 1, nq = nt / 4;
  V* s_t3 = (V*)s_raw;                    // [j2][p3], W x nt
  V* s_tab = s_t3 + (size_t)W * nt;       // (rw + 1) x nq
  V* s_c = s_tab + (size_t)(rw + 1) * nq; // [j2][j3], W x W
  const int j1 = blockIdx.x;
  const int slot = blockIdx.y;
  if constexpr (TL)
    for (int i = threadIdx.x; i < (rw + 1) * nq; i += blockDim.x) s_tab[i] = gtab[i];
  const V* tab = TL ? s_tab : gtab;
  const int band = slot_band(band_idx, band0, nvalid, nrows, slot);
  const double2* c = coef + (size_t)band * npw;
  if constexpr (CL) {
    const int32_t* map = wf_map + (size_t)j1 * W * W;
    for (int i = threadIdx.x; i < W * W; i += blockDim.x) {
      const int ig = map[i];
      const double2 v = ig >= 0 ? c[ig] : double2{0.0, 0.0};
      s_c[i] = V{T(v.x), T(v.y)};
    }
  }
  if constexpr (TL) __syncthreads();
  const int ng = (nq + kBq - 1) / kBq;    // groups of quads; the last one overlaps its neighbour
  for (int task = threadIdx.x; task < W * ng; task += blockDim.x) {
    const int j2 = task / ng, q0 = nq < kBq ? 0 : min((task % ng) * kBq, nq - kBq);
    const int32_t* map = wf_map + ((size_t)j1 * W + j2) * W + rw;   // index by n3
    double2 y[kBq][4];
    points_of_quads<double2, kBq>(
        rw, q0 == 0,
        [&](int n) {
          if constexpr (CL) return widen(s_c[j2 * W + rw + n]);
          const int ig = map[n];
          return ig >= 0 ? c[ig] : double2{0.0, 0.0};
        },
        [&](int n, int k) { return widen(tab[n * nq + min(q0 + k, nq - 1)]); }, y);
    V* dst = s_t3 + (size_t)j2 * nt + 4 * q0;
#pragma unroll
    for (int k = 0; k < kBq; ++k)
      if (q0 + k < nq) {
#pragma unroll
        for (int a = 0; a < 4; ++a) dst[4 * k + a] = narrow<T>(y[k][a]);
      }
  }
  __syncthreads();
  V* out = tB + ((size_t)slot * W + j1) * nt * row;
  for (int task = threadIdx.x; task < nt * ng; task += blockDim.x) {
    const int p3 = task % nt, q0 = nq < kBq ? 0 : min((task / nt) * kBq, nq - kBq);
    V y[kBq][4];
    points_of_quads<V, kBq>(
        rw, q0 == 0, [&](int n) { return s_t3[(size_t)(n + rw) * nt + p3]; },
        [&](int n, int k) { return tab[n * nq + min(q0 + k, nq - 1)]; }, y);
#pragma unroll
    for (int k = 0; k < kBq; ++k)
      if (q0 + k < nq) {
#pragma unroll
        for (int a = 0; a < 4; ++a) out[(size_t)(4 * (q0 + k) + a) * row + p3] = y[k][a];
      }
  }
}

// x1 lines: one (p2, p3) column and kBq quads per thread (wave-uniform quads: scalar factors),
// planes stored in natural x1 order.
template <typename T>
__global__ __launch_bounds__(256) void k_band_c(const cx<T>* __restrict__ tB, int rw, int nt, int row,
                                                const double2* __restrict__ tab, cx<T>* __restrict__ psi) {
  using V = cx<T>;
  const int W = 2 * rw + 1, nq = nt / 4;
  const int slot = blockIdx.y;
  const int q0 = nq < kBq ? 0 : min((int)blockIdx.z * kBq, nq - kBq);
  const int plane = nt * row;
  const int p23 = blockIdx.x * blockDim.x + threadIdx.x;
  if (p23 >= plane) return;
  const V* src = tB + ((size_t)slot * W + rw) * plane + p23;   // index by n1
  double2 y[kBq][4];
  points_of_quads<double2, kBq>(
      rw, q0 == 0, [&](int n) { return widen(src[(ptrdiff_t)n * plane]); },
      [&](int n, int k) { return tab[n * nq + min(q0 + k, nq - 1)]; }, y);
  V* dst = psi + (size_t)slot * nt * plane + p23;
#pragma unroll
  for (int k = 0; k < kBq; ++k)
    if (q0 + k < nq) {
#pragma unroll
      for (int a = 0; a < 4; ++a) dst[(size_t)quad_x(4 * (q0 + k) + a, nt) * plane] = narrow<T>(y[k][a]);
    }
}

template <typename T, bool TL, bool CL>
hipError_t allow_lds() {
  static OncePerDevice done;
  return allow_whole_lds(reinterpret_cast<const void*>(&k_band_ab<T, TL, CL>), done);
}

}  // namespace

size_t band_scratch_bytes(const Geom& g, int nslot, bool fp64) {
  return (size_t)nslot * g.W * g.nt * g.row(fp64) * (fp64 ? 16 : 8);
}

template <typename T>
hipError_t launch_band_to_real(const Geom& g, const double2* coef, int nrows, const int32_t* band_idx, int band0, int nvalid,
                               int nslot, void* tB, void* psi, hipStream_t st) {
  constexpr bool f64 = std::is_same<T, double>::value;
  const cx<T>* tab = f64 ? (const cx<T>*)g.d_pts64 : (const cx<T>*)g.d_pts32;
  const int nt = g.nt, W = g.W, row = g.row(f64), nq = nt / 4;
  const size_t slab = (size_t)W * nt * sizeof(cx<T>), both = slab + (size_t)(g.rw + 1) * nq * sizeof(cx<T>);
  // wavefunction spheres are limited by their slab on the stated grid
  if ((size_t)(128 + W * g.nd) * sizeof(cx<T>) > 160 * 1024 || slab > 160 * 1024) return hipErrorInvalidValue;
  const dim3 grid(W, nslot);
  const size_t all = both + (size_t)W * W * sizeof(cx<T>);
  const int ng = (nq + kBq - 1) / kBq;
  const int threads = std::min(kBandAbThreads, (nt * ng + 63) / 64 * 64);
  auto run = [&](auto f, hipError_t allowed, size_t lds) {
    if (allowed != hipSuccess) return allowed;
    f<<<grid, threads, lds, st>>>(coef, g.npw, band_idx, band0, nvalid, nrows, g.d_wf_map, g.rw, nt, row, tab,
                                  (cx<T>*)tB);
    return hipGetLastError();
  };
  hipError_t e = all <= kLdsBytes    ? run(k_band_ab<T, true, true>, allow_lds<T, true, true>(), all)
                 : both <= kLdsBytes ? run(k_band_ab<T, true, false>, allow_lds<T, true, false>(), both)
                                     : run(k_band_ab<T, false, false>, allow_lds<T, false, false>(), slab);
  if (e != hipSuccess) return e;
  k_band_c<T><<<dim3((nt * row + 255) / 256, nslot, ng), 256, 0, st>>>((const cx<T>*)tB, g.rw, nt, row, g.d_pts64,
                                                                       (cx<T>*)psi);
  return hipGetLastError();
}

template hipError_t launch_band_to_real<double>(const Geom&, const double2*, int, const int32_t*, int, int, int, void*,
                                                void*, hipStream_t);
template hipError_t launch_band_to_real<float>(const Geom&, const double2*, int, const int32_t*, int, int, int, void*,
                                               void*, hipStream_t);

}  // namespace gw
