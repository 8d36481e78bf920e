// The COH self-energy of Eq. (sigmach), static limit and plasmon-pole form.
//
// Static limit, summed with the same column form
// (bands and energy-window representatives with their weights) as Eq. (energyintegration):
//   S[n][n'] = 1/2 sum_c w_c sum_{G G'} M_{n c}(G) A_{G G'} conj(M_{n' c}(G')),
//   A = [eps^-1 - I] diag(v).
// The pair densities of a chunk come from the pair kernels; then Z = conj(M) A^T (one
// float64 MFMA GEMM) and S += X Z^T over the flattened (column, G) index with X = w_c M (split
// into blocks whose partial sums are added in a fixed order).
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace gw {

namespace {

// at[h][g] = A[g][h] = (eps_inv[g][h] - delta_gh) v[h] for g, h < ng (A transposed, so that
// Z = conj(M) A^T reads it row by row); zero in the padding up to ngp
__global__ void k_coh_kernel(const double2* __restrict__ eps_inv, const double* __restrict__ v, int ng, int ngp,
                             double2* __restrict__ a) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)ngp * ngp) return;
  const int h = (int)(e / ngp), g = (int)(e % ngp);
  double2 x{0.0, 0.0};
  if (g < ng && h < ng) {
    x = eps_inv[(size_t)g * ng + h];
    if (g == h) x.x -= 1.0;
    x.x *= v[h];
    x.y *= v[h];
  }
  a[e] = x;
}

constexpr int kCohTile = 32;     // k-values per LDS tile
constexpr int kCohMaxStates = 32;

// part[blk][n][n'] = sum over the block's k-range of w_c M[n][k] Z[n'][k], k = c ngp + G,
// rows of length cc ngp (pairs v-major), columns c >= nvalid weigh 0.
__global__ __launch_bounds__(256) void k_coh_reduce(const double2* __restrict__ m, const double2* __restrict__ z,
                                                    int ns, int cc, int ngp, int nvalid,
                                                    const double* __restrict__ n_col, int c0, long long kper,
                                                    double2* __restrict__ part) {
  __shared__ double2 sx[kCohMaxStates][kCohTile];
  __shared__ double2 sz[kCohMaxStates][kCohTile];
  const long long klen = (long long)cc * ngp;
  const long long k0 = (long long)blockIdx.x * kper;
  const long long k1 = k0 + kper < klen ? k0 + kper : klen;
  const int tid = threadIdx.x;
  const int nout = ns * ns;
  double2 acc[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] = double2{0.0, 0.0};
  for (long long kt = k0; kt < k1; kt += kCohTile) {
    __syncthreads();
    for (int e = tid; e < ns * kCohTile; e += 256) {
      const int n = e / kCohTile, j = e % kCohTile;
      const long long k = kt + j;
      double2 x{0.0, 0.0}, y{0.0, 0.0};
      if (k < k1) {
        const int c = (int)(k / ngp);
        const double w = c < nvalid ? (n_col ? n_col[c0 + c] : 1.0) : 0.0;
        x = m[(size_t)n * klen + k];
        x.x *= w;
        x.y *= w;
        y = z[(size_t)n * klen + k];
      }
      sx[n][j] = x;
      sz[n][j] = y;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = tid + 256 * r;
      if (o < nout) {
        const int n = o / ns, np = o % ns;
#pragma unroll 8
        for (int j = 0; j < kCohTile; ++j) cmac(acc[r], sx[n][j], sz[np][j]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = tid + 256 * r;
    if (o < nout) part[(size_t)blockIdx.x * nout + o] = acc[r];
  }
}

// s[o] += 1/2 sum_blk part[blk][o], blocks in order
__global__ void k_coh_sum(const double2* __restrict__ part, int nblk, int nout, double2* __restrict__ s) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nout) return;
  double2 t{0.0, 0.0};
  for (int b = 0; b < nblk; ++b) t = cadd(t, part[(size_t)b * nout + o]);
  s[o] = cadd(s[o], double2{0.5 * t.x, 0.5 * t.y});
}

// ---------------------------------------------------------------- plasmon-pole COH
// Eq. (sigmach) with the plasmon-pole eps^-1 (each element a single pole of weight Omega^2 at
// wt), after the E' integral:
//   S_j[n][n'] = 1/2 sum_c w_c sum_{G G'} M_{n c}(G) A_{GG'}(x_jc) conj(M_{n' c}(G')),
//   A_{GG'}(x) = B_{GG'} / (x - wt_{GG'}),  B = Omega^2 v(G') / wt,  x_jc = E_j - E_c + i delta.
// k_gpp_coh_prep forms (B, wt) once per call; k_coh_gpp keeps a 64 x 64 tile of them in registers and
// streams the columns c of a chunk and the energies E_j past it, both sums on float64 MFMA 16x16x4:
//   W[G'][n] = sum_G A_GG' M_n(G): A operand Re A^T and Im A^T (each lane evaluates its own element),
//     B operand [Re M | Im M] of 8 states, 16 columns in all; the two products X1, X2 combine to
//     W_re = X1_r - X2_i, W_im = X1_i + X2_r (lanes 8 apart);
//   Y[n'][n] += sum_G' w_c M_n'(G') W[G'][n]: an accumulator register of W holds four G' of each lane
//     group, which is the B operand's layout, so W goes straight into the second product.
// The states of a column come in by direct loads one column ahead.  Partial sums per (tile, share of
// the columns) are reduced in a fixed order.
constexpr int kGpT = 64;      // G rows and G' columns of a tile
constexpr int kGpWaves = 8;   // each wave 16 G' and half of the G: two or more waves per SIMD, so that one
                              // evaluates elements while another's products run
constexpr int kGpS = 8;       // states per block
constexpr int kGpE = 4;       // energies per pass
static_assert(kGpE <= kGpWaves, "a wave per energy adds the partial sums");
// Shares of the columns.  One workgroup runs per CU, so a launch lasts as long as its rounds over 256 CUs times
// the columns of a share; more shares are taken where that falls by two per cent or more (196 tiles of NG 800,
// 300 columns: five shares of 60 in four rounds, 2.70 ms a call; 13 shares of 24 in ten rounds, every wave with
// partial sums of its own, 2.83).  Every share keeps partial sums (4 KiB a tile): as many shares as keep
// them within 8 MiB a pass, up to 16, and up to eight on any sphere.
inline int gpp_tiles(int ngp) { return (ngp / kGpT) * (ngp / kGpT); }
inline int gpp_shares(int tiles, int columns, int most) {
  auto cost = [&](int s) { return (long long)((tiles * s + 255) / 256) * ((columns + s - 1) / s); };
  int best = 1;
  for (int s = 2; s <= std::min(most, columns); ++s)
    if (cost(s) * 50 < cost(best) * 49) best = s;
  return best;
}
// shares that the partial sums of a pass over chunks of cc columns have room for
inline int gpp_share_room(int tiles, int cc) {
  return gpp_shares(tiles, cc, std::min(16, std::max(8, 2048 / tiles)));
}

struct GppEnergies {
  double e[kGpE];
};

// principal square root (non-negative real part; the sign of the imaginary part follows the
// argument's, signed zeros included)
__device__ __forceinline__ double2 csqrt_principal(double2 z) {
  const double r = hypot(z.x, z.y);
  const double re = sqrt(0.5 * r + 0.5 * z.x);
  const double im = copysign(sqrt(0.5 * r - 0.5 * z.x), z.y);
  return double2{re, im};
}

// (B, wt) for G, G' < ngp (rows G); elements without a pole (wt^2 not finite), with Omega^2 = 0,
// or in the padding: B = 0, wt = 1, so that their term vanishes for every x
__global__ void k_gpp_coh_prep(const double2* __restrict__ om2, const double2* __restrict__ wt2,
                               const double* __restrict__ v, int ng, int ngp, double2* __restrict__ bb,
                               double2* __restrict__ ww) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)ngp * ngp) return;
  const int g = (int)(e / ngp), h = (int)(e % ngp);
  double2 b{0.0, 0.0}, w{1.0, 0.0};
  if (g < ng && h < ng) {
    const size_t i = (size_t)g * ng + h;
    const double2 o = om2[i], t = wt2[i];
    if (isfinite(t.x) && isfinite(t.y) && (o.x != 0.0 || o.y != 0.0)) {
      w = csqrt_principal(t);
      // B = o v(h) / w
      const double d = w.x * w.x + w.y * w.y;
      const double vr = v[h] / d;
      b = double2{(o.x * w.x + o.y * w.y) * vr, (o.y * w.x - o.x * w.y) * vr};
    }
  }
  bb[e] = b;
  ww[e] = w;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// the value of lane ^ 8 (within rows of 16 lanes: a rotation by 8)
__device__ __forceinline__ double lane_xor8(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, 0x128, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), 0x128, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// part[(slot * kGpE + j) * 64 + lane] += sum over this share of the chunk's columns for lane's
// (n, n') = (lane / 8, lane % 8) of state blocks (sa, sb), slot = tile * shares + share; states >= ns repeat
// the last one (their sums are not read).  Bound by float64 MFMA beside the
// evaluation of the elements on the VALU.  Measured (NG 800, 8 states, 300 columns, 4 energies): 1.84 ms;
// 13.3 with the sums on the VALU, W through LDS and divisions in place of a reciprocal.
__global__ __launch_bounds__(64 * kGpWaves, 2) void k_coh_gpp(const double2* __restrict__ bb, const double2* __restrict__ ww,
                                                    int ngp, int ntile1, const double2* __restrict__ m, int cc, int ns,
                                                    int sa, int sb, int nvalid, const double* __restrict__ e_col,
                                                    const double* __restrict__ n_col, int c0, GppEnergies en, int ne,
                                                    double delta, double2* __restrict__ part) {
  constexpr int LD = kGpT + 1;   // states are stored 1040 bytes apart: the 8 of a read on different banks
  __shared__ __align__(16) double2 s_m0[2 * kGpS * LD];   // M_n(G) of block sa, then M_n'(G') of block sb
  __shared__ __align__(16) double2 s_m1[2 * kGpS * LD];
  const int tile = blockIdx.x;
  const int t0 = tile / ntile1, t1 = tile % ntile1;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g0 = (wave >> 2) * (kGpT / 2), h0 = (wave & 3) * 16;   // this wave's G and G' in the tile
  const int li = lane & 15, lk = lane >> 4;
  const int n = li & 7, im = li >> 3;      // this lane's state and part as a column (or row) of the products
  const int per = (nvalid + gridDim.y - 1) / gridDim.y;
  const int cb = min(nvalid, (int)blockIdx.y * per), ce = min(nvalid, cb + per);
  // this lane's elements: G = t0 tile + g0 + 4 s + lk, G' = t1 tile + h0 + li
  double2 bq[kGpT / 8], wq[kGpT / 8];
#pragma unroll
  for (int s = 0; s < kGpT / 8; ++s) {
    const size_t e = (size_t)(t0 * kGpT + g0 + 4 * s + lk) * ngp + t1 * kGpT + h0 + li;
    bq[s] = bb[e];
    wq[s] = ww[e];
  }
  const size_t klen = (size_t)cc * ngp;
  // rows q = wave and wave + 8: 64 values (1 KB) of one state, one wave instruction each
  auto issue = [&](int c, double2* buf) {
#pragma unroll
    for (int i = 0; i < 2 * kGpS / kGpWaves; ++i) {
      const int q = kGpWaves * i + wave;
      const int st = min((q < kGpS ? sa : sb) * kGpS + q % kGpS, ns - 1);
      const double2* src = m + (size_t)st * klen + (size_t)c * ngp + (q < kGpS ? t0 : t1) * kGpT + lane;
      __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)&buf[q * LD], 16, 0, 0);
    }
  };
  f64x4 y[kGpE];
#pragma unroll
  for (int j = 0; j < kGpE; ++j) y[j] = f64x4{0, 0, 0, 0};
  const double sgn = im ? 1.0 : -1.0;
  auto column = [&](int c, const double2* cur, double2* nxt) {
    wait_vm<0>();
    lds_barrier();   // the column has landed; the other buffer is no longer read
    if (c + 1 < ce) issue(c + 1, nxt);
    const double wc = n_col ? n_col[c0 + c] : 1.0;
    const double ec = e_col[c0 + c];
    const double* ml = (const double*)(cur + n * LD + g0) + im;             // + 2 (G - g0)
    const double* mr = (const double*)(cur + (kGpS + n) * LD + h0) + im;    // + 2 (G' - h0)
    double r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = wc * mr[2 * (4 * k + lk)];
#pragma unroll
    for (int j = 0; j < kGpE; ++j) {
      if (j < ne) {   // uniform
        const double xr = en.e[j] - ec;
        f64x4 x1{0, 0, 0, 0}, x2{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < kGpT / 8; ++s) {
          const double dr = xr - wq[s].x, di = delta - wq[s].y;
          const double den = fma(dr, dr, di * di);
          double inv = __builtin_amdgcn_rcp(den);   // and two Newton steps: 1 / den
          inv = fma(fma(-den, inv, 1.0), inv, inv);
          inv = __builtin_amdgcn_div_fixup(fma(fma(-den, inv, 1.0), inv, inv), den, 1.0);   // 0 and infinite den
          const double ar = fma(bq[s].x, dr, bq[s].y * di) * inv;
          const double ai = fma(bq[s].y, dr, -(bq[s].x * di)) * inv;
          const double l = ml[2 * (4 * s + lk)];
          x1 = mfma64(ar, l, x1);
          x2 = mfma64(ai, l, x2);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double w = fma(sgn, lane_xor8(x2[k]), x1[k]);
          y[j] = mfma64(r[k], w, y[j]);
        }
        __builtin_amdgcn_sched_barrier(0);   // one energy at a time in registers
      }
    }
  };
  if (cb < ce) {
    issue(cb, s_m0);
    for (int c = cb; c < ce; c += 2) {
      column(c, s_m0, s_m1);
      if (c + 1 < ce) column(c + 1, s_m1, s_m0);
    }
  }
  wait_vm<0>();
  // Y rows (n', part') = lk + 4 r, columns (n, part) = li, through LDS to one (n, n') per lane, the waves' sums
  // added in their order (wave j takes energy j):
  // S_re = Y[re][re] + Y[im][im], S_im = Y[re][im] - Y[im][re]  (row part, column part)
  double* sy = (double*)s_m0;   // 256 per wave: 16 KB of the 16.25
  double2* dst = part + ((size_t)(tile * gridDim.y + blockIdx.y) * kGpE) * 64 + lane;
  const int pn = lane / kGpS, pm = lane % kGpS;
#pragma unroll
  for (int j = 0; j < kGpE; ++j) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) sy[wave * 256 + (lk + 4 * k) * 16 + li] = y[j][k];
    __syncthreads();
    if (wave == j) {
      double2 t = dst[(size_t)j * 64];
      for (int w = 0; w < kGpWaves; ++w) {
        const double* yw = sy + w * 256;
        t.x += yw[pm * 16 + pn] + yw[(pm + 8) * 16 + pn + 8];
        t.y += yw[pm * 16 + pn + 8] - yw[(pm + 8) * 16 + pn];
      }
      dst[(size_t)j * 64] = t;
    }
  }
}

// out[j][n][n'] += 1/2 sum over the slots of part (fixed order: each thread a fixed
// strided subset, then a fixed tree), one workgroup per (j, n, n') of the pass
__global__ __launch_bounds__(256) void k_coh_gpp_sum(const double2* __restrict__ part, int nslot, int ne, int ns,
                                                     int sa, int sb, int e0, double2* __restrict__ out) {
  __shared__ double2 red[256];
  const int o = blockIdx.x;   // j * 64 + lane
  const int j = o / 64, lane = o % 64;
  const int n = sa * kGpS + lane / kGpS, np = sb * kGpS + lane % kGpS;
  double2 t{0.0, 0.0};
  for (int sl = threadIdx.x; sl < nslot; sl += 256) t = cadd(t, part[((size_t)sl * kGpE + j) * 64 + lane]);
  red[threadIdx.x] = t;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] = cadd(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && j < ne && n < ns && np < ns) {
    double2* d = out + ((size_t)(e0 + j) * ns + n) * ns + np;
    *d = cadd(*d, double2{0.5 * red[0].x, 0.5 * red[0].y});
  }
}

}  // namespace

int coh_max_states() { return kCohMaxStates; }

int gpp_coh_tile() { return kGpT; }
int gpp_coh_states_per_block() { return kGpS; }
int gpp_coh_energies_per_pass() { return kGpE; }
size_t gpp_coh_part_bytes(int ngp, int cc) {
  const int tiles = gpp_tiles(ngp);
  return (size_t)tiles * gpp_share_room(tiles, cc) * kGpE * 64 * sizeof(double2);
}

hipError_t launch_gpp_coh_prep(const void* modes, const double* v, int ng, int ngp, void* b, void* w, hipStream_t st) {
  const size_t n = (size_t)ngp * ngp;
  const double2* om2 = (const double2*)modes;
  k_gpp_coh_prep<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(om2, om2 + (size_t)ng * ng, v, ng, ngp,
                                                               (double2*)b, (double2*)w);
  return hipGetLastError();
}

hipError_t launch_gpp_coh(const void* b, const void* w, int ngp, const void* m, int cc, int ns, int sa, int sb,
                          int nvalid, const double* e_col, const double* n_col, int c0, const double* energies, int ne,
                          double delta, void* part, hipStream_t st) {
  if (ngp % kGpT != 0 || ne < 1 || ne > kGpE || nvalid < 1 || nvalid > cc) return hipErrorInvalidValue;
  GppEnergies en{};
  for (int j = 0; j < ne; ++j) en.e[j] = energies[j];
  const int tiles = gpp_tiles(ngp), shares = gpp_shares(tiles, nvalid, gpp_share_room(tiles, cc));
  k_coh_gpp<<<dim3(tiles, shares), 64 * kGpWaves, 0, st>>>((const double2*)b, (const double2*)w, ngp, ngp / kGpT,
                                                           (const double2*)m, cc, ns, sa, sb, nvalid, e_col, n_col, c0,
                                                           en, ne, delta, (double2*)part);
  return hipGetLastError();
}

hipError_t launch_gpp_coh_sum(const void* part, size_t part_bytes, int ne, int ns, int sa, int sb, int e0, void* out,
                              hipStream_t st) {
  const int nslot = (int)(part_bytes / (kGpE * 64 * sizeof(double2)));
  k_coh_gpp_sum<<<kGpE * 64, 256, 0, st>>>((const double2*)part, nslot, ne, ns, sa, sb, e0, (double2*)out);
  return hipGetLastError();
}

hipError_t launch_coh_kernel(const void* eps_inv, const double* v, int ng, int ngp, void* a, hipStream_t st) {
  const size_t n = (size_t)ngp * ngp;
  k_coh_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const double2*)eps_inv, v, ng, ngp, (double2*)a);
  return hipGetLastError();
}

hipError_t launch_coh_reduce(const void* m, const void* z, int ns, int cc, int ngp, int nvalid, const double* n_col,
                             int c0, int nblk, void* part, void* s, hipStream_t st) {
  if (ns < 1 || ns > kCohMaxStates || nblk < 1) return hipErrorInvalidValue;
  const long long klen = (long long)cc * ngp;
  long long kper = (klen + nblk - 1) / nblk;
  kper = (kper + kCohTile - 1) / kCohTile * kCohTile;
  const int nb = (int)((klen + kper - 1) / kper);
  k_coh_reduce<<<nb, 256, 0, st>>>((const double2*)m, (const double2*)z, ns, cc, ngp, nvalid, n_col, c0, kper,
                                   (double2*)part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nout = ns * ns;
  k_coh_sum<<<(nout + 255) / 256, 256, 0, st>>>((const double2*)part, nb, nout, (double2*)s);
  return hipGetLastError();
}

}  // namespace gw
