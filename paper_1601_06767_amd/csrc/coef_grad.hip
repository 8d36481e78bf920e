// Gradients with respect to the wavefunction coefficients (float64): the adjoint of the
// path coefficients -> real-space bands -> pair densities of Eq. (chi0).
//
// With m_p = F(conj(u_v) u_c), F x (G) = (1/N) sum_r x(r) e^{iG.r}, and u_n = B c_n,
// B c (r) = sum_g c(g) e^{ig.r}, a real loss with chi0bar = dL/dRe chi0 + i dL/dIm chi0
// gives (same convention for every gradient):
//   mbar_p = sum_w [conj(w_p) chi0bar m_p + w_p chi0bar^H m_p]           (two GEMMs)
//   h_p    = F^H mbar_p,   h_p(r) = (1/N) sum_G mbar_p(G) e^{-iG.r}
//   ubar_c = sum_v h_vc u_v,   ubar_v = sum_c conj(h_vc) u_c
//   cbar_n = B^H ubar_n,   cbar_n(g) = sum_r ubar_n(r) e^{-ig.r}
// h_p is never stored: it is formed one x1 plane at a time, in the workgroup that
// accumulates the sum over partner bands for one band and one plane.  Each step is the
// transpose of a forward step, with the conjugate twiddles:
//   k_qbar      transpose of the pair finish stage (sphere scatter, x1 transform, 1/N)
//   k_ubar      transposes of the x2 and x3 stages of the pair kernel, times the partner
//               band, summed over the partners (conduction gradient: over the valence
//               bands; valence gradient: over the columns of the chunk, added up over chunks)
//   k_bandT_*   transpose of the band transform (x1, then x2 and x3, sphere gather), folded sums
// The inverse line transforms of k_qbar and k_ubar use the folded sums of fold.h, conjugated:
// conj(sum_n conj(t_n) e^{+2 pi i n x / N}) = sum_n t_n e^{-2 pi i n x / N}.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "fold.h"
#include "internal.h"

namespace gw {

namespace {

__device__ __forceinline__ double2 conjd(double2 a) { return double2{a.x, -a.y}; }

// a[p][G] = s_p m[p][G], s_p = w_p or conj(w_p) (w_p = w[p] + i w[np + p] when nparts == 2)
__global__ void k_weight_rows(const double2* __restrict__ m, int npair, int ngp, const double* __restrict__ w,
                              int nparts, int conj_w, double2* __restrict__ a) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)npair * ngp) return;
  const int p = (int)(e / ngp);
  double2 s{w[p], nparts == 2 ? w[(size_t)npair + p] : 0.0};
  if (conj_w) s.y = -s.y;
  a[e] = cmul(s, m[e]);
}

// qbar[pair][x1][l] = scale sum_{n1} e^{-2 pi i n1 x1 / N} mbar[pair][G(n1, l)], the transpose of the
// finish stage: per line l the points of each quad from the folded frequencies (the conjugate of
// points_of_quads' sum: A - i B); one workgroup per pair, quads wave-uniform (scalar factors).
template <int RC>
__global__ __launch_bounds__(256) void k_qbar(const double2* __restrict__ mbar, const int32_t* __restrict__ chi_map,
                                              int ngp, int nt, int nl, double scale, const double* __restrict__ fac,
                                              double2* __restrict__ qbar) {
  constexpr int K = 2 * RC + 1;
  const size_t pair = blockIdx.x;
  const int nq = nt / 4, h = nt / 2;
  const double2* src = mbar + pair * ngp;
  for (int l = threadIdx.x; l < nl; l += blockDim.x) {
    double2* dst = qbar + pair * nt * (size_t)nl + l;
    double2 e[RC + 1], o[RC + 1];   // folded frequencies
    double2 t[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const int ig = chi_map[(size_t)j * nl + l];
      t[j] = ig >= 0 ? src[ig] : double2{0.0, 0.0};
      t[j] = double2{t[j].x * scale, t[j].y * scale};
    }
    e[0] = t[RC];
#pragma unroll
    for (int n = 1; n <= RC; ++n) {
      e[n] = cadd(t[RC + n], t[RC - n]);
      o[n] = csub(t[RC + n], t[RC - n]);
    }
    auto mac = [](double2& a, double f, double2 x) {
      a.x = fma(f, x.x, a.x);
      a.y = fma(f, x.y, a.y);
    };
    {   // quad 0: x = 0, H / 2, H, 3 H / 2
      double2 ae = e[0], ao{0, 0}, be = e[0], bo{0, 0};
#pragma unroll
      for (int n = 1; n <= RC; ++n) {
        if (n % 2 == 0) {
          ae = cadd(ae, e[n]);
          be = n % 4 == 0 ? cadd(be, e[n]) : csub(be, e[n]);
        } else {
          ao = cadd(ao, e[n]);
          bo = n % 4 == 1 ? cadd(bo, o[n]) : csub(bo, o[n]);
        }
      }
      dst[0] = cadd(ae, ao);
      dst[(size_t)(h / 2) * nl] = minus_i(be, bo);
      dst[(size_t)h * nl] = csub(ae, ao);
      dst[(size_t)(h + h / 2) * nl] = plus_i(be, bo);
    }
#pragma unroll 1
    for (int j = 1; j < nq; ++j) {
      const double* f = fac + (size_t)j * (2 * RC + 2);
      double2 ae = e[0], ao{0, 0}, be{0, 0}, bo{0, 0};
#pragma unroll
      for (int n = 1; n <= RC; ++n) {
        mac(n % 2 == 0 ? ae : ao, f[n], e[n]);
        mac(n % 2 == 0 ? be : bo, f[RC + 1 + n], o[n]);
      }
      const double2 x = cadd(ae, ao), y = csub(ae, ao), sx = cadd(be, bo), sy = csub(bo, be);
      dst[(size_t)j * nl] = minus_i(x, sx);
      dst[(size_t)(h - j) * nl] = minus_i(y, sy);
      dst[(size_t)(h + j) * nl] = plus_i(y, sy);
      dst[(size_t)(nt - j) * nl] = plus_i(x, sx);
    }
  }
}

// Shape of a k_ubar workgroup: UQ x3 quads per wave, ROWS x2 rows and their U 16-byte units of the partner's
// plane (two buffers).  SMALL: two own bands share the partner's rows (twelve waves).
template <int RC, bool SMALL, int UQ_> struct UbarShape {
  static constexpr int K = 2 * RC + 1, UQ = UQ_, OWN = SMALL ? 2 : 1, ROWS = SMALL ? 48 : 64;
  static constexpr int NW = SMALL ? 6 : 8, QUADS = NW * UQ;           // waves per own band
  static constexpr int NT = 64 * NW * OWN;
  static constexpr int rest = OWN * (K * K + ROWS * K) + (RC + 1) * QUADS;   // lines, rows, factors
  static constexpr int U = SMALL ? 48 * 49 : (10240 - rest) / 2 / 64 * 64;
  static_assert(2 * U + rest <= 10240, "k_ubar workgroup exceeds the LDS");
  static bool fits(int nt, int row, int rq) {
    return 4 * rq <= ROWS && 4 * rq * row <= U && nt / 4 <= QUADS;
  }
};

// One workgroup per (OWN own bands, part of the x2 quads, x1 plane).  For every partner band: h of the pair on this
// plane from qbar (x2 transform into LDS, then the x3 transform), times the partner's plane, accumulated in
// registers; the plane of ubar is written (COND) or added (valence, accumulated over conduction chunks) at
// the end.
//   COND:  own = column c < ncs (pairs v * ncs + c, v < nvs), ubar_c += h_vc u_v
//   !COND: own = valence slot v < nvs (pairs v * ncs + c, c < ncs), ubar_v += conj(h_vc) u_c
// The inverse sums run on the conjugates (conj h), so that the factors are the forward ones.
// A wave takes UQ x3 quads (uniform: factors by scalar loads), a lane one row: the frequencies and the
// partner's rows are read from LDS at an odd stride.  The partner's rows come by direct loads and the pair's
// lines through registers, one partner ahead.  Lines and rows are kept folded over +-n3: slot n = sum,
// RC + n = difference.  Measured (RC 7 on 44^3, 64 x 256 pairs): conduction 3.9 ms, valence 4.1 (5.8 with
// one own band per workgroup: the direct loads of the rows bound it); 8.6 and 9.2 with the
// partner's rows read from memory by lanes a row apart and nothing in flight across partners.
template <int RC, bool COND, typename P>
__global__ __launch_bounds__(P::NT) void k_ubar(const double2* __restrict__ qbar, const double2* __restrict__ partner,
                                             int nvs, int ncs, int nt, int nl, int row, int nparts, int rq,
                                             const int32_t* __restrict__ rowtab, const double2* __restrict__ pts,
                                             double2* __restrict__ ubar) {
  constexpr int K = P::K, UQ = P::UQ;
  constexpr int NLD = 2;                          // (n2, n3 >= 0) entries per thread
  const int nq = nt / 4;
  // arrays of their own: reads of one do not wait for the direct loads into another
  __shared__ __align__(16) double2 s_u0[P::U], s_u1[P::U];
  __shared__ double2 s_qs[P::OWN * K * K];        // [n2][slot] conj of the pair's lines
  __shared__ double2 s_ts[P::OWN * P::ROWS * K];  // [row][slot]
  __shared__ double2 s_f[(RC + 1) * P::QUADS];    // [n][j] factors
  const int nown = ((COND ? ncs : nvs) + P::OWN - 1) / P::OWN;
  const int total = nt * nparts * nown, per = (total + 7) / 8;
  const int id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per || id >= total) return;
  const int own0 = id % nown * P::OWN, part = id / nown % nparts, x1 = id / (nown * nparts);
  const int q0 = part * rq, q1 = min(nq, q0 + rq), nrow = 4 * (q1 - q0);   // x2 quads [q0, q1)
  const int nu = nrow * row;
  // the waves of one own band (tid, wave) and all of them
  const int lane = threadIdx.x & 63, nth = blockDim.x / P::OWN;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int band = P::OWN == 1 ? 0 : wave_all / (nth / 64), wave = wave_all - band * (nth / 64), tid = wave * 64 + lane;
  const int own = min(own0 + band, (COND ? ncs : nvs) - 1);
  double2* s_q = s_qs + band * K * K;
  double2* s_t = s_ts + band * P::ROWS * K;
  const int npart = COND ? nvs : ncs;
  const int j0 = wave * UQ;
  // this thread's line entries: offsets of (n2, n3) and (n2, -n3) in the lines, -1 outside
  int lp[NLD], lm[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int e = tid + nth * i;
    lp[i] = lm[i] = -1;
    if (e < K * (RC + 1)) {
      const int32_t* t = rowtab + 3 * (e / (RC + 1));
      const int n = e % (RC + 1);
      if (RC + n >= t[1] && RC + n <= t[2]) lp[i] = t[0] + RC + n;
      if (RC - n >= t[1] && RC - n <= t[2]) lm[i] = t[0] + RC - n;
    }
  }
  for (int i = threadIdx.x; i < (RC + 1) * nq; i += blockDim.x) s_f[i] = pts[i];
  double2 gp[NLD], gm[NLD];
  auto fetch = [&](int q, double2* u) {
    const size_t pair = COND ? (size_t)q * ncs + own : (size_t)own * ncs + q;
    const double2* src = qbar + (pair * nt + x1) * (size_t)nl;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      gp[i] = lp[i] >= 0 ? src[lp[i]] : double2{0.0, 0.0};
      gm[i] = lm[i] >= 0 ? src[lm[i]] : double2{0.0, 0.0};
    }
    const double2* up = partner + (((size_t)q * nt + x1) * nt + 4 * q0) * (size_t)row;
    for (int u0 = wave_all * 64; u0 < nu; u0 += blockDim.x)
      if (u0 + lane < nu)
        __builtin_amdgcn_global_load_lds((const void*)(up + u0 + lane),
                                         (__attribute__((address_space(3))) void*)(u + u0), 16, 0, 0);
  };
  double2 acc[UQ][4];
#pragma unroll
  for (int a = 0; a < UQ; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = double2{0.0, 0.0};
  auto mac = [](double2& a, double f, double2 x) {
    a.x = fma(f, x.x, a.x);
    a.y = fma(f, x.y, a.y);
  };
  auto one = [&](int q, const double2* u, double2* unext) {
    wait_vm<0>();
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int e = tid + nth * i;
      if (e < K * (RC + 1)) {
        const int n2 = e / (RC + 1), n = e % (RC + 1);
        const double2 x = conjd(gp[i]), y = conjd(gm[i]);
        s_q[n2 * K + n] = n == 0 ? x : cadd(x, y);
        if (n > 0) s_q[n2 * K + RC + n] = csub(x, y);
      }
    }
    lds_barrier();   // the lines are folded, the partner's rows have landed, its other buffer is free
    if (q + 1 < npart) fetch(q + 1, unext);
    // x2: the four rows of a quad for one slot
    for (int task = tid; task < K * (q1 - q0); task += nth) {
      const int sl = task % K, ql = task / K, j = q0 + ql;
      double2 y[1][4];
      points_of_quads<double2, 1>(
          RC, j == 0, [&](int n) { return s_q[(n + RC) * K + sl]; }, [&](int n, int) { return s_f[n * nq + j]; }, y);
#pragma unroll
      for (int a = 0; a < 4; ++a) s_t[(4 * ql + a) * K + sl] = y[0][a];
    }
    lds_barrier();
    // x3: this wave's quads of the lane's row, times the partner's values
    auto sums = [&](auto zero) {
      constexpr bool Z = decltype(zero)::value;   // quad 0 is among them
      const double2* tr = s_t + lane * K;
      double2 ae[UQ], ao[UQ], be[UQ], bo[UQ];
      const double2 t0 = tr[0];
#pragma unroll
      for (int a = 0; a < UQ; ++a) {
        ae[a] = t0;
        ao[a] = bo[a] = double2{0.0, 0.0};
        be[a] = Z && a == 0 ? t0 : double2{0.0, 0.0};
      }
#pragma unroll
      for (int n = 1; n <= RC; ++n) {
        const double2 e = tr[n], o = tr[RC + n];
#pragma unroll
        for (int a = 0; a < UQ; ++a) {
          const double2 f = pts[n * nq + min(j0 + a, nq - 1)];   // wave-uniform
          mac(n % 2 ? ao[a] : ae[a], f.x, e);
          mac(n % 2 ? bo[a] : be[a], f.y, n % 2 == 0 && Z && a == 0 ? e : o);
        }
      }
#pragma unroll
      for (int a = 0; a < UQ; ++a) {
        const double2 x = cadd(ae[a], ao[a]), y = csub(ae[a], ao[a]);
        double2 h[4];   // conj h
        if (Z && a == 0) {
          h[0] = x;
          h[1] = plus_i(be[a], bo[a]);
          h[2] = y;
          h[3] = minus_i(be[a], bo[a]);
        } else {
          const double2 sx = cadd(be[a], bo[a]), sy = csub(bo[a], be[a]);
          h[0] = plus_i(x, sx);
          h[1] = plus_i(y, sy);
          h[2] = minus_i(y, sy);
          h[3] = minus_i(x, sx);
        }
        const double2* v = u + lane * row + 4 * min(j0 + a, nq - 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (COND) {
            acc[a][c].x = fma(h[c].x, v[c].x, fma(h[c].y, v[c].y, acc[a][c].x));
            acc[a][c].y = fma(h[c].x, v[c].y, fma(-h[c].y, v[c].x, acc[a][c].y));
          } else {
            cmac(acc[a][c], h[c], v[c]);
          }
        }
      }
    };
    if (lane < nrow) {
      if (wave == 0)
        sums(std::true_type{});
      else
        sums(std::false_type{});
    }
  };
  fetch(0, s_u0);
  for (int q = 0; q < npart; q += 2) {
    one(q, s_u0, s_u1);
    if (q + 1 < npart) one(q + 1, s_u1, s_u0);
  }
  double2* out = ubar + (((size_t)own * nt + x1) * nt + 4 * q0 + lane) * (size_t)row;
  if (lane < nrow && own == own0 + band) {   // a repeated last band is not written
#pragma unroll
    for (int a = 0; a < UQ; ++a)
      if (j0 + a < nq) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          double2* o = out + 4 * (j0 + a) + c;
          *o = COND ? acc[a][c] : cadd(*o, acc[a][c]);
        }
      }
  }
}

constexpr int kJn = 4;   // frequencies |n| per thread of the transposed band passes: n and -n share the sums

// Frequencies +-n, n = n0 .. n0 + kJn - 1, of a line with the conjugate factors: the folded sums of fold.h,
// F(-n) of the forward transform.  load(p): point at position p of the quad order; s_p[n][j]: (cos, sin)(n j theta),
// quad 0 as fold.h.  out(k, plus, minus) for n = n0 + k.
template <typename Load, typename Out>
__device__ __forceinline__ void conj_freqs(int n0, int nmax, int nq, const double2* s_p, Load load, Out out) {
  double2 c[kJn], s[kJn];
#pragma unroll
  for (int k = 0; k < kJn; ++k) c[k] = s[k] = double2{0.0, 0.0};
  auto mac = [](double2& a, double f, double2 x) {
    a.x = fma(f, x.x, a.x);
    a.y = fma(f, x.y, a.y);
  };
  for (int j = 0; j < nq; ++j) {
    const double2 p[4] = {load(4 * j), load(4 * j + 1), load(4 * j + 2), load(4 * j + 3)};
    const Fold<double2> h = j == 0 ? fold_quad0(p) : fold_quad(p);
#pragma unroll
    for (int k = 0; k < kJn; ++k) {   // n0 is even: the parity of n is that of k
      const double2 f = s_p[min(n0 + k, nmax) * nq + j];
      mac(c[k], f.x, k % 2 == 0 ? h.ce : h.co);
      if (k % 2 == 0 && j == 0)
        mac(c[k], f.y, h.se);
      else
        mac(s[k], f.y, k % 2 == 0 ? h.se : h.so);
    }
  }
#pragma unroll
  for (int k = 0; k < kJn; ++k) out(k, minus_i(c[k], s[k]), plus_i(c[k], s[k]));
}

// transpose of the x1 pass: tB[slot][j1][p23] = sum_{x1} e^{-2 pi i n1 x1 / N} ubar[slot][x1][p23]; the planes are in
// natural x1 order
__global__ __launch_bounds__(256) void k_bandT_c(const double2* __restrict__ ubar, int rw, int nt, int row,
                                                 const double2* __restrict__ pts, double2* __restrict__ tB) {
  extern __shared__ __align__(16) unsigned char s_raw[];
  double2* s_p = (double2*)s_raw;   // (rw + 1) x nq
  const int nq = nt / 4, W = 2 * rw + 1;
  for (int i = threadIdx.x; i < (rw + 1) * nq; i += blockDim.x) s_p[i] = pts[i];
  __syncthreads();
  const size_t plane = (size_t)nt * row;
  const int slot = blockIdx.y, n0 = blockIdx.z * kJn;
  const int p23 = blockIdx.x * blockDim.x + threadIdx.x;
  if (p23 >= (int)plane) return;
  const double2* src = ubar + (size_t)slot * nt * plane + p23;
  double2* dst = tB + ((size_t)slot * W + rw) * plane + p23;
  conj_freqs(
      n0, rw, nq, s_p, [&](int p) { return src[(size_t)quad_x(p, nt) * plane]; },
      [&](int k, double2 a, double2 b) {
        const int n = n0 + k;
        if (n > rw) return;
        dst[(ptrdiff_t)n * (ptrdiff_t)plane] = a;
        if (n > 0) dst[-(ptrdiff_t)n * (ptrdiff_t)plane] = b;
      });
}

// transposes of the x2 and x3 passes for one (slot, j1) slab, then the sphere gather:
// cbar[slot][ig] for ig = wf_map[j1][j2][j3] >= 0.  ld: stride between the lines of s_t (odd where it fits); TL:
// the factors in LDS too.
template <bool TL>
__global__ __launch_bounds__(256) void k_bandT_ab(const double2* __restrict__ tB, int rw, int nt, int row, int ld,
                                                  const int32_t* __restrict__ wf_map, int npw,
                                                  const double2* __restrict__ pts, double2* __restrict__ cbar) {
  extern __shared__ __align__(16) unsigned char s_raw[];
  const int W = 2 * rw + 1, nq = nt / 4;
  double2* s_t = (double2*)s_raw;           // [j2][p3], W x ld
  double2* s_tab = s_t + (size_t)W * ld;    // (rw + 1) x nq
  const double2* s_p = TL ? s_tab : pts;
  const int nblk = (rw + kJn) / kJn;        // groups of |n|
  const int j1 = blockIdx.x;
  const int slot = blockIdx.y;
  if constexpr (TL) {
    for (int i = threadIdx.x; i < (rw + 1) * nq; i += blockDim.x) s_tab[i] = pts[i];
    __syncthreads();
  }
  const double2* slab = tB + ((size_t)slot * W + j1) * nt * row;
  // x2: s_t[j2][p3] = sum_{x2} e^{-2 pi i n2 x2 / N} slab[p2(x2)][p3]
  for (int task = threadIdx.x; task < nt * nblk; task += blockDim.x) {
    const int p3 = task % nt, n0 = task / nt * kJn;
    conj_freqs(
        n0, rw, nq, s_p, [&](int p) { return slab[(size_t)p * row + p3]; },
        [&](int k, double2 a, double2 b) {
          const int n = n0 + k;
          if (n > rw) return;
          s_t[(size_t)(rw + n) * ld + p3] = a;
          if (n > 0) s_t[(size_t)(rw - n) * ld + p3] = b;
        });
  }
  __syncthreads();
  // x3: cbar(j1, j2, j3) = sum_{x3} e^{-2 pi i n3 x3 / N} s_t[j2][p3(x3)]
  for (int task = threadIdx.x; task < W * nblk; task += blockDim.x) {
    const int j2 = task % W, n0 = task / W * kJn;
    const double2* line = s_t + (size_t)j2 * ld;
    const int32_t* map = wf_map + ((size_t)j1 * W + j2) * W + rw;   // index by n3
    auto put = [&](int n, double2 x) {
      const int ig = map[n];
      if (ig >= 0) cbar[(size_t)slot * npw + ig] = x;
    };
    conj_freqs(
        n0, rw, nq, s_p, [&](int p) { return line[p]; },
        [&](int k, double2 a, double2 b) {
          const int n = n0 + k;
          if (n > rw) return;
          put(n, a);
          if (n > 0) put(-n, b);
        });
  }
}

// grad[row(c)][g] += cbar[c][g] for the valid columns c < ncol of a chunk, row(c) =
// col_band[c0 + c] (or c0 + c); one thread per g walks the columns in order.
__global__ void k_scatter_cols(const double2* __restrict__ cbar, int ncol, const int32_t* __restrict__ col_band,
                               int c0, int npw, int nband, double2* __restrict__ grad) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= npw) return;
  for (int c = 0; c < ncol; ++c) {
    const int row = col_band ? col_band[c0 + c] : c0 + c;
    if (row < 0 || row >= nband) continue;   // an out-of-range column row is never written
    double2* d = grad + (size_t)row * npw + g;
    *d = cadd(*d, cbar[(size_t)c * npw + g]);
  }
}

__global__ void k_fill_c128(double2* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = double2{0.0, 0.0};
}

template <int RC>
hipError_t run_qbar(const Geom& g, const void* mbar, int npair, void* qbar, hipStream_t st) {
  const int threads = std::min(256, (g.nl + 63) / 64 * 64);
  k_qbar<RC><<<npair, threads, 0, st>>>((const double2*)mbar, g.d_chi_map, g.ngp, g.nt, g.nl,
                                        1.0 / ((double)g.nt * g.nt * g.nt), g.d_fac64, (double2*)qbar);
  return hipGetLastError();
}

// The plane's x2 quads in the fewest parts whose rows fit.
template <int RC, typename P>
hipError_t run_ubar_shape(const Geom& g, const void* qbar, const void* partner, int nvs, int ncs, bool cond, void* ubar,
                          hipStream_t st) {
  const int nq = g.nt / 4, row = g.row(true);
  int rq = nq;
  for (int n = 1; !P::fits(g.nt, row, rq); rq = (nq + n - 1) / n)
    if (++n > nq) return hipErrorInvalidValue;
  const int nparts = (nq + rq - 1) / rq;
  const int total = g.nt * nparts * (((cond ? ncs : nvs) + P::OWN - 1) / P::OWN);
  const auto f = cond ? k_ubar<RC, true, P> : k_ubar<RC, false, P>;
  f<<<(total + 7) / 8 * 8, 64 * P::OWN * ((nq + P::UQ - 1) / P::UQ), 0, st>>>((const double2*)qbar, (const double2*)partner, nvs,
                                                                     ncs, g.nt, g.nl, row, nparts, rq, g.d_rowtab,
                                                                     g.d_pts64, (double2*)ubar);
  return hipGetLastError();
}

template <int RC>
hipError_t run_ubar(const Geom& g, const void* qbar, const void* partner, int nvs, int ncs, bool cond, void* ubar,
                    hipStream_t st) {
  if constexpr (RC <= 7) {   // whole planes of up to 48 points
    if (UbarShape<RC, true, 2>::fits(g.nt, g.row(true), g.nt / 4))
      return run_ubar_shape<RC, UbarShape<RC, true, 2>>(g, qbar, partner, nvs, ncs, cond, ubar, st);
  }
  if (g.nt <= 64) return run_ubar_shape<RC, UbarShape<RC, false, 2>>(g, qbar, partner, nvs, ncs, cond, ubar, st);
  return run_ubar_shape<RC, UbarShape<RC, false, 4>>(g, qbar, partner, nvs, ncs, cond, ubar, st);
}

template <bool TL>
hipError_t allow_bandT_lds() {
  static OncePerDevice done;
  return allow_whole_lds(reinterpret_cast<const void*>(&k_bandT_ab<TL>), done);
}

}  // namespace

hipError_t launch_weight_rows(const void* m, int npair, int ngp, const double* w, int nparts, bool conj_w, void* a,
                              hipStream_t st) {
  const size_t n = (size_t)npair * ngp;
  k_weight_rows<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const double2*)m, npair, ngp, w, nparts, conj_w ? 1 : 0,
                                                             (double2*)a);
  return hipGetLastError();
}

hipError_t launch_qbar(const Geom& g, const void* mbar, int npair, void* qbar, hipStream_t st) {
  switch (g.rchi) {
#define X(rc) \
  case rc: return run_qbar<rc>(g, mbar, npair, qbar, st);
    GW_RC_CASES(X)
#undef X
  }
  return hipErrorInvalidValue;
}

hipError_t launch_ubar(const Geom& g, const void* qbar, const void* partner, int nvs, int ncs, bool cond, void* ubar,
                       hipStream_t st) {
  switch (g.rchi) {
#define X(rc) \
  case rc: return run_ubar<rc>(g, qbar, partner, nvs, ncs, cond, ubar, st);
    GW_RC_CASES(X)
#undef X
  }
  return hipErrorInvalidValue;
}

hipError_t launch_band_from_real(const Geom& g, const void* ubar, int nslot, void* tB, void* cbar, hipStream_t st) {
  const int nt = g.nt, W = g.W, row = g.row(true);
  constexpr int kUnits = 160 * 1024 / (int)sizeof(double2);
  if (nt > 128 || 128 + W * nt > kUnits) return hipErrorInvalidValue;
  const int tab = (g.rw + 1) * (nt / 4);
  const bool tl = W * (nt + 1) + tab <= kUnits;
  const int ld = W * (nt + 1) <= kUnits ? nt + 1 : nt;
  const hipError_t ea = tl ? allow_bandT_lds<true>() : allow_bandT_lds<false>();
  if (ea != hipSuccess) return ea;
  const unsigned groups = (unsigned)((g.rw + kJn) / kJn);
  k_bandT_c<<<dim3((nt * row + 255) / 256, nslot, groups), 256, tab * sizeof(double2), st>>>(
      (const double2*)ubar, g.rw, nt, row, g.d_pts64, (double2*)tB);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const auto f = tl ? k_bandT_ab<true> : k_bandT_ab<false>;
  f<<<dim3(W, nslot), 256, (W * ld + (tl ? tab : 0)) * sizeof(double2), st>>>(
      (const double2*)tB, g.rw, nt, row, ld, g.d_wf_map, g.npw, g.d_pts64, (double2*)cbar);
  return hipGetLastError();
}

hipError_t launch_scatter_cols(const void* cbar, int ncol, const int32_t* col_band, int c0, int npw, int nband,
                               void* grad, hipStream_t st) {
  k_scatter_cols<<<(npw + 255) / 256, 256, 0, st>>>((const double2*)cbar, ncol, col_band, c0, npw, nband,
                                                    (double2*)grad);
  return hipGetLastError();
}

hipError_t launch_fill_c128(void* p, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 65536);
  k_fill_c128<<<(unsigned)blocks, 256, 0, st>>>((double2*)p, n);
  return hipGetLastError();
}

}  // namespace gw
