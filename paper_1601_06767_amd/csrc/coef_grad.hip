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
//   k_bandT_*   transpose of the band transform (x1, then x2 and x3, sphere gather)
// Every inverse line transform of k_qbar and k_ubar uses the radix split of the forward
// kernels, conjugated: conj(sum_n conj(t_n) e^{+2 pi i n x / N}) = sum_n t_n e^{-2 pi i n x / N}.
#include <algorithm>

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

// Threads of a k_ubar workgroup and quads of a row that a thread sums at once.
constexpr int kUt = 256, kUq = 2;

// One workgroup per (x1 plane, part of its x2 quads, own band).  For every partner band: h of the
// pair on this plane from qbar (x2 transform into LDS, then x3 transform per (row, quads) task), times
// the partner's plane, accumulated in registers; the plane of ubar is written (COND) or
// added (valence, accumulated over conduction chunks) at the end.  TPT tasks per thread.
//   COND:  own = column c < ncs (pairs v * ncs + c, v < nvs), ubar_c += h_vc u_v
//   !COND: own = valence slot v < nvs (pairs v * ncs + c, c < ncs), ubar_v += conj(h_vc) u_c
// The inverse sums run on the conjugates (conj h), so that the factors are the forward ones.
template <int RC, int TPT, bool COND>
__global__ __launch_bounds__(kUt) void k_ubar(const double2* __restrict__ qbar, const double2* __restrict__ partner,
                                              int nvs, int ncs, int nt, int nl, int row, int nparts, int rq,
                                              const int32_t* __restrict__ rowtab, const double2* __restrict__ pts,
                                              double2* __restrict__ ubar) {
  constexpr int K = 2 * RC + 1;
  const int nq = nt / 4;
  extern __shared__ __align__(16) unsigned char s_raw[];
  double2* s_q = (double2*)s_raw;                 // [n2][n3] conj of the pair's lines, K x K
  double2* s_f = s_q + K * K;                     // [n][j] factors, (RC + 1) x nq
  double2* s_t = s_f + (RC + 1) * nq;             // [row of the part][n3], 4 rq x (K + 1)
  constexpr int KS = K + 1;                       // even: rows of n3 folded in place below
  const int x1 = blockIdx.x % nt;
  const int part = (blockIdx.x / nt) % nparts;
  const int own = blockIdx.x / (nt * nparts);
  const int q0 = part * rq;                       // x2 quads [q0, q1)
  const int q1 = min(nq, q0 + rq);
  const int nrow = 4 * (q1 - q0);
  const int ngq = (nq + kUq - 1) / kUq;           // x3 quad groups of a row
  const int ntask = nrow * ngq;
  const int tid = threadIdx.x;
  const int npart = COND ? nvs : ncs;
  for (int i = tid; i < K * K; i += kUt) s_q[i] = double2{0.0, 0.0};   // outside the lines: zero
  for (int i = tid; i < (RC + 1) * nq; i += kUt) s_f[i] = pts[i];
  double2 acc[TPT][kUq][4];
#pragma unroll
  for (int k = 0; k < TPT; ++k)
#pragma unroll
    for (int a = 0; a < kUq; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[k][a][c] = double2{0.0, 0.0};
#pragma unroll 1
  for (int q = 0; q < npart; ++q) {
    const size_t pair = COND ? (size_t)q * ncs + own : (size_t)own * ncs + q;
    const double2* src = qbar + (pair * nt + x1) * (size_t)nl;
    __syncthreads();   // the previous partner's s_q / s_t are consumed
    for (int i = tid; i < K * K; i += kUt) {
      const int j2 = i / K, j3 = i % K;
      const int32_t* e = rowtab + 3 * j2;
      if (j3 >= e[1] && j3 <= e[2]) s_q[i] = conjd(src[e[0] + j3]);
    }
    __syncthreads();
    // x2: the four rows of a quad for one n3
    for (int task = tid; task < K * (q1 - q0); task += kUt) {
      const int j3 = task % K, ql = task / K, j = q0 + ql;
      double2 y[1][4];
      points_of_quads<double2, 1>(
          RC, j == 0, [&](int n) { return s_q[(n + RC) * K + j3]; }, [&](int n, int) { return s_f[n * nq + j]; }, y);
#pragma unroll
      for (int a = 0; a < 4; ++a) s_t[(4 * ql + a) * KS + j3] = y[0][a];
    }
    __syncthreads();
    // x3: quads of a row, times the partner's values
    const double2* up = partner + ((size_t)q * nt + x1) * (size_t)nt * row;
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int task = tid + kUt * k;
      if (task < ntask) {
        const int rl = task % nrow, jq = task / nrow;
        const int j0 = min(jq * kUq, nq - kUq);
        double2 y[kUq][4];
        const double2* tr = s_t + rl * KS + RC;
        points_of_quads<double2, kUq>(
            RC, j0 == 0, [&](int n) { return tr[n]; }, [&](int n, int a) { return s_f[n * nq + j0 + a]; }, y);
        const double2* u = up + (size_t)(4 * q0 + rl) * row + 4 * j0;
#pragma unroll
        for (int a = 0; a < kUq; ++a)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double2 v = u[4 * a + c];
            // y = conj h
            acc[k][a][c] = COND ? cadd(acc[k][a][c], cmulc(y[a][c], v)) : cadd(acc[k][a][c], cmul(y[a][c], v));
          }
      }
    }
  }
  double2* out = ubar + ((size_t)own * nt + x1) * (size_t)nt * row;
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const int task = tid + kUt * k;
    if (task < ntask) {
      const int rl = task % nrow, jq = task / nrow;
      const int j0 = min(jq * kUq, nq - kUq);
      // an overlapping last group repeats the quads of its neighbour: written by the group that owns them
      double2* o = out + (size_t)(4 * q0 + rl) * row + 4 * j0;
#pragma unroll
      for (int a = 0; a < kUq; ++a)
        if (j0 + a >= jq * kUq) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (COND)
              o[4 * a + c] = acc[k][a][c];
            else
              o[4 * a + c] = cadd(o[4 * a + c], acc[k][a][c]);
          }
        }
    }
  }
}

constexpr int kJB = 8;   // outputs per thread of the transposed band passes

// transpose of the x1 pass: tB[slot][j1][p23] = sum_{x1} e^{-2 pi i n1 x1 / N} ubar[slot][x1][p23]
__global__ __launch_bounds__(256) void k_bandT_c(const double2* __restrict__ ubar, int rw, int nd, int row,
                                                 const double2* __restrict__ tw, double2* __restrict__ tB) {
  __shared__ double2 s_tw[128];
  for (int i = threadIdx.x; i < nd; i += blockDim.x) s_tw[i] = conjd(tw[i]);
  __syncthreads();
  const int W = 2 * rw + 1;
  const int nblk = (W + kJB - 1) / kJB;
  const size_t plane = (size_t)nd * row;
  const int slot = blockIdx.y;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)nblk * (long long)plane) return;
  const int p23 = (int)(t % (long long)plane);
  const int jb = (int)(t / (long long)plane);
  const double2* src = ubar + (size_t)slot * nd * plane + p23;
  double2 acc[kJB];
  int idx[kJB], step[kJB];
#pragma unroll
  for (int k = 0; k < kJB; ++k) {
    acc[k] = double2{0.0, 0.0};
    step[k] = wrap(jb * kJB + k - rw, nd);   // n1 mod N; x1 advances the twiddle index by n1
    idx[k] = 0;
  }
  for (int x1 = 0; x1 < nd; ++x1) {
    const double2 v = src[(size_t)x1 * plane];
#pragma unroll
    for (int k = 0; k < kJB; ++k) {
      cmac(acc[k], v, s_tw[idx[k]]);
      idx[k] += step[k];
      if (idx[k] >= nd) idx[k] -= nd;
    }
  }
  double2* dst = tB + (size_t)slot * W * plane + p23;
#pragma unroll
  for (int k = 0; k < kJB; ++k)
    if (jb * kJB + k < W) dst[(size_t)(jb * kJB + k) * plane] = acc[k];
}

// transposes of the x2 and x3 passes for one (slot, j1) slab, then the sphere gather:
// cbar[slot][ig] for ig = wf_map[j1][j2][j3] >= 0
__global__ __launch_bounds__(256) void k_bandT_ab(const double2* __restrict__ tB, int rw, int nd, int row,
                                                  const int32_t* __restrict__ wf_map, int npw,
                                                  const double2* __restrict__ tw, double2* __restrict__ cbar) {
  extern __shared__ __align__(16) unsigned char s_raw[];
  double2* s_tw = (double2*)s_raw;   // conj twiddles, nd
  double2* s_t = s_tw + 128;         // [j2][p3], W x nd
  const int W = 2 * rw + 1;
  const int nblk = (W + kJB - 1) / kJB;
  const int j1 = blockIdx.x;
  const int slot = blockIdx.y;
  for (int i = threadIdx.x; i < nd; i += blockDim.x) s_tw[i] = conjd(tw[i]);
  __syncthreads();
  const double2* slab = tB + ((size_t)slot * W + j1) * nd * row;
  // x2: s_t[j2][p3] = sum_{x2} e^{-2 pi i n2 x2 / N} slab[p2(x2)][p3]
  for (int task = threadIdx.x; task < nd * nblk; task += blockDim.x) {
    const int p3 = task % nd, jb = task / nd;
    double2 acc[kJB];
#pragma unroll
    for (int k = 0; k < kJB; ++k) acc[k] = double2{0.0, 0.0};
    for (int p2 = 0; p2 < nd; ++p2) {
      const int x2 = quad_x(p2, nd);
      const double2 v = slab[(size_t)p2 * row + p3];
#pragma unroll
      for (int k = 0; k < kJB; ++k) cmac(acc[k], v, s_tw[wrap((jb * kJB + k - rw) * x2, nd)]);
    }
#pragma unroll
    for (int k = 0; k < kJB; ++k)
      if (jb * kJB + k < W) s_t[(size_t)(jb * kJB + k) * nd + p3] = acc[k];
  }
  __syncthreads();
  // x3: cbar(j1, j2, j3) = sum_{x3} e^{-2 pi i n3 x3 / N} s_t[j2][p3(x3)]
  for (int task = threadIdx.x; task < W * nblk; task += blockDim.x) {
    const int j2 = task % W, jb = task / W;
    double2 acc[kJB];
#pragma unroll
    for (int k = 0; k < kJB; ++k) acc[k] = double2{0.0, 0.0};
    for (int p3 = 0; p3 < nd; ++p3) {
      const int x3 = quad_x(p3, nd);
      const double2 v = s_t[(size_t)j2 * nd + p3];
#pragma unroll
      for (int k = 0; k < kJB; ++k) cmac(acc[k], v, s_tw[wrap((jb * kJB + k - rw) * x3, nd)]);
    }
#pragma unroll
    for (int k = 0; k < kJB; ++k) {
      const int j3 = jb * kJB + k;
      if (j3 < W) {
        const int ig = wf_map[((size_t)j1 * W + j2) * W + j3];
        if (ig >= 0) cbar[(size_t)slot * npw + ig] = acc[k];
      }
    }
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

template <int RC, int TPT, bool COND>
hipError_t run_ubar_tpt(const Geom& g, const void* qbar, const void* partner, int nvs, int ncs, int nparts, int rq,
                        void* ubar, hipStream_t st) {
  constexpr int K = 2 * RC + 1;
  const size_t lds = ((size_t)K * K + (RC + 1) * (g.nt / 4) + (size_t)4 * rq * (K + 1)) * sizeof(double2);
  static const hipError_t allowed = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ubar<RC, TPT, COND>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (allowed != hipSuccess) return allowed;
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(g.nt * nparts * (COND ? ncs : nvs));
  k_ubar<RC, TPT, COND><<<grid, kUt, lds, st>>>((const double2*)qbar, (const double2*)partner, nvs, ncs, g.nt, g.nl,
                                                g.row(true), nparts, rq, g.d_rowtab, g.d_pts64, (double2*)ubar);
  return hipGetLastError();
}

// A thread holds kUq quads (8 complex accumulators) per task; the plane's x2 quads are split over
// parts so that a thread has at most two tasks.
template <int RC>
hipError_t run_ubar(const Geom& g, const void* qbar, const void* partner, int nvs, int ncs, bool cond, void* ubar,
                    hipStream_t st) {
  const int nq = g.nt / 4, ngq = (nq + kUq - 1) / kUq;
  const int rq_max = std::max(1, 2 * kUt / (4 * ngq));   // x2 quads whose tasks fit two per thread
  const int nparts = (nq + rq_max - 1) / rq_max;
  const int rq = (nq + nparts - 1) / nparts;
  const int ntask = 4 * rq * ngq;
  if (ntask > 2 * kUt) return hipErrorInvalidValue;
  if (ntask <= kUt)
    return cond ? run_ubar_tpt<RC, 1, true>(g, qbar, partner, nvs, ncs, nparts, rq, ubar, st)
                : run_ubar_tpt<RC, 1, false>(g, qbar, partner, nvs, ncs, nparts, rq, ubar, st);
  return cond ? run_ubar_tpt<RC, 2, true>(g, qbar, partner, nvs, ncs, nparts, rq, ubar, st)
              : run_ubar_tpt<RC, 2, false>(g, qbar, partner, nvs, ncs, nparts, rq, ubar, st);
}

hipError_t allow_bandT_lds() {
  static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bandT_ab),
                                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  return e;
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
  const int nd = g.nt, W = g.W, row = g.row(true);
  const size_t lds = (size_t)(128 + W * nd) * sizeof(double2);
  if (nd > 128 || lds > 160 * 1024) return hipErrorInvalidValue;
  const hipError_t ea = allow_bandT_lds();
  if (ea != hipSuccess) return ea;
  const int nblk = (W + kJB - 1) / kJB;
  const long long n = (long long)nblk * nd * row;
  k_bandT_c<<<dim3((unsigned)((n + 255) / 256), nslot), 256, 0, st>>>((const double2*)ubar, g.rw, nd, row, g.d_tw64,
                                                                       (double2*)tB);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_bandT_ab<<<dim3(W, nslot), 256, lds, st>>>((const double2*)tB, g.rw, nd, row, g.d_wf_map, g.npw, g.d_tw64,
                                                (double2*)cbar);
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
