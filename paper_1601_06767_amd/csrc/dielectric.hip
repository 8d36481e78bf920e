// Dielectric matrix eps = I - diag(v) chi0 and its inverse in float64 (the RPA relation
// stated before Eq. (chi0); Table 3's eps_inf = 1/[eps^-1]_00).
//
// Inversion: in-place Gauss-Jordan elimination with partial (row) pivoting, blocked by
// panels of kNb columns.  The panel columns (all rows) are copied to a buffer; one workgroup
// takes S of them at a time into registers and runs their S pivot steps there (k_gj_sub), and a
// launch over all rows brings the panel's other columns up to date (k_gj_apply); matrices with more
// rows than its registers hold take one launch per pivot step instead (k_gj_step16).  After the panel,
// its row interchanges are applied to the other columns, the panel holds the columns T[:, J] of
// the accumulated elimination transform, and the remaining columns are brought up to
// date with one rank-kNb update A[:, rest] += (T[:, J] - I[:, J]) A_old[J, rest] on
// float64 MFMA.  The column interchanges implied by the row pivots are undone at the
// end.  A zero or non-finite pivot raises a device flag read by gw_eps_inv_status.
// Several matrices of a batch run together (blockIdx.y), each in its own slice of the workspace.
//
// zgemm: C = alpha op(A) op(B) + beta C for complex128 row-major matrices, op = identity
// or conjugate transpose, on MFMA f64 16x16x4 with 64 x 64 tiles.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace gw {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// blockIdx.y: matrix of the batch; v, chi and out advance by one matrix, the workspace by ws bytes
template <typename T> __device__ __forceinline__ T* slice(T* p, size_t ws) {
  return (T*)((char*)p + (size_t)blockIdx.y * ws);
}

__global__ void k_form_eps(const double* __restrict__ v, const double2* __restrict__ chi, int n, size_t ws,
                           double2* __restrict__ eps) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  const double2 c = chi[(size_t)blockIdx.y * n * n + e];
  const double vi = v[(size_t)blockIdx.y * n + i];
  slice(eps, ws)[e] = double2{(i == j ? 1.0 : 0.0) - vi * c.x, -vi * c.y};
}

__global__ void k_flag_clear(int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 0;
}

constexpr int kStepRows = 4;   // rows per workgroup of the panel kernels (one kNb-wide row per wave)

// Panel columns [j0, j0 + nbp) of a into p (n x kNb, zero padded).
__global__ __launch_bounds__(256) void k_panel_load(const double2* __restrict__ a, int n, int j0, int nbp, size_t ws,
                                                    double2* __restrict__ p) {
  const int i = blockIdx.x * kStepRows + (threadIdx.x >> 6);
  const int c = threadIdx.x & 63;
  if (i < n) slice(p, ws)[(size_t)i * kNb + c] = c < nbp ? slice(a, ws)[(size_t)i * n + j0 + c] : double2{0.0, 0.0};
}

// Largest of a wave's values, in every lane (data-parallel-primitive moves: no LDS).
__device__ __forceinline__ unsigned wave_max(unsigned k) {
  auto step = [](unsigned x, auto ctrl, auto rows) {
    const unsigned y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    return x > y ? x : y;
  };
  using std::integral_constant;
  k = step(k, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr 1, 2, 4, 8
  k = step(k, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  k = step(k, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  k = step(k, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  k = step(k, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast 15, 31
  k = step(k, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
  return (unsigned)__builtin_amdgcn_readlane((int)k, 63);
}

// 1 / d for d > 0 whose 1 / d is finite: the hardware estimate and two Newton steps
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}

// The S pivot steps of the panel columns [c0, c0 + sc), sc <= S, in one workgroup: each thread holds R
// rows of the S columns in registers.  Per step: the pivot as the largest |x|^2 of the rows from
// j on (the lower row on ties), its row and row j through LDS, then row j <- row p / d, row p <- row j (old) eliminated, every other
// row eliminated, column <- the corresponding column of the transform.  Register column 0 is the
// step's pivot column and every step rotates the columns by one: the loop stays rolled (unrolled, a
// launch spent its time on instruction fetch, 18 us per step).  Serial: two barriers and a
// reduction per step.
constexpr int kGjThreads = 512;
constexpr int kGjMaxRows = 2048;   // rows the registers hold
// A row and its |x|^2 as two words, the upper one raised by one: 0 for no row.  The largest is found by the
// upper words; only where lanes or waves tie there do the lower words and the row numbers decide (4 x 1114:
// 5.8 ms; 6.4 with every step over the whole value, 5.6 with a single word of 21 bits and the row, which
// lost the pivots whose squares are subnormal).
struct GjCandidate {
  unsigned hi, lo;
  int row, pad;
};
// the lane of the largest candidate among those of mask; top: its upper word
__device__ __forceinline__ int gj_winner(const GjCandidate& k, unsigned top, unsigned long long mask) {
  unsigned long long m = __ballot(k.hi == top) & mask;
  if ((m & (m - 1)) != 0) {
    const unsigned lo = wave_max(k.hi == top ? k.lo : 0u);
    const bool tie = k.hi == top && k.lo == lo;
    const unsigned last = wave_max(tie ? (unsigned)(kGjMaxRows - k.row) : 0u);   // the lowest row
    m = __ballot(tie && (unsigned)(kGjMaxRows - k.row) == last) & mask;
  }
  return __builtin_ctzll(m);
}
template <int R, int S>
__global__ __launch_bounds__(kGjThreads) void k_gj_sub(const double2* __restrict__ pin, int n, int j0, int c0, int sc,
                                                       size_t ws, double2* __restrict__ tout, int* __restrict__ piv,
                                                       int* __restrict__ flag) {
  static_assert(R * kGjThreads <= kGjMaxRows, "rows of the pivot steps");
  constexpr int NW = kGjThreads / 64;
  static_assert(NW == 8, "a candidate per wave, read by lane mod 8");
  __shared__ __align__(16) GjCandidate s_best[2][NW];
  __shared__ double2 s_prow[2][S], s_rowj[2][S];
  pin = slice(pin, ws);
  tout = slice(tout, ws);
  piv = slice(piv, ws);
  const int tid = threadIdx.x;
  double2 x[R][S];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = tid + kGjThreads * r;
#pragma unroll
    for (int c = 0; c < S; ++c)
      x[r][c] = i < n && c < sc ? pin[(size_t)i * kNb + c0 + c] : double2{0.0, 0.0};
  }
#pragma unroll 1
  for (int jc = 0; jc < sc; ++jc) {
    const int j = j0 + c0 + jc, b = jc & 1;
    double best = -1.0;   // no comparison holds for a NaN
    int row = kGjMaxRows;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = tid + kGjThreads * r;
      const double m = x[r][0].x * x[r][0].x + x[r][0].y * x[r][0].y;
      if (i >= j && i < n && m > best) {
        best = m;
        row = i;
      }
    }
    const unsigned long long bits = (unsigned long long)__double_as_longlong(best);
    GjCandidate k{row < kGjMaxRows ? (unsigned)(bits >> 32) + 1 : 0u, (unsigned)bits, row, 0};
    const unsigned most = wave_max(k.hi);
    if ((tid & 63) == (most != 0 ? gj_winner(k, most, ~0ull) : 0)) s_best[b][tid >> 6] = k;
    __syncthreads();
    k = s_best[b][tid & 7];
    unsigned top = k.hi;   // of the eight waves, in every lane
    top = max(top, (unsigned)__builtin_amdgcn_update_dpp(0, (int)top, 0xb1, 0xf, 0xf, false));    // lane ^ 1
    top = max(top, (unsigned)__builtin_amdgcn_update_dpp(0, (int)top, 0x4e, 0xf, 0xf, false));    // lane ^ 2
    top = max(top, (unsigned)__builtin_amdgcn_update_dpp(0, (int)top, 0x141, 0xf, 0xf, false));   // 7 - lane
    const int win = __builtin_amdgcn_readlane(k.row, gj_winner(k, top, (1ull << NW) - 1));
    const int p = win < n ? win : j;   // no finite candidate: row j, the flag reports it
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = tid + kGjThreads * r;
      if (i == p) {
#pragma unroll
        for (int c = 0; c < S; ++c) s_prow[b][c] = x[r][c];
      }
      if (i == j) {
#pragma unroll
        for (int c = 0; c < S; ++c) s_rowj[b][c] = x[r][c];
      }
    }
    __syncthreads();
    const double2 d = s_prow[b][0];
    const double den = d.x * d.x + d.y * d.y;
    if (tid == 0) {
      piv[j] = p;
      if (!(den > 0.0) || !isfinite(den)) *flag = 1;
    }
    double2 dinv{0.0, 0.0};
    if (den >= 0x1p-1021 && den <= 0x1p1021) {   // 1 / den normal too
      const double rden = recip(den);
      dinv = double2{d.x * rden, -d.y * rden};
    } else if (den > 0.0) {
      dinv = double2{d.x / den, -d.y / den};
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = tid + kGjThreads * r;
      if (i == p) {   // (p == j: row j itself, replaced below)
#pragma unroll
        for (int c = 0; c < S; ++c) x[r][c] = s_rowj[b][c];
      }
      // every row but j: x - f q; row j: q / d = 0 - (-1/d) q
      const bool isj = i == j;
      double2 f = cmul(x[r][0], dinv);
      if (isj) f = double2{-dinv.x, -dinv.y};
#pragma unroll
      for (int c = 0; c + 1 < S; ++c) {
        const double2 q = s_prow[b][c + 1];
        double2 y = x[r][c + 1];
        if (isj) y = double2{0.0, 0.0};
        x[r][c].x = fma(f.y, q.y, fma(-f.x, q.x, y.x));
        x[r][c].y = fma(-f.y, q.x, fma(-f.x, q.y, y.y));
      }
      x[r][S - 1] = double2{-f.x, -f.y};
    }
    // the LDS rows and candidates alternate between two sets: a wave that runs ahead into the next step
    // writes the other one
  }
  // after sc rotations register column c is panel column (sc + c) mod S
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = tid + kGjThreads * r;
    if (i < n) {
#pragma unroll
      for (int c = 0; c < S; ++c) {
        const int k = sc + c;
        tout[(size_t)i * S + (k >= S ? k - S : k)] = x[r][c];
      }
    }
  }
}

// Larger matrices: one launch per pivot step on a sub-panel of kGjSub columns (t buffers, n x kGjSub),
// all rows over the chip; the launch also leaves one pivot candidate (largest |x|^2, its row; the
// lower row on ties) per workgroup for the next step's column.
constexpr int kGjSub = 16;      // widest sub-panel
constexpr int kGjRows = 16;     // rows per workgroup of these launches (16 columns each)
__device__ __forceinline__ void gj_candidate(double m, int i, double* cm, int* ci) {
  // the 16 rows of the workgroup: thread 16 r holds row r's value
  __shared__ double s_m[kGjRows];
  __shared__ int s_i[kGjRows];
  const int r = threadIdx.x >> 4;
  if ((threadIdx.x & 15) == 0) {
    s_m[r] = m;
    s_i[r] = i;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double best = -1.0;
    int bi = 0x7fffffff;
    for (int k = 0; k < kGjRows; ++k)
      if (s_m[k] > best || (s_m[k] == best && s_i[k] < bi)) {
        best = s_m[k];
        bi = s_i[k];
      }
    cm[blockIdx.x] = best;
    ci[blockIdx.x] = bi;
  }
}

__global__ __launch_bounds__(256) void k_gj_load16(const double2* __restrict__ pin, int n, int j0, int c0, int sc,
                                                   size_t ws, double2* __restrict__ t, double* __restrict__ cm,
                                                   int* __restrict__ ci) {
  pin = slice(pin, ws);
  t = slice(t, ws);
  const int i = blockIdx.x * kGjRows + (threadIdx.x >> 4), c = threadIdx.x & 15;
  double2 x{0.0, 0.0};
  if (i < n && c < sc) x = pin[(size_t)i * kNb + c0 + c];
  if (i < n) t[(size_t)i * kGjSub + c] = x;
  gj_candidate(i < n && i >= j0 + c0 ? x.x * x.x + x.y * x.y : -1.0, i, slice(cm, ws), slice(ci, ws));
}

__global__ __launch_bounds__(256) void k_gj_step16(const double2* __restrict__ tin, double2* __restrict__ tout, int n,
                                                   int j, int jc, int ncand, size_t ws, const double* __restrict__ cm_in,
                                                   const int* __restrict__ ci_in, double* __restrict__ cm_out,
                                                   int* __restrict__ ci_out, int* __restrict__ piv,
                                                   int* __restrict__ flag) {
  __shared__ double s_m[4];
  __shared__ int s_i[4];
  tin = slice(tin, ws);
  tout = slice(tout, ws);
  cm_in = slice(cm_in, ws);
  ci_in = slice(ci_in, ws);
  const int tid = threadIdx.x, i = blockIdx.x * kGjRows + (tid >> 4), c = tid & 15;
  double2 x{0.0, 0.0};
  if (i < n) x = tin[(size_t)i * kGjSub + c];
  double best = -1.0;
  int bi = 0x7fffffff;
  auto take = [&](double m, int k) {
    if (m > best || (m == best && k < bi)) {
      best = m;
      bi = k;
    }
  };
  for (int k = tid; k < ncand; k += 256) take(cm_in[k], ci_in[k]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double m = __shfl_xor(best, o, 64);
    const int k = __shfl_xor(bi, o, 64);
    take(m, k);
  }
  if ((tid & 63) == 0) {
    s_m[tid >> 6] = best;
    s_i[tid >> 6] = bi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) take(s_m[w], s_i[w]);
  const int p = best >= 0.0 && bi < n ? bi : j;   // no finite candidate: keep row j, the flag reports it
  if (blockIdx.x == 0 && tid == 0) {
    slice(piv, ws)[j] = p;
    if (!(best > 0.0) || !isfinite(best)) *flag = 1;
  }
  const double2 d = tin[(size_t)p * kGjSub + jc], q = tin[(size_t)p * kGjSub + c];
  const double den = d.x * d.x + d.y * d.y;
  const double2 dinv = den > 0.0 ? double2{d.x / den, -d.y / den} : double2{0.0, 0.0};
  double2 out{0.0, 0.0};
  if (i < n) {
    if (i == j) {
      out = c == jc ? dinv : cmul(q, dinv);
    } else {
      const int src = i == p ? j : i;
      if (i == p) x = tin[(size_t)j * kGjSub + c];
      const double2 f = cmul(tin[(size_t)src * kGjSub + jc], dinv);
      const double2 r = cmul(f, q);
      out = c == jc ? double2{-f.x, -f.y} : double2{x.x - r.x, x.y - r.y};
    }
    tout[(size_t)i * kGjSub + c] = out;
  }
  // candidate of the next column: its value sits in lane jc + 1 of the row's 16
  const double m = out.x * out.x + out.y * out.y;
  const double mn = __shfl(m, ((tid & 63) & ~15) + min(jc + 1, 15), 64);
  gj_candidate(i < n && i > j ? mn : -1.0, i, slice(cm_out, ws), slice(ci_out, ws));
}

// The panel's other columns after S pivot steps (columns [c0, c0 + sc), rows J = j0 + c0 ..): with the
// steps' row interchanges, out[i][c] = in[src(i)][c] + sum_k (T - I)[i][k] in[src(J_k)][c], and T itself
// in the columns c0 ...  Reads pin, writes pout.
template <int S>
__global__ __launch_bounds__(256) void k_gj_apply(const double2* __restrict__ pin, double2* __restrict__ pout, int n,
                                                  int j0, int c0, int sc, size_t ws, const double2* __restrict__ t,
                                                  const int* __restrict__ piv) {
  __shared__ double2 s_row[S][kNb];
  pin = slice(pin, ws);
  pout = slice(pout, ws);
  t = slice(t, ws);
  piv = slice(piv, ws);
  const int jb = j0 + c0;
  int pv[S];
#pragma unroll
  for (int k = 0; k < S; ++k) pv[k] = k < sc ? piv[jb + k] : jb + k;
  auto source = [&](int i) {   // the row whose old content ends up in row i
#pragma unroll
    for (int k = S - 1; k >= 0; --k) {
      const int a = jb + k;
      i = i == a ? pv[k] : (i == pv[k] ? a : i);
    }
    return i;
  };
  const int wave = threadIdx.x >> 6, c = threadIdx.x & 63;
  for (int k = wave; k < sc; k += 4) s_row[k][c] = pin[(size_t)source(jb + k) * kNb + c];
  __syncthreads();
  const int i = blockIdx.x * kStepRows + wave;
  if (i >= n) return;
  double2 out;
  if (c >= c0 && c < c0 + sc) {
    out = t[(size_t)i * S + c - c0];
  } else {
    out = pin[(size_t)source(i) * kNb + c];
    for (int k = 0; k < sc; ++k) {
      double2 f = t[(size_t)i * S + k];
      if (i == jb + k) f.x -= 1.0;
      const double2 q = s_row[k][c];
      out.x = fma(-f.y, q.y, fma(f.x, q.x, out.x));
      out.y = fma(f.y, q.x, fma(f.x, q.y, out.y));
    }
  }
  pout[(size_t)i * kNb + c] = out;
}

// The panel's row interchanges, in order, on the columns outside the panel.
__global__ void k_row_swaps(double2* __restrict__ a, int n, int j0, int nbp, size_t ws, const int* __restrict__ piv) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n || (c >= j0 && c < j0 + nbp)) return;
  a = slice(a, ws);
  piv = slice(piv, ws);
  for (int j = j0; j < j0 + nbp; ++j) {
    const int p = piv[j];
    if (p != j && p >= 0 && p < n) {
      const double2 x = a[(size_t)j * n + c];
      a[(size_t)j * n + c] = a[(size_t)p * n + c];
      a[(size_t)p * n + c] = x;
    }
  }
}

// The finished panel T[:, J] back into a, and the operands of the rank-nbp update, 64 values per row:
// bp = T[:, J] - I[:, J] (in place in the panel buffer), tmp[col] = conj(A[J, col]), zero for the panel's
// own columns.
__global__ void k_panel_operands(double2* __restrict__ a, int n, int j0, int nbp, size_t ws, double2* __restrict__ bp,
                                 double2* __restrict__ tmp) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  a = slice(a, ws);
  bp = slice(bp, ws);
  tmp = slice(tmp, ws);
  if (e < (size_t)n * kNb) {
    const int i = (int)(e / kNb), c = (int)(e % kNb);
    double2 x{0.0, 0.0};
    if (c < nbp) {
      x = bp[e];
      a[(size_t)i * n + j0 + c] = x;
      if (i == j0 + c) x.x -= 1.0;
    }
    bp[e] = x;
  }
  // 8 columns by 8 rows of J per 64 threads: reads of whole 128-byte pieces of a row
  const int n8 = (n + 7) / 8;
  if (e < (size_t)n8 * 8 * kNb) {
    const int g = (int)(e / 64), l = (int)(e % 64);
    const int col = (g % n8) * 8 + (l & 7), c = (g / n8) * 8 + (l >> 3);
    if (col < n) {
      double2 x{0.0, 0.0};
      if (c < nbp && (col < j0 || col >= j0 + nbp)) {
        x = a[(size_t)(j0 + c) * n + col];
        x.y = -x.y;
      }
      tmp[(size_t)col * kNb + c] = x;
    }
  }
}

// out[:, c] = src[:, idx(c)], idx the columns after undoing the interchanges: idx(c) follows position c
// through the swaps (j, piv[j]), first to last.
__global__ __launch_bounds__(256) void k_col_perm(const int* __restrict__ piv, int n, size_t ws, int* __restrict__ idx) {
  __shared__ int s_p[1024];
  piv = slice(piv, ws);
  idx = slice(idx, ws);
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  int x = c;
  for (int b = 0; b < n; b += 1024) {
    const int m = min(1024, n - b);
    __syncthreads();
    for (int k = threadIdx.x; k < m; k += blockDim.x) s_p[k] = piv[b + k];
    __syncthreads();
    for (int k = 0; k < m; ++k) {
      const int p = s_p[k], j = b + k;
      x = x == j ? p : (x == p ? j : x);
    }
  }
  if (c < n) idx[c] = x;
}

__global__ void k_gather_cols(const double2* __restrict__ src, const int* __restrict__ idx, int n, size_t ws,
                              double2* __restrict__ dst) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const size_t i = e / n;
  const int c = (int)(e % n);
  dst[(size_t)blockIdx.y * n * n + e] = slice(src, ws)[i * n + slice(idx, ws)[c]];
}

// ---------------------------------------------------------------- zgemm
constexpr int ZT = 64, ZK = 16;

// element (r, k) of op(X) for X row-major with leading dimension ld; op: kOpN, kOpC
// (conjugate transpose), kOpT (transpose), kOpConj (conjugate)
__device__ __forceinline__ double2 opget(const double2* x, int ld, int r, int k, int op) {
  const bool tr = op == kOpC || op == kOpT;
  const double2 v = tr ? x[(size_t)k * ld + r] : x[(size_t)r * ld + k];
  return (op == kOpC || op == kOpConj) ? double2{v.x, -v.y} : v;
}

__global__ __launch_bounds__(256) void k_zgemm(int m, int n, int kd, double2 alpha, const double2* __restrict__ A,
                                               int lda, int opa, const double2* __restrict__ B, int ldb, int opb,
                                               double2 beta, double2* __restrict__ C, int ldc) {
  __shared__ double2 sA[ZK][ZT + 1];   // sA[k][row]
  __shared__ double2 sB[ZK][ZT + 1];   // sB[k][col]
  const int tiles_n = (n + ZT - 1) / ZT;
  const int r0 = (blockIdx.x / tiles_n) * ZT, c0 = (blockIdx.x % tiles_n) * ZT;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = wave >> 1, wc = wave & 1, li = lane & 15, lk = lane >> 4;
  f64x4 cre[2][2], cim[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      cre[i][j] = f64x4{0, 0, 0, 0};
      cim[i][j] = f64x4{0, 0, 0, 0};
    }
  for (int k0 = 0; k0 < kd; k0 += ZK) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (ZK * ZT) / 256; ++r) {
      const int e = tid + 256 * r;
      // consecutive threads walk the operand's contiguous index: k for A stored by rows (N,
      // conj) and for B stored transposed (T, C), the row / column index otherwise
      {
        const bool along_k = opa == kOpN || opa == kOpConj;
        const int kk = along_k ? e % ZK : e / ZT, rr = along_k ? e / ZK : e % ZT;
        double2 x{0.0, 0.0};
        if (r0 + rr < m && k0 + kk < kd) x = opget(A, lda, r0 + rr, k0 + kk, opa);
        sA[kk][rr] = x;
      }
      {
        const bool along_k = opb == kOpT || opb == kOpC;
        const int kk = along_k ? e % ZK : e / ZT, cc = along_k ? e / ZK : e % ZT;
        double2 x{0.0, 0.0};
        if (c0 + cc < n && k0 + kk < kd) x = opget(B, ldb, k0 + kk, c0 + cc, opb);
        sB[kk][cc] = x;
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < ZK / 4; ++s) {
      const int k = 4 * s + lk;
      double2 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = sA[k][32 * wr + 16 * i + li];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sB[k][32 * wc + 16 * j + li];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          cre[i][j] = mfma64(a[i].x, b[j].x, cre[i][j]);
          cre[i][j] = mfma64(-a[i].y, b[j].y, cre[i][j]);
          cim[i][j] = mfma64(a[i].x, b[j].y, cim[i][j]);
          cim[i][j] = mfma64(a[i].y, b[j].x, cim[i][j]);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + 32 * wr + 16 * i + lk + 4 * r;   // f64 MFMA output rows: lane/16 + 4 r
        const int col = c0 + 32 * wc + 16 * j + li;
        if (row < m && col < n) {
          const double2 ab{cre[i][j][r], cim[i][j][r]};
          double2 out = cmul(alpha, ab);
          double2* p = C + (size_t)row * ldc + col;
          if (beta.x != 0.0 || beta.y != 0.0) {
            const double2 o = cmul(beta, *p);
            out.x += o.x;
            out.y += o.y;
          }
          *p = out;
        }
      }
}

// The same for A by rows, n a multiple of 64, k of 16 and beta = 0, alpha = 1 (the products with pair
// densities, padded with zeros): both operands by direct loads into two buffers, the next 16 k under the
// current ones' MFMAs, one barrier per 16 k.  Rows [row][k] are swizzled (unit k ^ row mod 16) so that the 16
// rows of a fragment read different banks.  Tiles in bands of eight row tiles, a contiguous run per XCD.
// Bound by float64 MFMA: 16k x 2048 x 2000 in 8.0 ms (the general kernel 10.1; 7.3 at the rate of a large
// product).
template <bool CA, bool BT>   // A conjugated (kOpConj); B by rows of its transpose (kOpT), or by rows (kOpN)
__global__ __launch_bounds__(256, 2) void k_zgemm_rows(int m, int n, int kd, const double2* __restrict__ A, int lda,
                                                       const double2* __restrict__ B, int ldb, double2* __restrict__ C,
                                                       int ldc) {
  constexpr int U = ZT * ZK;   // 16-byte units of an operand's stage
  __shared__ __align__(16) double2 sA0[U], sB0[U], sA1[U], sB1[U];
  const int ntr = (m + ZT - 1) / ZT, ntc = n / ZT, nt = ntr * ntc;
  const int t = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
  if (t >= nt) return;
  const int band = t / (8 * ntc), in = t % (8 * ntc), wide = min(8, ntr - 8 * band);
  const int r0 = (8 * band + in % wide) * ZT, c0 = in / wide * ZT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1, li = lane & 15, lk = lane >> 4;
  // wave instruction i of an operand: rows 4 i .. 4 i + 3, 16 k each (B by rows: k = i, 64 columns)
  size_t offA[4], offB[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 4 * (4 * j + wave) + (lane >> 4), k = (lane & 15) ^ (row & 15);
    offA[j] = (size_t)min(r0 + row, m - 1) * lda + k;
    offB[j] = BT ? (size_t)(c0 + row) * ldb + k : (size_t)(4 * j + wave) * ldb + c0 + lane;
  }
  auto issue = [&](int k0, double2* a, double2* b) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      __builtin_amdgcn_global_load_lds((const void*)(A + offA[j] + k0),
                                       (__attribute__((address_space(3))) void*)(a + 64 * (4 * j + wave)), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)(B + offB[j] + (BT ? (size_t)k0 : (size_t)k0 * ldb)),
                                       (__attribute__((address_space(3))) void*)(b + 64 * (4 * j + wave)), 16, 0, 0);
    }
  };
  f64x4 cre[2][2], cim[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      cre[i][j] = f64x4{0, 0, 0, 0};
      cim[i][j] = f64x4{0, 0, 0, 0};
    }
  auto stage = [&](int k0, const double2* a, const double2* b, double2* an, double2* bn) {
    wait_vm<0>();
    lds_barrier();   // the stage has landed; the other buffers are no longer read
    if (k0 + ZK < kd) issue(k0 + ZK, an, bn);
#pragma unroll
    for (int s = 0; s < ZK / 4; ++s) {
      const int k = 4 * s + lk;
      double2 x[2], y[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = a[(32 * wr + 16 * i + li) * ZK + (k ^ li)];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = 32 * wc + 16 * j + li;
        y[j] = BT ? b[col * ZK + (k ^ li)] : b[k * ZT + col];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          cre[i][j] = mfma64(x[i].x, y[j].x, cre[i][j]);
          cim[i][j] = mfma64(x[i].x, y[j].y, cim[i][j]);
          cre[i][j] = mfma64(CA ? x[i].y : -x[i].y, y[j].y, cre[i][j]);
          cim[i][j] = mfma64(CA ? -x[i].y : x[i].y, y[j].x, cim[i][j]);
        }
    }
  };
  issue(0, sA0, sB0);
  int k0 = 0;
  for (; k0 + 2 * ZK <= kd; k0 += 2 * ZK) {
    stage(k0, sA0, sB0, sA1, sB1);
    stage(k0 + ZK, sA1, sB1, sA0, sB0);
  }
  if (k0 < kd) stage(k0, sA0, sB0, sA1, sB1);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = r0 + 32 * wr + 16 * i + lk + 4 * r;
      if (row < m)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          C[(size_t)row * ldc + c0 + 32 * wc + 16 * j + li] = double2{cre[i][j][r], cim[i][j][r]};
    }
}

// ---------------------------------------------------------------- static inverse by block sweeps
// For a static chi0 (Hermitian, negative semidefinite) and v > 0, eps~ = I - V^1/2 chi0 V^1/2 is
// Hermitian positive definite and eps^-1 = V^1/2 eps~^-1 V^-1/2.  The sweep operator on a block K
// of 64 indices, D = A_KK, X = A_.K, P = X D^-1:
//   A_ij -= P_i X_j^H (i, j outside K),  A_iK <- P_i,  A_Kj <- P_j^H,  A_KK <- -D^-1;
// sweeping every block in turn leaves -A^-1.  The part not yet swept is a Schur complement of
// eps~, positive definite, so D needs no pivoting.  Only the lower triangle is stored: half the
// arithmetic of the pivoted Gauss-Jordan path and three launches per block of 64 (D^-1 in one
// workgroup, P, the rank-64 update of the lower tiles).
constexpr int kSw = 64;

// lower triangle a[i][j] = delta_ij - sqrt(v_i) chi_ij sqrt(v_j) (i >= j), identity in the padding
__global__ void k_sweep_form(const double* __restrict__ v, const double2* __restrict__ chi, int n, int ldp, size_t ws,
                             double2* __restrict__ a, int* __restrict__ flag) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)ldp * ldp) return;
  v += (size_t)blockIdx.y * n;
  chi += (size_t)blockIdx.y * n * n;
  a = slice(a, ws);
  const int i = (int)(e / ldp), j = (int)(e % ldp);
  if (j > i) return;
  double2 x{i == j ? 1.0 : 0.0, 0.0};
  if (i < n && j < n) {
    const double vi = v[i], vj = v[j];
    double s = 0.0;   // a v <= 0 is reported; the entry is then left at the identity's
    if (!(vi > 0.0) || !(vj > 0.0))
      atomicOr(flag, 1);
    else
      s = sqrt(vi) * sqrt(vj);
    const double2 c = chi[(size_t)i * n + j];
    x.x -= s * c.x;
    x.y -= s * c.y;
  }
  a[e] = x;
}

// D^-1 of a 64 x 64 Hermitian pivot block by 64 Gauss-Jordan steps, a thread of 256 holding a 4 x 4
// piece [p][q] of rows ty + 16 p and columns tx + 16 q in registers.  Step j sweeps index j:
// A_jj <- -1/d, A_ij <- A_ij / d, A_ji <- conj(A_ij) / d, A_ik -= A_ij conj(A_kj) / d, Hermitian throughout,
// so it needs column j only, which its owners leave in LDS for the next step: one barrier, eight LDS
// reads and 64 FMAs per step.  The next step's column is brought up to date, stored and read back before the
// rest of the piece, whose FMAs run under the reads (NG 2000 in all: 2.07 ms, 2.12 with them before the
// store).  Row and column j come out of the same update with the factors -1/d for A_jj / d and -1 for A_jj,
// from zeroed entries.  A pivot that is not positive sets the flag.  (A Cholesky factor, its inverse and
// their product, all in LDS, took 126 us per block.)
__device__ __forceinline__ void diag_inverse(double (&xr)[4][4], double (&xi)[4][4], double2 (*s_col)[kSw],
                                             double2* __restrict__ dinv, int* __restrict__ flag) {
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  if (tx == 0) {
#pragma unroll
    for (int p = 0; p < 4; ++p) s_col[0][ty + 16 * p] = double2{xr[p][0], xi[p][0]};
  }
  __syncthreads();
  double d;
  double2 y[4], z[4];   // the step's pivot and the column's entries of this thread's rows and columns
  auto load = [&](int j) {
    const double2* col = s_col[j & 1];
    d = col[j].x;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      y[p] = col[ty + 16 * p];
      z[p] = col[tx + 16 * p];
    }
  };
  // step j = 16 jb + jt; the next step's column sits in piece nb
  auto step = [&](auto jbc, auto nbc, int jt) {
    constexpr int jb = decltype(jbc)::value, nb = decltype(nbc)::value;
    const int j = 16 * jb + jt;
    const bool bad = !(d > 0.0) || !isfinite(d);
    if (bad) d = 1.0;
    if (bad && tid == 0) atomicOr(flag, 1);
    const double rd = recip(d);
    const bool rj = ty == jt, cj = tx == jt;   // this thread's row / column piece jb is row / column j
    double fr[4], fi[4], cr[4], ci[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      fr[p] = y[p].x * rd;
      fi[p] = y[p].y * rd;
      cr[p] = z[p].x;
      ci[p] = z[p].y;
    }
    fr[jb] = rj ? -rd : fr[jb];
    fi[jb] = rj ? 0.0 : fi[jb];
    cr[jb] = cj ? -1.0 : cr[jb];
    ci[jb] = cj ? 0.0 : ci[jb];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      xr[jb][p] = rj ? 0.0 : xr[jb][p];
      xi[jb][p] = rj ? 0.0 : xi[jb][p];
      xr[p][jb] = cj ? 0.0 : xr[p][jb];
      xi[p][jb] = cj ? 0.0 : xi[p][jb];
    }
    auto update = [&](int q) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        xr[p][q] = fma(-fi[p], ci[q], fma(-fr[p], cr[q], xr[p][q]));
        xi[p][q] = fma(fr[p], ci[q], fma(-fi[p], cr[q], xi[p][q]));
      }
    };
    update(nb);
    if (j + 1 < kSw) {
      if (tx == (jt + 1) % 16) {
        double2* nxt = s_col[(j + 1) & 1];
#pragma unroll
        for (int p = 0; p < 4; ++p) nxt[ty + 16 * p] = double2{xr[p][nb], xi[p][nb]};
      }
      __syncthreads();
      load(j + 1);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q != nb) update(q);
  };
  load(0);
  auto block = [&](auto jbc) {   // sixteen steps whose row and column sit in piece jb
    constexpr int jb = decltype(jbc)::value;
#pragma unroll 1
    for (int jt = 0; jt < 15; ++jt) step(jbc, jbc, jt);
    step(jbc, std::integral_constant<int, jb < 3 ? jb + 1 : 3>{}, 15);
  };
  block(std::integral_constant<int, 0>{});
  block(std::integral_constant<int, 1>{});
  block(std::integral_constant<int, 2>{});
  block(std::integral_constant<int, 3>{});
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      dinv[(size_t)(ty + 16 * p) * kSw + tx + 16 * q] = double2{-xr[p][q], -xi[p][q]};
}

// The first block's D^-1 (the others come out of the preceding update).
__global__ __launch_bounds__(256) void k_sweep_diag(const double2* __restrict__ a, int ldp, size_t ws,
                                                    double2* __restrict__ dinv, int* __restrict__ flag) {
  __shared__ double2 s_col[2][kSw];
  a = slice(a, ws);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double xr[4][4], xi[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = ty + 16 * p, c = tx + 16 * q;
      const double2 y = a[(size_t)max(r, c) * ldp + min(r, c)];
      xr[p][q] = y.x;
      xi[p][q] = r == c ? 0.0 : (r > c ? y.y : -y.y);
    }
  diag_inverse(xr, xi, s_col, slice(dinv, ws), flag);
}

// 64 x 64 tile products on float64 MFMA, four waves of 32 x 32: c += A B^H for operands that hold KC
// consecutive inner values per row in LDS (odd row stride: the 16 rows of a fragment on different banks).
constexpr int kTc = 32;            // inner values per LDS stage
constexpr int kTcLd = kTc + 1;
template <int KC, int LD>
__device__ __forceinline__ void tile_abh(const double2* __restrict__ sa, const double2* __restrict__ sb, int ra, int rb,
                                         f64x4 (&cre)[2][2], f64x4 (&cim)[2][2]) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll 4
  for (int s = 0; s < KC / 4; ++s) {
    const int k = 4 * s + lk;
    double2 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = sa[(ra + 16 * i + li) * LD + k];
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = sb[(rb + 16 * j + li) * LD + k];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        cre[i][j] = mfma64(a[i].x, b[j].x, cre[i][j]);
        cre[i][j] = mfma64(a[i].y, b[j].y, cre[i][j]);
        cim[i][j] = mfma64(a[i].y, b[j].x, cim[i][j]);
        cim[i][j] = mfma64(-a[i].x, b[j].y, cim[i][j]);
      }
  }
}

// 16 rows i per workgroup: X_i = A_iK from the lower storage into xx[i][k], P_i = X_i D^-1 into pp[i][k] and
// into the swept entries of a (A_iK = P_i below the block, A_Ki = P_i^H above it, A_KK = -D^-1).  Each of
// the four waves forms 16 x 16 of P (16 rows per workgroup, so that also small matrices spread
// over the chip: one CU takes 7 us for 64 rows).
constexpr int kPr = 16;
__global__ __launch_bounds__(256) void k_sweep_panel(double2* __restrict__ a, int ldp, int k0, size_t ws,
                                                     const double2* __restrict__ dinv, double2* __restrict__ xx,
                                                     double2* __restrict__ pp) {
  constexpr int LD = kSw + 1;
  __shared__ double2 sx[kPr * LD];
  a = slice(a, ws);
  dinv = slice(dinv, ws);
  xx = slice(xx, ws);
  pp = slice(pp, ws);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i0 = blockIdx.x * kPr;
  if (i0 >= k0 && i0 < k0 + kSw) {
    for (int e = tid; e < kPr * kSw; e += 256) {
      const int r = i0 - k0 + e / kSw, c = e % kSw;
      const double2 d = dinv[(size_t)r * kSw + c];
      if (c <= r) a[(size_t)(k0 + r) * ldp + k0 + c] = double2{-d.x, -d.y};
    }
    return;
  }
  const bool below = i0 > k0;
  // this wave's 16 columns of D^-1, each value used once (D^-1 is Hermitian: X D^-1 = X (its rows)^H)
  const int li = lane & 15, lk = lane >> 4;
  double2 y[kSw / 4];
#pragma unroll
  for (int s = 0; s < kSw / 4; ++s) y[s] = dinv[(size_t)(16 * wave + li) * kSw + 4 * s + lk];
  if (below) {
#pragma unroll
    for (int rr = 0; rr < kPr / 4; ++rr) {
      const int r = 4 * rr + wave;
      sx[r * LD + lane] = a[(size_t)(i0 + r) * ldp + k0 + lane];
    }
  } else {   // rows of the block, columns i0 ..: conj-transposed
#pragma unroll
    for (int rr = 0; rr < kPr / 4; ++rr) {
      const int k = 16 * rr + (tid >> 4), r = tid & 15;
      const double2 z = a[(size_t)(k0 + k) * ldp + i0 + r];
      sx[r * LD + k] = double2{z.x, -z.y};
    }
  }
  __syncthreads();
  f64x4 cre{0, 0, 0, 0}, cim{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < kSw / 4; ++s) {
    const double2 x = sx[li * LD + 4 * s + lk];
    cre = mfma64(x.x, y[s].x, cre);
    cre = mfma64(x.y, y[s].y, cre);
    cim = mfma64(x.y, y[s].x, cim);
    cim = mfma64(-x.x, y[s].y, cim);
  }
#pragma unroll
  for (int rr = 0; rr < kPr / 4; ++rr) {
    const int r = 4 * rr + wave;
    xx[(size_t)(i0 + r) * kSw + lane] = sx[r * LD + lane];
  }
  __syncthreads();   // sx is read no more: P goes there
#pragma unroll
  for (int r = 0; r < 4; ++r) sx[(lk + 4 * r) * LD + 16 * wave + li] = double2{cre[r], cim[r]};
  __syncthreads();
#pragma unroll
  for (int rr = 0; rr < kPr / 4; ++rr) {
    const int r = 4 * rr + wave;
    const double2 x = sx[r * LD + lane];
    pp[(size_t)(i0 + r) * kSw + lane] = x;
    if (below) a[(size_t)(i0 + r) * ldp + k0 + lane] = x;
  }
  if (!below) {
#pragma unroll
    for (int rr = 0; rr < kPr / 4; ++rr) {
      const int k = 16 * rr + (tid >> 4), r = tid & 15;
      const double2 z = sx[r * LD + k];
      a[(size_t)(k0 + k) * ldp + i0 + r] = double2{z.x, -z.y};
    }
  }
}

// Rank-64 updates of 64 x 64 tiles, one workgroup per tile, operands with 64 values per row along the inner
// index, in two LDS stages of 32 (the second in registers while the first runs; 68 KB, two workgroups per CU).
//   SWEEP: A_ij -= P_i X_j^H on the lower tiles outside the block kt's row and column; the workgroup of the
//          next diagonal tile goes on to invert it (dinv), beside the other tiles.
//   else:  A_ij += L_i R_j^H for all i, j < n (leading dimension ld, edges masked).
template <bool SWEEP>
__global__ __launch_bounds__(256, 2) void k_rank64(double2* __restrict__ a, int ld, int n, int kt, size_t ws,
                                                   const double2* __restrict__ left, const double2* __restrict__ right,
                                                   double2* __restrict__ dinv, int* __restrict__ flag) {
  __shared__ double2 sl[kSw * kTcLd];
  __shared__ double2 sr[kSw * kTcLd];
  __shared__ double2 s_col[2][kSw];
  const int nt = (n + kSw - 1) / kSw;
  int ti, tj;
  bool next = false;
  if constexpr (SWEEP) {
    // tile t of the lower triangle of nt - 1 tile rows (the block's own left out), the next diagonal one first
    const int nl = (nt - 1) * nt / 2;
    const int first = kt + 1 < nt ? kt * (kt + 3) / 2 : 0;   // (kt, kt) of the reduced numbering
    const int b = (int)blockIdx.x;
    const int t = b == 0 ? first : (b <= first ? b - 1 : b);
    next = b == 0 && kt + 1 < nt;
    if (t >= nl) return;
    ti = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    while (ti * (ti + 1) / 2 > t) --ti;
    tj = t - ti * (ti + 1) / 2;
    ti += ti >= kt;
    tj += tj >= kt;
  } else {
    ti = (int)blockIdx.x / nt;
    tj = (int)blockIdx.x % nt;
  }
  a = slice(a, ws);
  left = slice(left, ws) + (size_t)ti * kSw * kSw;
  right = slice(right, ws) + (size_t)tj * kSw * kSw;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = 32 * (wave >> 1), wc = 32 * (wave & 1), li = lane & 15, lk = lane >> 4;
  const int r0 = ti * kSw + wr + lk, c0 = tj * kSw + wc + li;
  // staging: rows sr0 + 8 q, inner value tid % 32
  const int sk = tid & 31, sr0 = tid >> 5;
  double2 pl[8], pr[8];
  auto fetch = [&](int h) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = sr0 + 8 * q;
      const bool okl = SWEEP || ti * kSw + r < n, okr = SWEEP || tj * kSw + r < n;
      pl[q] = okl ? left[r * kSw + h * kTc + sk] : double2{0.0, 0.0};
      pr[q] = okr ? right[r * kSw + h * kTc + sk] : double2{0.0, 0.0};
    }
  };
  auto stash = [&] {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      sl[(sr0 + 8 * q) * kTcLd + sk] = pl[q];
      sr[(sr0 + 8 * q) * kTcLd + sk] = pr[q];
    }
  };
  f64x4 cre[2][2], cim[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) cre[i][j] = cim[i][j] = f64x4{0, 0, 0, 0};
  fetch(0);
  stash();
  __syncthreads();
  fetch(1);
  tile_abh<kTc, kTcLd>(sl, sr, wr, wc, cre, cim);
  __syncthreads();
  stash();
  // the tile of A, in flight while the second half runs
  double2 o[2][2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + 16 * i + 4 * r, col = c0 + 16 * j;
        o[i][j][r] = SWEEP || (row < n && col < n) ? a[(size_t)row * ld + col] : double2{0.0, 0.0};
      }
  __syncthreads();
  tile_abh<kTc, kTcLd>(sl, sr, wr, wc, cre, cim);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + 16 * i + 4 * r, col = c0 + 16 * j;
        const double s = SWEEP ? -1.0 : 1.0;
        const double2 v{fma(s, cre[i][j][r], o[i][j][r].x), fma(s, cim[i][j][r], o[i][j][r].y)};
        if (SWEEP || (row < n && col < n)) a[(size_t)row * ld + col] = v;
        o[i][j][r] = v;
      }
  if constexpr (SWEEP) {
    if (next) {   // workgroup-uniform
      // the updated tile through LDS (sl and sr hold 64 x 33 each: columns 0 .. 31 and 32 .. 63)
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            (wc ? sr : sl)[(wr + lk + 16 * i + 4 * r) * kTcLd + 16 * j + li] = o[i][j][r];
      __syncthreads();
      const int tx = tid & 15, ty = tid >> 4;
      double xr[4][4], xi[4][4];
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = ty + 16 * p, c = tx + 16 * q;
          const int hi = max(r, c), lo = min(r, c);   // the lower triangle
          const double2 y = (lo < 32 ? sl : sr)[hi * kTcLd + (lo & 31)];
          xr[p][q] = y.x;
          xi[p][q] = r == c ? 0.0 : (r > c ? y.y : -y.y);
        }
      diag_inverse(xr, xi, s_col, slice(dinv, ws), flag);
    }
  }
}

// eps^-1[i][j] = sqrt(v_i) (-A)_ij / sqrt(v_j) for i, j < n, A Hermitian from its lower triangle
__global__ void k_sweep_out(const double* __restrict__ v, const double2* __restrict__ a, int n, int ldp, size_t ws,
                            double2* __restrict__ out) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  v += (size_t)blockIdx.y * n;
  a = slice(a, ws);
  const int i = (int)(e / n), j = (int)(e % n);
  double2 x = i >= j ? a[(size_t)i * ldp + j] : a[(size_t)j * ldp + i];
  if (i < j) x.y = -x.y;
  if (i == j) x.y = 0.0;
  const double s = -sqrt(v[i]) / sqrt(v[j]);
  out[(size_t)blockIdx.y * n * n + e] = double2{s * x.x, s * x.y};
}

}  // namespace

hipError_t launch_zgemm_op(int m, int n, int k, double2 alpha, const double2* A, int lda, int opa, const double2* B,
                           int ldb, int opb, double2 beta, double2* C, int ldc, hipStream_t st) {
  if (m < 1 || n < 1 || k < 1 || opa < kOpN || opa > kOpConj || opb < kOpN || opb > kOpConj) return hipErrorInvalidValue;
  const int tiles = ((m + ZT - 1) / ZT) * ((n + ZT - 1) / ZT);
  // whole tiles and stages from rows: no bounds in the loads
  if ((opa == kOpN || opa == kOpConj) && (opb == kOpN || opb == kOpT) && n % ZT == 0 && k % ZK == 0 &&
      alpha.x == 1.0 && alpha.y == 0.0 && beta.x == 0.0 && beta.y == 0.0) {
    const auto f = opa == kOpN ? (opb == kOpT ? k_zgemm_rows<false, true> : k_zgemm_rows<false, false>)
                               : (opb == kOpT ? k_zgemm_rows<true, true> : k_zgemm_rows<true, false>);
    f<<<(tiles + 7) / 8 * 8, 256, 0, st>>>(m, n, k, A, lda, B, ldb, C, ldc);
    return hipGetLastError();
  }
  k_zgemm<<<tiles, 256, 0, st>>>(m, n, k, alpha, A, lda, opa, B, ldb, opb, beta, C, ldc);
  return hipGetLastError();
}

hipError_t launch_zgemm(int m, int n, int k, double2 alpha, const double2* A, int lda, bool cta, const double2* B,
                        int ldb, bool ctb, double2 beta, double2* C, int ldc, hipStream_t st) {
  return launch_zgemm_op(m, n, k, alpha, A, lda, cta ? kOpC : kOpN, B, ldb, ctb ? kOpC : kOpN, beta, C, ldc, st);
}

constexpr size_t up256(size_t x) { return (x + 255) / 256 * 256; }
constexpr size_t sweep_ld(int n) { return (size_t)((n + kSw - 1) / kSw * kSw); }
constexpr size_t sweep_bytes(int n) {
  return up256(sweep_ld(n) * sweep_ld(n) * sizeof(double2)) + 2 * up256(kSw * sweep_ld(n) * sizeof(double2)) +
         up256((size_t)kSw * kSw * sizeof(double2));
}

constexpr size_t gj_cands(int n) { return (size_t)(n + kGjRows - 1) / kGjRows; }
constexpr size_t gj_bytes(int n) {
  return up256((size_t)n * n * sizeof(double2)) + 2 * up256((size_t)n * kNb * sizeof(double2)) +
         2 * up256((size_t)n * kGjSub * sizeof(double2)) + 2 * up256((size_t)n * sizeof(int)) +
         2 * up256(gj_cands(n) * sizeof(double)) + 2 * up256(gj_cands(n) * sizeof(int));
}
// either route of the inverse (pivoted Gauss-Jordan, or the sweeps of the static form)
constexpr size_t eps_inv_bytes(int n) { return gj_bytes(n) > sweep_bytes(n) ? gj_bytes(n) : sweep_bytes(n); }

size_t eps_inv_workspace(int n) { return eps_inv_bytes(n); }

// ---------------------------------------------------------------- inverse without allocation
// Scratch of gw_eps_inv_noalloc: one file-scope device array, one copy per GPU, held until the
// process ends.  Host code never uses the array's name for its memory: the device address is
// looked up once per device (noalloc_scratch_init, called with the device current when a
// context is created there) and kept in noalloc_ptr.
constexpr size_t kNoAllocBytes = eps_inv_bytes(kNoAllocMaxNg);
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kNoAllocMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (g_noalloc_ptr[device]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e == hipSuccess) g_noalloc_ptr[device] = ptr;
  return e;
}

void* noalloc_scratch(int device) {
  if (device < 0 || device >= kNoAllocMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  return g_noalloc_ptr[device];
}

size_t noalloc_scratch_bytes() { return kNoAllocBytes; }

namespace {
struct GjWork {
  double2 *a, *pb[2], *t[2];   // matrix, panel buffers (afterwards the update's operands), sub-panels
  int *piv, *idx, *ci[2];      // row interchanges, column order, pivot candidates
  double* cm[2];
};

// R > 0: sub-panels of S columns in one workgroup with R rows per thread; R = 0: kGjSub columns, a launch
// per step
template <int R, int S>
hipError_t run_gj(int n, int nb, size_t ws, const GjWork& w, int* flag, hipStream_t st) {
  const unsigned rows = (unsigned)((n + kStepRows - 1) / kStepRows);
  const unsigned cand = (unsigned)gj_cands(n);
  for (int j0 = 0; j0 < n; j0 += kNb) {
    const int nbp = std::min(n - j0, kNb);
    k_panel_load<<<dim3(rows, nb), 256, 0, st>>>(w.a, n, j0, nbp, ws, w.pb[0]);
    int cur = 0;
    for (int c0 = 0; c0 < nbp; c0 += S) {
      const int sc = std::min(S, nbp - c0);
      const double2* t = w.t[0];
      if constexpr (R > 0) {
        k_gj_sub<R, S><<<dim3(1, nb), kGjThreads, 0, st>>>(w.pb[cur], n, j0, c0, sc, ws, w.t[0], w.piv, flag);
      } else {
        k_gj_load16<<<dim3(cand, nb), 256, 0, st>>>(w.pb[cur], n, j0, c0, sc, ws, w.t[0], w.cm[0], w.ci[0]);
        for (int jc = 0; jc < sc; ++jc) {
          const int i = jc & 1, o = i ^ 1;
          k_gj_step16<<<dim3(cand, nb), 256, 0, st>>>(w.t[i], w.t[o], n, j0 + c0 + jc, jc, (int)cand, ws, w.cm[i],
                                                      w.ci[i], w.cm[o], w.ci[o], w.piv, flag);
        }
        t = w.t[sc & 1];
      }
      k_gj_apply<S><<<dim3(rows, nb), 256, 0, st>>>(w.pb[cur], w.pb[cur ^ 1], n, j0, c0, sc, ws, t, w.piv);
      cur ^= 1;
    }
    double2* fin = w.pb[cur];
    double2* other = w.pb[cur ^ 1];
    if (nbp < n) k_row_swaps<<<dim3((n + 255) / 256, nb), 256, 0, st>>>(w.a, n, j0, nbp, ws, w.piv);
    const size_t nops = (size_t)(n + 7) / 8 * 8 * kNb;
    k_panel_operands<<<dim3((unsigned)((nops + 255) / 256), nb), 256, 0, st>>>(w.a, n, j0, nbp, ws, fin, other);
    if (nbp == n) break;   // a single panel: no other columns to update
    const unsigned nt = (unsigned)((n + kSw - 1) / kSw);
    k_rank64<false><<<dim3(nt * nt, nb), 256, 0, st>>>(w.a, n, n, 0, ws, fin, other, nullptr, nullptr);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_eps_inv(int n, int nb, const double* v, const double2* chi, double2* out, void* wsp, int* flag,
                          hipStream_t st) {
  const size_t ws = eps_inv_bytes(n);
  char* p = (char*)wsp;
  auto take = [&](size_t bytes) {
    char* q = p;
    p += up256(bytes);
    return q;
  };
  GjWork w;
  w.a = (double2*)take((size_t)n * n * sizeof(double2));
  for (auto& x : w.pb) x = (double2*)take((size_t)n * kNb * sizeof(double2));
  for (auto& x : w.t) x = (double2*)take((size_t)n * kGjSub * sizeof(double2));
  w.piv = (int*)take((size_t)n * sizeof(int));
  w.idx = (int*)take((size_t)n * sizeof(int));
  for (auto& x : w.cm) x = (double*)take(gj_cands(n) * sizeof(double));
  for (auto& x : w.ci) x = (int*)take(gj_cands(n) * sizeof(int));
  const dim3 gnn((unsigned)(((size_t)n * n + 255) / 256), nb);
  k_form_eps<<<gnn, 256, 0, st>>>(v, chi, n, ws, w.a);
  // columns per sub-panel: as many as the registers hold beside R rows per thread
  const int r = (n + kGjThreads - 1) / kGjThreads;
  const hipError_t e = r <= 1   ? run_gj<1, 16>(n, nb, ws, w, flag, st)
                       : r <= 2 ? run_gj<2, 16>(n, nb, ws, w, flag, st)
                       : r <= 3 ? run_gj<3, 8>(n, nb, ws, w, flag, st)
                       : r <= 4 ? run_gj<4, 8>(n, nb, ws, w, flag, st)
                                : run_gj<0, kGjSub>(n, nb, ws, w, flag, st);
  if (e != hipSuccess) return e;
  k_col_perm<<<dim3((n + 255) / 256, nb), 256, 0, st>>>(w.piv, n, ws, w.idx);
  k_gather_cols<<<gnn, 256, 0, st>>>(w.a, w.idx, n, ws, out);
  return hipGetLastError();
}

hipError_t launch_eps_inv_sweep(int n, int nb, const double* v, const double2* chi, double2* out, void* wsp, int* flag,
                                hipStream_t st) {
  const size_t ws = eps_inv_bytes(n);
  const int ldp = (int)sweep_ld(n);
  char* w = (char*)wsp;
  auto take = [&](size_t bytes) {
    char* p = w;
    w += up256(bytes);
    return p;
  };
  double2* a = (double2*)take((size_t)ldp * ldp * sizeof(double2));
  double2* xx = (double2*)take((size_t)kSw * ldp * sizeof(double2));
  double2* pp = (double2*)take((size_t)kSw * ldp * sizeof(double2));
  double2* dinv = (double2*)take((size_t)kSw * kSw * sizeof(double2));
  const size_t nn = (size_t)ldp * ldp;
  k_sweep_form<<<dim3((unsigned)((nn + 255) / 256), nb), 256, 0, st>>>(v, chi, n, ldp, ws, a, flag);
  const int nt = ldp / kSw;
  k_sweep_diag<<<dim3(1, nb), 256, 0, st>>>(a, ldp, ws, dinv, flag);
  for (int kt = 0; kt < nt; ++kt) {
    k_sweep_panel<<<dim3(ldp / kPr, nb), 256, 0, st>>>(a, ldp, kt * kSw, ws, dinv, xx, pp);
    if (nt > 1)
      k_rank64<true><<<dim3((nt - 1) * nt / 2, nb), 256, 0, st>>>(a, ldp, ldp, kt, ws, pp, xx, dinv, flag);
  }
  k_sweep_out<<<dim3((unsigned)(((size_t)n * n + 255) / 256), nb), 256, 0, st>>>(v, a, n, ldp, ws, out);
  return hipGetLastError();
}

// chibar = V Z^H Zbar Z^H  (V = diag v): t = Z^H Zbar, out = t Z^H, then rows scaled by v.
__global__ void k_scale_rows(double2* __restrict__ x, const double* __restrict__ v, int n) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const double s = v[e / n];
  x[e] = double2{x[e].x * s, x[e].y * s};
}

size_t eps_inv_backward_workspace(int n) { return (size_t)n * n * sizeof(double2) + 256; }

hipError_t launch_eps_inv_backward(int n, const double* v, const double2* z, const double2* zbar, double2* out,
                                   void* ws, hipStream_t st) {
  double2* t = (double2*)ws;
  hipError_t e = launch_zgemm(n, n, n, double2{1.0, 0.0}, z, n, true, zbar, n, false, double2{0.0, 0.0}, t, n, st);
  if (e != hipSuccess) return e;
  e = launch_zgemm(n, n, n, double2{1.0, 0.0}, t, n, false, z, n, true, double2{0.0, 0.0}, out, n, st);
  if (e != hipSuccess) return e;
  const size_t nn = (size_t)n * n;
  k_scale_rows<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(out, v, n);
  return hipGetLastError();
}

hipError_t launch_flag_clear(int* flag, hipStream_t st) {
  k_flag_clear<<<1, 64, 0, st>>>(flag);
  return hipGetLastError();
}

}  // namespace gw
