// Folded line transforms shared by the band, pair and gradient kernels.
//
// Every axis is transformed on the smallest alias-free grid: N = 4 nq points (a multiple of four).
// With theta = 2 pi / N and H = N / 2, the points come in nq quads that share their angles up to
// sign: quad j >= 1 holds x = (j, H - j, H + j, N - j), quad 0 holds (0, H/2, H, 3H/2).  A stored
// line is in quad order: position 4 j + t is entry t of quad j.
//
// Towards frequencies, F(n) = sum_x f(x) e^{i n x theta} = C(n) + i S(n), F(-n) = C(n) - i S(n):
// within a quad only four combinations of its entries (f0, f1, f2, f3) enter,
//   ce = f0 + f3 + (f1 + f2)  in C(n), n even      co = f0 + f3 - (f1 + f2)  in C(n), n odd
//   se = f0 - f3 - (f1 - f2)  in S(n), n even      so = f0 - f3 + (f1 - f2)  in S(n), n odd
// with the real factors cos(n j theta), sin(n j theta): K = 2 RC + 1 outputs take 2 K real FMAs per
// quad and 16 additions, instead of 8 K per point of the direct complex sum.  Quad 0 gives
// f0 + f2 to C even, f0 - f2 to C odd (factor 1), f1 + f3 to C even and f1 - f3 to S odd (factors
// cos(n pi/2), sin(n pi/2) = +-1).
// Towards points the same four real sums over the folded frequencies e_n = t_n + t_-n,
// o_n = t_n - t_-n give the four points of a quad.
#pragma once

#include "common.h"

namespace gw {

// the four combinations of an ordinary quad, and those of quad 0 (its second even sum in se)
template <typename V> struct Fold {
  V ce, co, se, so;
};
template <typename V> __device__ __forceinline__ Fold<V> fold_quad(const V (&p)[4]) {
  const V e1 = cadd(p[0], p[3]), o1 = csub(p[0], p[3]);
  const V e2 = cadd(p[1], p[2]), o2 = csub(p[1], p[2]);
  return Fold<V>{cadd(e1, e2), csub(e1, e2), csub(o1, o2), cadd(o1, o2)};
}
template <typename V> __device__ __forceinline__ Fold<V> fold_quad0(const V (&p)[4]) {
  return Fold<V>{cadd(p[0], p[2]), csub(p[0], p[2]), cadd(p[1], p[3]), csub(p[1], p[3])};
}

// Frequencies 0 .. RC of a line: NE even ones from 0, NO odd ones, NS = NE - 1 even ones from 2.
template <int RC> struct Freq {
  static constexpr int NE = RC / 2 + 1, NO = (RC + 1) / 2, NS = RC / 2;
  // groups of four rows of each sum, for the MFMA form
  static constexpr int GE = (NE + 3) / 4, GO = (NO + 3) / 4, GS = (NS + 3) / 4;
};

// Running sums of one line on the vector units.  Factors: row of quad j of the table written by
// gw_geom_create, cos(n j theta) at [n], sin(n j theta) at [RC + 1 + n]; row 0 holds cos(n pi/2)
// (n even) or sin(n pi/2) (n odd) at [n].  The row is wave-uniform (scalar loads).
template <typename T, int RC> struct LineSums {
  using V = cx<T>;
  using F = Freq<RC>;
  V ce[F::NE], co[F::NO], se[F::NS > 0 ? F::NS : 1], so[F::NO];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < F::NE; ++i) ce[i] = V{T(0), T(0)};
#pragma unroll
    for (int i = 0; i < F::NO; ++i) co[i] = so[i] = V{T(0), T(0)};
#pragma unroll
    for (int i = 0; i < F::NS; ++i) se[i] = V{T(0), T(0)};
  }
  static __device__ __forceinline__ void mac(V& a, T f, V x) {
    a.x = fma_t(f, x.x, a.x);
    a.y = fma_t(f, x.y, a.y);
  }
  __device__ __forceinline__ void add(const Fold<V>& q, const T* __restrict__ row) {
#pragma unroll
    for (int i = 0; i < F::NE; ++i) mac(ce[i], row[2 * i], q.ce);
#pragma unroll
    for (int i = 0; i < F::NO; ++i) mac(co[i], row[2 * i + 1], q.co);
#pragma unroll
    for (int i = 0; i < F::NS; ++i) mac(se[i], row[RC + 1 + 2 * i + 2], q.se);
#pragma unroll
    for (int i = 0; i < F::NO; ++i) mac(so[i], row[RC + 1 + 2 * i + 1], q.so);
  }
  __device__ __forceinline__ void add0(const Fold<V>& q, const T*) {
#pragma unroll
    for (int i = 0; i < F::NE; ++i) {
      ce[i] = cadd(ce[i], q.ce);
      ce[i] = i % 2 == 0 ? cadd(ce[i], q.se) : csub(ce[i], q.se);
    }
#pragma unroll
    for (int i = 0; i < F::NO; ++i) {
      co[i] = cadd(co[i], q.co);
      so[i] = i % 2 == 0 ? cadd(so[i], q.so) : csub(so[i], q.so);
    }
  }
  __device__ __forceinline__ V c(int n) const { return n % 2 == 0 ? ce[n / 2] : co[n / 2]; }
  __device__ __forceinline__ V s(int n) const { return n % 2 == 0 ? se[n / 2 - 1] : so[n / 2]; }
};

typedef float fold_f32x4 __attribute__((ext_vector_type(4)));

// The same in float32 on the matrix cores: v_mfma_f32_4x4x1 forms, in each of 16 blocks of four
// lanes, D[4 rows][4 columns] += A[4 rows] B[4 columns].  Each lane is one column (its own line)
// and holds four frequencies per accumulator; A holds the factors of the quad in the blocks of one
// register (block b: group b of even C, odd C, even S, odd S; lane 4 b + r: row r), and cbsz = 4 with
// abid = b broadcasts block b to all lanes, so one 4-byte register per lane serves a whole quad.
// Four FMAs per lane in 8 cycles of the matrix core, beside the products and folds on the VALU.
template <int RC> struct MfmaSums {
  using V = float2;
  using F = Freq<RC>;
  fold_f32x4 ce[F::GE][2], co[F::GO][2], se[F::GS > 0 ? F::GS : 1][2], so[F::GO][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
      for (int g = 0; g < F::GE; ++g) ce[g][k] = fold_f32x4{0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < F::GO; ++g) co[g][k] = so[g][k] = fold_f32x4{0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < F::GS; ++g) se[g][k] = fold_f32x4{0, 0, 0, 0};
    }
  }
  template <int B, int G> static __device__ __forceinline__ void mac(fold_f32x4 (*a)[2], float f, V x) {
    if constexpr (G > 0) {
      a[0][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(f, x.x, a[0][0], 4, B, 0);
      a[0][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(f, x.y, a[0][1], 4, B, 0);
      mac<B + 1, G - 1>(a + 1, f, x);
    }
  }
  __device__ __forceinline__ void add(const Fold<V>& q, float f) {
    mac<0, F::GE>(ce, f, q.ce);
    mac<F::GE, F::GO>(co, f, q.co);
    mac<F::GE + F::GO, F::GS>(se, f, q.se);
    mac<F::GE + F::GO + F::GS, F::GO>(so, f, q.so);
  }
  // quad 0: the blocks are even C (ones), odd C (ones), the second even C, odd S
  __device__ __forceinline__ void add0(const Fold<V>& q, float f) {
    mac<0, F::GE>(ce, f, q.ce);
    mac<F::GE, F::GO>(co, f, q.co);
    mac<F::GE + F::GO, F::GE>(ce, f, q.se);
    mac<2 * F::GE + F::GO, F::GO>(so, f, q.so);
  }
  __device__ __forceinline__ V c(int n) const {
    const int i = n / 2;
    return n % 2 == 0 ? V{ce[i / 4][0][i % 4], ce[i / 4][1][i % 4]} : V{co[i / 4][0][i % 4], co[i / 4][1][i % 4]};
  }
  __device__ __forceinline__ V s(int n) const {
    const int i = n % 2 == 0 ? n / 2 - 1 : n / 2;
    return n % 2 == 0 ? V{se[i / 4][0][i % 4], se[i / 4][1][i % 4]} : V{so[i / 4][0][i % 4], so[i / 4][1][i % 4]};
  }
};

// C + i S and C - i S
template <typename V> __device__ __forceinline__ V plus_i(V c, V s) { return V{c.x - s.y, c.y + s.x}; }
template <typename V> __device__ __forceinline__ V minus_i(V c, V s) { return V{c.x + s.y, c.y - s.x}; }

// Points of NQ quads from the frequencies |n| <= rw of a line: u(x) = sum_n t(n) e^{i n x theta}.
// load(n) gives t(n); fac(n, k) the pair (cos, sin)(n j_k theta) of quad k (for quad 0: 1, and
// cos(n pi/2) for n even or sin(n pi/2) for n odd).  first0: quad k = 0 of the group is quad 0.
// out[k][t] in the quad's order.
template <typename V, int NQ, typename Load, typename Fac>
__device__ __forceinline__ void points_of_quads(int rw, bool first0, Load load, Fac fac, V (&out)[NQ][4]) {
  V ae[NQ], ao[NQ], be[NQ], bo[NQ];
  const V t0 = load(0);
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    ae[k] = t0;
    ao[k] = bo[k] = V{0, 0};
    be[k] = k == 0 && first0 ? t0 : V{0, 0};
  }
  auto mac = [](V& a, auto f, V x) {
    a.x = fma_t(f, x.x, a.x);
    a.y = fma_t(f, x.y, a.y);
  };
  int n = 1;
  for (; n + 1 <= rw; n += 2) {
    const V p = load(n), m = load(-n), p2 = load(n + 1), m2 = load(-n - 1);
    const V e = cadd(p, m), o = csub(p, m);
    const V e2 = cadd(p2, m2), o2 = csub(p2, m2);
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const V f = fac(n, k), f2 = fac(n + 1, k);
      mac(ao[k], f.x, e);
      mac(bo[k], f.y, o);
      mac(ae[k], f2.x, e2);
      const bool z = k == 0 && first0;
      mac(be[k], f2.y, z ? e2 : o2);
    }
  }
  if (n <= rw) {
    const V p = load(n), m = load(-n);
    const V e = cadd(p, m), o = csub(p, m);
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const V f = fac(n, k);
      mac(ao[k], f.x, e);
      mac(bo[k], f.y, o);
    }
  }
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const V x = cadd(ae[k], ao[k]), y = csub(ae[k], ao[k]);
    if (k == 0 && first0) {
      out[k][0] = x;
      out[k][1] = plus_i(be[k], bo[k]);
      out[k][2] = y;
      out[k][3] = minus_i(be[k], bo[k]);
    } else {
      const V sx = cadd(be[k], bo[k]), sy = csub(bo[k], be[k]);
      out[k][0] = plus_i(x, sx);
      out[k][1] = plus_i(y, sy);
      out[k][2] = minus_i(y, sy);
      out[k][3] = minus_i(x, sx);
    }
  }
}

// x of position p of a line in quad order (nt points)
__host__ __device__ __forceinline__ int quad_x(int p, int nt) {
  const int j = p >> 2, t = p & 3, h = nt / 2;
  if (j == 0) return t * (h / 2);
  return t == 0 ? j : t == 1 ? h - j : t == 2 ? h + j : nt - j;
}

}  // namespace gw
