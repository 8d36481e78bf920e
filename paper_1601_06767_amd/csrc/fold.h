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

// Slots of the MFMA forms: four frequencies of one sum each, those of a line's C and S paired so that
// one lane holds both.  Slot (odd, part, g), part 0 = C, 1 = S: n = 2 (4 g + i) + odd, i = 0 .. 3
// (S of n = 0 has zero factors).  Factors of a quad: 32 floats, four of each slot in order; of quad 0,
// S even holds the second even sum of C.
template <int RC> struct Slots {
  using F = Freq<RC>;
  static constexpr int NG = RC >= 8 ? 2 : 1;
  static constexpr int N = 4 * NG;
  static constexpr int at(int odd, int part, int g) { return (odd * NG + g) * 2 + part; }
  static constexpr bool used(int i) { return 4 * (i / 2 % NG) < (i / 2 / NG ? F::NO : F::NE); }
  // the combination that slot i sums
  template <typename V> static __device__ __forceinline__ V part(const Fold<V>& q, int i) {
    return i / 2 / NG == 0 ? (i % 2 == 0 ? q.ce : q.se) : (i % 2 == 0 ? q.co : q.so);
  }
};

// Running sums of one line per lane in float32 on the matrix cores.  v_mfma_f32_4x4x1 forms, in each of
// 16 blocks of four lanes, D[4 rows][4 columns] += A[4 rows] B[4 columns].  Here each lane is one column
// (its own line) and holds four frequencies per accumulator; A holds the factors (lane 4 b + r: row r of
// slot b), and cbsz = 4 with abid = b broadcasts block b to all lanes, so one 4-byte register per lane
// serves a whole quad.  Four FMAs per lane in 8 cycles of the matrix core, beside the VALU.
template <int RC> struct MfmaSums {
  using V = float2;
  using S = Slots<RC>;
  fold_f32x4 a[S::N][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < S::N; ++i) a[i][0] = a[i][1] = fold_f32x4{0, 0, 0, 0};
  }
  template <int I> __device__ __forceinline__ void mac(fold_f32x4 (&d)[2], float f, V x) {
    d[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(f, x.x, d[0], 4, I, 0);
    d[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(f, x.y, d[1], 4, I, 0);
  }
  template <int I = 0> __device__ __forceinline__ void add(const Fold<V>& q, float f) {
    if constexpr (I < S::N) {
      if constexpr (S::used(I)) mac<I>(a[I], f, S::part(q, I));
      add<I + 1>(q, f);
    }
  }
  // quad 0: slots S even go to C even
  template <int I = 0> __device__ __forceinline__ void add0(const Fold<V>& q, float f) {
    if constexpr (I < S::N) {
      if constexpr (S::used(I)) mac<I>(a[I < S::N / 2 ? I & ~1 : I], f, S::part(q, I));
      add0<I + 1>(q, f);
    }
  }
  __device__ __forceinline__ V get(int part, int n) const {
    const int i = S::at(n % 2, part, n / 8);
    return V{a[i][0][n / 2 % 4], a[i][1][n / 2 % 4]};
  }
  __device__ __forceinline__ V c(int n) const { return get(0, n); }
  __device__ __forceinline__ V s(int n) const { return get(1, n); }
};

// The same sums with the roles exchanged: A holds the data of the block's four lanes (four lines), B the
// factors of a slot (blgp broadcasts one 16-lane section to all four: lane 16 s + 4 x + i holds factor i of
// slot s), so that lane 4 b + i receives frequency i of all four lines of its block in one accumulator.
template <int RC> struct MfmaTranspose {
  using V = float2;
  using S = Slots<RC>;
  fold_f32x4 a[S::N][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < S::N; ++i) a[i][0] = a[i][1] = fold_f32x4{0, 0, 0, 0};
  }
  template <int I> __device__ __forceinline__ void mac(fold_f32x4 (&d)[2], const float (&f)[S::NG], V x) {
    d[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(x.x, f[I / 4], d[0], 0, 0, 4 + I % 4);
    d[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(x.y, f[I / 4], d[1], 0, 0, 4 + I % 4);
  }
  template <int I = 0> __device__ __forceinline__ void add(const Fold<V>& q, const float (&f)[S::NG]) {
    if constexpr (I < S::N) {
      if constexpr (S::used(I)) mac<I>(a[I], f, S::part(q, I));
      add<I + 1>(q, f);
    }
  }
  template <int I = 0> __device__ __forceinline__ void add0(const Fold<V>& q, const float (&f)[S::NG]) {
    if constexpr (I < S::N) {
      if constexpr (S::used(I)) mac<I>(a[I < S::N / 2 ? I & ~1 : I], f, S::part(q, I));
      add0<I + 1>(q, f);
    }
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
