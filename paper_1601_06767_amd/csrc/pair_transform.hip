// Pair transform: the matrix element of Eq. (chi0),
//   M_vc(G) = (1/N) sum_r conj(u_v(r)) u_c(r) exp(iG.r),   G in the dielectric sphere,
// formed as the product of two real-space bands followed by a forward transform
// that only produces the K = 2 RC + 1 frequencies per axis the sphere needs, on the smallest
// alias-free grid (fold.h).
//
// k_pair_planes (float64) and k_pair_planes_mfma (float32), per x1 plane and TV valence x TC conduction
//   bands: over the plane's quads of x2 rows, the product along x3 and its folded x3 sums, then the folded
//   x2 sums over the quad's four rows, accumulated over the quads in registers;
//   output Q[pair][x1][l] for the lines l = (n2, n3) that hold a G of the sphere.
// k_pair_finish (one pair per workgroup): the folded x1 sums of Q's lines, the 1/N, and the
//   gather onto the sphere order: M[pair][G] (zero padded to ngp).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "fold.h"
#include "internal.h"

namespace gw {

namespace {

// Order of the planes' work: each XCD (workgroup b runs on XCD b mod 8) takes a contiguous run of the
// plane-major order; within a plane, strips of kStrip column tiles, their valence tiles in turn, so that the
// workgroups in flight on an XCD share their bands in its L2 (a plane of every band would not fit).
// False where index i of the XCD's run is past its end.
constexpr int kStrip = 8;
__device__ __forceinline__ bool plane_item(int i, int nt, int nbc, int nbv, int& x1, int& bc, int& bv) {
  const int total = nt * nbc * nbv;
  const int per = (total + 7) / 8;
  const int item = (int)(blockIdx.x % 8) * per + i;
  if (i >= per || item >= total) return false;
  x1 = item / (nbc * nbv);
  const int pb = item % (nbc * nbv);
  const int strip = pb / (kStrip * nbv), in = pb % (kStrip * nbv);
  const int wide = min(kStrip, nbc - strip * kStrip);
  bc = strip * kStrip + in % wide;
  bv = in / wide;
  return true;
}

// ---------------------------------------------------------------------------------------------
// float32: both sums on the matrix cores, without an exchange through LDS.
//
// A wave takes PW = 16 / QL pairs and QL quads of x2 rows; lane 4 b + t is row t of a quad of a pair (b:
// the quad in the high bits).  Stage 1 (MfmaTranspose) leaves in lane 4 b + i, per slot, the x3 sums of
// frequency i for the four rows of the quad: the fold of the rows is within the lane.  The C and S sums
// stay apart (x2 sums are linear); they meet at the end as C' +- i S' = Q(n2, +-n3).  With QL > 1
// v_permlane32_swap and v_permlane16_swap trade slots for quads between the lanes of one pair: each keeps
// NL = N / QL slots, for all the quads.  Stage 2 (MfmaSums) adds a quad's folded rows to the lane's
// running x2 sums.
// Rows come in by direct loads, a chunk of x3 quads of the QL row quads at a time into two buffers; the
// only barrier is the one per chunk.
template <int RC, int QL_, int WV_, int TV_, int TC_, int NU_, int MINW_> struct MfmaShape {
  using S = Slots<RC>;
  static constexpr int QL = QL_, WV = WV_, TV = TV_, TC = TC_, MINW = MINW_;
  static constexpr int NU = NU_;                       // 16-byte units of a buffer
  static constexpr int NT = 64 * WV;
  static constexpr int PW = 16 / QL;                   // pairs per wave, all of one valence band
  static constexpr int NL = S::N / QL;                 // slots a lane keeps
  static constexpr int NR = 4 * QL;                    // rows of a band in a step
  static constexpr int NQM = 32;                       // quads of the largest grid
  static constexpr int NF = 16 * S::NG;                // factors of a quad
  static constexpr int ND = (NU / 64 + WV - 1) / WV;   // direct loads of a wave per chunk
  static constexpr int NST = NL * (2 * RC + 1);        // stores of a wave per item
  static_assert(NST < 64, "stores in flight");
  static_assert(TV * TC == WV * PW && TC % PW == 0 && NL % 2 == 0, "planes shape");
  static_assert(2 * (NU + 2) * 16 + (NQM + 1) * NF * 4 + ND * NT * 4 + 124 <= 160 * 1024, "planes workgroup exceeds the LDS");
  // units of a row in LDS: an odd number of 64-byte groups, and one unit more per band, so that the 16
  // lanes of four rows and four bands read different banks
  static __host__ __device__ int row_units(int cq) { return 2 * cq + (12 - 2 * cq % 8) % 8; }
  static __host__ __device__ int band_units(int cq) { return NR * row_units(cq) + 1; }
  static __host__ __device__ int part_units(int nb, int cq) { return (nb * band_units(cq) + 63) / 64 * 64; }
  // chunks of x3 quads per row: an even number (two buffers in fixed roles) of equal size that fit a buffer
  static __host__ int chunks(int nq) {
    for (int n = 2; n <= nq; n += 2) {
      const int cq = (nq + n - 1) / n;
      if (part_units(TC, cq) + part_units(TV, cq) <= NU) return n;
    }
    return 0;
  }
};

// swap between lane halves: a = (a's, b's lower half), b = (a's, b's upper half)
__device__ __forceinline__ void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                  false, false);
  const unsigned x = r[0], y = r[1];   // an element of a vector cannot be bit-cast in place
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}
// the same between the even and odd 16-lane rows
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                  false, false);
  const unsigned x = r[0], y = r[1];   // an element of a vector cannot be bit-cast in place
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}

template <int RC, typename P>
__device__ __forceinline__ void planes_mfma(const float2* __restrict__ psi_v, const float2* __restrict__ psi_c, int nvs,
                                            int ncs, int nt, int nl, int nch, unsigned inv_r, unsigned inv_b,
                                            const int32_t* __restrict__ rowtab, const float* __restrict__ fac,
                                            float2* __restrict__ q) {
  using V = float2;
  using S = Slots<RC>;
  constexpr int NT = P::NT, TV = P::TV, TC = P::TC, QL = P::QL, NR = P::NR, NL = P::NL, N = S::N;
  // the TC columns, then the TV valence bands: [band][row][units of the chunk]
  __shared__ __align__(16) uint4 s_u0[P::NU + 2];   // the last quad's prefetch reads one quad on
  __shared__ __align__(16) uint4 s_u1[P::NU + 2];
  __shared__ __align__(16) float s_f[(P::NQM + 1) * P::NF];   // per quad [slot % 4][4 factors][slot / 4]
  __shared__ int s_row[2 * RC + 1];   // per n2: lowest n3, number of n3 << 8, (first line - lowest n3) << 16
  int it = blockIdx.x / 8, x1, c0, v0;
  if (!plane_item(it, nt, ncs / TC, nvs / TV, x1, c0, v0)) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // What a lane stands for is formed anew where it is needed: the accumulators leave no registers to keep it.
  struct Lane {
    int lane, ti, ql, pc;   // row of the quad, or frequency of the slot; quad of the step; column band
  };
  const int pc0 = wave % (TC / P::PW) * P::PW, pv = wave / (TC / P::PW);
  auto who = [&] {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return Lane{l, l & 3, (l >> 2) / P::PW, pc0 + (l >> 2) % P::PW};
  };

  const int row = nt + 2;                       // stored row length
  const int nq = nt / 4;
  const int nrs = (nq + QL - 1) / QL;           // row steps
  const int cq = (nq + nch - 1) / nch;          // x3 quads per chunk (the last ones may have fewer)
  const int lr = P::row_units(cq), lb = P::band_units(cq);
  const int nc = P::part_units(TC, cq), nslot = (nc + P::part_units(TV, cq)) / 64;
  const size_t band = (size_t)nt * nt * row;
  // Direct loads: slot s (64 units) of a chunk is loaded by wave s % WV from an offset per lane that is the
  // same for every chunk (no address arithmetic per chunk) plus a wave-uniform one.  Units that pad a row
  // or band, and rows and units past the end, are loaded and not used; the buffers' bounds end at the bands.
  const auto buffer = [&](const float2* psi, int nbands, int b0, int x) {
    const size_t first = (size_t)b0 * band + (size_t)x * nt * row;
    const size_t bytes = min(((size_t)nbands * band - first) * sizeof(V), (size_t)0xfffffff0u);
    return __builtin_amdgcn_make_buffer_rsrc((void*)(psi + first), 0, (int)(unsigned)bytes, 0x00020000);
  };
  auto rsrc_c = buffer(psi_c, ncs, c0 * TC, x1);
  auto rsrc_v = buffer(psi_v, nvs, v0 * TV, x1);
  // The offsets are kept in LDS: the accumulators leave no registers for them.
  __shared__ int s_off[P::ND * NT];
#pragma unroll 1
  for (int i = 0; i < P::ND; ++i) {
    const int s = wave + i * P::WV;
    const unsigned u = (64 * s >= nc ? 64 * s - nc : 64 * s) + (tid & 63);
    const unsigned b = min((unsigned)__umulhi(u, inv_b), (unsigned)((64 * s >= nc ? TV : TC) - 1));
    const unsigned in = min(u - b * lb, (unsigned)lb - 2);
    const unsigned y = __umulhi(in, inv_r);
    s_off[i * NT + tid] = (int)(b * (unsigned)(band * sizeof(V)) + y * (unsigned)(row * sizeof(V)) + (in - y * lr) * 16);
  }
  auto store = [](auto rsrc, unsigned at, V x) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__builtin_bit_cast(unsigned, x.x), __builtin_bit_cast(unsigned, x.y)},
                                          rsrc, (int)at, 0, 0);
  };
  auto issue = [&](int rs, int ch, uint4* dst) {
    const int at = rs * NR * row * (int)sizeof(V) + ch * cq * 32;
    const Lane w = who();
    int off[P::ND];
#pragma unroll
    for (int i = 0; i < P::ND; ++i) off[i] = s_off[i * NT + wave * 64 + w.lane];
#pragma unroll
    for (int i = 0; i < P::ND; ++i) {
      const int s = wave + i * P::WV;
      auto* to = (__attribute__((address_space(3))) void*)(dst + 64 * s);
      if (64 * s < nc)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_c, to, 16, off[i], at, 0, 0);
      else if (s < nslot)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_v, to, 16, off[i], at, 0, 0);
    }
  };
  constexpr int NF = P::NF;
  for (int i = tid; i < nq * NF; i += NT) {                 // visible after the first barrier
    const int j = i / NF, e = i % NF / S::NG, g = i % S::NG;
    s_f[i] = fac[32 * j + 16 * g + e];
  }
  if (tid < 2 * RC + 1) {   // rowtab: first line minus lowest n3, lowest and highest n3 (from 0)
    const int32_t* e = rowtab + 3 * tid;
    s_row[tid] = (int)((unsigned)e[0] << 16) | max(e[2] - e[1] + 1, 0) << 8 | e[1];
  }

  MfmaSums<RC> acc[NL];

  // one chunk: wait for it, start the next one (after the item's last, the next item's first), add its quads
  int nx1, nc0, nv0;
  bool more = false;
  auto chunk = [&](int rs, int ch, auto q0, auto first, MfmaTranspose<RC>& sm, const uint4* cur, uint4* nxt) {
    wait_vm<decltype(first)::value ? P::NST : 0>();   // an item's first chunk: its stores came after the loads
    lds_barrier();   // the chunk has landed; every wave is done with the other buffer
    const bool wrap = ch + 1 == nch, last = wrap && rs + 1 == nrs;
    if (last) {
      it += gridDim.x / 8;
      more = plane_item(it, nt, ncs / TC, nvs / TV, nx1, nc0, nv0);
      if (more) {
        rsrc_c = buffer(psi_c, ncs, nc0 * TC, nx1);
        rsrc_v = buffer(psi_v, nvs, nv0 * TV, nx1);
      }
    }
    if (!last || more) issue(last ? 0 : wrap ? rs + 1 : rs, wrap ? 0 : ch + 1, nxt);
    const Lane w = who();
    const V* rc = (const V*)(cur + w.pc * lb + (w.ql * 4 + w.ti) * lr);
    const V* rv = (const V*)(cur + nc + pv * lb + (w.ql * 4 + w.ti) * lr);
    const float* ff = s_f + (4 * (w.lane >> 4) + w.ti) * S::NG + ch * cq * NF;   // 16-lane section = slot
    const int ne = min(cq, nq - ch * cq);
    if (ne <= 0) return;
    // The MFMAs of a quad run beside the folds of the next one, with the operands of the one after in flight.
    V na[4], nb[4], p[4];
    auto load = [&](int j) {
      __builtin_memcpy(na, __builtin_assume_aligned(rv + 4 * j, 16), 4 * sizeof(V));
      __builtin_memcpy(nb, __builtin_assume_aligned(rc + 4 * j, 16), 4 * sizeof(V));
      asm volatile("" ::: "memory");   // the reads stay here, a quad ahead of their use
    };
    auto factors = [&](int j, float (&f)[S::NG]) {
#pragma unroll
      for (int g = 0; g < S::NG; ++g) f[g] = ff[NF * j + g];
    };
    auto product = [&] {
#pragma unroll
      for (int k = 0; k < 4; ++k) p[k] = cmulc(na[k], nb[k]);
      // the operands' registers are free: the next reads go out before the MFMAs
      asm volatile("" : "+v"(p[0].x), "+v"(p[0].y), "+v"(p[1].x), "+v"(p[1].y), "+v"(p[2].x), "+v"(p[2].y), "+v"(p[3].x),
                   "+v"(p[3].y)::"memory");
    };
    load(0);
    product();
    load(1);
    Fold<V> h;
    int j = 0;
    if constexpr (decltype(q0)::value) {
      h = fold_quad0(p);
      float f[S::NG];
      factors(0, f);
      if (ne > 1) product();
      load(2);
      sm.clear();
      sm.add0(h, f);
      if (ne == 1) return;
      j = 1;
    }
    h = fold_quad(p);
    auto quad = [&](int j, const Fold<V>& x) {
      float f[S::NG];
      factors(j, f);
      product();
      load(j + 2);
      __builtin_amdgcn_sched_barrier(0);
      const Fold<V> y = fold_quad(p);
      sm.add(x, f);
      return y;
    };
    // two quads per turn: no copies, half of the address arithmetic
#pragma unroll 1
    for (; j + 2 < ne; j += 2) {
      const Fold<V> g = quad(j, h);
      h = quad(j + 1, g);
    }
    if (j + 1 < ne) h = quad(j++, h);
    float f[S::NG];
    factors(j, f);
    sm.add(h, f);
  };
  auto step = [&](int rs, auto first) {
    constexpr bool kFirst = decltype(first)::value;
    MfmaTranspose<RC> sm;
    chunk(rs, 0, std::true_type{}, first, sm, s_u0, s_u1);
    chunk(rs, 1, std::false_type{}, std::false_type{}, sm, s_u1, s_u0);
#pragma unroll 1
    for (int ch = 2; ch < nch; ch += 2) {
      chunk(rs, ch, std::false_type{}, std::false_type{}, sm, s_u0, s_u1);
      chunk(rs, ch + 1, std::false_type{}, std::false_type{}, sm, s_u1, s_u0);
    }
    const Lane w = who();
    const float* f2 = s_f + (w.lane & 15) * S::NG + (w.lane >> 4) % S::NG;   // four lanes = slot
    // slots for quads: afterwards a[q NL + l] is slot l of this lane for quad q
    if constexpr (QL >= 2) {
#pragma unroll
      for (int i = 0; i < N / 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            float x = sm.a[i][k][t], y = sm.a[i + N / 2][k][t];
            swap32(x, y);
            sm.a[i][k][t] = x;
            sm.a[i + N / 2][k][t] = y;
          }
    }
    if constexpr (QL == 4) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < N / 4; ++i)
#pragma unroll
          for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              float x = sm.a[h * (N / 2) + i][k][t], y = sm.a[h * (N / 2) + i + N / 4][k][t];
              swap16(x, y);
              sm.a[h * (N / 2) + i][k][t] = x;
              sm.a[h * (N / 2) + i + N / 4][k][t] = y;
            }
    }
#pragma unroll
    for (int k = 0; k < QL; ++k) {
      if (kFirst && k == 0)
#pragma unroll
        for (int l = 0; l < NL; ++l) acc[l].clear();
      const int j2 = rs * QL + k;
      if (j2 < nq) {
        const float f = f2[NF * j2];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          const fold_f32x4 x = sm.a[k * NL + l][0], y = sm.a[k * NL + l][1];
          const V p[4] = {V{x[0], y[0]}, V{x[1], y[1]}, V{x[2], y[2]}, V{x[3], y[3]}};
          if (kFirst && k == 0)
            acc[l].add0(fold_quad0(p), f);
          else
            acc[l].add(fold_quad(p), f);
        }
      }
    }
  };
  issue(0, 0, s_u0);
  wait_vm<0>();
  for (;;) {
    step(0, std::true_type{});
#pragma unroll 1
    for (int rs = 1; rs < nrs; ++rs) step(rs, std::false_type{});
    const Lane w = who();
    // Q's lines; every wave issues the same number of stores (lanes out of range: beyond the buffer's bounds)
    const size_t first = (((size_t)(v0 * TV + pv) * ncs + c0 * TC) * nt + x1) * (size_t)nl;
    const size_t bytes = min(((size_t)nvs * ncs * nt * nl - first) * sizeof(V), (size_t)0xfffffff0u);
    const auto rsrc_q = __builtin_amdgcn_make_buffer_rsrc(q + first, 0, (int)(unsigned)bytes, 0x00020000);
#pragma unroll
    for (int l = 0; l < NL; l += 2) {
      const int sp = w.ql * (NL / 2) + l / 2;             // the (C, S) pair of slots
      const int n3 = 2 * (4 * (sp % S::NG) + w.ti) + sp / S::NG;
      const int jp = RC + n3, jm = n3 > 0 ? RC - n3 : -1;
      const unsigned at = (unsigned)(w.pc * nt) * (unsigned)(nl * sizeof(V));
      auto put = [&](int n2, V c, V s) {
        const int e = __builtin_amdgcn_readfirstlane(s_row[n2 + RC]);
        const int lo = e & 255, cnt = e >> 8 & 255, off = (e >> 16) * (int)sizeof(V);
        store(rsrc_q, (unsigned)(jp - lo) < (unsigned)cnt ? at + off + 8 * jp : 0xfffffff8u, plus_i(c, s));
        store(rsrc_q, (unsigned)(jm - lo) < (unsigned)cnt ? at + off + 8 * jm : 0xfffffff8u, minus_i(c, s));
      };
      put(0, acc[l].c(0), acc[l + 1].c(0));
#pragma unroll
      for (int n = 1; n <= RC; ++n) {
        put(n, plus_i(acc[l].c(n), acc[l].s(n)), plus_i(acc[l + 1].c(n), acc[l + 1].s(n)));
        put(-n, minus_i(acc[l].c(n), acc[l].s(n)), minus_i(acc[l + 1].c(n), acc[l + 1].s(n)));
      }
    }
    if (!more) break;
    x1 = nx1;
    c0 = nc0;
    v0 = nv0;
  }
}

template <int RC, typename P>
__global__ __launch_bounds__(P::NT, P::MINW) void k_pair_planes_mfma(const float2* __restrict__ psi_v,
                                                                     const float2* __restrict__ psi_c, int nvs,
                                                                     int ncs, int nt, int nl, int nch, unsigned inv_r,
                                                                     unsigned inv_b, const int32_t* __restrict__ rowtab,
                                                                     const float* __restrict__ fac,
                                                                     float2* __restrict__ q) {
  planes_mfma<RC, P>(psi_v, psi_c, nvs, ncs, nt, nl, nch, inv_r, inv_b, rowtab, fac, q);
}

// ---------------------------------------------------------------------------------------------
// float64, on the vector units: per step and lane one (pair, x2 row), the folded x3 sums of the product
// -> Z[pair][row][n3] in LDS; then per lane (pair, n3) the folded x2 sums over the quad's four rows,
// accumulated over the quads in registers.
//
// Shape of a workgroup.  HS: waves that share a line's x3 quads (partial sums added in LDS);
// QS: quads of x2 rows per step; NM: largest grid (the LDS row buffers).
// AL: the partial sums lie where the step's rows were, one set per share, and the next step's rows are loaded
// after them: half the LDS, for two workgroups per CU or for twice the row quads in one.
template <typename T, int RC, int HS_, int QS_, int TV_, int TC_, int NM_, int MINW_, bool AL_ = false>
struct PlaneShape {
  static constexpr int HS = HS_, QS = QS_, TV = TV_, TC = TC_, NM = NM_, MINW = MINW_;
  static constexpr bool AL = AL_;
  static constexpr int K = 2 * RC + 1;
  static constexpr int NP = TV * TC;               // pairs
  static constexpr int PG = NP / 16;               // waves per row quad and half: 16 pairs x 4 rows
  static constexpr int NT = 64 * HS * QS * PG;
  static constexpr int PS = 4 * K + 1;             // Z of a pair and quad: [row][n3], odd stride
  static constexpr int PADE = 16 / (int)sizeof(cx<T>);   // row padding (complex values): odd 16-byte units
  // row buffer: per band its QS quads of rows and one 16-byte unit (an odd stride between bands)
  static constexpr int NU = (TC + TV) * (QS * 4 * (NM + PADE) / PADE + 1);
  static constexpr int NB = AL ? HS : 1;           // sets of partial sums
  static constexpr int NZ = NB * QS * NP * PS;
  static constexpr size_t rows = (size_t)NU * 16, sums = (size_t)NZ * sizeof(cx<T>);
  static constexpr size_t lds = AL ? std::max(rows, sums) : rows + sums;
  static constexpr int NITEM = NP * K;
  static constexpr int IPL = (NITEM + NT - 1) / NT;
  static_assert(lds <= 160 * 1024, "planes workgroup exceeds the LDS");
  static_assert(HS == 1 || HS == 2, "shares of a line");
};

template <typename T, int RC, typename P>
__global__ __launch_bounds__(P::NT, P::MINW) void k_pair_planes(const cx<T>* __restrict__ psi_v,
                                                                const cx<T>* __restrict__ psi_c, int nvs, int ncs,
                                                                int nt, int nl, const int32_t* __restrict__ rowtab,
                                                                const T* __restrict__ fac, cx<T>* __restrict__ q) {
  using V = cx<T>;
  constexpr int K = P::K, NT = P::NT, TV = P::TV, TC = P::TC, HS = P::HS, QS = P::QS, PS = P::PS;
  constexpr int EPU = P::PADE;   // complex values per 16-byte unit
  // [band: TC columns, TV valence][quad][t][row], band stride odd
  __shared__ __align__(16) uint4 s_u[P::AL ? P::lds / 16 : P::NU];
  __shared__ __align__(16) V s_z0[P::AL ? 1 : P::NZ];
  V* s_z = P::AL ? (V*)s_u : s_z0;   // [set][quad][pair][t][n3]

  int x1, c0, v0;
  if (!plane_item(blockIdx.x / 8, nt, ncs / TC, nvs / TV, x1, c0, v0)) return;
  c0 *= TC;
  v0 *= TV;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int pg = wave % P::PG;                 // pair group
  const int hf = (wave / P::PG) % HS;          // share of the x3 quads
  const int qs = wave / (P::PG * HS);          // quad of the step
  const int t = lane >> 4;                     // row of the quad
  const int pair = pg * 16 + (lane & 15);
  const int pv = pair / TC, pc = pair % TC;

  const int row = nt + EPU;                    // stored row length
  const int ur = row / EPU;                    // its 16-byte units
  const int nq = nt / 4;
  const int nstep = (nq + QS - 1) / QS;
  const size_t band = (size_t)nt * nt * row;
  const size_t bb = band * sizeof(V);
  const int lb = QS * 4 * ur + 1;              // units per band in LDS
  const char* pcb = (const char*)(psi_c + (size_t)c0 * band + (size_t)x1 * nt * row);
  const char* pvb = (const char*)(psi_v + (size_t)v0 * band + (size_t)x1 * nt * row);
  // Direct loads of a step: the rows of a band's quads are contiguous in memory, taken 64 units per
  // wave instruction from a wave-uniform address (no registers but the lane's offset).
  auto issue = [&](int st) {
    const int lu = min(QS, nq - st * QS) * 4 * ur;   // units per band
    const int nch = (lu + 63) / 64;
    const size_t off = (size_t)st * QS * 4 * row * sizeof(V);
    int b = 0, ch = wave;
    for (;;) {
      while (ch >= nch) {
        ch -= nch;
        ++b;
      }
      if (b >= TC + TV) break;
      const char* src = (b < TC ? pcb + b * bb : pvb + (b - TC) * bb) + (off + (size_t)ch * 1024);
      if (ch * 64 + lane < lu)
        __builtin_amdgcn_global_load_lds((const void*)(src + 16 * lane),
                                         (__attribute__((address_space(3))) void*)&s_u[b * lb + ch * 64], 16, 0, 0);
      ch += NT / 64;
    }
  };
  auto factors = [&](int j) { return fac + (size_t)j * (2 * RC + 2); };   // wave-uniform row of quad j

  LineSums<T, RC> qa[P::IPL];
#pragma unroll
  for (int r = 0; r < P::IPL; ++r) qa[r].clear();

  const V* rc = (const V*)&s_u[pc * lb + (qs * 4 + t) * ur];
  const V* rv = (const V*)&s_u[(TC + pv) * lb + (qs * 4 + t) * ur];
  // this wave's quads: with HS = 2 the first half (which also adds the second one's sums) takes
  // the smaller share
  const int jm = HS == 1 ? nq : nq / 2;
  const int j0 = hf == 0 ? 1 : jm, j1 = hf == 0 ? jm : nq;

  // one step; the first (whose first row quad is quad 0) is instantiated by itself, so that the
  // accumulators of stage 2 stay in place over the loop
  auto step = [&](int st, auto first) {
    constexpr bool kFirst = decltype(first)::value;
    wait_vm<0>();
    lds_barrier();   // the step's rows have landed; stage 2 of the previous step is done with Z
    const bool live = QS == 1 || st * QS + qs < nq;
    LineSums<T, RC> sm;
    if (live) {
      sm.clear();
      // the operands of the next quad are read while the current one is summed
      V na[4], nb[4];
      auto load = [&](int j) {
        __builtin_memcpy(na, __builtin_assume_aligned(rv + 4 * j, 16), 4 * sizeof(V));
        __builtin_memcpy(nb, __builtin_assume_aligned(rc + 4 * j, 16), 4 * sizeof(V));
      };
      auto product = [&](V (&p)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = cmulc(na[k], nb[k]);
      };
      load(hf == 0 ? 0 : j0);
      auto nf = factors(hf == 0 ? 0 : j0);
      if (hf == 0) {
        V p[4];
        product(p);
        const auto f = nf;
        load(j0);
        nf = factors(j0);
        sm.add0(fold_quad0(p), f);
      }
#pragma unroll 1
      for (int j = j0; j < j1; ++j) {
        V p[4];
        product(p);
        const auto f = nf;
        const int jn = min(j + 1, nq - 1);
        load(jn);
        nf = factors(jn);
        sm.add(fold_quad(p), f);
      }
    }
    V* z = s_z + (((P::AL ? hf : 0) * QS + qs) * P::NP + pair) * PS + t * K + RC;
    if constexpr (P::AL) lds_barrier();   // every wave is done with the rows
    if (HS == 1 || P::AL || hf == 1) {
      if (live) {
        z[0] = sm.c(0);
#pragma unroll
        for (int n = 1; n <= RC; ++n) {
          z[n] = plus_i(sm.c(n), sm.s(n));
          z[-n] = minus_i(sm.c(n), sm.s(n));
        }
      }
    }
    lds_barrier();   // every wave is done with the rows
    if constexpr (!P::AL)
      if (st + 1 < nstep) issue(st + 1);
    if constexpr (HS == 2 && !P::AL) {
      if (live && hf == 0) {
        z[0] = cadd(z[0], sm.c(0));
#pragma unroll
        for (int n = 1; n <= RC; ++n) {
          z[n] = cadd(z[n], plus_i(sm.c(n), sm.s(n)));
          z[-n] = cadd(z[-n], minus_i(sm.c(n), sm.s(n)));
          if (n % 3 == 0) asm volatile("" ::: "memory");   // few Z values in registers at a time
        }
      }
      lds_barrier();
    }
    // stage 2
#pragma unroll
    for (int k = 0; k < QS; ++k) {
      const int j2 = st * QS + k;
      if (j2 < nq) {
        const auto f = factors(j2);
#pragma unroll
        for (int r = 0; r < P::IPL; ++r) {
          const int it = min(tid + NT * r, P::NITEM - 1);
          const V* y = s_z + (k * P::NP + it / K) * PS + it % K;
          V p[4] = {y[0], y[K], y[2 * K], y[3 * K]};
#pragma unroll
          for (int b = 1; b < P::NB; ++b) {
            const V* yb = y + b * QS * P::NP * PS;
#pragma unroll
            for (int a = 0; a < 4; ++a) p[a] = cadd(p[a], yb[a * K]);
          }
          if (kFirst && k == 0)
            qa[r].add0(fold_quad0(p), f);
          else
            qa[r].add(fold_quad(p), f);
        }
      }
    }
    if constexpr (P::AL) {
      lds_barrier();   // every wave is done with the sums
      if (st + 1 < nstep) issue(st + 1);
    }
  };
  issue(0);
  step(0, std::true_type{});
#pragma unroll 1
  for (int st = 1; st < nstep; ++st) step(st, std::false_type{});
  // rowtab[n2]: first line of n2 minus its lowest n3, lowest and highest n3 (all counted from 0)
#pragma unroll
  for (int r = 0; r < P::IPL; ++r) {
    const int it = tid + NT * r;
    if (it < P::NITEM) {
      const int pr = it / K, j3 = it % K;
      const size_t pgl = (size_t)(v0 + pr / TC) * ncs + (c0 + pr % TC);
      V* dst = q + (pgl * nt + x1) * (size_t)nl + j3;
      auto put = [&](int n2, V x) {
        const int32_t* e = rowtab + 3 * (n2 + RC);
        if (j3 >= e[1] && j3 <= e[2]) dst[e[0]] = x;
      };
      put(0, qa[r].c(0));
#pragma unroll
      for (int n = 1; n <= RC; ++n) {
        put(n, plus_i(qa[r].c(n), qa[r].s(n)));
        put(-n, minus_i(qa[r].c(n), qa[r].s(n)));
      }
    }
  }
}

// One workgroup per pair, one thread per line (n2, n3) that holds a G of the sphere.  HBM-bound:
// Q is read once, the next quad's planes in flight while the current one is summed.  The frequencies go to
// their places in the sphere's order in LDS and the row leaves in whole lines (32k pairs, float32: K 15, NG
// 2000 0.57 ms, 4.8 TB/s; K 25, NG 8000 2.42 ms, 5.1 TB/s; with 8-byte stores to memory and a wait for the map
// per frequency 0.69 and 3.2); RL false, rows larger than the LDS: straight to memory.
// Quad 0 stands before the loop and the map is read for eight frequencies at a time: with both in one piece the
// larger spheres took twice the registers, up to spills (float64, us: 2048 pairs, RC 12 593 -> 303; 4096 pairs, RC
// 13 519 -> 466, RC 15 2226 -> 1060).
// Float32 sums of small spheres run in float64 (24^3: 1.6e-7 -> 1.1e-7 of the norm, 11 -> 12 us); larger ones would
// hold too many registers (RC 12: 5.4 -> 10.6 ms).
constexpr int kFinishMax = 512;
template <typename T, int RC> using FinishSum = std::conditional_t<RC <= 4, double, T>;
template <typename T, int RC, bool RL>
__global__ __launch_bounds__(kFinishMax) void k_pair_finish(const cx<T>* __restrict__ q,
                                                            const int32_t* __restrict__ chi_map, int ng, int ngp,
                                                            int nt, int nl, FinishSum<T, RC> scale,
                                                            const FinishSum<T, RC>* __restrict__ fac,
                                                            cx<T>* __restrict__ m) {
  using V = cx<T>;
  using A = cx<FinishSum<T, RC>>;
  extern __shared__ __align__(16) unsigned char s_raw[];
  const size_t pair = blockIdx.x;
  const int nq = nt / 4, h = nt / 2;
  const V* src = q + pair * nt * (size_t)nl;
  V* dst = m + pair * ngp;
  V* row = RL ? (V*)s_raw : dst;
  for (int l = threadIdx.x; l < nl; l += blockDim.x) {
    LineSums<FinishSum<T, RC>, RC> s;
    s.clear();
    const V* p0 = src + l;
    V nx[4] = {p0[0], p0[(size_t)(h / 2) * nl], p0[(size_t)h * nl], p0[(size_t)(h + h / 2) * nl]};
    A x[4];
    auto next = [&](int j) {   // quad j's planes come in under the sums of the one before
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = A{nx[k].x, nx[k].y};
      if (j < nq) {
        nx[0] = p0[(size_t)j * nl];
        nx[1] = p0[(size_t)(h - j) * nl];
        nx[2] = p0[(size_t)(h + j) * nl];
        nx[3] = p0[(size_t)(nt - j) * nl];
      }
    };
    next(1);
    s.add0(fold_quad0(x), fac);
#pragma unroll 1
    for (int j = 1; j < nq; ++j) {
      next(j + 1);
      s.add(fold_quad(x), fac + (size_t)j * (2 * RC + 2));
    }
    // the map of up to kGroup frequencies at once: one wait, not one per frequency
    constexpr int kGroup = 8;
#pragma unroll
    for (int n0 = 0; n0 <= RC; n0 += kGroup) {
      int ig[2 * kGroup];
#pragma unroll
      for (int k = 0; k < 2 * kGroup; ++k) {
        const int n = n0 + k / 2;
        ig[k] = n <= RC && (n > 0 || k == 0) ? chi_map[(size_t)(RC + (k % 2 ? -n : n)) * nl + l] : -1;
      }
      if constexpr (RC > 10) asm volatile("" ::: "memory");   // few of the results in registers at a time
      auto put = [&](int k, A v) {
        if (ig[k] >= 0) row[ig[k]] = V{T(v.x * scale), T(v.y * scale)};
      };
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        const int n = n0 + k;
        if (n == 0) put(0, s.c(0));
        if (n > 0 && n <= RC) {
          put(2 * k, plus_i(s.c(n), s.s(n)));
          put(2 * k + 1, minus_i(s.c(n), s.s(n)));
        }
      }
    }
  }
  if constexpr (RL) {
    __syncthreads();
    for (int i = threadIdx.x; i < ngp; i += blockDim.x) dst[i] = i < ng ? row[i] : V{T(0), T(0)};
  } else {
    for (int i = ng + threadIdx.x; i < ngp; i += blockDim.x) dst[i] = V{T(0), T(0)};
  }
}

template <typename T, int RC, typename P>
hipError_t run_shape(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, hipStream_t st) {
  if (nvs % P::TV != 0 || ncs % P::TC != 0 || g.nt > P::NM) return hipErrorInvalidValue;
  const int total = g.nt * (nvs / P::TV) * (ncs / P::TC);
  k_pair_planes<T, RC, P><<<(total + 7) / 8 * 8, P::NT, 0, st>>>((const cx<T>*)psi_v, (const cx<T>*)psi_c, nvs, ncs,
                                                                 g.nt, g.nl, g.d_rowtab, (const T*)g.d_fac64,
                                                                 (cx<T>*)q);
  return hipGetLastError();
}

template <int RC, typename P>
hipError_t run_mfma(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, hipStream_t st) {
  const int nq = g.nt / 4, nch = P::chunks(nq);
  if (nvs % P::TV != 0 || ncs % P::TC != 0 || nq > P::NQM || nch < 1) return hipErrorInvalidValue;
  const int total = g.nt * (nvs / P::TV) * (ncs / P::TC);
  const int cq = (nq + nch - 1) / nch;
  auto inv = [](int d) { return (unsigned)((0x100000000ull + d - 1) / d); };   // u / d = mulhi(u, inv), u < 2^16
  // a fixed grid of one workgroup per CU where only one fits (the next item's rows load under the end of the
  // last one: 16.3 ms against 17.2); where several share a CU, one workgroup per item is as fast
  const int all = (total + 7) / 8 * 8;
  const int blocks = P::WV == 8 ? std::min(all, 256) : all;
  k_pair_planes_mfma<RC, P><<<blocks, P::NT, 0, st>>>((const float2*)psi_v, (const float2*)psi_c, nvs,
                                                                   ncs, g.nt, g.nl, nch, inv(P::row_units(cq)),
                                                                   inv(P::band_units(cq)), g.d_rowtab, g.d_amat,
                                                                   (float2*)q);
  return hipGetLastError();
}

// Shapes, per 32k-pair launch on one MI355X (before: both sums' partial results exchanged through LDS).
// float32, up to RC = 7: two row quads per wave, 64 accumulators, three waves per SIMD, workgroups of four
// waves: RC 7 on 44^3 2.06 ms (before 2.6; with one row quad per wave and two waves per SIMD 2.3, with
// workgroups of eight waves 2.5).  From RC = 8 a slot pair has twice the accumulators: four row quads per
// wave, two waves per SIMD, one workgroup of eight waves per CU over a fixed grid: RC 9 on 60^3 8.1 ms
// (before 10.3; workgroups of four waves 8.8), RC 12 on 80^3 16.2 ms (before 22; 17.9).
// float64: half a line per lane, at most 256 registers per lane for two waves per SIMD.
// Up to RC 7: workgroups of four waves, two per CU; RC 7 on 44^3 4.6 ms.  The rows of more than 64 points leave no
// room for the sums beside them, so these take the rows' place (4096 pairs, RC 7 on 72 points 3.35 -> 2.12 ms, RC 5
// on 68 2.78 -> 1.76).  Up to 64 points the next rows load under the sums.
// Up to RC 4 and 32 points the row buffers are half as long and the registers suffice for three waves per SIMD
// (24^3, RC 4 on 20^3, 3840 pairs: 74 us, 93 with two).
// RC 8 and 9: 32 pairs need two of stage 2's sums per lane, more than two waves' registers; 16 pairs and four (beyond
// 76 points three) row quads per step need one, one workgroup of eight (six) waves per CU, the sums in the rows'
// place: RC 9 on 60^3 16.6 ms (one wave per SIMD with 32 pairs 19.9); 4096 pairs, RC 8 on 68 points 2.82 (3.43), RC 9
// on 72 3.24 (3.89); 2048 pairs, RC 9 on 96 4.17 (4.21), on 104 5.14 (6.61).
// From RC 10 one wave per SIMD.  From RC 12 32 pairs' sums are more than its registers too: 16 pairs and two row
// quads, as far as the LDS allows (4096 pairs, RC 15 on 48 points 7.5 -> 2.46 ms, on 76 19.4 -> 7.0; RC 12 on 64 5.2 ->
// 4.0, 2048 pairs on 96 6.7 -> 5.4); RC 10 and 11 fit with 32.
template <typename T, int RC>
hipError_t run_planes(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, hipStream_t st) {
  if constexpr (std::is_same<T, float>::value) {
    if constexpr (RC <= 7)
      return run_mfma<RC, MfmaShape<RC, 2, 4, 4, 8, 1280, 3>>(g, psi_v, psi_c, nvs, ncs, q, st);
    else
      return run_mfma<RC, MfmaShape<RC, 4, 8, 4, 8, 4032, 2>>(g, psi_v, psi_c, nvs, ncs, q, st);
  } else {
    if constexpr (RC <= 4) {
      if (g.nt <= 32)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 32, 3>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    if constexpr (RC <= 7) {
      if (g.nt <= 64)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 64, 2>>(g, psi_v, psi_c, nvs, ncs, q, st);
      return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 104, 2, true>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    if constexpr (RC == 8 || RC == 9) {
      if (g.nt <= 76)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 4, 4, 4, 76, 2, true>>(g, psi_v, psi_c, nvs, ncs, q, st);
      return run_shape<T, RC, PlaneShape<T, RC, 2, 3, 4, 4, 104, 2, true>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    if constexpr (RC >= 12) {
      constexpr int nm = RC == 12 ? 104 : RC == 15 ? 88 : 96;
      if (g.nt <= nm)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 2, 4, 4, nm, 1>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    if constexpr (RC >= 10)
      return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 128, 1>>(g, psi_v, psi_c, nvs, ncs, q, st);
  }
}

template <typename T, int RC>
hipError_t run_finish(const Geom& g, const void* q, int npair, void* m, hipStream_t st) {
  using A = FinishSum<T, RC>;
  const A scale = A(1.0 / ((double)g.nt * g.nt * g.nt));
  const A* fac = std::is_same<A, float>::value ? (const A*)g.d_fac32 : (const A*)g.d_fac64;
  const int passes = (g.nl + kFinishMax - 1) / kFinishMax;
  const int threads = ((g.nl + passes - 1) / passes + 63) / 64 * 64;
  auto run = [&](auto f, size_t lds) {
    f<<<npair, threads, lds, st>>>((const cx<T>*)q, g.d_chi_map, g.ng, g.ngp, g.nt, g.nl, scale, fac, (cx<T>*)m);
  };
  const size_t lds = (size_t)g.ng * sizeof(cx<T>);
  if (lds <= kLdsBytes) {
    static OncePerDevice done;
    const hipError_t allowed = allow_whole_lds(reinterpret_cast<const void*>(&k_pair_finish<T, RC, true>), done);
    if (allowed != hipSuccess) return allowed;
    run(k_pair_finish<T, RC, true>, lds);
  } else {
    run(k_pair_finish<T, RC, false>, 0);
  }
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_pair_planes(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q,
                              hipStream_t st) {
  switch (g.rchi) {
#define X(rc) \
  case rc: return run_planes<T, rc>(g, psi_v, psi_c, nvs, ncs, q, st);
    GW_RC_CASES(X)
#undef X
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_pair_finish(const Geom& g, const void* q, int npair, void* m, hipStream_t st) {
  switch (g.rchi) {
#define X(rc) \
  case rc: return run_finish<T, rc>(g, q, npair, m, st);
    GW_RC_CASES(X)
#undef X
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_pair_planes<double>(const Geom&, const void*, const void*, int, int, void*, hipStream_t);
template hipError_t launch_pair_planes<float>(const Geom&, const void*, const void*, int, int, void*, hipStream_t);
template hipError_t launch_pair_finish<double>(const Geom&, const void*, int, void*, hipStream_t);
template hipError_t launch_pair_finish<float>(const Geom&, const void*, int, void*, hipStream_t);

}  // namespace gw
