// Pair transform: the matrix element of Eq. (chi0),
//   M_vc(G) = (1/N) sum_r conj(u_v(r)) u_c(r) exp(iG.r),   G in the dielectric sphere,
// formed as the product of two real-space bands followed by a forward transform
// that only produces the K = 2 RC + 1 frequencies per axis the sphere needs, on the smallest
// alias-free grid (fold.h).
//
// k_pair_planes (one x1 plane, TV valence x TC conduction bands per workgroup) walks the plane's
// quads of x2 rows:
//   stage 1, per lane one (pair, x2 row): the product along x3 and the folded x3 sums ->
//     Z[pair][row][n3] in LDS;
//   stage 2, per lane (pair, n3): the folded x2 sums over the quad's four rows, accumulated over
//     the quads in registers;
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

// Shape of a planes workgroup.  HS: waves that share a line's x3 quads (partial sums added in LDS);
// QS: quads of x2 rows per step; NM: largest grid (the LDS row buffers).
template <typename T, int RC, int HS_, int QS_, int TV_, int TC_, int NM_, int MINW_>
struct PlaneShape {
  static constexpr int HS = HS_, QS = QS_, TV = TV_, TC = TC_, NM = NM_, MINW = MINW_;
  static constexpr int K = 2 * RC + 1;
  static constexpr int NP = TV * TC;               // pairs
  static constexpr int PG = NP / 16;               // waves per row quad and half: 16 pairs x 4 rows
  static constexpr int NT = 64 * HS * QS * PG;
  static constexpr int PS = 4 * K + 1;             // Z of a pair and quad: [row][n3], odd stride
  static constexpr int PADE = 16 / (int)sizeof(cx<T>);   // row padding (complex values): odd 16-byte units
  // row buffer: per band its QS quads of rows and one 16-byte unit (an odd stride between bands)
  static constexpr int NU = (TC + TV) * (QS * 4 * (NM + PADE) / PADE + 1);
  static constexpr int NZ = QS * NP * PS;
  static constexpr size_t lds0 = (size_t)NU * 16 + (size_t)NZ * sizeof(cx<T>);
  // the MFMA factors of every quad in LDS too, where they fit
  static constexpr int NF = sizeof(T) == 4 && lds0 + NM / 4 * 256 <= 160 * 1024 ? NM / 4 * 64 : 0;
  static constexpr size_t lds = lds0 + 4 * NF;
  static constexpr int NITEM = NP * K;
  static constexpr int IPL = (NITEM + NT - 1) / NT;
  static_assert(lds <= 160 * 1024, "planes workgroup exceeds the LDS");
};

template <typename T, int RC> using Sums = std::conditional_t<std::is_same<T, float>::value, MfmaSums<RC>, LineSums<T, RC>>;

template <typename T, int RC, typename P>
__global__ __launch_bounds__(P::NT, P::MINW) void k_pair_planes(const cx<T>* __restrict__ psi_v,
                                                                const cx<T>* __restrict__ psi_c, int nvs, int ncs,
                                                                int nt, int nl, const int32_t* __restrict__ rowtab,
                                                                const T* __restrict__ fac, cx<T>* __restrict__ q) {
  using V = cx<T>;
  constexpr bool kMfma = std::is_same<T, float>::value;
  constexpr int K = P::K, NT = P::NT, TV = P::TV, TC = P::TC, HS = P::HS, QS = P::QS, PS = P::PS;
  constexpr int EPU = P::PADE;   // complex values per 16-byte unit
  __shared__ __align__(16) uint4 s_u[P::NU];   // [band: TC columns, TV valence][quad][t][row], band stride odd
  __shared__ __align__(16) V s_z[P::NZ];   // [quad][pair][t][n3]
  __shared__ float s_f[P::NF > 0 ? P::NF : 1];

  // The workgroups of one x1 plane read the same bands, so each XCD (workgroup b runs on XCD
  // b mod 8) takes a contiguous run of the plane-major order and its L2 holds about one plane.
  const int nbc = ncs / TC, nbv = nvs / TV;
  const int total = nt * nbc * nbv;
  const int per = (total + 7) / 8;
  const int item = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per || item >= total) return;
  const int x1 = item / (nbc * nbv);
  const int pb = item % (nbc * nbv);
  const int c0 = (pb % nbc) * TC;
  const int v0 = (pb / nbc) * TV;

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
  // factors of quad j: one register per lane (MFMA blocks), or a wave-uniform row
  if constexpr (P::NF > 0)
    for (int i = tid; i < nq * 64; i += NT) s_f[i] = fac[i];   // visible after the first step's barrier
  auto factors = [&](int j) {
    if constexpr (P::NF > 0)
      return s_f[64 * j + lane];
    else if constexpr (kMfma)
      return fac[64 * j + lane];
    else
      return fac + (size_t)j * (2 * RC + 2);
  };

  Sums<T, RC> qa[P::IPL];
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
    Sums<T, RC> sm;
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
    V* z = s_z + (qs * P::NP + pair) * PS + t * K + RC;
    if (HS == 1 || hf == 1) {
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
    if (st + 1 < nstep) issue(st + 1);
    if constexpr (HS == 2) {
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
          const V p[4] = {y[0], y[K], y[2 * K], y[3 * K]};
          if (kFirst && k == 0)
            qa[r].add0(fold_quad0(p), f);
          else
            qa[r].add(fold_quad(p), f);
        }
      }
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
// Q is read once, the next quad's planes in flight while the current one is summed.
constexpr int kFinishMax = 512;
template <typename T, int RC>
__global__ __launch_bounds__(kFinishMax) void k_pair_finish(const cx<T>* __restrict__ q,
                                                            const int32_t* __restrict__ chi_map, int ng, int ngp,
                                                            int nt, int nl, T scale, const T* __restrict__ fac,
                                                            cx<T>* __restrict__ m) {
  using V = cx<T>;
  const size_t pair = blockIdx.x;
  const int nq = nt / 4, h = nt / 2;
  const V* src = q + pair * nt * (size_t)nl;
  V* dst = m + pair * ngp;
  for (int l = threadIdx.x; l < nl; l += blockDim.x) {
    LineSums<T, RC> s;
    s.clear();
    const V* p0 = src + l;
    V nx[4] = {p0[0], p0[(size_t)(h / 2) * nl], p0[(size_t)h * nl], p0[(size_t)(h + h / 2) * nl]};
#pragma unroll 1
    for (int j = 0; j < nq; ++j) {
      V x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = nx[k];
      if (j + 1 < nq) {
        nx[0] = p0[(size_t)(j + 1) * nl];
        nx[1] = p0[(size_t)(h - j - 1) * nl];
        nx[2] = p0[(size_t)(h + j + 1) * nl];
        nx[3] = p0[(size_t)(nt - j - 1) * nl];
      }
      if (j == 0)
        s.add0(fold_quad0(x), fac);
      else
        s.add(fold_quad(x), fac + (size_t)j * (2 * RC + 2));
    }
    auto put = [&](int n1, V v) {
      const int ig = chi_map[(size_t)(n1 + RC) * nl + l];
      if (ig >= 0) dst[ig] = V{v.x * scale, v.y * scale};
    };
    put(0, s.c(0));
#pragma unroll
    for (int n = 1; n <= RC; ++n) {
      put(n, plus_i(s.c(n), s.s(n)));
      put(-n, minus_i(s.c(n), s.s(n)));
    }
  }
  for (int i = ng + threadIdx.x; i < ngp; i += blockDim.x) dst[i] = V{T(0), T(0)};
}

template <typename T, int RC, typename P>
hipError_t run_shape(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, hipStream_t st) {
  if (nvs % P::TV != 0 || ncs % P::TC != 0 || g.nt > P::NM) return hipErrorInvalidValue;
  const int total = g.nt * (nvs / P::TV) * (ncs / P::TC);
  const T* fac = std::is_same<T, float>::value ? (const T*)g.d_amat : (const T*)g.d_fac64;
  k_pair_planes<T, RC, P><<<(total + 7) / 8 * 8, P::NT, 0, st>>>((const cx<T>*)psi_v, (const cx<T>*)psi_c, nvs, ncs,
                                                                 g.nt, g.nl, g.d_rowtab, fac, (cx<T>*)q);
  return hipGetLastError();
}

// Shape of the planes kernel, per 32k-pair launch on one MI355X (before: the radix-split kernels
// on the stated grid).  float32 up to RC = 7: with a grid of at most 52 points two workgroups of
// eight waves share a CU (four waves per SIMD, form 2): RC 7 on 44^3 2.6 ms, 3.0 for form 1, 4.0 for
// form 3 (72^3 before: 8.7); on larger grids its rows would not leave room for a second workgroup,
// and the 64 pairs of form 1, with a whole line per lane, take over.  From RC = 8 the 64 accumulators
// per (pair, n3) item allow two waves per SIMD and one item for half the threads only with 32
// pairs per eight waves: RC 9 on 60^3 10.3 ms (96^3 before: 23), RC 12 on 80^3 22 ms (128^3
// before: 61).  float64: four waves, half a line per lane; RC 7 on 44^3 4.7 ms (72^3 before: 17.4),
// RC 9 on 60^3 20.3 (96^3 before: 68; one wave per SIMD beyond RC 7).
template <typename T, int RC>
hipError_t run_planes(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, int form,
                      hipStream_t st) {
  if constexpr (std::is_same<T, float>::value) {
    if constexpr (RC <= 7) {
      if (g.nt <= 52 && form != 1 && form != 3)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 2, 4, 8, 52, 4>>(g, psi_v, psi_c, nvs, ncs, q, st);
      if (form != 3 && ncs % 16 == 0) {
        if (g.nt <= 68)
          return run_shape<T, RC, PlaneShape<T, RC, 1, 1, 4, 16, 68, 2>>(g, psi_v, psi_c, nvs, ncs, q, st);
        return run_shape<T, RC, PlaneShape<T, RC, 1, 1, 4, 16, 128, 1>>(g, psi_v, psi_c, nvs, ncs, q, st);
      }
    }
    if constexpr (RC == 15) {   // the two-quad buffers of 128 points would not fit the LDS
      if (g.nt > 124) return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 128, 1>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    return run_shape<T, RC, PlaneShape<T, RC, 2, 2, 4, 8, RC == 15 ? 124 : 128, 2>>(g, psi_v, psi_c, nvs, ncs, q, st);
  } else {
    if constexpr (RC <= 7) {
      if (g.nt <= 64)
        return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 64, 2>>(g, psi_v, psi_c, nvs, ncs, q, st);
    }
    return run_shape<T, RC, PlaneShape<T, RC, 2, 1, 4, 8, 128, 1>>(g, psi_v, psi_c, nvs, ncs, q, st);
  }
}

template <typename T, int RC>
hipError_t run_finish(const Geom& g, const void* q, int npair, void* m, hipStream_t st) {
  const T scale = T(1.0 / ((double)g.nt * g.nt * g.nt));
  const T* fac = std::is_same<T, float>::value ? (const T*)g.d_fac32 : (const T*)g.d_fac64;
  const int passes = (g.nl + kFinishMax - 1) / kFinishMax;
  const int threads = ((g.nl + passes - 1) / passes + 63) / 64 * 64;
  k_pair_finish<T, RC><<<npair, threads, 0, st>>>((const cx<T>*)q, g.d_chi_map, g.ng, g.ngp, g.nt, g.nl, scale, fac,
                                                  (cx<T>*)m);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_pair_planes(const Geom& g, const void* psi_v, const void* psi_c, int nvs, int ncs, void* q, int form,
                              hipStream_t st) {
  switch (g.rchi) {
#define X(rc) \
  case rc: return run_planes<T, rc>(g, psi_v, psi_c, nvs, ncs, q, form, st);
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

template hipError_t launch_pair_planes<double>(const Geom&, const void*, const void*, int, int, void*, int,
                                               hipStream_t);
template hipError_t launch_pair_planes<float>(const Geom&, const void*, const void*, int, int, void*, int,
                                              hipStream_t);
template hipError_t launch_pair_finish<double>(const Geom&, const void*, int, void*, hipStream_t);
template hipError_t launch_pair_finish<float>(const Geom&, const void*, int, void*, hipStream_t);

}  // namespace gw
