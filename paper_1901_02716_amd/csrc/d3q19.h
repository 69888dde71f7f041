// Row pieces shared by the fast and the general D3Q19 step for gfx950: the
// link values of a node (Eq. (2), deviation form, times 36), the rolling plane
// accumulators they are pushed into, and the finalisation of a row (Eqs.
// (4)-(5)). T is the arithmetic type of the storage codec (FP64 or FP32). A link
// value and the order of every sum are the same wherever these are used.
#pragma once

#include <type_traits>

#include "device.h"

namespace maclab {

template <class C, int KX>
struct alignas(sizeof(typename C::elem) * KX) RowVec {
  typename C::elem v[KX];
};

template <class T, int KX>
struct PlaneAcc {
  T r[KX], mx[KX], my[KX], mz[KX];  // 36 * (drho', m')
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int e = 0; e < KX; ++e) r[e] = mx[e] = my[e] = mz[e] = (T)0;
  }
};

// Finalises the KX nodes of one row of destination plane accumulators a and
// encodes them: drho' = r / 36 and u~' = (m + 36 g) / (36 rho_ref + r)
// (Eqs. (4)-(5) with the sums carried times 36). The accumulators hold the
// sums times K = the codec's density scale (a power of two; see node_links),
// so K drho' = div36(a.r) and S u~' = S (a.m + 36 K g) / (36 K rho_ref + a.r)
// for the velocity scale S: every scale is exact, and the stored values
// carry them. Node e of the lane (dense node index node0 + e) draws its own
// rounding bits, sr_node_bits(key, node0 + e), the bits every kernel gives
// that node in that step, so the rounding decisions of neighbouring nodes are
// independent.
template <class C, int KX>
__device__ __forceinline__ void finalize_row(const PlaneAcc<typename C::T, KX>& a, typename C::T rho_ref,
                                             typename C::T g36x, typename C::T g36y, typename C::T g36z,
                                             uint32_t key, int64_t node0, RowVec<C, KX> (&o)[4]) {
#pragma clang fp contract(off)
  using T = typename C::T;
  constexpr T K = C::kScaleRho;
  T v[4][KX];
  uint32_t bits[KX];
#pragma unroll
  for (int e = 0; e < KX; ++e) {
    const T inv = recip<T>(K * ((T)36 * rho_ref) + a.r[e]) * C::kScaleU;
    v[0][e] = div36(a.r[e]);
    v[1][e] = (a.mx[e] + K * g36x) * inv;
    v[2][e] = (a.my[e] + K * g36y) * inv;
    v[3][e] = (a.mz[e] + K * g36z) * inv;
    bits[e] = needs_rng<C>::value ? sr_node_bits(key, node0 + e) : 0u;
  }
  if constexpr (sizeof(typename C::elem) == 2 && KX % 2 == 0) {
    struct Words { uint32_t w[KX / 2]; };
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      Words w;
#pragma unroll
      for (int e = 0; e < KX; e += 2) w.w[e / 2] = C::enc2_scaled(v[f][e], v[f][e + 1], f, bits[e], bits[e + 1]);
      o[f] = __builtin_bit_cast(RowVec<C, KX>, w);
    }
  } else {
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int e = 0; e < KX; ++e) o[f].v[e] = C::enc_scaled(v[f][e], f, bits[e]);
  }
}

// The 19 link values of one node, times 36, in deviation form (Eq. (2)):
//   36 F^_a = wnum_a [a + c.b + sum_i c_i^2 q_ii + sum_{i<j} c_i c_j q_ij]
// with a = drho - 1.5 rho |u|^2, b = 3 rho u, q_ii = 4.5 rho u_i^2,
// q_ij = 9 rho u_i u_j. The six axis links are carried halved (h = F/2).
template <class T>
struct Links {
  T f0, hxp, hxm, hyp, hym, hzp, hzm;
  T pp0, mm0, pm0, mp0;  // (1,1,0) (-1,-1,0) (1,-1,0) (-1,1,0)
  T p0p, m0m, p0m, m0p;  // (1,0,1) (-1,0,-1) (1,0,-1) (-1,0,1)
  T zpp, zmm, zpm, zmp;  // (0,1,1) (0,-1,-1) (0,1,-1) (0,-1,1)
};

// Contraction is off and every FMA is written out, so a link value has the
// same bits whichever wavefront (output or halo row) computes it and the
// result does not depend on the tiling.
//
// The inputs are the stored fields times the codec's storage scales, d =
// K drho and v = S u~ (K, S powers of two; 1 for FP32 storage), and every
// link value comes out times K: with r3 = (3 K / S) rho each b and each
// product c_ij = b_i v_j carries K resp. K S, and the constants that multiply
// the c_ij are divided by S. Powers of two commute with every rounding, so
// the scaled links are K times the unscaled ones, bit for bit.
template <class C>
__device__ __forceinline__ void node_links(typename C::T dr, typename C::T ux, typename C::T uy,
                                           typename C::T uz, typename C::T rho_ref, Links<typename C::T>& L) {
#pragma clang fp contract(off)
  using T = typename C::T;
  constexpr T K = C::kScaleRho, S = C::kScaleU;
  const T rho = K == (T)1 ? rho_ref + dr : fma_t(dr, (T)1 / K, rho_ref);
  const T r3 = ((T)3 * K / S) * rho;
  const T bx = r3 * ux, by = r3 * uy, bz = r3 * uz;    // 3 rho u          (times K)
  const T cxx = bx * ux, cyy = by * uy, czz = bz * uz;  // 3 rho u_i^2      (times K S; q_ii = 1.5 c_ii)
  const T cxy = bx * uy, cxz = bx * uz, cyz = by * uz;  // 3 rho u_i u_j    (times K S; q_ij = 3 c_ij)
  const T a = fma_t((cxx + cyy) + czz, (T)-0.5 / S, dr);
  const T sx = fma_t(cxx, (T)1.5 / S, a), sy = fma_t(cyy, (T)1.5 / S, a),
              sz = fma_t(czz, (T)1.5 / S, a);
  L.f0 = (T)12 * a;
  L.hxp = sx + bx;
  L.hxm = sx - bx;
  L.hyp = sy + by;
  L.hym = sy - by;
  L.hzp = sz + bz;
  L.hzm = sz - bz;
  T t, p, m, u, v;
  t = fma_t(cyy, (T)1.5 / S, sx);  // a + q_xx + q_yy
  p = fma_t(cxy, (T)3 / S, t);
  m = fma_t(cxy, (T)-3 / S, t);
  u = bx + by;
  v = bx - by;
  L.pp0 = p + u;
  L.mm0 = p - u;
  L.pm0 = m + v;
  L.mp0 = m - v;
  t = fma_t(czz, (T)1.5 / S, sx);  // a + q_xx + q_zz
  p = fma_t(cxz, (T)3 / S, t);
  m = fma_t(cxz, (T)-3 / S, t);
  u = bx + bz;
  v = bx - bz;
  L.p0p = p + u;
  L.m0m = p - u;
  L.p0m = m + v;
  L.m0p = m - v;
  t = fma_t(czz, (T)1.5 / S, sy);  // a + q_yy + q_zz
  p = fma_t(cyz, (T)3 / S, t);
  m = fma_t(cyz, (T)-3 / S, t);
  u = by + bz;
  v = by - bz;
  L.zpp = p + u;
  L.zmm = p - u;
  L.zpm = m + v;
  L.zmp = m - v;
}

// The c_y = 0 links of a row into the plane accumulators: rest, +-z, and the
// links moving in x, which cross to the neighbouring lane at the lane edges.
// Plane z+1 (ap) is first touched here, so it is assigned.
template <class T, int KX>
__device__ __forceinline__ void add_own_row(const T (&f0)[KX], const T (&hzp)[KX], const T (&hzm)[KX],
                                            const T (&hxp)[KX], const T (&p0p)[KX], const T (&p0m)[KX],
                                            const T (&hxm)[KX], const T (&m0p)[KX], const T (&m0m)[KX], T in_hxp,
                                            T in_p0p, T in_p0m, T in_hxm, T in_m0p, T in_m0m, PlaneAcc<T, KX>& am,
                                            PlaneAcc<T, KX>& ac, PlaneAcc<T, KX>& ap) {
#pragma clang fp contract(off)
#pragma unroll
  for (int d = 0; d < KX; ++d) {
    // links arriving at node d from d-1 (moving +x) and d+1 (moving -x)
    const T Phx = d > 0 ? hxp[d - 1] : in_hxp, Pzp = d > 0 ? p0p[d - 1] : in_p0p,
                Pzm = d > 0 ? p0m[d - 1] : in_p0m;
    const T Mhx = d < KX - 1 ? hxm[d + 1] : in_hxm, Mzp = d < KX - 1 ? m0p[d + 1] : in_m0p,
                Mzm = d < KX - 1 ? m0m[d + 1] : in_m0m;
    // plane z: rest and +-x
    const T A = Phx + Mhx, B = Phx - Mhx;
    ac.r[d] += fma_t((T)2, A, f0[d]);
    ac.mx[d] = fma_t((T)2, B, ac.mx[d]);
    // plane z+1: +z, +x+z, -x+z (first contributions to this plane)
    const T sp = fma_t((T)2, hzp[d], Pzp + Mzp);
    ap.r[d] = sp;
    ap.mz[d] = sp;
    ap.mx[d] = Pzp - Mzp;
    // plane z-1: -z, +x-z, -x-z
    const T sm = fma_t((T)2, hzm[d], Pzm + Mzm);
    am.r[d] += sm;
    am.mz[d] -= sm;
    am.mx[d] += Pzm - Mzm;
  }
}

template <class T, int KX>
__device__ __forceinline__ void own_row_links(const T (&f0)[KX], const T (&hzp)[KX], const T (&hzm)[KX],
                                              const T (&hxp)[KX], const T (&p0p)[KX], const T (&p0m)[KX],
                                              const T (&hxm)[KX], const T (&m0p)[KX], const T (&m0m)[KX],
                                              PlaneAcc<T, KX>& am, PlaneAcc<T, KX>& ac, PlaneAcc<T, KX>& ap) {
  const T in_hxp = dpp_from_left(hxp[KX - 1]), in_p0p = dpp_from_left(p0p[KX - 1]),
              in_p0m = dpp_from_left(p0m[KX - 1]);
  const T in_hxm = dpp_from_right(hxm[0]), in_m0p = dpp_from_right(m0p[0]), in_m0m = dpp_from_right(m0m[0]);
  add_own_row<T, KX>(f0, hzp, hzm, hxp, p0p, p0m, hxm, m0p, m0m, in_hxp, in_p0p, in_p0m, in_hxm, in_m0p, in_m0m, am,
                     ac, ap);
}

// Adds the contributions sent through LDS by the rows below (c_y = +1 links,
// S = +1) and above (c_y = -1 links, S = -1): s and d in the plane of the
// source, vp / vm moving to planes z+1 / z-1. The y momentum of plane z+1 is
// first touched by the row below, so it is assigned.
template <class T, int KX, int S>
__device__ __forceinline__ void add_sent(T s, T d, T vp, T vm, int e, PlaneAcc<T, KX>& am,
                                         PlaneAcc<T, KX>& ac, PlaneAcc<T, KX>& ap) {
#pragma clang fp contract(off)
  ac.r[e] += s;
  ac.mx[e] += d;
  ap.r[e] += vp;
  ap.mz[e] += vp;
  am.r[e] += vm;
  am.mz[e] -= vm;
  if constexpr (S > 0) {
    ac.my[e] += s;
    ap.my[e] = vp;
    am.my[e] += vm;
  } else {
    ac.my[e] -= s;
    ap.my[e] -= vp;
    am.my[e] -= vm;
  }
}

// Raw (stored) elements of one row of the four fields.
template <class C, int KX>
struct RawRow {
  RowVec<C, KX> f[4];
};

// c ? a : b on the bit patterns. A plain conditional between two elements of
// one row is turned by the compiler into a load at a selected index, which
// puts 16-bit rows in scratch memory.
template <class E>
__device__ __forceinline__ E pick_bits(bool c, E a, E b) {
  using U = std::conditional_t<sizeof(E) == 2, uint16_t, std::conditional_t<sizeof(E) == 4, uint32_t, uint64_t>>;
  static_assert(sizeof(U) == sizeof(E), "element size");
  const U m = (U)0 - (U)c;
  return __builtin_bit_cast(E, (U)((__builtin_bit_cast(U, a) & m) | (__builtin_bit_cast(U, b) & (U)~m)));
}


}  // namespace maclab
