// Node pieces shared by the D2Q9 step kernels for gfx950: the moments of a
// node's equilibrium and what it sends along x.
#pragma once

#include "device.h"

namespace maclab {

// The D2Q9 weights are a tensor product, 36 w_a = (6 w_x(c_x)) (6 w_y(c_y))
// with 6 w(0) = 4 and 6 w(+-1) = 1, and the link values of Eq. (2) in the
// deviation form F^_a = f_eq_a - w_a rho_ref are, times 36,
//   36 F^_a = (6 w_x)(6 w_y) [a + c_x bx + c_y by + 1.5 (c_x^2 cxx + c_y^2 cyy) + 3 c_x c_y cxy]
// with rho = rho_ref + drho, bx = 3 rho u_x, by = 3 rho u_y, cxx = bx u_x,
// cyy = by u_y, cxy = bx u_y and a = drho - (cxx + cyy) / 2. So the gather of
// Eqs. (4)-(5) runs as a pass along x and a pass along y over the six
// moments of each node instead of over its nine links. Along x, node x
// receives from x-1 and x+1 (c_x = +1 from the left, -1 from the right)
//   R0 = a + bx + 1.5 cxx,  R1 = by + 3 cxy,  R2 = cyy   (sent to the right)
//   L0 = a - bx + 1.5 cxx,  L1 = by - 3 cxy,  L2 = cyy   (sent to the left)
// and forms, per power of c_y, the x-gathered density (T) and x momentum (U)
// terms of its row:
//   T0 = 4 a + R0' + L0',  T1 = 4 by + R1' + L1',  T2 = 1.5 (4 cyy + R2' + L2')
//   U0 = R0' - L0',        U1 = R1' - L1',         U2 = 1.5 (R2' - L2').
// Along y the row above receives T0 + T1 + T2 (density and y momentum) and
// U0 + U1 + U2 (x momentum), the row below T0 - T1 + T2 (density, minus y
// momentum) and U0 - U1 + U2, and the row itself 4 T0 and 4 U0: together
// 36 drho' and 36 m' of Eqs. (4)-(5).
template <class T>
struct Mom2 {
  T a, bx, by, cxx, cyy, cxy;
};

template <class T>
__device__ __forceinline__ void moments2(T dr, T ux, T uy, T rho_ref, Mom2<T>& M) {
#pragma clang fp contract(off)
  const T rho = rho_ref + dr;
  const T r3 = (T)3 * rho;
  M.bx = r3 * ux;
  M.by = r3 * uy;
  M.cxx = M.bx * ux;
  M.cyy = M.by * uy;
  M.cxy = M.bx * uy;
  M.a = fma_t(M.cxx + M.cyy, (T)-0.5, dr);
}

// What a node sends along x: to the right (R0, R1; R2 = cyy) and to the
// left (L0, L1; L2 = cyy).
template <class T>
struct Send2 {
  T r0, r1, l0, l1, c2;
};

template <class T>
__device__ __forceinline__ Send2<T> send2(const Mom2<T>& M) {
#pragma clang fp contract(off)
  Send2<T> S;
  const T s = fma_t(M.cxx, (T)1.5, M.a);
  S.r0 = s + M.bx;
  S.l0 = s - M.bx;
  S.r1 = fma_t(M.cxy, (T)3, M.by);
  S.l1 = fma_t(M.cxy, (T)-3, M.by);
  S.c2 = M.cyy;
  return S;
}

template <class E, int KX>
struct alignas(sizeof(E) * KX) RowVec2 {
  E v[KX];
};

}  // namespace maclab
