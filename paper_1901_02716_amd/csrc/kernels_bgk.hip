// The lattice BGK scheme the paper starts from, Eq. (1) with relaxation time
// tau = 1, on gfx950: the Q populations of every node are stored, and a step
// streams them and relaxes them fully to the local equilibrium Eq. (2),
//
//   f_a(x + c_a, t + 1) = f_a(x, t) - (f_a(x, t) - f_eq_a(x, t)) / tau
//                       = f_eq_a(x, t)                         (tau = 1).
//
// This is the scheme MacLAB replaces: with tau = 1 the stored populations
// are exactly the equilibria of the macroscopic state, so they carry nothing
// that rho and u do not (Methods, Eqs. (9)-(10)). Both schemes give the same
// rho and u up to rounding; this one moves 2 Q values per node and step
// instead of 2 (d + 1).
//
// Storage: Q planes of `plane` elements, node (i, j, k) at i + nx (j + ny k)
// (no row padding), holding the post-collision populations as deviations
// F_a - w_a rho_ref (FP64 or FP32), so that sums of them stay small, as in
// the MacLAB state. Fixed (boundary) nodes hold f_eq(rho_b, u_b) in both
// buffers, and a step leaves their values as they are.
#include "internal.h"

namespace maclab {

namespace {

// KX neighbouring values of a plane, at any element: rows are not padded, and
// the streaming shift moves a vector by one element.
template <class T, int KX>
struct Vec {
  typedef T type __attribute__((ext_vector_type(KX), aligned(sizeof(T))));
};
template <class T>
struct Vec<T, 1> {
  using type = T;
};

// One wavefront per x-row, four rows per workgroup; a lane holds KX
// neighbouring nodes. The step pulls: destination x gathers population a from
// its upstream node x - c_a, so every stored population is read exactly once
// per step, in one vector load a link shifted by c_x.
//
// Bound: HBM (2 Q values a node). 16-byte accesses keep four times the bytes in
// flight per load of a wavefront: D3Q19 FP32 256^3 587 us a step with one node
// per lane, 485 with four (5.1 of the 6.75 TB/s of a copy; a copy has 2 streams,
// this 38); 251^3, whose rows end in part of a vector, 884 and 526; D2Q9 1024^2
// 31 and 13.4. Fewer workgroups on a CU change the time by under 3%.
//
// Stores: past the caches for a state that does not stay in the memory-side cache
// between steps (256^3 485 us, 500 device-scope, 504 cached), else device-scope, which
// leaves it there for the next step (D2Q9 1024^2 13.5 us, 19.3 non-temporal; D3Q19
// 64^3 7.0, 9.0). The end of a row is stored as the rest of it is: non-temporal among
// device-scope stores it cost 164 us a step against 94 (D3Q19 FP32 131^3).
//
// What a shifted vector takes from outside the row is replaced: on a periodic
// axis by the value across the wrap. A fixed node at a row's end is stored back
// with its own value, so that a lane's nodes are one vector store.
//
// Every FMA is written out, so that the populations have the same bits in every form of
// the kernel: left to the compiler, c.u of a diagonal link and the terms of phi were
// fused differently from one form to the next.
template <int Q, class T, int KX, bool TAIL, bool NT>
__global__ __launch_bounds__(256) void bgk_step_kernel(const T* __restrict__ src, T* __restrict__ dst, BgkParams p) {
#pragma clang fp contract(off)
  using Lt = Lattice<Q>;
  using V = typename Vec<T, KX>::type;
  const int64_t rows = p.ny * p.nz;
  // workgroups go to the eight XCDs in turn: give each XCD a contiguous
  // range of row groups, so neighbouring rows share its L2
  const int64_t nb = gridDim.x, bid = blockIdx.x;
  const int64_t per = nb >> 3, rem = nb & 7, xcd = bid & 7;
  const int64_t grp = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
  // One node per lane: a row is short, and its addresses are formed faster per lane than
  // in the scalar unit (twice the instructions: 4x60x60 FP32 7.4 us a step against 6.6).
  const int64_t row = grp * 4 + (KX == 1 ? (int)threadIdx.y : __builtin_amdgcn_readfirstlane((int)threadIdx.y));
  if (row >= rows) return;
  // (a 64-bit division is a long chain, and few lattices have so many rows)
  const int64_t k = rows <= 0x7fffffff ? (int64_t)((uint32_t)row / (uint32_t)p.ny) : row / p.ny;
  const int64_t j = row - k * p.ny;
  if ((p.fixed[1] && (j == 0 || j == p.ny - 1)) || (p.fixed[2] && (k == 0 || k == p.nz - 1))) return;
  // upstream rows (an interior node of a fixed axis never wraps)
  const int64_t jr[3] = {j + 1 < p.ny ? j + 1 : 0, j, j > 0 ? j - 1 : p.ny - 1};  // index 1 - c_y
  const int64_t kr[3] = {k + 1 < p.nz ? k + 1 : 0, k, k > 0 ? k - 1 : p.nz - 1};
  const T rho_ref = (T)p.rho_ref;
  const T g[3] = {(T)p.g[0], (T)p.g[1], (T)p.g[2]};
  const int nx = (int)p.nx;
  const int64_t own = p.nx * (j + p.ny * k);
  for (int i = (int)threadIdx.x * KX; i < nx; i += 64 * KX) {
    const bool lo = i == 0, hi = i + KX >= nx;  // the lane holds the row's first / last node
    // stream: the populations arriving at the lane's nodes
    T f[Q][KX];
    T edge[Q] = {};  // (KX > 1) at the row's ends: what crosses a periodic wrap, or the fixed node's own value
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      const T* const up = src + (int64_t)a * p.plane + p.nx * (jr[1 + Lt::cy[a]] + p.ny * kr[1 + Lt::cz[a]]);
      if constexpr (KX == 1) {
        const int x = i - Lt::cx[a];
        f[a][0] = up[x < 0 ? nx - 1 : (x < nx ? x : 0)];
      } else {
        const V v = *reinterpret_cast<const V*>(up + i - Lt::cx[a]);
        __builtin_memcpy(f[a], &v, sizeof v);
      }
    }
    if constexpr (KX > 1) {
      if (lo || hi) {
#pragma unroll
        for (int a = 0; a < Q; ++a) {
          const T* const up = src + (int64_t)a * p.plane + p.nx * (jr[1 + Lt::cy[a]] + p.ny * kr[1 + Lt::cz[a]]);
          if (p.fixed[0])
            edge[a] = src[(int64_t)a * p.plane + own + (lo ? 0 : nx - 1)];
          else if (Lt::cx[a])
            edge[a] = up[Lt::cx[a] > 0 ? nx - 1 : 0];
        }
      }
      if (!p.fixed[0]) {
#pragma unroll
        for (int a = 0; a < Q; ++a)
#pragma unroll
          for (int e = 0; e < KX; ++e) {
            if (Lt::cx[a] == 1 && e == 0) f[a][e] = lo ? edge[a] : f[a][e];
            if (Lt::cx[a] == -1) f[a][e] = i + e == nx - 1 ? edge[a] : f[a][e];
          }
      }
    }
    T r[KX], m0[KX], m1[KX], m2[KX], inv[KX], u0[KX], u1[KX], u2[KX], rho[KX], uu[KX];
#pragma unroll
    for (int e = 0; e < KX; ++e) {
      // density deviation and momentum (Eqs. (4)-(5) in population form)
      T m[3] = {0, 0, 0};
      r[e] = 0;
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        r[e] += f[a][e];
        m[0] = fma_t((T)Lt::cx[a], f[a][e], m[0]);
        m[1] = fma_t((T)Lt::cy[a], f[a][e], m[1]);
        m[2] = fma_t((T)Lt::cz[a], f[a][e], m[2]);
      }
      // collide with tau = 1: the new populations are the equilibria of the
      // new state (the body force of test 2 enters the momentum)
      rho[e] = rho_ref + r[e];
      inv[e] = (T)1 / rho[e];
      m0[e] = m[0] + g[0], m1[e] = m[1] + g[1], m2[e] = m[2] + g[2];
      u0[e] = m0[e] * inv[e], u1[e] = m1[e] * inv[e], u2[e] = m2[e] * inv[e];
      uu[e] = fma_t(u2[e], u2[e], fma_t(u0[e], u0[e], u1[e] * u1[e]));
    }
    const bool wall_lo = p.fixed[0] && lo, wall_hi = p.fixed[0] && hi;
    if (KX == 1 && (wall_lo || wall_hi)) continue;
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      const int64_t at = (int64_t)a * p.plane + own + i;
      T o[KX];
#pragma unroll
      for (int e = 0; e < KX; ++e) {
        // c.u: one of a diagonal link's two products m / rho enters unrounded
        constexpr bool d3 = Q == 19;
        const int cx = Lt::cx[a], cy = Lt::cy[a], cz = Lt::cz[a];
        const T cxy = cx && cy ? (d3 && cx < 0 && cy > 0 ? fma_t(m1[e], inv[e], -u0[e])
                                                         : fma_t((T)cx * m0[e], inv[e], (T)cy * u1[e]))
                               : fma_t((T)cy, u1[e], (T)cx * u0[e]);
        const T cu = cz ? fma_t((T)cz * m2[e], inv[e], cxy) : fma_t((T)0, u2[e], cxy);
        // phi_a - 1 = 3 c.u + 4.5 (c.u)^2 - 1.5 |u|^2
        const T phim1 = fma_t((T)-1.5, uu[e], fma_t((T)3, cu, ((T)4.5 * cu) * cu));
        // w_a (rho phi_a - rho_ref) = w_a (r + rho (phi_a - 1))
        o[e] = (T)Lt::wnum[a] * fma_t(rho[e], phim1, r[e]) * (T)(1.0 / 36.0);
        if (KX > 1 && ((wall_lo && e == 0) || (wall_hi && i + e == nx - 1))) o[e] = edge[a];
      }
      // device-scope: a state of under 148 MB, so a plane is within a buffer resource's range
      const buf_t to = make_buf(dst + (int64_t)a * p.plane, p.plane * (int)sizeof(T));
      const int off = (int)((own + i) * (int)sizeof(T));
      if (!TAIL || i + KX <= nx) {
        V v;
        __builtin_memcpy(&v, o, sizeof v);
        if constexpr (NT)
          __builtin_nontemporal_store(v, reinterpret_cast<V*>(dst + at));
        else
          buf_store<V, kStoreDevice>(v, to, off);
      } else {
#pragma unroll
        for (int e = 0; e < KX; ++e) {
          if constexpr (NT) {
            if (i + e < nx) __builtin_nontemporal_store(o[e], dst + at + e);
          } else {
            if (i + e >= nx) break;
            buf_store<T, kStoreDevice>(o[e], to, off + e * (int)sizeof(T));
          }
        }
      }
    }
  }
}

// Populations of the state (rho, u) given as FP64 physical fields of dense
// nodes first .. first+count-1: F_a - w_a rho_ref = w_a (drho + rho (phi_a - 1))
// with phi_a of Eq. (2) at u~ = u / e.
template <int Q, class T>
__global__ void bgk_encode_kernel(T* dst, int64_t plane, const double* __restrict__ rho,
                                  const double* __restrict__ ux, const double* __restrict__ uy,
                                  const double* __restrict__ uz, int64_t first, int64_t count, double rho_ref,
                                  double inv_e) {
  using Lt = Lattice<Q>;
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < count; s += (int64_t)gridDim.x * blockDim.x) {
    const double r = rho[s];
    const double u[3] = {ux[s] * inv_e, uy[s] * inv_e, Q == 19 ? uz[s] * inv_e : 0.0};
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    for (int a = 0; a < Q; ++a) {
      const double cu = Lt::cx[a] * u[0] + Lt::cy[a] * u[1] + Lt::cz[a] * u[2];
      const double phim1 = 3.0 * cu + 4.5 * cu * cu - 1.5 * uu;
      dst[(int64_t)a * plane + first + s] = (T)(Lt::wnum[a] / 36.0 * ((r - rho_ref) + r * phim1));
    }
  }
}

// The moments of the stored populations (the state they are the equilibria
// of): rho = rho_ref + sum_a F^_a, u = e (sum_a c_a F^_a) / rho, as FP64.
template <int Q, class T>
__global__ void bgk_decode_kernel(const T* __restrict__ src, int64_t plane, double* rho, double* ux, double* uy,
                                  double* uz, int64_t first, int64_t count, double rho_ref, double e) {
  using Lt = Lattice<Q>;
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < count; s += (int64_t)gridDim.x * blockDim.x) {
    double r = 0, m[3] = {0, 0, 0};
    for (int a = 0; a < Q; ++a) {
      const double f = (double)src[(int64_t)a * plane + first + s];
      r += f;
      m[0] += Lt::cx[a] * f;
      m[1] += Lt::cy[a] * f;
      m[2] += Lt::cz[a] * f;
    }
    const double rh = rho_ref + r;
    rho[s] = rh;
    ux[s] = e * m[0] / rh;
    uy[s] = e * m[1] / rh;
    if (Q == 19) uz[s] = e * m[2] / rh;
  }
}

// Fixed nodes of both buffers get f_eq(rho_b, u_b); a node on several fixed
// faces takes the values of the lowest-numbered one.
template <int Q, class T>
__global__ void bgk_impose_kernel(T* b0, T* b1, BgkParams p, FaceValues fv, double e) {
  using Lt = Lattice<Q>;
  const int64_t N = p.nx * p.ny * p.nz;
  const int64_t n[3] = {p.nx, p.ny, p.nz};
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < N; x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t idx[3] = {x % p.nx, (x / p.nx) % p.ny, x / (p.nx * p.ny)};
    int face = -1;
    for (int f = 0; f < 6 && face < 0; ++f) {
      if (fv.kind[f] != MACLAB_BC_FIXED) continue;
      const int ax = f / 2;
      if (idx[ax] == ((f & 1) ? n[ax] - 1 : 0)) face = f;
    }
    if (face < 0) continue;
    const double r = fv.rho[face];
    const double u[3] = {fv.u[face][0] / e, fv.u[face][1] / e, Q == 19 ? fv.u[face][2] / e : 0.0};
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    for (int a = 0; a < Q; ++a) {
      const double cu = Lt::cx[a] * u[0] + Lt::cy[a] * u[1] + Lt::cz[a] * u[2];
      const double phim1 = 3.0 * cu + 4.5 * cu * cu - 1.5 * uu;
      const T v = (T)(Lt::wnum[a] / 36.0 * ((r - p.rho_ref) + r * phim1));
      b0[(int64_t)a * p.plane + x] = v;
      b1[(int64_t)a * p.plane + x] = v;
    }
  }
}

template <int Q, class T>
size_t state_bytes(const BgkParams& p) {
  return (size_t)Q * (size_t)p.plane * sizeof(T);
}

// Whether the stores stream past the caches: where the two buffers no longer fit the
// 256 MB cache together and it holds little of what the next step reads. Time against one
// node per lane and streaming stores, widths of 32 to 1000 nodes: 120 MB device-scope
// 0.51..0.90, streaming 0.70..1.15; 140 MB 0.63..1.10 and 0.65..1.07; 160 MB device-scope
// about 1.03 (104^3 FP64 71.5 us a step, 67.4 streaming), 200 MB and more slower.
// Rows of 20 nodes lose from the sum of 256 MB on (140 MB 1.17). Fewer than
// eight rows are over before a device-scope store is (D2Q9 140x4 FP64 4.2, 3.7).
template <int Q, class T>
bool streams(const BgkParams& p) {
  return state_bytes<Q, T>(p) >= size_t(p.nx < 32 ? 128 : 148) << 20 || p.ny * p.nz < 8;
}

template <int Q, class T, int KX, bool TAIL>
hipError_t step_nt(const BgkParams& p, int groups, const void* src, void* dst, hipStream_t s) {
  if (streams<Q, T>(p))
    hipLaunchKernelGGL((bgk_step_kernel<Q, T, KX, TAIL, true>), dim3((unsigned)groups), dim3(64, 4), 0, s,
                       (const T*)src, (T*)dst, p);
  else
    hipLaunchKernelGGL((bgk_step_kernel<Q, T, KX, TAIL, false>), dim3((unsigned)groups), dim3(64, 4), 0, s,
                       (const T*)src, (T*)dst, p);
  return hipGetLastError();
}

template <int Q, class T, int KX>
hipError_t step_kx(const BgkParams& p, const void* src, void* dst, hipStream_t s) {
  const int64_t groups = (p.ny * p.nz + 3) / 4;
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
  if (p.nx % KX) return step_nt<Q, T, KX, true>(p, (int)groups, src, dst, s);
  return step_nt<Q, T, KX, false>(p, (int)groups, src, dst, s);
}

// Nodes per lane. A 16-byte access pays for what memory bounds; a smaller lattice is
// bound by the chain of a row (loads, edge values, stores), which is longer with more
// nodes per lane: D3Q19 FP32 129x16x16 7.9 us a step against 4.8, FP64 129x59x3 13.4
// against 5.5.
template <int Q, class T>
bool wide(const BgkParams& p) {
  constexpr int most = 16 / (int)sizeof(T);
  const size_t bytes = state_bytes<Q, T>(p);
  if (p.nx < 32 * most || p.ny * p.nz < 16) return false;
  if (bytes >= kStreamStoreBytes) return true;
  // Two nodes have to save more than a third of a row's passes (140 MB, against one node
  // per lane: 100 and 193 nodes 0.87, 0.92; 64, 129 and 160 nodes 1.03, 1.09, 1.07).
  const int64_t one = (p.nx + 63) / 64, vec = (p.nx + 64 * most - 1) / (64 * most);
  if (most == 2 && (2 * one <= 3 * vec || p.nx < 80)) return false;
  if (streams<Q, T>(p)) return true;
  // Within the cache, time wide and with one node per lane, against one node and streaming
  // stores: D2Q9 FP32 0.43..0.96 and 0.62..0.84 from 1 MB, FP64 0.57..0.78 and 0.57..0.68
  // at 40 MB; D3Q19 FP32 0.55..0.88 and 0.62..0.76 at 40 MB (0.71..1.08 and 0.72..0.88 at
  // 20), FP64 0.58..0.94 and 0.59..0.75 at 60 MB. Rows of eight passes and more gain at any
  // size in FP64 (D2Q9 600x60 9.1 and 10.8 us a step, 1000x291 13.2 and 16.1). Four FP32
  // nodes have to save two thirds of the passes (rows of 128 nodes, D3Q19 20..120 MB
  // 0.69..1.18 and 0.60..0.78; D2Q9 263x544 10.3 and 8.3 us a step).
  if (most == 4 && one < 3 * vec) return false;
  if (most == 2 && p.nx >= 512) return true;
  return bytes >= size_t(Q == 9 ? (most == 4 ? 0 : 40) : (most == 4 ? 40 : 60)) << 20;
}

template <int Q, class T>
hipError_t step_qt(const BgkParams& p, const void* src, void* dst, hipStream_t s) {
  if (wide<Q, T>(p)) return step_kx<Q, T, 16 / (int)sizeof(T)>(p, src, dst, s);
  return step_kx<Q, T, 1>(p, src, dst, s);
}

}  // namespace

hipError_t launch_bgk_step(int q, bool fp64, const BgkParams& p, const void* src, void* dst, hipStream_t s) {
  if (q == 9) return fp64 ? step_qt<9, double>(p, src, dst, s) : step_qt<9, float>(p, src, dst, s);
  return fp64 ? step_qt<19, double>(p, src, dst, s) : step_qt<19, float>(p, src, dst, s);
}

hipError_t launch_bgk_encode(int q, bool fp64, void* dst, int64_t plane, const double* rho, const double* ux,
                             const double* uy, const double* uz, int64_t first, int64_t count, double rho_ref,
                             double e, hipStream_t s) {
  const unsigned b = blocks_256(count);
  const double ie = 1.0 / e;
  if (q == 9) {
    if (fp64)
      hipLaunchKernelGGL((bgk_encode_kernel<9, double>), dim3(b), dim3(256), 0, s, (double*)dst, plane, rho, ux, uy,
                         uz, first, count, rho_ref, ie);
    else
      hipLaunchKernelGGL((bgk_encode_kernel<9, float>), dim3(b), dim3(256), 0, s, (float*)dst, plane, rho, ux, uy,
                         uz, first, count, rho_ref, ie);
  } else {
    if (fp64)
      hipLaunchKernelGGL((bgk_encode_kernel<19, double>), dim3(b), dim3(256), 0, s, (double*)dst, plane, rho, ux, uy,
                         uz, first, count, rho_ref, ie);
    else
      hipLaunchKernelGGL((bgk_encode_kernel<19, float>), dim3(b), dim3(256), 0, s, (float*)dst, plane, rho, ux, uy,
                         uz, first, count, rho_ref, ie);
  }
  return hipGetLastError();
}

hipError_t launch_bgk_decode(int q, bool fp64, const void* src, int64_t plane, double* rho, double* ux, double* uy,
                             double* uz, int64_t first, int64_t count, double rho_ref, double e, hipStream_t s) {
  const unsigned b = blocks_256(count);
  if (q == 9) {
    if (fp64)
      hipLaunchKernelGGL((bgk_decode_kernel<9, double>), dim3(b), dim3(256), 0, s, (const double*)src, plane, rho,
                         ux, uy, uz, first, count, rho_ref, e);
    else
      hipLaunchKernelGGL((bgk_decode_kernel<9, float>), dim3(b), dim3(256), 0, s, (const float*)src, plane, rho,
                         ux, uy, uz, first, count, rho_ref, e);
  } else {
    if (fp64)
      hipLaunchKernelGGL((bgk_decode_kernel<19, double>), dim3(b), dim3(256), 0, s, (const double*)src, plane, rho,
                         ux, uy, uz, first, count, rho_ref, e);
    else
      hipLaunchKernelGGL((bgk_decode_kernel<19, float>), dim3(b), dim3(256), 0, s, (const float*)src, plane, rho,
                         ux, uy, uz, first, count, rho_ref, e);
  }
  return hipGetLastError();
}

hipError_t launch_bgk_impose(int q, bool fp64, void* b0, void* b1, const BgkParams& p, const FaceValues& fv, double e,
                             hipStream_t s) {
  const unsigned b = blocks_256(p.nx * p.ny * p.nz);
  if (q == 9) {
    if (fp64)
      hipLaunchKernelGGL((bgk_impose_kernel<9, double>), dim3(b), dim3(256), 0, s, (double*)b0, (double*)b1, p, fv, e);
    else
      hipLaunchKernelGGL((bgk_impose_kernel<9, float>), dim3(b), dim3(256), 0, s, (float*)b0, (float*)b1, p, fv, e);
  } else {
    if (fp64)
      hipLaunchKernelGGL((bgk_impose_kernel<19, double>), dim3(b), dim3(256), 0, s, (double*)b0, (double*)b1, p, fv,
                         e);
    else
      hipLaunchKernelGGL((bgk_impose_kernel<19, float>), dim3(b), dim3(256), 0, s, (float*)b0, (float*)b1, p, fv, e);
  }
  return hipGetLastError();
}

}  // namespace maclab
