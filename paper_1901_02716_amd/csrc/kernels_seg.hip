// D3Q19 MacLAB step in FP64 for gfx950: rows of any width, periodic or between
// fixed faces.
//
// Bound: HBM (64 bytes a node) once the state is past the memory-side cache,
// else the latency of a plane step. A gather that loads the 19 upstream nodes
// of every node instead spends its time on 76 loads a node through the caches:
// 251^3 665 us a step against 191 us here (5.6 of the 6.75 TB/s of a copy),
// 48x40x36 8.0 us against 5.4.
//
// Work decomposition
//  - An x-row is cut into segments of 64 KX nodes; a wavefront owns one row
//    of one segment (lane l holds the nodes x0 + KX l .. + KX-1). A workgroup is
//    W output rows plus one halo row on each side and marches in z over a chunk
//    of planes, as the exchange kernel for whole rows does (2.5-D blocking):
//    links with c_y = +-1 go through LDS to the neighbouring row's wavefront,
//    links with c_z = +-1 into three rolling plane accumulators.
//  - In x the links move in registers and by DPP wave rotates. At the edges of
//    a segment that does not span the row (HALO), lanes 0 and 63 also load the
//    node just outside and evaluate the five links that enter from it; lane 63
//    does so for the mirrored node (u_x negated), so one evaluation serves both
//    sides. Negation commutes with every operation of a link value, so the
//    result has the bits of the unmirrored one and does not depend on the
//    segmentation.
//  - On a periodic axis the lanes past the end of a row load its first nodes
//    again, so that the last node's right neighbour is in the next lane.
#include "d3q19.h"
#include "internal.h"

namespace maclab {

struct Seg3DParams {
  int nx, ny, nz, px;
  int ylo, nyo, zlo, nzo;  // output rows and planes
  int xper, yper, zper;
  int nseg, nyb, nzb, nblocks;
  int64_t plane;           // elements per field plane
  double rho_ref;
  double g36x, g36y, g36z;  // 36 dt G / e
};

// The links that enter a segment from the node outside it, as seen from its
// left edge (moving +x); see the mirroring above.
struct EdgeLinks {
  double hxp, p0p, p0m, pp0, pm0;
};

__device__ __forceinline__ EdgeLinks edge_links(double dr, double ux, double uy, double uz, double rho_ref) {
  Links<double> L;
  node_links<CodecF64>(dr, ux, uy, uz, rho_ref, L);
  return {L.hxp, L.p0p, L.p0m, L.pp0, L.pm0};
}

template <int KX, int W, bool HALO, int AUX>
__global__ __launch_bounds__(64 * (W + 2)) void step_d3q19_seg(const double* __restrict__ src,
                                                              double* __restrict__ dst, Seg3DParams p) {
  using C = CodecF64;
  using T = double;
  using E = double;
  using V = RowVec<C, KX>;
  constexpr int SW = 64 * KX;
  constexpr int ROWS = W + 2;
  constexpr int EB = (int)sizeof(E);
  // LDS slots of 4 x SW values: ROWS-1 upward and ROWS-1 downward slots; two
  // such sets, so that one barrier per plane suffices.
  constexpr int SLOTS = 2 * (ROWS - 1) * 4 * SW;
  static_assert(2 * SLOTS * (int)sizeof(T) <= 160 * 1024, "two sets of slots fit the LDS");
  __shared__ T lds[2 * SLOTS];
  const int lane = threadIdx.x;
  const int wv = threadIdx.y;
  const int s_up = wv < ROWS - 1 ? wv : ROWS - 2;
  const int s_dn = wv > 0 ? wv - 1 : 0;
  T* const up0 = lds + s_up * 4 * SW;
  T* const dn0 = lds + (ROWS - 1 + s_dn) * 4 * SW;
  const T* const below0 = lds + s_dn * 4 * SW;
  const T* const above0 = lds + (ROWS - 1 + s_up) * 4 * SW;

  // XCD-aware tile numbering: XCD k (= blockIdx.x mod 8) gets a contiguous band
  const int bid = blockIdx.x;
  const int per = p.nblocks >> 3, rem = p.nblocks & 7, xcd = bid & 7;
  const int tile = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
  const int seg = tile % p.nseg, by = (tile / p.nseg) % p.nyb, bz = tile / (p.nseg * p.nyb);

  const int x0 = seg * SW;
  const int y0 = p.ylo + (int)((int64_t)by * p.nyo / p.nyb);
  const int y1 = p.ylo + (int)((int64_t)(by + 1) * p.nyo / p.nyb);
  const int z0 = p.zlo + (int)((int64_t)bz * p.nzo / p.nzb);
  const int z1 = p.zlo + (int)((int64_t)(bz + 1) * p.nzo / p.nzb);
  const int rows = y1 - y0;  // <= W
  // wave 0: halo row y0-1; waves 1..rows: output rows; wave rows+1: halo row
  // y1; any further waves idle (they only join the barriers)
  const int mode = wv == 0 ? 1 : (wv <= rows ? 0 : (wv == rows + 1 ? 2 : 3));
  const bool out_row = mode == 0;
  int yrow = y0 - 1 + wv;
  if (p.yper)
    yrow = (yrow % p.ny + p.ny) % p.ny;
  else
    yrow = yrow < 0 ? 0 : (yrow > p.ny - 1 ? p.ny - 1 : yrow);
  const int xb = x0 + KX * lane;
  const int xl = p.xper ? xb % p.nx : xb;          // the position this lane loads
  const bool in_row = p.xper || xb < p.nx;
  // the node outside the segment (lane 0: left, lane 63: right)
  const bool edge = HALO && ((lane == 0 && (x0 > 0 || p.xper)) || (lane == 63 && (x0 + SW < p.nx || p.xper)));
  const int hx = ((lane == 0 ? x0 - 1 : x0 + SW) % p.nx + p.nx) % p.nx;
  const T mirror = lane == 63 ? (T)-1 : (T)1;
  // What a lane stores: nothing past the row, and nothing where all its nodes
  // are walls. With KX = 2 (even row pitch) a wall node beside an updated one is
  // written back with its stored value: node 0 of the row (element 0) or, for
  // an even width, the last node (element 1).
  const bool wall_lo = !p.xper && xb == 0, wall_hi = !p.xper && xb + KX == p.nx;
  const bool stores = xb < p.nx && !(!p.xper && (KX == 1 ? (xb == 0 || xb == p.nx - 1) : xb == p.nx - 1));

  buf_t rs[4], rd[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    rs[f] = make_buf(src + f * p.plane, p.plane * EB);
    rd[f] = make_buf(dst + f * p.plane, p.plane * EB);
  }
  auto zwrap = [&](int z) { return p.zper ? (z + p.nz) % p.nz : z; };
  auto row_at = [&](int z) { return (int)(p.px * ((int64_t)yrow + (int64_t)p.ny * zwrap(z)) * EB); };
  const T rho_ref = (T)p.rho_ref;

  auto load_plane = [&](int z, bool valid, V (&b)[4], E (&h)[4]) {
    const int rb = row_at(z);
    const bool any = valid && mode != 3;
    const int off = any && in_row ? rb + xl * EB : kOutOfRange;
#pragma unroll
    for (int f = 0; f < 4; ++f) b[f] = buf_load<V>(rs[f], off);
    if constexpr (HALO) {
      const int hoff = any && edge ? rb + hx * EB : kOutOfRange;
#pragma unroll
      for (int f = 0; f < 4; ++f) h[f] = buf_load<E>(rs[f], hoff);
    }
  };

  E wcur[4], wprev[4];  // raw wall elements of the row pushed now and one step before (KX = 2)

  // One source plane: push its links, exchange the c_y = +-1 links through LDS,
  // then finalise and store destination plane zs-1. am / ac / ap are the
  // accumulators of destination planes zs-1, zs, zs+1; b holds plane zs and is
  // refilled with plane zs+1.
  auto source_plane = [&](auto store_c, int zs, PlaneAcc<T, KX>& am, PlaneAcc<T, KX>& ac, PlaneAcc<T, KX>& ap,
                          V (&b)[4], E (&h)[4], int set) {
#pragma clang fp contract(off)
    constexpr bool STORE = decltype(store_c)::value;
    const int so = set * SLOTS;
    T* const up = up0 + so;
    T* const dn = dn0 + so;
    T f0[KX], hzp[KX], hzm[KX], hxp[KX], p0p[KX], p0m[KX], hxm[KX], m0p[KX], m0m[KX];
    T hyp[KX], pp0[KX], mp0[KX], zpp[KX], zpm[KX];
    T hym[KX], pm0[KX], mm0[KX], zmp[KX], zmm[KX];
#pragma unroll
    for (int e = 0; e < KX; ++e) {
      Links<T> L;
      node_links<C>(b[0].v[e], b[1].v[e], b[2].v[e], b[3].v[e], rho_ref, L);
      f0[e] = L.f0, hzp[e] = L.hzp, hzm[e] = L.hzm;
      hxp[e] = L.hxp, p0p[e] = L.p0p, p0m[e] = L.p0m;
      hxm[e] = L.hxm, m0p[e] = L.m0p, m0m[e] = L.m0m;
      hyp[e] = L.hyp, pp0[e] = L.pp0, mp0[e] = L.mp0, zpp[e] = L.zpp, zpm[e] = L.zpm;
      hym[e] = L.hym, pm0[e] = L.pm0, mm0[e] = L.mm0, zmp[e] = L.zmp, zmm[e] = L.zmm;
    }
    EdgeLinks H{};
    if constexpr (HALO) H = edge_links(h[0], mirror * h[1], h[2], h[3], rho_ref);
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      wprev[f] = wcur[f];
      wcur[f] = KX == 1 ? b[f].v[0] : pick_bits(wall_lo, b[f].v[0], b[f].v[KX - 1]);
    }
    auto from_left = [&](T v, T outside) {
      const T r = dpp_from_left(v);
      return HALO && edge && lane == 0 ? outside : r;
    };
    auto from_right = [&](T v, T outside) {
      const T r = dpp_from_right(v);
      return HALO && edge && lane == 63 ? outside : r;
    };
    // what node x of the neighbouring row receives: density and x momentum in
    // the plane of the source, and the +-z diagonals
    auto send = [&](T* __restrict__ buf, const T (&hy)[KX], const T (&ep)[KX], const T (&em)[KX], const T (&vp)[KX],
                    const T (&vm)[KX], T outside) {
      const T in_ep = from_left(ep[KX - 1], outside), in_em = from_right(em[0], outside);
#pragma unroll
      for (int e = 0; e < KX; ++e) {
        const T a = e > 0 ? ep[e - 1] : in_ep, c = e < KX - 1 ? em[e + 1] : in_em;
        const int x = e * 64 + lane;
        buf[0 * SW + x] = fma_t((T)2, hy[e], a + c);
        buf[1 * SW + x] = a - c;
        buf[2 * SW + x] = vp[e];
        buf[3 * SW + x] = vm[e];
      }
    };
    if (mode == 0 || mode == 1) send(up, hyp, pp0, mp0, zpp, zpm, H.pp0);
    if (mode == 0 || mode == 2) send(dn, hym, pm0, mm0, zmp, zmm, H.pm0);
    if (mode == 0) {
      const T in_hxp = from_left(hxp[KX - 1], H.hxp), in_p0p = from_left(p0p[KX - 1], H.p0p),
              in_p0m = from_left(p0m[KX - 1], H.p0m);
      const T in_hxm = from_right(hxm[0], H.hxp), in_m0p = from_right(m0p[0], H.p0p),
              in_m0m = from_right(m0m[0], H.p0m);
      add_own_row<T, KX>(f0, hzp, hzm, hxp, p0p, p0m, hxm, m0p, m0m, in_hxp, in_p0p, in_p0m, in_hxm, in_m0p, in_m0m,
                         am, ac, ap);
    }
    load_plane(zs + 1, zs + 1 <= z1, b, h);
    __syncthreads();
    if (out_row) {
      const T* const fb = below0 + so;
      const T* const fa = above0 + so;
#pragma unroll
      for (int e = 0; e < KX; ++e) {
        const int x = e * 64 + lane;
        add_sent<T, KX, 1>(fb[0 * SW + x], fb[1 * SW + x], fb[2 * SW + x], fb[3 * SW + x], e, am, ac, ap);
        add_sent<T, KX, -1>(fa[0 * SW + x], fa[1 * SW + x], fa[2 * SW + x], fa[3 * SW + x], e, am, ac, ap);
      }
    }
    const int zd = zs - 1;
    V o[4] = {};
    if (STORE && out_row) {
      finalize_row<C, KX>(am, rho_ref, p.g36x, p.g36y, p.g36z, 0u, 0, o);  // (no rounding bits in FP64)
      if constexpr (KX > 1) {
        if (wall_lo || wall_hi) {
#pragma unroll
          for (int f = 0; f < 4; ++f) {
            if (wall_lo)
              o[f].v[0] = wprev[f];
            else
              o[f].v[KX - 1] = wprev[f];
          }
        }
      }
    }
    const int off = STORE && out_row && stores ? row_at(zd) + xb * EB : kOutOfRange;
#pragma unroll
    for (int f = 0; f < 4; ++f) buf_store<V, AUX>(o[f], rd[f], off);
  };

  using NoStore = std::integral_constant<bool, false>;
  using Store = std::integral_constant<bool, true>;
  PlaneAcc<T, KX> a0, a1, a2;
  a0.zero();
  a1.zero();
  V b[4];
  E h[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) wcur[f] = h[f] = E{};
  load_plane(z0 - 1, true, b, h);
  // Source planes z0-1 .. z1; the first two complete no plane of the tile. The
  // accumulator roles rotate with period 3, the LDS sets with period 2.
  source_plane(NoStore{}, z0 - 1, a0, a1, a2, b, h, 0);
  source_plane(NoStore{}, z0, a1, a2, a0, b, h, 1);
  for (int zs = z0 + 1; zs <= z1; zs += 6) {
    source_plane(Store{}, zs, a2, a0, a1, b, h, 0);
    if (zs + 1 > z1) break;
    source_plane(Store{}, zs + 1, a0, a1, a2, b, h, 1);
    if (zs + 2 > z1) break;
    source_plane(Store{}, zs + 2, a1, a2, a0, b, h, 0);
    if (zs + 3 > z1) break;
    source_plane(Store{}, zs + 3, a2, a0, a1, b, h, 1);
    if (zs + 4 > z1) break;
    source_plane(Store{}, zs + 4, a0, a1, a2, b, h, 0);
    if (zs + 5 > z1) break;
    source_plane(Store{}, zs + 5, a1, a2, a0, b, h, 1);
  }
}

// ------------------------------------------------------------------ launch
bool seg3d_supported(const Layout& L) {
  // (The FP32-arithmetic storages take the row kernel, whose sums run in
  // another order.) Three rows and planes; buffer offsets are 31-bit.
  return L.q == 19 && L.precision == MACLAB_FP64 && L.N >= kMarchNodes64 && L.ny >= 3 && L.nz >= 3 &&
         L.plane * L.bytes < (int64_t(1) << 31);
}

// One thread per node, with all its loads at once, takes 4.8 us a step as long as every
// SIMD has one wavefront (64 nodes of a row) at most; the chain of plane steps takes 5.2 to
// 6.5 (40x32x32 4.8 and 5.2 between walls, 4.8 and 6.4 periodic; 63x32x32 4.9, 6.5).
// With more wavefronts it is 7 and up (46x32 rows 7.6 and 6.5, 12x100x30 9.7 and 7.5), but
// not with one output row, where six of a workgroup's eight rows are idle (80x3x800
// 7.4 and 9.8, 300x3x800 even).
bool seg3d_pays(const Layout& L, const StepParams& p, int cus) {
  const int64_t nyo = p.fixed[1] ? L.ny - 2 : L.ny, nzo = p.fixed[2] ? L.nz - 2 : L.nz;
  return (L.nx + 63) / 64 * nyo * nzo > 4 * (int64_t)cus && nyo > 1;
}

// The tiling, from a model of the time: a workgroup's plane step costs each of
// its wavefronts a share of its CU for every node a lane holds (0.11 us per
// wavefront and node; a fifth more with one node per lane, half as much again
// for a state of 192 MB or more, which comes from memory in narrower accesses),
// workgroups on a CU add up, and a plane step takes at least the latency of its
// load, exchange and barrier (0.9 us). A tile also runs the two planes beside
// its chunk. So the rule weighs idle lanes in the last segment, halo rows and
// planes, and CUs without a tile. Measured (us per step, kx x w): 251^3 2x6 191, 1x14 227, 1x6
// 231; 130x129x131 1x14 36.5, 1x6 43.8, 2x6 57.5 (two segments for 130 nodes);
// 128x129x131 2x6 24.7, 1x14 35.8; 96^3 2x6 14.4, 1x14 17.6; 48x40x36 1x6 5.4,
// 1x14 7.3; 192^3 2x6 100, 1x14 114; 256^3 2x6 216 to 221, 1x14 238 to 261.
Seg3DShape seg3d_shape(const Layout& L, const StepParams& p, int cus) {
  const int nyo = p.fixed[1] ? (int)L.ny - 2 : (int)L.ny, nzo = p.fixed[2] ? (int)L.nz - 2 : (int)L.nz;
  const double unit = 0.11, latency = 0.9;
  static const int shapes[3][2] = {{1, 6}, {1, 14}, {2, 6}};
  Seg3DShape best;
  double best_cost = 1e300;
  for (const auto& kw : shapes) {
    const int kx = kw[0], w = kw[1];
    // a lane's nodes are one vector access, and a periodic wrap may not split them
    if (L.px % kx || (!p.fixed[0] && L.nx % kx)) continue;
    const int nseg = (int)((L.nx + 64 * kx - 1) / (64 * kx));
    const int nyb = (nyo + w - 1) / w;
    const double narrow = L.state_bytes < kStreamStoreBytes / 4 * 3 ? 1.2 : 1.5;
    const double work = (w + 2) * kx * unit * (kx > 1 ? 1.0 : narrow);
    for (int nzb = 1; nzb <= nzo; ++nzb) {
      const int64_t blocks = (int64_t)nseg * nyb * nzb;
      if (nzb > 1 && blocks > 16 * (int64_t)cus) break;  // enough tiles for any balance
      const int64_t planes = (nzo + nzb - 1) / nzb + 2;
      const double per_cu = (double)((blocks + cus - 1) / cus);
      const double cost = planes * (per_cu * work > latency ? per_cu * work : latency);
      if (cost < best_cost) {
        best_cost = cost;
        best.kx = kx;
        best.w = w;
        best.nyb = nyb;
        best.nzb = nzb;
      }
    }
  }
  return best;
}

template <int KX, int W, bool HALO, int AUX>
static hipError_t launch_seg(const void* src, void* dst, const Seg3DParams& sp, hipStream_t s) {
  hipLaunchKernelGGL((step_d3q19_seg<KX, W, HALO, AUX>), dim3(sp.nblocks), dim3(64, W + 2, 1), 0, s,
                     (const double*)src, (double*)dst, sp);
  return hipGetLastError();
}

template <int KX, int W>
static hipError_t launch_seg_h(const void* src, void* dst, const Seg3DParams& sp, hipStream_t s) {
  // one segment that spans the row: no node outside it matters (walls), or it wraps by the rotate
  const bool halo = !(sp.nseg == 1 && (!sp.xper || sp.nx == 64 * KX));
  // A state past the memory-side cache is stored non-temporally (251^3:
  // 191 us, 201 device-scope, 204 cached), a smaller one with device-scope
  // stores, which leave it there for the next step (128x129x131: 24.7 us, 31.0
  // non-temporal, 25.6 cached), as in the D2Q9 step.
  const bool stream = 4 * sp.plane * (int64_t)sizeof(double) >= (int64_t)kStreamStoreBytes;
  if (stream)
    return halo ? launch_seg<KX, W, true, kStoreStream>(src, dst, sp, s)
                : launch_seg<KX, W, false, kStoreStream>(src, dst, sp, s);
  return halo ? launch_seg<KX, W, true, kStoreDevice>(src, dst, sp, s)
              : launch_seg<KX, W, false, kStoreDevice>(src, dst, sp, s);
}

static hipError_t launch_seg_shape(const Seg3DShape& sh, const void* src, void* dst, const Seg3DParams& sp,
                                   hipStream_t s) {
  if (sh.kx == 1 && sh.w == 14) return launch_seg_h<1, 14>(src, dst, sp, s);
  if (sh.kx == 1 && sh.w == 6) return launch_seg_h<1, 6>(src, dst, sp, s);
  if (sh.kx == 2 && sh.w == 6) return launch_seg_h<2, 6>(src, dst, sp, s);
  return hipErrorInvalidValue;
}

hipError_t launch_step_seg(const Layout& L, const void* src, void* dst, const StepParams& p, const Seg3DShape& sh,
                           hipStream_t s) {
  Seg3DParams sp;
  sp.nx = (int)L.nx;
  sp.ny = (int)L.ny;
  sp.nz = (int)L.nz;
  sp.px = (int)L.px;
  sp.xper = !p.fixed[0];
  sp.yper = !p.fixed[1];
  sp.zper = !p.fixed[2];
  sp.ylo = p.fixed[1] ? 1 : 0;
  sp.zlo = p.fixed[2] ? 1 : 0;
  sp.nyo = sp.ny - 2 * sp.ylo;
  sp.nzo = sp.nz - 2 * sp.zlo;
  sp.nseg = (sp.nx + 64 * sh.kx - 1) / (64 * sh.kx);
  sp.nyb = sh.nyb;
  sp.nzb = sh.nzb;
  if (sp.nyb < 1 || sp.nzb < 1 || sp.nyb > sp.nyo || sp.nzb > sp.nzo || (sp.nyo + sp.nyb - 1) / sp.nyb > sh.w ||
      sp.px % sh.kx || (sp.xper && sp.nx % sh.kx))
    return hipErrorInvalidValue;
  sp.nblocks = sp.nseg * sp.nyb * sp.nzb;
  sp.plane = L.plane;
  sp.rho_ref = p.rho_ref;
  sp.g36x = 36.0 * p.g[0];
  sp.g36y = 36.0 * p.g[1];
  sp.g36z = 36.0 * p.g[2];
  return launch_seg_shape(sh, src, dst, sp, s);
}

}  // namespace maclab
