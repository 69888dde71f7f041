// General D3Q19 MacLAB step for gfx950: any node counts and boundary kinds, every
// storage, lattices past 2^31 bytes a plane.
//
// Work decomposition
//  - An x-row is cut into segments of 62 nodes; a wavefront owns the segment of
//    one row and a chunk of planes and marches in z, with the node beside the
//    segment in lanes 0 and 63 (wrapped on a periodic axis). There is no LDS and
//    no barrier.
//  - Per source plane it loads its own row and the rows below and above (which
//    the neighbouring wavefronts load too, so they come from the caches),
//    evaluates the 19 links of Eq. (2) that reach its row where they start, and
//    moves them in x by DPP wave rotates. Links that move up a plane wait in
//    registers.
//  - The links of a node are then summed in the order of the lattice table, as one
//    thread per node does that loads its 19 upstream nodes; those 76 loads a node are
//    what this form saves (300x67x93 FP32: 32.7 us a step, 17.8 here; 200x200x120 FP32
//    84.9, 39.2, S16 88.8, 43.4, split-bf16 95.3, 44.8). Bound by instructions: about 240 a wavefront and plane.
#include "internal.h"

#include <math.h>

namespace maclab {

struct RowsParams {
  int nx, ny, nz;
  int64_t px, plane;
  int ylo, nyo, zlo, nzo;  // output rows and planes
  int xper, yper, zper;
  int nseg, nzb;
  int64_t nwaves;
  double rho_ref;
  double g[3];
  uint32_t sr_key;
};

// 36 F^_a of one link with weight numerator w: w [drho + rho (3 cu + 4.5 cu^2 -
// 1.5 |u|^2)]. Every FMA is written out: a link has the same bits whichever
// wavefront evaluates it.
template <class T>
__device__ __forceinline__ T row_link(T w, T dr, T rho, T uu, T cu) {
#pragma clang fp contract(off)
  const T q = fma_t((T)-1.5, uu, fma_t((T)3, cu, ((T)4.5 * cu) * cu));
  return w * fma_t(rho, q, dr);
}

// A stored velocity component, m / rho. (Contraction is left to the compiler
// here: the split codec's low half is then the rounded remainder of the exact
// product, as in the other kernels that write the product into its encoding.)
template <class C>
__device__ __forceinline__ typename C::elem enc_velocity(typename C::T m, typename C::T inv, int field,
                                                         uint32_t bits) {
  return C::enc(m * inv, field, bits);
}

// Fields of the three source rows (below, own, above) of one plane, as stored.
template <class C>
struct RowsRaw {
  typename C::elem v[3][4];
};

// Wavefronts of a workgroup: neighbouring rows. Four share their rows' loads in
// one CU's cache and leave the scheduler small pieces (8: 10 to 20% slower).
constexpr int kRowsWaves = 4;

template <class C, bool NT>
__global__ __launch_bounds__(64 * kRowsWaves) void step_d3q19_rows(const typename C::elem* __restrict__ src,
                                                           typename C::elem* __restrict__ dst, RowsParams p) {
#pragma clang fp contract(off)
  using T = typename C::T;
  using E = typename C::elem;
  const int lane = threadIdx.x & 63;
  // XCD-aware numbering: XCD k takes a contiguous range of wavefronts, rows of a
  // segment and chunk next to each other
  // (a grid that needs a second dimension is long enough to be taken as it comes)
  const int nblk = (int)gridDim.x, bid = (int)blockIdx.x;
  const int per = nblk >> 3, rem = nblk & 7, xcd = bid & 7;
  const int64_t blk = gridDim.y > 1 ? (int64_t)blockIdx.y * nblk + bid
                                    : (int64_t)xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
  const int64_t g = blk * kRowsWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (g >= p.nwaves) return;
  const int row = (int)(g % p.nyo);
  const int seg = (int)(g / p.nyo % p.nseg), zc = (int)(g / p.nyo / p.nseg);
  const int y = p.ylo + row;
  const int z0 = p.zlo + (int)((int64_t)zc * p.nzo / p.nzb);
  const int z1 = p.zlo + (int)((int64_t)(zc + 1) * p.nzo / p.nzb);
  const int yb = p.yper && y == 0 ? p.ny - 1 : y - 1, ya = p.yper && y == p.ny - 1 ? 0 : y + 1;
  // periodic: the segment's first node is in lane 1; walls: node 0 is in lane 0
  const int x = seg * 62 + lane - (p.xper ? 1 : 0);
  // The position this lane loads: the first node for the lane past the last one on a
  // periodic axis, or the wall; no stored node depends on the lanes beyond, which load the
  // same. (A remainder for them cost 0.5 us a step, 16x40x40 FP32 5.7 against 4.7 with
  // one thread per node.)
  const int xl = p.xper ? (x < 0 ? p.nx - 1 : (x < p.nx ? x : 0)) : (x < p.nx ? x : p.nx - 1);
  const bool stores = lane > 0 && lane < 63 && x < p.nx - (p.xper ? 0 : 1);
  // (a remainder would be some thirty instructions)
  auto zwrap = [&](int z) { return z < 0 ? z + p.nz : (z >= p.nz ? z - p.nz : z); };
  auto load = [&](int z, RowsRaw<C>& b) {
    const int64_t zb = (int64_t)p.ny * zwrap(z);
    const int64_t at[3] = {p.px * (yb + zb) + xl, p.px * (y + zb) + xl, p.px * (ya + zb) + xl};
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int f = 0; f < 4; ++f) b.v[r][f] = src[f * p.plane + at[r]];
  };
  const T rho_ref = (T)p.rho_ref;
  const T g36x = (T)(36.0 * p.g[0]), g36y = (T)(36.0 * p.g[1]), g36z = (T)(36.0 * p.g[2]);

  // Links in flight, in x already where they arrive: the c_z = 0 links of the
  // plane being completed (rest, +-x, +-y, the xy diagonals), the c_z = +1 links
  // of the plane below it (+z axis, (0,1,1), (0,-1,1), (1,0,1), (-1,0,1)) and
  // those of the plane itself.
  T mid[9], low[5], next_low[5];
#pragma unroll
  for (int k = 0; k < 9; ++k) mid[k] = (T)0;
#pragma unroll
  for (int k = 0; k < 5; ++k) low[k] = next_low[k] = (T)0;

  // Source plane zs: its c_z = -1 links complete plane zs - 1, which is stored
  // if `store`.
  auto source_plane = [&](int zs, const RowsRaw<C>& b, bool store) {
#pragma clang fp contract(off)
    T dr[3], ux[3], uy[3], uz[3], rho[3], uu[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      dr[r] = C::dec(b.v[r][0], 0);
      ux[r] = C::dec(b.v[r][1], 1);
      uy[r] = C::dec(b.v[r][2], 2);
      uz[r] = C::dec(b.v[r][3], 3);
      rho[r] = rho_ref + dr[r];
      uu[r] = fma_t(uz[r], uz[r], fma_t(ux[r], ux[r], uy[r] * uy[r]));
    }
    auto link = [&](T w, int r, T cu) { return row_link<T>(w, dr[r], rho[r], uu[r], cu); };
    // c_z = -1: -z axis, (0,-1,-1) from above, (0,1,-1) from below, (-1,0,-1), (1,0,-1)
    const T m6 = link((T)2, 1, -uz[1]);
    const T m12 = link((T)1, 2, -uy[2] - uz[2]);
    const T m14 = link((T)1, 0, uy[0] - uz[0]);
    const T m16 = dpp_from_right(link((T)1, 1, -ux[1] - uz[1]));
    const T m18 = dpp_from_left(link((T)1, 1, ux[1] - uz[1]));
    if (store) {
      T r = (T)0 + mid[0], mx, my, mz;
      r += mid[1];
      mx = (T)0 + mid[1];
      r += mid[2];
      mx -= mid[2];
      r += mid[3];
      my = (T)0 + mid[3];
      r += mid[4];
      my -= mid[4];
      r += low[0];
      mz = (T)0 + low[0];
      r += m6;
      mz -= m6;
      r += mid[5];
      mx += mid[5];
      my += mid[5];
      r += mid[6];
      mx -= mid[6];
      my -= mid[6];
      r += mid[7];
      mx -= mid[7];
      my += mid[7];
      r += mid[8];
      mx += mid[8];
      my -= mid[8];
      r += low[1];
      my += low[1];
      mz += low[1];
      r += m12;
      my -= m12;
      mz -= m12;
      r += low[2];
      my -= low[2];
      mz += low[2];
      r += m14;
      my += m14;
      mz -= m14;
      r += low[3];
      mx += low[3];
      mz += low[3];
      r += m16;
      mx -= m16;
      mz -= m16;
      r += low[4];
      mx -= low[4];
      mz += low[4];
      r += m18;
      mx += m18;
      mz -= m18;
      // drho' = r / 36, u~' = (m + 36 g) / (36 rho_ref + r)
      const T inv = (T)1 / fma_t((T)36, rho_ref, r);
      const int64_t zb = (int64_t)p.ny * zwrap(zs - 1);
      const int64_t at = p.px * (y + zb) + x;
      uint32_t bits = 0;
      if constexpr (needs_rng<C>::value) bits = sr_node_bits(p.sr_key, x + (int64_t)p.nx * (y + zb));
      const E o[4] = {C::enc(div36(r), 0, bits), enc_velocity<C>(mx + g36x, inv, 1, bits),
                      enc_velocity<C>(my + g36y, inv, 2, bits), enc_velocity<C>(mz + g36z, inv, 3, bits)};
      if constexpr (NT) {
        if (stores) {
#pragma unroll
          for (int f = 0; f < 4; ++f) __builtin_nontemporal_store(o[f], dst + f * p.plane + at);
        }
      } else {
        // a state of under 256 MB: a plane is within a buffer resource's range
        const int64_t bytes = p.plane * (int64_t)sizeof(E);
        const int off = stores ? (int)(at * (int64_t)sizeof(E)) : kOutOfRange;
#pragma unroll
        for (int f = 0; f < 4; ++f)
          buf_store<E, kStoreDevice>(o[f], make_buf(dst + f * p.plane, bytes), off);
      }
    }
    // c_z = +1 of the plane below becomes due; this plane's c_z = 0 links
#pragma unroll
    for (int k = 0; k < 5; ++k) low[k] = next_low[k];
    mid[0] = link((T)12, 1, (T)0);
    mid[1] = dpp_from_left(link((T)2, 1, ux[1]));
    mid[2] = dpp_from_right(link((T)2, 1, -ux[1]));
    mid[3] = link((T)2, 0, uy[0]);
    mid[4] = link((T)2, 2, -uy[2]);
    mid[5] = dpp_from_left(link((T)1, 0, ux[0] + uy[0]));
    mid[6] = dpp_from_right(link((T)1, 2, -ux[2] - uy[2]));
    mid[7] = dpp_from_right(link((T)1, 0, -ux[0] + uy[0]));
    mid[8] = dpp_from_left(link((T)1, 2, ux[2] - uy[2]));
    next_low[0] = link((T)2, 1, uz[1]);
    next_low[1] = link((T)1, 0, uy[0] + uz[0]);
    next_low[2] = link((T)1, 2, -uy[2] + uz[2]);
    next_low[3] = dpp_from_left(link((T)1, 1, ux[1] + uz[1]));
    next_low[4] = dpp_from_right(link((T)1, 1, -ux[1] + uz[1]));
  };

  RowsRaw<C> b0, b1;
  load(z0 - 1, b0);
  load(z0, b1);
  for (int zs = z0 - 1; zs <= z1; zs += 2) {
    source_plane(zs, b0, zs - 1 >= z0);
    if (zs + 2 <= z1) load(zs + 2, b0);
    if (zs + 1 > z1) break;
    source_plane(zs + 1, b1, zs >= z0);
    if (zs + 3 <= z1) load(zs + 3, b1);
  }
}

// ------------------------------------------------------------------ launch
template <class C>
static hipError_t launch_rows(const Layout& L, const void* src, void* dst, const RowsParams& rp, hipStream_t s) {
  using E = typename C::elem;
  const int64_t blocks = (rp.nwaves + kRowsWaves - 1) / kRowsWaves;
  constexpr int64_t kRow = int64_t(1) << 22;  // workgroups in x: under 2^32 work-items
  const int64_t ny = (blocks + kRow - 1) / kRow;
  const dim3 grid((unsigned)(ny > 1 ? kRow : blocks), (unsigned)ny), block(64 * kRowsWaves);
  // Stores past the caches for a state larger than the memory-side cache
  // (301x256^2 FP32: 232 us a step, 248 device-scope, 240 cached), else
  // device-scope (300x67x93 FP32: 18.7, 24.3 non-temporal, 20.6 cached).
  if (L.state_bytes >= kStreamStoreBytes)
    hipLaunchKernelGGL((step_d3q19_rows<C, true>), grid, block, 0, s, (const E*)src, (E*)dst, rp);
  else
    hipLaunchKernelGGL((step_d3q19_rows<C, false>), grid, block, 0, s, (const E*)src, (E*)dst, rp);
  return hipGetLastError();
}

static int64_t row_segments(const Layout& L, const StepParams& p) {
  return p.fixed[0] ? (L.nx - 2 + 61) / 62 : (L.nx + 61) / 62;
}

// Chunks of planes, by a model of the time: a plane step takes a wavefront about
// 1 us (its loads and chain) and a SIMD 0.4 us for each of its wavefronts, and
// a chunk also runs the two planes beside it. Up to eight wavefronts a SIMD
// the last, nearly empty round counts in full.
int rows_chunks(const Layout& L, const StepParams& p, int cus) {
  const int64_t rows = row_segments(L, p) * (p.fixed[1] ? L.ny - 2 : L.ny), nzo = p.fixed[2] ? L.nz - 2 : L.nz;
  if (rows < 1) return 1;  // (such faces are refused before a launch)
  int64_t nzb = 1;
  double best = 1e300;
  for (int64_t k = 1; k <= nzo && (k == 1 || rows * k <= 32 * (int64_t)cus); ++k) {
    const double exact = (double)(rows * k) / (4.0 * cus);
    const double per_simd = exact < 8.0 ? ceil(exact) : exact;
    const double planes = (double)((nzo + k - 1) / k + 2);
    const double cost = planes * (0.4 * per_simd > 1.0 ? 0.4 * per_simd : 1.0);
    if (cost < best) {
      best = cost;
      nzb = k;
    }
  }
  return (int)nzb;
}

hipError_t launch_step_rows(const Layout& L, const void* src, void* dst, const StepParams& p, int nzb,
                            hipStream_t s) {
  RowsParams rp;
  rp.nx = (int)L.nx;
  rp.ny = (int)L.ny;
  rp.nz = (int)L.nz;
  rp.px = L.px;
  rp.plane = L.plane;
  rp.xper = !p.fixed[0];
  rp.yper = !p.fixed[1];
  rp.zper = !p.fixed[2];
  rp.ylo = p.fixed[1] ? 1 : 0;
  rp.zlo = p.fixed[2] ? 1 : 0;
  rp.nyo = rp.ny - 2 * rp.ylo;
  rp.nzo = rp.nz - 2 * rp.zlo;
  if (nzb < 1 || nzb > rp.nzo) return hipErrorInvalidValue;
  rp.nseg = (int)row_segments(L, p);
  rp.nzb = nzb;
  rp.nwaves = (int64_t)rp.nseg * rp.nyo * nzb;
  rp.rho_ref = p.rho_ref;
  for (int i = 0; i < 3; ++i) rp.g[i] = p.g[i];
  rp.sr_key = p.sr_key;
  switch (L.precision) {
    case MACLAB_FP64: return launch_rows<CodecF64>(L, src, dst, rp, s);
    case MACLAB_FP32: return launch_rows<CodecF32>(L, src, dst, rp, s);
    case MACLAB_HILO: return launch_rows<CodecHILO>(L, src, dst, rp, s);
    case MACLAB_S16: return launch_rows<CodecS16>(L, src, dst, rp, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace maclab
