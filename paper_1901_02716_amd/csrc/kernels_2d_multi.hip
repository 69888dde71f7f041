// Several D2Q9 MacLAB steps in one launch for gfx950, for one lattice or a
// batch of lattices.
//
// A step of a small lattice takes the latency of a launch and of one load chain
// (about 5 us), and a step of a large one moves the state through memory. Here a
// workgroup loads a tile of the lattice once, advances it T steps in registers,
// and stores the part that T steps of missing neighbours have not reached.
//
// Work decomposition
//  - A tile is 64 nodes wide (one per lane) and R NW rows high: wavefront w holds
//    rows R w .. R w + R-1 of the tile. Tiles overlap by T nodes on each side; at
//    a fixed face a tile begins or ends with the face, whose nodes keep their
//    values and need no overlap, and a periodic row of exactly 64 nodes wraps by
//    the rotate. On a periodic axis the overlap holds copies of the nodes across
//    the wrap.
//  - Per step the x pass runs by DPP rotates as in the single-step kernel, and
//    the y pass in registers; the sums that cross to the wavefront above or
//    below go through LDS (four values a node, two sets, one barrier a step).
//  - Between steps a value is encoded and decoded as the stored state would be
//    (with the rounding bits of its node and step), and the sums run in the order of
//    the single-step kernel, so T steps here have the bits of T single steps.
//  - TRACE: every step's state is stored, one behind the other, faces included
//    (the states a reverse sweep needs).
#include "d2q9.h"
#include "internal.h"

namespace maclab {

struct Multi2DParams {
  const Lattice2D* lat;  // device array (batch) ...
  Lattice2D one;         // ... or this single lattice when lat == nullptr
  const int4* items;     // device array of work items {lattice, x tile, y tile, 0} ...
  int nxt, nyt;          // ... or, when items == nullptr, nxt x nyt tiles of `one`
  int halo;              // overlap (>= steps)
  int steps;             // T
  int64_t stride;        // TRACE: elements between the stored states
  double rho_ref;
  uint64_t seed, step;   // S16 rounding: key of step + s
};

template <class C, int R, int NW, bool NT, bool TRACE>
__global__ __launch_bounds__(64 * NW) void step_d2q9_multi(const typename C::elem* __restrict__ src,
                                                          typename C::elem* __restrict__ dst, Multi2DParams p) {
#pragma clang fp contract(off)
  using T = typename C::T;
  using E = typename C::elem;
  constexpr int SW = 64;
  constexpr int H = R * NW;
  constexpr int EB = (int)sizeof(E);
  // per wavefront: density/y and x momentum sums for the row above it and for the row below it
  __shared__ T lds[2][NW][4][SW];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nblk = (int)gridDim.x, bid = (int)blockIdx.x;
  const int per = nblk >> 3, rem = nblk & 7, xcd = bid & 7;
  const int g = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);  // XCD k takes a contiguous range of tiles
  Lattice2D lt;
  int xt, yt;
  if (p.items) {
    const int4 it = p.items[g];
    lt = p.lat[it.x];
    xt = it.y;
    yt = it.z;
  } else {
    lt = p.one;
    xt = g % p.nxt;
    yt = g / p.nxt;
  }
  // first node of the tile and the nodes it stores, per axis
  const MultiSpan sx = multi_span(lt.nx, lt.xper, SW, p.halo, xt, lt.xper && lt.nx == SW);
  const MultiSpan sy = multi_span(lt.ny, lt.yper, H, p.halo, yt, false);
  const int xb = sx.start + lane;
  const int yb = sy.start + R * wv;
  const int xl = lt.xper ? wrap_near(xb, lt.nx) : xb;
  const bool in_row = lt.xper || xb < lt.nx;
  int yr[R];  // stored rows (wrapped)
#pragma unroll
  for (int i = 0; i < R; ++i) yr[i] = lt.yper ? wrap_near(yb + i, lt.ny) : yb + i;
  // rows past the last one any stored row depends on: the wavefront only joins the barriers
  const bool active = yb < sy.hi + p.halo && (lt.yper || yb < lt.ny);

  const int64_t pbytes = lt.plane * EB;
  buf_t rs[3];
#pragma unroll
  for (int f = 0; f < 3; ++f) rs[f] = make_buf(src + lt.base + f * lt.plane, pbytes);
  E st[R][3];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const bool ok = active && in_row && (lt.yper || yr[i] < lt.ny);
    const int off = ok ? (int)(((int64_t)lt.pitch * yr[i] + xl) * EB) : kOutOfRange;
#pragma unroll
    for (int f = 0; f < 3; ++f) st[i][f] = buf_load<E>(rs[f], off);
  }
  // nodes that keep their values: walls, and what lies past the row
  const bool keep_x = !lt.xper && (xb == 0 || xb >= lt.nx - 1);
  bool keep_y[R];
#pragma unroll
  for (int i = 0; i < R; ++i) keep_y[i] = !lt.yper && (yr[i] == 0 || yr[i] >= lt.ny - 1);

  const bool own_x = xb >= sx.lo && xb < sx.hi;
  auto store = [&](E* to) {
    buf_t rd[3];
#pragma unroll
    for (int f = 0; f < 3; ++f) rd[f] = make_buf(to + lt.base + f * lt.plane, pbytes);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool ok = own_x && yb + i >= sy.lo && yb + i < sy.hi && (TRACE || !keep_y[i]);
      const int off = ok ? (int)(((int64_t)lt.pitch * (yb + i) + xb) * EB) : kOutOfRange;
#pragma unroll
      for (int f = 0; f < 3; ++f) buf_store<E, NT ? kStoreStream : kStoreDevice>(st[i][f], rd[f], off);
    }
  };

  const T rho_ref = (T)p.rho_ref;
  const T g36x = (T)(36.0 * lt.gx), g36y = (T)(36.0 * lt.gy);
  const T den0 = (T)36 * rho_ref;
  for (int s = 0; s < p.steps; ++s) {
    T (*const box)[4][SW] = lds[s & 1];
    T t0[R], u0[R], up[R], dn[R], qup[R], qdn[R];
    if (active) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        Mom2<T> M;
        moments2<T>(C::dec(st[i][0], 0), C::dec(st[i][1], 1), C::dec(st[i][2], 2), rho_ref, M);
        const Send2<T> S = send2<T>(M);
        const T r0 = dpp_from_left(S.r0), r1 = dpp_from_left(S.r1), r2 = dpp_from_left(S.c2);
        const T l0 = dpp_from_right(S.l0), l1 = dpp_from_right(S.l1), l2 = dpp_from_right(S.c2);
        t0[i] = fma_t((T)4, M.a, r0 + l0);
        u0[i] = r0 - l0;
        const T t1 = fma_t((T)4, M.by, r1 + l1), u1 = r1 - l1;
        const T t2 = fma_t((T)4, M.cyy, r2 + l2), u2 = r2 - l2;
        const T pt = fma_t((T)1.5, t2, t0[i]), pu = fma_t((T)1.5, u2, u0[i]);
        up[i] = pt + t1;
        dn[i] = pt - t1;
        qup[i] = pu + u1;
        qdn[i] = pu - u1;
      }
      box[wv][0][lane] = up[R - 1];
      box[wv][1][lane] = qup[R - 1];
      box[wv][2][lane] = dn[0];
      box[wv][3][lane] = qdn[0];
    }
    __syncthreads();
    if (active) {
      const int below = wv > 0 ? wv - 1 : 0, above = wv < NW - 1 ? wv + 1 : NW - 1;
      const uint32_t key = needs_rng<C>::value ? sr_key(p.seed, p.step + (uint64_t)s) : 0u;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const T ub = i > 0 ? up[i > 0 ? i - 1 : 0] : box[below][0][lane];
        const T qb = i > 0 ? qup[i > 0 ? i - 1 : 0] : box[below][1][lane];
        const T da = i < R - 1 ? dn[i < R - 1 ? i + 1 : 0] : box[above][2][lane];
        const T qa = i < R - 1 ? qdn[i < R - 1 ? i + 1 : 0] : box[above][3][lane];
        const T r = fma_t((T)4, t0[i], ub) + da;
        const T mx = fma_t((T)4, u0[i], qb) + qa;
        const T my = ub - da;
        const T inv = recip<T>(den0 + r);
        uint32_t bits = 0;
        if constexpr (needs_rng<C>::value) bits = sr_node_bits(key, (int64_t)lt.nx * yr[i] + xl);
        const E e0 = C::enc(div36(r), 0, bits), e1 = C::enc((mx + g36x) * inv, 1, bits),
                e2 = C::enc((my + g36y) * inv, 2, bits);
        if (!(keep_x || keep_y[i])) {
          st[i][0] = e0;
          st[i][1] = e1;
          st[i][2] = e2;
        }
      }
    }
    if constexpr (TRACE) store(dst + s * p.stride);
  }
  if constexpr (!TRACE) store(dst);
}

// ------------------------------------------------------------------ launch
// Tiles: {R, NW}. One node per lane: two nodes per lane were never faster by more
// than 5% (1024^2 FP32 2.93 us a step against 3.07) and mostly slower.
static const int kMultiTiles[][2] = {{1, 16}, {2, 16}, {4, 16}, {6, 16}, {8, 8}};

int multi2d_tiles(const Layout& L, const StepParams& p, const Multi2DShape& sh, int halo) {
  return multi_tiles_x((int)L.nx, !p.fixed[0], halo) * multi_tiles((int)L.ny, !p.fixed[1], sh.r * sh.nw, halo, false);
}

bool multi2d_shape_valid(const Layout& L, const StepParams& p, const Multi2DShape& sh) {
  bool known = false;
  for (const auto& t : kMultiTiles) known |= t[0] == sh.r && t[1] == sh.nw;
  // something of a tile must be left after the overlap
  return known && sh.steps >= 2 && sh.steps <= multi2d_steps_max(sh) && fast2d_supported(L, p);
}

// The steps of a launch for a tile, from a model of the time: a launch costs 3.6 us
// and the transfer of the state; a step costs a CU a fixed time for every row
// of 64 nodes of its tiles (FP32 0.019 us, FP64 0.032, and 0.037 where values are
// encoded and decoded between steps), at least 0.4 us for its chain and barrier.
// More steps share the launch and the transfer, and lose more of a tile to the
// overlap. Measured, us a step in one launch per step, then at the best
// tile and T: 20x51 FP64 5.08, 1.19 (1x16, T 6); 64^2 FP64 5.3, 1.18 (1x16, 6); 401^2
// FP64 6.0, 1.69 (2x16, 8); 512^2 FP32 5.5, 1.69 (4x16, 12); 1024^2 FP32 6.9, 3.07
// (4x16, 8), FP64 9.7, 5.3; 2048^2 FP32 17.4, 8.45 (8x8, 4); 4096^2 FP32 82.9, 33.0
// (8x8, 6), bound by instructions, not by memory.
static double multi2d_cost(double state_bytes, int64_t tiles, const Multi2DShape& sh, int precision, int cus) {
  const int rows = sh.r * sh.nw, steps = sh.steps;
  double row = precision == MACLAB_FP32 ? 0.019 : (precision == MACLAB_FP64 ? 0.032 : 0.037);
  // With many tiles, FP32: the barriers of 8 wavefronts hold up less than those
  // of 16 (2048^2 8.5 us a step in 8x8 tiles, 9.3 in 4x16; 4096^2 32.7, 38.3). FP64: 8 rows a wavefront leave one workgroup to a CU, and
  // the tallest tile of 16 wavefronts loses least to the overlap (2048^2 20.4 in
  // 8x8, 18.0 in 6x16, 19.5 in 4x16).
  if (tiles > 4 * (int64_t)cus) {
    if (precision == MACLAB_FP64)
      row *= sh.r == 6 ? 0.9 : (sh.r == 8 ? 1.05 : 1.0);
    else if (sh.r == 8)
      row *= 0.9;
  }
  // tiles fill the CUs one by one; past a few each the share is continuous
  const double per_cu = tiles <= 4 * (int64_t)cus ? (double)((tiles + cus - 1) / cus) : (double)tiles / cus;
  const double step = per_cu * rows * row;
  return (3.6 + 2.0 * state_bytes / 8e6 + steps * (step > 0.4 ? step : 0.4)) / steps;
}

// The shapes in the order of their modelled time, one for each tile, for lattices
// of the given tile counts (`tiles(shape)` in all); returns how many.
template <class F>
static int multi2d_rank(double state_bytes, int precision, int cus, Multi2DShape* out, int max_out, F&& tiles) {
  Multi2DShape all[5];
  double cost[5];
  int n = 0;
  for (const auto& t : kMultiTiles) {
    // 6x16 pays where a step has more work a node (1024^2 FP64 5.8 -> 5.2 us a step,
    // split-bf16 4.6 -> 4.1, S16 5.2 -> 4.0); in FP32 it is even with 8x8 or behind
    if (t[0] == 6 && precision == MACLAB_FP32) continue;
    Multi2DShape best, sh;
    double best_cost = 1e300;
    sh.r = t[0];
    sh.nw = t[1];
    for (sh.steps = 2; sh.steps <= multi2d_steps_max(sh); ++sh.steps) {
      const int64_t count = tiles(sh);
      const double c = multi2d_cost(state_bytes, count, sh, precision, cus);
      if (c < best_cost && multi2d_fits(count, sh)) {
        best_cost = c;
        best = sh;
      }
    }
    if (best.steps == 0) continue;
    int at = n++;
    for (; at > 0 && cost[at - 1] > best_cost; --at) {
      cost[at] = cost[at - 1];
      all[at] = all[at - 1];
    }
    cost[at] = best_cost;
    all[at] = best;
  }
  if (n > max_out) n = max_out;
  for (int i = 0; i < n; ++i) out[i] = all[i];
  return n;
}

int multi2d_shapes(const Layout& L, const StepParams& p, int cus, Multi2DShape* out, int max_out) {
  if (!fast2d_supported(L, p)) return 0;
  return multi2d_rank((double)L.state_bytes, L.precision, cus, out, max_out,
                      [&](const Multi2DShape& s) { return (int64_t)multi2d_tiles(L, p, s, s.steps); });
}

int multi2d_batch_shapes(const Layout* L, const StepParams* p, int count, int cus, Multi2DShape* out, int max_out) {
  double bytes = 0;
  for (int i = 0; i < count; ++i) bytes += (double)L[i].state_bytes;
  return multi2d_rank(bytes, L[0].precision, cus, out, max_out, [&](const Multi2DShape& s) {
    int64_t n = 0;
    for (int i = 0; i < count; ++i) n += multi2d_tiles(L[i], p[i], s, s.steps);
    return n;
  });
}

template <class C, int R, int NW, bool NT, bool TRACE>
static hipError_t launch_multi(const void* src, void* dst, const Multi2DParams& mp, int tiles, hipStream_t s) {
  using E = typename C::elem;
  hipLaunchKernelGGL((step_d2q9_multi<C, R, NW, NT, TRACE>), dim3(tiles), dim3(64 * NW), 0, s, (const E*)src, (E*)dst,
                     mp);
  return hipGetLastError();
}

template <class C, bool NT, bool TRACE>
static hipError_t launch_multi_tile(const Multi2DShape& sh, const void* src, void* dst, const Multi2DParams& mp,
                                    int tiles, hipStream_t s) {
  if (sh.r == 1 && sh.nw == 16) return launch_multi<C, 1, 16, NT, TRACE>(src, dst, mp, tiles, s);
  if (sh.r == 2 && sh.nw == 16) return launch_multi<C, 2, 16, NT, TRACE>(src, dst, mp, tiles, s);
  if (sh.r == 4 && sh.nw == 16) return launch_multi<C, 4, 16, NT, TRACE>(src, dst, mp, tiles, s);
  if (sh.r == 6 && sh.nw == 16) return launch_multi<C, 6, 16, NT, TRACE>(src, dst, mp, tiles, s);
  if (sh.r == 8 && sh.nw == 8) return launch_multi<C, 8, 8, NT, TRACE>(src, dst, mp, tiles, s);
  return hipErrorInvalidValue;
}

template <bool NT, bool TRACE>
static hipError_t launch_multi_codec(int precision, const Multi2DShape& sh, const void* src, void* dst,
                                     const Multi2DParams& mp, int tiles, hipStream_t s) {
  switch (precision) {
    case MACLAB_FP64: return launch_multi_tile<CodecF64, NT, TRACE>(sh, src, dst, mp, tiles, s);
    case MACLAB_FP32: return launch_multi_tile<CodecF32, NT, TRACE>(sh, src, dst, mp, tiles, s);
    case MACLAB_HILO: return launch_multi_tile<CodecHILO, NT, TRACE>(sh, src, dst, mp, tiles, s);
    case MACLAB_S16: return launch_multi_tile<CodecS16, NT, TRACE>(sh, src, dst, mp, tiles, s);
  }
  return hipErrorInvalidValue;
}

// The parameters and the tile count of one lattice's launch.
static int multi_params(const Layout& L, const StepParams& p, const Multi2DShape& sh, int steps, Multi2DParams* mp) {
  *mp = Multi2DParams{};
  Lattice2D& lt = mp->one;
  lt.nx = (int)L.nx;
  lt.ny = (int)L.ny;
  lt.pitch = (int)L.px;
  lt.xper = !p.fixed[0];
  lt.yper = !p.fixed[1];
  lt.gx = p.g[0];
  lt.gy = p.g[1];
  lt.base = 0;
  lt.plane = L.plane;
  mp->halo = steps;
  mp->nxt = multi_tiles_x(lt.nx, lt.xper, steps);
  mp->nyt = multi_tiles(lt.ny, lt.yper, sh.r * sh.nw, steps, false);
  mp->steps = steps;
  mp->rho_ref = p.rho_ref;
  mp->seed = p.seed;
  mp->step = p.step;
  return mp->nxt * mp->nyt;
}

hipError_t launch_multi2d(const Layout& L, const void* src, void* dst, const StepParams& p, const Multi2DShape& sh,
                          int steps, hipStream_t s) {
  if (!multi2d_shape_valid(L, p, sh) || steps < 1 || steps > sh.steps) return hipErrorInvalidValue;
  Multi2DParams mp;
  const int tiles = multi_params(L, p, sh, steps, &mp);
  // stores past the caches for a state larger than the memory-side cache, as
  // in the single-step kernel
  return L.state_bytes >= kStreamStoreBytes ? launch_multi_codec<true, false>(L.precision, sh, src, dst, mp, tiles, s)
                                            : launch_multi_codec<false, false>(L.precision, sh, src, dst, mp, tiles, s);
}

hipError_t launch_multi2d_trace(const Layout& L, const void* src, void* states, const StepParams& p,
                                const Multi2DShape& sh, int steps, hipStream_t s) {
  if (!multi2d_shape_valid(L, p, sh) || steps < 1 || steps > sh.steps) return hipErrorInvalidValue;
  Multi2DParams mp;
  const int tiles = multi_params(L, p, sh, steps, &mp);
  mp.stride = (int64_t)(L.state_bytes / (size_t)L.bytes);
  return launch_multi_codec<false, true>(L.precision, sh, src, states, mp, tiles, s);
}

hipError_t launch_multi2d_items(int precision, const Multi2DShape& sh, const void* src, void* dst, const Lattice2D* lat,
                                const int4* items, int nitems, int steps, double rho_ref, uint64_t seed, uint64_t step,
                                bool stream_stores, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  if (steps < 1 || steps > sh.steps) return hipErrorInvalidValue;
  Multi2DParams mp{};
  mp.lat = lat;
  mp.items = items;
  mp.nxt = mp.nyt = 1;
  mp.halo = sh.steps;  // the items' tiles, whatever the steps of this launch
  mp.steps = steps;
  mp.rho_ref = rho_ref;
  mp.seed = seed;
  mp.step = step;
  return stream_stores ? launch_multi_codec<true, false>(precision, sh, src, dst, mp, nitems, s)
                       : launch_multi_codec<false, false>(precision, sh, src, dst, mp, nitems, s);
}

}  // namespace maclab
