// Several reverse steps of the D2Q9 MacLAB step in one launch for gfx950.
//
// A reverse step of one launch takes the latency of the launch and of one load
// chain (8 us on a 512^2 lattice, whose bytes take 1.3 us). Here a workgroup
// loads a tile of the adjoint, takes it back T steps in registers, reading the
// velocity of each step's state as it goes, and stores the part that T steps of
// missing neighbours have not reached. Measured, us a step with the recomputed
// forward step: 512^2 FP32 9.8 with one step per launch each, 3.7 with five of
// both; 64^2 FP64 7.5, 3.1; 1000x900 FP32 18.8, 9.1; 2048^2 FP32 65.9, 40.4 (bound by
// the velocities' and states' bytes and by instructions).
//
// Tiles, overlap and the exchange through LDS are those of the forward kernel
// of several steps (kernels_2d_multi.hip); the formulas and their order are those
// of the single reverse step (adjoint_d2q9_fast in kernels_adjoint.hip), so the
// adjoint has its bits. The derivative with respect to the force is summed per
// wavefront in FP64 and added once per step to a slot that the same wavefront owns:
// its value does not depend on how a sweep is cut into launches.
#include "d2q9.h"
#include "internal.h"

namespace maclab {

struct AdjMulti2DParams {
  int nx, ny, xper, yper;
  int64_t pitch, plane;   // elements
  int nxt, halo, steps;
  const char* ckpt;       // state 0 of the segment ...
  const char* states;     // ... and states 1, 2, ... behind each other
  int64_t state_bytes;
  int first;              // state of the first reverse step (then first - 1, ...)
};

// Time of a row of 64 nodes of a tile on a CU, us a step.
constexpr double kRowF32 = 0.03, kRowF64 = 0.045;

// Sum over the 64 lanes by DPP row shifts and broadcasts (no LDS
// access, whose latency would add to every step).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffff), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double lanes_sum(double v) {
  v = dpp_add<0x111>(v);  // row_shr:1
  v = dpp_add<0x112>(v);  // row_shr:2
  v = dpp_add<0x114>(v);  // row_shr:4
  v = dpp_add<0x118>(v);  // row_shr:8
  // lane 15 of each row of 16 holds its sum
  const long long b = __double_as_longlong(v);
  auto row = [&](int lane) {
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  };
  return ((row(15) + row(31)) + row(47)) + row(63);
}

template <class C, int R, int NW>
__global__ __launch_bounds__(64 * NW) void adjoint_d2q9_multi(const typename C::T* __restrict__ bn1,
                                                             typename C::T* __restrict__ bn, AdjMulti2DParams p,
                                                             double* __restrict__ gslots) {
#pragma clang fp contract(off)
  using T = typename C::T;
  using E = typename C::elem;
  constexpr int SW = 64;
  // per wavefront: the three sums for the row above it and for the row below it
  __shared__ T lds[2][NW][6][SW];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nblk = (int)gridDim.x, bid = (int)blockIdx.x;
  const int per = nblk >> 3, rem = nblk & 7, xcd = bid & 7;
  const int g = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);  // XCD k takes a contiguous range of tiles
  const MultiSpan sx = multi_span(p.nx, p.xper, SW, p.halo, g % p.nxt, p.xper && p.nx == SW);
  const MultiSpan sy = multi_span(p.ny, p.yper, R * NW, p.halo, g / p.nxt, false);
  const int xb = sx.start + lane, yb = sy.start + R * wv;
  const int xl = p.xper ? wrap_near(xb, p.nx) : xb;
  const bool in_row = p.xper || xb < p.nx;
  const bool active = yb < sy.hi + p.halo && (p.yper || yb < p.ny);
  const bool own_x = xb >= sx.lo && xb < sx.hi;
  const bool fixed_x = !p.xper && (xb == 0 || xb >= p.nx - 1);
  int64_t at[R];  // element of row i in a plane; negative: none
  bool own[R], fixed[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int y = yb + i, yw = p.yper ? wrap_near(y, p.ny) : y;
    at[i] = active && in_row && (p.yper || y < p.ny) ? p.pitch * yw + xl : -1;
    own[i] = own_x && y >= sy.lo && y < sy.hi;
    fixed[i] = fixed_x || (!p.yper && (y == 0 || y >= p.ny - 1));
  }
  // A plane of the adjoint may exceed a buffer resource's range: plain loads.
  T P[R], Mx[R], My[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const bool ok = at[i] >= 0;
    P[i] = ok ? bn1[at[i]] : (T)0;
    Mx[i] = ok ? bn1[p.plane + at[i]] : (T)0;
    My[i] = ok ? bn1[2 * p.plane + at[i]] : (T)0;
  }
  E ux[R], uy[R];
  auto load_u = [&](int n) {
    const char* const s = n == 0 ? p.ckpt : p.states + (int64_t)(n - 1) * p.state_bytes;
    const E* const u = reinterpret_cast<const E*>(s) + p.plane;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool ok = at[i] >= 0;
      ux[i] = ok ? u[at[i]] : E{};
      uy[i] = ok ? u[p.plane + at[i]] : E{};
    }
  };
  load_u(p.first);
  const T k36 = (T)(1.0 / 36.0);
  double* const slot = gslots + ((int64_t)g * NW + wv) * 4;
  double sum_x = slot[0], sum_y = slot[1];
  for (int s = 0; s < p.steps; ++s) {
    T (*const box)[6][SW] = lds[s & 1];
    T a0[R], a1[R], a2[R], b0[R], b1[R], b2[R], vx[R], vy[R];
    if (active) {
      double gx = 0, gy = 0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if (own[i]) {
          gx += (double)Mx[i];
          gy += (double)My[i];
        }
        const T PL = dpp_from_left(P[i]), XL = dpp_from_left(Mx[i]), YL = dpp_from_left(My[i]);
        const T PR = dpp_from_right(P[i]), XR = dpp_from_right(Mx[i]), YR = dpp_from_right(My[i]);
        const T sP = PL + PR, dX = XR - XL, sY = YL + YR;
        a2[i] = sP + dX;
        a0[i] = fma_t((T)4, P[i], a2[i]);
        a1[i] = (PR - PL) + (XR + XL);
        b0[i] = fma_t((T)4, My[i], sY);
        b1[i] = YR - YL;
        b2[i] = sY;
        vx[i] = C::dec(ux[i], 1);
        vy[i] = C::dec(uy[i], 2);
      }
      box[wv][0][lane] = a0[R - 1] - b0[R - 1];
      box[wv][1][lane] = a1[R - 1] - b1[R - 1];
      box[wv][2][lane] = a2[R - 1] - b2[R - 1];
      box[wv][3][lane] = a0[0] + b0[0];
      box[wv][4][lane] = a1[0] + b1[0];
      box[wv][5][lane] = a2[0] + b2[0];
      sum_x += lanes_sum(gx);
      sum_y += lanes_sum(gy);
      if (s + 1 < p.steps) load_u(p.first - s - 1);
    }
    __syncthreads();
    if (active) {
      const int below = wv > 0 ? wv - 1 : 0, above = wv < NW - 1 ? wv + 1 : NW - 1;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int im = i > 0 ? i - 1 : 0, ip = i < R - 1 ? i + 1 : 0;
        const T m0 = i > 0 ? a0[im] - b0[im] : box[below][0][lane], m1 = i > 0 ? a1[im] - b1[im] : box[below][1][lane],
                m2 = i > 0 ? a2[im] - b2[im] : box[below][2][lane];
        const T pa0 = i < R - 1 ? a0[ip] + b0[ip] : box[above][3][lane],
                pa1 = i < R - 1 ? a1[ip] + b1[ip] : box[above][4][lane],
                pa2 = i < R - 1 ? a2[ip] + b2[ip] : box[above][5][lane];
        const T S2yy = (m0 + pa0) * k36;
        const T S1y = (pa0 - m0) * k36;
        const T S0 = fma_t((T)4, a0[i], m0 + pa0) * k36;
        const T S2xy = (pa1 - m1) * k36;
        const T S1x = fma_t((T)4, a1[i], m1 + pa1) * k36;
        const T S2xx = fma_t((T)4, a2[i], m2 + pa2) * k36;
        const T u = vx[i], v = vy[i];
        const T uu = fma_t(u, u, v * v);
        const T su = fma_t(S2xx, u, S2xy * v), sv = fma_t(S2xy, u, S2yy * v);
        const T quad = fma_t(u, su, v * sv);
        P[i] = fixed[i] ? (T)0 : fma_t(S0, fma_t((T)1.5, uu, (T)1), (T)-4.5 * quad);
        Mx[i] = fixed[i] ? (T)0 : fma_t((T)3, S1x, fma_t((T)9, su, (T)-3 * u * S0));
        My[i] = fixed[i] ? (T)0 : fma_t((T)3, S1y, fma_t((T)9, sv, (T)-3 * v * S0));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (own[i]) {
      bn[at[i]] = P[i];
      bn[p.plane + at[i]] = Mx[i];
      bn[2 * p.plane + at[i]] = My[i];
    }
  }
  if (lane == 0) {
    slot[0] = sum_x;
    slot[1] = sum_y;
  }
}

// ------------------------------------------------------------------ launch
// The tile and the steps of a launch, for the lattice and its faces alone (the
// slots of the force derivative are laid out for them, and a slot's sum must
// not depend on the launch): the model of the forward kernel of several steps
// with the times of this one.
Multi2DShape adjoint_multi_shape(const Layout& L, bool fixed_x, bool fixed_y) {
  Multi2DShape best;
  if (L.q != 9 || L.ny < 3 || L.nx < (fixed_x ? 3 : 1)) return best;
  const double row = L.precision == MACLAB_FP64 ? kRowF64 : kRowF32;
  constexpr int kCus = 256;
  double best_cost = 1e300;
  for (int r : {1, 2, 4}) {
    if (r == 4 && L.precision == MACLAB_FP64) continue;  // its registers do not fit 16 wavefronts
    Multi2DShape sh;
    sh.r = r;
    sh.nw = 16;
    for (sh.steps = 2; sh.steps <= multi2d_steps_max(sh); ++sh.steps) {
      const int64_t tiles = adjoint_multi_tiles(L, fixed_x, fixed_y, sh);
      const double per_cu = tiles <= 4 * kCus ? (double)((tiles + kCus - 1) / kCus) : (double)tiles / kCus;
      const double step = per_cu * sh.r * sh.nw * row;
      const double cost = (4.0 + 2.0 * (double)L.state_bytes / 8e6) / sh.steps + (step > 0.7 ? step : 0.7);
      if (cost < best_cost) {
        best_cost = cost;
        best = sh;
      }
    }
  }
  return best;
}

int64_t adjoint_multi_tiles(const Layout& L, bool fixed_x, bool fixed_y, const Multi2DShape& sh) {
  return (int64_t)multi_tiles_x((int)L.nx, !fixed_x, sh.steps) *
         multi_tiles((int)L.ny, !fixed_y, sh.r * sh.nw, sh.steps, false);
}

template <class C>
static hipError_t launch_adjoint_multi_r(const Multi2DShape& sh, const void* an1, void* an, const AdjMulti2DParams& ap,
                                         int tiles, double* gslots, hipStream_t s) {
  using T = typename C::T;
  const dim3 grid(tiles), block(64 * sh.nw);
  switch (sh.r) {
    case 1:
      hipLaunchKernelGGL((adjoint_d2q9_multi<C, 1, 16>), grid, block, 0, s, (const T*)an1, (T*)an, ap, gslots);
      break;
    case 2:
      hipLaunchKernelGGL((adjoint_d2q9_multi<C, 2, 16>), grid, block, 0, s, (const T*)an1, (T*)an, ap, gslots);
      break;
    case 4:
      if constexpr (sizeof(T) == 4) {
        hipLaunchKernelGGL((adjoint_d2q9_multi<C, 4, 16>), grid, block, 0, s, (const T*)an1, (T*)an, ap, gslots);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_adjoint_multi(const Layout& L, const StepParams& p, const Multi2DShape& sh, const void* ckpt,
                                const void* states, int first, int steps, const void* an1, void* an, double* gslots,
                                hipStream_t s) {
  if (sh.steps < 1 || steps < 1 || steps > sh.steps || first < steps - 1 || (sh.r != 1 && sh.r != 2 && sh.r != 4) ||
      sh.nw != 16)
    return hipErrorInvalidValue;
  AdjMulti2DParams ap{};
  ap.nx = (int)L.nx;
  ap.ny = (int)L.ny;
  ap.xper = !p.fixed[0];
  ap.yper = !p.fixed[1];
  ap.pitch = L.px;
  ap.plane = L.plane;
  ap.halo = sh.steps;  // the shape's tiles, whatever the steps of this launch
  ap.steps = steps;
  ap.nxt = multi_tiles_x(ap.nx, ap.xper, sh.steps);
  ap.ckpt = (const char*)ckpt;
  ap.states = (const char*)states;
  ap.state_bytes = (int64_t)L.state_bytes;
  ap.first = first;
  const int tiles = (int)adjoint_multi_tiles(L, p.fixed[0], p.fixed[1], sh);
  switch (L.precision) {
    case MACLAB_FP64: return launch_adjoint_multi_r<CodecF64>(sh, an1, an, ap, tiles, gslots, s);
    case MACLAB_FP32: return launch_adjoint_multi_r<CodecF32>(sh, an1, an, ap, tiles, gslots, s);
    case MACLAB_HILO: return launch_adjoint_multi_r<CodecHILO>(sh, an1, an, ap, tiles, gslots, s);
    case MACLAB_S16: return launch_adjoint_multi_r<CodecS16>(sh, an1, an, ap, tiles, gslots, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace maclab
