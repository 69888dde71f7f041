// Host-side declarations shared by the library's translation units: the
// handle, and the launchers each kernel file provides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/maclab.h"
#include "device.h"

namespace maclab {

// Values of the six faces as the kernels see them (physical units except
// where noted).
struct FaceValues {
  int kind[6];
  double rho[6];
  double u[6][3];
};

struct Layout {
  int q = 0, d = 0, precision = 0, bytes = 0;
  int64_t nx = 0, ny = 0, nz = 0, N = 0;
  int64_t px = 0;             // elements between rows (nx, or nx rounded up to 128 bytes for D2Q9)
  int64_t plane = 0;          // elements between field planes (px ny nz rounded up, plus 256)
  size_t state_bytes = 0;     // (d + 1) planes
  size_t partial_bytes = 0;   // reduction partials
  size_t staging_bytes = 0;   // host transfer staging
  size_t adjoint_bytes = 0;   // per-workgroup FP64 slots of the force adjoint (+ fold result)
  size_t workspace_bytes = 0;
};

// A state buffer at least this large does not fit in the device's 256 MB
// last-level (memory-side) cache: what one step writes is evicted before the
// next step reads it, so the D2Q9 step streams its stores past the caches.
constexpr size_t kStreamStoreBytes = size_t(256) << 20;

constexpr int kDiagBlocks = 1024;  // partial sums of the diagnostics reduction
constexpr int kDiagValues = 8;     // M, Px, Py, Pz, E, max|u~|, non-finite, pad

// Workgroups of 256 for a per-element kernel over `count` elements. A grid
// dimension holds fewer than 2^32 work-items, and lattices may have more
// nodes, so these kernels stride over the elements and the grid is capped.
inline unsigned blocks_256(int64_t count) {
  const int64_t b = (count + 255) / 256;
  return (unsigned)(b < (int64_t(1) << 20) ? (b > 0 ? b : 1) : (int64_t(1) << 20));
}

// Launchers (kernels_generic.hip). All enqueue on `s` and return the launch
// status.
hipError_t launch_step_generic(const Layout& L, const void* src, void* dst, const StepParams& p,
                               hipStream_t s);
// Face values into `count` buffers, stride_bytes apart.
hipError_t launch_impose_bc(const Layout& L, void* base, int64_t stride_bytes, int count, const FaceValues& fv,
                            double rho_ref, double e, hipStream_t s);
// Faces with a zero normal gradient (MACLAB_BC_RHO_NEUMANN: density;
// MACLAB_BC_PRESSURE: velocity) copy it from their nearest interior nodes in
// `buf`; nothing is launched when no face is of those kinds.
bool has_derived_faces(const FaceValues& fv);
hipError_t launch_derive_faces(const Layout& L, void* buf, const FaceValues& fv, hipStream_t s);
// All fields of all nodes, from dense FP64 arrays into both buffers / to them.
hipError_t launch_encode_all(const Layout& L, void* b0, void* b1, const double* rho, const double* u, double rho_ref,
                             double e, hipStream_t s);
hipError_t launch_decode_all(const Layout& L, double* rho, double* u, const void* state, double rho_ref, double e,
                             hipStream_t s);
// Dense nodes first .. first+count-1 of one field plane (dense index: x
// fastest over nx, no row padding) from / to FP64 arrays of count values.
hipError_t launch_encode(const Layout& L, void* plane_dst, const double* src, int64_t first, int64_t count,
                         double offset, double mul, int field, hipStream_t s);
hipError_t launch_decode(const Layout& L, double* dst, const void* plane_src, int64_t first, int64_t count,
                         double offset, double mul, int field, hipStream_t s);
// Largest change of u~ and of drho from state `prev` to state `cur` and the
// count of non-finite nodes in `cur`, into result[0..2] (FP64, in storage
// units); partials holds kDiagBlocks x 4 doubles.
hipError_t launch_residual(const Layout& L, const void* prev, const void* cur, double* partials, double* result,
                           hipStream_t s);
// Streaming copy of `bytes` (a multiple of 16; 16-byte aligned, disjoint).
hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t s);
// Reads `bytes` (a multiple of 16, 16-byte aligned) with ordinary cached loads
// and keeps nothing (`sink` is written only if the data hash equals `key`,
// so the loads stay): it fills the caches with this buffer.
hipError_t launch_touch(const void* buf, size_t bytes, uint32_t* sink, uint32_t key, hipStream_t s);
hipError_t launch_diagnostics(const Layout& L, const void* state, double rho_ref, double e, double* partials,
                              double* result, hipStream_t s);

// Fast D3Q19 path (kernels_fast.hip). `supported` tells whether the fast
// kernels handle the layout; a FastShape selects one and its tiling.
// kind 0 (LDS exchange): W output rows per workgroup (one wavefront each,
// plus two halo rows), nyb x nzb workgroups with balanced ranges, pf source
// planes loaded ahead. kind 1 (independent wavefronts): W wavefronts per
// workgroup, each owning one row and one of nzb balanced z-chunks (nyb = 1,
// pf = 1).
struct FastShape {
  int W = 8, nyb = 1, nzb = 1;
  int pf = 1;
  int kind = 0;
};
bool fast_step_supported(const Layout& L, const StepParams& p);
bool fast_shape_valid(const Layout& L, const StepParams& p, const FastShape& sh);
FastShape fast_default_shape(const Layout& L, const StepParams& p, int cus);
int fast_candidates(const Layout& L, const StepParams& p, int cus, FastShape* out, int max_out);
hipError_t launch_step_fast(const Layout& L, const void* src, void* dst, const StepParams& p, const FastShape& sh,
                            hipStream_t s);

// D3Q19, any lattice (kernels_rows.hip), in nzb chunks of planes; rows_chunks: the
// chunks for a lattice and its faces.
hipError_t launch_step_rows(const Layout& L, const void* src, void* dst, const StepParams& p, int nzb, hipStream_t s);
int rows_chunks(const Layout& L, const StepParams& p, int cus);
// Nodes from which the FP64 D3Q19 step may be worth a march in z (by rows, or as below).
constexpr int64_t kMarchNodes64 = 40960;

// FP64 D3Q19 path (kernels_seg.hip), the general kernel's form for FP64: rows
// of any width cut into segments of 64 kx nodes, workgroups of w output rows,
// nyb x nzb of them per segment.
struct Seg3DShape {
  int kx = 1, w = 6, nyb = 1, nzb = 1;
};
bool seg3d_supported(const Layout& L);
bool seg3d_pays(const Layout& L, const StepParams& p, int cus);
Seg3DShape seg3d_shape(const Layout& L, const StepParams& p, int cus);
hipError_t launch_step_seg(const Layout& L, const void* src, void* dst, const StepParams& p, const Seg3DShape& sh,
                           hipStream_t s);

// Fast D2Q9 path (kernels_2d.hip): one wavefront per (x-segment of 64*kx
// nodes, band of rows); nband bands per segment.
struct Fast2DShape {
  int kx = 4, nband = 1;
};
bool fast2d_supported(const Layout& L, const StepParams& p);
bool fast2d_shape_valid(const Layout& L, const StepParams& p, const Fast2DShape& sh);
Fast2DShape fast2d_default_shape(const Layout& L, const StepParams& p, int cus);
int fast2d_candidates(const Layout& L, const StepParams& p, int cus, Fast2DShape* out, int max_out);
hipError_t launch_step_fast2d(const Layout& L, const void* src, void* dst, const StepParams& p,
                              const Fast2DShape& sh, hipStream_t s);

// Where one lattice of a batch lives in memory and how its boundaries behave
// (elements relative to the batch's state buffer).
struct Lattice2D {
  int nx, ny, pitch;  // node counts; elements between rows (>= nx)
  int xper, yper;     // periodic axes (else both faces fixed)
  double gx, gy;      // dt G / e
  int64_t base;       // element offset of the lattice's first field plane
  int64_t plane;      // elements between field planes
};
// A batch step: work item {lattice, x0, y0, y1} of a device table, one
// wavefront each, all lattices in one launch (every pitch a multiple of kx).
// stream_stores: non-temporal stores (a state buffer of kStreamStoreBytes or
// more).
hipError_t launch_step_fast2d_items(int precision, int kx, const void* src, void* dst, const Lattice2D* lat,
                                    const int4* items, int nitems, double rho_ref, uint32_t sr_key,
                                    bool stream_stores, hipStream_t s);

// Several D2Q9 steps per launch (kernels_2d_multi.hip): tiles of 64 nodes by
// r nw rows that overlap by the steps of the launch (`steps`, at most) on each
// side. multi2d_shapes: the best ones by a model of their time, best first.
struct Multi2DShape {
  int r = 1, nw = 16, steps = 0;  // steps 0: not used
};
constexpr int kMultiStepsMax = 12;  // steps of one launch
constexpr int kMultiRowsMin = 4;    // rows a tile stores, at least
inline int multi2d_steps_max(const Multi2DShape& sh) {
  const int by_rows = (sh.r * sh.nw - kMultiRowsMin) / 2;
  return by_rows < kMultiStepsMax ? by_rows : kMultiStepsMax;
}
// Whether a launch of so many tiles is within the 2^32 work-items of a grid dimension.
inline bool multi2d_fits(int64_t tiles, const Multi2DShape& sh) { return tiles * 64 * sh.nw < int64_t(1) << 32; }
bool multi2d_shape_valid(const Layout& L, const StepParams& p, const Multi2DShape& sh);
int multi2d_tiles(const Layout& L, const StepParams& p, const Multi2DShape& sh, int halo);
int multi2d_shapes(const Layout& L, const StepParams& p, int cus, Multi2DShape* out, int max_out);
int multi2d_batch_shapes(const Layout* L, const StepParams* p, int count, int cus, Multi2DShape* out, int max_out);
hipError_t launch_multi2d(const Layout& L, const void* src, void* dst, const StepParams& p, const Multi2DShape& sh,
                          int steps, hipStream_t s);
// `steps` steps from the state at src, each step's state stored: at `states`,
// one behind the other (L.state_bytes apart).
hipError_t launch_multi2d_trace(const Layout& L, const void* src, void* states, const StepParams& p,
                                const Multi2DShape& sh, int steps, hipStream_t s);
// The same for a batch: work items {lattice, x tile, y tile, 0} with the tiles
// of sh.steps, advanced by `steps` <= sh.steps.
hipError_t launch_multi2d_items(int precision, const Multi2DShape& sh, const void* src, void* dst, const Lattice2D* lat,
                                const int4* items, int nitems, int steps, double rho_ref, uint64_t seed, uint64_t step,
                                bool stream_stores, hipStream_t s);

// Tiles of `size` nodes along an axis of n nodes that overlap by h on each
// side. Periodic: tile k stores size - 2h nodes from k (size - 2h) and begins h
// before them (`wraps`: one tile is the whole axis). Between fixed faces the
// first tile begins and the last one ends at the face, without overlap there.
struct MultiSpan {
  int start, lo, hi;  // first node of the tile; nodes [lo, hi) that it stores
};
__host__ __device__ inline int multi_tiles(int n, int per, int size, int h, bool wraps) {
  if (wraps || (!per && n <= size)) return 1;
  const int u = size - 2 * h;
  return per ? (n + u - 1) / u : (n - 2 * h + u - 1) / u;
}
__host__ __device__ inline MultiSpan multi_span(int n, int per, int size, int h, int k, bool wraps) {
  if (wraps || (!per && n <= size)) return {0, 0, n};
  const int u = size - 2 * h;
  if (per) {
    const int hi = (k + 1) * u;
    return {k * u - h, k * u, hi < n ? hi : n};
  }
  const int last = k * u + size >= n;
  return {k * u, k == 0 ? 0 : k * u + h, last ? n : k * u + h + u};
}
// v wrapped into 0 .. n-1. A step across an edge takes two comparisons; the
// remainder, some forty instructions, only where a tile is wider than the axis.
__host__ __device__ inline int wrap_near(int v, int n) {
  v = v < 0 ? v + n : (v >= n ? v - n : v);
  return v >= 0 && v < n ? v : (v % n + n) % n;
}
inline int multi_tiles_x(int nx, int xper, int halo) { return multi_tiles(nx, xper, 64, halo, xper && nx == 64); }

// Reverse mode (kernels_adjoint.hip). Adjoint buffers hold (Rbar, Mbar) in
// the compute type, d + 1 planes of `plane` elements.
int64_t adjoint_slots(const Layout& L);
hipError_t launch_adjoint_step(const Layout& L, const void* sn, const void* an1, void* an, const StepParams& p,
                               double* gslots, hipStream_t s);
bool adjoint2d_supported(const Layout& L, const StepParams& p);
bool adjoint2d_shape_valid(const Layout& L, const StepParams& p, const Fast2DShape& sh);
Fast2DShape adjoint2d_default_shape(const Layout& L, const StepParams& p, int cus);
hipError_t launch_adjoint_fast2d(const Layout& L, const void* sn, const void* an1, void* an, const StepParams& p,
                                 const Fast2DShape& sh, double* gslots, hipStream_t s);
// Several reverse steps per launch (kernels_adjoint_multi.hip), D2Q9: states
// first, first - 1, ... of a segment (state 0 at ckpt, 1, 2, ... at states), the
// adjoint after the first of them at an1, the one before the last written to an.
Multi2DShape adjoint_multi_shape(const Layout& L, bool fixed_x, bool fixed_y);
int64_t adjoint_multi_tiles(const Layout& L, bool fixed_x, bool fixed_y, const Multi2DShape& sh);
hipError_t launch_adjoint_multi(const Layout& L, const StepParams& p, const Multi2DShape& sh, const void* ckpt,
                                const void* states, int first, int steps, const void* an1, void* an, double* gslots,
                                hipStream_t s);
hipError_t launch_adjoint_seed(const Layout& L, const void* sT, const double* dLdu, void* adj, const StepParams& p,
                               double e, hipStream_t s);
hipError_t launch_adjoint_result(const Layout& L, const void* s0, const void* adj, double* dLdu, double* dLdrho,
                                 double rho_ref, double e, hipStream_t s);
hipError_t launch_adjoint_fold(const double* slots, int64_t nslots, double* out, hipStream_t s);
hipError_t launch_zero_doubles(double* dst, int64_t count, hipStream_t s);

// Lattice BGK with tau = 1, populations stored (kernels_bgk.hip): Q planes
// of `plane` elements, dense rows, FP64 or FP32 deviations F_a - w_a rho_ref.
struct BgkParams {
  int64_t nx, ny, nz;   // node counts
  int64_t plane;        // elements between population planes
  int fixed[3];         // 1 if both faces of the axis are fixed
  double rho_ref;       // density the stored deviations refer to
  double g[3];          // dt G / e
};
hipError_t launch_bgk_step(int q, bool fp64, const BgkParams& p, const void* src, void* dst, hipStream_t s);
hipError_t launch_bgk_encode(int q, bool fp64, void* dst, int64_t plane, const double* rho, const double* ux,
                             const double* uy, const double* uz, int64_t first, int64_t count, double rho_ref,
                             double e, hipStream_t s);
hipError_t launch_bgk_decode(int q, bool fp64, const void* src, int64_t plane, double* rho, double* ux, double* uy,
                             double* uz, int64_t first, int64_t count, double rho_ref, double e, hipStream_t s);
hipError_t launch_bgk_impose(int q, bool fp64, void* b0, void* b1, const BgkParams& p, const FaceValues& fv, double e,
                             hipStream_t s);

}  // namespace maclab
