// HIP kernels for gfx950 and the C ABI of include/hweno.h.
//
// One workgroup advances one tile of cells through one Runge-Kutta stage
// (or evaluates the right-hand side on it):
//   1. the tile plus a two-cell halo of every field is staged in LDS with
//      coalesced row loads (boundary conditions are index maps on these
//      loads; there is no ghost-fill pass);
//   2. one thread per x-interface computes all interface fluxes
//      (characteristic HWENO f-hat, linear h-hat, mixed eta-hat) into an LDS
//      flux buffer; each thread then differences the two interfaces of its
//      own cell;
//   3. the same for the y-interfaces (same code, momenta swapped on load);
//   4. each thread limits the derivatives of its cell, applies the SSP-RK3
//      combination, stores its cell, and contributes its wave speeds to a
//      workgroup max that is folded into the next stage's global speed with
//      one 64-bit atomic max on the IEEE bit pattern.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/hweno.h"
#include "hweno_adjoint.h"
#include "hweno_math.h"

namespace hweno {

// ---------------------------------------------------------------------------
// launch arguments
// ---------------------------------------------------------------------------
template <typename T>
struct StageArgs {
  const T* in;        // stage input S_k (state layout)
  T* out;             // S_{k+1}, or the right-hand side (K == 0)
  const T* st0;       // S^n (stages 2 and 3 read U^n, and all of S^n without limiter)
  T* base;            // limited derivatives of S^n (written by stage 1, read by 2, 3)
  double* ctrl;       // step control block (stages only)
  double* fold;       // speed slots (stages only; see NSLOT)
  int slots;          // how many of them this grid uses: 1 or NSLOT
  unsigned long long* status;  // status word, or NULL
  const double* alpha;  // speeds for K == 0
  int nx, ny, bc_x, bc_y;
  long long fs;       // field stride nx * ny
  double dx, dy;
  double dt_fixed, t_end, cfl;
  int replay;
  int fold_next;      // stage 3 folds the new state's speeds for the next step
};

__device__ __forceinline__ int map_index(int i, int n, int bc) {
  if (bc == HWENO_BC_PERIODIC) {
    i %= n;
    return i < 0 ? i + n : i;
  }
  if (bc == HWENO_BC_REFLECT) {
    // mirror images repeat with period 2n; reducing first keeps every index
    // in range (halo loads deeper than n are never used in a result)
    i %= 2 * n;
    if (i < 0) i += 2 * n;
    return i < n ? i : 2 * n - 1 - i;
  }
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// map_index for the stage kernels, whose results use halos at most 2 deep: a
// reflecting wall has n >= 2 cells across, so one mirror step is exact for
// -2 <= i <= n + 1.  A partial tile also stages cells further out that no
// result uses; the clamp keeps those loads inside the grid.
__device__ __forceinline__ int map_index2(int i, int n, int bc) {
  if (bc == HWENO_BC_PERIODIC) {
    i %= n;
    return i < 0 ? i + n : i;
  }
  if (bc == HWENO_BC_REFLECT) i = i < 0 ? -1 - i : (i >= n ? 2 * n - 1 - i : i);
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// true when index i is a ghost that a reflecting boundary fills with signs
__device__ __forceinline__ bool mirrored(int i, int n, int bc) {
  return bc == HWENO_BC_REFLECT && (i < 0 || i >= n);
}

// Sign of field f (layout U[0..m), U_x[0..m), U_y[0..m)) in a ghost mirrored
// across a wall normal to direction d (0 = x, 1 = y): the wall-normal momentum
// (Euler component 1 + d) is odd, and so is every derivative along d; the
// two parities multiply.
__host__ __device__ __forceinline__ int mirror_sign(int f, int m, bool euler, int d) {
  const int c = f % m, g = f / m;
  int s = (euler && c == 1 + d) ? -1 : 1;
  if (g == 1 + d) s = -s;
  return s;
}

// Sides described by hweno_edge (HWENO_BC_EDGES) in kernel-argument form;
// sides 0..3 = x_lo, x_hi, y_lo, y_hi.
struct EdgeArgs {
  int kind[4][2];
  int mirror[4];  // the side stages with the mirror map (it has a wall segment)
  double split[4][3];
  double state[4][2][4];
  double t0;      // time of the state read by the right-hand side and the limiter entry points
  int oi, oj;     // solid cells i >= oi, j < oj (oj == 0: no obstacle)
};

// cell (i, j) of the grid is solid
__device__ __forceinline__ bool solid_cell(const EdgeArgs& e, int i, int j) {
  return j < e.oj && i >= e.oi && j >= 0;
}

// map_index2 with a per-side choice between mirror and copy on edge-described
// directions; always inside the grid
__device__ __forceinline__ int map_edge(int i, int n, int bc, int mlo, int mhi) {
  if (bc != HWENO_BC_EDGES) return map_index2(i, n, bc);
  if (i < 0)
    i = mlo ? -1 - i : 0;
  else if (i >= n)
    i = mhi ? 2 * n - 1 - i : n - 1;
  return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// Segment (0 or 1) of side `side` taken by a ghost cell at position `pos`
// along the side, `depth` beyond it, at time t: split = s0 + s1 t + s2 depth,
// evaluated in that order with separately rounded products and sums.
__device__ __forceinline__ int edge_segment(const EdgeArgs& e, int side, double pos, double depth,
                                            double t) {
  const double sp = __dadd_rn(__dadd_rn(e.split[side][0], __dmul_rn(e.split[side][1], t)),
                              __dmul_rn(e.split[side][2], depth));
  return pos < sp ? 0 : 1;
}

// Loads and stores through the global address space.  Pointers that arrive
// through memory (the batched instance descriptors) are generic to the
// compiler, which then cannot rule out aliasing with the LDS tile and
// serialises every HBM load against the LDS writes around it.
template <typename T>
__device__ __forceinline__ T gld(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ void gst(T* p, T v) {
  *(__attribute__((address_space(1))) T*)p = v;
}

__device__ __forceinline__ unsigned long long dbits(double x) {
  return (unsigned long long)__double_as_longlong(x);
}

// Maximum over a wave of non-negative values, on every lane; NaN wins.  Six DPP
// moves within the vector unit: a chain of LDS permutes took a tenth of the
// time of a small grid's stage.
template <int C>
__device__ __forceinline__ float dpp_shift(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), C, 0xf, 0xf, false));
}
template <int C>
__device__ __forceinline__ double dpp_shift(double x) {
  return __hiloint2double(
      __builtin_amdgcn_update_dpp(0, __double2hiint(x), C, 0xf, 0xf, false),
      __builtin_amdgcn_update_dpp(0, __double2loint(x), C, 0xf, 0xf, false));
}
__device__ __forceinline__ float last_lane(float x) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ double last_lane(double x) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                          __builtin_amdgcn_readlane(__double2loint(x), 63));
}
template <typename T>
__device__ __forceinline__ T wave_max(T x) {
  const bool nan = __builtin_amdgcn_ballot_w64(x != x) != 0;  // fmax drops NaN
  // lanes n-1, n-2, n-4, n-8 of a row of 16, then the last lanes of rows 0 and 2
  // to rows 1 and 3, and that of the lower half to the upper one; lanes without a
  // source read 0
  x = fmax(x, dpp_shift<0x111>(x));
  x = fmax(x, dpp_shift<0x112>(x));
  x = fmax(x, dpp_shift<0x114>(x));
  x = fmax(x, dpp_shift<0x118>(x));
  x = fmax(x, dpp_shift<0x142>(x));
  x = fmax(x, dpp_shift<0x143>(x));
  return nan ? T(__builtin_nan("")) : last_lane(x);
}

// The speeds of a grid are maxima over all its workgroups.  On one address their
// atomics queue, about 15 ns each: when the workgroups of a small grid finish
// together that was a third of a 240 x 240 step.  So the workgroups of a grid fold
// into NSLOT slots, one 128-byte line each, picked by blockIdx.x, and whoever needs
// the speeds takes the maximum over the slots.  Line s holds, at
// fold[s * SLOT_LEN + 2 q + direction], the speeds of the input of stage q + 1, and
// for q = 3 those of the next step's first stage.
// SLOT_FEW workgroups or fewer do not queue long enough to pay for reading several
// lines (eight steps of 60 x 60, 16 workgroups: 288 us on one slot, 296 on eight; 160
// x 120, 80 workgroups: 337 and 298): they use slot 0 alone, as any grid does whose
// workspace has no room for more (ws_bufs).
constexpr int NSLOT = 8, SLOT_LEN = 16, SLOT_FEW = 48;

__device__ __forceinline__ int my_slot(int slots) {
  return slots > 1 ? (int)(blockIdx.x & (NSLOT - 1)) * SLOT_LEN : 0;
}

// The maxima over the slots, in two ways; NaN wins.  By lanes (0..7 the x-speeds, 8..15
// the y-speeds), loaded before anything else so that nothing waits behind the halo
// loads: the shorter wait, for workgroups that all start at once.
__device__ __forceinline__ double slot_load(const double* fold, int q) {
  const int lane = threadIdx.x & 63;
  return lane < 2 * NSLOT ? gld(fold + (lane & (NSLOT - 1)) * SLOT_LEN + 2 * q + lane / NSLOT) : 0.0;
}
__device__ __forceinline__ void slot_max(double x, double& ax, double& ay) {
  const unsigned long long nan = __builtin_amdgcn_ballot_w64(x != x);
  x = fmax(x, dpp_shift<0x111>(x));  // lanes n-1, n-2, n-4 of the row
  x = fmax(x, dpp_shift<0x112>(x));
  x = fmax(x, dpp_shift<0x114>(x));
  const double q_nan = __builtin_nan("");
  ax = nan & 0xff ? q_nan : __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 7),
                                             __builtin_amdgcn_readlane(__double2loint(x), 7));
  ay = nan & 0xff00 ? q_nan : __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 15),
                                               __builtin_amdgcn_readlane(__double2loint(x), 15));
}
// By scalar loads, which later workgroups find in the scalar cache: nothing queues
// with the halo loads (FP32, 2047 x 1531, four steps: 2.42 ms, by lanes 2.59 ms).
__device__ __forceinline__ void slot_max_scalar(const double* fold, int q, double& ax, double& ay) {
  double x = fold[2 * q], y = fold[2 * q + 1], sx = x, sy = y;
#pragma unroll
  for (int s = 1; s < NSLOT; ++s) {
    const double u = fold[s * SLOT_LEN + 2 * q], v = fold[s * SLOT_LEN + 2 * q + 1];
    x = fmax(x, u), y = fmax(y, v);
    sx += u, sy += v;  // NaN, which fmax drops, stays in the sums
  }
  ax = sx != sx ? sx : x;
  ay = sy != sy ? sy : y;
}

// workgroup reduction of two non-negative speeds (compared as bit patterns, so NaN
// wins) and of status flags; thread 0 folds them into global memory.
template <int NT, typename T>
__device__ __forceinline__ void block_fold(T sx, T sy, uint32_t flags, double* slot,
                                           unsigned long long* status, bool do_speeds) {
  __shared__ unsigned long long red[NT / 64][2];
  __shared__ uint32_t redf[NT / 64];
  sx = wave_max(sx);
  sy = wave_max(sy);
  if (__builtin_amdgcn_ballot_w64(flags != 0)) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) flags |= __shfl_xor(flags, off);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    red[wv][0] = dbits(double(sx));
    red[wv][1] = dbits(double(sy));
    redf[wv] = flags;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long bx = red[0][0], by = red[0][1];
    for (int q = 1; q < NT / 64; ++q) {
      bx = red[q][0] > bx ? red[q][0] : bx;
      by = red[q][1] > by ? red[q][1] : by;
      flags |= redf[q];
    }
    // global-address-space atomics (see gld): the slot may come from memory.
    // The slots only grow during a launch, so a value read from them is a
    // lower bound of the final maximum: a workgroup whose maximum does not
    // exceed it has nothing to add.  Once the first workgroups have folded
    // theirs, almost every later one skips its atomic, and tens of thousands
    // of read-modify-writes no longer queue on one address.  A few workgroups do
    // not queue for long, and waiting for the read would cost them more.
    using gu64 = __attribute__((address_space(1))) unsigned long long;
    if (do_speeds) {
      unsigned long long cx = 0, cy = 0;
      if (gridDim.x > 512) {
        cx = __hip_atomic_load((gu64*)slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        cy = __hip_atomic_load((gu64*)slot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (bx > cx) __hip_atomic_fetch_max((gu64*)slot, bx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (by > cy)
        __hip_atomic_fetch_max((gu64*)slot + 1, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (flags && status)
      __hip_atomic_fetch_or((gu64*)status, (unsigned long long)flags, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------
// Tile order.  Workgroups are dispatched round-robin over the 8 XCDs (each
// with its own L2); renumbering so that each XCD receives a contiguous band
// of tiles keeps the halo rows shared by neighbouring tiles in one L2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int xcd_band(int b, int nb) {
  constexpr int NXCD = 8;
  const int per = nb / NXCD;
  if (b >= per * NXCD) return b;
  return (b % NXCD) * per + (b / NXCD);
}

// Persistent variant: the tile list is cut into 8 contiguous bands, band x
// is processed by the workgroups on XCD x (blockIdx % 8 == x), in order.
// Visits every t in [0, total) exactly once; `it` counts the iterations.
struct BandIter {
  int lb, nlb, band_lo, band_hi;
  __device__ __forceinline__ BandIter(int total) {
    constexpr int NXCD = 8;
    const int nb = (int)gridDim.x;
    if (nb < NXCD) {  // too few workgroups for one band each: plain striding
      nlb = nb;
      lb = (int)blockIdx.x;
      band_lo = 0;
      band_hi = total;
      return;
    }
    const int x = (int)blockIdx.x % NXCD;
    // workgroups of XCD x: x, x+8, ... (the last band may get fewer)
    nlb = nb / NXCD + ((nb % NXCD) > x ? 1 : 0);
    lb = (int)blockIdx.x / NXCD;
    const int per = (total + NXCD - 1) / NXCD;
    band_lo = min(x * per, total);
    band_hi = min(band_lo + per, total);
  }
  __device__ __forceinline__ int tile(int it) const { return band_lo + lb + it * nlb; }
  __device__ __forceinline__ bool valid(int it) const { return tile(it) < band_hi; }
};

// the time step from the stage-1 speeds (or the given one) at time t, clipped to
// t_end; 0 when it is not positive and finite (the step is skipped)
template <int DIM>
__device__ __forceinline__ double step_dt(double alx, double aly, double dt_fixed, double t_end,
                                          double t, double cfl, double dx, double dy) {
  double dt;
  if (dt_fixed > 0.0) {
    dt = dt_fixed;
  } else if (DIM == 1) {
    dt = cfl * dx / alx;
  } else {
    dt = cfl / (alx / dx + aly / dy);
  }
  const double left = t_end - t;
  if (t_end > 0.0 && dt > left) dt = left;  // a comparison: fmin would drop a NaN
  return (!(dt > 0.0) || !isfinite(dt)) ? 0.0 : dt;
}

// time step of stage K (uniform per grid), stage 1's from the speeds alx, aly; false
// when the step is skipped.  last, t: the control block's time step and time.
template <int DIM, int K>
__device__ __forceinline__ bool stage_dt(double* ctrl, double last, double t, double alx, double aly,
                                         double dt_fixed, double t_end, double cfl, double dx,
                                         double dy, int replay, bool leader,
                                         unsigned long long* status, double& dt) {
  if (K == 1 && !replay) {
    dt = step_dt<DIM>(alx, aly, dt_fixed, t_end, t, cfl, dx, dy);
    if (leader) {
      ctrl[6] = dt;
      if (dt == 0.0) atomicOr(status, (unsigned long long)HWENO_ST_SKIPPED);
    }
  } else {
    dt = last;
  }
  return dt > 0.0;
}

// Workgroups up to which the slots are read by lanes: what the chip holds at once
// (two FP64 or four FP32 per compute unit).  Eight steps, by lanes and by scalar
// loads: FP64 480 workgroups 454 and 457 us, 552 workgroups 610 and 601 us; FP32 552
// workgroups 431 and 438 us, 1120 workgroups 631 and 625 us.
template <typename T>
__device__ __forceinline__ constexpr int slot_lanes() {
  return sizeof(T) == 4 ? 1024 : 512;
}

// What a stage reads of the control block and the slots, before anything else and in
// one go: read where each value is used, they wait one after the other (0.25 us a
// stage).
struct Early {
  double lanes;     // slot_load's
  double f0, f1;    // slot 0
  double dt, time;  // ctrl[6], ctrl[7]
};
template <typename T, int K>
__device__ __forceinline__ Early read_early(const StageArgs<T>& a) {
  Early r = {0.0, 0.0, 0.0, 0.0, 0.0};
  if constexpr (K > 0) {
    r.dt = a.ctrl[6], r.time = a.ctrl[7];
    r.f0 = a.fold[2 * (K - 1)], r.f1 = a.fold[2 * (K - 1) + 1];
    if (a.slots > 1 && (int)gridDim.x <= slot_lanes<T>()) r.lanes = slot_load(a.fold, K - 1);
  }
  return r;
}

// what a stage (K > 0) or the right-hand side reads before it computes: the time
// step and the speeds it splits with (early: read_early's); false when the step is skipped
template <int DIM, int K, typename T>
__device__ __forceinline__ bool grid_begin(const StageArgs<T>& a, const Early& early, double& dt,
                                           double& alx, double& aly) {
  if constexpr (K == 0) {
    alx = a.alpha[0];
    aly = a.alpha[1];
    return true;
  } else {
    const bool leader = blockIdx.x == 0 && threadIdx.x == 0;
    if (a.replay) {
      alx = a.ctrl[2 * (K - 1)];
      aly = a.ctrl[2 * (K - 1) + 1];
    } else {
      if (a.slots == 1)
        alx = early.f0, aly = early.f1;
      else if ((int)gridDim.x <= slot_lanes<T>())
        slot_max(early.lanes, alx, aly);
      else
        slot_max_scalar(a.fold, K - 1, alx, aly);
    }
    const bool go = stage_dt<DIM, K>(a.ctrl, early.dt, early.time, alx, aly, a.dt_fixed, a.t_end,
                                     a.cfl, a.dx, a.dy, a.replay, leader, a.status, dt);
    // a skipped step leaves the speeds of its later stages at zero
    if (!a.replay && leader && (K == 1 || go)) {
      a.ctrl[2 * (K - 1)] = alx;
      a.ctrl[2 * (K - 1) + 1] = aly;
    }
    return go;
  }
}

// the LDS rectangle of columns [c0, c1) and rows [r0, r1) holds solid cells
__device__ __forceinline__ bool obstacle_near(const EdgeArgs& e, int c0, int c1, int r0, int r1) {
  return e.oj > 0 && c1 > e.oi && r0 < e.oj && r1 > 0;
}

// Field f as the stage tile holds it: derivatives times their cell size (the
// differences and linear forms of the scheme are in these units).
template <typename T>
__device__ __forceinline__ T staged(T x, int f, int m, T dx, T dy) {
  return f < m ? x : x * (f < 2 * m ? dx : dy);
}

// Solid cells of the staged tile take the mirror image of the fluid across the
// obstacle's front face (d = 0) or top face (d = 1), with the wall signs of
// that direction, read from the stage input.  Cells deeper than two inside the
// obstacle take a clamped, finite copy; no stencil that enters a result reads
// them.  Each thread rewrites the entries it staged.
template <typename T, int M, int NF, int HR, int W, int NT>
__device__ __forceinline__ void obstacle_mirror(const StageArgs<T>& a, const EdgeArgs& e, T* sm,
                                                int i0, int j0, int HY, int d) {
  const int nx = a.nx, ny = a.ny;
  for (int q = threadIdx.x; q < W * HR; q += NT) {
    const int lr = q / W, lc = q - lr * W;
    const int ii = i0 - 2 + lc, jj = j0 - HY + lr;
    if (!solid_cell(e, ii, jj)) continue;
    int si = d == 0 ? 2 * e.oi - 1 - ii : ii;
    int sj = d == 0 ? jj : 2 * e.oj - 1 - jj;
    si = si < 0 ? 0 : (si >= nx ? nx - 1 : si);
    sj = sj < 0 ? 0 : (sj >= ny ? ny - 1 : sj);
    const long long g = (long long)sj * nx + si;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const T x = staged(gld(a.in + f * a.fs + g), f, M, T(a.dx), T(a.dy));
      sm[f * HR * W + q] = mirror_sign(f, M, true, d) < 0 ? -x : x;
    }
  }
}

// 3/4 s0 + 1/4 x (stage 2) and 1/3 s0 + 2/3 x (stage 3).  FP32: from the difference,
// one rounding besides x's own, and a cell that does not change keeps its value; as a
// weighted sum the compiler rounds one product first, which left the conserved
// fields of three steps up to 1.3 times as far from 64 bits.  FP64: the weighted sum,
// which a 64-bit evaluation cannot tell from the other (3.2e-15 and 3.5e-15 apart from
// it, 1024^2).
template <typename T>
__device__ __forceinline__ T rk_combine(int K, T s0, T x) {
  const T w0 = (K == 2) ? T(0.75) : T(1.0 / 3.0);
  const T w1 = (K == 2) ? T(0.25) : T(2.0 / 3.0);
  if constexpr (sizeof(T) == 4) return mad(w1, x - s0, s0);
  return w0 * s0 + w1 * x;
}

// ---------------------------------------------------------------------------
// One tile of one stage (K = 1, 2, 3) or of the right-hand side (K = 0).
// NT threads; TX x TY cells (TX*TY <= NT); sm, fb: LDS staging buffers.
// begin(dt, alx, aly): the time step and the speeds from the control block, false
// when the step is skipped.
// Returns this thread's contribution to the next stage's speeds.
// ---------------------------------------------------------------------------
// MODE: which fields the reconstruction and the limiter of the Euler equations
// work on, separate instantiations because a branch between them costs the
// default kernels their registers (FP64: 250 instead of 220 VGPRs).  The scalar
// laws use MODE_COMP.
// EDG: edge-described sides (2D Euler; a separate instantiation), read from *e.
enum {
  MODE_CHAR = 0,       // characteristic reconstruction, limiter component by component
  MODE_CHAR_LIM = 1,   // characteristic reconstruction and limiter
  MODE_COMP = 2        // reconstruction component by component, either limiter
};

template <typename T, int PHYS, int DIM, int K, int TX, int TY, int NT, int MODE, bool EDG = false, typename Begin>
__device__ __forceinline__ void stage_tile(const StageArgs<T>& a, const Consts<T>& k,
                                           int tile_x, int tile_y, const Begin& begin,
                                           T* __restrict__ sm, T* __restrict__ fb,
                                           T& sx, T& sy, uint32_t& flags,
                                           const EdgeArgs* e = nullptr) {
  constexpr int M = Comps<PHYS, DIM>::M;
  constexpr int NF = Comps<PHYS, DIM>::NF;
  constexpr int HY = (DIM == 2) ? 2 : 0;
  constexpr int W = TX + 4;           // LDS row length (2-cell x halo each side)
  constexpr int HR = TY + 2 * HY;     // LDS rows
  constexpr int FW = TX + 1;          // flux buffer row length
  constexpr int FR = TY + 1;          // flux buffer rows
  static_assert(TX * TY <= NT, "one cell per thread");

  const int tid = threadIdx.x;
  const int i0 = tile_x * TX;
  const int j0 = tile_y * TY;
  const int nx = a.nx, ny = a.ny;
  const long long fs = a.fs;
  const T hx = T(a.dx), hy = T(a.dy);

  // ---- stage the tile and its halo in LDS ----
  // All rounds' loads are issued before the first LDS write, and before the control
  // block is waited for.  Tiles whose halo lies inside the grid need no boundary
  // map: a uniform base and one 32-bit offset per lane (nx <= 2^24 keeps it
  // in range) serve every field.
  constexpr int NS = (W * HR + NT - 1) / NT;
  T v[NS][NF];
  const bool inner = i0 >= 2 && i0 - 2 + W <= nx && (DIM == 1 || (j0 >= HY && j0 - HY + HR <= ny)) &&
                     (DIM == 1 || nx <= (1 << 24));
  if (inner) {
    const T* src = a.in + ((long long)(j0 - HY) * nx + (i0 - 2));
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int q = tid + r * NT;
      if (q < W * HR) {
        const unsigned lr = (unsigned)q / W, lc = (unsigned)q - lr * W;
        const unsigned o = lr * (unsigned)nx + lc;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[r][f] = gld(src + f * fs + o);
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int q = tid + r * NT;
      if (q < W * HR) {
        const int lr = q / W, lc = q - lr * W;
        const int ii = i0 - 2 + lc, jj = j0 - HY + lr;
        int gi, gj;
        if constexpr (EDG) {
          gi = map_edge(ii, nx, a.bc_x, e->mirror[0], e->mirror[1]);
          gj = map_edge(jj, ny, a.bc_y, e->mirror[2], e->mirror[3]);
        } else {
          gi = map_index2(ii, nx, a.bc_x);
          gj = (DIM == 2) ? map_index2(jj, ny, a.bc_y) : 0;
        }
        const long long g = (long long)gj * nx + gi;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[r][f] = gld(a.in + f * fs + g);
      }
    }
  }
  double dt = 0.0, alx, aly;
  if (!begin(dt, alx, aly)) return;  // the step is skipped (uniform over the workgroup)
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int q = tid + r * NT;
    if (q < W * HR) {
#pragma unroll
      for (int f = 0; f < NF; ++f) sm[f * HR * W + q] = staged(v[r][f], f, M, hx, hy);
    }
  }
  if constexpr (PHYS == PH_EULER) {
    // Reflecting walls: a ghost cell holds the mirror image of an interior
    // cell with its odd fields negated.  Only tiles whose halo crosses such a
    // wall (a uniform decision) fix their LDS entries, each thread the ones it
    // stored itself, so the staging above stays the same for every tile.
    const bool wx = a.bc_x == HWENO_BC_REFLECT && (i0 - 2 < 0 || i0 - 2 + W > nx);
    const bool wy = DIM == 2 && a.bc_y == HWENO_BC_REFLECT && (j0 - HY < 0 || j0 - HY + HR > ny);
    if (wx || wy) {
      for (int q = tid; q < W * HR; q += NT) {
        const int lr = q / W, lc = q - lr * W;
        const int ii = i0 - 2 + lc, jj = j0 - HY + lr;
        const bool mx = wx && (ii < 0 || ii >= nx), my = wy && (jj < 0 || jj >= ny);
        if (!(mx || my)) continue;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const int sg = (mx ? mirror_sign(f, M, true, 0) : 1) * (my ? mirror_sign(f, M, true, 1) : 1);
          if (sg < 0) sm[f * HR * W + q] = -sm[f * HR * W + q];
        }
      }
    }
  }
  if constexpr (EDG) {
    // Edge-described sides, at the time of this stage's input: ghost cells of
    // a wall segment take the mirror signs, those of an inflow segment the
    // prescribed state with zero derivatives; outflow segments keep the copy
    // staged above.  Corner ghosts take both rules; no stencil reads them.
    const bool ex = a.bc_x == HWENO_BC_EDGES && (i0 - 2 < 0 || i0 - 2 + W > nx);
    const bool ey = a.bc_y == HWENO_BC_EDGES && (j0 - HY < 0 || j0 - HY + HR > ny);
    if (ex || ey) {
      const double te = (K == 0) ? e->t0 : a.ctrl[7] + (K == 1 ? 0.0 : (K == 2 ? dt : 0.5 * dt));
      for (int q = tid; q < W * HR; q += NT) {
        const int lr = q / W, lc = q - lr * W;
        const int ii = i0 - 2 + lc, jj = j0 - HY + lr;
        auto apply = [&](int side, int d, double pos, double depth) {
          const int sg = edge_segment(*e, side, pos, depth, te);
          const int kd = e->kind[side][sg];
          if (kd == HWENO_SEG_REFLECT) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
              if (mirror_sign(f, M, true, d) < 0) sm[f * HR * W + q] = -sm[f * HR * W + q];
          } else if (kd == HWENO_SEG_STATE) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
              sm[f * HR * W + q] = f < M ? T(e->state[side][sg][f]) : T(0);
          }
        };
        if (ex && ii < 0) apply(0, 0, (jj + 0.5) * a.dy, (-ii - 0.5) * a.dx);
        if (ex && ii >= nx) apply(1, 0, (jj + 0.5) * a.dy, (ii - nx + 0.5) * a.dx);
        if (ey && jj < 0) apply(2, 1, (ii + 0.5) * a.dx, (-jj - 0.5) * a.dy);
        if (ey && jj >= ny) apply(3, 1, (ii + 0.5) * a.dx, (jj - ny + 0.5) * a.dy);
      }
    }
    // Obstacle, x-interfaces: a solid cell holds the mirror image of the fluid
    // across the front face x = oi dx (read from the stage input, wall signs)
    if (obstacle_near(*e, i0 - 2, i0 - 2 + W, j0 - HY, j0 - HY + HR))
      obstacle_mirror<T, M, NF, HR, W, NT>(a, *e, sm, i0, j0, HY, 0);
  }
  __syncthreads();

  const T idx = T(1.0 / a.dx), idy = T(1.0 / a.dy);
  const bool owner = tid < TX * TY;
  const int tx = tid % TX, ty = tid / TX;
  T LU[M], LV[M], LW[M];
  constexpr bool PROJ = PHYS == PH_EULER && MODE != MODE_COMP;

  // ---- x-interfaces: between local cells ix-1 and ix, ix = 0..TX ----
  for (int q = tid; q < FW * TY; q += NT) {
    const int r = q / FW, ix = q - r * FW;
    const T* row = sm + (r + HY) * W + ix;
    auto ld = [&](int s, T* U, T* Dn, T* Dt) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < M; ++c) {
        U[c] = row[(c * HR) * W + s];
        Dn[c] = row[((M + c) * HR) * W + s];
        if constexpr (DIM == 2) Dt[c] = row[((2 * M + c) * HR) * W + s];
      }
    };
    T fh[M], hh[M], xx[M];
    interface_fluxes<T, PHYS, M, DIM == 2, PROJ>(ld, T(alx), k.ax, k, fh, hh, xx);
#pragma unroll
    for (int c = 0; c < M; ++c) {
      fb[(c * FR + r) * FW + ix] = fh[c];
      fb[((M + c) * FR + r) * FW + ix] = hh[c];
      if constexpr (DIM == 2) fb[((2 * M + c) * FR + r) * FW + ix] = xx[c];
    }
  }
  __syncthreads();
  // the interfaces' fluxes are twice f-hat, 8 h h-hat and 12 times the mixed flux
  // of a derivative times its own cell size.  LV and LW leave out one factor idx
  // and idy until their own cell: the square of a cell size's reciprocal may leave
  // the range of T where the results do not.
  if (owner) {
#pragma unroll
    for (int c = 0; c < M; ++c) {
      const int b0 = (c * FR + ty) * FW + tx;
      LU[c] = (fb[b0] - fb[b0 + 1]) * (T(0.5) * idx);
      const int b1 = ((M + c) * FR + ty) * FW + tx;
      LV[c] = (fb[b1] - fb[b1 + 1]) * (T(0.125) * idx);
      if constexpr (DIM == 2) {
        const int b2 = ((2 * M + c) * FR + ty) * FW + tx;
        LW[c] = (fb[b2] - fb[b2 + 1]) * (T(1.0 / 12.0) * idx);
      }
    }
  }

  if constexpr (DIM == 2) {
    __syncthreads();
    if constexpr (EDG) {
      // Obstacle, y-interfaces: the mirror image across the top face y = oj dy
      if (obstacle_near(*e, i0 - 2, i0 - 2 + W, j0 - HY, j0 - HY + HR)) {
        obstacle_mirror<T, M, NF, HR, W, NT>(a, *e, sm, i0, j0, HY, 1);
        __syncthreads();
      }
    }
    // ---- y-interfaces: between local rows iy-1 and iy, iy = 0..TY ----
    for (int q = tid; q < TX * FR; q += NT) {
      const int iy = q / TX, cc = q - iy * TX;
      const T* col = sm + iy * W + cc + 2;
      auto ld = [&](int s, T* U, T* Dn, T* Dt) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < M; ++c) {
          // normal frame: swap the two momenta; Dn = U_y, Dt = U_x
          const int cs = (PHYS == PH_EULER && (c == 1 || c == 2)) ? 3 - c : c;
          U[c] = col[(cs * HR + s) * W];
          Dn[c] = col[((2 * M + cs) * HR + s) * W];
          Dt[c] = col[((M + cs) * HR + s) * W];
        }
      };
      T fh[M], hh[M], xx[M];
      interface_fluxes<T, PHYS, M, true, PROJ>(ld, T(aly), k.ay, k, fh, hh, xx);
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const int cs = (PHYS == PH_EULER && (c == 1 || c == 2)) ? 3 - c : c;
        fb[(cs * FR + iy) * FW + cc] = fh[c];
        fb[((M + cs) * FR + iy) * FW + cc] = hh[c];      // theta-hat -> L_W
        fb[((2 * M + cs) * FR + iy) * FW + cc] = xx[c];  // xi-hat -> L_V
      }
    }
    __syncthreads();
    if (owner) {
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const int b0 = (c * FR + ty) * FW + tx;
        LU[c] = mad(fb[b0] - fb[b0 + FW], T(0.5) * idy, LU[c]);
        const int b1 = ((M + c) * FR + ty) * FW + tx;
        LW[c] = mad(fb[b1] - fb[b1 + FW], T(0.125) * idy, LW[c]);
        const int b2 = ((2 * M + c) * FR + ty) * FW + tx;
        LV[c] = mad(fb[b2] - fb[b2 + FW], T(1.0 / 12.0) * idy, LV[c]);
      }
    }
  }

  // ---- own cell: limiter, Runge-Kutta combination, store ----
  const int gi = i0 + tx, gj = j0 + ty;
  const bool inside = owner && gi < nx && gj < ny;
  const long long g = (long long)gj * nx + gi;
  const T* own = sm + (ty + HY) * W + tx + 2;
  if (!inside) return;
  if constexpr (EDG) {
    if (solid_cell(*e, gi, gj)) {
      // solid: zero right-hand side, the state carried through unchanged
#pragma unroll
      for (int f = 0; f < NF; ++f) gst(a.out + f * fs + g, K == 0 ? T(0) : gld(a.in + f * fs + g));
      return;
    }
  }

  if constexpr (K == 0) {
#pragma unroll
    for (int c = 0; c < M; ++c) {
      gst(a.out + c * fs + g, LU[c]);
      gst(a.out + (M + c) * fs + g, LV[c] * idx);
      if constexpr (DIM == 2) gst(a.out + (2 * M + c) * fs + g, LW[c] * idy);
    }
  } else {
    // S^_k = (U_k, limited derivatives of S_k)
    T Sh[NF];
    const bool charlim = PHYS == PH_EULER && (MODE == MODE_CHAR_LIM || (MODE == MODE_COMP && k.limiter_char));
    const bool complim = k.limiter_on && !charlim;
    // the x-neighbour of a fluid cell next to the obstacle's front face is that
    // cell's own mirror image (the stage buffer holds the y-image there)
    bool front = false;
    if constexpr (EDG) front = gi == e->oi - 1 && gj < e->oj;
    // differences of one cell's x- or y-stencil (limit_blend), d = 0 or 1
    auto stencil = [&](int c, int d, T& d1, T& d2, T& vs, T& vd) __attribute__((always_inline)) {
      const T* u = own + (c * HR) * W;
      const T* v = own + (((1 + d) * M + c) * HR) * W;
      const int st = d == 0 ? 1 : W;
      T up = u[st], vp = v[st];
      if constexpr (EDG) {
        if (d == 0 && front) {
          up = mirror_sign(c, M, true, 0) < 0 ? -u[0] : u[0];
          vp = mirror_sign(M + c, M, true, 0) < 0 ? -v[0] : v[0];
        }
      }
      const T vm = v[-st];
      d1 = u[0] - u[-st], d2 = up - u[0];
      vs = vm + vp, vd = vm - vp;
    };
#pragma unroll
    for (int c = 0; c < M; ++c) {
      Sh[c] = own[(c * HR) * W];
      if (complim) {
        T d1, d2, vs, vd;
        stencil(c, 0, d1, d2, vs, vd);
        Sh[M + c] = idx * limit_blend(d1, d2, vs, vd, k.lb);
        if constexpr (DIM == 2) {
          stencil(c, 1, d1, d2, vs, vd);
          Sh[2 * M + c] = idy * limit_blend(d1, d2, vs, vd, k.lb);
        }
      } else if (!k.limiter_on) {
        // unlimited: the derivatives themselves, not their scaled copies
#pragma unroll
        for (int d = 0; d < DIM; ++d) Sh[(1 + d) * M + c] = gld(a.in + ((1 + d) * M + c) * fs + g);
      }
    }
    if constexpr (PHYS == PH_EULER && MODE != MODE_CHAR) {
      if (charlim && k.limiter_on) {
        // characteristic variant of the limiter, x then y (normal frame:
        // the two momenta swap places for y)
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
          T u0[M], d1[M], d2[M], vs[M], vd[M], r[M];
#pragma unroll
          for (int c = 0; c < M; ++c) {
            const int q = (d == 1 && (c == 1 || c == 2)) ? 3 - c : c;
            u0[c] = own[(q * HR) * W];
            stencil(q, d, d1[c], d2[c], vs[c], vd[c]);
          }
          limit_char_d<T, M>(u0, d1, d2, vs, vd, k.lb, k.gm1, r);
#pragma unroll
          for (int c = 0; c < M; ++c) {
            const int q = (d == 1 && (c == 1 || c == 2)) ? 3 - c : c;
            Sh[(1 + d) * M + q] = (d == 0 ? idx : idy) * r[c];
          }
        }
      }
    }
    T L[NF];
#pragma unroll
    for (int c = 0; c < M; ++c) {
      L[c] = LU[c];
      L[M + c] = LV[c] * idx;
      if constexpr (DIM == 2) L[2 * M + c] = LW[c] * idy;
    }
    const T tdt = T(dt);
    T out[NF];
    if constexpr (K == 1) {
#pragma unroll
      for (int f = 0; f < NF; ++f) out[f] = Sh[f] + tdt * L[f];
      if (k.limiter_on) {
#pragma unroll
        for (int f = M; f < NF; ++f) gst(a.base + (f - M) * fs + g, Sh[f]);
      }
    } else {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const T s0 = (f < M || !k.limiter_on) ? gld(a.st0 + f * fs + g) : gld(a.base + (f - M) * fs + g);
        out[f] = rk_combine(K, s0, Sh[f] + tdt * L[f]);
      }
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) gst(a.out + f * fs + g, out[f]);
    point_speeds<T, PHYS, DIM>(out, k, sx, sy, flags);
  }
  (void)alx;
  (void)aly;
}

// ---------------------------------------------------------------------------
// stage / right-hand-side kernel over one grid
// K = 0: right-hand side only; K = 1, 2, 3: SSP-RK3 stage K.
// ---------------------------------------------------------------------------
// Resident waves per SIMD the stage kernels are compiled for (the register
// budget is 512 / WAVES per lane; LDS allows five FP32 and two FP64
// workgroups per CU).  FP32: four, where every stage kernel fits (123-128
// VGPRs); at five (96) they spill 40 B per lane: 2.583 against 2.606 ms for
// four steps of 2047 x 1531, and 5.09 against 5.65 ms for a step of 256
// batched grids walked by resident workgroups, whose kernel spills most.  FP64: two
// (220-224 VGPRs, no spills); a third would need 168 and spills 352 B.
template <typename T>
struct StageOcc {
  static constexpr int WAVES = sizeof(T) == 4 ? 4 : 2;
};

template <typename T, int PHYS, int DIM, int K, int TX, int TY, int NT, int MODE>
__global__ __launch_bounds__(NT, StageOcc<T>::WAVES) void k_stage(StageArgs<T> a, Consts<T> k) {
  constexpr int M = Comps<PHYS, DIM>::M;
  constexpr int NF = Comps<PHYS, DIM>::NF;
  constexpr int HY = (DIM == 2) ? 2 : 0;
  constexpr int NQ = (DIM == 2) ? 3 : 2;
  __shared__ T sm[NF * (TY + 2 * HY) * (TX + 4)];
  __shared__ T fb[NQ * M * (TY + 1) * (TX + 1)];

  const int ntx = (a.nx + TX - 1) / TX;
  const int t = xcd_band(blockIdx.x, gridDim.x);
  const int tile_y = t / ntx, tile_x = t - tile_y * ntx;
  T sx = T(0), sy = T(0);
  uint32_t flags = 0;
  bool ran = true;
  const Early early = read_early<T, K>(a);
  const auto begin = [&](double& dt, double& alx, double& aly) {
    return ran = grid_begin<DIM, K>(a, early, dt, alx, aly);
  };
  stage_tile<T, PHYS, DIM, K, TX, TY, NT, MODE>(a, k, tile_x, tile_y, begin, sm, fb, sx, sy, flags);
  if (!ran) return;
  if constexpr (K > 0) {
    // speeds of the new stage state feed the next stage's splitting; after
    // stage 3 they are the next step's stage-1 speeds (multi-step calls)
    block_fold<NT>(sx, sy, flags, a.fold + my_slot(a.slots) + 2 * K, a.status,
                   !a.replay && (K < 3 || a.fold_next));
  }
}

// 2D Euler with edge-described sides.  The body
// repeats k_stage's: handing the kernel parameters to a shared device
// function by reference costs k_stage its register allocation (spills).
// (FP32 126-128 VGPRs, FP64 up to 226, without spills.)
template <typename T, int K, int TX, int TY, int NT, int MODE>
__global__ __launch_bounds__(NT, StageOcc<T>::WAVES) void k_stage_edges(StageArgs<T> a,
                                                                             Consts<T> k,
                                                                             EdgeArgs e) {
  constexpr int PHYS = PH_EULER, DIM = 2;
  constexpr int M = Comps<PHYS, DIM>::M;
  constexpr int NF = Comps<PHYS, DIM>::NF;
  constexpr int HY = (DIM == 2) ? 2 : 0;
  constexpr int NQ = (DIM == 2) ? 3 : 2;
  __shared__ T sm[NF * (TY + 2 * HY) * (TX + 4)];
  __shared__ T fb[NQ * M * (TY + 1) * (TX + 1)];

  const int ntx = (a.nx + TX - 1) / TX;
  const int t = xcd_band(blockIdx.x, gridDim.x);
  const int tile_y = t / ntx, tile_x = t - tile_y * ntx;
  T sx = T(0), sy = T(0);
  uint32_t flags = 0;
  bool ran = true;
  const Early early = read_early<T, K>(a);
  const auto begin = [&](double& dt, double& alx, double& aly) {
    return ran = grid_begin<2, K>(a, early, dt, alx, aly);
  };
  stage_tile<T, PH_EULER, 2, K, TX, TY, NT, MODE, true>(a, k, tile_x, tile_y, begin, sm, fb, sx, sy,
                                                        flags, &e);
  if (!ran) return;
  if constexpr (K > 0) {
    // speeds of the new stage state feed the next stage's splitting; after
    // stage 3 they are the next step's stage-1 speeds (multi-step calls)
    block_fold<NT>(sx, sy, flags, a.fold + my_slot(a.slots) + 2 * K, a.status,
                   !a.replay && (K < 3 || a.fold_next));
  }
}

// ---------------------------------------------------------------------------
// Batched 2D Euler: kernels over the flattened tile list of many independent
// instances, one tile per workgroup or striding.
// ---------------------------------------------------------------------------
template <int V>
struct BatchTile;
template <>
struct BatchTile<0> {  // 255 x- and 256 y-interfaces: one pass each
  static constexpr int TX = 16, TY = 15, NT = 256;
};
template <>
struct BatchTile<1> {  // 231 x- and 256 y-interfaces: one pass each, wider rows
  static constexpr int TX = 32, TY = 7, NT = 256;
};


template <typename T, int K>
__device__ __forceinline__ StageArgs<T> instance_args(const hweno_instance& I, double cfl) {
  StageArgs<T> a;
  char* ws = (char*)I.ws;
  a.ctrl = (double*)ws;
  a.status = (unsigned long long*)(a.ctrl + 8);
  a.alpha = nullptr;
  a.nx = I.nx;
  a.ny = I.ny;
  a.bc_x = I.bc_x;
  a.bc_y = I.bc_y;
  a.fs = (long long)I.nx * I.ny;
  a.dx = I.dx;
  a.dy = I.dy;
  a.dt_fixed = I.dt_fixed;
  a.t_end = I.t_end;
  a.cfl = cfl;
  a.replay = 0;
  a.st0 = (const T*)I.state;
  a.base = (T*)(ws + I.off_base);
  T* s1 = (T*)(ws + I.off_s1);
  T* s2 = (T*)(ws + I.off_s2);
  a.in = (K <= 1) ? (const T*)I.state : (K == 2 ? s1 : s2);
  a.out = (K <= 1) ? s1 : (K == 2 ? s2 : (T*)I.state);
  return a;
}

// One tile t of the flattened list; nothing is done when its instance's step
// is skipped (a decision uniform over the workgroup).
template <typename T, int V, int K, int MODE>
__device__ __forceinline__ void batched_tile(const hweno_instance* __restrict__ inst,
                                             const int* __restrict__ tile_map, int t, double cfl,
                                             const Consts<T>& k, T* sm, T* fb) {
  constexpr int TX = BatchTile<V>::TX, TY = BatchTile<V>::TY, NT = BatchTile<V>::NT;
  const hweno_instance& I = inst[tile_map[t]];
  StageArgs<T> a = instance_args<T, K>(I, cfl);
  const bool leader = t == I.tile_begin[V] && threadIdx.x == 0;
  bool ran = true;
  const auto begin = [&](double& dt, double& alx, double& aly) {
    alx = a.ctrl[2 * (K - 1)];
    aly = a.ctrl[2 * (K - 1) + 1];
    return ran = stage_dt<2, K>(a.ctrl, a.ctrl[6], a.ctrl[7], alx, aly, a.dt_fixed, a.t_end, cfl, a.dx, a.dy, 0, leader, a.status, dt);
  };
  const int lt = t - I.tile_begin[V];
  const int ntx = (I.nx + TX - 1) / TX;
  const int tile_y = lt / ntx, tile_x = lt - tile_y * ntx;
  T sx = T(0), sy = T(0);
  uint32_t flags = 0;
  stage_tile<T, PH_EULER, 2, K, TX, TY, NT, MODE>(a, k, tile_x, tile_y, begin, sm, fb, sx, sy, flags);
  if (!ran) return;
  block_fold<NT>(sx, sy, flags, a.ctrl + 2 * K, a.status, K < 3);
}

// ONE: exactly one tile per workgroup (grid = tile count, XCD-banded order).
// Nothing is written before the descriptor and control words are read, so
// those reads stay scalar and never queue behind the other workgroups'
// atomics on the same control line.  Otherwise: persistent, striding over
// XCD bands of the tile list.
template <typename T, int V, int K, bool ONE, int MODE>
__global__ __launch_bounds__(256, StageOcc<T>::WAVES) void k_stage_batched(
    const hweno_instance* __restrict__ inst, const int* __restrict__ tile_map, int total,
    double cfl, Consts<T> k) {
  constexpr int TX = BatchTile<V>::TX, TY = BatchTile<V>::TY;
  __shared__ T sm[12 * (TY + 4) * (TX + 4)];
  __shared__ T fb[12 * (TY + 1) * (TX + 1)];
  if constexpr (ONE) {
    batched_tile<T, V, K, MODE>(inst, tile_map, xcd_band(blockIdx.x, gridDim.x), cfl, k, sm, fb);
  } else {
    const BandIter bi(total);
    for (int it = 0; bi.valid(it); ++it) {
      batched_tile<T, V, K, MODE>(inst, tile_map, bi.tile(it), cfl, k, sm, fb);
      __syncthreads();  // LDS tile and fold slots are reused by the next tile
    }
  }
}

// speeds of every instance's state (slots pre-zeroed by k_begin_batched).
// Each workgroup walks one contiguous chunk of the tile list, keeps a running
// maximum while consecutive tiles belong to the same instance and folds it
// into that instance's slot only when the instance changes (cells are read
// once, so no halo locality is at stake here).
template <typename T, int V>
__global__ __launch_bounds__(256) void k_alpha_batched(const hweno_instance* __restrict__ inst,
                                                       const int* __restrict__ tile_map,
                                                       int total, Consts<T> k) {
  constexpr int TX = BatchTile<V>::TX, TY = BatchTile<V>::TY;
  const long long nb = gridDim.x;
  const int t_lo = (int)(total * (long long)blockIdx.x / nb);
  const int t_hi = (int)(total * ((long long)blockIdx.x + 1) / nb);
  int cur = -1;
  T sx = T(0), sy = T(0);
  uint32_t flags = 0;
  for (int t = t_lo; t < t_hi; ++t) {
    const int q = tile_map[t];
    if (q != cur) {  // uniform over the workgroup
      if (cur >= 0) {
        double* ctrl = (double*)inst[cur].ws;
        block_fold<256>(sx, sy, flags, ctrl, (unsigned long long*)(ctrl + 8), true);
        __syncthreads();  // the fold's LDS slots are reused by the next fold
        sx = sy = T(0);
        flags = 0;
      }
      cur = q;
    }
    const hweno_instance& I = inst[q];
    const int lt = t - I.tile_begin[V];
    const int ntx = (I.nx + TX - 1) / TX;
    const int tile_y = lt / ntx, tile_x = lt - tile_y * ntx;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int gi = tile_x * TX + tx, gj = tile_y * TY + ty;
    if (threadIdx.x < TX * TY && gi < I.nx && gj < I.ny) {
      const long long n = (long long)I.nx * I.ny;
      const long long g = (long long)gj * I.nx + gi;
      const T* S = (const T*)I.state;
      T U[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) U[c] = gld(S + c * n + g);
      T ax, ay;
      point_speeds<T, PH_EULER, 2>(U, k, ax, ay, flags);
      // bit-pattern max keeps NaN
      sx = (dbits(double(ax)) > dbits(double(sx))) ? ax : sx;
      sy = (dbits(double(ay)) > dbits(double(sy))) ? ay : sy;
    }
  }
  if (cur >= 0) {
    double* ctrl = (double*)inst[cur].ws;
    block_fold<256>(sx, sy, flags, ctrl, (unsigned long long*)(ctrl + 8), true);
  }
}

__global__ void k_begin_batched(const hweno_instance* __restrict__ inst, int n_inst) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n_inst) {
    double* ctrl = (double*)inst[q].ws;
#pragma unroll
    for (int j = 0; j < 6; ++j) ctrl[j] = 0.0;
  }
}

__global__ void k_finish_batched(const hweno_instance* __restrict__ inst, int n_inst) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n_inst) {
    double* ctrl = (double*)inst[q].ws;
    if (ctrl[6] > 0.0) {
      ctrl[7] += ctrl[6];
      ctrl[9] += 1.0;
    }
  }
}

// Fold the ghost-padded adjoint onto the grid and apply the pointwise
// Runge-Kutta transposes:
//   out  = [out] + fold(E) + cu * XU   (XU on U only, or on all fields when
//                                       identity_all; nothing when XU is NULL)
//   L0   = ca * A + cb * B + out       (when L0 is non-NULL)
template <typename T>
struct FoldArgs {
  const T* E;
  int nxe, nye;
  int nx, ny, bc_x, bc_y, dim, nf, m, euler;
  long long fs;
  T* out;
  int accumulate;
  const T* XU;
  double cu;
  int identity_all;
  T* L0;
  const T* A;
  const T* B;
  double ca, cb;
};

// The Runge-Kutta transposes of the NF fields of cell index q, given their
// folded adjoints v[].  Every load is issued before the first store: the
// output may not be proven distinct from the inputs, and interleaving them
// would serialise one memory round trip per field.
template <typename T, int NF>
__device__ __forceinline__ void fold_finish(const FoldArgs<T>& a, long long q, const T* v) {
  T r[NF], av[NF], bv[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const long long o = (long long)f * a.fs + q;
    r[f] = v[f];
    if (a.accumulate) r[f] += a.out[o];
    if (a.XU && (f < a.m || a.identity_all)) r[f] += T(a.cu) * a.XU[o];
    if (a.L0) {
      av[f] = a.A[o];
      bv[f] = a.B[o];
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const long long o = (long long)f * a.fs + q;
    a.out[o] = r[f];
    if (a.L0) a.L0[o] = T(a.ca) * av[f] + T(a.cb) * bv[f] + r[f];
  }
}

// field f of cell (i, j): its own entry of E plus every ghost entry the
// boundary maps read from it, then the Runge-Kutta transposes
template <typename T>
__device__ __forceinline__ void fold_cell_field(const FoldArgs<T>& a, int i, int j, int f) {
  const int GX = 2, GY = (a.dim == 2) ? 2 : 0;
  const int gx[4] = {-2, -1, a.nx, a.nx + 1};
  const int gy[4] = {-2, -1, a.ny, a.ny + 1};
  const long long q = (long long)j * a.nx + i;
  const T* Ef = a.E + (long long)f * a.nye * a.nxe;
  T v = Ef[(long long)(j + GY) * a.nxe + (i + GX)];
  // ghosts copied from this cell; a reflecting wall copied them with a sign
  const T sx = (a.bc_x == HWENO_BC_REFLECT) ? T(mirror_sign(f, a.m, a.euler, 0)) : T(1);
#pragma unroll
  for (int g = 0; g < 4; ++g)
    if (map_index(gx[g], a.nx, a.bc_x) == i) v += sx * Ef[(long long)(j + GY) * a.nxe + (gx[g] + GX)];
  if (a.dim == 2) {
    const T sy = (a.bc_y == HWENO_BC_REFLECT) ? T(mirror_sign(f, a.m, a.euler, 1)) : T(1);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (map_index(gy[g], a.ny, a.bc_y) == j) v += sy * Ef[(long long)(gy[g] + GY) * a.nxe + (i + GX)];
  }
  const long long o = (long long)f * a.fs + q;
  T r = v;
  if (a.accumulate) r += a.out[o];
  if (a.XU && (f < a.m || a.identity_all)) r += T(a.cu) * a.XU[o];
  T av = T(0), bv = T(0);
  if (a.L0) {
    av = a.A[o];
    bv = a.B[o];
  }
  a.out[o] = r;
  if (a.L0) a.L0[o] = T(a.ca) * av + T(a.cb) * bv + r;
}

// one thread per (field, cell)
template <typename T>
__global__ __launch_bounds__(256) void k_fold(FoldArgs<T> a) {
  const long long t = blockIdx.x * 256ll + threadIdx.x;
  if (t >= a.fs * a.nf) return;
  const int f = (int)(t / a.fs);
  const long long q = t - (long long)f * a.fs;
  const int j = (int)(q / a.nx), i = (int)(q - (long long)j * a.nx);
  fold_cell_field(a, i, j, f);
}

// 2D grids with nx, ny >= 4 after a fused adjoint: only the cells within two of
// a boundary (the only ones the boundary maps read ghost entries from) are
// folded here; every other cell was finished by the adjoint kernel itself.
// Band cells are enumerated as the four columns 0, 1, nx-2, nx-1 (4*ny cells)
// and then the four rows 0, 1, ny-2, ny-1 of the columns 2..nx-3; one thread
// per (field, band cell).
template <typename T>
__global__ __launch_bounds__(256) void k_fold_band(FoldArgs<T> a) {
  const int nxb = 4 * a.ny, nb = nxb + 4 * (a.nx - 4);
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= nb * a.nf) return;
  const int f = t / nb, q = t - f * nb;
  int i, j;
  if (q < nxb) {
    const int r = q & 3;
    j = q >> 2;
    i = r < 2 ? r : a.nx - 4 + r;
  } else {
    const int r = (q - nxb) & 3;
    i = 2 + ((q - nxb) >> 2);
    j = r < 2 ? r : a.ny - 4 + r;
  }
  fold_cell_field(a, i, j, f);
}

// ---------------------------------------------------------------------------
// Discrete adjoint.  The forward operator reads ghost cells through the
// boundary index maps; its adjoint scatters into a ghost-padded buffer E
// ([nf][ny+4][nx+4] in 2D, [nf][1][nx+4] in 1D) and k_fold then adds every
// ghost entry onto the cell it was copied from.
// ---------------------------------------------------------------------------
template <typename T>
struct AdjArgs {
  const T* S;           // state the operator is linearised at
  const T* XL;          // adjoint of L is cr * XL (nf fields)
  const T* XM;          // adjoint of the limited derivatives is cl * XM (m*dim fields) or NULL
  T* E;                 // ghost-padded output
  const double* alpha;  // speeds used by the forward evaluation
  const double* dtp;    // if non-NULL, cr is multiplied by *dtp
  double cr, cl;
  int nx, ny, bc_x, bc_y;
  long long fs;
  int nxe, nye;
  double dx, dy;
  // fused: entries of real cells at least two away from every boundary are
  // folded and finished (fo's transposes) here instead of being stored in E
  int fused;
  FoldArgs<T> fo;
};

constexpr int cmax(int x, int y) { return x > y ? x : y; }

// FP32 fits four waves per SIMD (126 VGPRs, 38 KB of LDS per workgroup), FP64
// two (235 VGPRs, 77 KB), both without spills.
template <typename T>
struct AdjOcc {
  static constexpr int WAVES = sizeof(T) == 4 ? 4 : 2;
};

// One output tile of E per workgroup (TX x TY entries, ghost entries
// included).  Every interface and limiter stencil that touches the tile is
// differentiated by one lane.
// The data of a cell enter its interfaces only through x+- = F +- alpha U and
// y+- = A Dn +- alpha Dn (interface_fluxes), so the interfaces' lanes add their
// adjoints of x+-, y+- to the cells' sums in LDS and the owner of each cell takes
// the sums through the point fluxes once per direction, instead of every
// interface and side doing so for each of its points.  The linear fluxes'
// adjoints are stencils of the incoming one: each lane leaves its interface's in
// LDS and the owners apply the four coefficients.  These pass the point fluxes
// by themselves, with the mixed flux's: within the sums, 15 times their size would
// have to cancel again in alpha U's share, whose rounding stays.
// The additions go point by point: in one phase all lanes add to stencil point s of
// their interfaces, which are distinct cells, and a barrier ends the phase.  So
// the sums need no atomics and have a fixed order.  The barriers also keep
// the compiler from holding the staged stencil in registers (loads after a
// barrier are reloads).  Lanes without an interface or with a zero adjoint run
// the same code on a valid stencil (every lane takes part in every barrier) and add
// nothing.  The state tile is staged cell-interleaved ([row][col][field],
// derivatives times their cell size) so that one stencil point's fields are read
// with a few wide LDS loads.
// Measured (one launch under the profiler): with every interface reversing the point
// fluxes of its six point data itself and handing 12 fields over per point, 512^2
// FP32 took 116 us (9278 VALU instructions per lane) and 128^2 FP64 47 us; in this
// form 77 us (5950) and 35 us.
template <typename T, int PHYS, int DIM, int TX, int TY, int NT, int MODE>
__global__ __launch_bounds__(NT, AdjOcc<T>::WAVES) void k_adjoint(AdjArgs<T> a, Consts<T> k) {
  constexpr int M = Comps<PHYS, DIM>::M;
  constexpr int NF = Comps<PHYS, DIM>::NF;
  constexpr int GX = 2, GY = (DIM == 2) ? 2 : 0;  // ghost width of E
  constexpr int HX = 3, HY = (DIM == 2) ? 3 : 0;  // state halo around the tile
  constexpr int W = TX + 2 * HX, HR = TY + 2 * HY;
  constexpr int NIX = TY * (TX + 3);                   // x-interfaces touching the tile
  constexpr int NIY = (DIM == 2) ? TX * (TY + 3) : 0;  // y-interfaces
  constexpr int NLX = TY * (TX + 2);                   // cells whose x-limiter touches it
  constexpr int NLY = (DIM == 2) ? TX * (TY + 2) : 0;
  constexpr int AS = TX * TY;                          // stride of the sums' fields
  constexpr int NG = DIM == 2 ? 2 * M : M;             // linear fluxes' adjoints of an interface
  constexpr bool EU = PHYS == PH_EULER;
  constexpr bool PROJ = EU && MODE != MODE_COMP;
  static_assert(TX * TY <= NT, "one output entry per thread");
  static_assert(NIX <= NT && NIY <= NT && NLX <= NT && NLY <= NT, "one stencil per lane");
  __shared__ __align__(16) T sm[HR * W * NF];
  __shared__ T accs[NF * AS];                          // adjoint of the cells' fields
  // the linear fluxes' adjoints by interface, then the sums of gx, gy by cell
  __shared__ T pool[cmax(NG * NT, 2 * M * AS)];
  const int nx = a.nx, ny = a.ny;
  const long long fs = a.fs;
  const int ntx = (a.nxe + TX - 1) / TX;
  const int t = xcd_band(blockIdx.x, gridDim.x);
  const int bty = t / ntx, btx = t - bty * ntx;
  const int rx0 = btx * TX - GX, ry0 = bty * TY - GY;  // real coordinates of tile entry (0, 0)
  const int tid = threadIdx.x;
  const T cr = T(a.cr * (a.dtp ? *a.dtp : 1.0));
  const T cl = T(a.cl);
  const T idx = T(1.0 / a.dx), hx = T(a.dx), idy = T(1.0 / a.dy), hy = T(a.dy);
  for (int q = tid; q < W * HR; q += NT) {
    const int lr = q / W, lc = q - lr * W;
    const int ii = rx0 - HX + lc, jj = ry0 - HY + lr;
    const int gi = map_index(ii, nx, a.bc_x);
    const int gj = (DIM == 2) ? map_index(jj, ny, a.bc_y) : 0;
    const long long g = (long long)gj * nx + gi;
    const bool mx = mirrored(ii, nx, a.bc_x), my = DIM == 2 && mirrored(jj, ny, a.bc_y);
    T x[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) x[f] = gld(a.S + f * fs + g);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int sg = (mx ? mirror_sign(f, M, EU, 0) : 1) * (my ? mirror_sign(f, M, EU, 1) : 1);
      sm[q * NF + f] = staged(sg < 0 ? -x[f] : x[f], f, M, hx, hy);
    }
  }

  auto xl = [&](int f, int i, int j) -> T {
    return (i >= 0 && i < nx && j >= 0 && j < ny) ? gld(a.XL + f * fs + (long long)j * nx + i) : T(0);
  };
  // cell (i, j) of the staged state
  auto cell = [&](int i, int j) -> const T* {
    return sm + ((j - (ry0 - HY)) * W + (i - (rx0 - HX))) * NF;
  };
  const bool owner = tid < AS;
  const int lx = tid % TX, ly = tid / TX;
  T* acc = accs + (owner ? tid : 0);
  if (owner) {
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f * AS] = T(0);
  }

  // ---- interfaces along direction d (0: x, 1: y) that touch the tile ----
  // interface q lies between points 1 and 2 of its stencil; its point s is the
  // tile's cell (sx + s, sy) along x, (sx, sy + s) along y
  auto direction = [&](auto dir) __attribute__((always_inline)) {
    constexpr int d = decltype(dir)::value;
    constexpr int NI = d == 0 ? NIX : NIY;
    constexpr int ST = d == 0 ? NF : W * NF;     // LDS step along the direction
    constexpr int CS = d == 0 ? 1 : TX;          // step of the tile's cells
    constexpr int ON = (1 + d) * M, OT = (2 - d) * M;  // normal and tangential derivatives
    // component c of the normal frame (normal momentum first)
    auto cs = [](int c) { return (EU && d == 1 && (c == 1 || c == 2)) ? 3 - c : c; };
    const T ihn = d == 0 ? idx : idy, iht = d == 0 ? idy : idx;
    const T alpha = T(a.alpha[d]), an = d == 0 ? k.ax : k.ay;
    // lanes past the last interface take the last one, with a zero adjoint
    const int q = tid < NI ? tid : NI - 1;
    const int qr = d == 0 ? q / (TX + 3) : q / TX;
    const int qc = d == 0 ? q - qr * (TX + 3) : q - qr * TX;
    const int sx = d == 0 ? qc - 3 : qc, sy = d == 0 ? qr : qr - 3;
    const int i1 = rx0 + sx + (d == 0 ? 1 : 0), j1 = ry0 + sy + (d == 1 ? 1 : 0);  // point 1
    const int i2 = i1 + (d == 0 ? 1 : 0), j2 = j1 + (d == 1 ? 1 : 0);
    const bool live = tid < NI && (d == 0 ? (j1 >= 0 && j1 < ny && i1 >= -1 && i1 <= nx - 1)
                                          : (i1 >= 0 && i1 < nx && j1 >= -1 && j1 <= ny - 1));
    T gf[M];
    bool any = false;
    {
      T gh[M], gx[M];
#pragma unroll
      for (int c = 0; c < M; ++c) {
        // adjoints of 2 f-hat, 8 h h-hat and 12 times the scaled mixed flux
        auto diff = [&](int f) { return live ? cr * (xl(f, i2, j2) - xl(f, i1, j1)) * ihn : T(0); };
        gf[c] = T(0.5) * diff(cs(c));
        gh[c] = (T(0.125) * ihn) * diff(ON + cs(c));
        gx[c] = DIM == 2 ? (T(1.0 / 12.0) * iht) * diff(OT + cs(c)) : T(0);
        any = any || gf[c] != T(0) || gh[c] != T(0) || gx[c] != T(0);
      }
#pragma unroll
      for (int c = 0; c < M; ++c) {
        pool[c * NT + tid] = gh[c];
        if constexpr (DIM == 2) pool[(M + c) * NT + tid] = gx[c];
      }
    }
    __syncthreads();
    // the cell's own state in the normal frame
    const T* own = sm + (((owner ? ly : 0) + HY) * W + (owner ? lx : 0) + HX) * NF;
    auto ld = [&](const T* p, T* U, T* Dn) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < M; ++c) U[c] = p[cs(c)], Dn[c] = p[ON + cs(c)];
    };
    // adjoint of the cell's fields (normal frame), nothing when it is zero
    auto add_cell = [&](const T* gU, const T* gN) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < M; ++c) acc[cs(c) * AS] += gU[c], acc[(ON + cs(c)) * AS] += gN[c];
    };
    if (owner) {
      // linear fluxes: the cell is point s of interface q0 + (3 - s) CS
      const int q0 = d == 0 ? ly * (TX + 3) + lx : ly * TX + lx;
      T lF[M], lA[M], gU[M], gN[M], gT[M], gB[M];
      bool some = false, mixed = false;
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T* g = pool + c * NT + q0;
        const T p3 = g[0], p2 = g[CS], p1 = g[2 * CS], p0 = g[3 * CS];
        lF[c] = mad(T(15), p2 - p1, p0 - p3);
        lA[c] = T(1.0 / 3.0) * mad(T(-7), p1 + p2, p0 + p3);
        gU[c] = alpha * ((p0 + p3) - (p1 + p2));
        gN[c] = (T(1.0 / 3.0) * alpha) * mad(T(3), p1 - p2, p0 - p3);
        some = some || p0 != T(0) || p1 != T(0) || p2 != T(0) || p3 != T(0);
        gT[c] = T(0);
        if constexpr (DIM == 2) {
          const T* x = g + M * NT;
          gB[c] = mad(T(7), x[CS] + x[2 * CS], -(x[0] + x[3 * CS]));
          mixed = mixed || gB[c] != T(0);
        }
      }
      if (some || mixed) {
        // fields that meet zero adjoints only stay out (they may not be finite)
        T U[M], Dn[M], Dt[M];
        ld(own, U, Dn);
#pragma unroll
        for (int c = 0; c < M; ++c) {
          Dn[c] = some ? Dn[c] : T(0);
          Dt[c] = DIM == 2 && mixed ? own[OT + cs(c)] : T(0);
        }
        point_fluxes_vjp<T, PHYS, M, DIM == 2>(U, Dn, Dt, k, an, lF, lA, gB, gU, gN, gT);
        add_cell(gU, gN);
        if constexpr (DIM == 2) {
#pragma unroll
          for (int c = 0; c < M; ++c) acc[(OT + cs(c)) * AS] += gT[c];
        }
      }
    }
    __syncthreads();
    if (owner) {
#pragma unroll
      for (int c = 0; c < 2 * M; ++c) pool[c * AS + tid] = T(0);
    }
    // ---- the nonlinear flux, "+" side then "-" side ----
    const T* base = cell(i1 - (d == 0 ? 1 : 0), j1 - (d == 1 ? 1 : 0));
    auto lds = [&](int s, T* U, T* Dn) __attribute__((always_inline)) { ld(base + s * ST, U, Dn); };
    Eigen<T, M> eg;
    EigenAdj<T> ge;
    T gw[M], w[M], gU1[M], gU2[M];
#pragma unroll
    for (int c = 0; c < M; ++c) w[c] = T(0);
    if constexpr (PROJ) {
      T U1[M], U2[M], dn[M];
      lds(1, U1, dn);
      lds(2, U2, dn);
      eg.roe(U1, U2, k.gm1);
      back_T(eg, gf, gw);
#pragma unroll
      for (int c = 0; c < M; ++c) gw[c] *= T(1.0 / 6.0);
    } else {
#pragma unroll
      for (int c = 0; c < M; ++c) gw[c] = T(1.0 / 6.0) * gf[c];
    }
    // one phase: gx, gy to point s's sums, gU (if any) to its cell
    auto add = [&](int s, const T* gx, const T* gy, const T* gU) __attribute__((always_inline)) {
      const int px = sx + (d == 0 ? s : 0), py = sy + (d == 1 ? s : 0);
      __syncthreads();
      if (any && px >= 0 && px < TX && py >= 0 && py < TY) {
        T* p = pool + py * TX + px;
        T* u = accs + py * TX + px;
#pragma unroll
        for (int c = 0; c < M; ++c) {
          p[c * AS] += gx[c];
          p[(M + c) * AS] += gy[c];
          if (gU) u[cs(c) * AS] += gU[c];
        }
      }
    };
    T gxa[M], gya[M], gxo[M], gyo[M], gxb[M], gyb[M], pF[M], pA[M];
    side_vjp<T, PHYS, M, PROJ>(lds, true, alpha, an, k, eg, gw, gf, w, ge, gxa, gya, gxo, gyo, gxb, gyb);
    add(0, gxa, gya, nullptr);
    add(1, gxo, gyo, nullptr);
    add(2, gxb, gyb, nullptr);
    __syncthreads();
    if (owner) {
#pragma unroll
      for (int c = 0; c < M; ++c) {
        pF[c] = pool[c * AS + tid], pA[c] = pool[(M + c) * AS + tid];
        pool[c * AS + tid] = pool[(M + c) * AS + tid] = T(0);
      }
    }
    side_vjp<T, PHYS, M, PROJ>(lds, false, alpha, an, k, eg, gw, gf, w, ge, gxa, gya, gxo, gyo, gxb, gyb);
    if constexpr (PROJ) {
      // the reconstructed fields' way back, then the Roe average
#pragma unroll
      for (int c = 0; c < M; ++c) w[c] *= T(1.0 / 6.0), gU1[c] = gU2[c] = T(0);
      back_eigen_adj(eg, w, gf, ge);
      T U1[M], U2[M], dn[M];
      lds(1, U1, dn);
      lds(2, U2, dn);
      roe_vjp<T, M>(U1, U2, k.gm1, ge, gU1, gU2);
    }
    add(3, gxa, gya, nullptr);
    add(2, gxo, gyo, PROJ ? gU2 : nullptr);
    add(1, gxb, gyb, PROJ ? gU1 : nullptr);
    __syncthreads();
    if (owner) {
      // through the point fluxes: x+- = F +- alpha U, y+- = A +- alpha Dn
      T gF[M], gA[M], gU[M], gN[M];
      bool some = false;
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T mF = pool[c * AS + tid], mA = pool[(M + c) * AS + tid];
        some = some || pF[c] != T(0) || pA[c] != T(0) || mF != T(0) || mA != T(0);
        gF[c] = pF[c] + mF, gU[c] = alpha * (pF[c] - mF);
        gA[c] = pA[c] + mA, gN[c] = alpha * (pA[c] - mA);
      }
      if (some) {
        T U[M], Dn[M];
        ld(own, U, Dn);
        point_fluxes_vjp<T, PHYS, M, false>(U, Dn, Dn, k, an, gF, gA, nullptr, gU, gN, nullptr);
        add_cell(gU, gN);
      }
    }
  };
  direction(std::integral_constant<int, 0>{});
  if constexpr (DIM == 2) {
    __syncthreads();  // the pool's last reads are done
    direction(std::integral_constant<int, 1>{});
  }

  // ---- limiter: U_x along x (and U_y along y) of cells near the tile ----
  // the limiter at cell C reads U at C-1, C, C+1 and the derivative at C-1, C+1
  auto limiter = [&](auto dir) __attribute__((always_inline)) {
    constexpr int d = decltype(dir)::value;
    constexpr int NL = d == 0 ? NLX : NLY;
    constexpr int ST = d == 0 ? NF : W * NF;
    constexpr int ON = (1 + d) * M;
    const T ihn = d == 0 ? idx : idy;
    const int q = tid < NL ? tid : NL - 1;
    const int qr = d == 0 ? q / (TX + 2) : q / TX;
    const int qc = d == 0 ? q - qr * (TX + 2) : q - qr * TX;
    const int sx = d == 0 ? qc - 1 : qc, sy = d == 0 ? qr : qr - 1;  // C in the tile
    const int ci = rx0 + sx, cj = ry0 + sy;
    const bool live = tid < NL && cj >= 0 && cj < ny && ci >= 0 && ci < nx;
    const T* p = live ? cell(ci, cj) : sm + ST;
    T gm[M], g0[M], gp[M], gvm[M], gvp[M], mu[M];
    bool any = false;
#pragma unroll
    for (int c = 0; c < M; ++c) {
      mu[c] = live ? cl * gld(a.XM + (d * M + c) * fs + (long long)cj * nx + ci) * ihn : T(0);
      any = any || mu[c] != T(0);
      gm[c] = g0[c] = gp[c] = gvm[c] = gvp[c] = T(0);
    }
    const bool charlim = EU && (MODE == MODE_CHAR_LIM || (MODE == MODE_COMP && k.limiter_char));
    auto cs = [&](int c) { return (EU && charlim && d == 1 && (c == 1 || c == 2)) ? 3 - c : c; };
    if (any) {
      auto args = [&](int f, T& d1, T& d2, T& vs, T& vd) __attribute__((always_inline)) {
        d1 = p[f] - p[f - ST], d2 = p[f + ST] - p[f];
        const T vm = p[ON + f - ST], vp = p[ON + f + ST];
        vs = vm + vp, vd = vm - vp;
      };
      if (!charlim) {
#pragma unroll
        for (int c = 0; c < M; ++c) {
          T d1, d2, vs, vd, g1, g2, gs, gd;
          args(c, d1, d2, vs, vd);
          limit_blend_vjp(d1, d2, vs, vd, k.lw.g1, k.lw.g2, k.lw.eps, mu[c], g1, g2, gs, gd);
          gm[c] = -g1, g0[c] = g1 - g2, gp[c] = g2, gvm[c] = gs + gd, gvp[c] = gs - gd;
        }
      } else if constexpr (EU && MODE != MODE_CHAR) {
        // characteristic variant, in the normal frame (the momenta swap places for y)
        T u0[M], d1[M], d2[M], vs[M], vd[M], go[M], gu[M], g1[M], g2[M], gs[M], gd[M];
#pragma unroll
        for (int c = 0; c < M; ++c) {
          const int f = d == 1 && (c == 1 || c == 2) ? 3 - c : c;
          u0[c] = p[f];
          go[c] = mu[f];
          args(f, d1[c], d2[c], vs[c], vd[c]);
        }
        limit_char_d_vjp<T, M>(u0, d1, d2, vs, vd, k.lw.g1, k.lw.g2, k.lw.eps, k.gm1, go, gu, g1, g2,
                               gs, gd);
#pragma unroll
        for (int c = 0; c < M; ++c) {
          const int f = d == 1 && (c == 1 || c == 2) ? 3 - c : c;
          gm[f] = -g1[c], g0[f] = gu[c] + (g1[c] - g2[c]), gp[f] = g2[c];
          gvm[f] = gs[c] + gd[c], gvp[f] = gs[c] - gd[c];
        }
      }
    }
    // phase: gu to U and gv (if any) to the derivative of cell C + s
    auto add = [&](int s, const T* gu, const T* gv) __attribute__((always_inline)) {
      const int px = sx + (d == 0 ? s : 0), py = sy + (d == 1 ? s : 0);
      __syncthreads();
      if (any && px >= 0 && px < TX && py >= 0 && py < TY) {
        T* u = accs + py * TX + px;
#pragma unroll
        for (int c = 0; c < M; ++c) {
          u[c * AS] += gu[c];
          if (gv) u[(ON + c) * AS] += gv[c];
        }
      }
    };
    add(-1, gm, gvm);
    add(0, g0, nullptr);
    add(1, gp, gvp);
  };
  if (a.XM) {
    limiter(std::integral_constant<int, 0>{});
    if constexpr (DIM == 2) limiter(std::integral_constant<int, 1>{});
  }
  __syncthreads();
  if (owner) {
    const int ex = btx * TX + lx, ey = bty * TY + ly;
    if (ex < a.nxe && ey < a.nye) {
      const int i = ex - GX, j = ey - GY;
      const bool inner = i >= 2 && i < nx - 2 && (DIM == 1 || (j >= 2 && j < ny - 2));
      T v[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) v[f] = staged(acc[f * AS], f, M, hx, hy);
      if (a.fused && inner) {
        fold_finish<T, NF>(a.fo, (long long)j * nx + i, v);
      } else {
#pragma unroll
        for (int f = 0; f < NF; ++f) a.E[((long long)f * a.nye + ey) * a.nxe + ex] = v[f];
      }
    }
  }
}

// global speeds of a state: the maximum over cells into the first two entries of
// `slots` slots that begin at alpha; pre-zeroed
// NT: 256 threads, or 1024 where every workgroup's atomics meet on one address.
template <typename T, int PHYS, int DIM, int NT>
__global__ __launch_bounds__(NT) void k_alpha(const T* __restrict__ S, long long n,
                                               Consts<T> k, double* alpha, int slots,
                                               unsigned long long* status) {
  constexpr int M = Comps<PHYS, DIM>::M;
  T mx = T(0), my = T(0);
  uint32_t flags = 0;
  for (long long i = (long long)blockIdx.x * NT + threadIdx.x; i < n; i += (long long)NT * gridDim.x) {
    T U[M];
#pragma unroll
    for (int c = 0; c < M; ++c) U[c] = gld(S + c * n + i);
    T sx, sy;
    point_speeds<T, PHYS, DIM>(U, k, sx, sy, flags);
    // bit-pattern max keeps NaN
    mx = (dbits(double(sx)) > dbits(double(mx))) ? sx : mx;
    my = (dbits(double(sy)) > dbits(double(my))) ? sy : my;
  }
  block_fold<NT>(mx, my, flags, alpha + my_slot(slots), status, true);
}

// k_alpha over the fluid cells of a 2D Euler grid with an obstacle (solid
// cells enter no speed)
template <typename T>
__global__ __launch_bounds__(256) void k_alpha_obstacle(const T* __restrict__ S, int nx, int ny,
                                                        int oi, int oj, Consts<T> k,
                                                        double* alpha, int slots,
                                                        unsigned long long* status) {
  const long long n = (long long)nx * ny;
  T mx = T(0), my = T(0);
  uint32_t flags = 0;
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += 256ll * gridDim.x) {
    const int j = (int)(i / nx), c = (int)(i - (long long)j * nx);
    if (j < oj && c >= oi) continue;
    T U[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) U[q] = S[q * n + i];
    T sx, sy;
    point_speeds<T, PH_EULER, 2>(U, k, sx, sy, flags);
    mx = (dbits(double(sx)) > dbits(double(mx))) ? sx : mx;
    my = (dbits(double(sy)) > dbits(double(my))) ? sy : my;
  }
  block_fold<256>(mx, my, flags, alpha + my_slot(slots), status, true);
}

// Start of a step: stage speeds and dt from the replay record, or speeds and speed
// slots cleared for the reductions.
__global__ void k_begin(double* ctrl, double* fold, int slots, const double* replay) {
  const int t = threadIdx.x;
  if (replay) {
    if (t < 7) ctrl[t] = replay[t];
  } else if (t < 6) {
    ctrl[t] = 0.0;
  }
  if (t == 10 || t == 11) ctrl[t] = 0.0;
  if (!replay)
    for (int q = t; q < slots * SLOT_LEN; q += 64) fold[q] = 0.0;
}

__global__ void k_zero(double* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0;
}

// End of a step: time and step count, tape record.  begin_next: also start the
// next step of a multi-step call (what k_begin does), with the stage-1 speeds that
// this step's third stage folded, or, after a skipped step, whose state is
// unchanged, with this step's own; so consecutive steps need one small launch
// between them instead of two.
// One wave: entry t of the control block is lane t's, all of it loaded at once.
__global__ __launch_bounds__(64) void k_finish(double* ctrl, double* fold, int slots, double* tape,
                                               int begin_next) {
  const int t = threadIdx.x;
  double v = t < 10 ? gld((const double*)ctrl + t) : 0.0;
  double* f = fold + (t & (NSLOT - 1)) * SLOT_LEN;
  double nx = 0.0, ny = 0.0;
  if (begin_next && t < slots) nx = gld((const double*)f + 6), ny = gld((const double*)f + 7);
  const double dt = __shfl(v, 6), ax = __shfl(v, 0), ay = __shfl(v, 1);
  const bool ran = dt > 0.0;
  if (ran && t == 7) v += dt;
  if (ran && t == 9) v += 1.0;
  if (tape && t < 10) gst(tape + t, v);
  if (ran && (t == 7 || t == 9)) gst(ctrl + t, v);
  if (begin_next) {
    if (t < 6) gst(ctrl + t, 0.0);
    if (t < slots) {
      if (ran) gst(f, nx), gst(f + 1, ny);
#pragma unroll
      for (int q = 2; q < 8; ++q) gst(f + q, 0.0);
    }
  } else if (!ran) {
    if (t == 10) gst(ctrl + 10, ax);
    if (t == 11) gst(ctrl + 11, ay);
  }
}

// ---------------------------------------------------------------------------
// n_steps whole steps of a 1D grid that one workgroup holds (nx < NT: one thread
// per cell and per interface).  The state stays in registers and LDS; each step
// does what k_begin, k_alpha, the three stages and k_finish do, with the same
// formulas in the same order, and leaves the same control block, tapes and
// stage states behind (up to the last bits: the compiler fuses other operations).
// A stage of such a grid is a few hundred instructions, and a step by launches was
// nothing but their cost: 64 steps of 200 cells of linear advection took 256
// launches at 3.6 us each, 0.93 ms, and take 0.25 ms in one.  Two barriers per stage
// order the two state buffers, the fluxes and the speeds: whoever writes one of them
// has passed a barrier after its last reads.
// ---------------------------------------------------------------------------
template <typename T, int PHYS, int NT, int MODE>
__global__ __launch_bounds__(NT) void k_steps_1d(StageArgs<T> a, Consts<T> k, T* s1, T* s2,
                                                 double* tapes, const double* replay,
                                                 int n_steps) {
  constexpr int M = Comps<PHYS, 1>::M;
  constexpr int NF = Comps<PHYS, 1>::NF;
  constexpr bool PROJ = PHYS == PH_EULER && MODE != MODE_COMP;
  constexpr int W = NT + 4;
  __shared__ T sm[2][NF * W];
  __shared__ T fb[2 * M * NT];
  __shared__ unsigned long long red[NT / 64];
  __shared__ uint32_t seen;  // status flags of the launch
  const int tid = threadIdx.x, nx = a.nx;
  const long long fs = a.fs;
  const bool owner = tid < nx;
  const T hx = T(a.dx), idx = T(1.0 / a.dx);
  if (tid == 0) seen = 0;

  // the ghosts (-2, -1, nx, nx + 1) that hold this cell
  uint32_t ghost = 0;
  if (owner) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (map_index2(g < 2 ? g - 2 : nx + g - 2, nx, a.bc_x) == tid) ghost |= 1u << g;
  }
  const bool wall = a.bc_x == HWENO_BC_REFLECT;
  T cur[NF], s0[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) cur[f] = owner ? gld(a.in + f * fs + tid) : T(0);
  auto publish = [&](int buf) __attribute__((always_inline)) {
    if (owner) {
#pragma unroll
      for (int f = 0; f < NF; ++f) sm[buf][f * W + 2 + tid] = staged(cur[f], f, M, hx, hx);
      if (ghost) {
        for (int g = 0; g < 4; ++g) {
          if (!(ghost >> g & 1)) continue;
          const int at = g < 2 ? g : nx + g;
#pragma unroll
          for (int f = 0; f < NF; ++f) {
            const T x = staged(cur[f], f, M, hx, hx);
            sm[buf][f * W + at] = wall && mirror_sign(f, M, true, 0) < 0 ? -x : x;
          }
        }
      }
    }
  };
  // speeds of the current state into red, flags into seen
  auto speeds = [&](bool fold) __attribute__((always_inline)) {
    T sx = T(0), sy = T(0);
    uint32_t flags = 0;
    if (owner) point_speeds<T, PHYS, 1>(cur, k, sx, sy, flags);
    if (fold) {
      sx = wave_max(sx);
      if ((tid & 63) == 0) red[tid >> 6] = dbits(double(sx));
    }
    if (flags) atomicOr(&seen, flags);
  };
  auto reduced = [&]() __attribute__((always_inline)) -> double {
    unsigned long long m = red[0];
#pragma unroll
    for (int q = 1; q < NT / 64; ++q) m = red[q] > m ? red[q] : m;
    return __longlong_as_double((long long)m);
  };

  // every thread keeps the step's scalars; thread 0 writes them
  double t = a.ctrl[7], count = a.ctrl[9];
  double al[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, dt = 0.0;
  unsigned long long status = dbits(a.ctrl[8]);
  __syncthreads();  // seen is cleared
  publish(0);
  if (!replay) speeds(true);
  __syncthreads();
  double next = replay ? 0.0 : reduced();  // stage-1 speed of the next step
  bool ran = false, skipped = false;
  int buf = 0;
  for (int n = 0; n < n_steps; ++n) {
    if (replay) {
#pragma unroll
      for (int q = 0; q < 6; ++q) al[q] = replay[q];
      dt = replay[6];
    } else {
      al[0] = next;
      al[2] = al[4] = 0.0;
      dt = step_dt<1>(next, 0.0, a.dt_fixed, a.t_end, t, a.cfl, a.dx, 1.0);
      if (dt == 0.0) status |= HWENO_ST_SKIPPED;
    }
    skipped = !(dt > 0.0);
    if (!skipped) {
      ran = true;
      const T tdt = T(dt);
#pragma unroll 1
      for (int K = 1; K <= 3; ++K) {
        const T* S = sm[buf];
        if (tid <= nx) {
          const T* row = S + tid;  // points of interface tid: cells tid - 2 .. tid + 1
          auto ld = [&](int p, T* U, T* Dn, T*) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < M; ++c) U[c] = row[c * W + p], Dn[c] = row[(M + c) * W + p];
          };
          T fh[M], hh[M], xx[M];
          interface_fluxes<T, PHYS, M, false, PROJ>(ld, T(K == 1 ? al[0] : (K == 2 ? al[2] : al[4])),
                                                    k.ax, k, fh, hh, xx);
#pragma unroll
          for (int c = 0; c < M; ++c) fb[c * NT + tid] = fh[c], fb[(M + c) * NT + tid] = hh[c];
        }
        __syncthreads();
        if (owner) {
          const T* own = S + tid + 2;
          T L[NF], Sh[NF];
#pragma unroll
          for (int c = 0; c < M; ++c) {
            L[c] = (fb[c * NT + tid] - fb[c * NT + tid + 1]) * (T(0.5) * idx);
            L[M + c] = (fb[(M + c) * NT + tid] - fb[(M + c) * NT + tid + 1]) * (T(0.125) * idx) * idx;
            Sh[c] = cur[c];
            Sh[M + c] = cur[M + c];
          }
          if (k.limiter_on) {
            T d1[M], d2[M], vs[M], vd[M];
#pragma unroll
            for (int c = 0; c < M; ++c) {
              const T* u = own + c * W;
              const T* v = own + (M + c) * W;
              d1[c] = u[0] - u[-1], d2[c] = u[1] - u[0];
              vs[c] = v[-1] + v[1], vd[c] = v[-1] - v[1];
            }
            bool charlim = false;
            if constexpr (PHYS == PH_EULER && MODE != MODE_CHAR) {
              charlim = MODE == MODE_CHAR_LIM || k.limiter_char;
              if (charlim) {
                T r[M];
                limit_char_d<T, M>(cur, d1, d2, vs, vd, k.lb, k.gm1, r);
#pragma unroll
                for (int c = 0; c < M; ++c) Sh[M + c] = idx * r[c];
              }
            }
            if (!charlim) {
#pragma unroll
              for (int c = 0; c < M; ++c) Sh[M + c] = idx * limit_blend(d1[c], d2[c], vs[c], vd[c], k.lb);
            }
          }
          if (K == 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) s0[f] = Sh[f], cur[f] = Sh[f] + tdt * L[f];
            if (k.limiter_on) {
#pragma unroll
              for (int f = M; f < NF; ++f) gst(a.base + (f - M) * fs + tid, Sh[f]);
            }
          } else {
#pragma unroll
            for (int f = 0; f < NF; ++f) cur[f] = rk_combine(K, s0[f], Sh[f] + tdt * L[f]);
          }
          if (K < 3) {
            T* st = K == 1 ? s1 : s2;
#pragma unroll
            for (int f = 0; f < NF; ++f) gst(st + f * fs + tid, cur[f]);
          }
        }
        buf ^= 1;
        publish(buf);
        speeds(!replay);
        __syncthreads();
        if (!replay) {
          const double m = reduced();
          if (K == 1) al[2] = m;
          else if (K == 2) al[4] = m;
          else next = m;
        }
      }
      t += dt;
      count += 1.0;
    }
    status |= seen;
    if (tapes && tid == 0) {
      double* tape = tapes + (long long)n * HWENO_CTRL_LEN;
      for (int q = 0; q < 6; ++q) tape[q] = al[q];
      tape[6] = dt;
      tape[7] = t;
      tape[8] = __longlong_as_double((long long)status);
      tape[9] = count;
    }
  }
  if (ran && owner) {
#pragma unroll
    for (int f = 0; f < NF; ++f) gst(a.out + f * fs + tid, cur[f]);
  }
  if (tid == 0) {
    for (int q = 0; q < 6; ++q) a.ctrl[q] = al[q];
    a.ctrl[6] = dt;
    a.ctrl[7] = t;
    a.ctrl[8] = __longlong_as_double((long long)status);
    a.ctrl[9] = count;
    // as k_finish leaves them after a step that was skipped, or was not
    a.ctrl[10] = skipped ? al[0] : 0.0;
    a.ctrl[11] = skipped ? al[1] : 0.0;
  }
}

// One neighbour of a cell for the limiter: its cell index and what a ghost
// there holds (0: a copy, 1: the mirror image with the wall signs, 2: the
// prescribed state `st` with zero derivatives).
struct LimNb {
  long long at;
  int mode;
  const double* st;
};

// Limited derivatives (Section 2.2), one thread per cell, all components; bound by
// memory, with the neighbours' reads answered by the caches.  A workgroup holds 2^lx
// columns of 256 / 2^lx rows, so that no thread divides to find its cell.  EDG:
// edge-described sides and obstacles; they index the kernel's arguments by lane, which
// the compiler serves from a copy in scratch memory (424 B a thread), and so are an
// instantiation of their own, which is as slow as every grid was before.  2D Euler
// without them, 1999 x 1501 FP64: 389 -> 130 us, 3.7 TB/s of one read and one write (a
// large copy reaches 5.1); 1024^2, whose 168 MB (FP64) partly stay in the last-level
// cache from call to call: FP64 138 -> 27 us, FP32 114 -> 19 us.
template <typename T, int PHYS, int DIM, bool EDG>
__global__ __launch_bounds__(256) void k_limit(const T* __restrict__ S, T* __restrict__ out,
                                               int nx, int ny, int lx, int bc_x, int bc_y,
                                               double dx, double dy, Consts<T> k, EdgeArgs e) {
  constexpr int M = Comps<PHYS, DIM>::M;
  const long long n = (long long)nx * ny;
  const int ntx = ((nx - 1) >> lx) + 1;
  const int tile_y = (int)blockIdx.x / ntx, tile_x = (int)blockIdx.x - tile_y * ntx;
  const int gi = (tile_x << lx) + ((int)threadIdx.x & ((1 << lx) - 1));
  const int gj = (tile_y << (8 - lx)) + ((int)threadIdx.x >> lx);
  if (gi >= nx || gj >= ny) return;
  const long long i = (long long)gj * nx + gi;
  constexpr bool EU = PHYS == PH_EULER;
  if constexpr (EDG) {
    if (e.oj > 0 && solid_cell(e, gi, gj)) {
      // solid cells keep their derivatives
      for (int f = 0; f < M * DIM; ++f) gst(out + f * n + i, gld(S + (M + f) * n + i));
      return;
    }
  }
  // neighbour at index q (column or row) along direction d; one cell deep,
  // so mirror and copy read the same interior cell
  auto neighbour = [&](int q, int d) -> LimNb {
    const int nn = d == 0 ? nx : ny, bc = d == 0 ? bc_x : bc_y;
    const int mq = map_index(q, nn, bc);
    LimNb r;
    r.at = d == 0 ? (long long)gj * nx + mq : (long long)mq * nx + gi;
    r.mode = mirrored(q, nn, bc) ? 1 : 0;
    r.st = nullptr;
    if constexpr (!EDG) return r;
    if (e.oj > 0 && (d == 0 ? solid_cell(e, q, gj) : solid_cell(e, gi, q))) {
      // a solid neighbour is the cell's own mirror image across the obstacle's face
      r.at = i;
      r.mode = 1;
      return r;
    }
    if (bc == HWENO_BC_EDGES && (q < 0 || q >= nn)) {
      const int side = 2 * d + (q < 0 ? 0 : 1);
      const double pos = d == 0 ? (gj + 0.5) * dy : (gi + 0.5) * dx;
      const int sg = edge_segment(e, side, pos, 0.5 * (d == 0 ? dx : dy), e.t0);
      const int kd = e.kind[side][sg];
      r.mode = kd == HWENO_SEG_REFLECT ? 1 : (kd == HWENO_SEG_STATE ? 2 : 0);
      r.st = e.state[side][sg];
    }
    return r;
  };
  const LimNb nxm = neighbour(gi - 1, 0), nxp = neighbour(gi + 1, 0);
  // value of field f at a neighbour: a copy, the wall signs of a mirrored
  // ghost, or an inflow state
  auto nbv = [&](int f, const LimNb& b, int d) -> T {
    if (EDG && b.mode == 2) return f < M ? T(b.st[f]) : T(0);
    const T x = gld(S + f * n + b.at);
    return (b.mode == 1 && mirror_sign(f, M, EU, d) < 0) ? -x : x;
  };
  if (EU && k.limiter_char) {
    // characteristic variant (normal frame: the momenta swap places for y)
    T um[M], u0[M], up[M], vm[M], vp[M], r[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
      um[c] = nbv(c, nxm, 0), u0[c] = gld(S + c * n + i), up[c] = nbv(c, nxp, 0);
      vm[c] = nbv(M + c, nxm, 0), vp[c] = nbv(M + c, nxp, 0);
    }
    limit_char<T, M>(um, u0, up, vm, vp, T(dx), T(1.0 / dx), k.lw, k.gm1, r);
#pragma unroll
    for (int c = 0; c < M; ++c) gst(out + c * n + i, r[c]);
    if constexpr (DIM == 2) {
      const LimNb nym = neighbour(gj - 1, 1), nyp = neighbour(gj + 1, 1);
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const int q = (c == 1) ? 2 : (c == 2) ? 1 : c;
        um[c] = nbv(q, nym, 1), u0[c] = gld(S + q * n + i), up[c] = nbv(q, nyp, 1);
        vm[c] = nbv(2 * M + q, nym, 1), vp[c] = nbv(2 * M + q, nyp, 1);
      }
      limit_char<T, M>(um, u0, up, vm, vp, T(dy), T(1.0 / dy), k.lw, k.gm1, r);
#pragma unroll
      for (int c = 0; c < M; ++c) gst(out + (M + ((c == 1) ? 2 : (c == 2) ? 1 : c)) * n + i, r[c]);
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < M; ++c) {
    gst(out + c * n + i, limit1(nbv(c, nxm, 0), gld(S + c * n + i), nbv(c, nxp, 0), nbv(M + c, nxm, 0),
                                nbv(M + c, nxp, 0), T(dx), T(1.0 / dx), k.lw));
  }
  if constexpr (DIM == 2) {
    const LimNb nym = neighbour(gj - 1, 1), nyp = neighbour(gj + 1, 1);
#pragma unroll
    for (int c = 0; c < M; ++c) {
      gst(out + (M + c) * n + i, limit1(nbv(c, nym, 1), gld(S + c * n + i), nbv(c, nyp, 1),
                                        nbv(2 * M + c, nym, 1), nbv(2 * M + c, nyp, 1), T(dy), T(1.0 / dy), k.lw));
    }
  }
}

}  // namespace hweno

// ===========================================================================
// host side
// ===========================================================================
using namespace hweno;

// Stage states and limited base derivatives of the allocation-free step
// (hweno_rk3_step_static).  Each GPU that runs the library holds its own copy
// for the life of the process.  On the host this name is only a handle for
// hipGetSymbolAddress: kernels receive the device address it returns.
static __device__ __align__(256) unsigned char scratch[HWENO_STATIC_SCRATCH_BYTES];
// its speed slots
static __device__ __align__(256) double scratch_fold[NSLOT * SLOT_LEN];

namespace {

thread_local std::string g_last_error;

// stage-kernel timing (diagnostics, per host thread)
struct Timing {
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  size_t used = 0;
};
thread_local Timing g_timing;

hipEvent_t* timing_pair(hipStream_t s, bool start) {
  (void)s;
  if (!g_timing.on) return nullptr;
  if (start) {
    if (g_timing.used == g_timing.ev.size()) {
      hipEvent_t a, b;
      if (hipEventCreate(&a) != hipSuccess) return nullptr;
      if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return nullptr; }
      g_timing.ev.emplace_back(a, b);
    }
    return &g_timing.ev[g_timing.used].first;
  }
  return &g_timing.ev[g_timing.used++].second;
}

void timing_release() {
  for (auto& e : g_timing.ev) {
    (void)hipEventDestroy(e.first);
    (void)hipEventDestroy(e.second);
  }
  g_timing.ev.clear();
  g_timing.used = 0;
  g_timing.on = false;
}

// launches one stage kernel, bracketed by timing events when enabled
template <typename Launch>
void timed(hipStream_t s, Launch&& launch) {
  hipEvent_t* a = timing_pair(s, true);
  if (a) (void)hipEventRecord(*a, s);
  launch();
  if (a) (void)hipEventRecord(*timing_pair(s, false), s);
}

hweno_status fail(hweno_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

hweno_status ok() {
  g_last_error.clear();
  return HWENO_OK;
}

int n_comp(const hweno_problem* p) {
  if (p->physics == HWENO_EULER) return p->dim == 1 ? 3 : 4;
  return 1;
}

int n_fields(const hweno_problem* p) { return n_comp(p) * (1 + p->dim); }

size_t elem_size(const hweno_problem* p) { return p->dtype == HWENO_F64 ? 8 : 4; }

bool weights_ok(const double* w) {
  if (!(w[0] > 0.0 && w[1] > 0.0 && w[2] > 0.0)) return false;
  if (!std::isfinite(w[0] + w[1] + w[2])) return false;
  return std::fabs(w[0] + w[1] + w[2] - 1.0) <= 1e-12;
}

bool has_edges(const hweno_problem* p) {
  return p->bc_x == HWENO_BC_EDGES || (p->dim == 2 && p->bc_y == HWENO_BC_EDGES);
}

hweno_status validate(const hweno_problem* p) {
  if (!p) return fail(HWENO_ERR_INVALID_ARG, "problem pointer is NULL");
  if (p->dim != 1 && p->dim != 2) return fail(HWENO_ERR_INVALID_ARG, "dim must be 1 or 2 (got %d)", p->dim);
  if (p->nx < 0 || p->ny < 0) return fail(HWENO_ERR_INVALID_ARG, "nx, ny must be >= 0");
  if (p->dim == 1 && p->ny != 1 && p->ny != 0)
    return fail(HWENO_ERR_INVALID_ARG, "ny must be 1 for dim == 1 (got %d)", p->ny);
  if (p->physics < HWENO_LINADV || p->physics > HWENO_EULER)
    return fail(HWENO_ERR_INVALID_ARG, "unknown physics %d", p->physics);
  if (p->dtype != HWENO_F32 && p->dtype != HWENO_F64)
    return fail(HWENO_ERR_INVALID_ARG, "unknown dtype %d", p->dtype);
  auto bc_ok = [](int b) {
    return b == HWENO_BC_PERIODIC || b == HWENO_BC_OUTFLOW || b == HWENO_BC_REFLECT ||
           b == HWENO_BC_EDGES;
  };
  if (!bc_ok(p->bc_x) || (p->dim == 2 && !bc_ok(p->bc_y)))
    return fail(HWENO_ERR_INVALID_ARG, "unknown boundary condition");
  if (p->obstacle[0] != 0 || p->obstacle[1] != 0) {
    if (p->dim != 2 || p->bc_x != HWENO_BC_EDGES)
      return fail(HWENO_ERR_UNSUPPORTED, "an obstacle needs a 2D grid with edge-described x sides");
    if (p->obstacle[0] < 2 || p->obstacle[0] > p->nx || p->obstacle[1] < 1 ||
        p->obstacle[1] > p->ny - 2)
      return fail(HWENO_ERR_INVALID_ARG,
                  "obstacle {%d, %d}: needs 2 <= i_s <= nx and 1 <= j_s <= ny - 2",
                  p->obstacle[0], p->obstacle[1]);
  }
  if (has_edges(p)) {
    if (p->physics != HWENO_EULER || p->dim != 2)
      return fail(HWENO_ERR_UNSUPPORTED, "edge-described sides are built for 2D Euler");
    for (int d = 0; d < 2; ++d) {
      if ((d == 0 ? p->bc_x : p->bc_y) != HWENO_BC_EDGES) continue;
      const int across = d == 0 ? p->nx : p->ny;
      for (int side = 0; side < 2; ++side) {
        const hweno_edge& e = p->edges[2 * d + side];
        bool out = false, wall = false;
        for (int sg = 0; sg < 2; ++sg) {
          const int kd = e.kind[sg];
          if (kd != HWENO_SEG_OUTFLOW && kd != HWENO_SEG_REFLECT && kd != HWENO_SEG_STATE)
            return fail(HWENO_ERR_INVALID_ARG, "edge %d: unknown segment kind %d", 2 * d + side, kd);
          out = out || kd == HWENO_SEG_OUTFLOW;
          wall = wall || kd == HWENO_SEG_REFLECT;
          if (kd == HWENO_SEG_STATE) {
            const double* q = e.state[sg];
            for (int c = 0; c < 4; ++c)
              if (!std::isfinite(q[c]))
                return fail(HWENO_ERR_INVALID_ARG, "edge %d: state %d is not finite", 2 * d + side, sg);
            const double pr =
                (p->gamma_gas - 1.0) * (q[3] - 0.5 * (q[1] * q[1] + q[2] * q[2]) / q[0]);
            if (!(q[0] > 0.0) || !(pr > 0.0))
              return fail(HWENO_ERR_INVALID_ARG,
                          "edge %d: state %d needs positive density and pressure", 2 * d + side, sg);
          }
        }
        for (int k = 0; k < 3; ++k)
          if (!std::isfinite(e.split[k]))
            return fail(HWENO_ERR_INVALID_ARG, "edge %d: split is not finite", 2 * d + side);
        if (out && wall)
          return fail(HWENO_ERR_INVALID_ARG, "edge %d combines an outflow and a wall segment",
                      2 * d + side);
        if (wall && across < 2)
          return fail(HWENO_ERR_INVALID_ARG, "a reflecting wall needs at least 2 cells across");
      }
    }
  }
  if (p->physics != HWENO_EULER &&
      (p->bc_x == HWENO_BC_REFLECT || (p->dim == 2 && p->bc_y == HWENO_BC_REFLECT)))
    return fail(HWENO_ERR_UNSUPPORTED, "reflecting walls are defined for the Euler equations only");
  // the two ghost cells mirror two distinct interior cells
  if ((p->bc_x == HWENO_BC_REFLECT && p->nx == 1) ||
      (p->dim == 2 && p->bc_y == HWENO_BC_REFLECT && p->ny == 1))
    return fail(HWENO_ERR_INVALID_ARG, "a reflecting wall needs at least 2 cells across");
  if (p->limiter_characteristic != 0 && p->limiter_characteristic != 1)
    return fail(HWENO_ERR_INVALID_ARG, "limiter_characteristic must be 0 or 1");
  if (!(p->dx > 0.0) || !std::isfinite(p->dx)) return fail(HWENO_ERR_INVALID_ARG, "dx must be > 0");
  if (p->dim == 2 && (!(p->dy > 0.0) || !std::isfinite(p->dy)))
    return fail(HWENO_ERR_INVALID_ARG, "dy must be > 0");
  if (!weights_ok(p->lin_w))
    return fail(HWENO_ERR_INVALID_ARG, "linear weights gamma must be > 0 and sum to 1 (got %.17g %.17g %.17g)",
                p->lin_w[0], p->lin_w[1], p->lin_w[2]);
  if (!weights_ok(p->lim_w))
    return fail(HWENO_ERR_INVALID_ARG, "limiter weights d must be > 0 and sum to 1 (got %.17g %.17g %.17g)",
                p->lim_w[0], p->lim_w[1], p->lim_w[2]);
  if (!(p->eps > 0.0) || !std::isfinite(p->eps)) return fail(HWENO_ERR_INVALID_ARG, "eps must be > 0");
  if (!(p->cfl > 0.0) || !std::isfinite(p->cfl)) return fail(HWENO_ERR_INVALID_ARG, "cfl must be > 0");
  if (p->physics == HWENO_EULER && (!(p->gamma_gas > 1.0) || !std::isfinite(p->gamma_gas)))
    return fail(HWENO_ERR_INVALID_ARG, "gamma_gas must be > 1");
  if (p->physics == HWENO_LINADV &&
      (!std::isfinite(p->adv_speed[0]) || !std::isfinite(p->adv_speed[1])))
    return fail(HWENO_ERR_INVALID_ARG, "advection speeds must be finite");
  const double cells = (double)p->nx * (double)(p->dim == 2 ? p->ny : 1);
  if (cells * n_fields(p) > 9.0e18 / 8.0) return fail(HWENO_ERR_INVALID_ARG, "grid too large");
  if (p->nx > (1 << 28) || p->ny > (1 << 28)) return fail(HWENO_ERR_INVALID_ARG, "grid side too large");
  return ok();
}

bool empty(const hweno_problem* p) { return p->nx == 0 || (p->dim == 2 && p->ny == 0); }

long long cells_of(const hweno_problem* p) {
  return (long long)p->nx * (p->dim == 2 ? p->ny : 1);
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct WsLayout {
  size_t ctrl, s1, s2, base, fold, total;
};

WsLayout ws_layout(const hweno_problem* p) {
  WsLayout L;
  const size_t fb = (size_t)cells_of(p) * elem_size(p);
  L.ctrl = 0;
  L.s1 = align256(HWENO_CTRL_LEN * sizeof(double));
  L.s2 = L.s1 + align256(fb * n_fields(p));
  L.base = L.s2 + align256(fb * n_fields(p));
  L.fold = L.base + align256(fb * n_comp(p) * p->dim);
  L.total = L.fold + NSLOT * SLOT_LEN * sizeof(double);
  return L;
}

template <typename T>
Consts<T> make_consts(const hweno_problem* p) {
  Consts<T> k;
  k.rw = {T(p->lin_w[0]), T(p->lin_w[1]), T(p->lin_w[2]), T(p->eps),
          T(p->lin_w[0]) + T(p->lin_w[1]) + T(p->lin_w[2])};
  k.lw = {T(p->lim_w[0]), T(p->lim_w[1]), T(p->lim_w[2]), T(p->eps),
          T(p->lim_w[0]) + T(p->lim_w[1]) + T(p->lim_w[2])};
  k.gm1 = T(p->gamma_gas - 1.0);
  k.gam = T(p->gamma_gas);
  k.ax = T(p->adv_speed[0]);
  k.ay = T(p->adv_speed[1]);
  k.limiter_on = p->limiter_on ? 1 : 0;
  k.limiter_char = p->limiter_characteristic ? 1 : 0;
  k.rb = recon_blend(T(p->lin_w[1]), T(p->lin_w[2]), T(p->eps));
  k.lb = limit_blend_weights(T(p->lim_w[1]), T(p->lim_w[2]), T(p->eps));
  return k;
}

// the characteristic limiter variant is in force (Euler with the limiter on)
bool char_limiter(const hweno_problem* p) {
  return p->physics == HWENO_EULER && p->limiter_on && p->limiter_characteristic;
}

// calls f(integral constant) with the stage kernels' MODE for an Euler problem
template <typename F>
void with_mode(const hweno_problem* p, F&& f) {
  if (!p->characteristic)
    f(std::integral_constant<int, MODE_COMP>{});
  else if (char_limiter(p))
    f(std::integral_constant<int, MODE_CHAR_LIM>{});
  else
    f(std::integral_constant<int, MODE_CHAR>{});
}

hweno_status launch_check(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HWENO_ERR_LAUNCH, "%s: %s", what, hipGetErrorString(e));
  return HWENO_OK;
}

// 2D tile: 16 x 15 cells on 256 threads gives 255 x-interfaces and 256
// y-interfaces, i.e. one balanced pass per direction.  1D tile: 255 cells have
// 256 interfaces, one per thread (with 256 cells the first wave took a second
// pass for the 257th, doubling the stage's critical path on small grids).
template <int DIM>
struct Tile {
  static constexpr int TX = (DIM == 2) ? 16 : 255;
  static constexpr int TY = (DIM == 2) ? 15 : 1;
  static constexpr int NT = 256;
};

// dispatch helper: calls F::template run<T, PHYS, DIM>(args...)
template <typename F, typename... Args>
hweno_status dispatch(const hweno_problem* p, Args&&... args) {
#define HWENO_CASE(TT, PH, D)                                                  \
  if (p->dtype == (sizeof(TT) == 8 ? HWENO_F64 : HWENO_F32) && p->physics == PH && \
      p->dim == D)                                                             \
    return F::template run<TT, PH, D>(p, args...);
  HWENO_CASE(double, HWENO_LINADV, 1)
  HWENO_CASE(double, HWENO_BURGERS, 1)
  HWENO_CASE(double, HWENO_EULER, 1)
  HWENO_CASE(double, HWENO_LINADV, 2)
  HWENO_CASE(double, HWENO_BURGERS, 2)
  HWENO_CASE(double, HWENO_EULER, 2)
  HWENO_CASE(float, HWENO_LINADV, 1)
  HWENO_CASE(float, HWENO_BURGERS, 1)
  HWENO_CASE(float, HWENO_EULER, 1)
  HWENO_CASE(float, HWENO_LINADV, 2)
  HWENO_CASE(float, HWENO_BURGERS, 2)
  HWENO_CASE(float, HWENO_EULER, 2)
#undef HWENO_CASE
  return fail(HWENO_ERR_UNSUPPORTED, "unsupported combination");
}

EdgeArgs edge_args(const hweno_problem* p) {
  EdgeArgs e;
  std::memset(&e, 0, sizeof e);
  for (int side = 0; side < 4; ++side) {
    const hweno_edge& h = p->edges[side];
    for (int sg = 0; sg < 2; ++sg) {
      e.kind[side][sg] = h.kind[sg];
      for (int c = 0; c < 4; ++c) e.state[side][sg][c] = h.state[sg][c];
    }
    e.mirror[side] = h.kind[0] == HWENO_SEG_REFLECT || h.kind[1] == HWENO_SEG_REFLECT;
    for (int q = 0; q < 3; ++q) e.split[side][q] = h.split[q];
  }
  e.t0 = 0.0;
  e.oi = p->obstacle[0];
  e.oj = p->obstacle[1];
  return e;
}

template <typename T, int PHYS, int DIM>
StageArgs<T> base_args(const hweno_problem* p) {
  StageArgs<T> a;
  std::memset(&a, 0, sizeof a);
  a.nx = p->nx;
  a.ny = DIM == 2 ? p->ny : 1;
  a.bc_x = p->bc_x;
  a.bc_y = p->bc_y;
  a.fs = cells_of(p);
  a.dx = p->dx;
  a.dy = DIM == 2 ? p->dy : 1.0;
  a.cfl = p->cfl;
  return a;
}

dim3 stage_grid(int dim, int nx, int ny) {
  if (dim == 2)
    return dim3(((nx + Tile<2>::TX - 1) / Tile<2>::TX) * ((ny + Tile<2>::TY - 1) / Tile<2>::TY));
  return dim3((nx + Tile<1>::TX - 1) / Tile<1>::TX);
}

// Workgroups of a speed reduction of 256 threads into the slots: two cells a thread
// (eight single steps of 96 x 64: 317 us, with eight cells a thread 340 us).
unsigned alpha_blocks(long long n) {
  return (unsigned)std::min<long long>(2048, std::max<long long>(1, (n + 511) / 512));
}

// Workgroups of 1024 threads of a reduction on one address, where each one's atomics
// queue behind the others' (15 ns).  With the one stage that follows, 512 workgroups of
// 256 threads, 256, 128 and 64 of 1024: 1024^2 FP32 76.9, 68.8, 67.4, 69.8 us; 2000^2
// FP64 384.8, 355.5, 362.8, 384.3 us.
unsigned alpha_blocks_one(long long n) {
  return (unsigned)std::min<long long>(256, std::max<long long>(1, (n + 4095) / 4096));
}

struct RunAlpha {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, const void* state, double* alpha,
                          unsigned long long* status, hipStream_t s) {
    const long long n = cells_of(p);
    k_zero<<<1, 64, 0, s>>>(alpha, 2);
    if constexpr (PHYS == PH_EULER && DIM == 2) {
      if (p->obstacle[1] > 0) {
        k_alpha_obstacle<T><<<std::min(alpha_blocks(n), 256u), 256, 0, s>>>(
            (const T*)state, p->nx, p->ny, p->obstacle[0], p->obstacle[1], make_consts<T>(p),
            alpha, 1, status);
        return launch_check("alpha");
      }
    }
    k_alpha<T, PHYS, DIM, 1024><<<alpha_blocks_one(n), 1024, 0, s>>>((const T*)state, n,
                                                                     make_consts<T>(p), alpha, 1, status);
    return launch_check("alpha");
  }
};

struct RunRhs {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, const void* state, void* rhs,
                          double* alpha, int compute, hipStream_t s) {
    if (compute) {
      hweno_status st = RunAlpha::run<T, PHYS, DIM>(p, state, alpha, nullptr, s);
      if (st) return st;
    }
    StageArgs<T> a = base_args<T, PHYS, DIM>(p);
    a.in = (const T*)state;
    a.out = (T*)rhs;
    a.alpha = alpha;
    constexpr int TX = Tile<DIM>::TX, TY = Tile<DIM>::TY, NT = Tile<DIM>::NT;
    const dim3 grid = stage_grid(DIM, a.nx, a.ny);
    const Consts<T> k = make_consts<T>(p);
    // the limiter plays no part in the right-hand side
    auto launch = [&](auto mode) {
      constexpr int MODE = decltype(mode)::value;
      if constexpr (PHYS == PH_EULER && DIM == 2) {
        if (has_edges(p)) {
          k_stage_edges<T, 0, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k, edge_args(p));
          return;
        }
      }
      k_stage<T, PHYS, DIM, 0, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k);
    };
    if (PHYS == PH_EULER && p->characteristic)
      launch(std::integral_constant<int, PHYS == PH_EULER ? MODE_CHAR : MODE_COMP>{});
    else
      launch(std::integral_constant<int, MODE_COMP>{});
    return launch_check("rhs");
  }
};

struct RunLimit {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, const void* state, void* out, hipStream_t s) {
    const int ny = DIM == 2 ? p->ny : 1;
    // rows of 64 cells, a wavefront's, or of all 256 where no rows share neighbours;
    // narrow grids take the power of two that holds them (a launch of 2^24 workgroups
    // or more fails: so do grids that only their padding would take there)
    auto tiles = [&](int l) {
      const long long rows = 256 >> l;
      return (((p->nx - 1) >> l) + 1) * ((ny + rows - 1) / rows);
    };
    int lx = DIM == 2 ? 6 : 8;
    while (lx > 0 && (p->nx <= 1 << (lx - 1) || tiles(lx) >= 1 << 24)) --lx;
    const unsigned blocks = (unsigned)tiles(lx);
    auto launch = [&](auto kernel) {
      kernel<<<blocks, 256, 0, s>>>((const T*)state, (T*)out, p->nx, ny, lx, p->bc_x, p->bc_y, p->dx,
                                    DIM == 2 ? p->dy : 1.0, make_consts<T>(p), edge_args(p));
    };
    if constexpr (PHYS == PH_EULER && DIM == 2) {
      if (has_edges(p)) {
        launch(k_limit<T, PHYS, DIM, true>);
        return launch_check("limit");
      }
    }
    launch(k_limit<T, PHYS, DIM, false>);
    return launch_check("limit");
  }
};

// where one step keeps its control block, its two stage states, the limited base
// derivatives and the speed slots, and how many of these there are
struct StepBufs {
  double* ctrl;
  void* s1;
  void* s2;
  void* base;
  double* fold;
  int slots;
};

// A workspace that ends before the slots (L.fold bytes or more) has one of them behind
// the control block, in the rest of its 256 bytes.
static_assert((HWENO_CTRL_LEN + SLOT_LEN) * sizeof(double) <= 256, "one slot fits behind the control block");
StepBufs ws_bufs(const hweno_problem* p, void* ws, size_t ws_bytes) {
  const WsLayout L = ws_layout(p);
  char* w = (char*)ws;
  double* ctrl = (double*)(w + L.ctrl);
  const bool all = ws_bytes >= L.total;
  return StepBufs{ctrl, w + L.s1, w + L.s2, w + L.base,
                  all ? (double*)(w + L.fold) : ctrl + HWENO_CTRL_LEN, all ? NSLOT : 1};
}

struct RunStep {
  template <typename T, int PHYS, int DIM>
  // take_next: stage-1 speeds come from the previous step's stage 3 (the state
  // has not changed since); fold_next: this step's stage 3 provides them
  // (multi-step calls: the previous step's k_finish already began this one when
  // take_next, and this one's k_finish begins the next when fold_next).
  // may_time: stage launches may be bracketed by the diagnostic timer's events
  static hweno_status run(const hweno_problem* p, void* state, StepBufs b, double dt_fixed,
                          double t_end, double* tape, const double* replay, bool take_next,
                          bool fold_next, bool may_time, hipStream_t s) {
    double* ctrl = b.ctrl;
    auto timed = [&](hipStream_t st, auto&& launch) {
      if (may_time)
        ::timed(st, launch);
      else
        launch();
    };
    const long long n = cells_of(p);
    const Consts<T> k = make_consts<T>(p);
    const dim3 grid = stage_grid(DIM, p->nx, p->ny);
    const int slots = (int)grid.x > SLOT_FEW ? b.slots : 1;
    if (!(take_next && !replay)) k_begin<<<1, 64, 0, s>>>(ctrl, b.fold, slots, replay);
    if (!replay && !take_next) {
      bool done = false;
      if constexpr (PHYS == PH_EULER && DIM == 2) {
        if (p->obstacle[1] > 0) {
          k_alpha_obstacle<T><<<alpha_blocks(n), 256, 0, s>>>(
              (const T*)state, p->nx, p->ny, p->obstacle[0], p->obstacle[1], k, b.fold, slots,
              (unsigned long long*)(ctrl + 8));
          done = true;
        }
      }
      if (!done)
        k_alpha<T, PHYS, DIM, 256><<<alpha_blocks(n), 256, 0, s>>>(
            (const T*)state, n, k, b.fold, slots, (unsigned long long*)(ctrl + 8));
    }
    StageArgs<T> a = base_args<T, PHYS, DIM>(p);
    a.ctrl = ctrl;
    a.fold = b.fold;
    a.slots = slots;
    a.status = (unsigned long long*)(ctrl + 8);
    a.st0 = (const T*)state;
    a.base = (T*)b.base;
    a.dt_fixed = dt_fixed;
    a.t_end = t_end;
    a.replay = replay ? 1 : 0;
    a.fold_next = (fold_next && !replay) ? 1 : 0;
    T* s1 = (T*)b.s1;
    T* s2 = (T*)b.s2;
    constexpr int TX = Tile<DIM>::TX, TY = Tile<DIM>::TY, NT = Tile<DIM>::NT;
    auto stages = [&](auto mode) {
      constexpr int MODE = decltype(mode)::value;
      a.in = (const T*)state;
      a.out = s1;
      timed(s, [&] { k_stage<T, PHYS, DIM, 1, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k); });
      a.in = s1;
      a.out = s2;
      timed(s, [&] { k_stage<T, PHYS, DIM, 2, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k); });
      a.in = s2;
      a.out = (T*)state;
      timed(s, [&] { k_stage<T, PHYS, DIM, 3, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k); });
    };
    if constexpr (PHYS == PH_EULER) {
      if constexpr (DIM == 2) {
        if (has_edges(p)) {
          const EdgeArgs e = edge_args(p);
          auto edge_stages = [&](auto mode) {
            constexpr int MODE = decltype(mode)::value;
            a.in = (const T*)state;
            a.out = s1;
            timed(s, [&] { k_stage_edges<T, 1, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k, e); });
            a.in = s1;
            a.out = s2;
            timed(s, [&] { k_stage_edges<T, 2, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k, e); });
            a.in = s2;
            a.out = (T*)state;
            timed(s, [&] { k_stage_edges<T, 3, TX, TY, NT, MODE><<<grid, NT, 0, s>>>(a, k, e); });
          };
          with_mode(p, edge_stages);
          k_finish<<<1, 64, 0, s>>>(ctrl, b.fold, slots, tape, fold_next && !replay ? 1 : 0);
          return launch_check("rk3_step");
        }
      }
      with_mode(p, stages);
    } else {
      stages(std::integral_constant<int, MODE_COMP>{});
    }
    k_finish<<<1, 64, 0, s>>>(ctrl, b.fold, slots, tape, fold_next && !replay ? 1 : 0);
    return launch_check("rk3_step");
  }
};

// 1D grids whose steps run in one workgroup (k_steps_1d): fewer than NT2 cells, on NT1
// threads (one wave per SIMD) below NT1.  FP64, 32 steps a call, one workgroup
// against launches, per step: Euler 255 cells 8.7 against 18.3 us, 511 cells 14.3
// against 20.6; linear advection 255 cells 4.1 against 14.6, 1000 cells 10.0
// against 16.1.  Twice as many cells would take twice as long (the waves share the
// SIMDs), more than the launches.
template <int PHYS>
struct OneBlock {
  static constexpr int NT1 = 256, NT2 = PHYS == PH_EULER ? 512 : 1024;
};

// n steps (replay: n == 1); tapes: n records or NULL
struct RunSteps {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, void* state, StepBufs b, int n, double dt_fixed,
                          double t_end, double* tapes, const double* replay, bool may_time,
                          hipStream_t s) {
    if constexpr (DIM == 1) {
      if (p->nx < OneBlock<PHYS>::NT2) {
        StageArgs<T> a = base_args<T, PHYS, 1>(p);
        a.ctrl = b.ctrl;
        a.in = (const T*)state;
        a.out = (T*)state;
        a.base = (T*)b.base;
        a.dt_fixed = dt_fixed;
        a.t_end = t_end;
        const Consts<T> k = make_consts<T>(p);
        // at most 256 steps a launch, so that none runs long
        for (int n0 = 0; n0 < n; n0 += 256) {
          const int m = std::min(256, n - n0);
          double* tp = tapes ? tapes + (size_t)n0 * HWENO_CTRL_LEN : nullptr;
          auto launch = [&](auto mode) {
            constexpr int MODE = decltype(mode)::value;
            constexpr int NT1 = OneBlock<PHYS>::NT1, NT2 = OneBlock<PHYS>::NT2;
            auto steps = [&] {
              if (p->nx < NT1)
                k_steps_1d<T, PHYS, NT1, MODE><<<1, NT1, 0, s>>>(a, k, (T*)b.s1, (T*)b.s2, tp, replay, m);
              else
                k_steps_1d<T, PHYS, NT2, MODE><<<1, NT2, 0, s>>>(a, k, (T*)b.s1, (T*)b.s2, tp, replay, m);
            };
            if (may_time)
              timed(s, steps);
            else
              steps();
          };
          if constexpr (PHYS == PH_EULER)
            with_mode(p, launch);
          else
            launch(std::integral_constant<int, MODE_COMP>{});
          hweno_status st = launch_check("rk3_steps");
          if (st) return st;
        }
        return HWENO_OK;
      }
    }
    for (int q = 0; q < n; ++q) {
      hweno_status st = RunStep::run<T, PHYS, DIM>(
          p, state, b, dt_fixed, t_end, tapes ? tapes + (size_t)q * HWENO_CTRL_LEN : nullptr, replay,
          q > 0, q + 1 < n, may_time, s);
      if (st) return st;
    }
    return HWENO_OK;
  }
};

// 2D adjoint tile: 15 x 14 cells, so the 18 x 14 x-interfaces and the
// 15 x 17 y-interfaces touching it each fit one pass of 256 threads
template <int DIM>
struct AdjTile {
  static constexpr int TX = (DIM == 2) ? 15 : 253;
  static constexpr int TY = (DIM == 2) ? 14 : 1;
  static constexpr int NT = 256;
};

struct AdjLayout {
  size_t e, y2, y1, l0, total;
  int nxe, nye;
};

AdjLayout adj_layout(const hweno_problem* p) {
  AdjLayout L;
  L.nxe = p->nx + 4;
  L.nye = p->dim == 2 ? p->ny + 4 : 1;
  const size_t es = elem_size(p);
  const size_t st = (size_t)cells_of(p) * es * n_fields(p);
  L.e = 0;
  L.y2 = align256((size_t)L.nxe * L.nye * es * n_fields(p));
  L.y1 = L.y2 + align256(st);
  L.l0 = L.y1 + align256(st);
  L.total = L.l0 + align256(st);
  return L;
}

// one adjoint evaluation into E followed by one fold
struct RunAdj {
  template <typename T, int PHYS, int DIM>
  // fuse: finish interior cells inside the adjoint kernel (the fold's output
  // buffers must then not alias S, XL or XM)
  static hweno_status run(const hweno_problem* p, const void* S, const void* XL, double cr,
                          const double* dtp, const void* XM, double cl, const double* alpha,
                          void* ws, FoldArgs<T> fo, bool fuse, hipStream_t s) {
    const AdjLayout L = adj_layout(p);
    AdjArgs<T> a;
    a.S = (const T*)S;
    a.XL = (const T*)XL;
    a.XM = (const T*)XM;
    a.E = (T*)((char*)ws + L.e);
    a.alpha = alpha;
    a.dtp = dtp;
    a.cr = cr;
    a.cl = cl;
    a.nx = p->nx;
    a.ny = DIM == 2 ? p->ny : 1;
    a.bc_x = p->bc_x;
    a.bc_y = p->bc_y;
    a.fs = cells_of(p);
    a.nxe = L.nxe;
    a.nye = L.nye;
    a.dx = p->dx;
    a.dy = DIM == 2 ? p->dy : 1.0;
    fo.E = a.E;
    fo.nxe = L.nxe;
    fo.nye = L.nye;
    fo.nx = a.nx;
    fo.ny = a.ny;
    fo.bc_x = p->bc_x;
    fo.bc_y = p->bc_y;
    fo.dim = DIM;
    fo.nf = Comps<PHYS, DIM>::NF;
    fo.m = Comps<PHYS, DIM>::M;
    fo.euler = PHYS == PH_EULER;
    fo.fs = a.fs;
    a.fused = (fuse && DIM == 2 && a.nx >= 4 && a.ny >= 4) ? 1 : 0;
    a.fo = fo;
    constexpr int TX = AdjTile<DIM>::TX, TY = AdjTile<DIM>::TY, NT = AdjTile<DIM>::NT;
    const unsigned tiles = (unsigned)(((L.nxe + TX - 1) / TX) * ((L.nye + TY - 1) / TY));
    auto launch = [&](auto mode) {
      timed(s, [&] {
        k_adjoint<T, PHYS, DIM, TX, TY, NT, decltype(mode)::value><<<tiles, NT, 0, s>>>(a, make_consts<T>(p));
      });
    };
    if constexpr (PHYS == PH_EULER)
      with_mode(p, launch);
    else
      launch(std::integral_constant<int, MODE_COMP>{});
    if (a.fused) {
      const long long nb = (4ll * a.ny + 4ll * (a.nx - 4)) * fo.nf;
      k_fold_band<T><<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(fo);
    } else {
      k_fold<T><<<(unsigned)((a.fs * fo.nf + 255) / 256), 256, 0, s>>>(fo);
    }
    return launch_check("adjoint");
  }
};

template <typename T>
FoldArgs<T> fold_args(void* out, int accumulate, const void* XU, double cu, int identity_all) {
  FoldArgs<T> f;
  std::memset(&f, 0, sizeof f);
  f.out = (T*)out;
  f.accumulate = accumulate;
  f.XU = (const T*)XU;
  f.cu = cu;
  f.identity_all = identity_all;
  return f;
}

struct RunRhsAdj {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, const void* state, const double* alpha,
                          const void* lam_rhs, const void* lam_lim, void* lam_state, void* ws,
                          hipStream_t s) {
    // the caller's buffers may alias: fold in a separate pass
    return RunAdj::run<T, PHYS, DIM>(p, state, lam_rhs, 1.0, nullptr, lam_lim, 1.0, alpha, ws,
                                     fold_args<T>(lam_state, 1, nullptr, 0.0, 0), false, s);
  }
};

struct RunStepAdj {
  template <typename T, int PHYS, int DIM>
  static hweno_status run(const hweno_problem* p, const void* state0, const void* step_ws,
                          const double* tape, void* lam, void* ws, hipStream_t s) {
    const WsLayout F = ws_layout(p);
    const AdjLayout L = adj_layout(p);
    const char* sw = (const char*)step_ws;
    const void* S1 = sw + F.s1;
    const void* S2 = sw + F.s2;
    char* w = (char*)ws;
    T* Y2 = (T*)(w + L.y2);
    T* Y1 = (T*)(w + L.y1);
    T* L0 = (T*)(w + L.l0);
    const bool lim = p->limiter_on != 0;
    const long long mN = (long long)n_comp(p) * cells_of(p);
    const int ida = lim ? 0 : 1;
    hweno_status st;
    // stage 3: S^{n+1} = 1/3 S^0 + 2/3 (S^2 + dt L(S2)),  S^ = (U, Lim(S))
    // (each stage's fold writes a buffer its adjoint kernel does not read: fused)
    st = RunAdj::run<T, PHYS, DIM>(p, S2, lam, 2.0 / 3.0, tape + 6,
                                   lim ? (const T*)lam + mN : nullptr, 2.0 / 3.0, tape + 4, ws,
                                   fold_args<T>(Y2, 0, lam, 2.0 / 3.0, ida), true, s);
    if (st) return st;
    // stage 2: S2 = 3/4 S^0 + 1/4 (S^1 + dt L(S1));  L0 = lam/3 + 3/4 Y2 + Y1
    FoldArgs<T> f2 = fold_args<T>(Y1, 0, Y2, 0.25, ida);
    f2.L0 = L0;
    f2.A = (const T*)lam;
    f2.B = Y2;
    f2.ca = 1.0 / 3.0;
    f2.cb = 0.75;
    st = RunAdj::run<T, PHYS, DIM>(p, S1, Y2, 0.25, tape + 6, lim ? Y2 + mN : nullptr, 0.25,
                                   tape + 2, ws, f2, true, s);
    if (st) return st;
    // stage 1: S1 = S^0 + dt L(S0); the base S^0 collects L0
    return RunAdj::run<T, PHYS, DIM>(p, state0, Y1, 1.0, tape + 6, lim ? L0 + mN : nullptr, 1.0,
                                     tape + 0, ws, fold_args<T>(lam, 0, L0, 1.0, ida), true, s);
  }
};

int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
  }
  return cus;
}

template <int V>
int tiles_of(int nx, int ny) {
  return ((nx + BatchTile<V>::TX - 1) / BatchTile<V>::TX) *
         ((ny + BatchTile<V>::TY - 1) / BatchTile<V>::TY);
}

// workgroups of a batched stage that can be resident at once
template <typename T, int V>
int batched_resident() {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_stage_batched<T, V, 1, false, MODE_CHAR>, 256, 0) !=
          hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  return per_cu * device_cus();
}

// workgroups of one batched stage launch: `blocks`, never more than the tiles, or (0)
// one per tile.  Walking the tiles instead costs the kernel registers and the
// workgroups' waits no longer overlap: 256 grids of 64..512 a side, FP32, a step by
// resident workgroups 4.68 ms, by one per tile 3.87 ms; 20 grids of 60..200, FP64, 187
// and 160 us.  (A launch holds less than 2^32 threads: past 2^22 workgroups they walk.)
int batched_grid(int blocks, int total) { return std::min(blocks <= 0 ? 1 << 22 : blocks, total); }

template <typename T, int V>
hweno_status run_batched(const hweno_problem* p, const hweno_instance* inst, const int* map, int n,
                         int total, int blocks, hipStream_t s) {
  const Consts<T> k = make_consts<T>(p);
  const int grid = batched_grid(blocks, total);
  const unsigned small = (unsigned)((n + 255) / 256);
  k_begin_batched<<<small, 256, 0, s>>>(inst, n);
  k_alpha_batched<T, V><<<std::min(total, 4 * device_cus()), 256, 0, s>>>(inst, map, total, k);
  with_mode(p, [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
    auto stages = [&](auto one) {
      constexpr bool ONE = decltype(one)::value;
      timed(s, [&] { k_stage_batched<T, V, 1, ONE, MODE><<<grid, 256, 0, s>>>(inst, map, total, p->cfl, k); });
      timed(s, [&] { k_stage_batched<T, V, 2, ONE, MODE><<<grid, 256, 0, s>>>(inst, map, total, p->cfl, k); });
      timed(s, [&] { k_stage_batched<T, V, 3, ONE, MODE><<<grid, 256, 0, s>>>(inst, map, total, p->cfl, k); });
    };
    if (grid == total)
      stages(std::true_type{});
    else
      stages(std::false_type{});
  });
  k_finish_batched<<<small, 256, 0, s>>>(inst, n);
  return launch_check("rk3_step_batched");
}

hweno_status run_batched_any(const hweno_problem* p, const hweno_instance* inst, const int* map,
                             int n, int total, int variant, int blocks, hipStream_t s) {
  if (p->dtype == HWENO_F64)
    return variant == 0 ? run_batched<double, 0>(p, inst, map, n, total, blocks, s)
                        : run_batched<double, 1>(p, inst, map, n, total, blocks, s);
  return variant == 0 ? run_batched<float, 0>(p, inst, map, n, total, blocks, s)
                      : run_batched<float, 1>(p, inst, map, n, total, blocks, s);
}

// the autotuner's grid-size candidates for one tile variant: the resident
// capacity, two and four workgroups per compute unit, one per tile
void autotune_candidates(const hweno_problem* p, int variant, int total,
                         int out[HWENO_AUTOTUNE_CANDIDATES]) {
  const int cus = device_cus();
  if (p->dtype == HWENO_F64)
    out[0] = variant == 0 ? batched_resident<double, 0>() : batched_resident<double, 1>();
  else
    out[0] = variant == 0 ? batched_resident<float, 0>() : batched_resident<float, 1>();
  out[1] = 2 * cus;
  out[2] = 4 * cus;
  out[3] = total;
}

// timing of the autotuner's steps: two events, destroyed on every path
struct EventPair {
  hipEvent_t a = nullptr, b = nullptr;
  ~EventPair() {
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
  }
};

hweno_status batch_common_ok(const hweno_problem* common) {
  if (!common) return fail(HWENO_ERR_INVALID_ARG, "problem pointer is NULL");
  if (common->dim != 2 || common->physics != HWENO_EULER)
    return fail(HWENO_ERR_UNSUPPORTED, "batched stepping is built for 2D Euler only");
  if (has_edges(common))
    return fail(HWENO_ERR_UNSUPPORTED, "batched stepping has no edge-described sides");
  hweno_problem q = *common;
  if (q.nx < 1) q.nx = 1;
  if (q.ny < 1) q.ny = 1;
  return validate(&q);
}

// device address of `scratch` on every device, looked up once per device
// with that device current (each device holds its own copy of the array)
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
void* g_scratch_fold[kMaxDevices] = {};

hweno_status static_scratch(hipStream_t s, void** out, double** fold) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(HWENO_ERR_LAUNCH, "hipGetDevice: %s", hipGetErrorString(e));
  if (s) {
    hipDevice_t sdev = -1;
    e = hipStreamGetDevice(s, &sdev);
    if (e != hipSuccess) return fail(HWENO_ERR_LAUNCH, "hipStreamGetDevice: %s", hipGetErrorString(e));
    if ((int)sdev != dev)
      return fail(HWENO_ERR_INVALID_ARG, "the stream belongs to device %d but device %d is current",
                  (int)sdev, dev);
  }
  if (dev < 0 || dev >= kMaxDevices) return fail(HWENO_ERR_UNSUPPORTED, "device index %d", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(HWENO_ERR_LAUNCH, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                  hipGetErrorString(e));
    void* slots = nullptr;
    e = hipGetSymbolAddress(&slots, HIP_SYMBOL(scratch_fold));
    if (e != hipSuccess || !slots)
      return fail(HWENO_ERR_LAUNCH, "hipGetSymbolAddress(scratch_fold) on device %d: %s", dev,
                  hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
    g_scratch_fold[dev] = slots;
  }
  *out = g_scratch_ptr[dev];
  *fold = (double*)g_scratch_fold[dev];
  return HWENO_OK;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

hweno_status hweno_validate(const hweno_problem* prob) { return validate(prob); }

size_t hweno_workspace_bytes(const hweno_problem* prob) {
  if (validate(prob) != HWENO_OK) return 0;
  return ws_layout(prob).total;
}

hweno_status hweno_alpha(const hweno_problem* prob, const void* state, double* alpha,
                         void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (empty(prob)) return ok();
  if (!state || !alpha) return fail(HWENO_ERR_INVALID_ARG, "state and alpha must be non-NULL");
  st = dispatch<RunAlpha>(prob, state, alpha, (unsigned long long*)nullptr, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_rhs(const hweno_problem* prob, const void* state, void* rhs,
                       double* alpha, int32_t compute_alpha, void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (empty(prob)) return ok();
  if (!state || !rhs || !alpha) return fail(HWENO_ERR_INVALID_ARG, "state, rhs and alpha must be non-NULL");
  if (state == rhs) return fail(HWENO_ERR_INVALID_ARG, "state and rhs must not alias");
  st = dispatch<RunRhs>(prob, state, rhs, alpha, (int)compute_alpha, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_limit(const hweno_problem* prob, const void* state, void* dlim,
                         void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (empty(prob)) return ok();
  if (!state || !dlim) return fail(HWENO_ERR_INVALID_ARG, "state and dlim must be non-NULL");
  st = dispatch<RunLimit>(prob, state, dlim, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_rk3_step(const hweno_problem* prob, void* state, void* ws, size_t ws_bytes,
                            double dt_fixed, double t_end, double* tape, const double* replay,
                            void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (empty(prob)) return ok();
  if (!state || !ws) return fail(HWENO_ERR_INVALID_ARG, "state and ws must be non-NULL");
  const size_t need = ws_layout(prob).fold;  // the slots are not required (ws_bufs)
  if (ws_bytes < need)
    return fail(HWENO_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  if (((uintptr_t)ws & 255u) != 0) return fail(HWENO_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (!std::isfinite(dt_fixed) || !std::isfinite(t_end))
    return fail(HWENO_ERR_INVALID_ARG, "dt_fixed and t_end must be finite");
  st = dispatch<RunSteps>(prob, state, ws_bufs(prob, ws, ws_bytes), 1, dt_fixed, t_end, tape, replay, true,
                          (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_rk3_steps(const hweno_problem* prob, void* state, void* ws, size_t ws_bytes,
                             int32_t n_steps, double dt_fixed, double t_end, double* tapes,
                             void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (n_steps < 0) return fail(HWENO_ERR_INVALID_ARG, "n_steps must be >= 0");
  if (empty(prob) || n_steps == 0) return ok();
  if (!state || !ws) return fail(HWENO_ERR_INVALID_ARG, "state and ws must be non-NULL");
  const size_t need = ws_layout(prob).fold;  // the slots are not required (ws_bufs)
  if (ws_bytes < need)
    return fail(HWENO_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  if (((uintptr_t)ws & 255u) != 0) return fail(HWENO_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (!std::isfinite(dt_fixed) || !std::isfinite(t_end))
    return fail(HWENO_ERR_INVALID_ARG, "dt_fixed and t_end must be finite");
  st = dispatch<RunSteps>(prob, state, ws_bufs(prob, ws, ws_bytes), (int)n_steps, dt_fixed, t_end, tapes,
                          (const double*)nullptr, true, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_rk3_step_static(const hweno_problem* prob, void* state, double* ctrl,
                                   double dt_fixed, double t_end, double* tape,
                                   const double* replay, void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (empty(prob)) return ok();
  if (!state || !ctrl) return fail(HWENO_ERR_INVALID_ARG, "state and ctrl must be non-NULL");
  if (((uintptr_t)ctrl & 7u) != 0) return fail(HWENO_ERR_INVALID_ARG, "ctrl must be 8-byte aligned");
  if (!std::isfinite(dt_fixed) || !std::isfinite(t_end))
    return fail(HWENO_ERR_INVALID_ARG, "dt_fixed and t_end must be finite");
  // the stage states and base derivatives, laid out as in a workspace but
  // without its control block
  const WsLayout L = ws_layout(prob);
  const size_t need = L.fold - L.s1;
  if (need > (size_t)HWENO_STATIC_SCRATCH_BYTES)
    return fail(HWENO_ERR_WORKSPACE,
                "grid too large for the static scratch: needs %zu bytes, the maximum is %zu",
                need, (size_t)HWENO_STATIC_SCRATCH_BYTES);
  void* base = nullptr;
  double* fold = nullptr;
  st = static_scratch((hipStream_t)stream, &base, &fold);
  if (st) return st;
  char* w = (char*)base;
  const StepBufs b{ctrl, w, w + (L.s2 - L.s1), w + (L.base - L.s1), fold, NSLOT};
  st = dispatch<RunSteps>(prob, state, b, 1, dt_fixed, t_end, tape, replay, false,
                          (hipStream_t)stream);
  if (st) return st;
  return ok();
}

size_t hweno_adjoint_workspace_bytes(const hweno_problem* prob) {
  if (validate(prob) != HWENO_OK || has_edges(prob)) return 0;
  return adj_layout(prob).total;
}

hweno_status hweno_rhs_adjoint(const hweno_problem* prob, const void* state, const double* alpha,
                               const void* lam_rhs, const void* lam_lim, void* lam_state, void* ws,
                               size_t ws_bytes, void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (has_edges(prob)) return fail(HWENO_ERR_UNSUPPORTED, "the adjoint has no edge-described sides");
  if (empty(prob)) return ok();
  if (!state || !alpha || !lam_rhs || !lam_state || !ws)
    return fail(HWENO_ERR_INVALID_ARG, "state, alpha, lam_rhs, lam_state and ws must be non-NULL");
  if (ws_bytes < adj_layout(prob).total)
    return fail(HWENO_ERR_WORKSPACE, "adjoint workspace too small: %zu < %zu bytes", ws_bytes,
                adj_layout(prob).total);
  if (((uintptr_t)ws & 255u) != 0) return fail(HWENO_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  st = dispatch<RunRhsAdj>(prob, state, alpha, lam_rhs, lam_lim, lam_state, ws, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_rk3_step_adjoint(const hweno_problem* prob, const void* state0,
                                    const void* step_ws, size_t step_ws_bytes, const double* tape,
                                    void* lam, void* ws, size_t ws_bytes, void* stream) {
  hweno_status st = validate(prob);
  if (st) return st;
  if (has_edges(prob)) return fail(HWENO_ERR_UNSUPPORTED, "the adjoint has no edge-described sides");
  if (empty(prob)) return ok();
  if (!state0 || !step_ws || !tape || !lam || !ws)
    return fail(HWENO_ERR_INVALID_ARG, "state0, step_ws, tape, lam and ws must be non-NULL");
  // the speed slots at its end are not read: a saved copy may lack them
  if (step_ws_bytes < ws_layout(prob).fold)
    return fail(HWENO_ERR_WORKSPACE, "step workspace too small");
  if (ws_bytes < adj_layout(prob).total)
    return fail(HWENO_ERR_WORKSPACE, "adjoint workspace too small: %zu < %zu bytes", ws_bytes,
                adj_layout(prob).total);
  if (((uintptr_t)ws & 255u) != 0 || ((uintptr_t)step_ws & 255u) != 0)
    return fail(HWENO_ERR_WORKSPACE, "workspaces must be 256-byte aligned");
  {
    // the stage adjoints read state0, step_ws and lam while writing lam and ws
    const size_t sb = (size_t)cells_of(prob) * elem_size(prob) * n_fields(prob);
    auto overlap = [](const void* a, size_t na, const void* b, size_t nb) {
      const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
      return x < y + nb && y < x + na;
    };
    if (overlap(lam, sb, state0, sb) || overlap(lam, sb, step_ws, step_ws_bytes) ||
        overlap(lam, sb, ws, ws_bytes) || overlap(ws, ws_bytes, state0, sb) ||
        overlap(ws, ws_bytes, step_ws, step_ws_bytes))
      return fail(HWENO_ERR_INVALID_ARG, "lam, state0, step_ws and ws must not overlap");
  }
  st = dispatch<RunStepAdj>(prob, state0, step_ws, tape, lam, ws, (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_batch_prepare(const hweno_problem* common, hweno_instance* inst,
                                 int32_t n_inst, int32_t* total_tiles) {
  hweno_status st = batch_common_ok(common);
  if (st) return st;
  if (!inst || !total_tiles || n_inst < 1)
    return fail(HWENO_ERR_INVALID_ARG, "inst, total_tiles must be non-NULL and n_inst >= 1");
  long long tot[HWENO_BATCH_VARIANTS] = {0, 0};
  for (int q = 0; q < n_inst; ++q) {
    hweno_instance& I = inst[q];
    hweno_problem p = *common;
    p.nx = I.nx;
    p.ny = I.ny;
    p.bc_x = I.bc_x;
    p.bc_y = I.bc_y;
    p.dx = I.dx;
    p.dy = I.dy;
    if (has_edges(&p))
      return fail(HWENO_ERR_UNSUPPORTED, "instance %d: batched stepping has no edge-described sides", q);
    st = validate(&p);
    if (st) return fail(st, "instance %d: %s", q, g_last_error.c_str());
    if (I.nx < 1 || I.ny < 1) return fail(HWENO_ERR_INVALID_ARG, "instance %d: nx, ny must be >= 1", q);
    if (!std::isfinite(I.dt_fixed) || !std::isfinite(I.t_end))
      return fail(HWENO_ERR_INVALID_ARG, "instance %d: dt_fixed, t_end must be finite", q);
    const WsLayout L = ws_layout(&p);
    I.ws_bytes = (int64_t)L.fold;  // a batch folds its speeds into the control blocks
    I.off_s1 = (int64_t)L.s1;
    I.off_s2 = (int64_t)L.s2;
    I.off_base = (int64_t)L.base;
    const int nt[HWENO_BATCH_VARIANTS] = {tiles_of<0>(I.nx, I.ny), tiles_of<1>(I.nx, I.ny)};
    for (int v = 0; v < HWENO_BATCH_VARIANTS; ++v) {
      I.tile_begin[v] = (int32_t)tot[v];
      I.n_tiles[v] = nt[v];
      tot[v] += nt[v];
      if (tot[v] > (1ll << 30)) return fail(HWENO_ERR_INVALID_ARG, "too many tiles");
    }
  }
  for (int v = 0; v < HWENO_BATCH_VARIANTS; ++v) total_tiles[v] = (int32_t)tot[v];
  return ok();
}

hweno_status hweno_batch_tile_map(const hweno_instance* inst, int32_t n_inst, int32_t variant,
                                  int32_t* map, int32_t total_tiles) {
  if (!inst || !map || n_inst < 1 || variant < 0 || variant >= HWENO_BATCH_VARIANTS)
    return fail(HWENO_ERR_INVALID_ARG, "inst, map must be non-NULL, n_inst >= 1, variant valid");
  long long filled = 0;
  for (int q = 0; q < n_inst; ++q) {
    const int b = inst[q].tile_begin[variant], n = inst[q].n_tiles[variant];
    if (b != filled || n < 1 || (long long)b + n > total_tiles)
      return fail(HWENO_ERR_INVALID_ARG, "instance %d: descriptors not prepared for %d tiles", q,
                  total_tiles);
    for (int t = 0; t < n; ++t) map[b + t] = q;
    filled += n;
  }
  if (filled != total_tiles) return fail(HWENO_ERR_INVALID_ARG, "tile count mismatch");
  return ok();
}

hweno_status hweno_rk3_step_batched(const hweno_problem* common, const hweno_instance* inst_dev,
                                    const int32_t* tile_map_dev, int32_t n_inst,
                                    int32_t total_tiles, int32_t variant, int32_t blocks,
                                    void* stream) {
  hweno_status st = batch_common_ok(common);
  if (st) return st;
  if (!inst_dev || !tile_map_dev || n_inst < 1 || total_tiles < n_inst)
    return fail(HWENO_ERR_INVALID_ARG,
                "inst_dev, tile_map_dev must be non-NULL, n_inst >= 1, total_tiles >= n_inst");
  if (variant < 0 || variant >= HWENO_BATCH_VARIANTS)
    return fail(HWENO_ERR_INVALID_ARG, "variant must be in [0, %d)", HWENO_BATCH_VARIANTS);
  if (blocks < 0) return fail(HWENO_ERR_INVALID_ARG, "blocks must be >= 0");
  st = run_batched_any(common, inst_dev, tile_map_dev, n_inst, total_tiles, variant, blocks,
                       (hipStream_t)stream);
  if (st) return st;
  return ok();
}

hweno_status hweno_autotune(const hweno_problem* common, const hweno_instance* inst_dev,
                            const int32_t* const* tile_maps_dev, int32_t n_inst,
                            const int32_t* total_tiles, int32_t trials, void* stream,
                            int32_t* variant, int32_t* blocks, double* times_ms,
                            int32_t* grid_sizes) {
  hweno_status st = batch_common_ok(common);
  if (st) return st;
  if (!inst_dev || !tile_maps_dev || !total_tiles || !variant || !blocks || n_inst < 1)
    return fail(HWENO_ERR_INVALID_ARG,
                "inst_dev, tile_maps_dev, total_tiles, variant, blocks must be non-NULL, n_inst >= 1");
  if (trials < 1 || trials > 1000) return fail(HWENO_ERR_INVALID_ARG, "trials must be in [1, 1000]");
  for (int v = 0; v < HWENO_BATCH_VARIANTS; ++v) {
    if (!tile_maps_dev[v]) return fail(HWENO_ERR_INVALID_ARG, "tile map of variant %d is NULL", v);
    if (total_tiles[v] < n_inst)
      return fail(HWENO_ERR_INVALID_ARG, "variant %d: total_tiles must be >= n_inst", v);
  }
  hipStream_t s = (hipStream_t)stream;
  // the diagnostic stage timer must not see the autotuner's launches
  const bool timing_was_on = g_timing.on;
  g_timing.on = false;
  struct Restore {
    bool on;
    ~Restore() { g_timing.on = on; }
  } restore{timing_was_on};
  EventPair ev;
  hipError_t e = hipEventCreate(&ev.a);
  if (e == hipSuccess) e = hipEventCreate(&ev.b);
  if (e != hipSuccess) return fail(HWENO_ERR_LAUNCH, "hipEventCreate: %s", hipGetErrorString(e));
  double best = 0.0;
  int best_v = -1, best_b = 0;
  for (int v = 0; v < HWENO_BATCH_VARIANTS; ++v) {
    int cand[HWENO_AUTOTUNE_CANDIDATES];
    autotune_candidates(common, v, total_tiles[v], cand);
    for (int c = 0; c < HWENO_AUTOTUNE_CANDIDATES; ++c) {
      const int b = cand[c];
      // one warm-up step, then `trials` timed steps between two events
      st = run_batched_any(common, inst_dev, tile_maps_dev[v], n_inst, total_tiles[v], v, b, s);
      if (st) return st;
      if ((e = hipEventRecord(ev.a, s)) != hipSuccess)
        return fail(HWENO_ERR_LAUNCH, "hipEventRecord: %s", hipGetErrorString(e));
      for (int q = 0; q < trials; ++q) {
        st = run_batched_any(common, inst_dev, tile_maps_dev[v], n_inst, total_tiles[v], v, b, s);
        if (st) return st;
      }
      if ((e = hipEventRecord(ev.b, s)) != hipSuccess ||
          (e = hipEventSynchronize(ev.b)) != hipSuccess)
        return fail(HWENO_ERR_LAUNCH, "event: %s", hipGetErrorString(e));
      float ms = 0.f;
      if ((e = hipEventElapsedTime(&ms, ev.a, ev.b)) != hipSuccess)
        return fail(HWENO_ERR_LAUNCH, "hipEventElapsedTime: %s", hipGetErrorString(e));
      const double per = (double)ms / trials;
      const int k = v * HWENO_AUTOTUNE_CANDIDATES + c;
      if (times_ms) times_ms[k] = per;
      if (grid_sizes) grid_sizes[k] = batched_grid(b, total_tiles[v]);
      if (best_v < 0 || per < best) {
        best = per;
        best_v = v;
        best_b = b;
      }
    }
  }
  *variant = best_v;
  // the grid size itself, which launches the same kernels as the candidate when
  // passed back as `blocks`
  *blocks = batched_grid(best_b, total_tiles[best_v]);
  return ok();
}

hweno_status hweno_timing_begin(int32_t enable) {
  timing_release();
  g_timing.on = enable != 0;
  return ok();
}

hweno_status hweno_timing_end(int64_t* launches, double* total_ms) {
  double tot = 0.0;
  for (size_t q = 0; q < g_timing.used; ++q) {
    if (hipEventSynchronize(g_timing.ev[q].second) != hipSuccess) {
      timing_release();
      return fail(HWENO_ERR_LAUNCH, "event synchronisation failed");
    }
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, g_timing.ev[q].first, g_timing.ev[q].second) != hipSuccess) {
      timing_release();
      return fail(HWENO_ERR_LAUNCH, "event timing failed");
    }
    tot += ms;
  }
  if (launches) *launches = (int64_t)g_timing.used;
  if (total_ms) *total_ms = tot;
  timing_release();
  return ok();
}

const char* hweno_status_string(int32_t s) {
  switch (s) {
    case HWENO_OK: return "HWENO_OK";
    case HWENO_ERR_INVALID_ARG: return "HWENO_ERR_INVALID_ARG";
    case HWENO_ERR_UNSUPPORTED: return "HWENO_ERR_UNSUPPORTED";
    case HWENO_ERR_WORKSPACE: return "HWENO_ERR_WORKSPACE";
    case HWENO_ERR_LAUNCH: return "HWENO_ERR_LAUNCH";
    default: return "HWENO_ERR_UNKNOWN";
  }
}

const char* hweno_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
