// Fused pull-stream / boundary / wall-model / MRT-Smagorinsky collision
// kernel for the D3Q19 channel (Algorithm 1 of Xue, Yao, Davidson,
// arXiv 2304.04214), plus the initialisation, import/export, stream-only and
// copy kernels.
//
// Population layout: 64-node bricks.  The 19 populations of the 64 nodes
// (x, y, 64 zc .. 64 zc + 63) are one contiguous block of 19 x 64 elements,
// and bricks are ordered (x, zc, y): element (i, x, y, z) sits at
// ((x zc_n + z/64) ny + y) 1216 + 64 i + z%64.  A wave (64 lanes) owns one
// brick: its 19 stores are one contiguous 4864-byte (float) run, and its pulls
// come from the 3 x 3 neighbouring (x, y) bricks plus one element of the
// z-neighbouring bricks for the +-1 z shifts.
//
// Mapping: one thread per node.  A block is 4 consecutive y rows (4 waves) of
// one (x, z-chunk).  x and y are wave-uniform (scalar registers), so every
// boundary decision is a scalar select and each population load is
// scalar base + per-lane column offset.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "collide.h"
#include "internal.h"
#include "stream.h"



namespace lbm {
namespace {

// Node of the calling thread: block = 4 consecutive y rows of one (x, z-chunk),
// blocks ordered like the bricks (y-groups fastest, then z-chunks, then x).
struct Node {
  int x, y, zci, base, gy, lane, z;
  bool owned, active;
};
__device__ __forceinline__ Node decode(const CollideArgs& a) {
  Node n;
  const int L = blockIdx.x;
  n.gy = L % a.yg;
  const int rest = L / a.yg;
  n.zci = rest % a.zc;
  n.x = rest / a.zc;
  n.lane = threadIdx.x & (ZT - 1);
  n.base = min(YROWS * n.gy, a.ny - YROWS);
  n.y = n.base + uni(threadIdx.x >> 6);
  n.owned = n.y >= YROWS * n.gy;  // rows shared with the previous group (ragged ny) are helpers only
  const int zraw = n.zci * ZT + n.lane;
  n.active = zraw < a.nz;
  n.z = n.active ? zraw : a.nz - 1;  // inactive lanes compute a valid node and store nothing
  return n;
}

// Boundary rules, wall model, collision, store and statistics of one node
// whose pulled populations are in f (Algorithm 1 for one cell).
// The outlet and inlet rules of an open channel on the pulled populations f
// of node (x, y, z); store: write the outlet history of the step.
template <bool F16>
__device__ __forceinline__ void x_rules(const CollideArgs& a, int x, int y, int z, const Col& col, float f[Q],
                                        bool store) {
  const bool inflow = a.xbc == LBM_X_INFLOW;
  if (inflow && x == a.nx - 1) {  // convective outlet for c_x < 0
    const Geo g2 = make_geo(a, x - 1, y);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const int i = OUT5[k];
      const float up = pull_dir<F16>(a, g2, i, col, 0.f);
      const int hidx = (k * a.ny + y) * a.nz + z;
      const float v = outlet_value(a, a.hist_in[hidx], up);
      f[i] = v;
      if (store) a.hist_out[hidx] = v;
    }
  }
  if (inflow && x == 0) inlet_regularize(a, y, z, f);
}

// NT: non-temporal population stores (see CollideArgs::nt_store).
// LATE: the storage offsets are loaded with their stores, not ahead of them.
template <bool F16, bool NT = true, int ZL = ZT, bool LATE = true>
__device__ __forceinline__ void node_update(const CollideArgs& a, int x, int y, int z, int lane, int base, int zci,
                                            bool owned, bool active, const Col& col, float f[Q],
                                            float (*lds_u2)[2][ZL]) {
  x_rules<F16>(a, x, y, z, col, f, active && owned);

  // density and momentum before the force (Eq. (10)-(11)), summed directly
  // so that the collision's pair sums are not live across the wall force
  float rho = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    rho += f[i];
    if (CX[i]) jx += CX[i] * f[i];
    if (CY[i]) jy += CY[i] * f[i];
    if (CZ[i]) jz += CZ[i] * f[i];
  }

  float Fx = 0.f, Fy = 0.f, Fz = 0.f;
  bool force = a.has_g != 0;
  if (force) {
    Fx = rho * a.g[0];
    Fy = rho * a.g[1];
    Fz = rho * a.g[2];
  }
  if (a.wall_model) {
    const bool bot = base == 0, top = base == a.ny - YROWS;
    if (bot || top) {  // block-uniform: the block holds a wall row and its neighbour
      const float ir = 1.f / rho;
      if (bot && y == 1) {
        lds_u2[0][0][lane] = jx * ir;
        lds_u2[0][1][lane] = jz * ir;
      }
      if (top && y == a.ny - 2) {
        lds_u2[1][0][lane] = jx * ir;
        lds_u2[1][1][lane] = jz * ir;
      }
      __syncthreads();
      const bool wb = bot && y == 0, wt = top && y == a.ny - 1;
      if (wb || wt) {
        const int w = wb ? 0 : 1;
        float fwx, fwz, ut;
        wall_force(a, rho, jx * ir, jz * ir, lds_u2[w][0][lane], lds_u2[w][1][lane], fwx, fwz, ut, w, x);
        Fx += fwx;
        Fz += fwz;
        force = true;
        if (a.wall_acc) {  // wall statistics: sum over the wave's z of u_tau (FP64, one writer per slot)
          double v = active ? (double)ut : 0.0;
#pragma unroll
          for (int off = ZL / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, ZT);
          if (lane == 0) a.wall_acc[((size_t)w * a.nx + x) * a.zc + zci] += v;
        }
      }
    }
  }

  float ux, uy, uz;
  const Tau0 t0 = tau0_of_x(a, x);
  const Pairs pr = make_pairs(f);
  if (force)
    collide<true>(a, t0, f, pr, rho, jx, jy, jz, Fx, Fy, Fz, ux, uy, uz);
  else
    collide<false>(a, t0, f, pr, rho, jx, jy, jz, 0.f, 0.f, 0.f, ux, uy, uz);

  if (!(rho > 0.f && rho < 1e30f)) atomicOr(a.err, ERRBIT_NONFINITE);

  if (active && owned) {
    char* p = const_cast<char*>(row_ptr<F16>(a.dst, rowpart(a, x, y)));
    // The offsets are loaded before the first store: between stores each load would wait for its own
    // (us per six steps 48x64x64 81.7 -> 77.0, 16x90x100 85.0 -> 80.3).  On lattices beyond the caches,
    // where other waves fill that wait, 64-lane rows keep theirs with the stores (914x90x100, twelve
    // sampled planes, four steps 723, ahead 737).
    float ref[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) ref[i] = F16 && !LATE ? ref_off(a, i, y) : 0.f;
#pragma unroll
    for (int i = 0; i < Q; ++i)
      Pop<F16>::template stp<NT>(p + i * ZT * Pop<F16>::ES, i, col.b0, f[i], LATE ? ref_off(a, i, y) : ref[i]);
  }

  if (a.stats_on) {
    const int p = a.plane_of_x[x];
    if (p >= 0 && owned) {
      const bool on = active;
      double v[9];
      const double dx = ux, dy = uy, dz = uz;
      v[0] = on ? dx : 0.0;
      v[1] = on ? dy : 0.0;
      v[2] = on ? dz : 0.0;
      v[3] = on ? dx * dx : 0.0;
      v[4] = on ? dy * dy : 0.0;
      v[5] = on ? dz * dz : 0.0;
      v[6] = on ? dx * dy : 0.0;
      v[7] = on ? dx * dz : 0.0;
      v[8] = on ? dy * dz : 0.0;
#pragma unroll
      for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int off = ZL / 2; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, ZT);
      if (lane == 0) {
        double* s = a.stats + (((size_t)p * a.ny + y) * a.zc + zci) * 9;
#pragma unroll
        for (int k = 0; k < 9; ++k) s[k] += v[k];
      }
    }
  }
}

// With FP16 storage the collide-stream step runs as two kernels over
// disjoint block sets (a block = 4 consecutive y rows of one (x, z-chunk)):
//  * bulk blocks (every block away from the inlet, outlet and statistics
//    planes): interior blocks, whose 3 x 3 source rows all lie inside the
//    lattice, and the y-groups holding a wall row, in one lean kernel that
//    keeps few registers and many waves in flight to hide HBM latency;
//  * boundary blocks (inlet and outlet planes, sampled statistics planes):
//    the general kernel with every rule of Algorithm 1.
// On lattices up to FUSED_MAX_NODES the two lists run as one launch
// (collide_fused_kernel).  With FP32 storage the general kernel takes every
// block.  All read s_n and write disjoint nodes of s_{n+1}.  Each walks a
// block list (columns (x, y-group) dealt to the XCDs by xcd_order).

// Row of the calling thread in its block: rows of ZL lanes (64: one wave a row,
// a scalar).
template <int ZL>
__device__ __forceinline__ int row_of_thread() {
  return ZL == ZT ? uni(threadIdx.x >> 6) : (int)threadIdx.x / ZL;
}

// Storage offsets of the block's rows and one beyond each side, by short rows
// (ZL < 64) from LDS: loaded before the pulls go out, stored behind them, so
// that no pull waits for them.
template <int ZL>
struct RowRef {
  static constexpr int N = (YROWS + 2) * Q, PER = (N + YROWS * ZL - 1) / (YROWS * ZL);
  float v[PER];
  __device__ __forceinline__ void load(const CollideArgs& a, const float* __restrict__ dref, int base) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int k = min((int)threadIdx.x + j * YROWS * ZL, N - 1), q = k / Q;
      int y = base - 1 + q;
      y = y < 0 ? y + a.ny : (y >= a.ny ? y - a.ny : y);
      v[j] = dref[y * Q + (k - q * Q)];
    }
  }
  __device__ __forceinline__ void store(float* lref) const {
#pragma unroll
    for (int j = 0; j < PER; ++j) lref[min((int)threadIdx.x + j * YROWS * ZL, N - 1)] = v[j];
    __syncthreads();
  }
};

// FP16 storage: a block whose 3 x 3 source rows all lie inside the lattice (see
// the block lists): plain shifted pulls, no boundary rule.
// dref / dpull: the reference offsets (REF), passed as restrict kernel
// arguments so that their loads need not be ordered after the stores.
// ZL < 64: lref takes the offsets (RowRef).
template <bool FORCE, bool REF, bool NT = true, int ZL = ZT>
__device__ __forceinline__ void plain_block(const CollideArgs& a, int x, int zci, int gy,
                                            const float* __restrict__ dref, const float* __restrict__ dpull,
                                            float* lref = nullptr) {
  const int lane = threadIdx.x & (ZL - 1);
  const int base = min(YROWS * gy, a.ny - YROWS);
  const int w = row_of_thread<ZL>(), y = base + w;
  const bool owned = y >= YROWS * gy;
  const int zraw = zci * ZT + lane;
  const bool active = zraw < a.nz;
  const int z = active ? zraw : a.nz - 1;
  const Col col = make_col<true>(a, z);
  const Geo g = make_geo(a, x, y);
  RowRef<ZL> rr;
  if (REF && ZL < ZT) rr.load(a, dref, base);
  Pop<true>::Raw r[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const uint32_t cs = CZ[i] == 1 ? col.bm : (CZ[i] == -1 ? col.bp : col.b0);
    r[i] = Pop<true>::raw(row_ptr<true>(a.src, rowpart(a, g.xs[CX[i] + 1], g.ys[CY[i] + 1]) + (uint32_t)i * ZT), cs);
  }
  if (REF && ZL < ZT) rr.store(lref);
  // on the deviations h = f - w directly (no w added on load or subtracted on store)
  float f[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    if (REF)
      f[i] = Pop<true>::cvt_dev(r[i], ZL < ZT ? lref[(w + 1 - CY[i]) * Q + i] : dpull[y * Q + i]);  // uniform row: scalar loads
    else
      f[i] = Pop<true>::cvt_dev(r[i]);
  }
  const Pairs pr = make_pairs(f);
  const float rhoh = pr.A + pr.Bx + f[9], rho = 1.f + rhoh;
  const float jx = (pr.d[3] + pr.d[7]) - (pr.d[1] + pr.d[5] + pr.d[8]);
  const float jy = pr.d[4] - (pr.d[0] + pr.d[5] + pr.d[6] + pr.d[7]);
  const float jz = -(pr.d[0] + pr.d[1] + pr.d[2] + pr.d[3] + pr.d[4]);
  float ux, uy, uz;
  const Tau0 t0 = tau0_of_x(a, x);
  if (FORCE)
    collide<true, true>(a, t0, f, pr, rho, jx, jy, jz, rho * a.g[0], rho * a.g[1], rho * a.g[2], ux, uy, uz, rhoh);
  else
    collide<false, true>(a, t0, f, pr, rho, jx, jy, jz, 0.f, 0.f, 0.f, ux, uy, uz, rhoh);
  if (!(rho > 0.f && rho < 1e30f)) atomicOr(a.err, ERRBIT_NONFINITE);
  if (active && owned) {
    char* p = const_cast<char*>(row_ptr<true>(a.dst, rowpart(a, x, y)));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (REF)
        Pop<true>::stp_dev<NT>(p + i * ZT * Pop<true>::ES, col.b0, f[i], ZL < ZT ? lref[(w + 1) * Q + i] : dref[y * Q + i]);
      else
        Pop<true>::stp_dev<NT>(p + i * ZT * Pop<true>::ES, col.b0, f[i]);
    }
  }
}

// A y-group holding a wall row, away from the inlet, outlet and statistics
// planes: the plain block's data flow plus the wall rules of the pull and
// the wall model (the wall row's neighbour velocity through LDS).  Density
// and momentum are summed directly so that the pair sums of the collision
// are not live across the Newton solve (fewer registers).
template <bool REF, bool NT = true, int ZL = ZT>
__device__ __forceinline__ void wall_block(const CollideArgs& a, int x, int zci, int gy, float (*lds_u2)[2][ZL],
                                           const float* __restrict__ dref, float* lref = nullptr) {
  const int lane = threadIdx.x & (ZL - 1);
  const int base = min(YROWS * gy, a.ny - YROWS);
  const int w = row_of_thread<ZL>(), y = base + w;
  const bool owned = y >= YROWS * gy;
  const int zraw = zci * ZT + lane;
  const bool active = zraw < a.nz;
  const int z = active ? zraw : a.nz - 1;
  const Col col = make_col<true>(a, z);
  const Geo g = make_geo(a, x, y);
  RowRef<ZL> rr;
  if (REF && ZL < ZT) rr.load(a, dref, base);
  Pop<true>::Raw r[Q];
  issue_pulls<true, ZL == ZT>(a, g, col, r);  // every x source exists; the y walls redirect
  if (REF && ZL < ZT) rr.store(lref);
  float f[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    if (REF && ZL < ZT) {
      int plane, ysrc;
      pull_plane_row(a, g, i, plane, ysrc);
      f[i] = Pop<true>::cvt_dev(r[i], lref[(CY[i] != 0 && g.yout[CY[i] + 1] ? w + 1 : w + 1 - CY[i]) * Q + plane]);
    } else if (REF)
      f[i] = Pop<true>::cvt_dev(r[i], pull_ref(a, g, i));
    else
      f[i] = Pop<true>::cvt_dev(r[i]);
  }
  // density and momentum first; the pair sums of the collision are formed
  // after the wall force, so they are not live across the Newton solve
  float rhoh = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    rhoh += f[i];
    if (CX[i]) jx += CX[i] * f[i];
    if (CY[i]) jy += CY[i] * f[i];
    if (CZ[i]) jz += CZ[i] * f[i];
  }
  const float rho = 1.f + rhoh;
  float Fx = rho * a.g[0], Fy = rho * a.g[1], Fz = rho * a.g[2];
  if (a.wall_model) {
    const bool bot = base == 0, top = base == a.ny - YROWS;
    const float ir = 1.f / rho;
    if (bot && y == 1) {
      lds_u2[0][0][lane] = jx * ir;
      lds_u2[0][1][lane] = jz * ir;
    }
    if (top && y == a.ny - 2) {
      lds_u2[1][0][lane] = jx * ir;
      lds_u2[1][1][lane] = jz * ir;
    }
    __syncthreads();
    const bool wb = bot && y == 0, wt = top && y == a.ny - 1;
    if (wb || wt) {
      const int wl = wb ? 0 : 1;
      float fwx, fwz, ut;
      wall_force(a, rho, jx * ir, jz * ir, lds_u2[wl][0][lane], lds_u2[wl][1][lane], fwx, fwz, ut, wl, x);
      Fx += fwx;
      Fz += fwz;
      if (a.wall_acc) {
        double v = active ? (double)ut : 0.0;
#pragma unroll
        for (int off = ZL / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, ZT);
        if (lane == 0) a.wall_acc[((size_t)wl * a.nx + x) * a.zc + zci] += v;
      }
    }
  }
  float ux, uy, uz;
  const Pairs pr = make_pairs(f);
  collide<true, true>(a, tau0_of_x(a, x), f, pr, rho, jx, jy, jz, Fx, Fy, Fz, ux, uy, uz, rhoh);
  if (!(rho > 0.f && rho < 1e30f)) atomicOr(a.err, ERRBIT_NONFINITE);
  if (active && owned) {
    char* p = const_cast<char*>(row_ptr<true>(a.dst, rowpart(a, x, y)));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (REF)
        Pop<true>::stp_dev<NT>(p + i * ZT * Pop<true>::ES, col.b0, f[i], ZL < ZT ? lref[(w + 1) * Q + i] : dref[y * Q + i]);
      else
        Pop<true>::stp_dev<NT>(p + i * ZT * Pop<true>::ES, col.b0, f[i]);
    }
  }
}

// Interior and wall blocks (block-uniform choice): the lean kernel, so it
// keeps few registers and many waves in flight to hide HBM latency.
template <bool FORCE, bool REF>
__global__ __launch_bounds__(BLOCK) void collide_bulk_kernel(CollideArgs a, const int* __restrict__ blist,
                                                             const float* __restrict__ dref,
                                                             const float* __restrict__ dpull) {
  __shared__ float lds_u2[2][2][ZT];
  const int e = blist[blockIdx.x];
  if (e < 0) return;  // padding of the XCD-ordered list (whole block: no barrier is skipped by part of it)
  int x, zci, gy;
  block_coords(a, e, x, zci, gy);
  const int base = min(YROWS * gy, a.ny - YROWS);
  if (a.ywall != LBM_Y_PERIODIC && (base == 0 || base == a.ny - YROWS))
    wall_block<REF>(a, x, zci, gy, lds_u2, dref);
  else
    plain_block<FORCE, REF>(a, x, zci, gy, dref, dpull);
}

template <bool F16, bool NT = true>
__global__ __launch_bounds__(BLOCK) void collide_general_kernel(CollideArgs a, const int* __restrict__ blist) {
  __shared__ float lds_u2[2][2][ZT];
  const int e = blist[blockIdx.x];
  if (e < 0) return;  // padding of the XCD-ordered list (whole block: no barrier is skipped by part of it)
  int x, zci, gy;
  block_coords(a, e, x, zci, gy);
  const int lane = threadIdx.x & (ZT - 1);
  const int base = min(YROWS * gy, a.ny - YROWS);
  const int y = base + uni(threadIdx.x >> 6);
  const bool owned = y >= YROWS * gy;  // rows shared with the previous group (ragged ny) are helpers only
  const int zraw = zci * ZT + lane;
  const bool active = zraw < a.nz;
  const int z = active ? zraw : a.nz - 1;  // inactive lanes compute a valid node and store nothing
  const Col col = make_col<F16>(a, z);
  const Geo g = make_geo(a, x, y);
  typename Pop<F16>::Raw r[Q];
  issue_pulls<F16>(a, g, col, r);
  float f[Q];
  convert_pulls<F16>(a, g, r, f);
  node_update<F16, NT>(a, x, y, z, lane, base, zci, owned, active, col, f, lds_u2);
}

// Waves per SIMD that the fused kernel with short rows is held to: 71 VGPRs
// without spills.  At eight, as with 64-lane rows, it spills and loses what the
// short rows give (400x40x32: 20.6 us per step at six, 26.3 at eight).
constexpr int FUSED_SHORT_WAVES = 6;

// FP16 storage on lattices up to FUSED_MAX_NODES: both block lists in one
// launch, the general blocks (gl, n_gen entries) first so that their longer
// work overlaps the bulk blocks (bl).  Held to 64 VGPRs (8 waves per SIMD, as
// the bulk kernel; the general path spills a few).  A separate general launch
// costs a fixed ~10 us (its blocks run alone as a latency-bound wave), more
// than the fused kernel's slower bulk path on small lattices, less on large.
//
// ZL: lanes of a row (row_lanes).  Lattices of at most 32 (16) spanwise nodes
// give a row 32 (16) lanes, so that a wave holds two (four) rows of the block's
// four and fewer lanes are without a node.  us per step with 64 lanes -> with these:
// 400x40x32 24.1 -> 20.6, 64x32x32 9.9 -> 7.6, 600x60x24 32.2 -> 28.7,
// 200x20x16 13.4 -> 10.3.
template <bool FORCE, bool REF, bool NT, int ZL, bool LATE = false>
__global__ __launch_bounds__(YROWS* ZL) __attribute__((amdgpu_waves_per_eu(ZL == ZT ? 8 : FUSED_SHORT_WAVES)))
void collide_fused_kernel(CollideArgs a, const int* __restrict__ gl, int n_gen, const int* __restrict__ bl,
                          const float* __restrict__ dref, const float* __restrict__ dpull) {
  __shared__ float lds_u2[2][2][ZL];
  const int b = (int)blockIdx.x;
  if (b < n_gen) {  // a general block (block-uniform)
    const int e = gl[b];
    if (e < 0) return;  // padding of the XCD-ordered list (whole block)
    int x, zci, gy;
    block_coords(a, e, x, zci, gy);
    const int lane = threadIdx.x & (ZL - 1);
    const int base = min(YROWS * gy, a.ny - YROWS);
    const int y = base + row_of_thread<ZL>();
    const bool owned = y >= YROWS * gy;
    const int zraw = zci * ZT + lane;
    const bool active = zraw < a.nz;
    const int z = active ? zraw : a.nz - 1;
    const Col col = make_col<true>(a, z);
    const Geo g = make_geo(a, x, y);
    Pop<true>::Raw r[Q];
    issue_pulls<true, ZL == ZT>(a, g, col, r);
    float f[Q];
    convert_pulls<true, ZL == ZT>(a, g, r, f);
    node_update<true, NT, ZL, LATE>(a, x, y, z, lane, base, zci, owned, active, col, f, lds_u2);
    return;
  }
  const int e = bl[b - n_gen];
  if (e < 0) return;
  int x, zci, gy;
  block_coords(a, e, x, zci, gy);
  const int base = min(YROWS * gy, a.ny - YROWS);
  __shared__ float lref[REF && ZL < ZT ? RowRef<ZL>::N : 1];
  if (a.ywall != LBM_Y_PERIODIC && (base == 0 || base == a.ny - YROWS))
    wall_block<REF, NT, ZL>(a, x, zci, gy, lds_u2, dref, lref);
  else
    plain_block<FORCE, REF, NT, ZL>(a, x, zci, gy, dref, dpull, lref);
}

// Pre-force velocity (u_x, u_z) of node (x, y, z) after streaming and the
// boundary rules, as node_update forms it.
template <bool F16>
__device__ __forceinline__ void pre_force_uxz(const CollideArgs& a, int x, int y, int z, const Col& col, float& ux,
                                              float& uz) {
  const Geo g = make_geo(a, x, y);
  typename Pop<F16>::Raw r[Q];
  issue_pulls<F16>(a, g, col, r);
  float f[Q];
  convert_pulls<F16>(a, g, r, f);
  x_rules<F16>(a, x, y, z, col, f, false);
  const Pairs pr = make_pairs(f);
  const float rho = pr.A + pr.Bx + f[9];
  const float jx = (pr.d[3] + pr.d[7]) - (pr.d[1] + pr.d[5] + pr.d[8]);
  const float jz = -(pr.d[0] + pr.d[1] + pr.d[2] + pr.d[3] + pr.d[4]);
  const float ir = 1.f / rho;
  ux = jx * ir;
  uz = jz * ir;
}

// Line-averaged wall model: one block per wall line (x, wall).  Its four
// waves sum u_hat = u_w . e_x (Eq. (19), 0 where u_2 has no tangential part)
// over z in FP64 in a fixed order; the line's u_tau solves Eq. (20) for the
// mean's magnitude and is stored with the mean's sign.
template <bool F16>
__global__ __launch_bounds__(BLOCK) void wall_line_kernel(CollideArgs a, float* line) {
  __shared__ double part[BLOCK / ZT];
  const int x = blockIdx.x, w = blockIdx.y;
  const int yw = w ? a.ny - 1 : 0, y2 = w ? a.ny - 2 : 1;
  const int lane = threadIdx.x & (ZT - 1), wave = uni(threadIdx.x >> 6);
  double acc = 0.0;
  for (int zci = wave; zci < a.zc; zci += BLOCK / ZT) {
    const int zraw = zci * ZT + lane;
    const bool active = zraw < a.nz;
    const int z = active ? zraw : a.nz - 1;
    const Col col = make_col<F16>(a, z);
    float uwx, uwz, u2x, u2z;
    pre_force_uxz<F16>(a, x, yw, z, col, uwx, uwz);
    pre_force_uxz<F16>(a, x, y2, z, col, u2x, u2z);
    const float tn2 = u2x * u2x + u2z * u2z;
    float uh = 0.f;
    if (tn2 > 0.f) {
      const float itn = 1.f / sqrtf(tn2);
      uh = uwx * (u2x * itn) + uwz * (u2z * itn);
    }
    acc += active ? (double)uh : 0.0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, ZT);
  if (lane == 0) part[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < BLOCK / ZT; ++k) s += part[k];
    const float ub = (float)(s / a.nz);
    const float ut = ub != 0.f ? newton_utau(a, fabsf(ub)) : 0.f;
    line[w * a.nx + x] = ub > 0.f ? ut : -ut;
  }
}

// Pull with the wall rules only (debug map); unset populations are -1.
__global__ __launch_bounds__(BLOCK) void stream_only_kernel(CollideArgs a) {
  const Node nd = decode(a);
  if (!nd.active || !nd.owned) return;
  const Col col = make_col<false>(a, nd.z);
  const Geo g = make_geo(a, nd.x, nd.y);
  const uint32_t row = rowpart(a, nd.x, nd.y);
#pragma unroll
  for (int i = 0; i < Q; ++i) Pop<false>::st_plain(a.dst, i, row + (uint32_t)i * ZT + col.c0, pull_dir<false>(a, g, i, col, -1.f), 0.f);
}

// f_i = f_eq_i(rho, u) + eps w_i pert_i from SoA node fields [.][N], N = (x ny + y) nz + z,
// in the precision T of the inputs (float or double), rounded once to the
// storage: FP32 populations, or with FP16 storage the deviation f - w - r
// formed in T.
template <bool F16, typename T>
__global__ __launch_bounds__(BLOCK) void init_kernel(CollideArgs a, float* hist, const T* rho, const T* u,
                                                     const T* pert, T eps) {
  const Node nd = decode(a);
  if (!nd.active || !nd.owned) return;
  const int N = a.nx * a.ny * a.nz;
  const int n = (nd.x * a.ny + nd.y) * a.nz + nd.z;
  const T r = rho ? rho[n] : T(1);
  const T ux = u[n], uy = u[N + n], uz = u[2 * N + n];
  const T uu15 = T(1.5) * (ux * ux + uy * uy + uz * uz);
  const uint32_t e0 = rowpart(a, nd.x, nd.y) + colpart(a, nd.z);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const T cu = CX[i] * ux + CY[i] * uy + CZ[i] * uz;
    T v = (T)WD[i] * r * (T(1) + T(3) * cu + T(4.5) * cu * cu - uu15);
    if (pert) v += eps * (T)WD[i] * pert[(size_t)i * N + n];
    const float ref = ref_off(a, i, nd.y);
    if (F16 && sizeof(T) == 8)
      static_cast<_Float16*>(a.dst)[e0 + (uint32_t)i * ZT] = (_Float16)(float)((v - WD[i]) - (T)ref);
    else
      Pop<F16>::st_plain(a.dst, i, e0 + (uint32_t)i * ZT, (float)v, ref);
    if (hist && nd.x == a.nx - 1) {
#pragma unroll
      for (int k = 0; k < 5; ++k)
        if (OUT5[k] == i) hist[(k * a.ny + nd.y) * a.nz + nd.z] = (float)v;
    }
  }
}

// State (bricks) -> float SoA [19][N].
template <bool F16>
__global__ __launch_bounds__(BLOCK) void export_kernel(CollideArgs a, float* out) {
  const Node nd = decode(a);
  if (!nd.active || !nd.owned) return;
  const size_t N = (size_t)a.nx * a.ny * a.nz;
  const size_t n = ((size_t)nd.x * a.ny + nd.y) * a.nz + nd.z;
  const uint32_t e0 = rowpart(a, nd.x, nd.y) + colpart(a, nd.z);
#pragma unroll
  for (int i = 0; i < Q; ++i) out[(size_t)i * N + n] = Pop<F16>::ld_plain(a.src, i, e0 + (uint32_t)i * ZT, ref_off(a, i, nd.y));
}

// Float SoA [19][N] -> state (bricks), rounded to the storage type.
template <bool F16>
__global__ __launch_bounds__(BLOCK) void import_kernel(CollideArgs a, const float* in) {
  const Node nd = decode(a);
  if (!nd.active || !nd.owned) return;
  const size_t N = (size_t)a.nx * a.ny * a.nz;
  const size_t n = ((size_t)nd.x * a.ny + nd.y) * a.nz + nd.z;
  const uint32_t e0 = rowpart(a, nd.x, nd.y) + colpart(a, nd.z);
#pragma unroll
  for (int i = 0; i < Q; ++i)
    Pop<F16>::st_plain(a.dst, i, e0 + (uint32_t)i * ZT, in[(size_t)i * N + n], ref_off(a, i, nd.y));
}

// FP16 storage reference offsets r_i(y) = f_eq_i(1, u_ref(y)) - w_i (second-order
// equilibrium, FP64, stored as float); u_ref == nullptr gives r = 0.
__device__ double dref_value(const double* u_ref, int ny, int y, int i) {
#pragma clang fp contract(off)  // plain multiplies and adds: reproducible off the device
  const double ux = u_ref[y], uy = u_ref[ny + y], uz = u_ref[2 * ny + y];
  const double cu = CX[i] * ux + CY[i] * uy + CZ[i] * uz;
  return WD[i] * (3.0 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy + uz * uz));
}

// dref[y][i] = r_i(y); dpull[y][i] = r_i of the row a plain pull of direction i
// reads into row y (y - c_y, periodic in y like the plain pull rows).
__global__ void dref_kernel(const double* u_ref, int ny, float* dref, float* dpull) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ny * Q) return;
  const int y = k / Q, i = k % Q;
  const int ys = (y - CY[i] + ny) % ny;
  dref[k] = (float)dref_value(u_ref, ny, y, i);
  dpull[k] = (float)dref_value(u_ref, ny, ys, i);
}

// The current FP16 state re-encoded in place from offsets dold to dnew (either
// may be null: 0).
__global__ __launch_bounds__(BLOCK) void recode_kernel(CollideArgs a, _Float16* state, const float* dold,
                                                       const float* dnew) {
  const Node nd = decode(a);
  if (!nd.active || !nd.owned) return;
  const uint32_t e0 = rowpart(a, nd.x, nd.y) + colpart(a, nd.z);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const float ro = dold ? dold[nd.y * Q + i] : 0.f, rn = dnew ? dnew[nd.y * Q + i] : 0.f;
    _Float16& h = state[e0 + (uint32_t)i * ZT];
    h = (_Float16)(((float)h + ro) - rn);
  }
}

// One 16-byte vector per thread, non-temporal load and store (the bandwidth
// reference of the benchmark: 6.54-6.58 TB/s for 2-11 GiB, against 6.20-6.36
// with plain loads and 5.6-6.1 with 2-8 vectors per thread).  The pull kernels
// keep plain loads: each source row is read by up to nine destination rows,
// which must hit in L2.
typedef float vec4f __attribute__((ext_vector_type(4)));
__global__ void copy_kernel(const vec4f* __restrict__ src, vec4f* __restrict__ dst, int64_t n4) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n4) __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

}  // namespace

// Kernel arguments of a launch reading buffer src and writing buffer dst.
void fill_args(lbm_ctx* h, CollideArgs& a, int src, int dst) {
  const lbm_config& c = h->cfg;
  a.src = h->f[src];
  a.dst = h->f[dst];
  a.hist_in = h->hist[src];
  a.hist_out = h->hist[dst];
  a.u_in = h->stg_bound ? h->stg.u_in : nullptr;
  a.stats = h->d_stats;
  a.wall_acc = h->stats_on ? h->d_wall_acc : nullptr;
  a.wall_line = nullptr;
  a.dref = h->d_dref;
  a.dpull = h->d_dpull;
  a.plane_of_x = h->d_plane_of_x;
  a.err = h->d_err;
  a.nx = c.nx;
  a.ny = c.ny;
  a.nz = c.nz;
  a.zc = h->zc;
  a.yg = h->yg;
  a.nblocks = h->nblocks;
  a.ywall = c.ywall;
  a.xbc = c.xbc;
  a.wall_model = c.wall_model;
  a.wall_law = c.wall_law;
  a.newton_iters = c.newton_iters;
  a.stats_on = h->stats_on && h->d_stats != nullptr;
  // Population stores bypass the caches (non-temporal) unless the next step finds
  // much of the state the last one wrote in the Infinity Cache (the limits are at
  // their constants).
  const int64_t touched = touched_bytes(c);
  a.nt_store = touched > nt_store_min(c) || (h->split && c.nz > 32 && touched < NT_STORE_BELOW_F16) ||
               (h->last_step && touched > NT_LAST_MIN_BYTES[h->split]);
  a.has_g = (c.g[0] != 0.0 || c.g[1] != 0.0 || c.g[2] != 0.0) ? 1 : 0;
  a.tau0 = (float)c.tau0;
  a.tau0sq = (float)(c.tau0 * c.tau0);
  a.smag = (float)(18.0 * std::sqrt(2.0) * c.cs_smag * c.cs_smag);
  for (int k = 0; k < 3; ++k) a.g[k] = (float)c.g[k];
  const double nu0 = (c.tau0 - 0.5) / 3.0;
  a.nu0 = (float)nu0;
  a.inv_nu0 = (float)(1.0 / nu0);
  a.y_wall = (float)c.y_wall;
  a.kappa = (float)c.kappa;
  a.inv_kappa = (float)(1.0 / c.kappa);
  a.b_reich = (float)c.b_reich;
  if (c.outlet == LBM_OUTLET_ZERO_GRADIENT) {
    a.out_wh = 0.f;
    a.out_wu = 1.f;
  } else {  // convective: (f^prev + U_c f(x-1)) / (1 + U_c)
    a.out_wh = (float)(1.0 / (1.0 + c.u_conv));
    a.out_wu = (float)(c.u_conv / (1.0 + c.u_conv));
  }
  a.sponge_x0 = c.sponge_cells > 0 ? c.nx - c.sponge_cells : c.nx;
  a.sponge_inv_len = c.sponge_cells > 0 ? (float)(1.0 / c.sponge_cells) : 0.f;
  a.sponge_dnu = c.sponge_cells > 0 ? (float)(c.sponge_nu - nu0) : 0.f;
  for (int k = 0; k < Q; ++k) {
    a.rs[k] = (float)(c.s[k] / DNORM[k]);
    a.rf[k] = (float)((1.0 - 0.5 * c.s[k]) / DNORM[k]);
  }
}


// The line-averaged u_tau of the step a describes, into h->d_wall_line (a
// no-op unless that model is configured); a.wall_line then points there.
hipError_t launch_wall_line(lbm_ctx* h, CollideArgs& a, hipStream_t stream) {
  const lbm_config& c = h->cfg;
  if (c.wall_avg != LBM_WALL_AVG_LINE || !c.wall_model || c.ywall == LBM_Y_PERIODIC) return hipSuccess;
  if (!h->d_wall_line) {
    hipError_t e = hipMalloc(&h->d_wall_line, sizeof(float) * 2 * c.nx);
    if (e != hipSuccess) return e;
  }
  dim3 grid(c.nx, 2);
  if (c.storage == LBM_STORE_F16DEV)
    wall_line_kernel<true><<<grid, BLOCK, 0, stream>>>(a, h->d_wall_line);
  else
    wall_line_kernel<false><<<grid, BLOCK, 0, stream>>>(a, h->d_wall_line);
  a.wall_line = h->d_wall_line;
  return hipGetLastError();
}

// The bulk blocks of one step (FP16 storage; none with FP32): the kernel
// variant for the body force and the reference offsets.
void launch_bulk_kernel(lbm_ctx* h, const CollideArgs& a, hipStream_t stream) {
  const int n = h->n_int;
  const int* bl = h->d_blist_int;
  if (h->fused) {
    const int ng = h->n_bnd, nt = ng + n;
    const int* gl = h->d_blist_bnd;
    if (nt == 0) return;
    auto go = [&](auto FORCE, auto REF, auto NT) {
      constexpr bool F = FORCE.value, R = REF.value, N = NT.value;
      const int lanes = row_lanes(h->cfg);
      if (lanes == 16)
        collide_fused_kernel<F, R, N, 16><<<nt, YROWS * 16, 0, stream>>>(a, gl, ng, bl, a.dref, a.dpull);
      else if (lanes == 32)
        collide_fused_kernel<F, R, N, 32><<<nt, YROWS * 32, 0, stream>>>(a, gl, ng, bl, a.dref, a.dpull);
      else if (R && N && touched_bytes(h->cfg) > nt_store_min(h->cfg))
        collide_fused_kernel<F, R, N, ZT, R && N><<<nt, BLOCK, 0, stream>>>(a, gl, ng, bl, a.dref, a.dpull);
      else
        collide_fused_kernel<F, R, N, ZT><<<nt, BLOCK, 0, stream>>>(a, gl, ng, bl, a.dref, a.dpull);
    };
    auto store = [&](auto FORCE, auto REF) {
      a.nt_store ? go(FORCE, REF, std::true_type{}) : go(FORCE, REF, std::false_type{});
    };
    auto ref = [&](auto FORCE) { a.dref ? store(FORCE, std::true_type{}) : store(FORCE, std::false_type{}); };
    a.has_g ? ref(std::true_type{}) : ref(std::false_type{});
    return;
  }
  if (n == 0) return;
  // With reference offsets one dispatch over the list, without them one per
  // x-chunk of it (see CHUNK_BLOCKS_F16).
  if (a.dref) {
    if (a.has_g)
      collide_bulk_kernel<true, true><<<n, BLOCK, 0, stream>>>(a, bl, a.dref, a.dpull);
    else
      collide_bulk_kernel<false, true><<<n, BLOCK, 0, stream>>>(a, bl, a.dref, a.dpull);
    return;
  }
  for (size_t k = 0; k + 1 < h->int_off.size(); ++k) {
    const int m = h->int_off[k + 1] - h->int_off[k];
    const int* bk = bl + h->int_off[k];
    if (a.has_g)
      collide_bulk_kernel<true, false><<<m, BLOCK, 0, stream>>>(a, bk, nullptr, nullptr);
    else
      collide_bulk_kernel<false, false><<<m, BLOCK, 0, stream>>>(a, bk, nullptr, nullptr);
  }
}

// The general blocks of one step: one dispatch per x-chunk of the list (the
// chunks update disjoint nodes from s_n, so their order is free).
void launch_edge_kernels(lbm_ctx* h, const CollideArgs& a, hipStream_t stream) {
  const bool f16 = h->cfg.storage == LBM_STORE_F16DEV;
  if (h->rows && !(a.stats_on && h->rows_lose_sampled)) {
    launch_rows(h, a, stream);  // all blocks
    return;
  }
  for (size_t k = 0; k + 1 < h->bnd_off.size(); ++k) {
    const int n = h->bnd_off[k + 1] - h->bnd_off[k];
    const int* bl = h->d_blist_bnd + h->bnd_off[k];
    if (n <= 0) continue;
    if (f16)
      collide_general_kernel<true><<<n, BLOCK, 0, stream>>>(a, bl);
    else if (a.nt_store)
      collide_general_kernel<false, true><<<n, BLOCK, 0, stream>>>(a, bl);
    else
      collide_general_kernel<false, false><<<n, BLOCK, 0, stream>>>(a, bl);
  }
}

// The step's line u_tau (line-averaged wall model; also when no general block
// exists, e.g. a periodic channel with FP16 storage) and the general blocks
// (unless the fused kernel takes them with the bulk blocks).
hipError_t launch_boundary(lbm_ctx* h, int src, int dst, hipStream_t stream, const float* u_in) {
  CollideArgs a;
  fill_args(h, a, src, dst);
  if (u_in) a.u_in = u_in;
  hipError_t e = launch_wall_line(h, a, stream);
  if (e != hipSuccess || h->n_bnd == 0 || h->fused) return e;
  launch_edge_kernels(h, a, stream);
  return hipGetLastError();
}

// One step between caller buffers (statistics off), on one stream: the
// boundary and bulk block lists with FP16 storage, the single list with FP32.
hipError_t launch_step_explicit(lbm_ctx* h, const void* src, void* dst, const float* hist_in, float* hist_out,
                                const float* u_in, hipStream_t stream) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  a.src = src;
  a.dst = dst;
  a.hist_in = hist_in;
  a.hist_out = hist_out;
  a.u_in = u_in;
  a.stats_on = 0;
  a.wall_acc = nullptr;
  hipError_t e = launch_wall_line(h, a, stream);
  if (e != hipSuccess) return e;
  if (!h->fused) launch_edge_kernels(h, a, stream);
  launch_bulk_kernel(h, a, stream);
  return hipGetLastError();
}

// The bulk blocks of one step (with the general blocks when fused; u_in, when
// given, replaces the bound inlet plane).  With the line-averaged wall model
// the step's line u_tau must already be in h->d_wall_line on this stream
// (launch_boundary).
hipError_t launch_bulk(lbm_ctx* h, int src, int dst, hipStream_t stream, const float* u_in) {
  CollideArgs a;
  fill_args(h, a, src, dst);
  if (u_in) a.u_in = u_in;
  if (h->cfg.wall_avg == LBM_WALL_AVG_LINE && h->cfg.wall_model && h->cfg.ywall != LBM_Y_PERIODIC)
    a.wall_line = h->d_wall_line;
  launch_bulk_kernel(h, a, stream);
  return hipGetLastError();
}

// Arrange a list of blocks for dispatch.  Blocks are handed to the 8 XCDs
// round-robin (block b runs on XCD b mod 8), and each XCD has its own L2.
// The only cache lines two blocks share are the edge lines of the +-1 z
// shifts between z-neighbouring bricks of one (x, y-group) column, so every
// column is given to one XCD and its z-chunks run back to back there.
// Columns go to XCDs in turn, each class of column (heavy[c]: wall groups,
// whose blocks take longer) with its own turn, so that every XCD gets its
// share of both; queues are padded with -1 (empty block).
std::vector<int> xcd_order(const std::vector<int>& entries, int zc, const std::vector<char>* heavy) {
  constexpr int NX = 8;
  std::vector<std::vector<int>> q(NX);
  const size_t ncol = entries.size() / zc;
  size_t turn[2] = {0, 0};
  for (size_t c = 0; c < ncol; ++c) {
    const int k = heavy ? ((*heavy)[c] ? 1 : 0) : 0;
    const size_t xcd = turn[k]++ % NX;
    for (int j = 0; j < zc; ++j) q[xcd].push_back(entries[c * zc + j]);
  }
  size_t len = 0;
  for (auto& v : q) len = std::max(len, v.size());
  std::vector<int> out(len * NX, -1);
  for (int k = 0; k < NX; ++k)
    for (size_t j = 0; j < q[k].size(); ++j) out[j * NX + k] = q[k][j];
  return out;
}

// Split the blocks (x, z-chunk, y-group) into bulk and boundary lists,
// each ordered by xcd_order (see collide_bulk_kernel / collide_general_kernel).
// The planes of plane_of_x (the attached statistics planes) are boundary
// blocks whether or not statistics are being accumulated: the two kernels
// round FP16 deviations differently (the bulk kernel computes on deviations),
// and a recompute with statistics off must reproduce the forward run.
// With FP32 storage the boundary list (all blocks) is cut into x-chunks of
// about CHUNK_BLOCKS blocks, with FP16 storage the bulk list into chunks of
// about CHUNK_BLOCKS_F16 (unless it is part of a fused launch), each ordered by
// xcd_order on its own, since every chunk is a dispatch of its own.
hipError_t build_block_lists(lbm_ctx* h, const std::vector<int>& plane_of_x) {
  const lbm_config& c = h->cfg;
  std::vector<int> in, bd;
  std::vector<char> in_heavy;  // per bulk column: a wall group
  in.reserve((size_t)c.nx * h->zc * h->yg);
  int64_t int_nodes = 0;
  const bool split = h->split;
  // columns (x, y-group) in memory order, each with its zc z-chunks
  for (int x = 0; x < c.nx; ++x) {
    // statistics planes (attached, accumulating or not) take the general kernel
    const bool xb = (c.xbc == LBM_X_INFLOW && (x == 0 || x == c.nx - 1)) || plane_of_x[x] >= 0;
    for (int gy = 0; gy < h->yg; ++gy) {
      const int base = std::min(YROWS * gy, c.ny - YROWS);
      const bool bulk_block = split && !xb;  // wall groups take the bulk kernel's wall branch
      if (bulk_block) in_heavy.push_back(c.ywall != LBM_Y_PERIODIC && (base == 0 || base == c.ny - YROWS));
      for (int zc = 0; zc < h->zc; ++zc) {
        const int e = (x * h->zc + zc) * h->yg + gy;
        (bulk_block ? in : bd).push_back(e);
        if (bulk_block) {
          const int owned_rows = YROWS - (YROWS * gy - base);
          const int lanes = std::min(ZT, c.nz - ZT * zc);
          int_nodes += (int64_t)owned_rows * lanes;
        }
      }
    }
  }
  const int per_plane = h->zc * h->yg;
  // General blocks: the outlet plane's and the inlet plane's first, so that the
  // longest are not the launch's tail (256x64x64 FP32 27.2 -> 26.2 us per step,
  // 768x64x192 242 -> 239).  The sampled planes' too where the launch is little
  // more than one round of blocks (64x64x64 10.9 -> 9.9 us); on larger lattices
  // they are no tail, and many of them out of turn cost (128x96x336 with twelve,
  // 112 -> 114.5).  Few blocks go first only where a plane's columns fill the XCDs
  // evenly (four steps with four planes, 41x64x64 44.1 -> 38.3 us, 20x30x128 36.8 ->
  // 33.8): otherwise they cost (41x22x64 34.3 -> 36.4, 30x22x100 31.2 -> 33.0,
  // 41x50x40 32.8 -> 34.8, 100x22x64 38.0 -> 39.2; 55x22x100, 660 blocks, 40.6 -> 38.0).  FP16's general blocks run before the bulk blocks in any case
  // and keep the order of x (64x64x64 10.4 us, outlet first 11.0).
  auto first_the_longest = [&](std::vector<int>& v) {
    const bool open = c.xbc == LBM_X_INFLOW;
    const bool one_round = v.size() <= 2048 && (v.size() > 640 || h->yg % 8 == 0);
    std::vector<int> part[4];
    for (int e : v) {
      const int x = e / per_plane;
      part[open && x == c.nx - 1 ? 0 : (one_round && plane_of_x[x] >= 0 ? 1 : (open && x == 0 ? 2 : 3))].push_back(e);
    }
    v.clear();
    for (const std::vector<int>& p : part) v.insert(v.end(), p.begin(), p.end());
  };
  // Cut a list in memory order (x-major: an x-range is a contiguous run of it)
  // into ranges of `planes` planes, each ordered for the XCDs.
  auto chunk = [&](std::vector<int>& v, int planes, const std::vector<char>* heavy, std::vector<int>& off) {
    std::vector<int> out;
    off.assign(1, 0);
    size_t i = 0;
    for (int x0 = 0; x0 < c.nx; x0 += planes) {
      std::vector<int> part;
      std::vector<char> hv;
      while (i < v.size() && v[i] / per_plane < x0 + planes) {
        if (heavy && i % h->zc == 0) hv.push_back((*heavy)[i / h->zc]);
        part.push_back(v[i++]);
      }
      if (part.empty()) continue;
      if (!split) first_the_longest(part);
      part = xcd_order(part, h->zc, heavy ? &hv : nullptr);
      out.insert(out.end(), part.begin(), part.end());
      off.push_back((int)out.size());
    }
    v.swap(out);
  };
  auto chunk_planes = [&](int blocks) {
    const int n = (int)std::min<int64_t>(c.nx, std::max<int64_t>(1, std::llround((double)h->nblocks / blocks)));
    return (c.nx + n - 1) / n;
  };
  const int planes = split ? c.nx : chunk_planes(CHUNK_BLOCKS);
  chunk(bd, planes, nullptr, h->bnd_off);
  h->int_planes = h->fused ? c.nx : chunk_planes(CHUNK_BLOCKS_F16);
  chunk(in, h->int_planes, &in_heavy, h->int_off);
  h->chunk_planes = planes;
  hipError_t err;
  for (int k = 0; k < 2; ++k) {
    std::vector<int>& v = k == 0 ? in : bd;
    int** d = k == 0 ? &h->d_blist_int : &h->d_blist_bnd;
    int* cap = k == 0 ? &h->cap_int : &h->cap_bnd;
    if (*cap < (int)v.size() || !*d) {
      if (*d && (err = hipFree(*d)) != hipSuccess) return err;
      *d = nullptr;
      if ((err = hipMalloc(d, sizeof(int) * std::max<size_t>(v.size(), 1))) != hipSuccess) return err;
      *cap = (int)std::max<size_t>(v.size(), 1);
    }
    if (!v.empty() && (err = hipMemcpy(*d, v.data(), sizeof(int) * v.size(), hipMemcpyHostToDevice)) != hipSuccess)
      return err;
  }
  h->n_int = (int)in.size();
  h->n_bnd = (int)bd.size();
  h->int_nodes = int_nodes;
  return hipSuccess;
}

hipError_t launch_stream_only(lbm_ctx* h, int src, int dst) {
  CollideArgs a;
  fill_args(h, a, src, dst);
  stream_only_kernel<<<h->nblocks, BLOCK, 0, h->stream>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_init_t(lbm_ctx* h, const T* rho, const T* u, const T* pert, T eps) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  float* hist = h->cfg.xbc == LBM_X_INFLOW ? h->hist[h->cur] : nullptr;
  if (h->cfg.storage == LBM_STORE_F16DEV)
    init_kernel<true, T><<<h->nblocks, BLOCK, 0, h->stream>>>(a, hist, rho, u, pert, eps);
  else
    init_kernel<false, T><<<h->nblocks, BLOCK, 0, h->stream>>>(a, hist, rho, u, pert, eps);
  return hipGetLastError();
}

hipError_t launch_init(lbm_ctx* h, const float* rho, const float* u, const float* pert, float eps) {
  return launch_init_t(h, rho, u, pert, eps);
}

hipError_t launch_init(lbm_ctx* h, const double* rho, const double* u, const double* pert, double eps) {
  return launch_init_t(h, rho, u, pert, eps);
}

hipError_t launch_export(lbm_ctx* h, float* out) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  if (h->cfg.storage == LBM_STORE_F16DEV)
    export_kernel<true><<<h->nblocks, BLOCK, 0, h->stream>>>(a, out);
  else
    export_kernel<false><<<h->nblocks, BLOCK, 0, h->stream>>>(a, out);
  return hipGetLastError();
}

hipError_t launch_import(lbm_ctx* h, const float* in) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  if (h->cfg.storage == LBM_STORE_F16DEV)
    import_kernel<true><<<h->nblocks, BLOCK, 0, h->stream>>>(a, in);
  else
    import_kernel<false><<<h->nblocks, BLOCK, 0, h->stream>>>(a, in);
  return hipGetLastError();
}

// Replace the FP16 storage reference (u_ref: device double [3][ny], or null
// for none) and re-encode the current state.  Synchronises the stream.
hipError_t launch_set_reference(lbm_ctx* h, const double* u_ref) {
  const int ny = h->cfg.ny;
  if (!u_ref && !h->d_dref) return hipSuccess;  // no reference before or after
  float* dnew = nullptr;  // [ny][19] offsets, then [ny][19] pull offsets
  hipError_t e = hipSuccess;
  if (u_ref) {
    if ((e = hipMalloc(&dnew, sizeof(float) * 2 * ny * Q)) != hipSuccess) return e;
    dref_kernel<<<(ny * Q + 255) / 256, 256, 0, h->stream>>>(u_ref, ny, dnew, dnew + ny * Q);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    CollideArgs a;
    fill_args(h, a, h->cur, h->cur);
    recode_kernel<<<h->nblocks, BLOCK, 0, h->stream>>>(a, static_cast<_Float16*>(h->f[h->cur]), h->d_dref, dnew);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) {  // the handle keeps its old reference
    if (dnew) (void)hipFree(dnew);
    return e;
  }
  if (h->d_dref && (e = hipFree(h->d_dref)) != hipSuccess) return e;
  h->d_dref = dnew;
  h->d_dpull = dnew ? dnew + ny * Q : nullptr;
  return hipSuccess;
}

// Float bricks <-> float SoA [19][N] for adjoint fields (always FP32).
hipError_t launch_field_export(lbm_ctx* h, const float* bricks, float* soa) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  a.src = bricks;
  export_kernel<false><<<h->nblocks, BLOCK, 0, h->stream>>>(a, soa);
  return hipGetLastError();
}

hipError_t launch_field_import(lbm_ctx* h, const float* soa, float* bricks) {
  CollideArgs a;
  fill_args(h, a, h->cur, h->cur);
  a.dst = bricks;
  import_kernel<false><<<h->nblocks, BLOCK, 0, h->stream>>>(a, soa);
  return hipGetLastError();
}

hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s) {
  const int64_t n4 = bytes / 16;
  const int64_t nb = (n4 + 255) / 256;
  if (nb < 1 || nb > 0x7fffffff) return hipErrorInvalidValue;
  copy_kernel<<<(unsigned)nb, 256, 0, s>>>(static_cast<const vec4f*>(src), static_cast<vec4f*>(dst), n4);
  return hipGetLastError();
}

}  // namespace lbm
