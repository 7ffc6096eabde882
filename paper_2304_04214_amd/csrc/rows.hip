// The collide-stream step on lattices of few spanwise nodes, FP32 storage
// (Algorithm 1 as in collide.hip's general kernel, with the same arithmetic:
// the states are equal bit for bit).
//
// The kernels of collide.hip give every row (x, y) of 64 spanwise nodes a wave,
// so with nz <= 32 half the lanes or more hold no node (three quarters at
// nz = 16).  Here a block takes whole rows of one x-plane, as many as its
// threads hold, and a thread the node t % nz of row t / nz: the row is a
// per-lane value, the plane a scalar.  Bound by the latency of one round of
// blocks on small lattices, on large ones by the 128-byte lines of the padded
// bricks, of which nz = 16 uses half.  Per step, general kernel -> this one:
// 200x20x16 8.2 -> 6.5 us, 64x32x32 7.3 -> 6.3, 400x40x32 18.5 -> 15.3,
// 603x63x16 39.7 -> 24.6, 603x63x28 41.7 -> 34.0.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "collide.h"
#include "internal.h"
#include "stream.h"

namespace lbm {
namespace {

constexpr int MAXT = 256, MAXZ = 32;  // threads of a block, spanwise nodes

struct RowsLds {
  float u2[2][2][MAXZ];  // (u_x, u_z) of the rows next to the walls
  float ut[2][MAXZ];     // u_tau of the wall rows
  float u[3][MAXT];      // velocities of a sampled plane
};

// Sum over a wave; the order of the reductions in collide.hip.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, ZT);
  return v;
}

// v of the lane N places on in its 16 lanes.
template <int N>
__device__ __forceinline__ double rotate16(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  constexpr int ROW_ROR = 0x120;
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, ROW_ROR + N, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), ROW_ROR + N, 0xf, 0xf, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over each 16 (or 32) lanes: the additions of wave_sum, whose other operands
// are zero.  After the step of 8 the lanes repeat with period 8, and so on, so
// that rotations give what lane ^ 8, ^ 4, ^ 2, ^ 1 hold.
__device__ __forceinline__ double row_sum(double v, bool of32) {
  if (of32) v += __shfl_xor(v, 16, ZT);  // wave-uniform
  v += rotate16<8>(v);
  v += rotate16<4>(v);
  v += rotate16<2>(v);
  v += rotate16<1>(v);
  return v;
}

// rb rows of one x-plane a block, `groups` blocks a plane, the planes x0 .. x0 + planes
// - 1 (all of them: without the two arguments the compiler's registers fall otherwise
// and a step of 200x20x16 takes 6.65 us, with them 6.61).  The stores go through the caches: blocks end within rows,
// and lines written in parts bypassing the caches cost more than what the next
// step reads (521x60x16 27.9 -> 21.2 us per step, 347x60x24 24.3 -> 18.0).
__global__ __launch_bounds__(MAXT) void collide_rows_kernel(CollideArgs a, int x0, int planes, int rb, int groups,
                                                            const int* __restrict__ plane_of_x) {
  __shared__ RowsLds L;
  const int gy = blockIdx.x % groups, xq = blockIdx.x / groups;
  const int x = x0 + (xq == 0 ? planes - 1 : xq - 1);  // the end planes, whose nodes have more to do, go first
  const bool inflow = a.xbc == LBM_X_INFLOW, walls = a.ywall != LBM_Y_PERIODIC;
  const bool bb = a.ywall == LBM_Y_BOUNCEBACK;
  const bool outlet = inflow && x == a.nx - 1, inlet = inflow && x == 0;
  const int t = threadIdx.x;
  const int row = t / a.nz, z = t - row * a.nz;
  const int base = min(rb * gy, a.ny - rb);
  const bool valid = row < rb;  // threads without a node compute another one and store nothing
  const int y = valid ? base + row : base;
  const bool mine = valid && y >= rb * gy;  // rows shared with the previous group are helpers only

  // ---- pulls (the wall rules of issue_pulls): plane by c_x (scalar), row and column by lane ----
  const Geo gx = make_geo(a, x, 0);
  const int zs[3] = {z == a.nz - 1 ? 0 : z + 1, z, z == 0 ? a.nz - 1 : z - 1};  // source z for c_z = -1, 0, 1
  const bool bot = walls && y == 0, top = walls && y == a.ny - 1;
  uint32_t srow[3], scol[3];
#pragma unroll
  for (int c = -1; c <= 1; ++c) {
    int ys = y - c;
    ys = ys < 0 ? ys + a.ny : (ys >= a.ny ? ys - a.ny : ys);
    if (c == 1 ? bot : (c == -1 && top)) ys = y;
    srow[c + 1] = (uint32_t)ys * (BRICK * 4u);
    scol[c + 1] = (uint32_t)zs[c + 1] * 4u;
  }
  const char* s0 = static_cast<const char*>(a.src);
  const size_t plane = (size_t)a.ny * BRICK * 4u;  // bytes per x-plane (one z-chunk)
  const uint32_t self = srow[1] + scol[1];
  auto out = [&](int i) { return CY[i] == 1 ? bot : (CY[i] == -1 && top); };
  // population i as the node of plane xn pulls it, xsrc = xn - c_x: beyond a
  // wall the mirrored one of the own row, or the opposite one of the own node
  auto pull = [&](int xn, int xsrc, int i) {
    const bool own = CY[i] != 0 && bb && out(i);
    const int m = out(i) ? (bb ? opp(i) : REFLY[i]) : i;
    const char* p = s0 + (size_t)xsrc * plane;
    if (CY[i] != 0 && bb) p = own ? s0 + (size_t)xn * plane : p;
    return *reinterpret_cast<const float*>(p + ((own ? self : srow[CY[i] + 1] + scol[CZ[i] + 1]) + (uint32_t)m * (ZT * 4u)));
  };
  // What the end planes read besides the pulls is loaded with them: their nodes
  // are the launch's longest, and the loads' latency would come on top.
  const int pz = y * a.nz + z;
  float e0[5], e1[5];
  if (outlet) {
    const Geo g2 = make_geo(a, x - 1, 0);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      e0[k] = a.hist_in[k * a.ny * a.nz + pz];
      e1[k] = pull(x - 1, g2.xs[CX[OUT5[k]] + 1], OUT5[k]);
    }
  }
  if (inlet) {
#pragma unroll
    for (int k = 0; k < 3; ++k) e0[k] = a.u_in[k * a.ny * a.nz + pz];
  }
  // a sampled plane: this wave's first rows q1 .., their lanes, and what was summed so far
  const int sample = a.stats_on ? plane_of_x[x] : -1;
  const int lanes = a.nz <= 16 ? 16 : 32, per = ZT / lanes, zl = t & (lanes - 1);
  const int q1 = rb * gy - base + uni(t >> 6) * per, qt = q1 + (t & (ZT - 1)) / lanes;
  double* const stat = a.stats + ((size_t)max(sample, 0) * a.ny + base) * 9 + zl;
  const double before = sample >= 0 && qt < rb && zl < 9 ? stat[9 * qt] : 0.0;
  float f[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) f[i] = pull(x, gx.xs[CX[i] + 1], i);
#pragma unroll
  for (int i = 0; i < Q; ++i)
    if (CX[i] != 0) f[i] = gx.xok[CX[i] + 1] || (CY[i] != 0 && bb && out(i)) ? f[i] : 0.f;

  // ---- outlet and inlet (x_rules) ----
  if (outlet) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const float v = outlet_value(a, e0[k], e1[k]);
      f[OUT5[k]] = v;
      if (mine) a.hist_out[k * a.ny * a.nz + pz] = v;
    }
  }
  if (inlet) inlet_regularize(e0[0], e0[1], e0[2], f);

  // ---- density, momentum, forces, collision (node_update) ----
  float rho = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    rho += f[i];
    if (CX[i]) jx += CX[i] * f[i];
    if (CY[i]) jy += CY[i] * f[i];
    if (CZ[i]) jz += CZ[i] * f[i];
  }
  float Fx = 0.f, Fy = 0.f, Fz = 0.f;
  if (a.has_g) {
    Fx = rho * a.g[0];
    Fy = rho * a.g[1];
    Fz = rho * a.g[2];
  }
  const bool wblock = a.wall_model && (base == 0 || base == a.ny - rb);  // block-uniform
  const bool wrow = a.wall_model && (bot || top);
  if (wblock) {  // the block holds a wall row and its neighbour
    const float ir = 1.f / rho;
    if (valid && base == 0 && y == 1) {
      L.u2[0][0][z] = jx * ir;
      L.u2[0][1][z] = jz * ir;
    }
    if (valid && base == a.ny - rb && y == a.ny - 2) {
      L.u2[1][0][z] = jx * ir;
      L.u2[1][1][z] = jz * ir;
    }
    __syncthreads();
    if (wrow) {
      const int w = bot ? 0 : 1;
      float fwx, fwz, ut;
      wall_force(a, rho, jx * ir, jz * ir, L.u2[w][0][z], L.u2[w][1][z], fwx, fwz, ut, w, x);
      Fx += fwx;
      Fz += fwz;
      if (mine) L.ut[w][z] = ut;
    }
  }
  float ux, uy, uz;
  const Tau0 t0 = tau0_of_x(a, x);
  const Pairs pr = make_pairs(f);
  if (a.has_g || wrow)
    collide<true>(a, t0, f, pr, rho, jx, jy, jz, Fx, Fy, Fz, ux, uy, uz);
  else
    collide<false>(a, t0, f, pr, rho, jx, jy, jz, 0.f, 0.f, 0.f, ux, uy, uz);
  if (valid && !(rho > 0.f && rho < 1e30f)) atomicOr(a.err, ERRBIT_NONFINITE);
  if (mine) {
    char* d = static_cast<char*>(a.dst) + (size_t)x * plane;
#pragma unroll
    for (int i = 0; i < Q; ++i) Pop<false>::stp<false>(d + i * (ZT * 4), i, self, f[i], 0.f);
  }

  // ---- statistics: sums over z of the block's own rows ----
  // A wave takes as many rows at a time as have 16 or 32 lanes each, and nine lanes
  // add the nine sums of a row: row after row, and one sum after the other, the
  // sampled blocks were the launch's tail (62x22x9 with twelve planes 22.6 us per
  // step, now 7.6; 200x20x16 18.0, now 7.8).
  const int lane = t & (ZT - 1), wave = uni(t >> 6), nw = blockDim.x / ZT;
  if (sample >= 0) {  // block-uniform
    L.u[0][t] = ux;
    L.u[1][t] = uy;
    L.u[2][t] = uz;
    __syncthreads();
    for (int q0 = q1; q0 < rb; q0 += nw * per) {
      const int q = min(q0 + lane / lanes, rb - 1);
      const bool row = q == q0 + lane / lanes, node = row && zl < a.nz, out = row && zl < 9;
      const double s = q0 == q1 ? before : (out ? stat[9 * q] : 0.0);
      const int k0 = q * a.nz + (node ? zl : 0);
      const double dx = L.u[0][k0], dy = L.u[1][k0], dz = L.u[2][k0];
      const double v[9] = {dx, dy, dz, dx * dx, dy * dy, dz * dz, dx * dy, dx * dz, dy * dz};
      double mine9 = 0.0;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const double sum = row_sum(node ? v[k] : 0.0, lanes == 32);
        mine9 = zl == k ? sum : mine9;
      }
      if (out) stat[9 * q] = s + mine9;
    }
  }
  if (wblock && a.wall_acc) {  // block-uniform: sums of u_tau, by the blocks that own a wall row
    __syncthreads();
    for (int w = wave; w < 2; w += nw) {
      if (w == 0 ? gy != 0 : gy != groups - 1) continue;
      const double sum = wave_sum(lane < a.nz ? (double)L.ut[w][lane] : 0.0);
      if (lane == 0) a.wall_acc[(size_t)w * a.nx + x] += sum;
    }
  }
}

}  // namespace

// Touched bytes up to which the row kernel is taken: us per five steps, general
// kernel -> this one, 1028x60x16 (300 MB) 260 -> 210, 617x100x24 289 -> 274, 617x100x32
// 277 -> 251; rows that are no multiple of 32 bytes lose near the Infinity Cache's
// size, 3084x20x17 (300 MB) 283 -> 298, 2878x20x17 (280 MB) 267 -> 275, 1028x60x3 257 ->
// 267, 545x100x17 (265 MB) 258 -> 245, and earlier the longest of them, 617x100x28 289 ->
// 306, 524x100x28 (255 MB) 249 -> 254, 442x100x28 (215 MB) 215 -> 206.
int64_t rows_max(const lbm_config& c) {
  const int mib = c.nz % 8 == 0 ? 288 : (c.nz <= 24 ? 264 : 224);
  return (int64_t)mib << 20;
}

// Rows per block and blocks per plane of the row kernel (0 rows: not used).
// FP32 storage with nz <= 32, where a step's stores stay in the caches for the
// next (rows_max): us per step, general kernel -> this one, 625x96x24
// (60,000 rows) 58.5 -> 48.3, 687x104x28 (71,000) 65 -> 108, with non-temporal
// stores 82.  Beyond 32 a row leaves less than half the wave idle and little is
// won by more nodes a wave (190x63x48 18.3 -> 18.4, 400x75x40 42.5 -> 46.5).
// The rows are those that leave the fewest threads without a row of their own.
// Up to 2^17 nodes the chip takes all blocks in one round and the smallest such
// blocks are taken (200x20x16: 6.5 us per step with one wave a block, 7.4 with two
// of which a quarter idles); above, the largest of up to 256 threads (400x40x32
// 15.3 us, 16.9 with 128).  Every block has at least two rows, a wall row and the
// row next to it.
// A closed channel of up to one general block a CU keeps the general kernel with
// the wall model, whose Newton steps and plain rows then share a wave here: us per
// four steps, general -> this one, 13x10x6 20.4 -> 22.0, 13x60x14 20.7 -> 23.0, 40x24x6
// (240 blocks) 20.9 -> 21.9, 24x60x8 (360) -> 1.09x; with one or two spanwise nodes, 64
// rows a wave, up to 640: 13x60x2 20.7 -> 24.6, without walls 17.7 -> 19.6, 40x60x1
// 25.9 -> 27.2.  In an open channel the end planes are the longest and their loads go
// out earlier here: 1.00x to 1.29x from 24 blocks on.
// A wave sums a sampled plane's rows a few at a time (four of up to 16 lanes, two
// of 32, at twice the adds), the general kernel one each: where a block's rows
// take several turns and the launch is short enough to wait for them, sampled steps
// go to the general kernel.  us per two steps, general -> this one, by turns (twice
// as many with 32 lanes) and blocks of the general kernel, two planes: 2 turns
// 24x50x8 (312) 13.9 -> 14.2, 41x50x12 (533) 14.2 -> 15.4, 168x16x5 (672, six steps,
// eight planes) 43.0 -> 49.2, 70x50x8 (910) 16.6 -> 15.5;
// 3 turns 41x50x6 (533) 14.1 -> 16.8, 70x50x6 (910) 16.5 -> 17.3, 120x50x6 (1560) 19.7 ->
// 19.3; 4 turns 41x50x24 (533) 14.8 -> 17.4, 89x64x3 (1424) 18.5 -> 20.9; four
// planes: 103x60x24 (1545) 30.1 -> 27.4;
// 8 turns 41x60x2 (615) 22.7 -> 29.0, 240x60x2 (3600) 38.9 -> 41.3, 308x60x2 (4620)
// 44.7 -> 42.4; one turn 16x50x16 13.8 -> 13.3, 21x20x28 19.2 -> 18.2.
void plan_rows(lbm_ctx* h) {
  const lbm_config& c = h->cfg;
  h->rows = 0;
  if (c.storage != LBM_STORE_F32 || c.nz > MAXZ || touched_bytes(c) > rows_max(c)) return;
  if (c.xbc != LBM_X_INFLOW && (int64_t)c.nx * h->yg <= (c.nz <= 2 ? 640 : (c.wall_model ? 256 : 0))) return;
  const bool small = h->N <= (int64_t(1) << 17);
  const int most = std::min((small ? MAXT / 2 : MAXT) / c.nz, c.ny);
  int64_t least = 0;  // threads of a plane
  for (int k = 2; k <= most; ++k) {
    const int rb = small ? k : most + 2 - k;
    const int threads = (rb * c.nz + ZT - 1) / ZT * ZT, groups = (c.ny + rb - 1) / rb;
    if (h->rows && (int64_t)threads * groups >= least) continue;
    least = (int64_t)threads * groups;
    h->rows = rb;
    h->row_threads = threads;
    h->row_groups = groups;
  }
  if (!h->rows) return;
  const int per = c.nz <= 16 ? 4 : 2, at_once = h->row_threads / ZT * per;
  const int turns = (h->rows + at_once - 1) / at_once;
  const int64_t w = turns * (4 / per);
  h->rows_lose_sampled = turns > 1 && (int64_t)c.nx * h->yg < 560 + 60 * w * w;
}

// One dispatch, as the general kernel's of lattices this small.  The caller reads the
// launch error: reading clears it.
void launch_rows(lbm_ctx* h, const CollideArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)h->cfg.nx * h->row_groups);
  collide_rows_kernel<<<grid, h->row_threads, 0, stream>>>(a, 0, h->cfg.nx, h->rows, h->row_groups, a.plane_of_x);
}

}  // namespace lbm
