// cfd_kernels.hip -- gfx950 kernels of libcfd: metrics, viscous prepass, AFWENO direction
// sweeps with the fused RK3 update, halo copies, boundary fills and reductions.
//
// Method: Ye et al., arXiv 2006.07964, Sec. 2 (Eqs 1-21) and Sec. 4.5 (modified AFWENO).
#include <type_traits>
#include <hip/hip_runtime.h>

#include "../../include/cfd.h"
#include "cfd_kernels.hpp"

namespace cfd {

// Workgroups are handed to the eight XCDs round-robin (id mod 8).  Remap the id so that
// each XCD walks a contiguous range of logical tiles; with the sweep-direction tile index
// fastest, tiles that share halo rows run back to back on the same L2.
__device__ __forceinline__ int xcd_remap(int wg, int nwg) {
  const int x = wg & 7, local = wg >> 3;
  const int q = nwg >> 3, r = nwg & 7;
  return x * q + (x < r ? x : r) + local;
}

// Persistent schedule: the `total` work items are split into eight contiguous ranges, one
// per XCD; this workgroup is number *lane_wg of the *nwg_x workgroups on its XCD.
__device__ __forceinline__ void xcd_range(int total, int* start, int* count, int* lane_wg, int* nwg_x) {
  const int x = blockIdx.x & 7;
  const int q = total >> 3, r = total & 7;
  *start = x * q + (x < r ? x : r);
  *count = q + (x < r ? 1 : 0);
  *lane_wg = blockIdx.x >> 3;
  const int G = gridDim.x;
  *nwg_x = (G >> 3) + (x < (G & 7) ? 1 : 0);
}

// =====================================================================================
// Metrics (Sec. 2, Eqs 7-8), FP64, setup only.
// =====================================================================================
struct CBox {
  int sx, sy, sz;  // extents of the tight coordinate-box layout (n + 12)
};

__device__ __forceinline__ int64_t cat(const MetricArgs& a, int i, int j, int k) {
  return ((int64_t)(k + kCHalo) * a.cld_j + (j + kCHalo)) * a.cld_i + (i + kCHalo);
}
__device__ __forceinline__ int64_t tat(const CBox& b, int i, int j, int k) {
  return ((int64_t)(k + kCHalo) * b.sy + (j + kCHalo)) * b.sx + (i + kCHalo);
}

// Pass 1: inner derivatives dX_c/d(dir) for every coordinate-box point whose 7-point
// stencil along dir fits in the box.  Plane 3*c + dir of dcoord.
__global__ __launch_bounds__(256) void k_metric_inner(MetricArgs a) {
  const CBox b{a.g.ni + 12, a.g.nj + 12, a.g.nk + 12};
  const int i = blockIdx.x * 64 + (threadIdx.x & 63) - kCHalo;
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6) - kCHalo;
  const int k = blockIdx.z - kCHalo;
  if (i >= a.g.ni + kCHalo || j >= a.g.nj + kCHalo) return;
  const int64_t plane = (int64_t)b.sx * b.sy * b.sz;
  const int n[3] = {a.g.ni, a.g.nj, a.g.nk};
  const int idx[3] = {i, j, k};
  for (int dir = 0; dir < 3; ++dir) {
    if (idx[dir] < -3 || idx[dir] >= n[dir] + 3) continue;
    const int64_t st = dir == 0 ? 1 : dir == 1 ? a.cld_i : a.cld_i * a.cld_j;
    for (int c = 0; c < 3; ++c) {
      const double* X = a.xyz + c * a.cplane + cat(a, i, j, k);
      a.dcoord[(3 * c + dir) * plane + tat(b, i, j, k)] =
          d6<double>([&](int m) { return X[m * st]; });
    }
  }
}

// Pass 2: conservative metrics (Eq 7) and Jacobian (Eq 8) on the halo-3 box.
// hatted metric (d, c) = d/d(d2) (X_{c1,d1} X_{c2}) - d/d(d1) (X_{c1,d2} X_{c2}) with
// c1 = c+1, c2 = c+2, d1 = d+1, d2 = d+2 (mod 3).
__global__ __launch_bounds__(256) void k_metric_outer(MetricArgs a) {
  const CBox b{a.g.ni + 12, a.g.nj + 12, a.g.nk + 12};
  const int i = blockIdx.x * 64 + (threadIdx.x & 63) - kHalo;
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6) - kHalo;
  const int k = blockIdx.z - kHalo;
  if (i >= a.g.ni + kHalo || j >= a.g.nj + kHalo) return;
  const int64_t cplane = (int64_t)b.sx * b.sy * b.sz;
  const int64_t tp = tat(b, i, j, k);
  const int64_t cp = cat(a, i, j, k);
  const int64_t tst[3] = {1, b.sx, (int64_t)b.sx * b.sy};
  const int64_t cst[3] = {1, a.cld_i, a.cld_i * a.cld_j};
  const int64_t p = at(a.g, i, j, k);
  for (int d = 0; d < 3; ++d) {
    const int d1 = (d + 1) % 3, d2 = (d + 2) % 3;
    for (int c = 0; c < 3; ++c) {
      const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
      const double* Xb = a.xyz + c2 * a.cplane + cp;
      const double* Da = a.dcoord + (3 * c1 + d1) * cplane + tp;  // X_{c1} along d1
      const double* Db = a.dcoord + (3 * c1 + d2) * cplane + tp;  // X_{c1} along d2
      const double t1 = d6<double>([&](int m) { return Da[m * tst[d2]] * Xb[m * cst[d2]]; });
      const double t2 = d6<double>([&](int m) { return Db[m * tst[d1]] * Xb[m * cst[d1]]; });
      a.met[(3 * d + c) * a.g.plane + p] = t1 - t2;
    }
  }
  double D[3][3];  // D[c][dir] = dX_c/d(dir)
  for (int c = 0; c < 3; ++c)
    for (int dir = 0; dir < 3; ++dir) D[c][dir] = a.dcoord[(3 * c + dir) * cplane + tp];
  const double jinv = D[0][0] * D[1][1] * D[2][2] - D[0][0] * D[1][2] * D[2][1] + D[0][1] * D[1][2] * D[2][0] -
                      D[0][1] * D[1][0] * D[2][2] + D[0][2] * D[1][0] * D[2][1] - D[0][2] * D[1][1] * D[2][0];
  if (!(jinv > 0.0)) atomicOr(a.bad, 1);
  a.met[9 * a.g.plane + p] = 1.0 / jinv;
}

hipError_t launch_metrics(const MetricArgs& a, hipStream_t s) {
  dim3 blk(256);
  dim3 g1((a.g.ni + 12 + 63) / 64, (a.g.nj + 12 + 3) / 4, a.g.nk + 12);
  hipLaunchKernelGGL(k_metric_inner, g1, blk, 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 g2((a.g.ni + 6 + 63) / 64, (a.g.nj + 6 + 3) / 4, a.g.nk + 6);
  hipLaunchKernelGGL(k_metric_outer, g2, blk, 0, s, a);
  return hipGetLastError();
}

// =====================================================================================
// Viscous prepass (Eqs 5, 6, 21): nodal viscous fluxes of all three directions.
// Plane 4*d + (n-1) holds component n = 1..4 of the direction-d flux, divided by J.
//
// A workgroup owns a VI x VJ tile of (i, j) columns and marches along k through a chunk
// of kc planes.  Each thread keeps the primitives (u, v, w, T) of its own column at
// k-3..k+3 in registers for the zeta derivative; the primitives of plane k, with three
// halo columns / rows, go through LDS for the xi and eta derivatives.  Every primitive is
// formed about twice per chunk instead of at each of its eighteen stencil uses, and Q is
// read once per column.
// =====================================================================================
constexpr int kViscChunk = 128;  // most planes per workgroup (fewer when nk is smaller)

// Two tile shapes.  64 x 16 columns (1024 threads, one workgroup per CU) read the fewest halo
// nodes of Q per output and stream a large block at the copy rate; 32 x 8 (256 threads, four
// workgroups per CU) suit blocks whose Q stays in the 256 MB last-level cache, where the wider
// halo costs little and finer, independently waiting workgroups fill the chip and leave less
// of it idle in the last round.  FP64 prepass, 64 x 16 against 32 x 8, each at its best chunk:
// 32^3 11.1 / 7.4 us, 101x94x99 54.2 / 55.5, 96x100x98 56.3 / 47.7, 130x96x120 95 / 89, 160^3
// 189 / 172, 190x131x93 113 / 113, 186x150x181 227 / 240, 201x187x168 314 / 298, 256^3
// 755 / 793; FP32: 32^3 8.9 / 7.5, 101x94x99 39.1 / 45.0, 96x100x98 37.0 / 36.8, 160^3
// 130 / 124, 190x131x93 76 / 84, 201x187x168 200 / 221, 256^3 521 / 596.
template <bool SMALL>
struct ViscTile {
  static constexpr int VI = SMALL ? 32 : 64, VJ = SMALL ? 8 : 16, NT = VI * VJ;
  static constexpr int NHALO = 6 * (VI + VJ);  // halo nodes of a plane (a cross, no corners)
  static constexpr int NBUF = SMALL ? 2 : 1;   // LDS planes: two need one barrier per plane
  static constexpr int SLOTS = SMALL ? 1024 : 256;  // workgroups the chip holds at once
  static_assert(NHALO <= NT, "one halo node per thread");
};
// At most kViscLatency points: 32 x 8, a round of a few planes whose latencies count.  Above,
// the shape with the fewer rounds x planes (visc_plan), a plane of 32 x 8 taking 8% (FP64) or
// 24% (FP32) longer; from kViscTraffic points on the halo traffic reaches memory: 64 x 16.
constexpr int64_t kViscLatency = 600000, kViscTraffic = 7000000;
constexpr double kViscSmallPlane[2] = {1.08, 1.24};  // FP64, FP32

template <typename R, bool SMALL>
struct ViscShared {
  // (u, v, w, T) of plane k at (j - j0 + 3, i - i0 + 3)
  R p[ViscTile<SMALL>::NBUF][4][ViscTile<SMALL>::VJ + 6][ViscTile<SMALL>::VI + 6];
};

template <typename R>
__device__ __forceinline__ void primitives(GP<const double> Q, int64_t plane, uint32_t p, R gg, R out[4]) {
  R q[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) q[v] = R(ldg(plane_ptr(Q, v * plane), p));
  const R rinv = rcp(q[0]);
  out[0] = q[1] * rinv;
  out[1] = q[2] * rinv;
  out[2] = q[3] * rinv;
  out[3] = gg * (q[4] * rinv - R(0.5) * (out[0] * out[0] + out[1] * out[1] + out[2] * out[2]));
}

// One-sided closure of the viscous derivatives (Sec. 4.5.2 mentions one-sided differences
// near block boundaries without giving them): the derivative at node r = 0, 1, 2 of a face
// of the degree-6 polynomial through the seven nodes nearest it (node 0 on the face, node
// m at distance m inside) is sum_m kOS6[r][m] f(m) (Lagrange derivative weights, unit
// spacing); a node r away from the high face takes the mirror image with the opposite sign.
__constant__ double kOS6[3][7] = {
    {-49.0 / 20.0, 6.0, -15.0 / 2.0, 20.0 / 3.0, -15.0 / 4.0, 6.0 / 5.0, -1.0 / 6.0},
    {-1.0 / 6.0, -77.0 / 60.0, 5.0 / 2.0, -5.0 / 3.0, 5.0 / 6.0, -1.0 / 4.0, 1.0 / 30.0},
    {1.0 / 30.0, -2.0 / 5.0, -7.0 / 12.0, 4.0 / 3.0, -1.0 / 2.0, 2.0 / 15.0, -1.0 / 60.0}};

// Window of the one-sided closure for the node at index n of an axis of nd nodes, given
// the face mask bits of that axis (bit 0: low face one-sided, bit 1: high face): returns
// false for a central node, else the first window node, the weight row and the sign.
__device__ __forceinline__ bool one_sided_window(int bits, int n, int nd, int* first, int* row, int* sign) {
  if ((bits & 1) && n < 3) {
    *first = 0;
    *row = n;
    *sign = 1;
    return true;
  }
  if ((bits & 2) && n > nd - 4) {
    *first = nd - 7;
    *row = nd - 1 - n;
    *sign = -1;
    return true;
  }
  return false;
}
__device__ __forceinline__ double os6_weight(int row, int sign, int m) {
  return sign > 0 ? kOS6[row][m] : -kOS6[row][6 - m];
}

// The weight table in LDS, for kernels whose lanes look up different rows (a load from memory
// for each of seven dependent terms held up every tile next to a wall).  Every thread of the
// workgroup calls it before a barrier.
template <typename R>
__device__ __forceinline__ void os6_stage(R* tab) {
  if (threadIdx.x < 21) tab[threadIdx.x] = R(kOS6[threadIdx.x / 7][threadIdx.x % 7]);
}
template <typename R>
__device__ __forceinline__ R os6_weight(const R* tab, int row, int sign, int m) {
  return sign > 0 ? tab[row * 7 + m] : -tab[row * 7 + 6 - m];
}

// d/dn of a field on a 7-point line, g(m) = value at offset m (sixth-order central)
template <typename R, typename F>
__device__ __forceinline__ R grad6(F g) {
  R s = R(0);
#pragma unroll
  for (int m = -3; m <= 3; ++m) {
    if (m == 0) continue;
    const R wgt = (m == 1 || m == -1) ? R(0.75) : (m == 2 || m == -2) ? R(-0.15) : R(1.0 / 60.0);
    s += (m > 0 ? wgt : -wgt) * g(m);
  }
  return s;
}

// OS: the block may have faces with the one-sided closure (a separate instantiation, so
// that blocks without them keep the register budget of the plain prepass)
template <typename R, bool OS, bool SMALL>
__device__ __forceinline__ void visc_tile(const ViscArgs& a, int t, ViscShared<R, SMALL>& sh) {
  constexpr int VI = ViscTile<SMALL>::VI, VJ = ViscTile<SMALL>::VJ, NBUF = ViscTile<SMALL>::NBUF;
  const Geom& g = a.g;
  const int nti = (g.ni + VI - 1) / VI, ntj = (g.nj + VJ - 1) / VJ;
  const int i0 = (t % nti) * VI, j0 = ((t / nti) % ntj) * VJ;
  const int k0 = (t / (nti * ntj)) * a.kc;
  const int k1 = min(k0 + a.kc, g.nk);
  const int ti = threadIdx.x % VI, tj = threadIdx.x / VI;
  const int i = i0 + ti, j = j0 + tj;
  const bool own = i < g.ni + kHalo && j < g.nj + kHalo;  // column inside the stored array
  const bool act = i < g.ni && j < g.nj;                  // column with outputs
  const uint32_t sk = (uint32_t)(g.ld_i * g.ld_j);
  const uint32_t pc = (uint32_t)at(g, own ? i : 0, own ? j : 0, 0);  // (i, j, k = 0); plane < 2^29
  // halo node of this thread in plane k: eta rows below / above the tile, xi columns
  // left / right of it (the stencil is a cross, corners are not needed)
  int hi = 0, hj = 0;
  const int h = threadIdx.x;
  if (h < 2 * 3 * VI) {
    hi = i0 + h % VI;
    hj = h < 3 * VI ? j0 - 3 + h / VI : j0 + VJ + (h - 3 * VI) / VI;
  } else if (h < 2 * 3 * VI + 2 * 3 * VJ) {
    const int e = h - 2 * 3 * VI;
    hj = j0 + (e % (3 * VJ)) / 3;
    hi = e < 3 * VJ ? i0 - 3 + e % 3 : i0 + VI + e % 3;
  } else {
    hi = g.ni + kHalo;  // no halo node
  }
  const bool hval = hi < g.ni + kHalo && hj < g.nj + kHalo;
  const uint32_t ph = (uint32_t)at(g, hval ? hi : 0, hval ? hj : 0, 0);

  const R gg = R(a.ph.gamma) * (R(a.ph.gamma) - R(1));
  const GP<const double> Q = to_global(a.q);
  const GP<const R> met = to_global(static_cast<const R*>(a.met_r));
  const GP<R> out = to_global(static_cast<R*>(a.vis));
  const int64_t plane = g.plane;
  __shared__ R os_tab[OS ? 21 : 1];
  if constexpr (OS) os6_stage(os_tab);  // the barrier of the first plane orders it
  R P[7][4];  // own column, planes k-3 .. k+3
  if (own) {
#pragma unroll
    for (int m = 0; m < 6; ++m) primitives<R>(Q, plane, pc + (uint32_t)(k0 - 3 + m) * sk, gg, P[m]);
  }
  for (int k = k0; k < k1; ++k) {
    if (own) primitives<R>(Q, plane, pc + (uint32_t)(k + 3) * sk, gg, P[6]);
    auto& sp = sh.p[NBUF == 2 ? (k & 1) : 0];
    if (own) {
#pragma unroll
      for (int n = 0; n < 4; ++n) sp[n][tj + 3][ti + 3] = P[3][n];
    }
    if (hval) {
      R ph4[4];
      primitives<R>(Q, plane, ph + (uint32_t)k * sk, gg, ph4);
#pragma unroll
      for (int n = 0; n < 4; ++n) sp[n][hj - j0 + 3][hi - i0 + 3] = ph4[n];
    }
    // the metrics and the flux planes stream through (read or written once): streaming
    // accesses leave L2 to the Q rows and columns that the neighbouring tiles read as
    // their halo (measured on the 512 x 512 x 384 channel: 4% faster in FP64).  The small
    // tile, whose chunks are a plane or a few, requests its metrics before the barrier (32^3
    // FP64 9.9 -> 7.4 us); the closure's kernels have no registers left for that.
    constexpr bool EARLY = SMALL && !OS;
    R mh[3][3], J;
    auto load_metrics = [&]() {
      const uint32_t p = pc + (uint32_t)k * sk;
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int c = 0; c < 3; ++c) mh[d][c] = ldg_nt(plane_ptr(met, (3 * d + c) * plane), p);
      J = ldg_nt(plane_ptr(met, 9 * plane), p);
    };
    if (EARLY && act) load_metrics();
    __syncthreads();
    if (act) {
      R gr[4][3];  // d(u, v, w, T)/d(xi, eta, zeta)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        gr[n][0] = grad6<R>([&](int m) { return sp[n][tj + 3][ti + 3 + m]; });
        gr[n][1] = grad6<R>([&](int m) { return sp[n][tj + 3 + m][ti + 3]; });
        gr[n][2] = grad6<R>([&](int m) { return P[3 + m][n]; });
      }
      const uint32_t p = pc + (uint32_t)k * sk;
      if constexpr (OS) {
        // nodes next to a one-sided face of direction d: the seven-point one-sided
        // derivative over the nodes nearest the face replaces the central one (whose
        // ghost values it ignores).  Along xi and eta the LDS plane holds the window's
        // primitives (unless a last tile has fewer than four columns or rows), else they
        // come from Q, whose loads one after the other would hold up the whole tile
        const int idx[3] = {i, j, k};
        const int nds[3] = {g.ni, g.nj, g.nk};
        const uint32_t st[3] = {1u, (uint32_t)g.ld_i, sk};
#pragma unroll 1
        for (int d = 0; d < 3; ++d) {
          int first, row, sign;
          if (!one_sided_window((a.one_sided >> (2 * d)) & 3, idx[d], nds[d], &first, &row, &sign)) continue;
          R acc[4] = {R(0), R(0), R(0), R(0)};
          const int at0 = first - (d == 0 ? i0 : j0) + 3;  // the window in the LDS plane
          if (d < 2 && at0 >= 0 && at0 + 6 < (d == 0 ? VI : VJ) + 6) {
            const R* w0 = d == 0 ? &sp[0][tj + 3][at0] : &sp[0][at0][ti + 3];
            const int next = d == 0 ? 1 : VI + 6;
#pragma unroll 1
            for (int m = 0; m < 7; ++m) {
              const R wgt = os6_weight(os_tab, row, sign, m);
#pragma unroll
              for (int n = 0; n < 4; ++n) acc[n] += wgt * w0[n * (VJ + 6) * (VI + 6) + m * next];
            }
          } else {
#pragma unroll 1
            for (int m = 0; m < 7; ++m) {
              R pr[4];
              primitives<R>(Q, plane, p + (uint32_t)(first + m - idx[d]) * st[d], gg, pr);
              const R wgt = os6_weight(os_tab, row, sign, m);
#pragma unroll
              for (int n = 0; n < 4; ++n) acc[n] += wgt * pr[n];
            }
          }
#pragma unroll
          for (int n = 0; n < 4; ++n) gr[n][d] = acc[n];
        }
      }
      if constexpr (!EARLY) load_metrics();
      R dx[4][3];  // d(u, v, w, T)/d(x, y, z), Eq 21
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int c = 0; c < 3; ++c) dx[n][c] = J * (mh[0][c] * gr[n][0] + mh[1][c] * gr[n][1] + mh[2][c] * gr[n][2]);
      const R u = P[3][0], v = P[3][1], w = P[3][2];
      const R mu = viscosity(P[3][3], R(a.ph.suth));
      const R vs = R(a.ph.visc_scale) * mu;
      const R lam = R(-2.0 / 3.0) * vs;
      const R div = dx[0][0] + dx[1][1] + dx[2][2];
      R tau[3][3];
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) tau[r][c] = vs * (dx[r][c] + dx[c][r]) + (r == c ? lam * div : R(0));
      const R hs = R(a.ph.heat_scale) * mu;
      R bet[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) bet[c] = u * tau[0][c] + v * tau[1][c] + w * tau[2][c] + hs * dx[3][c];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        R f[4];
#pragma unroll
        for (int n = 0; n < 3; ++n) f[n] = mh[d][0] * tau[n][0] + mh[d][1] * tau[n][1] + mh[d][2] * tau[n][2];
        f[3] = mh[d][0] * bet[0] + mh[d][1] * bet[1] + mh[d][2] * bet[2];
#pragma unroll
        for (int n = 0; n < 4; ++n) stg_nt(plane_ptr(out, (4 * d + n) * plane), p, f[n]);
        // a block periodic with itself along d: the node's image in the halo across the
        // d-faces (the direction-d flux is the one the d sweep differentiates)
        if (a.periodic & (1 << d)) {
          const int idx = d == 0 ? i : d == 1 ? j : k;
          const int nd = d == 0 ? g.ni : d == 1 ? g.nj : g.nk;
          const uint32_t sd = d == 0 ? 1u : d == 1 ? (uint32_t)g.ld_i : sk;
          if (idx < kHalo || idx >= nd - kHalo) {
            const uint32_t pi = idx < kHalo ? p + (uint32_t)nd * sd : p - (uint32_t)nd * sd;
#pragma unroll
            for (int n = 0; n < 4; ++n) stg_nt(plane_ptr(out, (4 * d + n) * plane), pi, f[n]);
          }
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 6; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n) P[m][n] = P[m + 1][n];
    // plane k of the LDS tile is consumed; with two buffers the next plane goes to the other
    // one, and the barrier of the plane after next orders that write behind these reads
    if constexpr (NBUF == 1) __syncthreads();
  }
}

template <typename R, bool OS, bool SMALL>
__global__ __launch_bounds__(ViscTile<SMALL>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_visc(ViscArgs a) {
  __shared__ ViscShared<R, SMALL> sh;
  visc_tile<R, OS, SMALL>(a, xcd_remap(blockIdx.x, gridDim.x), sh);
}

__global__ __launch_bounds__(256) void k_round(const double* __restrict__ src, float* __restrict__ dst, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) dst[e] = float(src[e]);
}

hipError_t launch_round(const double* src, float* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nwg = (n + 255) / 256;
  hipLaunchKernelGGL(k_round, dim3((unsigned)(nwg < 65536 ? nwg : 65536)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

// Half-point metrics of a mixed-precision block (one thread per stored node and direction).
__global__ __launch_bounds__(256) void k_half_metric(Geom g, const double* __restrict__ met, float* __restrict__ hm) {
  const int64_t pl = g.plane;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < 3 * pl; e += (int64_t)gridDim.x * 256) {
    const int d = (int)(e / pl);
    const int64_t p = e - d * pl;
    const int64_t ij = g.ld_i * g.ld_j;
    const int idx = d == 0 ? (int)(p % g.ld_i) - kHalo
                  : d == 1 ? (int)((p / g.ld_i) % g.ld_j) - kHalo
                           : (int)(p / ij) - kHalo;
    const int nd = d == 0 ? g.ni : d == 1 ? g.nj : g.nk;
    if (idx < -1 || idx > nd - 1) continue;  // the stencil idx-2 .. idx+3 stays in the halo
    const int64_t st = d == 0 ? 1 : d == 1 ? g.ld_i : ij;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double* m = met + (3 * d + c) * pl + p;
      hm[(3 * d + c) * pl + p] = float(half_metric([&](int o) { return m[o * st]; }));
    }
  }
}

hipError_t launch_half_metrics(const Geom& g, const double* met, float* hm, hipStream_t s) {
  const int64_t nwg = (3 * g.plane + 255) / 256;
  hipLaunchKernelGGL(k_half_metric, dim3((unsigned)(nwg < 65536 ? nwg : 65536)), dim3(256), 0, s, g, met, hm);
  return hipGetLastError();
}

static int visc_cols(const Geom& g, bool small) {
  const int vi = small ? ViscTile<true>::VI : ViscTile<false>::VI, vj = small ? ViscTile<true>::VJ : ViscTile<false>::VJ;
  return ((g.ni + vi - 1) / vi) * ((g.nj + vj - 1) / vj);
}

// Tile shape, chunk lengths and tile counts of a launch over nb blocks (i-tile fastest, then
// j-tile, then k-chunk).  For a shape, the chunk bound c (<= kViscChunk) with the least rounds
// x (c + 3), rounds the times the tiles fill the chip and 3 the measured cost of the six
// priming planes of a chunk in units of an output plane; nk is then split into the fewest
// equal chunks under c.  (160^3 FP64 before, with a bound halved until 256 tiles were reached:
// 300 tiles of 1024 threads, two rounds, 258 us.)  A batch of kViscTraffic points or more has
// several rounds in any case and keeps chunks of at most kViscChunk, halved (down to 8) where
// a block has fewer than kViscMinTilesBatch tiles.
static int64_t visc_chunk(const Geom* gs, int nb, int nkmax, bool small, int* chunk) {
  const int slots = small ? ViscTile<true>::SLOTS : ViscTile<false>::SLOTS;
  int64_t best = INT64_MAX;
  for (int c = nkmax < kViscChunk ? nkmax : kViscChunk; c >= 1; --c) {
    int64_t t = 0;
    for (int b = 0; b < nb; ++b) t += (int64_t)visc_cols(gs[b], small) * ((gs[b].nk + c - 1) / c);
    const int64_t cost = ((t + slots - 1) / slots) * (c + 3);
    if (cost < best) best = cost, *chunk = c;
  }
  return best;
}

void visc_plan(const Geom* gs, int nb, bool batch, bool fp64, bool* small_out, int* kc, int* tiles) {
  int64_t points = 0;
  int nkmax = 0;
  for (int b = 0; b < nb; ++b) {
    points += (int64_t)gs[b].ni * gs[b].nj * gs[b].nk;
    nkmax = gs[b].nk > nkmax ? gs[b].nk : nkmax;
  }
  int chunk[2] = {0, 0};  // 64 x 16, 32 x 8
  bool small = points <= kViscLatency;
  const int64_t small_cost = visc_chunk(gs, nb, nkmax, true, &chunk[1]);
  if (!small) {
    const int64_t large_cost = visc_chunk(gs, nb, nkmax, false, &chunk[0]);
    small = points < kViscTraffic && kViscSmallPlane[fp64 ? 0 : 1] * small_cost < large_cost;
  }
  *small_out = small;
  for (int b = 0; b < nb; ++b) {
    const int cols = visc_cols(gs[b], small), nk = gs[b].nk;
    int c = chunk[small ? 1 : 0];
    if (batch && points >= kViscTraffic)
      for (c = kViscChunk; c > 8 && cols * ((nk + c - 1) / c) < kViscMinTilesBatch;) c /= 2;
    const int nch = (nk + c - 1) / c;
    kc[b] = (nk + nch - 1) / nch;
    tiles[b] = cols * ((nk + kc[b] - 1) / kc[b]);
  }
}

// one workgroup per tile of the concatenated list (ids remapped XCD-contiguously)
template <typename R, bool OS, bool SMALL>
__global__ __launch_bounds__(ViscTile<SMALL>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_visc_batch(const ViscArgs* __restrict__ args, TileList tl) {
  __shared__ ViscShared<R, SMALL> sh;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  int blk = 0;
  while (t >= tl.prefix[blk + 1]) ++blk;
  visc_tile<R, OS, SMALL>(args[blk], t - tl.prefix[blk], sh);
}

template <typename R, bool SMALL>
static void launch_visc_shape(const ViscArgs& a, int tiles, hipStream_t s) {
  if (a.one_sided)
    hipLaunchKernelGGL((k_visc<R, true, SMALL>), dim3(tiles), dim3(ViscTile<SMALL>::NT), 0, s, a);
  else
    hipLaunchKernelGGL((k_visc<R, false, SMALL>), dim3(tiles), dim3(ViscTile<SMALL>::NT), 0, s, a);
}

template <typename R>
hipError_t launch_visc(const ViscArgs& a, bool small, int tiles, hipStream_t s) {
  if (small)
    launch_visc_shape<R, true>(a, tiles, s);
  else
    launch_visc_shape<R, false>(a, tiles, s);
  return hipGetLastError();
}
template hipError_t launch_visc<double>(const ViscArgs&, bool, int, hipStream_t);
template hipError_t launch_visc<float>(const ViscArgs&, bool, int, hipStream_t);

template <typename R, bool SMALL>
static void launch_visc_batch_shape(const ViscArgs* args_dev, const TileList& tl, bool one_sided, hipStream_t s) {
  const dim3 grid(tl.prefix[tl.nblk]), wg(ViscTile<SMALL>::NT);
  if (one_sided)
    hipLaunchKernelGGL((k_visc_batch<R, true, SMALL>), grid, wg, 0, s, args_dev, tl);
  else
    hipLaunchKernelGGL((k_visc_batch<R, false, SMALL>), grid, wg, 0, s, args_dev, tl);
}

// small, args_dev[b].kc and the tile counts of tl must be those of visc_plan
template <typename R>
hipError_t launch_visc_batch(const ViscArgs* args_dev, const TileList& tl, bool small, bool one_sided, hipStream_t s) {
  if (small)
    launch_visc_batch_shape<R, true>(args_dev, tl, one_sided, s);
  else
    launch_visc_batch_shape<R, false>(args_dev, tl, one_sided, s);
  return hipGetLastError();
}
template hipError_t launch_visc_batch<double>(const ViscArgs*, const TileList&, bool, bool, hipStream_t);
template hipError_t launch_visc_batch<float>(const ViscArgs*, const TileList&, bool, bool, hipStream_t);

// =====================================================================================
// Direction sweep: modified AFWENO inviscid derivative (Sec. 4.5.1, Figs 10-11, Eq 19),
// the sixth-order derivative of the viscous flux, and the output (partial sum, R, or the
// RK3 stage of Eq 20).
//
// A workgroup owns a tile of TW grid lines (cross direction c1) by TS output nodes along
// the sweep direction.  It stages Q, the direction's node metrics and the viscous
// fluxes of nodes d0-3 .. d0+TS+2 in LDS; evaluates per node the characteristic WENO pair
// and the two split fluxes (nodes d0-1 .. d0+TS, one per thread) into interface fluxes;
// replaces the staged Q by the nodal fluxes; and assembles Eq 19, the viscous derivative
// and the output per output node (one per thread).
// =====================================================================================
template <int DIR, int TW>
struct LdsIdx {
  // LDS order puts the lane-fastest tile axis innermost: along the line for DIR 0
  // (lanes walk i), across lines otherwise.
  static __device__ __forceinline__ int f(int v, int w, int s, int len) {
    return DIR == 0 ? (v * TW + w) * len + s : (v * len + s) * TW + w;
  }
};

template <int TW, int TS>
struct SweepLds {
  static constexpr int NH = TS + 1;  // half points
  static constexpr int NN = TS + 6;  // nodes with a nodal flux
  static constexpr int NW = TS + 2;  // nodes with a WENO evaluation
};

// Inviscid scheme of a sweep (Sec. 4.5.1): characteristic space at the nodes (modified
// AFWENO, Figs 10-11) or at the half points (original AFWENO, Fig 9).
constexpr int kModified = 0, kOriginal = 1;

// Metrics of a sweep in mixed precision: the node metrics are staged from their FP32
// copy (every use rounds them to FP32) and the half-point metrics from the planes that
// cfd_metrics interpolated once in FP64 and rounded (the values an FP64 interpolation in
// the sweep would give, without its FP64 arithmetic in the FP32 sweeps, whose VALU issue
// is their bound).  FP64 sweeps stage the FP64 node metrics and interpolate.
template <typename R>
constexpr bool kHalfPre = sizeof(R) == 4;
template <typename R>
using StageM = typename std::conditional<kHalfPre<R>, R, double>::type;

// LDS of one workgroup for the largest tile configuration in use.  The staged Q /
// nodal-flux tile is in the compute type: an FP64 tile gives the RK combination Q_cur from
// LDS; a mixed-precision RK sweep reads Q_cur again (from L2, moments after the staging
// read it) rather than convert an FP64 tile at every use (its FP32 tile runs that sweep 3%
// faster on the 512 x 512 x 384 channel).
template <typename R, int TW, int TS>
struct SweepShared {
  R F[5 * TW * SweepLds<TW, TS>::NH];   // interface fluxes f(n+1/2)
  R Fn[5 * TW * SweepLds<TW, TS>::NN];  // staged Q, then nodal fluxes
  StageM<R> M[3 * TW * SweepLds<TW, TS>::NN];  // node metrics of the sweep direction
  R V[4 * TW * SweepLds<TW, TS>::NN];  // viscous fluxes of the direction
  R H[kHalfPre<R> ? 3 * TW * SweepLds<TW, TS>::NH : 1];  // half-point metrics (mixed precision)
};

// One tile of a direction sweep: t is the logical tile index inside the block (sweep-
// direction tile fastest, then the cross tile c1, then the cross index c2).
// OS: some block of the launch has faces with the one-sided viscous closure (a separate
// instantiation keeps the register budget of the others)
template <int DIR, typename R, int TW, int TS, int NT, int SCHEME = kModified, bool OS = false>
__device__ __forceinline__ void sweep_tile(const SweepCommon& c, const SweepBlock& b, int t,
                                           SweepShared<R, TW, TS>& sh) {
  R* const sF = sh.F;
  R* const sFn = sh.Fn;
  StageM<R>* const sM = sh.M;
  R* const sV = sh.V;
  R* const sH = sh.H;
  constexpr int NH = SweepLds<TW, TS>::NH;
  constexpr int NN = SweepLds<TW, TS>::NN;
  constexpr int NW = SweepLds<TW, TS>::NW;
  using L = LdsIdx<DIR, TW>;
  // xi tiles with 64 threads per line: a wave owns a line, reads no other wave's LDS and so
  // needs no barrier, only the order of its own LDS accesses; the waves of a workgroup drift
  // apart, which overlaps one's staging with another's arithmetic
  constexpr bool WAVE_LINE = DIR == 0 && NT == 64 * TW && NW <= 64;
  constexpr int SPAN = WAVE_LINE ? 64 : NT;  // threads that share the items of a phase
  // item e of a phase with len entries per line: its line and entry
  auto line_of = [](int e, int len) { return WAVE_LINE ? (int)(threadIdx.x >> 6) : DIR == 0 ? e / len : e % TW; };
  auto node_of = [](int e, int len) { return WAVE_LINE ? e : DIR == 0 ? e % len : e / TW; };
  constexpr int LINES = WAVE_LINE ? 1 : TW;  // lines behind the items of a phase
  const int tid = WAVE_LINE ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
  auto tile_sync = []() {
    if constexpr (WAVE_LINE) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };

  const Geom& g = b.g;
  const int nd = DIR == 0 ? g.ni : DIR == 1 ? g.nj : g.nk;
  const int n1 = DIR == 0 ? g.nj : g.ni;
  // element offsets inside one plane fit in 32 bits (checked on the host); every array
  // is addressed as a uniform plane base plus a 32-bit per-lane offset
  const uint32_t sd = DIR == 0 ? 1u : DIR == 1 ? (uint32_t)g.ld_i : (uint32_t)(g.ld_i * g.ld_j);
  const uint32_t s1 = DIR == 0 ? (uint32_t)g.ld_i : 1u;
  const uint32_t s2 = DIR == 2 ? (uint32_t)g.ld_i : (uint32_t)(g.ld_i * g.ld_j);
  const int ts = b.tile_len;  // output nodes per tile along the sweep (<= TS)
  const int nw = ts + 2;      // WENO nodes
  const int nn = ts + 6;      // nodal-flux nodes
  const int tiled = t % b.tiles_d;
  const int rest = t / b.tiles_d;
  const int tile1 = rest % b.tiles_c1;
  const int c2 = rest / b.tiles_c1;
  const int c1_0 = tile1 * TW;
  const int d0 = tiled * ts;
  // offset of (c1 = 0, c2, n = 0)
  const uint32_t origin = (uint32_t)at(g, 0, 0, 0) + (uint32_t)c2 * s2;
  const int64_t plane = g.plane;
  const GP<const double> Q = to_global(b.q);
  const GP<const double> met = to_global(b.met);
  const Gas<R> G(c.ph);
  const R eps = R(c.ph.eps);
  const bool linear = c.ph.linear != 0;
  using MT = StageM<R>;
  // node metrics of the direction (FP64, or their FP32 copy), half-point metrics (mixed)
  const GP<const MT> mbase =
      kHalfPre<R> ? (GP<const MT>)to_global(b.met_r) : (GP<const MT>)to_global(b.met);
  const GP<const MT> mx = plane_ptr(mbase, (3 * DIR + 0) * plane);
  const GP<const MT> my = plane_ptr(mbase, (3 * DIR + 1) * plane);
  const GP<const MT> mz = plane_ptr(mbase, (3 * DIR + 2) * plane);
  const GP<const float> hbase = kHalfPre<R> ? to_global(b.met_r) + (10 + 3 * DIR) * plane : nullptr;

  // ---- the output node of this thread (at most one per thread) and its global operands,
  // requested before the last barrier so that their latency overlaps the nodal-flux phase
  static_assert(LINES * TS <= SPAN, "one output node per thread");
  const GP<const R> vis = to_global(static_cast<const R*>(b.vis)) + (4 * DIR) * plane;
  const GP<const R> rin = to_global(static_cast<const R*>(b.rt_in));
  const int so = node_of(tid, TS), wo = line_of(tid, TS);
  const bool out_here = tid < LINES * TS && so < ts && c1_0 + wo < n1 && d0 + so < nd;
  const uint32_t po = origin + (uint32_t)(c1_0 + wo) * s1 + (uint32_t)(d0 + so) * sd;
  R vm[4][6];  // viscous fluxes of the direction at offsets -3, -2, -1, 1, 2, 3
  R rp[5];     // partial sums of the earlier directions
  double Jo = 0.0, qno[5], qco[5];
  auto fetch = [&]() {
    if (!out_here) return;
    if (c.do_vis && !c.do_inv) {  // else staged with the tile
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const GP<const R> vp = plane_ptr(vis, v * plane);
#pragma unroll
        for (int m = 0; m < 6; ++m) vm[v][m] = ldg(vp, po + (uint32_t)(m < 3 ? m - 3 : m - 2) * sd);
      }
    }
    if (c.has_prev) {
#pragma unroll
      for (int v = 0; v < 5; ++v) rp[v] = ldg(plane_ptr(rin, v * plane), po);
    }
    if (c.out_kind != kOutPartial) Jo = ldg(plane_ptr(met, 9 * plane), po);
    if (c.out_kind == kOutRK) {
      // Q at the output node (an inviscid FP64 sweep took it from its tile already)
      if (!(sizeof(R) == 8 && c.do_inv)) {
#pragma unroll
        for (int v = 0; v < 5; ++v) qco[v] = ldg(plane_ptr(Q, v * plane), po);
      }
      // stage 0 has Qn = Q
      if (b.qn == b.q) {
#pragma unroll
        for (int v = 0; v < 5; ++v) qno[v] = qco[v];
      } else {
        const GP<const double> qn = to_global(b.qn);
#pragma unroll
        for (int v = 0; v < 5; ++v) qno[v] = ldg(plane_ptr(qn, v * plane), po);
      }
    }
  };

  __shared__ R os_tab[OS ? 21 : 1];
  if constexpr (OS) {
    os6_stage(os_tab);
    __syncthreads();
  }
  if (c.do_inv) {
    // ---- stage Q (compute type) and the sweep direction's node metrics (FP64) of nodes
    // d0-3 .. d0+ts+2 of the tile's lines in LDS; sFn holds Q until the nodal fluxes
    // replace it.  Items are laid out with the compile-time extents NN / NW / TS so that
    // the index split needs no runtime division; slots beyond the tile's length idle.
    // A thread's items (at most ITEMS) have all their loads issued before the first LDS
    // store, so the tile waits for one memory round trip rather than one per item.
    {
      constexpr int ITEMS = (LINES * NN + SPAN - 1) / SPAN;
      double ld[ITEMS][12];  // Q, then (FP64) node metrics and viscous fluxes
      R lr[ITEMS][10];       // mixed precision: node metrics, viscous fluxes, half-point metrics
      bool ok[ITEMS], okh[ITEMS];
      int li[ITEMS], lhi[ITEMS];
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        const int e = tid + it * SPAN;
        const int s = node_of(e, NN), w = line_of(e, NN);
        const int n = d0 - 3 + s;
        const int c1 = c1_0 + w;
        ok[it] = e < LINES * NN && s < nn && c1 < n1 && n <= nd + 2;
        li[it] = L::f(0, w, s, NN);
        if (ok[it]) {
          const uint32_t p = origin + (uint32_t)c1 * s1 + (uint32_t)n * sd;
#pragma unroll
          for (int v = 0; v < 5; ++v) ld[it][v] = ldg(plane_ptr(Q, v * plane), p);
          if constexpr (kHalfPre<R>) {
            lr[it][0] = ldg(mx, p);
            lr[it][1] = ldg(my, p);
            lr[it][2] = ldg(mz, p);
            if (c.do_vis) {
#pragma unroll
              for (int v = 0; v < 4; ++v) lr[it][3 + v] = ldg(plane_ptr(vis, v * plane), p);
            }
            // the half point n+1/2 is interface slot s-2 (slots 0 .. ts, n <= nd-1)
            okh[it] = s >= 2 && s <= ts + 2 && n <= nd - 1;
            lhi[it] = L::f(0, w, s - 2, NH);
            if (okh[it]) {
#pragma unroll
              for (int v = 0; v < 3; ++v) lr[it][7 + v] = ldg(plane_ptr(hbase, v * plane), p);
            }
          } else {
            ld[it][5] = ldg(mx, p);
            ld[it][6] = ldg(my, p);
            ld[it][7] = ldg(mz, p);
            if (c.do_vis) {
#pragma unroll
              for (int v = 0; v < 4; ++v) ld[it][8 + v] = double(ldg(plane_ptr(vis, v * plane), p));
            }
          }
        }
      }
      // plane v of an LDS array starts TW*NN (TW*NH) entries after plane v-1 (both layouts)
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        if (!ok[it]) continue;
#pragma unroll
        for (int v = 0; v < 5; ++v) sFn[li[it] + v * TW * NN] = R(ld[it][v]);
        if constexpr (kHalfPre<R>) {
#pragma unroll
          for (int v = 0; v < 3; ++v) sM[li[it] + v * TW * NN] = lr[it][v];
          if (c.do_vis) {
#pragma unroll
            for (int v = 0; v < 4; ++v) sV[li[it] + v * TW * NN] = lr[it][3 + v];
          }
          if (okh[it]) {
#pragma unroll
            for (int v = 0; v < 3; ++v) sH[lhi[it] + v * TW * NH] = lr[it][7 + v];
          }
        } else {
#pragma unroll
          for (int v = 0; v < 3; ++v) sM[li[it] + v * TW * NN] = ld[it][5 + v];
          if (c.do_vis) {
#pragma unroll
            for (int v = 0; v < 4; ++v) sV[li[it] + v * TW * NN] = R(ld[it][8 + v]);
          }
        }
      }
    }
    tile_sync();
    R Fkeep[5];
    bool need_m = false;
    int ww = 0, sw_ = 0;
    if constexpr (SCHEME == kModified) {
      // ---- characteristic WENO pair and split fluxes (one node per thread); node n = d0-1+s
      // sits at staged index s+2.  F+ at n+1/2 goes to LDS now; F- at n-1/2 is added to the
      // same interface after the barrier, so sF holds f(n+1/2) = F+(n) + F-(n+1). ----------
      static_assert(LINES * NW <= SPAN, "one WENO node per thread");
      sw_ = node_of(tid, NW);
      ww = line_of(tid, NW);
      const bool wvalid = tid < LINES * NW && sw_ < nw && c1_0 + ww < n1 && d0 - 1 + sw_ <= nd;
      const bool need_p = wvalid && sw_ <= ts && d0 - 1 + sw_ <= nd - 1;  // F+ at n+1/2
      need_m = wvalid && sw_ >= 1;                                        // F- at n-1/2
      if (need_p || need_m) {
        const int s = sw_, w = ww;
        const int sc = s + 2;
        R q0[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) q0[v] = R(sFn[L::f(v, w, sc, NN)]);
        const R m0 = R(sM[L::f(0, w, sc, NN)]), m1 = R(sM[L::f(1, w, sc, NN)]), m2 = R(sM[L::f(2, w, sc, NN)]);
        if constexpr (kHalfPre<R>) {
          const Basis<R> B = make_basis(q0, m0, m1, m2, G);
          R V[5][5];  // V[t][field] at node n + t - 2
#pragma unroll
          for (int tt = 0; tt < 5; ++tt) {
            R qq[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) qq[v] = R(sFn[L::f(v, w, s + tt, NN)]);
            project(B, G, qq, V[tt]);
          }
          R vl[5], vr[5];
#pragma unroll
          for (int f = 0; f < 5; ++f)
            weno_pair<R>(V[0][f], V[1][f], V[2][f], V[3][f], V[4][f], eps, linear, vl[f], vr[f]);
          // half-point metrics from LDS: slot s holds n+1/2, slot s-1 holds n-1/2
          if (need_p) {
            R ul[5], F[5];
            unproject(B, G, vl, ul);
            const R hx = sH[L::f(0, w, s, NH)], hy = sH[L::f(1, w, s, NH)], hz = sH[L::f(2, w, s, NH)];
            sw_flux<+1>(ul, hx, hy, hz, G, F);
#pragma unroll
            for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] = F[v];
          }
          if (need_m) {
            R ur[5];
            unproject(B, G, vr, ur);
            const R hx = sH[L::f(0, w, s - 1, NH)], hy = sH[L::f(1, w, s - 1, NH)], hz = sH[L::f(2, w, s - 1, NH)];
            sw_flux<-1>(ur, hx, hy, hz, G, Fkeep);
          }
        } else {
          const NodeSpace<R> B = node_space(q0, m0, m1, m2, G);
          R D[4][5];  // projected first differences of Q along n-2 .. n+2
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) {
            R t[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) t[v] = sFn[L::f(v, w, s + tt + 1, NN)] - sFn[L::f(v, w, s + tt, NN)];
            project_diff(B, t, D[tt]);
          }
          R vl[5], vr[5];
          const R eps4 = R(4) * eps;
#pragma unroll
          for (int f = 0; f < 5; ++f) weno_diff<R>(D[0][f], D[1][f], D[2][f], D[3][f], eps4, linear, vl[f], vr[f]);
          // half-point metrics interpolated from the staged node metrics; the half point n-1/2
          // = (n-1)+1/2 is centred on staged index sc-1
          auto half = [&](int at, R h[3], R& mag, R& minv) {
#pragma unroll
            for (int d = 0; d < 3; ++d) h[d] = half_metric([&](int m) { return sM[L::f(d, w, at + m, NN)]; });
            const R hh = h[0] * h[0] + h[1] * h[1] + h[2] * h[2];
            minv = rsq(hh);
            mag = hh * minv;
          };
          R h[3], mag, minv;
          if (need_p) {
            R F[5];
            half(sc, h, mag, minv);
            half_flux<+1>(B, G, vl, h[0], h[1], h[2], mag, minv, F);
#pragma unroll
            for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] = F[v];
          }
          if (need_m) {
            half(sc - 1, h, mag, minv);
            half_flux<-1>(B, G, vr, h[0], h[1], h[2], mag, minv, Fkeep);
          }
        }
      }
    } else {
      // ---- original AFWENO: one half point per thread.  Slot s holds n+1/2 with
      // n = d0-1+s (staged index s+2), whose stencil is staged s .. s+5.  The
      // characteristic space sits at the half point: the mean state of n and n+1 and the
      // direction of the half-point metric; the value left of n+1/2 comes from nodes
      // n-2..n+2, the value right of it from n-1..n+3, and f(n+1/2) = F+ + F- directly.
      static_assert(LINES * NH <= SPAN, "one half point per thread");
      const int s = node_of(tid, NH), w = line_of(tid, NH);
      if (tid < LINES * NH && s <= ts && c1_0 + w < n1 && d0 - 1 + s <= nd - 1) {
        const int sc = s + 2;
        R qa[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) qa[v] = R(0.5) * (R(sFn[L::f(v, w, sc, NN)]) + R(sFn[L::f(v, w, sc + 1, NN)]));
        // this thread alone writes slot s: F+ goes to LDS, F- is added to it
        if constexpr (kHalfPre<R>) {
          auto hm = [&](int c) { return sH[L::f(c, w, s, NH)]; };
          const Basis<R> B = make_basis(qa, hm(0), hm(1), hm(2), G);
          // V[t][field] at node n + t - 2; node n+3 replaces node n-2 once the left value is
          // formed, which keeps five stencil points live instead of six
          R V[5][5];
          auto proj = [&](int tt, R out[5]) {
            R qq[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) qq[v] = R(sFn[L::f(v, w, s + tt, NN)]);
            project(B, G, qq, out);
          };
#pragma unroll
          for (int tt = 0; tt < 5; ++tt) proj(tt, V[tt]);
          R vl[5], vr[5], uh[5], F[5];
#pragma unroll
          for (int f = 0; f < 5; ++f) vl[f] = weno_left(V[0][f], V[1][f], V[2][f], V[3][f], V[4][f], eps, linear);
          proj(5, V[0]);
#pragma unroll
          for (int f = 0; f < 5; ++f) vr[f] = weno_left(V[0][f], V[4][f], V[3][f], V[2][f], V[1][f], eps, linear);
          unproject(B, G, vl, uh);
          sw_flux<+1>(uh, hm(0), hm(1), hm(2), G, F);
#pragma unroll
          for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] = F[v];
          unproject(B, G, vr, uh);
          sw_flux<-1>(uh, hm(0), hm(1), hm(2), G, F);
#pragma unroll
          for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] += F[v];
        } else {
          R h[3];
#pragma unroll
          for (int d = 0; d < 3; ++d) h[d] = half_metric([&](int m) { return sM[L::f(d, w, sc + m, NN)]; });
          const NodeSpace<R> B = node_space(qa, h[0], h[1], h[2], G);
          R D[5][5];  // projected first differences of Q along n-2 .. n+3
#pragma unroll
          for (int tt = 0; tt < 5; ++tt) {
            R t[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) t[v] = sFn[L::f(v, w, s + tt + 1, NN)] - sFn[L::f(v, w, s + tt, NN)];
            project_diff(B, t, D[tt]);
          }
          R vl[5], vr[5], q[5], u[5], F[5];
          const R eps4 = R(4) * eps;
#pragma unroll
          for (int f = 0; f < 5; ++f) {
            vl[f] = weno_left_diff(D[0][f], D[1][f], D[2][f], D[3][f], eps4, linear);
            vr[f] = weno_left_diff(-D[4][f], -D[3][f], -D[2][f], -D[1][f], eps4, linear);
          }
          const R hh = h[0] * h[0] + h[1] * h[1] + h[2] * h[2];
          const R minv = rsq(hh), mag = hh * minv;
#pragma unroll
          for (int v = 0; v < 5; ++v) q[v] = sFn[L::f(v, w, sc, NN)];
          unproject_diff(B, G, vl, q, u);
          state_flux<+1>(u, G, h[0], h[1], h[2], mag, minv, F);
#pragma unroll
          for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] = F[v];
#pragma unroll
          for (int v = 0; v < 5; ++v) q[v] = sFn[L::f(v, w, sc + 1, NN)];
          unproject_diff(B, G, vr, q, u);
          state_flux<-1>(u, G, h[0], h[1], h[2], mag, minv, F);
#pragma unroll
          for (int v = 0; v < 5; ++v) sF[L::f(v, w, s, NH)] += F[v];
        }
      }
    }
    // a staged Q in FP64 is exact: the output node's copy for the RK combination is read
    // here, before the barrier after which the nodal fluxes overwrite it
    if (sizeof(R) == 8 && c.out_kind == kOutRK && out_here) {
#pragma unroll
      for (int v = 0; v < 5; ++v) qco[v] = double(sFn[L::f(v, wo, so + 3, NN)]);
    }
    tile_sync();
    if (need_m) {  // each interface receives exactly one F-
#pragma unroll
      for (int v = 0; v < 5; ++v) sF[L::f(v, ww, sw_ - 1, NH)] += Fkeep[v];
    }
    fetch();
    // ---- nodal fluxes, Eq 4, in place of the staged Q ------------------------------------
    for (int e = tid; e < LINES * NN; e += SPAN) {
      const int s = node_of(e, NN), w = line_of(e, NN);
      const int n = d0 - 3 + s;
      const int c1 = c1_0 + w;
      if (s >= nn || c1 >= n1 || n > nd + 2) continue;
      R q[5], F[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) q[v] = R(sFn[L::f(v, w, s, NN)]);
      phys_flux(q, R(sM[L::f(0, w, s, NN)]), R(sM[L::f(1, w, s, NN)]), R(sM[L::f(2, w, s, NN)]), G, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) sFn[L::f(v, w, s, NN)] = F[v];
    }
    tile_sync();
  }

  // ---- assembly at the output node ------------------------------------------------------
  if (!c.do_inv) fetch();
  if (!out_here) return;
  const int s = so, w = wo;
  R r[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) r[v] = R(0);
  if (c.do_inv) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const R fp = sF[L::f(v, w, s + 1, NH)];
      const R fm = sF[L::f(v, w, s, NH)];
      auto fn = [&](int m) { return R(sFn[L::f(v, w, s + m, NN)]); };
      const R D = fp - fm + R(17.0 / 256.0) * (fn(4) - fn(2)) - R(13.0 / 320.0) * (fn(5) - fn(1)) +
                  R(19.0 / 3840.0) * (fn(6) - fn(0));
      r[v] = -D;
    }
  }
  if (c.do_vis) {
    int first = 0, row = 0, sign = 0;
    if (OS && one_sided_window((b.one_sided >> (2 * DIR)) & 3, d0 + s, nd, &first, &row, &sign)) {
      // a node next to a one-sided face: seven-point one-sided derivative over the nodes
      // nearest the face, from the staged tile where it holds them (all but a last tile of
      // fewer than four nodes), else from memory
      R acc[4] = {R(0), R(0), R(0), R(0)};
      const int at0 = first - (d0 - 3);  // staged index of the window
      if (c.do_inv && at0 >= 0 && at0 + 6 < nn) {
#pragma unroll 1
        for (int m = 0; m < 7; ++m) {
          const R wgt = os6_weight(os_tab, row, sign, m);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[v] += wgt * sV[L::f(v, w, at0 + m, NN)];
        }
      } else {
#pragma unroll 1
        for (int m = 0; m < 7; ++m) {
          const R wgt = os6_weight(os_tab, row, sign, m);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            acc[v] += wgt * ldg(plane_ptr(vis, v * plane), po + (uint32_t)(first + m - d0 - s) * sd);
        }
      }
#pragma unroll
      for (int v = 1; v < 5; ++v) r[v] += acc[v - 1];
    } else if (c.do_inv) {
#pragma unroll
      for (int v = 1; v < 5; ++v) r[v] += d6<R>([&](int m) { return sV[L::f(v - 1, w, s + 3 + m, NN)]; });
    } else {
#pragma unroll
      for (int v = 1; v < 5; ++v) r[v] += d6<R>([&](int m) { return vm[v - 1][m < 0 ? m + 3 : m + 2]; });
    }
  }
  if (c.has_prev) {
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] += rp[v];
  }
  if (c.out_kind == kOutPartial) {
    const GP<R> ro = to_global(static_cast<R*>(b.rt_out));
#pragma unroll
    for (int v = 0; v < 5; ++v) stg(plane_ptr(ro, v * plane), po, r[v]);
  } else {
    const GP<double> out = to_global(b.out);
    if (c.out_kind == kOutRhs) {
#pragma unroll
      for (int v = 0; v < 5; ++v) stg(plane_ptr(out, v * plane), po, Jo * double(r[v]));
    } else {
      // local time stepping reads the point's own step here rather than with the other
      // operands: the common scalar-step path keeps its register budget
      const double dt = b.dt_field ? ldg(to_global(b.dt_field), po) : c.dt_dev ? *c.dt_dev : c.dt;
      const double cdt = c.cc * dt * Jo;
#pragma unroll
      for (int v = 0; v < 5; ++v) stg(plane_ptr(out, v * plane), po, c.ca * qno[v] + c.cb * qco[v] + cdt * double(r[v]));
    }
  }
}

// Single block: one workgroup per tile, ids remapped XCD-contiguously.
template <int DIR, typename R, int TW, int TS, int NT, int SCHEME, bool OS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_sweep(SweepArgs a) {
  __shared__ SweepShared<R, TW, TS> sh;
  sweep_tile<DIR, R, TW, TS, NT, SCHEME, OS>(a.c, a.b, xcd_remap(blockIdx.x, gridDim.x), sh);
}
// the original scheme in FP64 holds five projected differences and the half-point basis at
// once (141-160 VGPRs): three waves per SIMD give it what four would make it spill
template <int DIR, typename R, int TW, int TS, int NT, bool OS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void k_sweep_w3(SweepArgs a) {
  __shared__ SweepShared<R, TW, TS> sh;
  sweep_tile<DIR, R, TW, TS, NT, kOriginal, OS>(a.c, a.b, xcd_remap(blockIdx.x, gridDim.x), sh);
}

// Batched blocks: one launch walks a work list covering the tiles of every block
// (prefix[b] = first tile of block b).  The list is split into eight contiguous ranges, one
// per XCD.  PERSIST: a fixed grid of workgroups strides through its XCD's range; otherwise
// one workgroup per tile (ids remapped XCD-contiguously).  Blocks with one-sided faces (OS)
// run one workgroup per tile.
template <int DIR, typename R, int TW, int TS, int NT, bool PERSIST, bool OS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(PERSIST && sizeof(R) == 8 ? 3 : 4))) void k_sweep_batch(
    const SweepBlock* __restrict__ blocks, SweepCommon c, TileList tl) {
  __shared__ SweepShared<R, TW, TS> sh;
  const int total = tl.prefix[tl.nblk];
  if (!PERSIST) {
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    int blk = 0;
    while (t >= tl.prefix[blk + 1]) ++blk;
    sweep_tile<DIR, R, TW, TS, NT, kModified, OS>(c, blocks[blk], t - tl.prefix[blk], sh);
    return;
  }
  static_assert(!(PERSIST && OS), "the persistent schedule is not built for one-sided closures");
  int start, count, lane_wg, nwg_x;
  xcd_range(total, &start, &count, &lane_wg, &nwg_x);
  int blk = 0;
  for (int u = lane_wg; u < count; u += nwg_x) {
    const int t = start + u;
    while (t >= tl.prefix[blk + 1]) ++blk;  // t only grows, so the scan resumes
    sweep_tile<DIR, R, TW, TS, NT>(c, blocks[blk], t - tl.prefix[blk], sh);
    __syncthreads();  // the next tile overwrites the LDS this one read
  }
}

// Batched original-scheme sweep (one workgroup per tile).  FP64 gets three waves per SIMD
// (see k_sweep_w3), FP32 the usual four.
template <int DIR, typename R, int TW, int TS, int NT, bool OS>
__device__ __forceinline__ void batch_orig_tile(const SweepBlock* __restrict__ blocks, const SweepCommon& c,
                                                const TileList& tl, SweepShared<R, TW, TS>& sh) {
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  int blk = 0;
  while (t >= tl.prefix[blk + 1]) ++blk;
  sweep_tile<DIR, R, TW, TS, NT, kOriginal, OS>(c, blocks[blk], t - tl.prefix[blk], sh);
}
template <int DIR, typename R, int TW, int TS, int NT, bool OS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 3 : 4))) void k_sweep_batch_orig(
    const SweepBlock* __restrict__ blocks, SweepCommon c, TileList tl) {
  __shared__ SweepShared<R, TW, TS> sh;
  batch_orig_tile<DIR, R, TW, TS, NT, OS>(blocks, c, tl, sh);
}

// tile configurations (lines across x nodes along the sweep x threads)
template <int CFG>
struct TileCfg;
template <>
struct TileCfg<0> {
  static constexpr int TW = 16, TS = 30, NT = 512;
};
template <>
struct TileCfg<1> {
  static constexpr int TW = 32, TS = 14, NT = 512;
};
template <>
struct TileCfg<2> {
  static constexpr int TW = 16, TS = 14, NT = 256;
};
template <>
struct TileCfg<3> {
  static constexpr int TW = 8, TS = 62, NT = 512;
};
template <>
struct TileCfg<4> {
  static constexpr int TW = 8, TS = 26, NT = 256;
};
template <>
struct TileCfg<5> {
  static constexpr int TW = 4, TS = 58, NT = 256;
};
// shapes whose WENO nodes (lines x (nodes + 2)) fill the 256 threads exactly
template <>
struct TileCfg<6> {
  static constexpr int TW = 8, TS = 30, NT = 256;
};
template <>
struct TileCfg<7> {
  static constexpr int TW = 4, TS = 62, NT = 256;
};

void sweep_tiling(int dir, int cfg, const Geom& g, int* tiles_c1, int* tiles_d, int* tile_len) {
  static const int tw[kTileCfgs] = {TileCfg<0>::TW, TileCfg<1>::TW, TileCfg<2>::TW,
                                    TileCfg<3>::TW, TileCfg<4>::TW, TileCfg<5>::TW,
                                    TileCfg<6>::TW, TileCfg<7>::TW};
  static const int tsz[kTileCfgs] = {TileCfg<0>::TS, TileCfg<1>::TS, TileCfg<2>::TS,
                                     TileCfg<3>::TS, TileCfg<4>::TS, TileCfg<5>::TS,
                                     TileCfg<6>::TS, TileCfg<7>::TS};
  const int nd = dir == 0 ? g.ni : dir == 1 ? g.nj : g.nk;
  const int n1 = dir == 0 ? g.nj : g.ni;
  *tiles_c1 = (n1 + tw[cfg] - 1) / tw[cfg];
  *tiles_d = (nd + tsz[cfg] - 1) / tsz[cfg];
  *tile_len = (nd + *tiles_d - 1) / *tiles_d;  // balanced tiles along the sweep
}

void tile_shape(int cfg, int* tw, int* ts, int* nt) {
  static const int w[kTileCfgs] = {TileCfg<0>::TW, TileCfg<1>::TW, TileCfg<2>::TW,
                                   TileCfg<3>::TW, TileCfg<4>::TW, TileCfg<5>::TW,
                                   TileCfg<6>::TW, TileCfg<7>::TW};
  static const int l[kTileCfgs] = {TileCfg<0>::TS, TileCfg<1>::TS, TileCfg<2>::TS,
                                   TileCfg<3>::TS, TileCfg<4>::TS, TileCfg<5>::TS,
                                   TileCfg<6>::TS, TileCfg<7>::TS};
  *tw = w[cfg];
  *ts = l[cfg];
  *nt = sweep_threads(cfg);
}

int sweep_threads(int cfg) {
  static const int nt[kTileCfgs] = {TileCfg<0>::NT, TileCfg<1>::NT, TileCfg<2>::NT,
                                    TileCfg<3>::NT, TileCfg<4>::NT, TileCfg<5>::NT,
                                    TileCfg<6>::NT, TileCfg<7>::NT};
  return nt[cfg];
}

template <typename R, int CFG, int SCHEME, bool OS>
hipError_t launch_sweep_scheme(int dir, const SweepArgs& a, int64_t nwg, hipStream_t s) {
  using C = TileCfg<CFG>;
  dim3 grid((unsigned)nwg);
  if constexpr (SCHEME == kOriginal && sizeof(R) == 8) {
    if (dir == 0)
      hipLaunchKernelGGL((k_sweep_w3<0, R, C::TW, C::TS, C::NT, OS>), grid, dim3(C::NT), 0, s, a);
    else if (dir == 1)
      hipLaunchKernelGGL((k_sweep_w3<1, R, C::TW, C::TS, C::NT, OS>), grid, dim3(C::NT), 0, s, a);
    else
      hipLaunchKernelGGL((k_sweep_w3<2, R, C::TW, C::TS, C::NT, OS>), grid, dim3(C::NT), 0, s, a);
    return hipGetLastError();
  } else {
    if (dir == 0)
      hipLaunchKernelGGL((k_sweep<0, R, C::TW, C::TS, C::NT, SCHEME, OS>), grid, dim3(C::NT), 0, s, a);
    else if (dir == 1)
      hipLaunchKernelGGL((k_sweep<1, R, C::TW, C::TS, C::NT, SCHEME, OS>), grid, dim3(C::NT), 0, s, a);
    else
      hipLaunchKernelGGL((k_sweep<2, R, C::TW, C::TS, C::NT, SCHEME, OS>), grid, dim3(C::NT), 0, s, a);
    return hipGetLastError();
  }
}

template <typename R, int CFG>
hipError_t launch_sweep_cfg(int dir, const SweepArgs& a, int64_t nwg, hipStream_t s) {
  const bool os = (a.b.one_sided >> (2 * dir)) & 3;  // the closure acts on faces across the sweep
  if (a.c.ph.scheme == kOriginal)
    return os ? launch_sweep_scheme<R, CFG, kOriginal, true>(dir, a, nwg, s)
              : launch_sweep_scheme<R, CFG, kOriginal, false>(dir, a, nwg, s);
  return os ? launch_sweep_scheme<R, CFG, kModified, true>(dir, a, nwg, s)
            : launch_sweep_scheme<R, CFG, kModified, false>(dir, a, nwg, s);
}

// FP64 xi sweep with a workgroup of one wave per line of up to 58 nodes: the wave-per-line tile
// (4 x 58) without three neighbours whose LDS and registers wait for the slowest of the four.
// xi + RK sweep, 4 x 58 / one line: 128^3 122 / 117 us, 160^3 218 / 201, 256^3 862 / 835,
// 512 x 512 x 384 4.95 / 4.83 ms (5.28 before waves owned lines).
constexpr int kRowNodes = 58;

hipError_t launch_sweep_rows(SweepArgs a, hipStream_t s) {
  const Geom& g = a.b.g;
  a.b.tiles_c1 = g.nj;
  a.b.tiles_d = (g.ni + kRowNodes - 1) / kRowNodes;
  a.b.tile_len = (g.ni + a.b.tiles_d - 1) / a.b.tiles_d;
  const int64_t nwg = (int64_t)a.b.tiles_c1 * a.b.tiles_d * g.nk;
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nwg), wg(64);
  const bool os = a.b.one_sided & 3;
  if (a.c.ph.scheme == kOriginal) {
    if (os)
      hipLaunchKernelGGL((k_sweep_w3<0, double, 1, kRowNodes, 64, true>), grid, wg, 0, s, a);
    else
      hipLaunchKernelGGL((k_sweep_w3<0, double, 1, kRowNodes, 64, false>), grid, wg, 0, s, a);
  } else if (os) {
    hipLaunchKernelGGL((k_sweep<0, double, 1, kRowNodes, 64, kModified, true>), grid, wg, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_sweep<0, double, 1, kRowNodes, 64, kModified, false>), grid, wg, 0, s, a);
  }
  return hipGetLastError();
}

template <typename R>
hipError_t launch_sweep(int dir, SweepArgs a, hipStream_t s, int cfg) {
  const int n2 = dir == 2 ? a.b.g.nj : a.b.g.nk;
  sweep_tiling(dir, cfg, a.b.g, &a.b.tiles_c1, &a.b.tiles_d, &a.b.tile_len);
  const int64_t nwg = (int64_t)a.b.tiles_c1 * a.b.tiles_d * n2;
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  switch (cfg) {
    case 0: return launch_sweep_cfg<R, 0>(dir, a, nwg, s);
    case 1: return launch_sweep_cfg<R, 1>(dir, a, nwg, s);
    case 2: return launch_sweep_cfg<R, 2>(dir, a, nwg, s);
    case 3: return launch_sweep_cfg<R, 3>(dir, a, nwg, s);
    case 4: return launch_sweep_cfg<R, 4>(dir, a, nwg, s);
    case 5: return launch_sweep_cfg<R, 5>(dir, a, nwg, s);
    case 6: return launch_sweep_cfg<R, 6>(dir, a, nwg, s);
    case 7: return launch_sweep_cfg<R, 7>(dir, a, nwg, s);
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_sweep<double>(int, SweepArgs, hipStream_t, int);
template hipError_t launch_sweep<float>(int, SweepArgs, hipStream_t, int);

template <typename R, int CFG, bool P, bool OS>
hipError_t launch_sweep_batch_os(int dir, const SweepBlock* blocks, const SweepCommon& c, const TileList& tl, int nwg,
                                 hipStream_t s) {
  using C = TileCfg<CFG>;
  if (c.ph.scheme == kOriginal) {
    // the original scheme runs one workgroup per tile (the persistent schedule is not built
    // for it); in FP64 at three waves per SIMD like its single-block kernels
    if (P) return hipErrorInvalidValue;
    if (dir == 0)
      hipLaunchKernelGGL((k_sweep_batch_orig<0, R, C::TW, C::TS, C::NT, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    else if (dir == 1)
      hipLaunchKernelGGL((k_sweep_batch_orig<1, R, C::TW, C::TS, C::NT, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    else
      hipLaunchKernelGGL((k_sweep_batch_orig<2, R, C::TW, C::TS, C::NT, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    return hipGetLastError();
  }
  if constexpr (P && OS) {
    return hipErrorInvalidValue;
  } else {
    if (dir == 0)
      hipLaunchKernelGGL((k_sweep_batch<0, R, C::TW, C::TS, C::NT, P, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    else if (dir == 1)
      hipLaunchKernelGGL((k_sweep_batch<1, R, C::TW, C::TS, C::NT, P, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    else
      hipLaunchKernelGGL((k_sweep_batch<2, R, C::TW, C::TS, C::NT, P, OS>), dim3(nwg), dim3(C::NT), 0, s, blocks, c, tl);
    return hipGetLastError();
  }
}
template <typename R, int CFG, bool P>
hipError_t launch_sweep_batch_cfg(int dir, const SweepBlock* blocks, const SweepCommon& c, const TileList& tl, int nwg,
                                  hipStream_t s) {
  return c.one_sided ? launch_sweep_batch_os<R, CFG, P, true>(dir, blocks, c, tl, nwg, s)
                     : launch_sweep_batch_os<R, CFG, P, false>(dir, blocks, c, tl, nwg, s);
}

// persist: nwg workgroups stride through the list; otherwise nwg must equal the tile count
template <typename R>
hipError_t launch_sweep_batch(int dir, int cfg, bool persist, const SweepBlock* blocks, const SweepCommon& c,
                              const TileList& tl, int nwg, hipStream_t s) {
  if (persist) {
    switch (cfg) {
      case 0: return launch_sweep_batch_cfg<R, 0, true>(dir, blocks, c, tl, nwg, s);
      case 1: return launch_sweep_batch_cfg<R, 1, true>(dir, blocks, c, tl, nwg, s);
      case 2: return launch_sweep_batch_cfg<R, 2, true>(dir, blocks, c, tl, nwg, s);
      case 3: return launch_sweep_batch_cfg<R, 3, true>(dir, blocks, c, tl, nwg, s);
      case 4: return launch_sweep_batch_cfg<R, 4, true>(dir, blocks, c, tl, nwg, s);
      case 5: return launch_sweep_batch_cfg<R, 5, true>(dir, blocks, c, tl, nwg, s);
      case 6: return launch_sweep_batch_cfg<R, 6, true>(dir, blocks, c, tl, nwg, s);
      case 7: return launch_sweep_batch_cfg<R, 7, true>(dir, blocks, c, tl, nwg, s);
    }
  } else {
    switch (cfg) {
      case 0: return launch_sweep_batch_cfg<R, 0, false>(dir, blocks, c, tl, nwg, s);
      case 1: return launch_sweep_batch_cfg<R, 1, false>(dir, blocks, c, tl, nwg, s);
      case 2: return launch_sweep_batch_cfg<R, 2, false>(dir, blocks, c, tl, nwg, s);
      case 3: return launch_sweep_batch_cfg<R, 3, false>(dir, blocks, c, tl, nwg, s);
      case 4: return launch_sweep_batch_cfg<R, 4, false>(dir, blocks, c, tl, nwg, s);
      case 5: return launch_sweep_batch_cfg<R, 5, false>(dir, blocks, c, tl, nwg, s);
      case 6: return launch_sweep_batch_cfg<R, 6, false>(dir, blocks, c, tl, nwg, s);
      case 7: return launch_sweep_batch_cfg<R, 7, false>(dir, blocks, c, tl, nwg, s);
    }
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_sweep_batch<double>(int, int, bool, const SweepBlock*, const SweepCommon&, const TileList&, int,
                                               hipStream_t);
template hipError_t launch_sweep_batch<float>(int, int, bool, const SweepBlock*, const SweepCommon&, const TileList&, int,
                                              hipStream_t);

// =====================================================================================
// Small blocks: the viscous prepass and the three direction sweeps in one launch.  The
// inviscid partial sums are independent of each other and of the viscous fluxes, so one grid
// covers the tiles of the prepass, then of zeta, eta and xi, each direction writing its own
// five planes; a second launch adds the derivative of the viscous flux to each and then the
// three, in the order of the sequential sweeps, and writes R or the RK stage.  Two dependent
// launches instead of four, with all their workgroups at once for blocks that do not fill the
// chip: a launch that waits for another costs 3-4 us before its own work, and a sweep of 32^3
// takes 6-7 us with that.  Where the fluxes exist already (the split form), the sweeps take
// them as usual (WITH_VISC false in both kernels).
// =====================================================================================
template <typename R>
constexpr int kAllTW = sizeof(R) == 8 ? 8 : 16;  // eta and zeta tiles (configurations 6 and 2)
template <typename R>
constexpr int kAllTS = sizeof(R) == 8 ? 30 : 14;
constexpr int kAllNT = 256;

template <typename R>
union AllShared {
  ViscShared<R, true> visc;
  SweepShared<R, 4, 58> xi;  // configuration 5
  SweepShared<R, kAllTW<R>, kAllTS<R>> across;
};

// a.b[d]: arguments and tiling of direction d; the prepass has tiles [0, nv), zeta the next nz,
// eta the next ne
template <typename R, bool WITH_VISC>
__global__ __launch_bounds__(kAllNT) __attribute__((amdgpu_waves_per_eu(4))) void k_sweep_all(
    ViscArgs va, SweepCommon c, AllBlocks a, int nv, int nz, int ne) {
  __shared__ AllShared<R> sh;
  int t = blockIdx.x;
  if (WITH_VISC && t < nv) {
    visc_tile<R, false, true>(va, xcd_remap(t, nv), sh.visc);
    return;
  }
  t -= nv;
  if (t < nz)
    sweep_tile<2, R, kAllTW<R>, kAllTS<R>, kAllNT>(c, a.b[2], xcd_remap(t, nz), sh.across);
  else if (t < nz + ne)
    sweep_tile<1, R, kAllTW<R>, kAllTS<R>, kAllNT>(c, a.b[1], xcd_remap(t - nz, ne), sh.across);
  else
    sweep_tile<0, R, 4, 58, kAllNT>(c, a.b[0], xcd_remap(t - nz - ne, gridDim.x - nv - nz - ne), sh.xi);
}

// The same over every block of a batch: nb xi blocks, then nb eta, then nb zeta.
struct AllLists {
  TileList v, z, e, x;  // prepass, zeta, eta, xi
};
template <typename R, bool WITH_VISC>
__global__ __launch_bounds__(kAllNT) __attribute__((amdgpu_waves_per_eu(4))) void k_sweep_all_batch(
    const ViscArgs* __restrict__ va, const SweepBlock* __restrict__ blocks, SweepCommon c, AllLists tl) {
  __shared__ AllShared<R> sh;
  const int nb = tl.x.nblk, nv = WITH_VISC ? tl.v.prefix[nb] : 0, nz = tl.z.prefix[nb], ne = tl.e.prefix[nb];
  int t = blockIdx.x, blk = 0;
  if (WITH_VISC && t < nv) {
    while (t >= tl.v.prefix[blk + 1]) ++blk;
    visc_tile<R, false, true>(va[blk], t - tl.v.prefix[blk], sh.visc);
    return;
  }
  t -= nv;
  if (t < nz) {
    while (t >= tl.z.prefix[blk + 1]) ++blk;
    sweep_tile<2, R, kAllTW<R>, kAllTS<R>, kAllNT>(c, blocks[2 * nb + blk], t - tl.z.prefix[blk], sh.across);
  } else if (t < nz + ne) {
    t -= nz;
    while (t >= tl.e.prefix[blk + 1]) ++blk;
    sweep_tile<1, R, kAllTW<R>, kAllTS<R>, kAllNT>(c, blocks[nb + blk], t - tl.e.prefix[blk], sh.across);
  } else {
    t -= nz + ne;
    while (t >= tl.x.prefix[blk + 1]) ++blk;
    sweep_tile<0, R, 4, 58, kAllNT>(c, blocks[blk], t - tl.x.prefix[blk], sh.xi);
  }
}

// R or the RK stage from the three partial sums (b: the xi block; rt: zeta's five planes, then
// eta's, then xi's); WITH_VISC: those are inviscid and the derivatives of the viscous fluxes
// are added here
template <typename R, bool WITH_VISC>
__device__ __forceinline__ void combine_block(const SweepCommon& c, const SweepBlock& b) {
  const Geom& g = b.g;
  const GP<const R> rt = (GP<const R>)to_global(static_cast<const R*>(b.rt_in));
  const int total = g.ni * g.nj * g.nk;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int i = e % g.ni, jk = e / g.ni;
    const uint32_t p = (uint32_t)at(g, i, jk % g.nj, jk / g.nj);
    R part[3][5], r[5];  // zeta, eta, xi
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int v = 0; v < 5; ++v) part[d][v] = ldg(plane_ptr(rt, (5 * d + v) * g.plane), p);
    if constexpr (WITH_VISC) {
      const GP<const R> vis = to_global(static_cast<const R*>(b.vis));
      const uint32_t st[3] = {(uint32_t)(g.ld_i * g.ld_j), (uint32_t)g.ld_i, 1u};
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = 1; v < 5; ++v) {
          const GP<const R> vp = plane_ptr(vis, (4 * (2 - d) + v - 1) * g.plane);
          part[d][v] += d6<R>([&](int m) { return ldg(vp, p + (uint32_t)m * st[d]); });
        }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] = part[2][v] + (part[1][v] + part[0][v]);
    const double Jo = ldg(plane_ptr(to_global(b.met), 9 * g.plane), p);
    const GP<double> out = to_global(b.out);
    if (c.out_kind == kOutRhs) {
#pragma unroll
      for (int v = 0; v < 5; ++v) stg(plane_ptr(out, v * g.plane), p, Jo * double(r[v]));
    } else {
      double qno[5], qco[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        qco[v] = ldg(plane_ptr(to_global(b.q), v * g.plane), p);
        qno[v] = b.qn == b.q ? qco[v] : ldg(plane_ptr(to_global(b.qn), v * g.plane), p);
      }
      const double dt = b.dt_field ? ldg(to_global(b.dt_field), p) : c.dt_dev ? *c.dt_dev : c.dt;
      const double cdt = c.cc * dt * Jo;
#pragma unroll
      for (int v = 0; v < 5; ++v) stg(plane_ptr(out, v * g.plane), p, c.ca * qno[v] + c.cb * qco[v] + cdt * double(r[v]));
    }
  }
}
template <typename R, bool WITH_VISC>
__global__ __launch_bounds__(256) void k_combine(SweepCommon c, SweepBlock b) {
  combine_block<R, WITH_VISC>(c, b);
}
template <typename R, bool WITH_VISC>
__global__ __launch_bounds__(256) void k_combine_batch(const SweepBlock* __restrict__ blocks, SweepCommon c) {
  combine_block<R, WITH_VISC>(c, blocks[blockIdx.y]);
}

template <typename R>
hipError_t launch_sweep_all(const ViscArgs* visc, int nv, const SweepArgs& a, hipStream_t s) {
  const Geom& g = a.b.g;
  ViscArgs va{};
  if (visc)
    va = *visc;
  else
    nv = 0;
  SweepCommon part = a.c;
  part.has_prev = 0;
  part.out_kind = kOutPartial;
  if (visc) part.do_vis = 0;
  AllBlocks all;
  int n[3];
  for (int d = 0; d < 3; ++d) {
    SweepBlock& b = all.b[d] = a.b;
    sweep_tiling(d, kAllCfg[sizeof(R) == 8 ? 0 : 1][d], g, &b.tiles_c1, &b.tiles_d, &b.tile_len);
    n[d] = b.tiles_c1 * b.tiles_d * (d == 2 ? g.nj : g.nk);
    b.rt_out = static_cast<R*>(a.b.rt_out) + (2 - d) * 5 * g.plane;
  }
  const dim3 grid(nv + n[0] + n[1] + n[2]), wg(kAllNT);
  if (visc)
    hipLaunchKernelGGL((k_sweep_all<R, true>), grid, wg, 0, s, va, part, all, nv, n[2], n[1]);
  else
    hipLaunchKernelGGL((k_sweep_all<R, false>), grid, wg, 0, s, va, part, all, nv, n[2], n[1]);
  return hipGetLastError();
}
template hipError_t launch_sweep_all<double>(const ViscArgs*, int, const SweepArgs&, hipStream_t);
template hipError_t launch_sweep_all<float>(const ViscArgs*, int, const SweepArgs&, hipStream_t);

template <typename R>
hipError_t launch_combine(bool with_visc, const SweepArgs& a, hipStream_t s) {
  const dim3 grid((a.b.g.ni * a.b.g.nj * a.b.g.nk + 255) / 256), wg(256);
  if (with_visc)
    hipLaunchKernelGGL((k_combine<R, true>), grid, wg, 0, s, a.c, a.b);
  else
    hipLaunchKernelGGL((k_combine<R, false>), grid, wg, 0, s, a.c, a.b);
  return hipGetLastError();
}
template hipError_t launch_combine<double>(bool, const SweepArgs&, hipStream_t);
template hipError_t launch_combine<float>(bool, const SweepArgs&, hipStream_t);

template <typename R>
hipError_t launch_sweep_all_batch(const ViscArgs* visc, const TileList* visc_tl, const SweepBlock* blocks,
                                  const SweepCommon& c, const TileList tl[3], hipStream_t s) {
  const int nb = tl[0].nblk;
  SweepCommon part = c;
  part.has_prev = 0;
  part.out_kind = kOutPartial;
  AllLists l{};
  l.x = tl[0];
  l.e = tl[1];
  l.z = tl[2];
  const int n = tl[0].prefix[nb] + tl[1].prefix[nb] + tl[2].prefix[nb];
  if (visc) {
    part.do_vis = 0;
    l.v = *visc_tl;
    hipLaunchKernelGGL((k_sweep_all_batch<R, true>), dim3(l.v.prefix[nb] + n), dim3(kAllNT), 0, s, visc, blocks, part, l);
  } else {
    hipLaunchKernelGGL((k_sweep_all_batch<R, false>), dim3(n), dim3(kAllNT), 0, s, visc, blocks, part, l);
  }
  return hipGetLastError();
}
template hipError_t launch_sweep_all_batch<double>(const ViscArgs*, const TileList*, const SweepBlock*, const SweepCommon&,
                                                   const TileList[3], hipStream_t);
template hipError_t launch_sweep_all_batch<float>(const ViscArgs*, const TileList*, const SweepBlock*, const SweepCommon&,
                                                  const TileList[3], hipStream_t);

template <typename R>
hipError_t launch_combine_batch(bool with_visc, const SweepBlock* blocks, const SweepCommon& c, int nb, int max_points,
                                hipStream_t s) {
  const dim3 grid((max_points + 255) / 256, nb), wg(256);
  if (with_visc)
    hipLaunchKernelGGL((k_combine_batch<R, true>), grid, wg, 0, s, blocks, c);
  else
    hipLaunchKernelGGL((k_combine_batch<R, false>), grid, wg, 0, s, blocks, c);
  return hipGetLastError();
}
template hipError_t launch_combine_batch<double>(bool, const SweepBlock*, const SweepCommon&, int, int, hipStream_t);
template hipError_t launch_combine_batch<float>(bool, const SweepBlock*, const SweepCommon&, int, int, hipStream_t);

// =====================================================================================
// Marching sweep (FP64, eta and zeta, partial sums): one thread per grid line, lanes along i.
//
// A thread walks its line of nodes through a chunk of `len` outputs.  At node p it adds the
// nodal and viscous flux of p to the seven outputs p-3 .. p+3 (kept in registers), evaluates
// the characteristic WENO pair and split fluxes of node n = p-2, whose stencil p-4 .. p is
// now complete, and stores output p-4, finished one step earlier.  The last four nodes' Q and
// metrics sit in LDS slots that only this thread touches, so there is no barrier; the
// operands of node p+1 are requested before the arithmetic of node p, which takes several
// memory latencies.
//
// Why: the tile kernels issue VALU work on 76% of the cycles of the clock that the chip holds
// under this load (1.76-1.87 GHz), 936 (zeta) and 970 (eta) instructions per point, on rows that
// they recompute (WENO 32/30, nodal fluxes 36/30, half-point metrics twice) and on tile
// addressing; this form takes 725, a quarter of the LDS instructions and reads Q once.  Two waves
// per SIMD with 230-254 VGPRs: the outputs in flight and the node's basis do not fit less.  It
// issues on 70-78% of the cycles and moves its bytes at 83-90% of the rate of a device copy.
// Measured, 512 x 512 x 384: zeta 4.26 -> 3.31 ms, eta 4.64 -> 3.90 ms; 160^3 193 -> 153 us and
// 239 -> 168 us.
//
// The original scheme walks the same way with one slot more: node p completes the stencil
// p-5 .. p of the half point p-5/2, whose flux goes to outputs p-3 and p-2 at once (160^3 eta
// 242 -> 179 us, zeta 234 -> 172 us).  Outputs next to a face with the one-sided viscous
// closure are left out of the scatter of viscous fluxes and take their seven-point sum when
// they are stored (190 x 131 x 93 with walls in eta: 131 -> 117 us).
// =====================================================================================
constexpr int kMarchNT = 256;  // threads (grid lines) of a workgroup; two workgroups per CU
constexpr int kMarchSlot = 8 * kMarchNT;  // LDS doubles of one node: Q (5) and the metric (3)

template <int DIR, int SCHEME, bool VIS, bool PREV, bool OS>
__device__ __forceinline__ void march_lines(const SweepCommon& c, const SweepBlock& b, int grp, int chunk, int len,
                                            double* sh) {
  static_assert(DIR == 1 || DIR == 2, "lanes run along i");
  constexpr int NT = kMarchNT;
  using R = double;
  const Geom& g = b.g;
  const int nd = DIR == 1 ? g.nj : g.nk;
  const int n2 = DIR == 1 ? g.nk : g.nj;
  const uint32_t sd = DIR == 1 ? (uint32_t)g.ld_i : (uint32_t)(g.ld_i * g.ld_j);
  const uint32_t s2 = DIR == 1 ? (uint32_t)(g.ld_i * g.ld_j) : (uint32_t)g.ld_i;
  const int lines = g.ni * n2;
  const int line = min(grp * NT + (int)threadIdx.x, lines - 1);
  const bool act = grp * NT + (int)threadIdx.x < lines;  // the others repeat the last line, storing nothing
  const int o0 = chunk * len, o1 = min(o0 + len, nd);
  const uint32_t base = (uint32_t)at(g, 0, 0, 0) + (uint32_t)(line % g.ni) + (uint32_t)(line / g.ni) * s2;
  const Gas<R> G(c.ph);
  const R eps4 = 4.0 * c.ph.eps;
  const int faces = OS ? (b.one_sided >> (2 * DIR)) & 3 : 0;  // with the one-sided closure

  GP<const double> Q[5], V[4], I[5], M[3];
  GP<double> O[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    Q[v] = plane_ptr(to_global(b.q), v * g.plane);
    I[v] = plane_ptr((GP<const double>)to_global(static_cast<const double*>(b.rt_in)), v * g.plane);
    O[v] = plane_ptr(to_global(static_cast<double*>(b.rt_out)), v * g.plane);
    if (v < 4) V[v] = plane_ptr((GP<const double>)to_global(static_cast<const double*>(b.vis)), (4 * DIR + v) * g.plane);
    if (v < 3) M[v] = plane_ptr(to_global(b.met), (3 * DIR + v) * g.plane);
  }

  struct Operands {
    R q[5], v[4], m[3];  // Q and viscous flux of node p, metric of node p+1
  };
  auto load = [&](Operands& x, int n) {  // indices past the stored planes belong to discarded outputs
    const uint32_t e = base + (uint32_t)min(n, nd + 2) * sd, em = base + (uint32_t)min(n + 1, nd + 2) * sd;
#pragma unroll
    for (int v = 0; v < 5; ++v) x.q[v] = ldg(Q[v], e);
    if constexpr (VIS) {
#pragma unroll
      for (int v = 0; v < 4; ++v) x.v[v] = ldg(V[v], e);
    }
#pragma unroll
    for (int v = 0; v < 3; ++v) x.m[v] = ldg(M[v], em);
  };

  // A[o]: right-hand side of output p-3+o so far (two steps per loop round shift it by two)
  R A[8][5];
#pragma unroll
  for (int o = 0; o < 6; ++o)
#pragma unroll
    for (int v = 0; v < 5; ++v) A[o][v] = 0.0;
  R done[5], rr[5];  // output p-4, finished, and its partial sum of the earlier directions
  auto put = [&](int o) {
    if (o >= o0 && o < o1 && act) {
      const uint32_t e = base + (uint32_t)o * sd;
      if constexpr (OS && VIS) {
        int first, row, sign;
        if (one_sided_window(faces, o, nd, &first, &row, &sign)) {
#pragma unroll
          for (int v = 1; v < 5; ++v) {  // seven loads in flight
            R y[7];
#pragma unroll
            for (int m = 0; m < 7; ++m) y[m] = ldg(V[v - 1], base + (uint32_t)(first + m) * sd);
#pragma unroll
            for (int m = 0; m < 7; ++m) done[v] += os6_weight(row, sign, m) * y[m];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) stg(O[v], e, PREV ? done[v] + rr[v] : done[v]);
    }
  };
  // modified scheme: F+ of the node before at its n+1/2, and the metric of that half point
  double* const SF = sh + 4 * kMarchSlot + threadIdx.x;
  if constexpr (SCHEME == kModified) {
#pragma unroll
    for (int v = 0; v < 8; ++v) SF[v * NT] = 1.0;
  }
  R mag = 1.0, minv = 1.0;
  R mc[3];  // metric of node p

  // one node; S[0] .. are the slots of the nodes before it (p-4 .. p-1, original scheme p-5 ..
  // p-1) starting with slot k, the oldest, which takes node p
  constexpr int SLOTS = SCHEME == kModified ? 4 : 5;
  double* S[SLOTS];
#pragma unroll
  for (int n = 0; n < SLOTS; ++n) S[n] = sh + n * kMarchSlot + threadIdx.x;
  auto step = [&](int p, R(*A)[5], const Operands& x, Operands& next, int k) {
    auto slot = [&](int n) { return S[(n + k) % SLOTS]; };
    double* const S0 = slot(0);
    const double* const S1 = slot(1);
    const double* const S2 = slot(2);
    const double* const S3 = slot(3);
    load(next, p + 1);
    __builtin_amdgcn_sched_barrier(0);  // phase borders: the scheduler would overlap phases into spills
    R F[5];
    phys_flux(x.q, mc[0], mc[1], mc[2], G, F);
#pragma unroll
    for (int v = 0; v < 5; ++v) {  // Eq 19
      A[0][v] -= R(19.0 / 3840.0) * F[v];
      A[1][v] += R(13.0 / 320.0) * F[v];
      A[2][v] -= R(17.0 / 256.0) * F[v];
      A[4][v] += R(17.0 / 256.0) * F[v];
      A[5][v] -= R(13.0 / 320.0) * F[v];
      A[6][v] = R(19.0 / 3840.0) * F[v];
    }
    if constexpr (VIS) {  // d6 of the viscous flux; outputs next to a one-sided face take theirs in put
      auto add = [&](auto central) {
#pragma unroll
        for (int v = 1; v < 5; ++v) {
          const R y = x.v[v - 1];
          if (central(p - 3)) A[0][v] += R(1.0 / 60.0) * y;
          if (central(p - 2)) A[1][v] -= R(0.15) * y;
          if (central(p - 1)) A[2][v] += R(0.75) * y;
          if (central(p + 1)) A[4][v] -= R(0.75) * y;
          if (central(p + 2)) A[5][v] += R(0.15) * y;
          if (central(p + 3)) A[6][v] -= R(1.0 / 60.0) * y;
        }
      };
      if (OS && (((faces & 1) && p < 6) || ((faces & 2) && p > nd - 7)))
        add([&](int o) { return !(((faces & 1) && o < 3) || ((faces & 2) && o > nd - 4)); });
      else
        add([](int) { return true; });
    }
    __builtin_amdgcn_sched_barrier(0);
    put(p - 4);
    if (SCHEME == kModified && p > o0) {  // node n = p-2, from n = o0-1 on
      R qn[5], mn[3], h[3];
#pragma unroll
      for (int v = 0; v < 5; ++v) qn[v] = S2[v * NT];
#pragma unroll
      for (int v = 0; v < 3; ++v) {  // half_metric at n+1/2
        mn[v] = S2[(5 + v) * NT];
        h[v] = R(3.0 / 256.0) * (S0[(5 + v) * NT] + x.m[v]) - R(25.0 / 256.0) * (S1[(5 + v) * NT] + mc[v]) +
               R(150.0 / 256.0) * (mn[v] + S3[(5 + v) * NT]);
      }
      const NodeSpace<R> B = node_space(qn, mn[0], mn[1], mn[2], G);
      R D[4][5];  // projected first differences of Q along p-4 .. p
      {
        R a[5], d[5], t[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) a[v] = S1[v * NT], t[v] = a[v] - S0[v * NT];
        project_diff(B, t, D[0]);
#pragma unroll
        for (int v = 0; v < 5; ++v) t[v] = qn[v] - a[v];
        project_diff(B, t, D[1]);
#pragma unroll
        for (int v = 0; v < 5; ++v) d[v] = S3[v * NT], t[v] = d[v] - qn[v];
        project_diff(B, t, D[2]);
#pragma unroll
        for (int v = 0; v < 5; ++v) t[v] = x.q[v] - d[v], S0[v * NT] = x.q[v];
#pragma unroll
        for (int v = 0; v < 3; ++v) S0[(5 + v) * NT] = mc[v];
        project_diff(B, t, D[3]);
      }
      __builtin_amdgcn_sched_barrier(0);
      R vl[5], vr[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        weno_diff<R>(D[0][f], D[1][f], D[2][f], D[3][f], eps4, false, vl[f], vr[f]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PREV) {  // requested here, past the peak of register use, for the next step's put
        const uint32_t e = base + (uint32_t)max(p - 3, 0) * sd;
#pragma unroll
        for (int v = 0; v < 5; ++v) rr[v] = ldg(I[v], e);
      }
      half_flux<-1>(B, G, vr, SF[5 * NT], SF[6 * NT], SF[7 * NT], mag, minv, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const R f = SF[v * NT] + F[v];  // f(n-1/2) = F+(n-1) + F-(n)
        A[0][v] -= f;
        A[1][v] += f;
      }
      __builtin_amdgcn_sched_barrier(0);
      const R m2 = h[0] * h[0] + h[1] * h[1] + h[2] * h[2];
      minv = rsq(m2);
      mag = m2 * minv;
      half_flux<+1>(B, G, vl, h[0], h[1], h[2], mag, minv, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) SF[v * NT] = F[v];
#pragma unroll
      for (int v = 0; v < 3; ++v) SF[(5 + v) * NT] = h[v];
    } else if (SCHEME == kOriginal && p > o0 + 1) {  // half point n+1/2, n = p-3, from n = o0-1 on
      const double* const S4 = slot(SLOTS - 1);
      R h[3], qa[5];
#pragma unroll
      for (int v = 0; v < 3; ++v)
        h[v] = R(3.0 / 256.0) * (S0[(5 + v) * NT] + mc[v]) - R(25.0 / 256.0) * (S1[(5 + v) * NT] + S4[(5 + v) * NT]) +
               R(150.0 / 256.0) * (S2[(5 + v) * NT] + S3[(5 + v) * NT]);
#pragma unroll
      for (int v = 0; v < 5; ++v) qa[v] = R(0.5) * (S2[v * NT] + S3[v * NT]);
      const NodeSpace<R> B = node_space(qa, h[0], h[1], h[2], G);
      R D[5][5];  // projected first differences of Q along p-5 .. p
      {
        const double* const line[5] = {S0, S1, S2, S3, S4};
        R t[5];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
#pragma unroll
          for (int v = 0; v < 5; ++v) t[v] = line[n + 1][v * NT] - line[n][v * NT];
          project_diff(B, t, D[n]);
        }
#pragma unroll
        for (int v = 0; v < 5; ++v) t[v] = x.q[v] - S4[v * NT], S0[v * NT] = x.q[v];
#pragma unroll
        for (int v = 0; v < 3; ++v) S0[(5 + v) * NT] = mc[v];
        project_diff(B, t, D[4]);
      }
      __builtin_amdgcn_sched_barrier(0);
      R vl[5], vr[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        vl[f] = weno_left_diff<R>(D[0][f], D[1][f], D[2][f], D[3][f], eps4, false);
        vr[f] = weno_left_diff<R>(-D[4][f], -D[3][f], -D[2][f], -D[1][f], eps4, false);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PREV) {
        const uint32_t e = base + (uint32_t)max(p - 3, 0) * sd;
#pragma unroll
        for (int v = 0; v < 5; ++v) rr[v] = ldg(I[v], e);
      }
      const R m2 = h[0] * h[0] + h[1] * h[1] + h[2] * h[2];
      minv = rsq(m2);
      mag = m2 * minv;
      R q[5], u[5], Fm[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) q[v] = S2[v * NT];
      unproject_diff(B, G, vl, q, u);
      state_flux<+1>(u, G, h[0], h[1], h[2], mag, minv, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) q[v] = S3[v * NT];
      unproject_diff(B, G, vr, q, u);
      state_flux<-1>(u, G, h[0], h[1], h[2], mag, minv, Fm);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const R f = F[v] + Fm[v];
        A[0][v] -= f;
        A[1][v] += f;
      }
    } else {
#pragma unroll
      for (int v = 0; v < 5; ++v) S0[v * NT] = x.q[v];
#pragma unroll
      for (int v = 0; v < 3; ++v) S0[(5 + v) * NT] = mc[v];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 5; ++v) done[v] = A[0][v];
#pragma unroll
    for (int v = 0; v < 3; ++v) mc[v] = x.m[v];
  };

  int p = o0 - 3;
#pragma unroll
  for (int v = 0; v < 3; ++v) mc[v] = ldg(M[v], base + (uint32_t)p * sd);
  Operands even, odd;
  load(even, p);
  // output o is final after step o+3; the last step may be one past the chunk
#pragma unroll 1
  for (; p < o1 + 3; p += 2) {
    step(p, A, even, odd, 0);
    step(p + 1, A + 1, odd, even, 1);
    double* old[SLOTS];
#pragma unroll
    for (int n = 0; n < SLOTS; ++n) old[n] = S[n];
#pragma unroll
    for (int n = 0; n < SLOTS; ++n) S[n] = old[(n + 2) % SLOTS];
#pragma unroll
    for (int o = 0; o < 6; ++o)
#pragma unroll
      for (int v = 0; v < 5; ++v) A[o][v] = A[o + 2][v];
  }
  if (p == o1 + 3) put(o1 - 1);  // no step past the chunk stored it
}

template <int DIR, int SCHEME, bool VIS, bool PREV, bool OS>
__global__ __launch_bounds__(kMarchNT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_march(SweepArgs a, int groups,
                                                                                              int len) {
  __shared__ double sh[5 * kMarchSlot];
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  march_lines<DIR, SCHEME, VIS, PREV, OS>(a.c, a.b, t % groups, t / groups, len, sh);
}

// Chunk length of the marching sweep, or 0 where the tiles are faster: a plan of the block,
// made once (the search takes up to 2 sqrt(nd) lengths).  A workgroup puts one
// wave on each SIMD of its CU, two keep the SIMDs busy, and a step of a wave takes one unit
// (2.45 us in eta with a partial sum, 2.2 us in zeta without) of SIMD time; a chunk of len
// outputs costs len + 2.6 steps (two more WENO nodes, four nodes without), and a launch takes
// the time of the CU with most workgroups, 15% more where that is one workgroup, whose
// latencies nothing fills.  The tiles take 46-58 ps per point (eta) and 44-53 (zeta), i.e. a
// unit per 47000 points.  Measured eta, tiles / march: 96x80x72 31 / 32 us (tiles kept),
// 144x120x100 83 / 79 (tiles kept: 456 workgroups of 16 outputs, two rounds, cost 1% more by the
// rule), 160x88x96 64 / 61, 192x112x72 74 / 69, 128^3 110 / 89, 190x131x93 125 / 103, 256^3
// 890 / 641.
int march_len(int dir, const Geom& g) {
  const int nd = dir == 1 ? g.nj : g.nk, n2 = dir == 1 ? g.nk : g.nj;
  const int64_t groups = ((int64_t)g.ni * n2 + kMarchNT - 1) / kMarchNT;
  const double points = (double)g.ni * g.nj * g.nk;
  double best = points / 47000.0;
  int best_len = 0;
  for (int chunks = 1; chunks <= nd;) {
    const int part = (nd + chunks - 1) / chunks;
    const int len = part + (part & 1);  // steps come in pairs
    const int64_t wgs = groups * ((nd + len - 1) / len);
    if (wgs > 16 * 1024 && chunks > 1) break;  // many rounds already
    const int64_t rounds = (wgs + 255) / 256;
    const double cost = (rounds == 1 ? 1.15 : (double)rounds) * (len + 2.6);
    if (cost < best) best = cost, best_len = len;
    if (part == 1) break;
    chunks = (nd + part - 2) / (part - 1);  // the first count whose chunks are shorter
  }
  return best_len;
}

template <int DIR, int SCHEME, bool OS>
static void launch_march_dir(const SweepArgs& a, int groups, int chunks, int len, hipStream_t s) {
  const dim3 grid(groups * chunks), wg(kMarchNT);
  if (a.c.do_vis && a.c.has_prev)
    hipLaunchKernelGGL((k_march<DIR, SCHEME, true, true, OS>), grid, wg, 0, s, a, groups, len);
  else if (a.c.do_vis)
    hipLaunchKernelGGL((k_march<DIR, SCHEME, true, false, OS>), grid, wg, 0, s, a, groups, len);
  else if (a.c.has_prev)
    hipLaunchKernelGGL((k_march<DIR, SCHEME, false, true, false>), grid, wg, 0, s, a, groups, len);
  else
    hipLaunchKernelGGL((k_march<DIR, SCHEME, false, false, false>), grid, wg, 0, s, a, groups, len);
}
template <int DIR>
static void launch_march_scheme(const SweepArgs& a, int groups, int chunks, int len, hipStream_t s) {
  const bool os = (a.b.one_sided >> (2 * DIR)) & 3;
  if (a.c.ph.scheme == kOriginal)
    os ? launch_march_dir<DIR, kOriginal, true>(a, groups, chunks, len, s)
       : launch_march_dir<DIR, kOriginal, false>(a, groups, chunks, len, s);
  else
    os ? launch_march_dir<DIR, kModified, true>(a, groups, chunks, len, s)
       : launch_march_dir<DIR, kModified, false>(a, groups, chunks, len, s);
}

hipError_t launch_march(int dir, const SweepArgs& a, int len, hipStream_t s) {
  const int nd = dir == 1 ? a.b.g.nj : a.b.g.nk, n2 = dir == 1 ? a.b.g.nk : a.b.g.nj;
  const int groups = (int)(((int64_t)a.b.g.ni * n2 + kMarchNT - 1) / kMarchNT), chunks = (nd + len - 1) / len;
  if (dir == 1)
    launch_march_scheme<1>(a, groups, chunks, len, s);
  else
    launch_march_scheme<2>(a, groups, chunks, len, s);
  return hipGetLastError();
}

// =====================================================================================
// Halo copies across 1-to-1 faces (ghost layer m of the destination face <- interior
// layer m-1 inside the source face), boundary fills.
// =====================================================================================
template <typename T>
__device__ __forceinline__ void copy_segment(const CopySeg& S, const PtrTable& t) {
  const int per_plane = S.na * S.nb * kHalo;
  const int total = per_plane * S.nplanes;
  T* dst = static_cast<T*>(t.p[S.dst]);
  const T* src = static_cast<const T*>(t.p[S.src]);
  const int64_t pd = t.plane[S.dst], ps = t.plane[S.src];
  for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int vv = e / per_plane;
    int r = e % per_plane;
    int a, l;
    if (S.layer_fast) {
      l = r % kHalo;
      r /= kHalo;
      a = r % S.na;
      r /= S.na;
    } else {
      a = r % S.na;
      r /= S.na;
      l = r % kHalo;
      r /= kHalo;
    }
    const int b = r;
    const T x = src[(S.src_plane0 + vv) * ps + S.src_off + a * S.src_sa + b * S.src_sb + l * S.src_sl];
    dst[(S.plane0 + vv) * pd + S.dst_off + a * S.dst_sa + b * S.dst_sb + l * S.dst_sl] = S.negate ? -x : x;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_copy(const CopySeg* segs, PtrTable t) {
  copy_segment<T>(segs[blockIdx.y], t);
}

template <typename T>
hipError_t launch_copy(const CopySeg* segs_dev, int nseg, int max_elems, const PtrTable& t, hipStream_t s) {
  if (nseg == 0) return hipSuccess;
  int bx = (max_elems + 255) / 256;
  if (bx > 256) bx = 256;  // grid-stride: more workgroups mostly idle on short segments
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(k_copy<T>, dim3(bx, nseg), dim3(256), 0, s, segs_dev, t);
  return hipGetLastError();
}
template hipError_t launch_copy<double>(const CopySeg*, int, int, const PtrTable&, hipStream_t);
template hipError_t launch_copy<float>(const CopySeg*, int, int, const PtrTable&, hipStream_t);

__global__ __launch_bounds__(256) void k_wall_reset(const BcSeg* segs, BcArgs A) {
  const BcSeg S = segs[blockIdx.y];
  if (S.kind != CFD_BC_WALL) return;
  double* Q = static_cast<double*>(A.t.p[S.blk]);
  const int64_t pl = A.t.plane[S.blk];
  const int64_t total = (int64_t)S.na * S.nb;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int a = (int)(e % S.na), b = (int)(e / S.na);
    const int64_t p = S.wall_off + a * S.sa + b * S.sb;
    Q[1 * pl + p] = 0.0;
    Q[2 * pl + p] = 0.0;
    Q[3 * pl + p] = 0.0;
    Q[4 * pl + p] = Q[p] * A.t_wall / (A.gamma * (A.gamma - 1.0));
  }
}

// Characteristic far-field state for the boundary node's conserved state qb, the outward
// unit normal n and the far-field state qf: Riemann invariants u_n +- 2c/(gamma-1) along n,
// the outgoing one from qb and the incoming one from qf; entropy p/rho^gamma and the
// tangential velocity from qb on outflow, from qf on inflow; at supersonic normal speed
// the whole state of the upwind side.
__device__ void char_farfield(const double qb[5], const double n[3], const double qf[5], double gamma, double qg[5]) {
  const double gm1 = gamma - 1.0;
  const double rb = qb[0], ub = qb[1] / rb, vb = qb[2] / rb, wb = qb[3] / rb;
  const double pb = gm1 * (qb[4] - 0.5 * rb * (ub * ub + vb * vb + wb * wb));
  const double cb = sqrt(gamma * pb / rb);
  const double unb = ub * n[0] + vb * n[1] + wb * n[2];
  if (unb >= cb || unb <= -cb) {
    const double* src = unb >= cb ? qb : qf;
    for (int v = 0; v < 5; ++v) qg[v] = src[v];
    return;
  }
  const double rf = qf[0], uf = qf[1] / rf, vf = qf[2] / rf, wf = qf[3] / rf;
  const double pf = gm1 * (qf[4] - 0.5 * rf * (uf * uf + vf * vf + wf * wf));
  const double cf = sqrt(gamma * pf / rf);
  const double unf = uf * n[0] + vf * n[1] + wf * n[2];
  const double rplus = unb + 2.0 * cb / gm1, rminus = unf - 2.0 * cf / gm1;
  const double un = 0.5 * (rplus + rminus), c = 0.25 * gm1 * (rplus - rminus);
  const bool out = un > 0.0;
  const double s = out ? pb / pow(rb, gamma) : pf / pow(rf, gamma);
  const double un_s = out ? unb : unf;
  const double tx = (out ? ub : uf) - un_s * n[0], ty = (out ? vb : vf) - un_s * n[1], tz = (out ? wb : wf) - un_s * n[2];
  const double rho = pow(c * c / (gamma * s), 1.0 / gm1);
  const double p = rho * c * c / gamma;
  const double u = tx + un * n[0], v = ty + un * n[1], w = tz + un * n[2];
  qg[0] = rho;
  qg[1] = rho * u;
  qg[2] = rho * v;
  qg[3] = rho * w;
  qg[4] = p / gm1 + 0.5 * rho * (u * u + v * v + w * w);
}

__device__ __forceinline__ void ghost_segment(const BcSeg& S, const BcArgs& A) {
  double* Q = static_cast<double*>(A.t.p[S.blk]);
  const int64_t pl = A.t.plane[S.blk];
  const int64_t total = (int64_t)S.na * S.nb * kHalo;
  const double gm1 = A.gamma - 1.0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int a = (int)(e % S.na);
    const int64_t r = e / S.na;
    const int m = 1 + (int)(r % kHalo);
    const int b = (int)(r / kHalo);
    const int64_t pw = S.wall_off + a * S.sa + b * S.sb;
    const int64_t pg = pw + m * S.sout, pm = pw - m * S.sout;
    if (S.kind == CFD_BC_FARFIELD) {
      for (int v = 0; v < 5; ++v) Q[v * pl + pg] = A.qinf[v];
    } else if (S.kind == CFD_BC_FARFIELD_CHAR) {
      // outward unit normal: the face-normal direction's hatted metric at the boundary node
      const double* M = static_cast<const double*>(A.mt.p[S.blk]);
      double nv[3] = {M[(3 * S.axis) * pl + pw], M[(3 * S.axis + 1) * pl + pw], M[(3 * S.axis + 2) * pl + pw]};
      const double scale = (S.sout > 0 ? 1.0 : -1.0) / sqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
      for (int d = 0; d < 3; ++d) nv[d] *= scale;
      double qb[5], qg[5];
      for (int v = 0; v < 5; ++v) qb[v] = Q[v * pl + pw];
      char_farfield(qb, nv, A.qinf, A.gamma, qg);
      for (int v = 0; v < 5; ++v) Q[v * pl + pg] = qg[v];
    } else {
      const double rho = Q[pm], rinv = 1.0 / rho;
      const double u = Q[pl + pm] * rinv, v = Q[2 * pl + pm] * rinv, w = Q[3 * pl + pm] * rinv;
      const double ke = 0.5 * (u * u + v * v + w * w);
      const double p = gm1 * (Q[4 * pl + pm] - rho * ke);
      const double T = A.gamma * p * rinv;
      // reflection of T - T_w, floored at T_w / 2 (positive ghost density)
      const double Tg = fmax(2.0 * A.t_wall - T, 0.5 * A.t_wall);
      const double rg = A.gamma * p / Tg;
      Q[pg] = rg;
      Q[pl + pg] = -rg * u;
      Q[2 * pl + pg] = -rg * v;
      Q[3 * pl + pg] = -rg * w;
      Q[4 * pl + pg] = p / gm1 + rg * ke;
    }
  }
}

template <typename T>
__device__ __forceinline__ void visc_ghost_segment(const BcSeg& S, const PtrTable& t) {
  T* V = static_cast<T*>(t.p[S.blk]);
  const int64_t pl = t.plane[S.blk];
  const int64_t total = (int64_t)S.na * S.nb * kHalo * 4;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int a = (int)(e % S.na);
    int64_t r = e / S.na;
    const int m = 1 + (int)(r % kHalo);
    r /= kHalo;
    const int n = (int)(r % 4);
    const int b = (int)(r / 4);
    const int64_t pw = S.wall_off + a * S.sa + b * S.sb;
    T* P = V + (4 * S.axis + n) * pl;
    P[pw + m * S.sout] = T(2) * P[pw] - P[pw - m * S.sout];
  }
}

// Halo copies and ghost fills in one launch: both read nodes of the blocks and write halo nodes
// beyond different rectangles of their faces, so neither waits for the other.
__global__ __launch_bounds__(256) void k_halo(const CopySeg* copies, int ncopy, const BcSeg* bcs, BcArgs A) {
  if ((int)blockIdx.y < ncopy)
    copy_segment<double>(copies[blockIdx.y], A.t);
  else
    ghost_segment(bcs[blockIdx.y - ncopy], A);
}
template <typename T>
__global__ __launch_bounds__(256) void k_visc_halo(const CopySeg* copies, int ncopy, const BcSeg* bcs, PtrTable t) {
  if ((int)blockIdx.y < ncopy)
    copy_segment<T>(copies[blockIdx.y], t);
  else
    visc_ghost_segment<T>(bcs[blockIdx.y - ncopy], t);
}
template <typename T>
__global__ __launch_bounds__(256) void k_visc_ghost(const BcSeg* segs, PtrTable t) {
  visc_ghost_segment<T>(segs[blockIdx.y], t);
}

static dim3 bc_grid(int max_elems, int nseg) {
  int bx = (max_elems + 255) / 256;
  if (bx > 256) bx = 256;  // grid-stride: more workgroups mostly idle on short segments
  if (bx < 1) bx = 1;
  return dim3(bx, nseg);
}

hipError_t launch_wall_reset(const BcSeg* segs_dev, int nseg, int max_elems, const BcArgs& a, hipStream_t s) {
  if (nseg == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wall_reset, bc_grid(max_elems, nseg), dim3(256), 0, s, segs_dev, a);
  return hipGetLastError();
}
hipError_t launch_halo(const CopySeg* copies, int ncopy, int max_copy, const BcSeg* bcs, int nbc, int max_bc,
                       const BcArgs& a, hipStream_t s) {
  if (nbc == 0) return launch_copy<double>(copies, ncopy, max_copy, a.t, s);
  const int most = ncopy && max_copy > max_bc * kHalo ? max_copy : max_bc * kHalo;
  hipLaunchKernelGGL(k_halo, bc_grid(most, ncopy + nbc), dim3(256), 0, s, copies, ncopy, bcs, a);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_visc_halo(const CopySeg* copies, int ncopy, int max_copy, const BcSeg* bcs, int nbc, int max_bc,
                            const PtrTable& t, hipStream_t s) {
  if (nbc == 0) return launch_copy<T>(copies, ncopy, max_copy, t, s);
  const int most = ncopy && max_copy > max_bc * kHalo * 4 ? max_copy : max_bc * kHalo * 4;
  hipLaunchKernelGGL(k_visc_halo<T>, bc_grid(most, ncopy + nbc), dim3(256), 0, s, copies, ncopy, bcs, t);
  return hipGetLastError();
}
template hipError_t launch_visc_halo<double>(const CopySeg*, int, int, const BcSeg*, int, int, const PtrTable&, hipStream_t);
template hipError_t launch_visc_halo<float>(const CopySeg*, int, int, const BcSeg*, int, int, const PtrTable&, hipStream_t);
template <typename T>
hipError_t launch_visc_ghost(const BcSeg* segs_dev, int nseg, int max_elems, const PtrTable& t, hipStream_t s) {
  if (nseg == 0) return hipSuccess;
  hipLaunchKernelGGL(k_visc_ghost<T>, bc_grid(max_elems * kHalo * 4, nseg), dim3(256), 0, s, segs_dev, t);
  return hipGetLastError();
}
template hipError_t launch_visc_ghost<double>(const BcSeg*, int, int, const PtrTable&, hipStream_t);
template hipError_t launch_visc_ghost<float>(const BcSeg*, int, int, const PtrTable&, hipStream_t);

// =====================================================================================
// Reductions: CFL spectral-radius maximum and finiteness.
// =====================================================================================
// Slots of the maxima of one CFL step, one per workgroup of its launches.  The launch over the
// first block stores its slots and clears the others, the launches over the other blocks raise
// them, so what a step needs is in its own launches: nothing is cleared before it, and nothing
// that a call leaves behind matters to the next one, whether it ran, failed half-way or was
// recorded into a graph.  A slot per workgroup also spares the atomics on one address that a
// single accumulator takes: 100^3 host step 47 -> 38 us, 224 x 200 x 176 179 -> 172, 32^3
// 17.8 us as before.
//
// FIRST is a template so that the kernel of the other blocks keeps its arguments in the loads at
// its entry: behind a branch at the end their fetch is one more latency of every launch (64 blocks
// of 10^3 291 us so, 269 this way).
template <bool FIRST>
__global__ __launch_bounds__(256) void k_dt_max(Geom g, const double* q, const double* met, double gamma,
                                                unsigned long long* slots, int nslots) {
  __shared__ uint64_t red[256];
  uint64_t best = 0;  // bit pattern of the largest spectral radius (+0.0 to start)
  const int64_t total = (int64_t)g.ni * g.nj * g.nk;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int i = (int)(e % g.ni);
    const int64_t r = e / g.ni;
    const int j = (int)(r % g.nj), k = (int)(r / g.nj);
    const int64_t p = at(g, i, j, k);
    const double rho = q[p], rinv = 1.0 / rho;
    const double u = q[g.plane + p] * rinv, v = q[2 * g.plane + p] * rinv, w = q[3 * g.plane + p] * rinv;
    const double pr = (gamma - 1.0) * (q[4 * g.plane + p] - 0.5 * rho * (u * u + v * v + w * w));
    const double c = sqrt(gamma * pr * rinv);
    const double J = met[9 * g.plane + p];
    double sum = 0.0;
    for (int d = 0; d < 3; ++d) {
      const double ax = J * met[(3 * d) * g.plane + p], ay = J * met[(3 * d + 1) * g.plane + p],
                   az = J * met[(3 * d + 2) * g.plane + p];
      sum += fabs(ax * u + ay * v + az * w) + c * sqrt(ax * ax + ay * ay + az * az);
    }
    // a non-finite point (NaN or infinite spectral radius) becomes the quiet-NaN pattern,
    // which orders above +inf as an unsigned integer, so the maximum keeps it
    const uint64_t bits = sum <= 1.7976931348623157e308 ? (uint64_t)__double_as_longlong(sum) : 0x7ff8000000000000ull;
    best = best > bits ? best : bits;
  }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + h] ? red[threadIdx.x] : red[threadIdx.x + h];
    __syncthreads();
  }
  // non-negative doubles order like their bit patterns
  if constexpr (FIRST) {
    if (threadIdx.x == 0) slots[blockIdx.x] = red[0];
    for (int n = gridDim.x + blockIdx.x * 256 + threadIdx.x; n < nslots; n += gridDim.x * 256) slots[n] = 0;
  } else if (threadIdx.x == 0) {
    atomicMax(slots + blockIdx.x, (unsigned long long)red[0]);  // nobody waits for it (a load would be waited for)
  }
}

int dt_slots(const Geom& g) {
  const int64_t wgs = ((int64_t)g.ni * g.nj * g.nk + 255) / 256;
  return (int)(wgs < kDtSlots ? wgs : kDtSlots);  // kDtSlots workgroups fill the chip
}

hipError_t launch_dt_max(const Geom& g, const double* q, const double* met, double gamma, bool first, int nslots,
                         unsigned long long* slots, hipStream_t s) {
  if (first)
    hipLaunchKernelGGL(k_dt_max<true>, dim3(dt_slots(g)), dim3(256), 0, s, g, q, met, gamma, slots, nslots);
  else
    hipLaunchKernelGGL(k_dt_max<false>, dim3(dt_slots(g)), dim3(256), 0, s, g, q, met, gamma, slots, nslots);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_finite(Geom g, const double* q, int* flag) {
  const int64_t total = (int64_t)g.ni * g.nj * g.nk;
  int bad = 0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int i = (int)(e % g.ni);
    const int64_t r = e / g.ni;
    const int j = (int)(r % g.nj), k = (int)(r / g.nj);
    const int64_t p = at(g, i, j, k);
    for (int v = 0; v < 5; ++v) bad |= !isfinite(q[v * g.plane + p]);
  }
  if (bad) *flag = 1;  // every writer stores the same
}

hipError_t launch_finite(const Geom& g, const double* q, int* flag, hipStream_t s) {
  const int64_t total = (int64_t)g.ni * g.nj * g.nk;
  int bx = (int)((total + 255) / 256);
  if (bx > 8192) bx = 8192;
  hipLaunchKernelGGL(k_finite, dim3(bx), dim3(256), 0, s, g, q, flag);
  return hipGetLastError();
}

// ---- local time steps: the CFL step of every interior point ---------------------------
__global__ __launch_bounds__(256) void k_dt_local(Geom g, const double* q, const double* met, double gamma, double cfl,
                                                  double* dt_field) {
  const int64_t total = (int64_t)g.ni * g.nj * g.nk;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int i = (int)(e % g.ni);
    const int64_t r = e / g.ni;
    const int j = (int)(r % g.nj), k = (int)(r / g.nj);
    const int64_t p = at(g, i, j, k);
    const double rho = q[p], rinv = 1.0 / rho;
    const double u = q[g.plane + p] * rinv, v = q[2 * g.plane + p] * rinv, w = q[3 * g.plane + p] * rinv;
    const double pr = (gamma - 1.0) * (q[4 * g.plane + p] - 0.5 * rho * (u * u + v * v + w * w));
    const double c = sqrt(gamma * pr * rinv);
    const double J = met[9 * g.plane + p];
    double sum = 0.0;
    for (int d = 0; d < 3; ++d) {
      const double ax = J * met[(3 * d) * g.plane + p], ay = J * met[(3 * d + 1) * g.plane + p],
                   az = J * met[(3 * d + 2) * g.plane + p];
      sum += fabs(ax * u + ay * v + az * w) + c * sqrt(ax * ax + ay * ay + az * az);
    }
    dt_field[p] = cfl / sum;
  }
}

hipError_t launch_dt_local(const Geom& g, const double* q, const double* met, double gamma, double cfl,
                           double* dt_field, hipStream_t s) {
  const int64_t total = (int64_t)g.ni * g.nj * g.nk;
  int bx = (int)((total + 255) / 256);
  if (bx > 8192) bx = 8192;
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(k_dt_local, dim3(bx), dim3(256), 0, s, g, q, met, gamma, cfl, dt_field);
  return hipGetLastError();
}

// ---- CFL time step from the maxima (no host round trip) --------------------------------
__global__ __launch_bounds__(256) void k_dt_finish(const unsigned long long* __restrict__ slots, int nslots, double cfl,
                                                   double* dt) {
  __shared__ unsigned long long red[4];
  unsigned long long best = 0;
  for (int n = threadIdx.x; n < nslots; n += 256) best = best > slots[n] ? best : slots[n];
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) {
    const unsigned long long other = __shfl_down(best, h);
    best = best > other ? best : other;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < 4; ++w) best = best > red[w] ? best : red[w];
  const double smax = __longlong_as_double((long long)best);
  *dt = (smax > 0.0 && smax <= 1.7976931348623157e308) ? cfl / smax : __builtin_nan("");
}

hipError_t launch_dt_finish(const unsigned long long* slots, int nslots, double cfl, double* dt, hipStream_t s) {
  hipLaunchKernelGGL(k_dt_finish, dim3(1), dim3(256), 0, s, slots, nslots, cfl, dt);
  return hipGetLastError();
}

// ---- residual norms: reduced-dimensional reductions (Sec. 4.5) ------------------------
// 3D -> lines: each wave walks grid lines (j, k) of the block, its lanes striding along i
// (coalesced), and keeps per lane the sums of squares and the maxima of the five fields of
// scale * (a - b) (b may be null); lanes -> wave: a fixed-order shuffle tree; waves ->
// workgroup: their rows in LDS in order; the kResGroups partial rows of every block are then
// reduced by one workgroup, again in a fixed order, so the result does not depend on timing.
// Bound by HBM reads where there are enough: sixteen waves per workgroup, one workgroup per CU,
// keep ten loads per lane in flight (with four, the call on 256^3 with b took 668 us, now 268).
// Small blocks take four waves (residual_waves).
template <int NT>
__global__ __launch_bounds__(NT) void k_res_partial(Geom g, const double* __restrict__ a, const double* __restrict__ b,
                                                    double scale, double* __restrict__ part) {
  __shared__ double red[NT / 64][10];
  double sq[5] = {0, 0, 0, 0, 0}, mx[5] = {0, 0, 0, 0, 0};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lines = g.nj * g.nk;
  for (int l = blockIdx.x * (NT / 64) + wave; l < lines; l += gridDim.x * (NT / 64)) {
    const int64_t line = at(g, 0, l % g.nj, l / g.nj);
    for (int i = lane; i < g.ni; i += 64) {
      const int64_t p = line + i;
      double d[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) d[v] = a[v * g.plane + p];
      if (b) {
#pragma unroll
        for (int v = 0; v < 5; ++v) d[v] -= b[v * g.plane + p];
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        d[v] *= scale;
        sq[v] += d[v] * d[v];
        mx[v] = fmax(mx[v], fabs(d[v]));
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) {
      sq[v] += __shfl_down(sq[v], h);
      mx[v] = fmax(mx[v], __shfl_down(mx[v], h));
    }
    if (lane == 0) red[wave][v] = sq[v], red[wave][5 + v] = mx[v];
  }
  __syncthreads();
  if (threadIdx.x < 10) {
    double r = red[0][threadIdx.x];
    for (int w = 1; w < NT / 64; ++w) r = threadIdx.x < 5 ? r + red[w][threadIdx.x] : fmax(r, red[w][threadIdx.x]);
    part[(int64_t)blockIdx.x * 10 + threadIdx.x] = r;
  }
}

__global__ __launch_bounds__(256) void k_res_final(const double* __restrict__ part, int nparts, double inv_n,
                                                   double* __restrict__ out) {
  __shared__ double red[10][256];
  double sq[5] = {0, 0, 0, 0, 0}, mx[5] = {0, 0, 0, 0, 0};
  for (int r = threadIdx.x; r < nparts; r += 256) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      sq[v] += part[(int64_t)r * 10 + v];
      mx[v] = fmax(mx[v], part[(int64_t)r * 10 + 5 + v]);
    }
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    red[v][threadIdx.x] = sq[v];
    red[5 + v][threadIdx.x] = mx[v];
  }
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        red[v][threadIdx.x] += red[v][threadIdx.x + h];
        red[5 + v][threadIdx.x] = fmax(red[5 + v][threadIdx.x], red[5 + v][threadIdx.x + h]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 5) out[threadIdx.x] = sqrt(red[threadIdx.x][0] * inv_n);
  else if (threadIdx.x < 10) out[threadIdx.x] = red[threadIdx.x][0];
}

// Waves of a workgroup: four times as many cost 3.5 us more to start and finish, and save that
// once a wave of the smaller launch makes four more passes over 64 nodes than one of the larger.
// Call with 4 / 16 waves and b: 32^3 30.4 / 34.4 us, 64^3 33.7 / 34.6, 128 x 64 x 48 39.2 / 36.9,
// 80^3 52.5 / 41.5, 512 x 32 x 32 43.3 / 47.6, 512 x 64 x 64 84 / 57; 64 blocks of 10^3 402 / 639.
static int residual_waves(const Geom& g) {
  const int64_t lines = (int64_t)g.nj * g.nk, row = (g.ni + 63) / 64;
  auto passes = [&](int waves) { return (lines + kResGroups * waves - 1) / (kResGroups * waves) * row; };
  return passes(4) - passes(16) < 4 ? 4 : 16;
}

hipError_t launch_res_partial(const Geom& g, const double* a, const double* b, double scale, double* part,
                              hipStream_t s) {
  if (residual_waves(g) == 4)
    hipLaunchKernelGGL(k_res_partial<256>, dim3(kResGroups), dim3(256), 0, s, g, a, b, scale, part);
  else
    hipLaunchKernelGGL(k_res_partial<1024>, dim3(kResGroups), dim3(1024), 0, s, g, a, b, scale, part);
  return hipGetLastError();
}
hipError_t launch_res_final(const double* part, int nparts, double inv_n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_res_final, dim3(1), dim3(256), 0, s, part, nparts, inv_n, out);
  return hipGetLastError();
}

}  // namespace cfd
