// Device helpers shared by the mechanics kernels (mech.hip) and the
// multigrid preconditioner (mg.hip): node-grid launch shape, wave64 and block
// reductions in FP64, and the matrix-free HEX8 stiffness of Eq. (8) applied
// cell by cell.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "etm_internal.h"

namespace etm {
namespace mech {

constexpr int BX = 64, BY = 4;

inline dim3 node_grid(const DevGrid &g) { return dim3((g.nx + 1 + BX - 1) / BX, (g.ny + 1 + BY - 1) / BY, g.nz + 1); }

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block sums of NS values into out[0..NS) (any block size that is a multiple of 64, <= 1024).
template <int NS>
__device__ __forceinline__ void block_sums(const double (&v)[NS], double *out) {
  __shared__ double red[16][NS];
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int lane = tid & 63, wv = tid >> 6;
  double r[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) r[q] = wsum(v[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NS; ++q) red[wv][q] = r[q];
  __syncthreads();
  if (tid == 0) {
    const int nw = (blockDim.x * blockDim.y) / 64;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      double acc = red[0][q];
      for (int w = 1; w < nw; ++w) acc += red[w][q];
      out[q] = acc;
    }
  }
}

// Fixed-order sum of partials[nb][kRedWidth] columns 0..NS-1 by one block of 256.
template <int NS>
__device__ __forceinline__ void sum_partials(const double *part, int64_t nb, double *out) {
  double v[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) v[q] = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += blockDim.x)
#pragma unroll
    for (int q = 0; q < NS; ++q) v[q] += part[b * kRedWidth + q];
  block_sums<NS>(v, out);
}

// ---- cell-based HEX8 apply ---------------------------------------------------
// For a box cell the element stiffness is a sum of Kronecker products of 1D
// 2x2 factors: mass m(a,b) = int phi_a phi_b, stiffness k = int phi_a' phi_b',
// and the mixed g = int phi_a' phi_b, g^T.  In the per-axis basis
// (sum, difference) = (v0 + v1, v1 - v0) each factor is diagonal or a swap:
//   m: diag(h/2, h/6)   k: diag(0, 2/h)   g: sum -> difference   g^T: difference -> sum
// so K_e u = H^-1 D H u with H the tensor sum/difference transform, and D
// has 24 diagonal entries and 24 single-entry couplings between components.
// The in-plane part of H belongs to a node plane, not to a cell: a column of
// cells transforms each plane once, as the top of one layer and the bottom
// of the next, and adds both layers' results before it transforms back.

// In-plane transform of a cell's four corner values (index ax + 2 ay).
template <typename T>
__device__ __forceinline__ void haar2(T v[4]) {
  const T a = v[0] + v[1], b = v[1] - v[0], c = v[2] + v[3], d = v[3] - v[2];
  v[0] = a + c; v[1] = b + d; v[2] = c - a; v[3] = d - b;
}
// Its inverse without the factor 1/4 (folded, with z's 1/2, into the operator).
template <typename T>
__device__ __forceinline__ void ihaar2(T v[4]) {
  const T a = v[0] - v[2], b = v[1] - v[3], c = v[0] + v[2], d = v[1] + v[3];
  v[0] = a - b; v[1] = a + b; v[2] = c - d; v[3] = c + d;
}

// The in-plane factors of a column of cells, fixed while it marches up z:
// the mass of the sum modes along x and y (the difference modes have a third
// of it), and stiffness along one times mass along the other.
template <typename T>
struct HexColumn {
  T mx, my, a1, a2;
  __device__ __forceinline__ HexColumn(T hx, T hy, T ihx, T ihy)
      : mx(hx * T(0.5)), my(hy * T(0.5)), a1(ihx * hy), a2(ihy * hx) {}
};

// One cell layer of a column in the transformed basis: lo / up are the
// in-plane modes of the bottom and top plane (component, px + 2 py); lo
// becomes the cell's result on the bottom plane, vt its result on the top.
template <typename T>
__device__ __forceinline__ void hex8_layer(const HexColumn<T> &C, T hz, T ihz, T lam, T mu, T lo[3][4],
                                           const T up[3][4], T vt[3][4]) {
  const T el = T(0.125) * lam, em = T(0.125) * mu;
  const T mz[2] = {hz * T(0.5), hz * T(1.0 / 6.0)}, kz = T(2) * ihz;
  T u[3][8], v[3][8];  // index px + 2 py + 4 pz
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u[c][q] = lo[c][q] + up[c][q];
      u[c][q + 4] = up[c][q] - lo[c][q];
    }
  const T L[2] = {el * mz[0], el * mz[1]}, M[2] = {em * mz[0], em * mz[1]};
  constexpr T third = T(1.0 / 3.0);
  const T ma = C.mx * C.my;
  const T Kz = em * kz * ma, Lz = el * kz * ma + Kz;
  const T fz[4] = {T(1), third, third, T(1.0 / 9.0)};  // mass times mass of mode px + 2 py, over ma
  const T pxy[4] = {T(0), C.a1, C.a2, (C.a1 + C.a2) * third};
#pragma unroll
  for (int pz = 0; pz < 2; ++pz) {
    const T lm = L[pz] + M[pz];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int px = q & 1, py = q >> 1, p = q + 4 * pz;
      T base = q ? M[pz] * pxy[q] : T(0);
      if (pz) base += Kz * fz[q];
      const T dx = px ? base + lm * (py ? C.a1 * third : C.a1) : base,
              dy = py ? base + lm * (px ? C.a2 * third : C.a2) : base, dz = pz ? base + Lz * fz[q] : base;
      v[0][p] = dx * u[0][p];
      v[1][p] = dy * u[1][p];
      v[2][p] = dz * u[2][p];
    }
  }
#pragma unroll
  for (int pz = 0; pz < 2; ++pz) {  // x-y coupling: (sum x, diff y) <-> (diff x, sum y)
    const int ai = 2 + 4 * pz, ao = 1 + 4 * pz;
    v[0][ao] += L[pz] * u[1][ai]; v[0][ai] += M[pz] * u[1][ao];
    v[1][ai] += L[pz] * u[0][ao]; v[1][ao] += M[pz] * u[0][ai];
  }
#pragma unroll
  for (int py = 0; py < 2; ++py) {  // x-z coupling
    const int ai = 2 * py + 4, ao = 1 + 2 * py;
    const T my = py ? C.my * third : C.my, l = el * my, m = em * my;
    v[0][ao] += l * u[2][ai]; v[0][ai] += m * u[2][ao];
    v[2][ai] += l * u[0][ao]; v[2][ao] += m * u[0][ai];
  }
#pragma unroll
  for (int px = 0; px < 2; ++px) {  // y-z coupling
    const int ai = px + 4, ao = px + 2;
    const T mx = px ? C.mx * third : C.mx, l = el * mx, m = em * mx;
    v[1][ao] += l * u[2][ai]; v[1][ai] += m * u[2][ao];
    v[2][ai] += l * u[1][ao]; v[2][ao] += m * u[1][ai];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lo[c][q] = v[c][q] - v[c][q + 4];
      vt[c][q] = v[c][q] + v[c][q + 4];
    }
}

// A node as a plane (the same for every thread of a block, so its part of an
// address stays in scalar registers) and a place in the plane (below 2^32
// bytes at the largest mesh a plan accepts).
struct NodeAt {
  int64_t plane;
  uint32_t off;
};
// The place as a value the compiler cannot tell from a new one each time
// round a loop: it otherwise keeps 64-bit addresses of every array per lane
// (two more registers and a vector add per access) instead of a scalar base.
__device__ __forceinline__ uint32_t fresh(uint32_t off) {
  asm("" : "+v"(off));
  return off;
}
template <typename T>
__device__ __forceinline__ T ld(const T *p, const NodeAt &n) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p + n.plane) + n.off * uint32_t(sizeof(T)));
}
template <typename T>
__device__ __forceinline__ void st(T *p, const NodeAt &n, T v) {
  *reinterpret_cast<T *>(reinterpret_cast<char *>(p + n.plane) + n.off * uint32_t(sizeof(T))) = v;
}
template <typename T>
__device__ __forceinline__ T ld(const T *p, int64_t n) { return p[n]; }
template <typename T>
__device__ __forceinline__ void st(T *p, int64_t n, T v) { p[n] = v; }

// y = K x over the mesh, cell by cell, with an epilogue per node.
// A block of CX x CY threads owns a tile of CX x CY columns of cells and the
// (CX-1) x (CY-1) nodes whose four in-plane cells all lie in the tile, and
// marches up z over kchunk node planes.  Per layer: plane ck + 1 of x goes
// to LDS, one barrier, then (1) the owned nodes add the four columns'
// results on plane ck - 1, left in LDS by the layer below, in a fixed order
// (y is deterministic) and run the epilogue; (2) the next plane of x, its
// materials and the epilogue's inputs of plane ck are requested; (3) every
// thread transforms its four values of plane ck + 1, applies its cell and
// leaves the column's result on plane ck, the layer's bottom plus the top of
// the layer below, in the other half of the LDS buffer.
// Bound by VALU issue (about 300 instructions per wave and layer) together
// with HBM: on 257x257x65 nodes in FP32 the plain residual takes 56 us (179 MB
// of counted traffic, 3.2 TB/s), a smoothing step 84 us (350 MB, 4.2 TB/s), or
// 96 us (392 MB) where it stores its direction.
// A form that transformed each cell's eight corners by itself and left 24
// results per cell in LDS (two barriers a layer, every load masked where it
// was issued) took 84 and (every step storing a direction) 110 us; in FP64 on
// 98x84x34 nodes 19.1 and 21.2 us against 14.6 and 16.9 us now.
// Fixed DOFs give zero rows; x is taken as zero on them.  The Lame constants
// come from a per-block LDS copy of the material table (both zero for a void
// material and outside the mesh).  The epilogue sees (n, y, x at the node,
// its prefetched inputs, per-thread partial sums).
constexpr int CX = 32, CY = 8;
constexpr int kMatMaxMech = 256;  // material ids are 8-bit

inline dim3 cell_grid(const DevGrid &g, int kchunk) {
  return dim3((g.nx + 1 + CX - 2) / (CX - 1), (g.ny + 1 + CY - 2) / (CY - 1), (g.nz + 1 + kchunk - 1) / kchunk);
}
// Planes per block.  The resident blocks (4 per CU in FP32, 2 in FP64, by
// registers and LDS) march in step, so a launch takes about (generations of
// blocks) x (planes per block + 2: the layer below the chunk and the start).
// The number of chunks that makes this smallest is taken, within the rows that
// the reduction's partials always hold (one per block: max(1024, node blocks));
// a mesh whose tiles alone are more takes one chunk, and a plan gives its
// partials a row for each (mech_part_rows).  On
// 257x257x65 nodes in FP32 that is 22 planes: 55 us for the residual and
// 85 us for a smoothing step, against 69 and 98 us at 5 planes; on
// 161x153x49 nodes 7 planes, 21.6 and 24.8 us against 25.2 and 29.2 us at 4.
template <typename T>
inline int cell_kchunk(const DevGrid &g) {
  const int64_t tiles = int64_t((g.nx + 1 + CX - 2) / (CX - 1)) * ((g.ny + 1 + CY - 2) / (CY - 1));
  const dim3 nb = node_grid(g);
  const int64_t rows = std::max<int64_t>(1024, int64_t(nb.x) * nb.y * nb.z), resident = sizeof(T) == 4 ? 1024 : 512;
  int best = g.nz + 1;
  int64_t least = INT64_MAX;
  // from one chunk of all planes on, each number of chunks at its shortest (a
  // longer one costs more): some 2 sqrt(nz) candidates, as this runs at every launch
  for (int kc = g.nz + 1; kc >= 2; --kc) {
    const int chunks = (g.nz + 1 + kc - 1) / kc;
    kc = (g.nz + 1 + chunks - 1) / chunks;
    const int64_t blocks = tiles * chunks;
    if (blocks > rows && kc <= g.nz) break;
    const int64_t cost = (blocks + resident - 1) / resident * (kc + 2);
    if (cost < least) {
      least = cost;
      best = kc;
    }
  }
  return best;
}

template <typename T, int NS, class Epi>
__global__ __launch_bounds__(CX * CY, sizeof(T) == 4 ? 4 : 2) void hex8_cell_kernel(MechGrid M, const T *x0, const T *x1, const T *x2,
                                                             int kchunk, Epi epi, double *partials,
                                                             const DevScalars *sc) {
  if (sc && sc->done) return;
  const DevGrid &g = M.g;
  constexpr int PL = (CY + 1) * (CX + 1);          // nodes per staged plane
  constexpr int PT = (PL + CX * CY - 1) / (CX * CY);  // plane entries per thread
  __shared__ T xs[3][3][CY + 1][CX + 1];
  __shared__ T co[2][12][CY][CX];
  __shared__ T lm_tab[kMatMaxMech][2];
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * CX + tx;
  for (int m = tid; m < g.n_mat; m += CX * CY) {
    const double *row = g.mtab + m * kMatStride;
    const bool solid = row[MC_VOID] == 0.0;
    lm_tab[m][0] = solid ? T(row[MC_LAMBDA]) : T(0);
    lm_tab[m][1] = solid ? T(row[MC_MU]) : T(0);
  }
  // logical tile of this block, x fastest: tiles that share cache lines at
  // their x and y borders mostly share an L2
  const int nbx = int(gridDim.x), nby = int(gridDim.y);
  const int lb =
      grouped_block((int(blockIdx.z) * nby + int(blockIdx.y)) * nbx + int(blockIdx.x), nbx * nby * int(gridDim.z));
  const int bx = lb % nbx, by = (lb / nbx) % nby, bz = lb / (nbx * nby);
  const int i0 = bx * (CX - 1), j0 = by * (CY - 1);
  const int k0 = bz * kchunk, k1 = min(k0 + kchunk, g.nz + 1);
  const int ci = i0 - 1 + tx, cj = j0 - 1 + ty;
  const bool cin = ci >= 0 && ci < g.nx && cj >= 0 && cj < g.ny;
  const int ni = i0 + tx, nj = j0 + ty;
  const bool own = tx < CX - 1 && ty < CY - 1 && ni <= g.nx && nj <= g.ny;
  const HexColumn<T> C(cin ? T(g.dx[ci]) : T(1), cin ? T(g.dy[cj]) : T(1), cin ? T(g.idx[ci]) : T(1),
                       cin ? T(g.idy[cj]) : T(1));
  const uint32_t sy = uint32_t(g.sy), own_at = uint32_t(nj) * sy + uint32_t(ni);
  const T *xv[3] = {x0, x1, x2};
  double red[NS > 0 ? NS : 1];
#pragma unroll
  for (int q = 0; q < (NS > 0 ? NS : 1); ++q) red[q] = 0.0;
  // Plane k of x into registers (this thread's share), then into LDS.  Entries
  // off the mesh read the first of a plane, so no load waits behind a branch
  // (but the second entry is one per wave); they are masked when they are
  // staged, a layer later, so nothing waits for the loads before that.
  T pf[PT][3];
  int pm = 0;       // material id of cell (ci, cj, k - 1), fetched with plane k
  bool pk = false;  // plane k is in the mesh
  uint32_t at[PT];
  bool in[PT];
#pragma unroll
  for (int e = 0; e < PT; ++e) {
    const int t = tid + e * CX * CY;
    const int r = t / (CX + 1), c = t - r * (CX + 1);
    const int i = i0 - 1 + c, j = j0 - 1 + r;
    in[e] = t < PL && i >= 0 && i <= g.nx && j >= 0 && j <= g.ny;
    at[e] = in[e] ? uint32_t(j) * sy + uint32_t(i) : 0u;
#pragma unroll
    for (int q = 0; q < 3; ++q) pf[e][q] = T(0);
  }
  const uint32_t cell_at = cin ? uint32_t(cj) * sy + uint32_t(ci) : 0u;
  auto fetch = [&](int k) {
    const int kk = min(max(k, 0), g.nz), kl = min(max(k - 1, 0), g.nz - 1);
    pk = k == kk;
    pm = int(ld(g.mat, NodeAt{int64_t(kl) * g.sz, fresh(cell_at)}));
    const int64_t plane = int64_t(kk) * g.sz;
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      if (e > 0 && tid + e * CX * CY >= PL) continue;
      const NodeAt n{plane, fresh(at[e])};
#pragma unroll
      for (int q = 0; q < 3; ++q) pf[e][q] = ld(xv[q], n);
    }
  };
  auto stage = [&](int k) {
    T(*dst)[CY + 1][CX + 1] = xs[(k + 3) % 3];
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      const int t = tid + e * CX * CY;
      if (t < PL) {
        const int r = t / (CX + 1), c = t - r * (CX + 1);
#pragma unroll
        for (int q = 0; q < 3; ++q) dst[q][r][c] = in[e] && pk ? pf[e][q] : T(0);
      }
    }
  };
  // the cell's four values of plane k, as in-plane modes
  auto modes = [&](int k, T s[3][4]) {
    const T(*pl)[CY + 1][CX + 1] = xs[(k + 3) % 3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int a = 0; a < 4; ++a) s[q][a] = pl[q][ty + (a >> 1)][tx + (a & 1)];
      haar2(s[q]);
    }
  };
  T lo[3][4], top[3][4], xc[3];  // xc: x at the owned node on the plane whose results were left last
  typename Epi::Pre pre;
  uint8_t fix = 0;
  auto emit = [&](int k) {
    const T(*cp)[CY][CX] = co[k & 1];
    // node (ni, nj) is corner (1,1) of cell (tx,ty), (0,1) of (tx+1,ty),
    // (1,0) of (tx,ty+1) and (0,0) of (tx+1,ty+1)
    T y[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
      y[q] = cp[3 * 3 + q][ty][tx] + cp[2 * 3 + q][ty][tx + 1] + cp[1 * 3 + q][ty + 1][tx] + cp[q][ty + 1][tx + 1];
    if (fix & 1) y[0] = T(0);
    if (fix & 2) y[1] = T(0);
    if (fix & 4) y[2] = T(0);
    epi(NodeAt{int64_t(k) * g.sz, fresh(own_at)}, y, xc, pre, red);
  };
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int a = 0; a < 4; ++a) top[q][a] = T(0);
  fetch(k0 - 1);
  stage(k0 - 1);
  fetch(k0);
  __syncthreads();
  modes(k0 - 1, lo);
  for (int ck = k0 - 1; ck < k1; ++ck) {
    stage(ck + 1);
    const int m = pm;  // cell layer ck (fetched with plane ck + 1)
    const bool solid = cin && ck >= 0 && ck < g.nz;
    __syncthreads();
    if (own && ck > k0) emit(ck - 1);
    if (ck + 2 <= k1) fetch(ck + 2);
    if (own && ck >= k0) {
      const NodeAt n{int64_t(ck) * g.sz, fresh(own_at)};
      pre = epi.load(n);
      fix = ld(M.fixed, n);
    }
    const int kc = min(max(ck, 0), g.nz - 1);
    const T lam = solid ? lm_tab[m][0] : T(0), mu = solid ? lm_tab[m][1] : T(0);
    T up[3][4], vt[3][4];
    // (here and not in emit: by then a faster wave may be staging over the plane)
    for (int q = 0; q < 3; ++q) xc[q] = xs[(ck + 3) % 3][q][ty + 1][tx + 1];
    modes(ck + 1, up);
    hex8_layer<T>(C, T(g.dz[kc]), T(g.idz[kc]), lam, mu, lo, up, vt);
    T(*cp)[CY][CX] = co[ck & 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        lo[q][a] += top[q][a];
        top[q][a] = vt[q][a];
      }
      ihaar2(lo[q]);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        cp[a * 3 + q][ty][tx] = lo[q][a];
        lo[q][a] = up[q][a];
      }
    }
  }
  __syncthreads();
  if (own) emit(k1 - 1);
  if constexpr (NS > 0) {
    const int64_t b = (int64_t(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    block_sums<NS>(red, partials + b * kRedWidth);
  }
}

template <typename T>
inline int64_t cell_blocks(const DevGrid &g) {
  const dim3 d = cell_grid(g, cell_kchunk<T>(g));
  return int64_t(d.x) * d.y * d.z;
}

template <typename T, int NS, class Epi>
inline hipError_t launch_hex8(const MechGrid &M, const T *const x[3], Epi epi, double *partials, const DevScalars *sc,
                              hipStream_t s) {
  const int kc = cell_kchunk<T>(M.g);
  hipLaunchKernelGGL((hex8_cell_kernel<T, NS, Epi>), cell_grid(M.g, kc), dim3(CX, CY), 0, s, M, x[0], x[1], x[2], kc,
                     epi, partials, sc);
  return hipGetLastError();
}

}  // namespace mech
}  // namespace etm
