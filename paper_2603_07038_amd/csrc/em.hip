// gfx950 kernels of the coupled EM + Joule + thermal march (arXiv 2603.07038,
// Sec. II-A): the explicit central-difference EM update of Eq. (2)-(3) with
// sigma(T) from Eq. (6), the Joule source D_sigma e^2, the forward-Euler
// conduction step of Eq. (5), and the history diagnostics.
//
// Scaled form used on the device (both precisions).  Dividing Eq. (2) for an
// edge by eps0 and by the edge volume L*A gives
//   (er + a) e^{n+1} = 2 er e^n - (c0 dt)^2 (C e^n) - (er - a) e^{n-1} - jd
// with er the edge's mean relative permittivity, a = dt sigma_e / (2 eps0)
// (port conductances included), C the purely geometric curl-curl
// (curl mu0^-1 curl = C / mu0) and jd = dt (J^{n+1/2} - J^{n-1/2}) / eps0.
// The mixed path marches the same scheme as leapfrog on (e^n, h^{n-1/2}),
// both stored in FP32 and combined in FP64, with an 8-bit residual that
// extends the stored e below its FP32 rounding (e_join).  Edge
// coefficients are always formed in FP64 and rounded once.
//
// March kernels.  A block owns a column of nodes and marches up a chunk of z
// planes (FP64: 32 x 8 or 64 x 4 nodes staged in LDS with a one-node halo; mixed:
// 64 x 4 of them, or barrier-free waves of 62 nodes each).  A node updates the x-,
// y- and z-edges that start at it.  The Joule source is gathered one step late: the
// node sums sigma e^2 L A over its six incident edges of the *input* field
// e^n, which the stencil already holds, so no edge update is recomputed.
// The power of the last step of a thermal block is added by the thermal
// kernel (or by a flush kernel at the end of an advance call) before
// temperature changes.
#include <algorithm>
#include <type_traits>

#include "etm_internal.h"

namespace etm {

namespace {

constexpr int BX = 64, BY = 4;             // threads per block (x, y)
// nodes of an FP64 march tile (x, y), one per thread: see em_flat
constexpr int kTileX = 32, kTileY = 8, kFlatX = 64, kFlatY = 4;

// ---- field accessors: value of component c at node offset (di, dj, dk) --
template <typename T>
struct GAcc {  // global memory around node n
  const T *e[3];
  int64_t n, sy, sz;
  __device__ __forceinline__ T raw(int c, int di, int dj, int dk) const { return e[c][n + di + dj * sy + dk * sz]; }
  __device__ __forceinline__ double operator()(int c, int di, int dj, int dk) const { return double(raw(c, di, dj, dk)); }
};

// ---- geometric curl-curl (C e) at the edge of direction D starting at node
// (i,j,k).  h on a primal face = circulation / area (mu0 dropped); faces
// outside the domain carry zero (PMC truncation).
template <typename T, typename A>
__device__ __forceinline__ T curl_x(const DevGrid &g, const A &E, int i, int j, int k) {
  const T idxi = T(g.idx[i]);
  T s = T(0);
  if (j < g.ny) s += ((E.raw(0, 0, 0, 0) - E.raw(0, 0, 1, 0)) * T(g.idy[j]) + (E.raw(1, 1, 0, 0) - E.raw(1, 0, 0, 0)) * idxi) * T(g.ihy[j]);
  if (j > 0) s -= ((E.raw(0, 0, -1, 0) - E.raw(0, 0, 0, 0)) * T(g.idy[j - 1]) + (E.raw(1, 1, -1, 0) - E.raw(1, 0, -1, 0)) * idxi) * T(g.ihy[j]);
  if (k < g.nz) s -= ((E.raw(2, 0, 0, 0) - E.raw(2, 1, 0, 0)) * idxi + (E.raw(0, 0, 0, 1) - E.raw(0, 0, 0, 0)) * T(g.idz[k])) * T(g.ihz[k]);
  if (k > 0) s += ((E.raw(2, 0, 0, -1) - E.raw(2, 1, 0, -1)) * idxi + (E.raw(0, 0, 0, 0) - E.raw(0, 0, 0, -1)) * T(g.idz[k - 1])) * T(g.ihz[k]);
  return s;
}
template <typename T, typename A>
__device__ __forceinline__ T curl_y(const DevGrid &g, const A &E, int i, int j, int k) {
  const T idyj = T(g.idy[j]);
  T s = T(0);
  if (k < g.nz) s += ((E.raw(2, 0, 1, 0) - E.raw(2, 0, 0, 0)) * idyj - (E.raw(1, 0, 0, 1) - E.raw(1, 0, 0, 0)) * T(g.idz[k])) * T(g.ihz[k]);
  if (k > 0) s -= ((E.raw(2, 0, 1, -1) - E.raw(2, 0, 0, -1)) * idyj - (E.raw(1, 0, 0, 0) - E.raw(1, 0, 0, -1)) * T(g.idz[k - 1])) * T(g.ihz[k]);
  if (i < g.nx) s -= ((E.raw(0, 0, 0, 0) - E.raw(0, 0, 1, 0)) * idyj + (E.raw(1, 1, 0, 0) - E.raw(1, 0, 0, 0)) * T(g.idx[i])) * T(g.ihx[i]);
  if (i > 0) s += ((E.raw(0, -1, 0, 0) - E.raw(0, -1, 1, 0)) * idyj + (E.raw(1, 0, 0, 0) - E.raw(1, -1, 0, 0)) * T(g.idx[i - 1])) * T(g.ihx[i]);
  return s;
}
template <typename T, typename A>
__device__ __forceinline__ T curl_z(const DevGrid &g, const A &E, int i, int j, int k) {
  const T idzk = T(g.idz[k]);
  T s = T(0);
  if (i < g.nx) s += ((E.raw(2, 0, 0, 0) - E.raw(2, 1, 0, 0)) * T(g.idx[i]) + (E.raw(0, 0, 0, 1) - E.raw(0, 0, 0, 0)) * idzk) * T(g.ihx[i]);
  if (i > 0) s -= ((E.raw(2, -1, 0, 0) - E.raw(2, 0, 0, 0)) * T(g.idx[i - 1]) + (E.raw(0, -1, 0, 1) - E.raw(0, -1, 0, 0)) * idzk) * T(g.ihx[i]);
  if (j < g.ny) s -= ((E.raw(2, 0, 1, 0) - E.raw(2, 0, 0, 0)) * T(g.idy[j]) - (E.raw(1, 0, 0, 1) - E.raw(1, 0, 0, 0)) * idzk) * T(g.ihy[j]);
  if (j > 0) s += ((E.raw(2, 0, 0, 0) - E.raw(2, 0, -1, 0)) * T(g.idy[j - 1]) - (E.raw(1, 0, -1, 1) - E.raw(1, 0, -1, 0)) * idzk) * T(g.ihy[j]);
  return s;
}

__device__ __forceinline__ bool pec_edge(const DevGrid &g, int D, int i, int j, int k) {
  const int b = g.pec;
  if (D != 0 && ((i == 0 && (b & 1)) || (i == g.nx && (b & 2)))) return true;
  if (D != 1 && ((j == 0 && (b & 4)) || (j == g.ny && (b & 8)))) return true;
  if (D != 2 && ((k == 0 && (b & 16)) || (k == g.nz && (b & 32)))) return true;
  return false;
}

// ---- 1D tables, from one base pointer (dx, dy, dz, idx, idy, idz, hx, hy, hz,
// ihx, ihy, ihz, then alpha_lo / alpha_hi per axis on nodes).
struct Geo {
  const double *dx, *dy, *dz, *idx, *idy, *idz, *ihx, *ihy, *ihz, *axl, *axh, *ayl, *ayh, *azl, *azh;
  __device__ __forceinline__ Geo(const double *g, int nx, int ny, int nz) {
    dx = g; dy = dx + nx; dz = dy + ny;
    idx = dz + nz; idy = idx + nx; idz = idy + ny;
    const double *hx = idz + nz, *hy = hx + nx + 1, *hz = hy + ny + 1;
    ihx = hz + nz + 1; ihy = ihx + nx + 1; ihz = ihy + ny + 1;
    axl = ihz + nz + 1; axh = axl + nx + 1; ayl = axh + nx + 1; ayh = ayl + ny + 1;
    azl = ayh + ny + 1; azh = azl + nz + 1;
  }
};

// ---- edge coefficients from the cells around a node -----------------------
// Cell (i-1+ox, j-1+oy, k-1+oz) touches the node's x-edge on side ox (the
// edge starting at the node if ox = 1, the low-side edge i-1 if ox = 0), its
// y-edge on side oy and its z-edge on side oz.  An edge property is the mean
// over its cells weighted by the share of the edge's dual area in each cell;
// on a rectilinear grid that share factors into alpha_y(oy) * alpha_z(oz)
// for an x-edge (alpha = half the cell width over the node's dual width, 0 for
// a cell outside the mesh).  sigma follows Eq. (6) per cell at the
// edge-midpoint rise.  Returned: the normalised conductance
// a = dt sigma / (2 eps0) and (own edges) the mean eps_r.  FP64 with explicit
// FMAs and contraction off, so every kernel that calls it gets the same bits.
struct CellV {
  double er, sg;  // eps_r, sigma0 * dt / (2 eps0)
  int tf, m;      // sigma depends on temperature; material id
};

template <int D, typename CELL, typename TCR, typename TH>
__device__ __forceinline__ double edge_coef(int side, const double (&ax)[2], const double (&ay)[2],
                                            const double (&az)[2], const CELL &cell, const TCR &tcr_of, const TH &th,
                                            double *er_out) {
#pragma clang fp contract(off)
  double er = 0.0, sg = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int p0 = q & 1, p1 = q >> 1;  // offsets in the two transverse directions
    const int ox = D == 0 ? side : p0, oy = D == 1 ? side : (D == 0 ? p0 : p1), oz = D == 2 ? side : p1;
    const double w = D == 0 ? ay[oy] * az[oz] : D == 1 ? ax[ox] * az[oz] : ax[ox] * ay[oy];
    const CellV v = cell(ox, oy, oz);
    double s0 = v.sg;
    if (v.tf && w != 0.0) {
      const double t0 = th(0, 0, 0);
      const double t1 = D == 0 ? th(side ? 1 : -1, 0, 0) : D == 1 ? th(0, side ? 1 : -1, 0) : th(0, 0, side ? 1 : -1);
      s0 = s0 / (1.0 + tcr_of(v.m) * (0.5 * (t0 + t1)));
    }
    sg = fma(w, s0, sg);
    if (er_out) er = fma(w, v.er, er);
  }
  if (er_out) *er_out = er;
  return sg;
}

// Joule power density at the node from its six incident edges of field e:
//   P_n = sum_e 1/2 sigma_e e^2 L A / V_n = jf * sum_e a_e e^2 (L / dual width),
// with L / dual width = 2 alpha on the edge's side (0 for a missing edge).
// a[0..5], v[0..5]: own x, y, z then low-side x, y, z.
__device__ __forceinline__ double node_joule(const double (&a)[6], const double (&ax)[2], const double (&ay)[2],
                                             const double (&az)[2], const double (&v)[6], double jf) {
#pragma clang fp contract(off)
  double s = 0.0;
  s = fma(ax[1] * a[0], v[0] * v[0], s);
  s = fma(ay[1] * a[1], v[1] * v[1], s);
  s = fma(az[1] * a[2], v[2] * v[2], s);
  s = fma(ax[0] * a[3], v[3] * v[3], s);
  s = fma(ay[0] * a[4], v[4] * v[4], s);
  s = fma(az[0] * a[5], v[5] * v[5], s);
  return (2.0 * jf) * s;
}

// The temperatures an own edge of the node reads, loaded beforehand: the
// node's and its +x, +y, +z neighbours'.
struct PTh {
  double t[4];
  __device__ __forceinline__ double operator()(int di, int dj, int dk) const {
    return di > 0 ? t[1] : dj > 0 ? t[2] : dk > 0 ? t[3] : t[0];
  }
};

// The per-material EM constants in LDS: eps_r, the scaled conductance
// (stored negated where sigma depends on T, so one load gives both) and the
// temperature coefficient.  Loaded once per block; every thread of the block
// must reach the barrier.
constexpr int kMatMax = 256;
struct LdsMat {
  double er[kMatMax], sg[kMatMax], tcr[kMatMax];
};
__device__ __forceinline__ void lds_mat_load(const DevGrid &g, LdsMat &M) {
  const int tid = threadIdx.x + threadIdx.y * blockDim.x, nt = blockDim.x * blockDim.y;
  for (int m = tid; m < g.n_mat; m += nt) {
    const double *row = g.mtab + m * kMatStride;
    const bool tf = row[MC_TCR] != 0.0 && row[MC_SIGS] != 0.0;
    M.er[m] = row[MC_EPSR];
    M.sg[m] = tf ? -row[MC_SIGS] : row[MC_SIGS];
    M.tcr[m] = row[MC_TCR];
  }
  __syncthreads();
}
// The 8 cells around a node by id (index ox + 2 oy + 4 oz), values from LDS;
// material 0 for a cell outside the mesh (its weights are 0).
struct LCell {
  const LdsMat *M;
  int id[8];
  __device__ __forceinline__ CellV operator()(int ox, int oy, int oz) const {
    const int m = id[ox + 2 * oy + 4 * oz];
    const double sg = M->sg[m];
    CellV v;
    v.er = M->er[m];
    v.sg = fabs(sg);
    v.tf = sg < 0.0 ? 1 : 0;
    v.m = m;
    return v;
  }
};
struct LTcr {
  const LdsMat *M;
  __device__ __forceinline__ double operator()(int m) const { return M->tcr[m]; }
};

__device__ __forceinline__ int find_port(const DevPorts &P, int64_t key) {
  int lo = 0, hi = P.n_edges - 1;
  while (lo <= hi) {
    int mid = (lo + hi) >> 1;
    int64_t km = P.key[mid];
    if (km == key) return mid;
    if (km < key) lo = mid + 1; else hi = mid - 1;
  }
  return -1;
}

// Value at time t of a closed-form wave (the excitation scheme of Sec. III-B):
// a Ricker wavelet, a sine, or a Gaussian pulse train on a carrier, zero
// outside [t_on, t_off).  Record: kind, n_pulses, amp, t0, width, freq,
// t_on, t_off, pulse centres.
__device__ __forceinline__ double wave_value(const double *w, double t) {
  if (!(t >= w[6] && t < w[7])) return 0.0;
  const int kind = int(w[0]);
  const double amp = w[2], t0 = w[3], width = w[4], f = w[5];
  if (kind == ETM_WAVE_RICKER) {
    const double u = (t - t0) / width;
    const double a = u * u;
    return amp * (1.0 - 2.0 * a) * exp(-a);
  }
  if (kind == ETM_WAVE_SINE) return amp * sin(2.0 * M_PI * f * (t - t0));
  double env = 0.0;
  const int np = int(w[1]);
  for (int q = 0; q < np; ++q) {
    const double u = (t - w[8 + q]) / width;
    env += exp(-(u * u));
  }
  return amp * env * cos(2.0 * M_PI * f * (t - t0));
}

// Samples s = base .. base + kWaveBlock of every closed-form wave: J at
// t = (s - 1/2) dt, the same instants as a tabulated wave's samples.
__global__ __launch_bounds__(256) void wave_sample_kernel(const double *aw, int n, double dt, int64_t base,
                                                          double *Ja) {
  const int64_t per = kWaveBlock + 1;
  const int64_t id = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (id >= int64_t(n) * per) return;
  const int64_t w = id / per, q = id - w * per;
  Ja[id] = wave_value(aw + w * kWaveStride, (double(base + q) - 0.5) * dt);
}

// Entry of a port edge in the place of its eps_r among the coefficients.  The
// marches index DevPorts::rec and er with what they find there and check only
// the node's port flag, so every slot of a flagged edge has to hold an entry:
// flags and entries come from one list at plan creation, only the full refresh
// writes these slots, and it runs at bind and at restore, before any march.  A
// kernel that changes eps_r of a port edge has to write DevPorts::er instead.
__device__ __forceinline__ float port_code(int q, float) { return __int_as_float(q); }
__device__ __forceinline__ double port_code(int q, double) { return __longlong_as_double(q); }
__device__ __forceinline__ int port_entry(float c) { return __float_as_int(c); }
__device__ __forceinline__ int port_entry(double c) { return int(__double_as_longlong(c)); }

// Source, lumped conductance and eps_r of port edge q at this step.  The
// entry's first source term sits in its record, so a port costs two dependent
// reads (record, wave sample) behind the coefficients.  On a small mesh the
// waves that hold ports end last, and the launch with them: with a binary
// search over the keys and a read per array here, a step of a 61 x 61 x 38
// package took 26.1 us in mixed precision, against 11.9 us with its ports
// taken out; with the record 13.2 us.
//
// Port source of EM step n at an edge: jd = dt (J^{n+1/2} - J^{n-1/2}) / eps0
// (three-level form), jn = dt J^{n+1/2} / eps0 (leapfrog form), and the
// lumped conductance g (scaled like the a-coefficient).  J^{n+1/2} is the
// sampled value n+1 of a tabulated wave, or of a closed-form wave (sampled on
// the device, see wave_sample_kernel).
struct PortTerm {
  double jd, jn, g, er;
};
__device__ __forceinline__ PortTerm port_terms(const DevPorts &P, int q, int64_t step) {
  const PortRec R = P.rec[q];
  PortTerm r{0.0, 0.0, R.gs, P.er[q]};
  const int64_t s1 = step + 1, s0 = step, ns = P.n_samples;
  int w = R.wave;
  double wt = R.wt;
  for (int t = 0;;) {
    double j1, j0;
    if (w < P.n_table) {
      const double *Jw = P.J + int64_t(w) * ns;
      j1 = s1 < ns ? Jw[s1] : 0.0;
      j0 = s0 < ns ? Jw[s0] : 0.0;
    } else {
      const double *Jw = P.Ja + int64_t(w - P.n_table) * (kWaveBlock + 1) - P.a_base;
      j1 = Jw[s1];
      j0 = Jw[s0];
    }
    r.jd += wt * (j1 - j0);
    r.jn += wt * j1;
    if (++t >= R.n) break;
    w = P.wave[R.more + t - 1];
    wt = P.wt[R.more + t - 1];
  }
  return r;
}

// The mixed path keeps each e component as an FP32 value plus an 8-bit
// residual: e = hi + lo * ulp(hi) / 256.  The stencil reads hi; the own-edge
// accumulation e^{n+1} = e^n + (e^{n+1} - e^n) runs on the full value, so
// the per-step rounding of e (which otherwise dominates the error of the
// temperature rise over long windows) is 256 times smaller.
// log2 of ulp(hi) / 256 (subnormals share the smallest binade's ulp)
__device__ __forceinline__ int lo_exp(float hi) {
  const int E = int((__float_as_uint(hi) >> 23) & 0xFFu);
  return max(E, 1) - 158;
}
__device__ __forceinline__ double e_join(float hi, int8_t lo) { return double(hi) + ldexp(double(lo), lo_exp(hi)); }
__device__ __forceinline__ void e_split(double x, float &hi, int8_t &lo) {
  hi = float(x);
  const double r = rint(ldexp(x - double(hi), -lo_exp(hi)));  // exact scaling by a power of two
  lo = int8_t(fmax(-128.0, fmin(127.0, r)));
}

// Face value of the leapfrog field h^{n+1/2} = h^{n-1/2} + c0 dt (curl e^n)
// (per unit area), from the face's four edge values in the fixed order
// (a - b) s + (c - d) t.  Every thread that needs a face computes it with
// this one expression, so a face computed at a tile or chunk border is
// bitwise the value its owner stores.
__device__ __forceinline__ float hface(float hold, float a, float b, double s, float c, float d, double t,
                                       double cdt) {
  const double q = __builtin_fma(double(a) - double(b), s, (double(c) - double(d)) * t);
  return float(__builtin_fma(cdt, q, double(hold)));
}

// 1/x in FP64: hardware reciprocal and two Newton steps (full precision).
__device__ __forceinline__ double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// LDS of one FP64 block: four e planes (k - 1, k, k + 1 and the one being
// staged) of the TX x TY node column with a one-node halo, and the dual-width
// shares of its columns and rows.  Four blocks fit on a CU.
template <typename T, int TX, int TY>
struct MarchSmem {
  T e[4][3][TY + 2][TX + 2];
  double ax[2][TX], ay[2][TY];
};

template <typename T>
struct EmPtrs {
  const T *e;    // e^n (component c at + c*cs)
  const T *aux;  // FP64: e^{n-1};  mixed: h^{n-1/2} (faces: x-normal, y-normal, z-normal at + c*cs)
  T *oe;         // e^{n+1}
  T *oaux;       // mixed: h^{n+1/2}
};

// Joule power density at node n from the stored coefficients of its six
// incident edges and their field values v (own x, y, z, low x, y, z).  For the
// flush kernel; the marches and the thermal kernel hold these values already
// and form the same six products in the same order.
// The mixed path stores 2a, so its conductances are halved (exactly) here.
template <typename T>
__device__ __forceinline__ double joule_from_coef(const T *cf, uint32_t cs, uint32_t n, uint32_t sy, uint32_t sz,
                                                  int i, int j, int k, const double (&ax)[2], const double (&ay)[2],
                                                  const double (&az)[2], const double (&v)[6], double jf) {
  const double h = sizeof(T) == 4 ? 0.5 : 1.0;
  const double a6[6] = {h * double(cf[3 * cs + n]), h * double(cf[4 * cs + n]), h * double(cf[5 * cs + n]),
                        i > 0 ? h * double(cf[3 * cs + n - 1]) : 0.0, j > 0 ? h * double(cf[4 * cs + n - sy]) : 0.0,
                        k > 0 ? h * double(cf[5 * cs + n - sz]) : 0.0};
  return node_joule(a6, ax, ay, az, v, jf);
}

// ---- addressing of the marches ------------------------------------------------
// Every access is an array's base plus the plane and component (the same for
// the block: scalar registers) plus the lane's place in the plane (32 bits,
// below 2^32 bytes at the largest mesh a plan accepts).

// The lane's place as a value that the compiler cannot carry round the loop
// as a 64-bit address per array.
__device__ __forceinline__ uint32_t fresh(uint32_t off) {
  asm("" : "+v"(off));
  return off;
}

// A value handed on to the next plane, moved here: without this the move can
// end up behind the loads that refill its source, at the loop's head, and
// wait there for all of them.
template <typename T>
__device__ __forceinline__ T handed_on(T v) {
  asm("" : "+v"(v));
  return v;
}

// A table entry at an index that is the same for the wave, as a scalar load:
// read through a plain pointer in a loop that stores, it becomes a vector load
// whose latency every plane waits for.  (The tables are constant while a
// kernel runs.)
__device__ __forceinline__ double uniform_entry(const double *t, int i) {
  using Table = const __attribute__((address_space(4))) double *;
  return ((Table)(uintptr_t)t)[i];
}

template <bool NT = false, typename T>
__device__ __forceinline__ T ld_plane(const T *base, int64_t o, uint32_t r) {
  const T *a = reinterpret_cast<const T *>(reinterpret_cast<const char *>(base + o) + r * uint32_t(sizeof(T)));
  if constexpr (NT) return __builtin_nontemporal_load(a);
  return *a;
}

// Store to entry r of the n entries of a plane; r = 0xffffffff stores nothing:
// the plane is a buffer of its own, and a buffer drops stores past its end.
// So a store needs no branch: the waits for loads count requests in order, and
// requests that a branch may skip have to be waited for with the ones before.
template <bool NT = false, typename T>
__device__ __forceinline__ void st_plane(T *base, int64_t o, uint32_t n, uint32_t r, T v) {
  constexpr uint32_t B = sizeof(T);  // (0xffffffff * B wraps to at least 0xfffffff8, still past the end)
  const auto buf = __builtin_amdgcn_make_buffer_rsrc(base + o, 0, int(n * B), 0x00027000);
  constexpr int kAux = NT ? 2 : 0;
  if constexpr (B == 1) {
    __builtin_amdgcn_raw_buffer_store_b8(uint8_t(v), buf, r, 0, kAux);
  } else if constexpr (B == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), buf, r * B, 0, kAux);
  } else {
    using U2 = uint32_t __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), buf, r * B, 0, kAux);
  }
}

// ---- FP64: the three-level form of Eq. (2)-(3) on (e^n, e^{n-1}) -----------
// One block: the TX x TY node column (tx, ty) over the z planes of chunk kc.
// Per plane: stage e plane k+1, update the own edges of the nodes of plane
// k from their stored coefficients, and gather the Joule power of e^n at the
// node from its six incident edges.  Plane k + 2 and the node inputs of plane
// k + 1 are requested while plane k is computed, with no select and no branch
// between a request and its use (see st_plane), and one barrier per plane.
// Bound by HBM: 95 us on 257x257x65 nodes, 765 us on 1025x513x65.  There the
// loads that are used once and the stores bypass the caches (em_streams; with
// blocks in eight ranges, grouped_block, 101.5 and 883 us; 127 and 928 without
// either), and a
// 32 x 8 tile reads 1.33 nodes per node where 64 x 4 reads 1.55 (52.6 against
// 58.5 us on 2.06 M nodes, 64 against 75 on 2.49 M, 101.5 against 104 on the
// first; 16 x 16 rows are too short: 109).  With the node inputs read where
// they are used, masks, and two barriers around a three-plane ring it took 162
// and 1137 us.
template <typename T, int TX, int TY, bool NT>
__device__ __forceinline__ void em_march_tile(const EmLaunch &L, const EmPtrs<T> &p, int64_t step, int tx, int ty,
                                              int kc, int kchunk, int acc_joule, MarchSmem<T, TX, TY> &S) {
  constexpr int TXH = TX + 2, TYH = TY + 2;  // staged tile with halo
  const DevGrid &g = L.g;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const uint32_t sy = uint32_t(g.sy), sz = uint32_t(g.sz);
  const int64_t cs = g.cs;
  const Geo G(g.geo, nx, ny, nz);
  const T *cf = static_cast<const T *>(L.coef);
  const int tid = int(threadIdx.y) * BX + int(threadIdx.x), lx = tid % TX, ly = tid / TX;
  const int i0 = tx * TX, j0 = ty * TY;
  const int i = i0 + lx, j = j0 + ly;
  const int k0 = kc * kchunk, k1 = min(k0 + kchunk, nz + 1);
  // per-thread x / y factors (clamped indices)
  const bool active = i <= nx && j <= ny;
  const int ic = min(i, nx), jc = min(j, ny);
  if (tid < TX) {
    S.ax[0][tid] = G.axl[min(i0 + tid, nx)];
    S.ax[1][tid] = G.axh[min(i0 + tid, nx)];
  }
  if (tid < TY) {
    S.ay[0][tid] = G.ayl[min(j0 + tid, ny)];
    S.ay[1][tid] = G.ayh[min(j0 + tid, ny)];
  }
  // (a factor is 0 where its cell does not exist: with the zeros staged there
  // the faces outside the mesh come out as 0 without a mask)
  const T idx_i = i < nx ? T(G.idx[ic]) : T(0), idx_m = i > 0 ? T(G.idx[ic - 1]) : T(0), ihx_i = T(G.ihx[ic]);
  const T idy_j = j < ny ? T(G.idy[jc]) : T(0), idy_m = j > 0 ? T(G.idy[jc - 1]) : T(0), ihy_j = T(G.ihy[jc]);
  const T c2 = T(L.c2dt2);
  const int pec = g.pec;
  const bool pec_i = (i == 0 && (pec & 1)) || (i == nx && (pec & 2));
  const bool pec_j = (j == 0 && (pec & 4)) || (j == ny && (pec & 8));
  // own edges held at zero on every plane (on PEC faces, or not in the mesh)
  const bool zx = pec_j || i >= nx, zy = pec_i || j >= ny, zz = pec_i || pec_j;
  const uint32_t rj = uint32_t(jc) * sy + uint32_t(ic);
  const uint32_t rx = ic > 0 ? rj - 1 : rj, ry = jc > 0 ? rj - sy : rj;
  const uint32_t so = active ? rj : 0xffffffffu;
  auto plane = [&](int kk) -> int64_t { return int64_t(min(max(kk, 0), nz)) * int64_t(sz); };

  // This thread's entries of a staged plane.  Entries off the mesh read the
  // nearest node and are cleared when they are staged; threads without a
  // second entry read their first again.
  constexpr int NPF = (TYH * TXH + TX * TY - 1) / (TX * TY);
  struct Staged {
    T v[NPF][3];
  };
  uint32_t at[NPF];
  bool in[NPF];
#pragma unroll
  for (int q = 0; q < NPF; ++q) {
    const int t = tid + q * TX * TY < TYH * TXH ? tid + q * TX * TY : tid;
    const int r = t / TXH, c = t - r * TXH;
    const int gi = i0 - 1 + c, gj = j0 - 1 + r;
    in[q] = gi >= 0 && gi <= nx && gj >= 0 && gj <= ny;
    at[q] = uint32_t(min(max(gj, 0), ny)) * sy + uint32_t(min(max(gi, 0), nx));
  }
  auto fetch = [&](int kk, Staged &pf) {
    const int64_t o = plane(kk);
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      const uint32_t a = fresh(at[q]);
#pragma unroll
      for (int c = 0; c < 3; ++c) pf.v[q][c] = ld_plane(p.e, o + c * cs, a);
    }
  };
  auto commit = [&](int kk, const Staged &pf) {
    const bool pk = kk >= 0 && kk <= nz;
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      const int t = tid + q * TX * TY;
      if (t < TYH * TXH) {
        const int r = t / TXH, c = t - r * TXH;
#pragma unroll
        for (int d = 0; d < 3; ++d) S.e[kk & 3][d][r][c] = pk && in[q] ? pf.v[q][d] : T(0);
      }
    }
  };

  // Inputs of a node, each requested for the next plane as soon as this
  // plane's has been used.  A node with no conducting cell around it has a = 0
  // on its six incident edges: a wave without one skips those loads (a scalar
  // branch on flags that were loaded a plane ahead).
  struct Node {
    T er[3], pv[3];
    double a[3], axm, aym;
    uint32_t fl;
  };
  auto load_flags = [&](int kk) -> uint32_t { return ld_plane(g.flags, plane(kk), fresh(rj)); };
  Node nd;
  auto load_edge = [&](int kk, int d) {
    const int64_t o = plane(kk) + d * cs;
    const uint32_t q = fresh(rj);
    nd.er[d] = ld_plane<NT>(cf, o, q);
    nd.pv[d] = ld_plane<NT>(p.aux, o, q);
  };
  auto load_loss = [&](int kk) {
    const int64_t o = plane(kk);
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, am = 0.0, an = 0.0;
    if (__any(nd.fl & kFlagSigma)) {
      const uint32_t q2 = fresh(rj);
      a0 = double(ld_plane(cf, o + 3 * cs, q2));
      a1 = double(ld_plane(cf, o + 4 * cs, q2));
      a2 = double(ld_plane(cf, o + 5 * cs, q2));
      am = double(ld_plane(cf, o + 3 * cs, fresh(rx)));
      an = double(ld_plane(cf, o + 4 * cs, fresh(ry)));
    }
    nd.a[0] = a0; nd.a[1] = a1; nd.a[2] = a2;
    nd.axm = am; nd.aym = an;
  };

  // (the three planes are requested at once: one after the other, they made
  // up half a chunk's latency)
  Staged pf;
  nd.fl = load_flags(k0);
  {
    Staged lo, mid;
    fetch(k0 - 1, lo);
    fetch(k0, mid);
    fetch(k0 + 1, pf);
#pragma unroll
    for (int d = 0; d < 3; ++d) load_edge(k0, d);
    load_loss(k0);
    commit(k0 - 1, lo);
    commit(k0, mid);
  }
  uint32_t fl_next = load_flags(k0 + 1);
  double azm = k0 > 0 ? double(ld_plane(cf, plane(k0 - 1) + 5 * cs, rj)) : 0.0;

  auto step_plane = [&](int k, auto more) {
    constexpr bool kMore = decltype(more)::value;
    commit(k + 1, pf);
    __syncthreads();
    if constexpr (kMore) fetch(k + 2, pf);
    const bool pec_k = (k == 0 && (pec & 16)) || (k == nz && (pec & 32));
    auto E = [&](int c, int di, int dj, int dk) -> T { return S.e[(k + dk) & 3][c][ly + 1 + dj][lx + 1 + di]; };
    const T e0x = E(0, 0, 0, 0), e0y = E(1, 0, 0, 0), e0z = E(2, 0, 0, 0);
    const bool zero_d[3] = {zx || pec_k, zy || pec_k, zz || k >= nz};
    const T idz_k = k < nz ? T(uniform_entry(G.idz, k)) : T(0), idz_m = k > 0 ? T(uniform_entry(G.idz, k - 1)) : T(0),
            ihz_k = T(uniform_entry(G.ihz, k));
    // curl-curl of e^n on the three own edges
    const T hz_c = (e0x - E(0, 0, 1, 0)) * idy_j + (E(1, 1, 0, 0) - e0y) * idx_i;        // hz(i, j)
    const T hy_c = (e0z - E(2, 1, 0, 0)) * idx_i + (E(0, 0, 0, 1) - e0x) * idz_k;        // hy(i, k)
    const T hx_c = (E(2, 0, 1, 0) - e0z) * idy_j - (E(1, 0, 0, 1) - e0y) * idz_k;        // hx(j, k)
    const int64_t o = int64_t(k) * int64_t(sz);
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      T cc;
      if (D == 0) {
        const T hz_jm = (E(0, 0, -1, 0) - e0x) * idy_m + (E(1, 1, -1, 0) - E(1, 0, -1, 0)) * idx_i;
        const T hy_km = (E(2, 0, 0, -1) - E(2, 1, 0, -1)) * idx_i + (e0x - E(0, 0, 0, -1)) * idz_m;
        cc = (hz_c - hz_jm) * ihy_j - (hy_c - hy_km) * ihz_k;
      } else if (D == 1) {
        const T hx_km = (E(2, 0, 1, -1) - E(2, 0, 0, -1)) * idy_j - (e0y - E(1, 0, 0, -1)) * idz_m;
        const T hz_im = (E(0, -1, 0, 0) - E(0, -1, 1, 0)) * idy_j + (e0y - E(1, -1, 0, 0)) * idx_m;
        cc = (hx_c - hx_km) * ihz_k - (hz_c - hz_im) * ihx_i;
      } else {
        const T hy_im = (E(2, -1, 0, 0) - e0z) * idx_m + (E(0, -1, 0, 1) - E(0, -1, 0, 0)) * idz_k;
        const T hx_jm = (e0z - E(2, 0, -1, 0)) * idy_m - (E(1, 0, -1, 1) - E(1, 0, -1, 0)) * idz_k;
        cc = (hy_c - hy_im) * ihx_i - (hx_c - hx_jm) * ihy_j;
      }
      const T e0 = D == 0 ? e0x : D == 1 ? e0y : e0z;
      T er = nd.er[D], a = T(nd.a[D]), jd = T(0);
      if (nd.fl & (1 << D)) {
        const PortTerm pt = port_terms(L.ports, port_entry(er), step);
        er = T(pt.er);
        a = T(double(a) + pt.g);
        jd = T(pt.jd);
      }
      const T inv = T(rcp64(double(er) + double(a)));
      const T v = (T(2) * er * e0 - c2 * cc - (er - a) * nd.pv[D] - jd) * inv;
      st_plane<NT>(p.oe, o + D * cs, sz, so, zero_d[D] ? T(0) : v);
      if constexpr (kMore) load_edge(k + 1, D);
    }
    if (acc_joule && active && (nd.fl & kFlagSigma)) {
      const double ax[2] = {S.ax[0][lx], S.ax[1][lx]}, ay[2] = {S.ay[0][ly], S.ay[1][ly]};
      const double az[2] = {uniform_entry(G.azl, k), uniform_entry(G.azh, k)};
      const double a6[6] = {nd.a[0], nd.a[1], nd.a[2], i > 0 ? nd.axm : 0.0, j > 0 ? nd.aym : 0.0, k > 0 ? azm : 0.0};
      const double v[6] = {double(e0x), double(e0y), double(e0z), double(E(0, -1, 0, 0)), double(E(1, 0, -1, 0)),
                           double(E(2, 0, 0, -1))};
      const double P = node_joule(a6, ax, ay, az, v, L.jf);
      // one thread per node: the add is not contended and its result is the plain sum
      if (P != 0.0) unsafeAtomicAdd(L.psum + o + fresh(rj), P);
    }
    azm = handed_on(nd.a[2]);
    if constexpr (kMore) {
      nd.fl = handed_on(fl_next);
      load_loss(k + 1);
      fl_next = load_flags(k + 2);
    }
  };
  for (int k = k0; k + 1 < k1; ++k) step_plane(k, std::true_type{});
  step_plane(k1 - 1, std::false_type{});
}

// ---- mixed: the same scheme as leapfrog on (e^n, h^{n-1/2}) ----------------
// Both fields are stored in FP32 and combined in FP64:
//   h^{n+1/2} = h^{n-1/2} + c0 dt curl e^n                       (faces)
//   (er + a) (e^{n+1} - e^n) = -2a e^n - c0 dt curl^T h^{n+1/2} - jn + K
// Eliminating h gives Eq. (2) exactly; K (per edge, zero until sigma changes)
// carries the difference the three-level form keeps when a changes at a
// thermal step.  Rounding errors of h reach e only through curl^T, so they
// never feed the gradient (static-charge) modes the curl-curl leaves
// undamped in dielectrics; the increment form e^{n+1} - e^n stored in FP32
// lets them accumulate.

// Per-node inputs of one plane for the edge update.
struct YeeNode {
  float er[3], a2[3], K[3];
  float a2ym;  // 2a of the y-edge at j-1 (Joule)
  int8_t lo[3];
  uint32_t fl;
};

// One wave per run of nodes, no barriers.  A wave owns WX = 62 consecutive
// nodes of a plane numbered x fastest (a run may cross the end of a row) and
// marches up its z-chunk on its own: lanes 0 and 63 overlap the neighbouring
// runs, so every x-neighbour a face or the Joule gather needs is one lane
// away (whole-wave DPP shifts).  The rows j - 1 and j + 1 of each lane's node
// are read directly (their own waves read the same lines, so they are L2
// hits), and the faces of row j - 1 that the edge update needs are
// recomputed in-wave with the same expression their owner uses.  No barriers:
// each wave's loads for the next plane are in flight while it computes the
// current one, and its neighbours on the SIMD fill the gaps.  Bound by the
// latency of a plane's loads on small meshes and by the L2 lines it requests
// (62 per wave and plane) on larger ones; 20.1 us on 153x121x44 nodes, 37.0 on
// 201x201x51 (21.3 and 38.8 with loads and stores behind branches, whose waits
// cover all that was requested before).
constexpr int WX = 62;

// Whether a step over `nodes` nodes (of all variants of its launch) touches
// more than the 256 MB last-level cache holds, so that nothing it writes, or
// reads once, is still there at the next step: such data then goes past the
// caches (non-temporal).  Bytes per node and step: FP64 113 (three fields,
// eps_r, flags, part of the loss terms), mixed 85 (four fields, residuals,
// eps_r, flags, part of the loss terms and K).  FP64 us per step without |
// with, by million nodes:
//   0.81  23.0 | 27.6   1.69  41.0 | 48.3   2.06  52.2 | 57.7
//   2.49  68.0 | 64.5   3.03  94.5 | 82.1   4.29  132 | 106   9.63  284 | 260
__host__ __device__ inline bool em_streams(int64_t nodes, bool fp64) {
  return nodes * (fp64 ? 113 : 85) > (int64_t(1) << 28);
}

// Which of the two mixed marches a mesh takes when no tuning table says so:
// the tiles when a step streams and their padding is below 30 % of the plane,
// the runs (no idle lanes, no barriers) otherwise.  us per step, runs | tiles,
// by million nodes:
//   0.46  13.7 | 18.5   1.21  26.5 | 33.5   2.06  37.0 | 54.1   2.49  43.4 | 57.7
//   3.03  67.9 | 67.7   4.29  102.8 | 92.9 (26 % padding)   5.89  135 | 113
//   9.63  214 | 202     34.2  708 | 644    135.5  2712 | 2496
constexpr int MX = 64, MY = 4;  // nodes of a mixed tile (x, y): a wave is a row
__host__ __device__ inline bool em_runs(const DevGrid &g) {
  if (g.layout != kLayoutAuto) return g.layout == kLayoutRuns;
  const int64_t plane = int64_t(g.nx + 1) * (g.ny + 1);
  const int64_t padded = int64_t((g.nx + MX) / MX) * ((g.ny + MY) / MY) * (MX * MY);
  return !em_streams(g.ntot, false) || padded * 10 > plane * 13;
}

__device__ __forceinline__ float lane_next(float v) {  // value of lane + 1 (0 past the last lane)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_prev(float v) {  // value of lane - 1 (0 before the first lane)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}

struct RowE {  // e of one row and plane (x, y, z components)
  float x, y, z;
};

// The in-plane dual-width shares of a lane's node, which only the Joule gather
// reads: in LDS they cost no registers in the waves without a conductor.
struct YeeSmem {
  double a[4][BY][BX];  // x low, x high, y low, y high
};

__device__ __forceinline__ void em_march_run_yee(const EmLaunch &L, const EmPtrs<float> &p, int64_t step, int ts,
                                                 int kc, int kchunk, int acc_joule, YeeSmem &S) {
  const DevGrid &g = L.g;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const uint32_t sy = uint32_t(g.sy), sz = uint32_t(g.sz), cs = g.cs;
  const int lane = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.y));
  // Wave w owns the nodes t = WX w .. WX w + WX - 1 of the plane numbered x
  // fastest (t = j (nx + 1) + i); lane L holds t = WX w - 1 + L.  A run may
  // cross the end of a row (the lane after node (nx, j) holds (0, j + 1)):
  // every term that would read across -- the faces at i = nx, and through them
  // the faces and x-edge at i - 1 of node 0 -- does not exist and is masked,
  // so short rows leave no lanes idle.
  const int nx1 = nx + 1, nplane = nx1 * (ny + 1);
  const int w = ts * BY + wave;
  if (WX * w >= nplane) return;  // the whole wave is past the plane
  const int t = WX * w - 1 + lane;
  const bool inb = t >= 0 && t < nplane;
  const int tc = min(max(t, 0), nplane - 1);
  const Geo G(g.geo, nx, ny, nz);
  const float *cf = static_cast<const float *>(L.coef);
  const float *Kp = L.K;
  int8_t *elo = L.elo;
  const double cdt = L.cdt;
  const int j = tc / nx1, ic = tc - j * nx1;                // (clamped for lanes off the plane)
  const int i = inb ? ic : -1;
  const bool own = lane >= 1 && lane <= WX && inb;          // node updated by this lane
  const int k0 = kc * kchunk, k1 = min(k0 + kchunk, nz + 1);
  const bool jm_ok = j > 0, jp_ok = j < ny;                 // rows j - 1, j + 1 exist
  const uint32_t rj = uint32_t(j) * sy + uint32_t(ic);
  const uint32_t rm = jm_ok ? rj - sy : rj, rp = jp_ok ? rj + sy : rj;

  // Every access is an array's base plus the plane and component (the same
  // for the wave: scalar registers) plus the lane's place in the plane (32
  // bits, below 2^32 bytes at the largest mesh a plan accepts).  Nothing is
  // masked where it is loaded: a lane off the plane, a row or a plane that
  // does not exist reads its nearest node, and the faces formed from it are
  // cleared below.  (A select on a load's result makes the wave wait for it
  // there; 64-bit addresses per lane cost two vector adds per access.)
  auto plane = [&](int kk, int c) -> int64_t { return int64_t(c) * cs + int64_t(min(max(kk, 0), nz)) * int64_t(sz); };
  auto ld = [&](const float *base, int64_t o, uint32_t r) -> float {
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base + o) + r * 4u);
  };
  auto row3 = [&](int kk, uint32_t r) -> RowE {
    return RowE{ld(p.e, plane(kk, 0), r), ld(p.e, plane(kk, 1), r), ld(p.e, plane(kk, 2), r)};
  };

  // per-lane x and y factors
  const double dxi = G.idx[min(ic, nx - 1)], dhx = G.ihx[ic];
  const double dyj = G.idy[min(j, ny - 1)], dym = G.idy[max(j - 1, 0)], dhy = G.ihy[j];
  S.a[0][wave][lane] = G.axl[ic];  // (a lane reads its own entries only)
  S.a[1][wave][lane] = G.axh[ic];
  S.a[2][wave][lane] = G.ayl[j];
  S.a[3][wave][lane] = G.ayh[j];
  const int pec = g.pec;
  const bool pec_i = (i == 0 && (pec & 1)) || (i == nx && (pec & 2));
  const bool pec_j = (j == 0 && (pec & 4)) || (j == ny && (pec & 8));
  // faces that exist (independent of the plane, apart from k < nz)
  const bool fz = inb && i < nx && j < ny;         // z-normal (i, j)
  const bool fzm = inb && i < nx && jm_ok;         // z-normal (i, j - 1)
  const bool fy = inb && i < nx;                   // y-normal (i, j, k), k < nz
  const bool fx = inb && j < ny;                   // x-normal (i, j, k), k < nz
  const bool fxm = inb && jm_ok;                   // x-normal (i, j - 1, k), k < nz
  // own edges held at zero on every plane
  const bool zx = pec_j || i >= nx, zy = pec_i || j >= ny, zz = pec_i || pec_j;
  const uint32_t so = own ? rj : 0xffffffffu;

  // A node with no conducting cell around it has 2a = 0 on its own edges,
  // on the y-edge of its j - 1 neighbour and (through the previous lane and
  // plane) on the other incident edges, and K = 0: a wave none of whose
  // nodes has a conducting cell skips those loads.  The test is wave-wide
  // (a scalar branch) and reads flags loaded one plane ahead, so no load
  // waits behind it; gating the loads lane by lane measured slower.
  auto load_flags = [&](int kk) -> uint32_t { return (g.flags + plane(kk, 0))[fresh(rj)]; };
  auto load_node = [&](int kk, uint32_t flk, YeeNode &c) {
    const uint32_t q = fresh(rj);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      c.er[d] = ld(cf, plane(kk, d), q);
      c.lo[d] = (elo + plane(kk, d))[q];
    }
    c.fl = flk;
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, am = 0.0f, K0 = 0.0f, K1 = 0.0f, K2 = 0.0f;
    if (__any(flk & kFlagSigma)) {
      const uint32_t q2 = fresh(rj);
      a0 = ld(cf, plane(kk, 3), q2);
      a1 = ld(cf, plane(kk, 4), q2);
      a2 = ld(cf, plane(kk, 5), q2);
      am = ld(cf, plane(kk, 4), fresh(rm));
      if (Kp) {
        const uint32_t q3 = fresh(rj);
        K0 = ld(Kp, plane(kk, 0), q3);
        K1 = ld(Kp, plane(kk, 1), q3);
        K2 = ld(Kp, plane(kk, 2), q3);
      }
    }
    c.a2[0] = a0; c.a2[1] = a1; c.a2[2] = a2;
    c.a2ym = am;
    c.K[0] = K0; c.K[1] = K1; c.K[2] = K2;
  };
  struct Hold {
    float x, y, z, xm, zm;  // old faces at (i, j, k) and at (i, j - 1, k)
  };
  auto load_hold = [&](int kk, Hold &h) {
    const uint32_t q = fresh(rj), m = fresh(rm);
    h.x = ld(p.aux, plane(kk, 0), q);
    h.y = ld(p.aux, plane(kk, 1), q);
    h.z = ld(p.aux, plane(kk, 2), q);
    h.xm = ld(p.aux, plane(kk, 0), m);
    h.zm = ld(p.aux, plane(kk, 2), m);
  };

  // ---- prologue
  RowE c0 = row3(k0, rj), m0 = row3(k0, rm);
  RowE c1 = row3(k0 + 1, rj), m1 = row3(k0 + 1, rm);
  float p0x = ld(p.e, plane(k0, 0), rp), p0z = ld(p.e, plane(k0, 2), rp);
  float p1x = ld(p.e, plane(k0 + 1, 0), rp), p1z = ld(p.e, plane(k0 + 1, 2), rp);
  YeeNode nd;
  load_node(k0, load_flags(k0), nd);
  uint32_t fl_next = load_flags(k0 + 1);  // flags of the plane after nd's
  Hold ho;
  load_hold(k0, ho);
  float ezm = 0.0f, hy_km = 0.0f, hx_km = 0.0f, a2zm = 0.0f;
  if (k0 > 0) {
    // the x- and y-edges of plane k0 need the x- and y-normal faces of plane k0 - 1
    const RowE cm = row3(k0 - 1, rj);
    const float pmz = ld(p.e, plane(k0 - 1, 2), rp);
    const double dzm = G.idz[k0 - 1];
    const float hy = hface(ld(p.aux, plane(k0 - 1, 1), rj), cm.z, lane_next(cm.z), dxi, c0.x, cm.x, dzm, cdt);
    const float hx = hface(ld(p.aux, plane(k0 - 1, 0), rj), pmz, cm.z, dyj, cm.y, c0.y, dzm, cdt);
    hy_km = fy ? hy : 0.0f;
    hx_km = fx ? hx : 0.0f;
    ezm = cm.z;
    a2zm = ld(cf, plane(k0 - 1, 5), rj);
  }

  // One plane.  All but the last also request what the planes after it need,
  // with no branch round a request or a store (see st_plane).
  auto step_plane = [&](int k, auto more) {
    constexpr bool kMore = decltype(more)::value;
    // next plane's e in flight while this plane is computed
    RowE c2{0.0f, 0.0f, 0.0f}, m2{0.0f, 0.0f, 0.0f};
    float p2x = 0.0f, p2z = 0.0f;
    if constexpr (kMore) {
      const uint32_t qj = fresh(rj), qm = fresh(rm), qp = fresh(rp);
      c2 = row3(k + 2, qj);
      m2 = row3(k + 2, qm);
      p2x = ld(p.e, plane(k + 2, 0), qp);
      p2z = ld(p.e, plane(k + 2, 2), qp);
    }
    const double dzk = uniform_entry(G.idz, min(k, nz - 1)), dhz = uniform_entry(G.ihz, k);
    const bool kin = k < nz;
    // h^{n+1/2}: own faces and the z- and x-normal faces of row j - 1
    const float ey_n = lane_next(c0.y), ez_n = lane_next(c0.z), eym_n = lane_next(m0.y);
    float hz_c = hface(ho.z, c0.x, p0x, dyj, ey_n, c0.y, dxi, cdt);
    float hy_c = hface(ho.y, c0.z, ez_n, dxi, c1.x, c0.x, dzk, cdt);
    float hx_c = hface(ho.x, p0z, c0.z, dyj, c0.y, c1.y, dzk, cdt);
    float hz_jm = hface(ho.zm, m0.x, c0.x, dym, eym_n, m0.y, dxi, cdt);
    float hx_jm = hface(ho.xm, c0.z, m0.z, dym, m0.y, m1.y, dzk, cdt);
    hz_c = fz ? hz_c : 0.0f;
    hy_c = (fy && kin) ? hy_c : 0.0f;
    hx_c = (fx && kin) ? hx_c : 0.0f;
    hz_jm = fzm ? hz_jm : 0.0f;
    hx_jm = (fxm && kin) ? hx_jm : 0.0f;
    const float hz_im = lane_prev(hz_c), hy_im = lane_prev(hy_c);
    // (faces that do not exist are 0 and their entries stay 0)
    st_plane(p.oaux, plane(k, 0), sz, so, hx_c);
    st_plane(p.oaux, plane(k, 1), sz, so, hy_c);
    st_plane(p.oaux, plane(k, 2), sz, so, hz_c);
    if constexpr (kMore) load_hold(k + 1, ho);

    // e^{n+1} on the own x-, y-, z-edges (0 on PEC faces and on edges that do
    // not exist)
    const bool pec_k = (k == 0 && (pec & 16)) || (k == nz && (pec & 32));
    const bool zero_d[3] = {zx || pec_k, zy || pec_k, zz || !kin};
    const double cc[3] = {
        (double(hz_c) - double(hz_jm)) * dhy - (double(hy_c) - double(hy_km)) * dhz,
        (double(hx_c) - double(hx_km)) * dhz - (double(hz_c) - double(hz_im)) * dhx,
        (double(hy_c) - double(hy_im)) * dhx - (double(hx_c) - double(hx_jm)) * dhy};
    const float e0[3] = {c0.x, c0.y, c0.z};
    float eh[3];
    int8_t el[3];
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      // 1/(er + a) is formed here in FP64 from the stored er and 2a, so the
      // recurrence is exactly Eq. (2) for the stored pair: two separately
      // rounded FP32 coefficients would perturb the multiplier (er - a) /
      // (er + a) of the odd-even mode of good conductors (a ~ 1e4) by ~1e-7
      // per step.
      double er = double(nd.er[D]), a2 = double(nd.a2[D]), jn = 0.0;
      if (nd.fl & (1 << D)) {
        const PortTerm pt = port_terms(L.ports, port_entry(nd.er[D]), step);
        a2 = 2.0 * (0.5 * a2 + pt.g);
        er = pt.er;
        jn = pt.jn;
      }
      const double inv = rcp64(er + 0.5 * a2);
      // the loss term takes the full e (FP32 part + residual): in a good
      // conductor 2a / (er + a) ~ 2, so a residual left out of it would come
      // back into e at FP32 size every step
      const double ef = e_join(e0[D], nd.lo[D]);
      const double dl = -(a2 * ef + cdt * cc[D] + jn - double(nd.K[D])) * inv;
      e_split(ef + dl, eh[D], el[D]);
      eh[D] = zero_d[D] ? 0.0f : eh[D];
      el[D] = zero_d[D] ? int8_t(0) : el[D];
    }
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      st_plane(p.oe, plane(k, D), sz, so, eh[D]);
      st_plane(elo, plane(k, D), sz, so, el[D]);
    }
    // Joule power of e^n at the node, from its six incident edges
    const float a2xm = lane_prev(nd.a2[0]), exm = lane_prev(c0.x);
    if (acc_joule && own && (nd.fl & kFlagSigma)) {
      const double az[2] = {uniform_entry(G.azl, k), uniform_entry(G.azh, k)};
      const double ax[2] = {S.a[0][wave][lane], S.a[1][wave][lane]}, ay[2] = {S.a[2][wave][lane], S.a[3][wave][lane]};
      const double a6[6] = {0.5 * double(nd.a2[0]), 0.5 * double(nd.a2[1]), 0.5 * double(nd.a2[2]),
                            i > 0 ? 0.5 * double(a2xm) : 0.0, jm_ok ? 0.5 * double(nd.a2ym) : 0.0,
                            k > 0 ? 0.5 * double(a2zm) : 0.0};
      const double v[6] = {double(c0.x), double(c0.y), double(c0.z), double(exm), double(m0.y), double(ezm)};
      const double P = node_joule(a6, ax, ay, az, v, L.jf);
      // one thread per node: the add is not contended and its result is the plain sum
      if (P != 0.0) unsafeAtomicAdd(L.psum + plane(k, 0) + fresh(rj), P);
    }
    ezm = c0.z;
    hy_km = hy_c;
    hx_km = hx_c;
    a2zm = handed_on(nd.a2[2]);
    if constexpr (kMore) {
      load_node(k + 1, handed_on(fl_next), nd);
      fl_next = load_flags(k + 2);
    }
    c0 = c1; c1 = c2;
    m0 = m1; m1 = m2;
    p0x = p1x; p0z = p1z; p1x = p2x; p1z = p2z;
  };
  for (int k = k0; k + 1 < k1; ++k) step_plane(k, std::true_type{});
  step_plane(k1 - 1, std::false_type{});
}

// ---- mixed, tiles: the same march for meshes that stream from HBM ------------
// One block: 64 x 4 nodes (a wave is a row, so that its loads and stores are
// runs of whole 64-byte sectors) over a z-chunk.  e is staged in LDS with its
// halo; the new faces of a plane are formed once per block, one plane ahead of
// the edges, and handed on through LDS: waves 0 and 1 form the ones of row
// j0 - 1 and column i0 - 1 in addition.  One barrier per plane; every load is
// requested a plane before its use and every store is unconditional (st_plane).
//
// Bound by HBM.  Arithmetic costs nothing here (with the faces in FP32 and a
// 1-instruction reciprocal, in a timing copy, the step takes the same time),
// and time goes with bytes: without the residuals 2489 of 2753 us on the
// 1024x1024x128 package, without the h stores 2338, without the old h 2423.  A
// kernel that only moves this march's 66 bytes per node in its order takes
// 2000 us there (in plane order, without neighbours, 1510).  The rows' pitch
// of 64 bytes makes every other row straddle 128-byte lines, which costs that
// kernel 10 %.  What is left is the halo.  Runs | tiles before and after
// the blocks were grouped (grouped_block): package 2936 | 2754 | 2496 us,
// 1024x512x64 809 | 744 | 644, 384x384x96 351 | 333 | 291, 256x256x64
// 102.4 | 100.7 | 90.
//
// LDS of one block: four e planes (one of them being staged) and two planes of
// new faces, both with the halo that the block's nodes read, and the
// dual-width shares of its columns and rows.
struct YeeTile {
  float e[4][3][MY + 2][MX + 2];
  float h[2][3][MY + 1][MX + 1];
  double ax[2][MX], ay[2][MY];
};

template <bool NT>
__device__ __forceinline__ void em_march_tile_yee(const EmLaunch &L, const EmPtrs<float> &p, int64_t step, int tx,
                                                  int ty, int kc, int kchunk, int acc_joule, YeeTile &S) {
  const DevGrid &g = L.g;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const uint32_t sy = uint32_t(g.sy), sz = uint32_t(g.sz), cs = g.cs;
  const Geo G(g.geo, nx, ny, nz);
  const float *cf = static_cast<const float *>(L.coef);
  const float *Kp = L.K;
  int8_t *elo = L.elo;
  const double cdt = L.cdt;
  const int tid = int(threadIdx.y) * BX + int(threadIdx.x), lx = tid % MX, ly = tid / MX;
  const int i0 = tx * MX, j0 = ty * MY, i = i0 + lx, j = j0 + ly;
  const int k0 = kc * kchunk, k1 = min(k0 + kchunk, nz + 1);
  const bool active = i <= nx && j <= ny;
  const int ic = min(i, nx), jc = min(j, ny);
  if (tid < MX) {
    S.ax[0][tid] = G.axl[min(i0 + tid, nx)];
    S.ax[1][tid] = G.axh[min(i0 + tid, nx)];
  }
  if (tid < MY) {
    S.ay[0][tid] = G.ayl[min(j0 + tid, ny)];
    S.ay[1][tid] = G.ayh[min(j0 + tid, ny)];
  }
  const double dxi = G.idx[min(i, nx - 1)], dhx = G.ihx[ic];
  const double dyj = G.idy[min(j, ny - 1)], dhy = G.ihy[jc];
  const int pec = g.pec;
  const bool pec_i = (i == 0 && (pec & 1)) || (i == nx && (pec & 2));
  const bool pec_j = (j == 0 && (pec & 4)) || (j == ny && (pec & 8));
  const bool zx = pec_j || i >= nx, zy = pec_i || j >= ny, zz = pec_i || pec_j;
  const uint32_t rj = uint32_t(jc) * sy + uint32_t(ic);
  const uint32_t rx = ic > 0 ? rj - 1 : rj, ry = jc > 0 ? rj - sy : rj;
  const uint32_t so = active ? rj : 0xffffffffu;
  auto plane = [&](int kk, int c) -> int64_t { return int64_t(c) * cs + int64_t(min(max(kk, 0), nz)) * int64_t(sz); };
  // own faces that exist (independent of the plane, apart from k < nz)
  const bool fz = i < nx && j < ny, fy = i < nx && j <= ny, fx = i <= nx && j < ny;
  // the block's faces of row j0 - 1 (wave 0: hz, hx) and of column i0 - 1
  // (wave 1: hz, hy)
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const bool hrow = wave == 0, hcol = wave == 1;
  const int hq = min(tid % 64, MY - 1);  // lanes past the column repeat its last row
  const int hi = hcol ? i0 - 1 : i, hj = hcol ? j0 + hq : j0 - 1;
  const bool hin = hi >= 0 && hj >= 0 && hi <= nx && hj <= ny;
  const bool hfz = hin && hi < nx && hj < ny;
  const uint32_t rh = uint32_t(min(max(hj, 0), ny)) * sy + uint32_t(min(max(hi, 0), nx));
  const double hdx = G.idx[min(max(hi, 0), nx - 1)], hdy = G.idy[min(max(hj, 0), ny - 1)];
  const int hlx = hcol ? 0 : lx + 1, hly = hcol ? hq + 1 : 0;

  constexpr int NPF = ((MY + 2) * (MX + 2) + MX * MY - 1) / (MX * MY);
  struct Staged {
    float v[NPF][3];
  };
  uint32_t at[NPF];
  bool in[NPF];
#pragma unroll
  for (int q = 0; q < NPF; ++q) {
    const int t = tid + q * MX * MY < (MY + 2) * (MX + 2) ? tid + q * MX * MY : tid;
    const int r = t / (MX + 2), c = t - r * (MX + 2);
    const int gi = i0 - 1 + c, gj = j0 - 1 + r;
    in[q] = gi >= 0 && gi <= nx && gj >= 0 && gj <= ny;
    at[q] = uint32_t(min(max(gj, 0), ny)) * sy + uint32_t(min(max(gi, 0), nx));
  }
  auto fetch = [&](int kk, Staged &pf) {
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      const uint32_t a = fresh(at[q]);
#pragma unroll
      for (int c = 0; c < 3; ++c) pf.v[q][c] = ld_plane(p.e, plane(kk, c), a);
    }
  };
  auto commit = [&](int kk, const Staged &pf) {
    const bool pk = kk >= 0 && kk <= nz;
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      const int t = tid + q * MX * MY;
      if (t < (MY + 2) * (MX + 2)) {
        const int r = t / (MX + 2), c = t - r * (MX + 2);
#pragma unroll
        for (int d = 0; d < 3; ++d) S.e[kk & 3][d][r][c] = pk && in[q] ? pf.v[q][d] : 0.0f;
      }
    }
  };
  struct Hold {
    float x, y, z, a, b;  // old own faces, and the halo's z and x or y
  };
  Hold ho;
  auto load_hold = [&](int kk) {
    const uint32_t q = fresh(rj);
    ho.x = ld_plane<NT>(p.aux, plane(kk, 0), q);
    ho.y = ld_plane<NT>(p.aux, plane(kk, 1), q);
    ho.z = ld_plane<NT>(p.aux, plane(kk, 2), q);
    if (wave < 2) {
      const uint32_t m = fresh(rh);
      ho.a = ld_plane(p.aux, plane(kk, 2), m);
      ho.b = ld_plane(p.aux, plane(kk, hrow ? 0 : 1), m);
    }
  };
  YeeNode nd;
  float a2xm = 0.0f;
  auto load_node = [&](int kk) {
    const uint32_t q = fresh(rj);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      nd.er[d] = ld_plane<NT>(cf, plane(kk, d), q);
      nd.lo[d] = ld_plane(elo, plane(kk, d), q);
    }
  };
  auto load_loss = [&](int kk) {
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, am = 0.0f, an = 0.0f, K0 = 0.0f, K1 = 0.0f, K2 = 0.0f;
    if (__any(nd.fl & kFlagSigma)) {
      const uint32_t q2 = fresh(rj);
      a0 = ld_plane(cf, plane(kk, 3), q2);
      a1 = ld_plane(cf, plane(kk, 4), q2);
      a2 = ld_plane(cf, plane(kk, 5), q2);
      an = ld_plane(cf, plane(kk, 3), fresh(rx));
      am = ld_plane(cf, plane(kk, 4), fresh(ry));
      if (Kp) {
        const uint32_t q3 = fresh(rj);
        K0 = ld_plane(Kp, plane(kk, 0), q3);
        K1 = ld_plane(Kp, plane(kk, 1), q3);
        K2 = ld_plane(Kp, plane(kk, 2), q3);
      }
    }
    nd.a2[0] = a0; nd.a2[1] = a1; nd.a2[2] = a2;
    nd.a2ym = am;
    a2xm = an;
    nd.K[0] = K0; nd.K[1] = K1; nd.K[2] = K2;
  };
  auto load_flags = [&](int kk) -> uint32_t { return ld_plane(g.flags, plane(kk, 0), fresh(rj)); };
  struct Faces {
    float x, y, z;
  };
  // faces of plane kk from the staged e, own ones returned and stored, all of
  // them left in LDS for the block
  auto faces = [&](int kk) -> Faces {
    const double dz = uniform_entry(G.idz, min(kk, nz - 1));
    const bool kin = kk < nz;
    const int sl = kk & 3, su = (kk + 1) & 3, hs = kk & 1;
    const int r = ly + 1, c = lx + 1;
    Faces f;
    const float ex = S.e[sl][0][r][c], ey = S.e[sl][1][r][c], ez = S.e[sl][2][r][c];
    f.z = hface(ho.z, ex, S.e[sl][0][r + 1][c], dyj, S.e[sl][1][r][c + 1], ey, dxi, cdt);
    f.y = hface(ho.y, ez, S.e[sl][2][r][c + 1], dxi, S.e[su][0][r][c], ex, dz, cdt);
    f.x = hface(ho.x, S.e[sl][2][r + 1][c], ez, dyj, ey, S.e[su][1][r][c], dz, cdt);
    f.z = fz ? f.z : 0.0f;
    f.y = fy && kin ? f.y : 0.0f;
    f.x = fx && kin ? f.x : 0.0f;
    S.h[hs][0][r][c] = f.x;
    S.h[hs][1][r][c] = f.y;
    S.h[hs][2][r][c] = f.z;
    if (wave < 2) {
      const int hr = hly, hc = hlx, dr = hrow ? 1 : 0, dc = hrow ? 0 : 1;
      const float x0 = S.e[sl][0][hr][hc], y0 = S.e[sl][1][hr][hc], z0 = S.e[sl][2][hr][hc];
      const float z = hface(ho.a, x0, S.e[sl][0][hr + 1][hc], hdy, S.e[sl][1][hr][hc + 1], y0, hdx, cdt);
      S.h[hs][2][hr][hc] = hfz ? z : 0.0f;
      // hx: (ez(j+1) - ez) / dy + (ey - ey(k+1)) / dz; hy: (ez - ez(i+1)) / dx + (ex(k+1) - ex) / dz
      const float zn = S.e[sl][2][hr + dr][hc + dc], u0 = hrow ? y0 : x0, un = S.e[su][hrow ? 1 : 0][hr][hc];
      const float w = hface(ho.b, hrow ? zn : z0, hrow ? z0 : zn, hrow ? hdy : hdx, hrow ? u0 : un, hrow ? un : u0,
                            dz, cdt);
      S.h[hs][hrow ? 0 : 1][hr][hc] = hin && kin ? w : 0.0f;
    }
    const int64_t o = int64_t(kk) * int64_t(sz);
    st_plane<NT>(p.oaux, o, sz, so, f.x);
    st_plane<NT>(p.oaux, o + cs, sz, so, f.y);
    st_plane<NT>(p.oaux, o + 2 * int64_t(cs), sz, so, f.z);
    return f;
  };

  // ---- prologue
  nd.fl = load_flags(k0);
  float hx_km = 0.0f, hy_km = 0.0f, ezm = 0.0f, a2zm = 0.0f;
  float oy = ld_plane(p.aux, plane(k0 - 1, 1), rj), ox = ld_plane(p.aux, plane(k0 - 1, 0), rj);
  a2zm = ld_plane(cf, plane(k0 - 1, 5), rj);
  load_hold(k0);
  {
    Staged q0, q1, q2, q3;
    fetch(k0 - 1, q0);
    fetch(k0, q1);
    fetch(k0 + 1, q2);
    fetch(k0 + 2, q3);
    commit(k0 - 1, q0);
    commit(k0, q1);
    commit(k0 + 1, q2);
    commit(k0 + 2, q3);
  }
  __syncthreads();
  if (k0 > 0) {
    const double dzm = G.idz[k0 - 1];
    const int sl = (k0 - 1) & 3, su = k0 & 3, r = ly + 1, c = lx + 1;
    ezm = S.e[sl][2][r][c];
    hy_km = hface(oy, ezm, S.e[sl][2][r][c + 1], dxi, S.e[su][0][r][c], S.e[sl][0][r][c], dzm, cdt);
    hx_km = hface(ox, S.e[sl][2][r + 1][c], ezm, dyj, S.e[sl][1][r][c], S.e[su][1][r][c], dzm, cdt);
    hy_km = fy ? hy_km : 0.0f;
    hx_km = fx ? hx_km : 0.0f;
  }
  Staged pf;
  Faces h = faces(k0);
  load_hold(k0 + 1);
  load_node(k0);
  load_loss(k0);
  uint32_t fl_next = load_flags(k0 + 1);
  __syncthreads();

  // kStage 2: planes k + 1 and k + 2 follow; 1: plane k + 1 follows; 0: the last
  auto step_plane = [&](int k, auto stage) {
    constexpr int kStage = decltype(stage)::value;
    Faces hn{0.0f, 0.0f, 0.0f};
    if constexpr (kStage == 2) fetch(k + 3, pf);
    if constexpr (kStage >= 1) hn = faces(k + 1);
    if constexpr (kStage == 2) load_hold(k + 2);
    const int r = ly + 1, c = lx + 1, sl = k & 3, hs = k & 1;
    const double dhz = uniform_entry(G.ihz, k);
    const bool kin = k < nz;
    const bool pec_k = (k == 0 && (pec & 16)) || (k == nz && (pec & 32));
    const bool zero_d[3] = {zx || pec_k, zy || pec_k, zz || !kin};
    const float hz_jm = S.h[hs][2][r - 1][c], hx_jm = S.h[hs][0][r - 1][c];
    const float hz_im = S.h[hs][2][r][c - 1], hy_im = S.h[hs][1][r][c - 1];
    const double cc[3] = {(double(h.z) - double(hz_jm)) * dhy - (double(h.y) - double(hy_km)) * dhz,
                          (double(h.x) - double(hx_km)) * dhz - (double(h.z) - double(hz_im)) * dhx,
                          (double(h.y) - double(hy_im)) * dhx - (double(h.x) - double(hx_jm)) * dhy};
    const float e0[3] = {S.e[sl][0][r][c], S.e[sl][1][r][c], S.e[sl][2][r][c]};
    const int64_t o = int64_t(k) * int64_t(sz);
#pragma unroll
    for (int D = 0; D < 3; ++D) {
      double er = double(nd.er[D]), a2 = double(nd.a2[D]), jn = 0.0;
      if (nd.fl & (1 << D)) {
        const PortTerm pt = port_terms(L.ports, port_entry(nd.er[D]), step);
        a2 = 2.0 * (0.5 * a2 + pt.g);
        er = pt.er;
        jn = pt.jn;
      }
      const double inv = rcp64(er + 0.5 * a2);
      const double ef = e_join(e0[D], nd.lo[D]);
      const double dl = -(a2 * ef + cdt * cc[D] + jn - double(nd.K[D])) * inv;
      float eh;
      int8_t el;
      e_split(ef + dl, eh, el);
      st_plane<NT>(p.oe, o + D * int64_t(cs), sz, so, zero_d[D] ? 0.0f : eh);
      st_plane<NT>(elo, o + D * int64_t(cs), sz, so, zero_d[D] ? int8_t(0) : el);
    }
    if constexpr (kStage >= 1) load_node(k + 1);
    if (acc_joule && active && (nd.fl & kFlagSigma)) {
      const double az[2] = {uniform_entry(G.azl, k), uniform_entry(G.azh, k)};
      const double ax[2] = {S.ax[0][lx], S.ax[1][lx]}, ay[2] = {S.ay[0][ly], S.ay[1][ly]};
      const double a6[6] = {0.5 * double(nd.a2[0]), 0.5 * double(nd.a2[1]), 0.5 * double(nd.a2[2]),
                            i > 0 ? 0.5 * double(a2xm) : 0.0, j > 0 ? 0.5 * double(nd.a2ym) : 0.0,
                            k > 0 ? 0.5 * double(a2zm) : 0.0};
      const double v[6] = {double(e0[0]), double(e0[1]), double(e0[2]), double(S.e[sl][0][r][c - 1]),
                           double(S.e[sl][1][r - 1][c]), double(ezm)};
      const double P = node_joule(a6, ax, ay, az, v, L.jf);
      if (P != 0.0) unsafeAtomicAdd(L.psum + o + fresh(rj), P);
    }
    ezm = e0[2];
    hy_km = h.y;
    hx_km = h.x;
    a2zm = handed_on(nd.a2[2]);
    if constexpr (kStage >= 1) {
      h = hn;
      nd.fl = handed_on(fl_next);
      load_loss(k + 1);
      fl_next = load_flags(k + 2);
    }
    if constexpr (kStage == 2) commit(k + 3, pf);
    if constexpr (kStage >= 1) __syncthreads();
  };
  int k = k0;
  for (; k + 2 < k1; ++k) step_plane(k, std::integral_constant<int, 2>{});
  if (k + 1 < k1) step_plane(k++, std::integral_constant<int, 1>{});
  step_plane(k, std::integral_constant<int, 0>{});
}

// Which of the two FP64 tiles a mesh takes.  32 x 8 reads the smaller halo; 64 x 4
// leaves fewer lanes idle where the rows of nodes are few, and is taken where
// that makes its blocks a fifth fewer, unless all blocks find a CU of their own
// anyway (chunks of one plane).  us per step, 32 x 8 | 64 x 4:
//   4001x2x61 nodes 27.6 | 16.1   1001x4x401 42.7 | 33.1   97x4x1501 22.9 | 16.7
//   501x9x443 56.7 | 42.3   501x12x332 46.9 | 41.0 (blocks 0.75 of the others')
//   501x17x234 45.3 | 43.1   501x20x59 16.1 | 16.8 (0.83)   64x4x64 5.2 | 5.6 (128 blocks)
__host__ __device__ inline bool em_flat(const DevGrid &g) {
  const int64_t tile = int64_t((g.nx + kTileX) / kTileX) * ((g.ny + kTileY) / kTileY),
                flat = int64_t((g.nx + kFlatX) / kFlatX) * ((g.ny + kFlatY) / kFlatY);
  return flat * 5 <= tile * 4 && tile * (g.nz + 1) > 256;
}

// MARCH: the FP64 march in 32 x 8 or 64 x 4 tiles, the mixed runs or tiles, or
// whichever of a precision's two the mesh takes.  NT: data used once goes past
// the caches (FP64, mixed tiles).
enum { kMarchFp64, kMarchRuns, kMarchTiles, kMarchMixed, kMarchFp64Flat, kMarchFp64Any };
template <typename T, int MARCH, bool NT>
__device__ __forceinline__ void march_tile(const EmLaunch &L, const EmPtrs<T> &p, int64_t step, int tx, int ty, int kc,
                                           int kchunk, int acc_joule) {
  using Tile = MarchSmem<T, kTileX, kTileY>;
  using Flat = MarchSmem<T, kFlatX, kFlatY>;
  if constexpr (MARCH == kMarchFp64) {
    __shared__ Tile S;
    em_march_tile<T, kTileX, kTileY, NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, S);
  } else if constexpr (MARCH == kMarchFp64Flat) {
    __shared__ Flat S;
    em_march_tile<T, kFlatX, kFlatY, NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, S);
  } else if constexpr (MARCH == kMarchFp64Any) {
    __shared__ __align__(16) char S[std::max(sizeof(Tile), sizeof(Flat))];
    if (em_flat(L.g))
      em_march_tile<T, kFlatX, kFlatY, NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, *reinterpret_cast<Flat *>(S));
    else
      em_march_tile<T, kTileX, kTileY, NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, *reinterpret_cast<Tile *>(S));
  } else if constexpr (MARCH == kMarchRuns) {
    __shared__ YeeSmem S;
    em_march_run_yee(L, p, step, tx, kc, kchunk, acc_joule, S);
  } else if constexpr (MARCH == kMarchTiles) {
    __shared__ YeeTile S;
    em_march_tile_yee<NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, S);
  } else {
    __shared__ __align__(16) char S[std::max(sizeof(YeeTile), sizeof(YeeSmem))];
    if (em_runs(L.g))
      em_march_run_yee(L, p, step, tx, kc, kchunk, acc_joule, *reinterpret_cast<YeeSmem *>(S));
    else
      em_march_tile_yee<NT>(L, p, step, tx, ty, kc, kchunk, acc_joule, *reinterpret_cast<YeeTile *>(S));
  }
}

template <typename T, int MARCH, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void em_march_kernel(
    EmLaunch L, EmPtrs<T> p, int ntx, int nty, int nkc, int kchunk, int acc_joule) {
  const int b = grouped_block(blockIdx.x, ntx * nty * nkc);
  const int tx = b % ntx, ty = (b / ntx) % nty, kc = b / (ntx * nty);
  march_tile<T, MARCH, NT>(L, p, L.step, tx, ty, kc, kchunk, acc_joule);
}

// ---- two steps as a wavefront over z-slabs (temporal blocking) -------------
// One launch runs the tiles of two z-ranges of chunks: blocks [0, nA) make
// step n on chunks [kcA, kcA + nkcA) with pointer set pa, blocks [nA, nb)
// make step n + 1 on chunks [kcB, kcB + nkcB) with pb.  The host orders the
// launches so that the n + 1 range runs only after the step-n tiles it
// reads (its own slab and the planes next to it) are complete and after
// every step-n tile that reads the planes it overwrites; see
// launch_em_pair_schedule.  Each tile computes exactly what it computes in
// a one-step launch, so the two steps are bitwise those of two launches.
template <typename T, int MARCH>
__global__ __launch_bounds__(256) void em_march_pair_kernel(EmLaunch L, EmPtrs<T> pa, EmPtrs<T> pb, int ntx, int nty,
                                                            int kcA, int nkcA, int kcB, int nkcB, int kchunk,
                                                            int acc_a) {
  const int cols = ntx * nty, nA = cols * nkcA, nb = nA + cols * nkcB;
  const int b = xcd_remap(blockIdx.x, nb);
  const bool second = b >= nA;
  const int r = second ? b - nA : b;
  const int tx = r % ntx, ty = (r / ntx) % nty, kc = (second ? kcB : kcA) + r / cols;
  if (second)
    march_tile<T, MARCH, false>(L, pb, L.step + 1, tx, ty, kc, kchunk, 1);
  else
    march_tile<T, MARCH, false>(L, pa, L.step, tx, ty, kc, kchunk, acc_a);
}

// A pointer that was itself loaded from memory, as one into global memory: the
// compiler knows that only of kernel arguments, and reads through any other
// with flat loads, which need 64-bit addresses per lane and are counted with
// the LDS accesses, so that every wait for LDS waits for them as well.  A step
// of twelve uneven variants (8.0 M nodes): 224 -> 185 us in mixed precision,
// 234 -> 210 in FP64.
template <typename T>
__device__ __forceinline__ T *in_global(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}

// ---- batched: one launch walks the (variant, tile) list of all variants ----
// Item = (variant, tile x, tile y, z chunk).  s is the step's offset from the
// descriptors' step, so a captured segment of steps can be replayed after the
// descriptors are staged again.  (As a launch argument: a counter in device
// memory took a second launch per step, about 4 us.)  Held to 4 waves per SIMD
// (at most 128 VGPRs).
template <typename T, int MARCH, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void em_march_batched(const BatchVar *vars,
                                                                                               const int4 *items,
                                                                                               int n_items, int64_t s) {
  const int b = grouped_block(blockIdx.x, n_items);
  const int4 it = items[b];
  const BatchVar &V = vars[it.x];
  const int64_t step = V.step0 + s;
  EmPtrs<T> p;
  if (MARCH == kMarchMixed) {
    const int cur = int((V.cur0 + s) & 1), o = 1 - cur;
    p.e = in_global((const T *)V.e[cur][0]);
    p.aux = in_global((const T *)V.h[cur][0]);
    p.oe = in_global((T *)V.e[o][0]);
    p.oaux = in_global((T *)V.h[o][0]);
  } else {
    const int cur = int((V.cur0 + s) % 3), prv = (cur + 2) % 3, nxt = (cur + 1) % 3;
    p.e = in_global((const T *)V.e[cur][0]);
    p.aux = in_global((const T *)V.e[prv][0]);
    p.oe = in_global((T *)V.e[nxt][0]);
    p.oaux = nullptr;
  }
  const int acc = (s == 0) ? V.acc_joule0 : int(step % V.R != 0);
  EmLaunch L = V.L;
  L.g.geo = in_global(L.g.geo);
  L.g.flags = in_global(L.g.flags);
  L.ports.rec = in_global(L.ports.rec);
  L.ports.wave = in_global(L.ports.wave);
  L.ports.wt = in_global(L.ports.wt);
  L.ports.J = in_global(L.ports.J);
  L.ports.Ja = in_global(L.ports.Ja);
  L.ports.er = in_global(L.ports.er);
  L.psum = in_global(L.psum);
  L.coef = in_global(static_cast<const T *>(L.coef));
  L.K = in_global(L.K);
  L.elo = in_global(L.elo);
  march_tile<T, MARCH, NT>(L, p, step, it.y, it.z, it.w, V.kchunk, acc);
}

// ---- block reductions (wave64 shuffles, then LDS across the waves) --------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

template <int NS, int NM>
__device__ __forceinline__ void block_reduce_store(const double (&sums)[NS], const double (&maxs)[NM], double *out) {
  __shared__ double red[4][NS + NM];
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int lane = tid & 63, wv = tid >> 6;
  double v[NS + NM];
#pragma unroll
  for (int q = 0; q < NS; ++q) v[q] = wave_sum(sums[q]);
#pragma unroll
  for (int q = 0; q < NM; ++q) v[NS + q] = wave_max(maxs[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < NS + NM; ++q) red[wv][q] = v[q];
  __syncthreads();
  if (tid == 0) {
    const int nw = (blockDim.x * blockDim.y + 63) / 64;
#pragma unroll
    for (int q = 0; q < NS + NM; ++q) {
      double acc = red[0][q];
      for (int w = 1; w < nw; ++w) acc = q < NS ? acc + red[w][q] : fmax(acc, red[w][q]);
      out[q] = acc;
    }
  }
}

inline dim3 node_grid(const DevGrid &g) { return dim3((g.nx + 1 + BX - 1) / BX, (g.ny + 1 + BY - 1) / BY, g.nz + 1); }

// Joule of the current field (the deferred last step) at node (i,j,k), with
// the same arithmetic as the march kernel (missing low-side edges read 0).
template <typename T>
__device__ __forceinline__ double pending_joule(const DevGrid &g, const T *const *e, const T *cf, int i, int j, int k,
                                                int64_t n, double jf) {
  const double ax[2] = {g.al[0][i], g.ah[0][i]}, ay[2] = {g.al[1][j], g.ah[1][j]}, az[2] = {g.al[2][k], g.ah[2][k]};
  const double v[6] = {double(e[0][n]), double(e[1][n]), double(e[2][n]), i > 0 ? double(e[0][n - 1]) : 0.0,
                       j > 0 ? double(e[1][n - g.sy]) : 0.0, k > 0 ? double(e[2][n - g.sz]) : 0.0};
  return joule_from_coef(cf, g.cs, uint32_t(n), uint32_t(g.sy), uint32_t(g.sz), i, j, k, ax, ay, az, v, jf);
}

// Per-node coefficients of the own x, y, z edges: eps_r and the normalised
// material conductance a = dt sigma(T) / (2 eps0), formed in FP64 from the
// cells around the node (their ids read once, the material table in LDS) and
// stored at the field precision.  An edge that does not exist keeps eps_r =
// 1 and a = 0 and reads no temperature.
//
// FULL: every node, with eps_r and the ports' entries (at bind and restore).
// Otherwise the refresh after a temperature change: only edges next to a cell
// whose sigma depends on it change, and eps_r never does.  One block: 64 x 4
// nodes over up to 8 planes (launch_coef; the mask of planes has room for 32),
// whose flags it reads at once; planes without such
// a node cost nothing more, and a block without one leaves before it loads the
// material table.
// Bound by the bytes of those nodes (about 80 each in mixed precision): 95 us
// on 385x385x97 nodes, 112 before in blocks of one plane.
template <typename T, bool FULL>
__global__ __launch_bounds__(256) void coef_kernel(DevGrid g, DevPorts P, const T *th, T *cf, CoefK ck, int ntx,
                                                   int nty, int kchunk) {
  __shared__ LdsMat MT;
  const int b = grouped_block(blockIdx.x, gridDim.x);
  const int i = (b % ntx) * BX + int(threadIdx.x), j = (b / ntx) % nty * BY + int(threadIdx.y);
  const int k0 = b / (ntx * nty) * kchunk, k1 = min(k0 + kchunk, g.nz + 1);
  const bool in = i <= g.nx && j <= g.ny;
  const int64_t n0 = in ? int64_t(j) * g.sy + i : 0;
  uint32_t planes = 0;  // bit k - k0: the node needs work
  if (FULL) {
    planes = in ? ~0u : 0;
  } else {
    for (int k = k0; k < k1; ++k)
      planes |= uint32_t(in && (g.flags[n0 + k * g.sz] & kFlagTcr)) << (k - k0);
    if (!__syncthreads_or(planes != 0)) return;
  }
  lds_mat_load(g, MT);
  if (!planes) return;
  const double ax[2] = {g.al[0][i], g.ah[0][i]}, ay[2] = {g.al[1][j], g.ah[1][j]};
  const LTcr TC{&MT};
  for (int k = k0; k < k1; ++k) {
    if (!(planes >> (k - k0) & 1)) continue;
    const int64_t n = n0 + k * g.sz;
    const double az[2] = {g.al[2][k], g.ah[2][k]};
    LCell CL;
    CL.M = &MT;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int ox = q & 1, oy = (q >> 1) & 1, oz = q >> 2;
      const int ci = i - 1 + ox, cj = j - 1 + oy, ck2 = k - 1 + oz;
      const bool ok = ci >= 0 && ci < g.nx && cj >= 0 && cj < g.ny && ck2 >= 0 && ck2 < g.nz;
      CL.id[q] = int(g.mat[ok ? n + (ox - 1) + (oy - 1) * g.sy + (oz - 1) * g.sz : n]);
      CL.id[q] = ok ? CL.id[q] : 0;
    }
    const bool ex[3] = {i < g.nx, j < g.ny, k < g.nz};
    // every load up front: the temperatures the own edges may read and, for a
    // K update, the old 2a, K and the two fields (clamped where an edge does
    // not exist), so none waits behind a branch
    const PTh TH{{double(th[n]), double(th[ex[0] ? n + 1 : n]), double(th[ex[1] ? n + g.sy : n]),
                  double(th[ex[2] ? n + g.sz : n])}};
    const uint32_t cs = g.cs;
    float a2o[3] = {0.0f, 0.0f, 0.0f}, Ko[3] = {0.0f, 0.0f, 0.0f}, ec[3] = {0.0f, 0.0f, 0.0f},
          ep[3] = {0.0f, 0.0f, 0.0f};
    if (sizeof(T) == 4 && ck.K) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const uint32_t o = d * cs + uint32_t(n);
        a2o[d] = float(cf[(3 + d) * cs + n]);
        Ko[d] = ck.K[o];
        ec[d] = ck.e_cur[o];
        ep[d] = ck.e_prev[o];
      }
    }
    double er[3] = {1.0, 1.0, 1.0}, a[3] = {0.0, 0.0, 0.0};
    if (ex[0]) a[0] = edge_coef<0>(1, ax, ay, az, CL, TC, TH, FULL ? &er[0] : nullptr);
    if (ex[1]) a[1] = edge_coef<1>(1, ax, ay, az, CL, TC, TH, FULL ? &er[1] : nullptr);
    if (ex[2]) a[2] = edge_coef<2>(1, ax, ay, az, CL, TC, TH, FULL ? &er[2] : nullptr);
    const uint8_t fl = FULL ? g.flags[n] : 0;
    for (int d = 0; d < 3; ++d) {
      if (sizeof(T) == 4) {
        const float a2 = float(2.0 * a[d]);
        if (ck.K && ex[d]) {
          // leapfrog form: a changed from a_old to a between e_prev = e^{n-1}
          // and e_cur = e^n; K += (a - a_old) (e^n + e^{n-1})
          if (a2 != a2o[d]) {
            const uint32_t o = d * cs + uint32_t(n);
            ck.K[o] = float(double(Ko[d]) + 0.5 * (double(a2) - double(a2o[d])) * (double(ec[d]) + double(ep[d])));
          }
        }
        cf[(3 + d) * cs + n] = T(a2);
      } else {
        cf[(3 + d) * cs + n] = T(a[d]);
      }
      if (FULL) {
        const double e = er[d] > 0.0 ? er[d] : 1.0;  // an edge without cells keeps a harmless 1
        const int q = fl & (1 << d) ? find_port(P, int64_t(d) * g.ntot + n) : -1;
        if (q >= 0) P.er[q] = e;
        cf[d * cs + n] = q >= 0 ? port_code(q, T(0)) : T(e);
      }
    }
  }
}

// ---- thermal step, Eq. (5) ------------------------------------------------
// C_n V_n (theta' - theta) = dt*psum*V_n - R*dt*sum_e G_e (theta_n - theta_m),
// G_e = sum over the edge's cells of (quarter transverse area) k_c / L,
// C_n V_n = sum over the node's cell octants of rho_cp * octant volume.
// The pending Joule power of the block's last EM step is added first, with
// the conductivity of the temperature the block ran at.
//
// One block: 64 x 4 nodes (a wave is a row) over a z-chunk.  A layer of cells
// is turned into its shares of G_e and C_n V_n once, for the two node planes it
// bounds, and every node reads its temperature neighbours, material ids and
// source once per plane, requested as soon as the plane before has used its
// own.  The factors of cells, edges and neighbours that do not
// exist are 0 and their loads read the nearest entry, so no load waits behind
// a branch; only a wave with a conducting cell loads the conductances.
// Bound by HBM and the order in which it is read (about 50 bytes per node at
// 4 TB/s): 178 us on 385x385x97 nodes with the pending Joule power, 357 before
// as one node per thread, which read every neighbour, and formed each cell's
// shares, once per node.
struct TherSmem {
  double2 kr[kMatMax];    // k, rho c_p of every material
  double dx[2][BX], ix[2][BX], ax[2][BX], hx[BX];  // widths, 1 / width and dual-width shares on both sides, dual width
};

template <typename T>
struct ThermIn {
  double th, xl, xh, yl, yh, ps;  // theta of the node above, and of the four beside; source
  uint32_t m00, m10, m01, m11;    // cells of the layer above, (x, y) low or high
  uint32_t fl;                    // flags of the plane after
  T e0, e1, e2;                   // JOULE: the field on the own edges
  T a0, a1, a2, a3, a4, v3, v4;   // and, by a conductor, conductances of five edges, field on the low x, y edges
};

// JOULE: with the pending Joule power of the block's last EM step.
template <typename T, bool JOULE>
__global__ __launch_bounds__(256) void thermal_kernel(
    ThermalLaunch L, const T *e0, const T *e1, const T *e2, const T *cf, int ntx, int nty, int kchunk) {
  __shared__ TherSmem S;
  const DevGrid &g = L.g;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int lane = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.y)), tid = wave * BX + lane;
  const int b = grouped_block(blockIdx.x, gridDim.x);
  const int i0 = (b % ntx) * BX, i = i0 + lane, j = (b / ntx) % nty * BY + wave;
  const int k0 = b / (ntx * nty) * kchunk, k1 = min(k0 + kchunk, nz + 1);
  const bool in = i <= nx && j <= ny;
  const int ic = min(i, nx), jc = min(j, ny);
  const bool xl = ic > 0, xh = ic < nx, yl = jc > 0, yh = jc < ny;
  const uint32_t sy = uint32_t(g.sy), sz = uint32_t(g.sz);
  const int64_t cs = g.cs;
  const uint32_t r = uint32_t(jc) * sy + uint32_t(ic), so = in ? r : 0xffffffffu;
  const uint32_t rxl = xl ? r - 1 : r, rxh = xh ? r + 1 : r, ryl = yl ? r - sy : r, ryh = yh ? r + sy : r;
  const uint32_t rll = yl ? rxl - sy : rxl;  // the cell on both low sides
  auto plane = [&](int kk) -> int64_t { return int64_t(min(max(kk, 0), nz)) * int64_t(sz); };
  ThermIn<T> q;
  auto load = [&](int kk, bool first) {
    const int64_t o = plane(kk);
    const uint32_t c = fresh(r), cxl = fresh(rxl), cyl = fresh(ryl);
    q.m11 = ld_plane(g.mat, o, c);
    q.m01 = ld_plane(g.mat, o, cxl);
    q.m10 = ld_plane(g.mat, o, cyl);
    q.m00 = ld_plane(g.mat, o, fresh(rll));
    q.xl = ld_plane(L.theta_in, o, cxl);
    q.xh = ld_plane(L.theta_in, o, fresh(rxh));
    q.yl = ld_plane(L.theta_in, o, cyl);
    q.yh = ld_plane(L.theta_in, o, fresh(ryh));
    q.th = ld_plane(L.theta_in, plane(kk + 1), c);
    q.ps = ld_plane(L.psum, o, c);
    if constexpr (JOULE) {
      q.e0 = ld_plane(e0, o, c);
      q.e1 = ld_plane(e1, o, c);
      q.e2 = ld_plane(e2, o, c);
      T a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0, v3 = 0, v4 = 0;
      if (first || __any(q.fl & kFlagSigma)) {
        a0 = ld_plane(cf, o + 3 * cs, c);
        a1 = ld_plane(cf, o + 4 * cs, c);
        a2 = ld_plane(cf, o + 5 * cs, c);
        a3 = ld_plane(cf, o + 3 * cs, cxl);
        a4 = ld_plane(cf, o + 4 * cs, cyl);
        v3 = ld_plane(e0, o, cxl);
        v4 = ld_plane(e1, o, cyl);
      }
      q.a0 = a0; q.a1 = a1; q.a2 = a2; q.a3 = a3; q.a4 = a4; q.v3 = v3; q.v4 = v4;
      q.fl = ld_plane(g.flags, plane(kk + 1), c);
    }
  };

  const int64_t om = plane(k0 - 1);
  const uint32_t n00 = ld_plane(g.mat, om, rll), n10 = ld_plane(g.mat, om, ryl), n01 = ld_plane(g.mat, om, rxl),
                 n11 = ld_plane(g.mat, om, r);
  double tm = ld_plane(L.theta_in, om, r), t0 = ld_plane(L.theta_in, plane(k0), r);
  double a2m = 0.0, vm = 0.0;  // conductance and field of the low z edge
  if constexpr (JOULE) {
    const double h = k0 > 0 ? 1.0 : 0.0;
    a2m = h * double(ld_plane(cf, om + 5 * cs, r));
    vm = double(ld_plane(e2, om, r));
  }
  load(k0, true);  // (one round trip: the conductances do not wait for the flags)
  for (int m = tid; m < g.n_mat; m += BX * BY)
    S.kr[m] = make_double2(g.mtab[m * kMatStride + MC_K], g.mtab[m * kMatStride + MC_RHOCP]);
  if (wave == 0) {
    const int il = max(ic - 1, 0), ih = min(ic, nx - 1);
    S.dx[0][lane] = xl ? g.dx[il] : 0.0;
    S.dx[1][lane] = xh ? g.dx[ih] : 0.0;
    S.ix[0][lane] = xl ? g.idx[il] : 0.0;
    S.ix[1][lane] = xh ? g.idx[ih] : 0.0;
    S.ax[0][lane] = g.al[0][ic];
    S.ax[1][lane] = g.ah[0][ic];
    S.hx[lane] = g.hx[ic];
  }
  // a wave is a row: its y factors are scalars
  const int jl = max(jc - 1, 0), jh = min(jc, ny - 1);
  const double dy0 = yl ? uniform_entry(g.dy, jl) : 0.0, dy1 = yh ? uniform_entry(g.dy, jh) : 0.0;
  const double iy0 = yl ? uniform_entry(g.idy, jl) : 0.0, iy1 = yh ? uniform_entry(g.idy, jh) : 0.0;
  const double hy = uniform_entry(g.hy, jc);
  __syncthreads();
  // shares of one layer of cells: X, Y per side (without 1 / width), Z, C_n V_n
  struct Layer {
    double x0, x1, y0, y1, z, c;
  };
  auto layer = [&](int kk, uint32_t m00, uint32_t m10, uint32_t m01, uint32_t m11) -> Layer {
    const bool ok = kk >= 0 && kk < nz;
    const int kx = min(max(kk, 0), nz - 1);
    const double dzk = uniform_entry(g.dz, kx), izk = uniform_entry(g.idz, kx);
    const double dz = ok ? dzk : 0.0, iz = ok ? izk : 0.0;
    const double2 a = S.kr[m00], c = S.kr[m10], d = S.kr[m01], f = S.kr[m11];
    const double dx0 = S.dx[0][lane], dx1 = S.dx[1][lane];
    const double y0 = fma(c.x, dx1, a.x * dx0), y1 = fma(f.x, dx1, d.x * dx0), w = 0.25 * dz;
    Layer l;
    l.x0 = fma(d.x, dy1, a.x * dy0) * w;
    l.x1 = fma(f.x, dy1, c.x * dy0) * w;
    l.y0 = y0 * w;
    l.y1 = y1 * w;
    l.z = fma(y1, dy1, y0 * dy0) * (0.25 * iz);
    l.c = fma(fma(f.y, dx1, d.y * dx0), dy1, fma(c.y, dx1, a.y * dx0) * dy0) * (0.125 * dz);
    return l;
  };
  Layer lo = layer(k0 - 1, n00, n10, n01, n11);
  double e_part = 0.0, m_part = -1.0e300;
  for (int k = k0; k < k1; ++k) {
    const int64_t o = plane(k);
    const double ps0 = q.ps;
    double ps = ps0;
    if constexpr (JOULE) {
      // the pending Joule power of the current field (as joule_from_coef); in a
      // wave without a conductor every conductance is 0, and so is the power
      // unless the field has overflowed, which has to show
      const double h = sizeof(T) == 4 ? 0.5 : 1.0;
      const double ax[2] = {S.ax[0][lane], S.ax[1][lane]},
                   ay[2] = {uniform_entry(g.al[1], jc), uniform_entry(g.ah[1], jc)},
                   az[2] = {uniform_entry(g.al[2], k), uniform_entry(g.ah[2], k)};
      const double a6[6] = {h * double(q.a0), h * double(q.a1), h * double(q.a2), xl ? h * double(q.a3) : 0.0,
                            yl ? h * double(q.a4) : 0.0, h * a2m};
      const double v[6] = {double(q.e0), double(q.e1), double(q.e2), xl ? double(q.v3) : 0.0,
                           yl ? double(q.v4) : 0.0, k > 0 ? vm : 0.0};
      const double P = node_joule(a6, ax, ay, az, v, L.jf);
      if (P != 0.0) ps += P;
      a2m = double(q.a2);
      vm = double(q.e2);
    }
    const Layer up = layer(k, q.m00, q.m10, q.m01, q.m11);
    const double gx0 = (lo.x0 + up.x0) * S.ix[0][lane], gx1 = (lo.x1 + up.x1) * S.ix[1][lane],
                 gy0 = (lo.y0 + up.y0) * iy0, gy1 = (lo.y1 + up.y1) * iy1;
    double flux = gx0 * (t0 - q.xl);
    flux = fma(gx1, t0 - q.xh, flux);
    flux = fma(gy0, t0 - q.yl, flux);
    flux = fma(gy1, t0 - q.yh, flux);
    flux = fma(lo.z, t0 - tm, flux);
    flux = fma(up.z, t0 - q.th, flux);
    tm = t0;
    const double tc = t0;
    t0 = q.th;
    double src = L.dt * ps * (S.hx[lane] * hy * uniform_entry(g.hz, k));
    uint32_t sp = ps0 != 0.0 ? so : 0xffffffffu;  // a source of 0 stays as it is
    // formed here: sunk below the loads, these would keep the old inputs alive
    // beside the new ones, which then cost registers and a copy that waits
    asm volatile("" : "+v"(src), "+v"(flux), "+v"(t0), "+v"(tm), "+v"(a2m), "+v"(vm), "+v"(sp));
    load(min(k + 1, k1 - 1), false);
    const double tn = tc + (src - double(L.R) * L.dt * flux) / (lo.c + up.c);
    st_plane(L.theta_out, o, sz, so, tn);
    st_plane(L.psum, o, sz, sp, 0.0);
    if (L.theta32) st_plane(L.theta32, o, sz, so, float(tn));
    // the max reduction (fmax) drops NaN: a non-finite temperature is carried
    // in the energy sum, which the finalize kernel checks
    e_part += src + (tn - tn);
    m_part = fmax(m_part, tn);
    lo = up;
  }
  const double s[1] = {in ? e_part : 0.0}, m[1] = {in ? m_part : -1.0e300};
  block_reduce_store<1, 1>(s, m, L.partials + int64_t(blockIdx.x) * kRedWidth);
}

// Add the pending Joule power of the current field to psum.
template <typename T>
__global__ __launch_bounds__(256) void joule_flush_kernel(DevGrid g, const T *e0, const T *e1, const T *e2,
                                                          const T *cf, double *psum, double jf) {
  const int i = blockIdx.x * BX + threadIdx.x, j = blockIdx.y * BY + threadIdx.y, k = blockIdx.z;
  if (i > g.nx || j > g.ny) return;
  const int64_t n = int64_t(k) * g.sz + int64_t(j) * g.sy + i;
  const T *e[3] = {e0, e1, e2};
  const double P = pending_joule<T>(g, e, cf, i, j, k, n, jf);
  if (P != 0.0) psum[n] += P;
}

// Sum partials [nb][kRedWidth] in a fixed order (one block of 256).
__device__ void reduce_partials(const double *part, int64_t nb, int n_sum, int n_max, double *out) {
  __shared__ double red[4][kRedWidth];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double v[kRedWidth];
  for (int q = 0; q < kRedWidth; ++q) v[q] = q < n_sum ? 0.0 : -1.0e300;
  for (int64_t b = tid; b < nb; b += blockDim.x)
    for (int q = 0; q < n_sum + n_max; ++q) v[q] = q < n_sum ? v[q] + part[b * kRedWidth + q] : fmax(v[q], part[b * kRedWidth + q]);
  for (int q = 0; q < n_sum + n_max; ++q) v[q] = q < n_sum ? wave_sum(v[q]) : wave_max(v[q]);
  if (lane == 0)
    for (int q = 0; q < n_sum + n_max; ++q) red[wv][q] = v[q];
  __syncthreads();
  if (tid == 0)
    for (int q = 0; q < n_sum + n_max; ++q) {
      double acc = red[0][q];
      for (int w = 1; w < (int)(blockDim.x / 64); ++w) acc = q < n_sum ? acc + red[w][q] : fmax(acc, red[w][q]);
      out[q] = acc;
    }
}

// First stage of a two-stage reduction: block b folds rows [b per, (b+1) per)
// of the partials, in a fixed order, into row b of out.
__global__ __launch_bounds__(256) void reduce_rows_kernel(const double *part, int64_t nb, int64_t per, int n_sum,
                                                          int n_max, double *out) {
  __shared__ double o[kRedWidth];
  const int64_t b0 = int64_t(blockIdx.x) * per, b1 = b0 + per < nb ? b0 + per : nb;
  reduce_partials(part + b0 * kRedWidth, b1 > b0 ? b1 - b0 : 0, n_sum, n_max, o);
  if (threadIdx.x == 0)
    for (int q = 0; q < n_sum + n_max; ++q) out[int64_t(blockIdx.x) * kRedWidth + q] = o[q];
}

__global__ __launch_bounds__(256) void thermal_finalize(const double *part, int64_t nb, DevScalars *sc) {
  __shared__ double out[kRedWidth];
  reduce_partials(part, nb, 1, 1, out);
  if (threadIdx.x == 0) {
    sc->ejoule += out[0];
    sc->theta_max = out[1];
    if (!isfinite(out[0]) || !isfinite(out[1])) { if (sc->status == 0) sc->status = ETM_E_UNSTABLE; }
  }
}

// ---- diagnostics -------------------------------------------------------------
// W = eps0/(2 dt^2) sum_e L A [ er delta^2 + (c0 dt)^2 e^{n+1} (C e^n) ]
// One thread per node.  Its eight cells' ids are read once and their constants
// from LDS: 31 us on 132x78x46 nodes in FP64 (40 with a read of id and
// constants per edge and cell).
template <typename T>
__global__ __launch_bounds__(256) void diag_kernel(DiagLaunch L) {
  const DevGrid &g = L.g;
  const int i = blockIdx.x * BX + threadIdx.x, j = blockIdx.y * BY + threadIdx.y, k = blockIdx.z;
  __shared__ LdsMat MT;
  double w_part = 0.0, j_part = 0.0, m_part = -1.0e300;
  const bool in = i <= g.nx && j <= g.ny;
  const int64_t n = in ? int64_t(k) * g.sz + int64_t(j) * g.sy + i : 0;
  LCell CL;
  CL.M = &MT;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int ox = q & 1, oy = (q >> 1) & 1, oz = q >> 2;
    const int ci = i - 1 + ox, cj = j - 1 + oy, ck = k - 1 + oz;
    const bool ok = in && ci >= 0 && ci < g.nx && cj >= 0 && cj < g.ny && ck >= 0 && ck < g.nz;
    const int m = int(g.mat[ok ? n + (ox - 1) + (oy - 1) * g.sy + (oz - 1) * g.sz : n]);
    CL.id[q] = ok ? m : 0;
  }
  lds_mat_load(g, MT);
  if (in) {
    const T *en[3] = {(const T *)L.e_new[0], (const T *)L.e_new[1], (const T *)L.e_new[2]};
    const T *eo[3] = {(const T *)L.e_old[0], (const T *)L.e_old[1], (const T *)L.e_old[2]};
    const double ax[2] = {g.al[0][i], g.ah[0][i]}, ay[2] = {g.al[1][j], g.ah[1][j]}, az[2] = {g.al[2][k], g.ah[2][k]};
    const LTcr TC{&MT};
    auto zero_th = [](int, int, int) { return 0.0; };
    double er3[3];
    (void)edge_coef<0>(1, ax, ay, az, CL, TC, zero_th, &er3[0]);
    (void)edge_coef<1>(1, ax, ay, az, CL, TC, zero_th, &er3[1]);
    (void)edge_coef<2>(1, ax, ay, az, CL, TC, zero_th, &er3[2]);
    double acc = 0.0;
    for (int D = 0; D < 3; ++D) {
      if ((D == 0 && i == g.nx) || (D == 1 && j == g.ny) || (D == 2 && k == g.nz)) continue;
      if (pec_edge(g, D, i, j, k)) continue;
      GAcc<T> E{{eo[0], eo[1], eo[2]}, n, g.sy, g.sz};
      const double cc = D == 0 ? double(curl_x<T>(g, E, i, j, k))
                               : D == 1 ? double(curl_y<T>(g, E, i, j, k)) : double(curl_z<T>(g, E, i, j, k));
      const double Lh = D == 0 ? g.dx[i] : D == 1 ? g.dy[j] : g.dz[k];
      const double A = D == 0 ? g.hy[j] * g.hz[k] : D == 1 ? g.hx[i] * g.hz[k] : g.hx[i] * g.hy[j];
      const double e1 = double(en[D][n]);
      const double dl = e1 - double(eo[D][n]);
      acc += Lh * A * (er3[D] * dl * dl + L.c2dt2 * e1 * cc);
    }
    w_part = acc;
    j_part = L.psum[n] * (g.hx[i] * g.hy[j] * g.hz[k]);
    m_part = L.theta[n];
  }
  const double s[2] = {w_part, j_part}, m[1] = {m_part};
  const int64_t b = (int64_t(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
  block_reduce_store<2, 1>(s, m, L.partials + b * kRedWidth);
}

template <typename T>
__global__ __launch_bounds__(256) void diag_finalize(DiagLaunch L, int64_t nb) {
  __shared__ double out[kRedWidth];
  reduce_partials(L.partials, nb, 2, 1, out);
  if (threadIdx.x == 0) {
    const double W = out[0] * kEps0 / (2.0 * L.dt * L.dt);
    if (!isfinite(W)) { if (L.sc->status == 0) L.sc->status = ETM_E_UNSTABLE; }
    if (L.rec < L.cap) {
      double *row = L.hist_row;
      row[0] = double(L.step);
      row[1] = W;
      row[2] = L.sc->ejoule + L.dt * out[1];
      row[3] = out[2];
      for (int q = 0; q < L.n_probes; ++q) {
        const int f = int(L.probes[2 * q]);
        const int64_t idx = L.probes[2 * q + 1];
        row[4 + q] = f == 3 ? L.theta[idx] : double(((const T *)L.e_new[f])[idx]);
      }
      L.sc->n_records = L.rec + 1;
    }
  }
}

// ---- layout conversion and fills -------------------------------------------
__global__ void pack_kernel(const void *src, int src_f32, int64_t sy, int64_t sz, int ni, int nj, int nk, double *dst) {
  const int64_t total = int64_t(ni) * nj * nk;
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < total; t += int64_t(gridDim.x) * blockDim.x) {
    const int i = int(t % ni);
    const int64_t r = t / ni;
    const int j = int(r % nj), k = int(r / nj);
    const int64_t s = int64_t(k) * sz + int64_t(j) * sy + i;
    dst[t] = src_f32 ? double(((const float *)src)[s]) : ((const double *)src)[s];
  }
}

__global__ void unpack_kernel(const double *src, int ni, int nj, int nk, void *dst, int dst_f32, int64_t sy, int64_t sz) {
  const int64_t total = int64_t(ni) * nj * nk;
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < total; t += int64_t(gridDim.x) * blockDim.x) {
    const int i = int(t % ni);
    const int64_t r = t / ni;
    const int j = int(r % nj), k = int(r / nj);
    const int64_t s = int64_t(k) * sz + int64_t(j) * sy + i;
    if (dst_f32) ((float *)dst)[s] = float(src[t]); else ((double *)dst)[s] = src[t];
  }
}

__global__ void fill_kernel(uint32_t *dst, int64_t n_words) {
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n_words; t += int64_t(gridDim.x) * blockDim.x)
    dst[t] = 0u;
}

}  // namespace

void em_tiles(const DevGrid &g, int precision, int kchunk, int *ntx, int *nty, int *nkc) {
  if (precision == ETM_PREC_MIXED && em_runs(g)) {
    // BY runs of WX nodes of the x-fastest plane per block, one row of blocks
    const int64_t plane = int64_t(g.nx + 1) * (g.ny + 1), per = int64_t(WX) * BY;
    *ntx = int((plane + per - 1) / per);
    *nty = 1;
  } else if (precision == ETM_PREC_MIXED) {
    // MX x MY node tiles
    *ntx = (g.nx + 1 + MX - 1) / MX;
    *nty = (g.ny + 1 + MY - 1) / MY;
  } else {
    const int tx = em_flat(g) ? kFlatX : kTileX, ty = em_flat(g) ? kFlatY : kTileY;
    *ntx = (g.nx + 1 + tx - 1) / tx;
    *nty = (g.ny + 1 + ty - 1) / ty;
  }
  *nkc = (g.nz + 1 + kchunk - 1) / kchunk;
}

int64_t em_list_tiles(const DevGrid &g, int precision, int kchunk) {
  const int64_t nx1 = g.nx + 1, ny1 = g.ny + 1, nkc = (g.nz + 1 + kchunk - 1) / kchunk;
  if (precision == ETM_PREC_FP64) return (nx1 + 63) / 64 * ((ny1 + 3) / 4) * nkc;
  if (g.layout == kLayoutRuns || (g.layout == kLayoutAuto && nx1 < 1024)) return (nx1 * ny1 + 247) / 248 * nkc;
  return (nx1 + 61) / 62 * ((ny1 + 3) / 4) * nkc;
}

int em_kchunk(const DevGrid &g, int precision, bool alone) {
  // Planes per block: long chunks on many columns, short ones otherwise, and
  // shorter still (down to 4) while there would be fewer than 2048 blocks to
  // spread over the 256 CUs.  Blocks are those of em_list_tiles here (up to
  // twice or half the launch's own), whose limit the chunk also decides.
  // us per step at 4, 6, 11 and 17 planes: mixed
  // 256x256x64 96.8, 94.3, 93.1, 97.7, 384x384x96 299, 296, 303, 313,
  // 1024x1024x128 2592, 2569, 2557, 2604; FP64 256x256x64 98.7, 96.1, 94.5, 97.4,
  // 384x384x96 332, 336, 345, 356.
  int64_t cols = em_list_tiles(g, precision, g.nz + 1);
  auto blocks = [&](int kc) { return cols * ((g.nz + 1 + kc - 1) / kc); };
  int kc = blocks(12) >= 8192 ? 12 : 6;
  while (kc > 4 && blocks(kc) < 2048) kc = std::max(4, kc - 2);
  // A launch of one mesh that fits on the GPU at once (1024 blocks
  // at 4 waves per SIMD) lasts as long as one block: a chunk's planes are a
  // serial chain of 1.5 to 2 us each, so the shortest chunk that still fits is
  // taken.  It is taken too where other plans march at the same time on streams
  // of their own: us per step and plan at chunks of 4 | the shortest, mixed, two
  // plans of 32x32x16 5.1 | 4.6, 61x61x38 6.1 | 5.5, 110x100x40 8.8 | 8.8, four
  // plans 5.3 | 4.4, 6.0 | 5.9, 9.2 | 9.3.  One plan, us per step in FP64 | mixed
  // at chunks of 1, 2, 3, 4:
  //   32x32x16    5.7  7.3  8.4  9.5 |  5.4  7.3  8.8 10.1
  //   61x61x38    9.1  9.0 10.4 12.2 |  8.6  9.2 10.4 12.7
  //   80x77x48   13.1 12.8 13.7 16.5 | 11.1 11.2 13.4 15.8
  //   110x100x40 16.5 15.3 16.6 18.1 | 14.4 13.3 13.6 15.6
  //   152x120x43 25.2 21.9 22.1 21.6 | 22.0 19.2 19.2 19.9
  // (one generation from chunks 1, 1, 2, 3, 4 | 1, 1, 2, 2, 4 on).  Larger meshes
  // keep the rule above: 192x192x48 takes 42.7 | 34.9 at 4, 44.8 | 36.7 at 2.
  int ntx, nty, nkc;
  em_tiles(g, precision, 1, &ntx, &nty, &nkc);
  cols = int64_t(ntx) * nty;
  if (alone && blocks(4) <= 1024)
    for (kc = 1; blocks(kc) > 1024;) ++kc;
  return kc;
}

hipError_t launch_em_step(const EmLaunch &L, hipStream_t s) {
  int ntx, nty, nkc;
  const int kc = L.kchunk > 0 ? L.kchunk : em_kchunk(L.g, L.precision, true);
  em_tiles(L.g, L.precision, kc, &ntx, &nty, &nkc);
  const int nb = ntx * nty * nkc;
  const dim3 block(BX, BY, 1);
  if (L.precision == ETM_PREC_FP64) {
    EmPtrs<double> p{(const double *)L.e0[0], (const double *)L.e1[0], (double *)L.out0[0], nullptr};
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(nb), block, 0, s, L, p, ntx, nty, nkc, kc, L.acc_joule);
    };
    if (em_streams(L.g.ntot, true))
      launch(em_flat(L.g) ? em_march_kernel<double, kMarchFp64Flat, true> : em_march_kernel<double, kMarchFp64, true>);
    else
      launch(em_flat(L.g) ? em_march_kernel<double, kMarchFp64Flat, false> : em_march_kernel<double, kMarchFp64, false>);
  } else {
    EmPtrs<float> p{(const float *)L.e0[0], (const float *)L.e1[0], (float *)L.out0[0], (float *)L.out1[0]};
    if (em_runs(L.g))
      hipLaunchKernelGGL((em_march_kernel<float, kMarchRuns, false>), dim3(nb), block, 0, s, L, p, ntx, nty, nkc, kc,
                         L.acc_joule);
    else
      hipLaunchKernelGGL((em_march_kernel<float, kMarchTiles, true>), dim3(nb), block, 0, s, L, p, ntx, nty, nkc, kc,
                         L.acc_joule);
  }
  return hipGetLastError();
}

// Steps n and n + 1 (La: pointers and Joule flag of step n; Lb: pointers of
// step n + 1) as a wavefront over n_slabs z-slabs of whole chunks.  Launch t
// runs step n on slab t + 1 (slabs 0 and 1 in launch 0) and step n + 1 on
// slab t - 1 (slabs S - 2 and S - 1 in the last launch), so step n + 1 on a
// slab follows step n on that slab and its two neighbours, and no step-n
// tile still to run reads a plane step n + 1 overwrites (slab s + 2 reads
// down to the last plane of slab s + 1 only).  S launches for the two steps.
hipError_t launch_em_pair_schedule(const EmLaunch &La, const EmLaunch &Lb, int n_slabs, hipStream_t s) {
  int ntx, nty, nkc;
  const int kc = La.kchunk > 0 ? La.kchunk : em_kchunk(La.g, La.precision, false);
  em_tiles(La.g, La.precision, kc, &ntx, &nty, &nkc);
  const int S = std::max(2, std::min(n_slabs, nkc));
  auto first = [&](int q) { return int(int64_t(q) * nkc / S); };  // first chunk of slab q
  const dim3 block(BX, BY, 1);
  for (int t = 0; t < S; ++t) {
    // step-n slabs [a0, a1), step-(n + 1) slabs [b0, b1) of this launch
    int a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    if (t == 0) {
      a1 = 2;
    } else if (t == S - 1) {
      b0 = S - 2;
      b1 = S;
    } else {
      a0 = t + 1; a1 = t + 2;
      b0 = t - 1; b1 = t;
    }
    const int kcA = a0 < a1 ? first(a0) : 0, nkcA = a0 < a1 ? first(a1) - first(a0) : 0;
    const int kcB = b0 < b1 ? first(b0) : 0, nkcB = b0 < b1 ? first(b1) - first(b0) : 0;
    const int nb = ntx * nty * (nkcA + nkcB);
    if (nb == 0) continue;
    if (La.precision == ETM_PREC_FP64) {
      EmPtrs<double> pa{(const double *)La.e0[0], (const double *)La.e1[0], (double *)La.out0[0], nullptr};
      EmPtrs<double> pb{(const double *)Lb.e0[0], (const double *)Lb.e1[0], (double *)Lb.out0[0], nullptr};
      const auto kernel =
          em_flat(La.g) ? em_march_pair_kernel<double, kMarchFp64Flat> : em_march_pair_kernel<double, kMarchFp64>;
      hipLaunchKernelGGL(kernel, dim3(nb), block, 0, s, La, pa, pb, ntx, nty, kcA, nkcA, kcB, nkcB, kc, La.acc_joule);
    } else {
      EmPtrs<float> pa{(const float *)La.e0[0], (const float *)La.e1[0], (float *)La.out0[0], (float *)La.out1[0]};
      EmPtrs<float> pb{(const float *)Lb.e0[0], (const float *)Lb.e1[0], (float *)Lb.out0[0], (float *)Lb.out1[0]};
      hipLaunchKernelGGL((em_march_pair_kernel<float, kMarchMixed>), dim3(nb), block, 0, s, La, pa, pb, ntx, nty, kcA, nkcA,
                         kcB, nkcB, kc, La.acc_joule);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool em_tile_is_flat(const DevGrid &g) { return em_flat(g); }

hipError_t launch_em_batched(const BatchVar *vars, const int4 *items, int n_items, int64_t s, int precision,
                             int64_t nodes, bool any_flat, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  const bool nt = em_streams(nodes, precision == ETM_PREC_FP64);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(n_items), dim3(BX, BY), 0, st, vars, items, n_items, s);
  };
  if (precision != ETM_PREC_FP64)
    launch(nt ? em_march_batched<float, kMarchMixed, true> : em_march_batched<float, kMarchMixed, false>);
  else if (any_flat)  // (the kernel of both tiles is 1 to 3 % slower on batches of ordinary meshes)
    launch(nt ? em_march_batched<double, kMarchFp64Any, true> : em_march_batched<double, kMarchFp64Any, false>);
  else
    launch(nt ? em_march_batched<double, kMarchFp64, true> : em_march_batched<double, kMarchFp64, false>);
  return hipGetLastError();
}

hipError_t launch_wave_sample(const double *aw, int n, double dt, int64_t base, double *Ja, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t total = int64_t(n) * (kWaveBlock + 1);
  hipLaunchKernelGGL(wave_sample_kernel, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, aw, n, dt, base, Ja);
  return hipGetLastError();
}

// Columns of 64 x 4 nodes and planes per block of the thermal and coefficient
// kernels: the longest chunk, up to `most` planes, that leaves `least` blocks.
// A chunk reads a plane beyond its own and waits for its first loads alone, so
// the thermal kernel takes few long ones (least 700); the coefficient kernel
// only skips through most planes, and the many round trips of the others run
// side by side (least 4800).  us per step at one thermal block per EM step,
// mixed, by planes per block:
//   thermal  131x77x45  1: 49.4  2: 42.7  4: 39.1  8: 41.8   256x256x64  2: 222  4: 205  8: 199  12: 193
//   coef     131x77x45  1: 48.2  2: 48.5  4: 53.1  8: 61.8   256x256x64  1: 206  2: 196  4: 195  8: 199
static int column_chunk(const DevGrid &g, int most, int64_t least, int *ntx, int *nty) {
  *ntx = (g.nx + BX) / BX;
  *nty = (g.ny + BY) / BY;
  for (int kc : {12, 8, 6, 4, 3, 2})
    if (kc <= most && int64_t(*ntx) * *nty * ((g.nz + 1 + kc - 1) / kc) >= least) return kc;
  return 1;
}

hipError_t launch_thermal(const ThermalLaunch &L, hipStream_t s) {
  int ntx, nty;
  const int kc = column_chunk(L.g, 12, 700, &ntx, &nty);
  const dim3 grid(unsigned(ntx) * unsigned(nty) * unsigned((L.g.nz + 1 + kc - 1) / kc)), block(BX, BY, 1);
  auto launch = [&](auto kernel, auto zero) {
    using T = decltype(zero);
    hipLaunchKernelGGL(kernel, grid, block, 0, s, L, (const T *)L.e[0], (const T *)L.e[1], (const T *)L.e[2],
                       (const T *)L.coef, ntx, nty, kc);
  };
  if (L.precision == ETM_PREC_FP64)
    launch(L.acc_joule ? thermal_kernel<double, true> : thermal_kernel<double, false>, 0.0);
  else
    launch(L.acc_joule ? thermal_kernel<float, true> : thermal_kernel<float, false>, 0.0f);
  const int64_t nb = int64_t(grid.x) * grid.y * grid.z;
  if (nb > 4 * kFinalizeRows) {
    // two stages: rows [nb, nb + kFinalizeRows) of the partials hold the first
    const int64_t per = (nb + kFinalizeRows - 1) / kFinalizeRows, nb2 = (nb + per - 1) / per;
    hipLaunchKernelGGL(reduce_rows_kernel, dim3(unsigned(nb2)), dim3(256), 0, s, (const double *)L.partials, nb, per,
                       1, 1, L.partials + nb * kRedWidth);
    hipLaunchKernelGGL(thermal_finalize, dim3(1), dim3(256), 0, s, (const double *)(L.partials + nb * kRedWidth),
                       nb2, L.sc);
  } else {
    hipLaunchKernelGGL(thermal_finalize, dim3(1), dim3(256), 0, s, (const double *)L.partials, nb, L.sc);
  }
  return hipGetLastError();
}

hipError_t launch_joule_flush(const DevGrid &g, int precision, const void *const *e, const void *coef, double *psum,
                              double jf, hipStream_t s) {
  const dim3 grid = node_grid(g), block(BX, BY, 1);
  if (precision == ETM_PREC_FP64)
    hipLaunchKernelGGL((joule_flush_kernel<double>), grid, block, 0, s, g, (const double *)e[0], (const double *)e[1],
                       (const double *)e[2], (const double *)coef, psum, jf);
  else
    hipLaunchKernelGGL((joule_flush_kernel<float>), grid, block, 0, s, g, (const float *)e[0], (const float *)e[1],
                       (const float *)e[2], (const float *)coef, psum, jf);
  return hipGetLastError();
}

hipError_t launch_coef(const DevGrid &g, const DevPorts &P, int precision, const void *theta, void *coef, CoefK ck,
                       hipStream_t s) {
  int ntx, nty;
  const int kc = column_chunk(g, 8, 4800, &ntx, &nty);
  const dim3 grid(unsigned(ntx) * unsigned(nty) * unsigned((g.nz + 1 + kc - 1) / kc)), block(BX, BY, 1);
  auto launch = [&](auto kernel, auto zero, CoefK c) {
    using T = decltype(zero);
    hipLaunchKernelGGL(kernel, grid, block, 0, s, g, P, (const T *)theta, (T *)coef, c, ntx, nty, kc);
  };
  const CoefK ck64{nullptr, nullptr, nullptr, ck.tcr_only};
  if (precision == ETM_PREC_FP64)
    launch(ck.tcr_only ? coef_kernel<double, false> : coef_kernel<double, true>, 0.0, ck64);
  else
    launch(ck.tcr_only ? coef_kernel<float, false> : coef_kernel<float, true>, 0.0f, ck);
  return hipGetLastError();
}

hipError_t launch_diag(const DiagLaunch &L, hipStream_t s) {
  const dim3 grid = node_grid(L.g), block(BX, BY, 1);
  const int64_t nb = int64_t(grid.x) * grid.y * grid.z;
  if (L.precision == ETM_PREC_FP64) {
    hipLaunchKernelGGL((diag_kernel<double>), grid, block, 0, s, L);
    hipLaunchKernelGGL((diag_finalize<double>), dim3(1), dim3(256), 0, s, L, nb);
  } else {
    hipLaunchKernelGGL((diag_kernel<float>), grid, block, 0, s, L);
    hipLaunchKernelGGL((diag_finalize<float>), dim3(1), dim3(256), 0, s, L, nb);
  }
  return hipGetLastError();
}

hipError_t launch_pack(const void *src, int src_f32, int64_t sy, int64_t sz, int ni, int nj, int nk, double *dst,
                       hipStream_t s) {
  const int64_t total = int64_t(ni) * nj * nk;
  if (total <= 0) return hipSuccess;
  const int blocks = int(std::min<int64_t>((total + 255) / 256, 65536));
  hipLaunchKernelGGL(pack_kernel, dim3(blocks), dim3(256), 0, s, src, src_f32, sy, sz, ni, nj, nk, dst);
  return hipGetLastError();
}

hipError_t launch_unpack(const double *src, int ni, int nj, int nk, void *dst, int dst_f32, int64_t sy, int64_t sz,
                         hipStream_t s) {
  const int64_t total = int64_t(ni) * nj * nk;
  if (total <= 0) return hipSuccess;
  const int blocks = int(std::min<int64_t>((total + 255) / 256, 65536));
  hipLaunchKernelGGL(unpack_kernel, dim3(blocks), dim3(256), 0, s, src, ni, nj, nk, dst, dst_f32, sy, sz);
  return hipGetLastError();
}

hipError_t launch_fill(void *dst, int64_t n_bytes, hipStream_t s) {
  const int64_t words = n_bytes / 4;
  if (words <= 0) return hipSuccess;
  const int blocks = int(std::min<int64_t>((words + 255) / 256, 65536));
  hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, s, (uint32_t *)dst, words);
  return hipGetLastError();
}

}  // namespace etm
