// Cell-centred multigrid solver and elliptic divergence cleaning for MI355X
// (gfx950): level hierarchy, kernels and the C ABI of include/gmunu_mg.h.
//
// Cheong et al., "Gmunu" (arXiv 2012.07322), section 2.7 and section 2.2.
// On fine levels an operation of a cycle is one launch over the level's cells:
// the smoother (red-black, i + j + k even first: in place one colour per
// launch, on large levels sweep pairs out of place), the residual and its
// restriction (volume-weighted mean of the children), the FAS coarse
// right-hand side and the Kwak prolongation of the coarse correction; the
// coarse levels run as one workgroup.  The geometry of the reference-metric
// Laplacian factorises into per-axis 1D tables per level (weights toward the
// lower and upper neighbour, the metric factors of the transverse terms, cell
// volumes), Cartesian weights are scalars, so a cell's operator is a handful
// of loads and FMAs.  The residual norm is a grid-stride maximum with
// wavefront shuffles, one partial per workgroup and one finishing workgroup:
// no atomics, no memset.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/gmunu.h"
#include "../../include/gmunu_mg.h"
#include "gmunu_dev.hpp"
#include "gmunu_host.hpp"
#include "gmunu_tile.hpp"

using namespace gm;

namespace {

constexpr int kMaxLevels = 16;
constexpr int kNormParts = 16384;
// after the norm's result: the state of a chunk of dynamical-metric steps
// (gmunu_mg_dynamical_steps: trigger step, time at that step)
constexpr int kGateSlots = 2;

// One level as the kernels see it.
struct MgGeo {
  int ndim, coord;
  int n[3], g[3];
  long s1, s2, nt;  // strides of axes 1 and 2, entries
  double ih2_2;     // 1 / h^2 along axis 2
  double h[3];
  // per axis-0 index (ghosts included)
  const double *a0m, *a0p, *g1, *g2, *vol0, *sg0;
  // per axis-1 index
  const double *a1m, *a1p, *s2t, *vol1, *sg1;
  int bc[3][2];
  double rob_lo, rob_hi;  // Robin ghost factors on axis 0 (centre inside / centre of the ghost)
  double x0[3];           // lower face coordinate per axis (Cartesian Robin factors)
  unsigned vodd[3][2];    // vector equations: components odd across each mirror face (bit q)
  int power, power2;
  double offset;
  int line;  // smoother: alternating zebra line relaxation (else red-black points)
  // vector operator (Cartesian): 1/h_a^2, 1/(4 h_a h_b) for the axis pairs
  // (0,1), (0,2), (1,2), and the inverse diagonal of each component's row
  double vih2[3], vmix[3], vidg[3];
};

// Running maximum of |v|; a NaN counts as infinite, so that a solution gone
// NaN never reads as converged.
__device__ __forceinline__ double mg_absmax(double m, double v) { return v != v ? INFINITY : fmax(m, fabs(v)); }

__device__ __forceinline__ long mg_off(const MgGeo &G, int i, int j, int k) {
  return (long)(k + G.g[2]) * G.s2 + (long)(j + G.g[1]) * G.s1 + (i + G.g[0]);
}

// 1 / x; IEEE: with a division's results where the refinement gives NaN (0 and
// infinity).
template <bool IEEE>
__device__ __forceinline__ double mg_rcp(double x) {
  return IEEE ? __builtin_amdgcn_div_fixup(rcp(x), x, 1.0) : rcp(x);
}

// sqrt(ri / rg): the ratio of two distances from the origin from their squares,
// as one refined root of their product; 0 and infinity where the one or the
// other is the origin.
__device__ __forceinline__ double mg_dist_ratio(double ri, double rg) {
  return __builtin_amdgcn_div_fixup(ri * rsq(ri * rg), rg, ri);
}

// w^q, q >= 0.
__device__ __forceinline__ double mg_ipow(double w, int q) {
  double r = 1.0;
#pragma unroll 1
  for (; q > 0; q--) r *= w;
  return r;
}

// a (u + c)^p + a2 (u + c)^q and its derivative in u.  IEEE: at a zero of a
// negative power the infinities of a division, for the operator itself (a
// sweep or a norm ends in NaN or infinity there either way, and the fix-ups
// would take 8% of the general sweep pairs: 472 us at 256^3 with Robin faces,
// 434 without).
template <bool IEEE = false>
__device__ __forceinline__ double mg_nl_both(int power, int power2, double offset, double a, double a2, double u,
                                             double &du) {
  const double w = u + offset;
  double nl = a, rw = 0.0;
  du = 0.0;
  if (power == 1) {
    nl = a * w;
    du = a;
  } else if (power == -1) {
    rw = mg_rcp<IEEE>(w);
    nl = a * rw;
    du = -nl * rw;
  }
  if (a2 != 0.0) {
    if (power2 <= 0 && power != -1) rw = mg_rcp<IEEE>(w);
    if (power2 == -7) {
      const double r2 = rw * rw, t = a2 * (r2 * r2) * (r2 * rw);
      nl += t;
      du += power2 * t * rw;
    } else {
      // (a positive power without a reciprocal: u + c may be 0)
      const bool pos = power2 > 0;
      const double b = pos ? w : rw, v = a2 * mg_ipow(b, (pos ? power2 : -power2) - 1);
      nl += v * b;
      du += power2 * (pos ? v : v * b * b);
    }
  }
  return nl;
}

// Robin ghost factor r_in / r_ghost for the ghost of boundary cell c across
// face (a, up): on spherical grids (axis 0) the level's constants; on
// Cartesian and cylindrical grids r is the distance of the cell centres
// from the origin (x, y, z; or R, z) -- the conditions u + x.grad u = 0 and
// u + R du/dR + z du/dz = 0 of section 2.6 as a 1/r fall-off between the
// cell and its ghost.
__device__ __forceinline__ double mg_rob(const MgGeo &G, int i, int j, int k, int a, bool up) {
  if (G.coord == GMUNU_SPH) return up ? G.rob_hi : G.rob_lo;
  const int c[3] = {i, j, k};
  const int nb = G.coord == GMUNU_CYL ? 2 : 3;
  double ri = 0.0, rg = 0.0;
#pragma unroll
  for (int b = 0; b < 3; b++) {
    if (b >= G.ndim || b >= nb) continue;
    const double xi = G.x0[b] + (c[b] + 0.5) * G.h[b];
    const double xg = b == a ? G.x0[b] + (c[b] + (up ? 1 : -1) + 0.5) * G.h[b] : xi;
    ri += xi * xi;
    rg += xg * xg;
  }
  return mg_dist_ratio(ri, rg);
}

// Neighbour of interior cell (i, j, k) along axis a (stride S) on the side
// `up`: the stored value inside, else the boundary rule applied to the cell
// itself (the value a ghost fill would store there).
__device__ __forceinline__ double mg_nb(const MgGeo &G, const double *__restrict__ u, long o, int i, int j, int k,
                                        int a, int S, bool up) {
  const int n = G.n[a], c = a == 0 ? i : a == 1 ? j : k, kind = G.bc[a][up ? 1 : 0];
  const bool face = up ? c == n - 1 : c == 0;
  const int in = up ? S : -S, out = kind == GMUNU_MG_PERIODIC ? (up ? -(n - 1) * S : (n - 1) * S) : 0;
  double v = u[o + (face ? out : in)];
  if (kind == GMUNU_MG_DIRICHLET) v = face ? -v : v;
  if (kind == GMUNU_MG_ROBIN && face) v *= mg_rob(G, i, j, k, a, up);
  return v;
}

// L(u) at interior cell (i,j,k) (linear offset o) and dL/du there.  GH:
// neighbours across the boundary from u's ghost entries as stored; else
// from the boundary rule (mg_nb), so that no ghost fill is needed.
template <bool GH>
__device__ __forceinline__ double mg_L(const MgGeo &G, const double *__restrict__ u, double av, double a2v, int i,
                                       int j, int k, long o, double *dg) {
  const int I = i + G.g[0], J = j + G.g[1], S1 = (int)G.s1, S2 = (int)G.s2;
  const bool ca = G.coord == GMUNU_CART;  // Cartesian weights are scalars
  const double uc = u[o];
  double wm = ca ? G.vih2[0] : G.a0m[I], wp = ca ? G.vih2[0] : G.a0p[I];
  double um = GH ? u[o - 1] : mg_nb(G, u, o, i, j, k, 0, 1, false);
  double up = GH ? u[o + 1] : mg_nb(G, u, o, i, j, k, 0, 1, true);
  double lap = wp * (up - uc) - wm * (uc - um);
  double d = -(wm + wp);
  if (G.ndim > 1) {
    wm = wp = G.vih2[1];
    if (!ca) {
      const double gi = G.g1[I];
      wm = gi * G.a1m[J];
      wp = gi * G.a1p[J];
    }
    um = GH ? u[o - S1] : mg_nb(G, u, o, i, j, k, 1, S1, false);
    up = GH ? u[o + S1] : mg_nb(G, u, o, i, j, k, 1, S1, true);
    lap += wp * (up - uc) - wm * (uc - um);
    d -= wm + wp;
  }
  if (G.ndim > 2) {
    const double w = ca ? G.vih2[2] : G.g2[I] * G.s2t[J] * G.ih2_2;
    um = GH ? u[o - S2] : mg_nb(G, u, o, i, j, k, 2, S2, false);
    up = GH ? u[o + S2] : mg_nb(G, u, o, i, j, k, 2, S2, true);
    lap += w * (up - uc) - w * (uc - um);
    d -= 2.0 * w;
  }
  double du;
  const double nl = mg_nl_both<GH>(G.power, G.power2, G.offset, av, a2v, uc, du);
  if (dg) *dg = d - du;
  return lap - nl;
}

// Interior cell number t (x fastest); 32-bit arithmetic (a level has fewer
// than 2^32 cells, which validation ensures).
__device__ __forceinline__ void mg_cell(const MgGeo &G, long t, int &i, int &j, int &k) {
  const unsigned u = (unsigned)t, n0 = (unsigned)G.n[0], n1 = (unsigned)G.n[1];
  const unsigned r = u / n0;
  i = (int)(u - r * n0);
  k = (int)(r / n1);
  j = (int)(r - (unsigned)k * n1);
}

__device__ __forceinline__ long mg_cells(const MgGeo &G) { return (long)G.n[0] * G.n[1] * G.n[2]; }

// Face-adjacent ghost number t: axis, side, transverse cell.
__device__ __forceinline__ void mg_ghost_one(const MgGeo &G, double *u, long t) {
  for (int a = 0; a < G.ndim; a++) {
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    const long per = 2L * G.n[b1] * G.n[b2];
    if (t >= per) {
      t -= per;
      continue;
    }
    const int side = (int)(t & 1);
    const long tr = t >> 1;
    int gc[3], sc[3];
    gc[b1] = sc[b1] = (int)(tr % G.n[b1]);
    gc[b2] = sc[b2] = (int)(tr / G.n[b1]);
    gc[a] = side == 0 ? -1 : G.n[a];
    const int kind = G.bc[a][side];
    double v;
    if (kind == GMUNU_MG_PERIODIC) {
      sc[a] = side == 0 ? G.n[a] - 1 : 0;
      v = u[mg_off(G, sc[0], sc[1], sc[2])];
    } else {
      sc[a] = side == 0 ? 0 : G.n[a] - 1;
      const double ui = u[mg_off(G, sc[0], sc[1], sc[2])];
      v = kind == GMUNU_MG_DIRICHLET ? -ui
          : kind == GMUNU_MG_NEUMANN ? ui
                                     : ui * mg_rob(G, sc[0], sc[1], sc[2], a, side == 1);
    }
    u[mg_off(G, gc[0], gc[1], gc[2])] = v;
    return;
  }
}

__device__ __forceinline__ long mg_ghost_count(const MgGeo &G) {
  long s = 0;
  for (int a = 0; a < G.ndim; a++) {
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    s += 2L * G.n[b1] * G.n[b2];
  }
  return s;
}

// Face ghost t of component q of a vector field: periodic wrap or mirror
// with the component's parity across that face.
__device__ __forceinline__ void mgv_ghost_one(const MgGeo &G, double *u, int q, long t) {
  for (int a = 0; a < G.ndim; a++) {
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    const long per = 2L * G.n[b1] * G.n[b2];
    if (t >= per) {
      t -= per;
      continue;
    }
    const int side = (int)(t & 1);
    const long tr = t >> 1;
    int gc[3], sc[3];
    gc[b1] = sc[b1] = (int)(tr % G.n[b1]);
    gc[b2] = sc[b2] = (int)(tr / G.n[b1]);
    gc[a] = side == 0 ? -1 : G.n[a];
    double v;
    if (G.bc[a][side] == GMUNU_MG_PERIODIC) {
      sc[a] = side == 0 ? G.n[a] - 1 : 0;
      v = u[mg_off(G, sc[0], sc[1], sc[2])];
    } else {
      sc[a] = side == 0 ? 0 : G.n[a] - 1;
      const double ui = u[mg_off(G, sc[0], sc[1], sc[2])];
      v = (G.vodd[a][side] >> q) & 1 ? -ui : ui;
    }
    u[mg_off(G, gc[0], gc[1], gc[2])] = v;
    return;
  }
}

template <int NC>
__global__ __launch_bounds__(NT) void k_mg_ghosts(const MgGeo G, double *u) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
#pragma unroll
  for (int q = 0; q < NC; q++) {
    if (NC == 1)
      mg_ghost_one(G, u, t);
    else
      mgv_ghost_one(G, u + q * G.nt, q, t);
  }
}

// One colour of red-black Newton-Gauss-Seidel in place: thread t -> the t-th
// cell of that colour (every other cell of a row).
__global__ __launch_bounds__(NT) void k_mg_smooth(const MgGeo G, double *u, const double *__restrict__ f,
                                                  const double *__restrict__ a, const double *__restrict__ a2,
                                                  int colour) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  const unsigned hrow = (unsigned)(G.n[0] + 1) >> 1, n1 = (unsigned)G.n[1];
  if (t >= (long)hrow * G.n[1] * G.n[2]) return;
  const unsigned row = (unsigned)t / hrow;
  const int k = (int)(row / n1), j = (int)(row - (unsigned)k * n1);
  const int i = (int)((unsigned)t - row * hrow) * 2 + ((j + k + colour) & 1);
  if (i >= G.n[0]) return;
  const long o = mg_off(G, i, j, k);
  double dg;
  const double Lu = mg_L<false>(G, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, i, j, k, o, &dg);
  u[o] -= (Lu - f[o]) * rcp(dg);
}

// ---- Line relaxation --------------------------------------------------------
// An alternative to the paper's point smoother for the anisotropic cells on
// which section 2.7 notes that point smoothers converge slowly (spherical
// polar grids).  One workgroup per line, a lane per cell (lines have at most
// kMaxLine cells).  The lane builds its row of the line's tridiagonal system
// (couplings toward the lower and upper neighbour along the line, right-hand
// side, all over the diagonal) in registers; parallel cyclic reduction then
// solves it: at stride s every row eliminates its couplings to the rows s
// below and s above, which it reads from LDS, so after ceil(log2 n)
// doublings each row holds one unknown.  Two copies of the three arrays
// alternate between doublings.
//
// Bound by latency (a line is a chain of loads and log2 n doublings on a few
// wavefronts): the diagonal kept at 1 takes one refined reciprocal per
// doubling where the four-array form took two divisions (scalar lines, 32 of
// 640 cells: 9.1 us, 13.1 before; 320 of 64: 6.3, 7.4 before).

constexpr int kLineWave = 64;
constexpr int kCoarseLineThreads = 1024;  // one-workgroup coarsest-level line solvers
constexpr int kMaxLine = 1024;

// Weights of the flux-form Laplacian from cell (I, J) (ghost-inclusive
// indices) toward its lower and upper neighbour along axis a: the terms
// of mg_L.
__device__ __forceinline__ void mg_w(const MgGeo &G, int I, int J, int a, double &wm, double &wp) {
  if (a == 0) {
    wm = G.a0m[I];
    wp = G.a0p[I];
  } else if (a == 1) {
    wm = G.g1[I] * G.a1m[J];
    wp = G.g1[I] * G.a1p[J];
  } else {
    wm = wp = G.g2[I] * G.s2t[J] * G.ih2_2;
  }
}

// Factor s of the boundary rule ghost = s u_cell across the non-periodic
// face (a, up) of boundary cell c.
__device__ __forceinline__ double mg_fold(const MgGeo &G, const int c[3], int a, bool up) {
  const int kind = G.bc[a][up ? 1 : 0];
  return kind == GMUNU_MG_DIRICHLET ? -1.0 : kind == GMUNU_MG_NEUMANN ? 1.0 : mg_rob(G, c[0], c[1], c[2], a, up);
}

// First cell of line t of colour `colour` along axis a: the transverse
// axes b1 < b2, each active one coloured by its index parity (bit 0: b1,
// bit 1: b2).  False past the last line.
__device__ __forceinline__ bool mg_line(const MgGeo &G, int a, int colour, long t, int c[3]) {
  const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
  const int p1 = colour & 1, p2 = (colour >> 1) & 1;
  const long h1 = b1 < G.ndim ? (G.n[b1] - p1 + 1) >> 1 : 1;
  const long h2 = b2 < G.ndim ? (G.n[b2] - p2 + 1) >> 1 : 1;
  if (t >= h1 * h2) return false;
  const int t1 = b1 < G.ndim ? 2 * (int)(t % h1) + p1 : 0;
  const int t2 = b2 < G.ndim ? 2 * (int)(t / h1) + p2 : 0;
  // (b1, b2) = (1, 2), (0, 2), (0, 1) for a = 0, 1, 2 (no dynamic indexing of c)
  c[0] = a == 0 ? 0 : t1;
  c[1] = a == 0 ? t1 : a == 1 ? 0 : t2;
  c[2] = a == 2 ? 0 : t2;
  return true;
}

// Order of LDS accesses between the lanes of one wavefront.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Orders the LDS accesses of the lanes of a line: those of one wavefront, or
// of the workgroup.
__device__ __forceinline__ void mg_line_sync(bool one_wave) {
  if (one_wave)
    wave_fence();
  else
    __syncthreads();
}

// This workgroup's place in the contiguous runs of a 1D grid, one run per XCD
// (workgroups are dispatched round-robin over the eight XCDs).  Lines along y
// and z whose cells share cache lines are then in flight beside each other on
// one L2: 162 us per colour of z-lines at 256^3, against 525 with neighbouring
// lines on different XCDs, each of which fetched every cache line.
__device__ __forceinline__ int mg_xcd_run() {
  const int nt = gridDim.x, b = blockIdx.x, x = b % 8, q = nt / 8, r = nt % 8;
  return x * q + (x < r ? x : r) + b / 8;
}

// Parallel cyclic reduction of NS systems of n rows at once, row m in this
// lane's registers (a x_{m-s} + x_m + c x_{m+s} = d, s = 1; rows of lanes with
// !on do not exist): on return d is the solution.  sm: 6 NS n doubles.
template <int NS>
__device__ __forceinline__ void mg_pcr(double *sm, int n, int m, bool on, bool one_wave, double *a, double *c,
                                       double *d) {
  for (int s = 1, p = 0; s < n; s <<= 1, p ^= 1) {
    double *R = sm + p * 3 * NS * n;
    if (on) {
#pragma unroll
      for (int q = 0; q < NS; q++) {
        R[3 * q * n + m] = a[q];
        R[(3 * q + 1) * n + m] = c[q];
        R[(3 * q + 2) * n + m] = d[q];
      }
    }
    mg_line_sync(one_wave);
    if (on) {
      // (a row without a neighbour s away has no coupling to it)
      const int lo = m >= s ? m - s : m, hi = m + s < n ? m + s : m;
#pragma unroll
      for (int q = 0; q < NS; q++) {
        const double *A = R + 3 * q * n, *C = A + n, *D = C + n;
        const double al = -a[q], ga = -c[q];
        const double ib = rcp(1.0 + al * C[lo] + ga * A[hi]);
        a[q] = al * A[lo] * ib;
        c[q] = ga * C[hi] * ib;
        d[q] = (d[q] + al * D[lo] + ga * D[hi]) * ib;
      }
    }
  }
}

// One Newton step of the line through cell c along axis ax, cell m of it in
// this lane (live: the line exists): the residual's derivative on the line
// from the operator's couplings and diagonal (boundary faces folded in),
// everything off the line at its current value.  sm: 6 n doubles of the line.
__device__ __forceinline__ void mg_line_step(const MgGeo &G, double *u, const double *__restrict__ f,
                                             const double *__restrict__ a, const double *__restrict__ a2, int ax,
                                             const int c[3], bool live, double *sm, int m, bool one_wave) {
  const int n = G.n[ax];
  const bool on = live && m < n;
  double wm = 0.0, wp = 0.0, d = 0.0;
  long o = 0;
  if (on) {
    const int cc[3] = {ax == 0 ? m : c[0], ax == 1 ? m : c[1], ax == 2 ? m : c[2]};
    o = mg_off(G, cc[0], cc[1], cc[2]);
    double dg;
    const double Lu = mg_L<false>(G, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, cc[0], cc[1], cc[2], o, &dg);
#pragma unroll
    for (int b = 0; b < 3; b++) {
      if (b >= G.ndim || G.bc[b][0] == GMUNU_MG_PERIODIC || (cc[b] > 0 && cc[b] < G.n[b] - 1)) continue;
      mg_w(G, cc[0] + G.g[0], cc[1] + G.g[1], b, wm, wp);
      if (cc[b] == 0) dg += wm * mg_fold(G, cc, b, false);
      if (cc[b] == G.n[b] - 1) dg += wp * mg_fold(G, cc, b, true);
    }
    mg_w(G, cc[0] + G.g[0], cc[1] + G.g[1], ax, wm, wp);
    const double id = rcp(dg);
    wm = m == 0 ? 0.0 : wm * id;
    wp = m == n - 1 ? 0.0 : wp * id;
    d = (f[o] - Lu) * id;
  }
  mg_pcr<1>(sm, n, m, on, one_wave, &wm, &wp, &d);
  if (on) u[o] += d;
}

__global__ __launch_bounds__(kMaxLine) void k_mg_line(const MgGeo G, double *u, const double *__restrict__ f,
                                                      const double *__restrict__ a, const double *__restrict__ a2,
                                                      int ax, int colour) {
  extern __shared__ double sm[];
  int c[3];
  if (!mg_line(G, ax, colour, mg_xcd_run(), c)) return;
  mg_line_step(G, u, f, a, a2, ax, c, true, sm, threadIdx.x, blockDim.x == kLineWave);
}

// Number of lines of colour `colour` along axis a.
__host__ __device__ __forceinline__ long mg_line_count(const MgGeo &G, int a, int colour) {
  const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
  const long h1 = b1 < G.ndim ? (G.n[b1] - (colour & 1) + 1) >> 1 : 1;
  const long h2 = b2 < G.ndim ? (G.n[b2] - ((colour >> 1) & 1) + 1) >> 1 : 1;
  return h1 * h2;
}

// The coarsest-level solver of the line smoother: `sweeps` line sweeps by
// one workgroup, `lanes` lanes to a line, a colour's lines in rounds, colours
// and axes separated by barriers.  Dynamic LDS: the level's u, f (and the
// given a, a2) copied in and u copied back, then 6 nmax doubles per line at
// work.  No more wavefronts than a colour has lines, and no barrier inside a
// line of one wavefront: 10 wavefronts on 20x2 cells take 54.6 us, 16 meeting
// at a barrier per doubling took 86.8.
__global__ __launch_bounds__(kCoarseLineThreads) void k_mg_line_coarse(const MgGeo G, double *u,
                                                                       const double *__restrict__ f,
                                                                       const double *__restrict__ a,
                                                                       const double *__restrict__ a2, int sweeps,
                                                                       int nmax, int lanes) {
  extern __shared__ double sm[];
  double *p = sm, *uu = p;
  for (long e = threadIdx.x; e < G.nt; e += blockDim.x) p[e] = u[e];
  p += G.nt;
  for (long e = threadIdx.x; e < G.nt; e += blockDim.x) p[e] = f[e];
  const double *ff = p, *aa = nullptr, *aa2 = nullptr;
  p += G.nt;
  if (a) {
    for (long e = threadIdx.x; e < G.nt; e += blockDim.x) p[e] = a[e];
    aa = p;
    p += G.nt;
  }
  if (a2) {
    for (long e = threadIdx.x; e < G.nt; e += blockDim.x) p[e] = a2[e];
    aa2 = p;
    p += G.nt;
  }
  __syncthreads();
  const int w = threadIdx.x / lanes, ln = threadIdx.x % lanes, nw = blockDim.x / lanes;
  for (int s = 0; s < sweeps; s++)
    for (int ax = 0; ax < G.ndim; ax++) {
      if (G.bc[ax][0] == GMUNU_MG_PERIODIC) continue;
      for (int col = 0; col < 1 << (G.ndim - 1); col++) {
        const long nl = mg_line_count(G, ax, col);
        for (long t0 = 0; t0 < nl; t0 += nw) {
          int c[3] = {0, 0, 0};
          const bool live = mg_line(G, ax, col, t0 + w, c);
          mg_line_step(G, uu, ff, aa, aa2, ax, c, live, p + (long)w * 6 * nmax, ln, lanes == kLineWave);
          __syncthreads();
        }
      }
    }
  for (long e = threadIdx.x; e < G.nt; e += blockDim.x) u[e] = uu[e];
}

// out = L(u) on the interior.
__global__ __launch_bounds__(NT) void k_mg_apply(const MgGeo G, const double *__restrict__ u,
                                                 const double *__restrict__ a, const double *__restrict__ a2,
                                                 double *__restrict__ out) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = mg_off(G, i, j, k);
  out[o] = mg_L<true>(G, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, i, j, k, o, nullptr);
}

// Per-workgroup maxima of |f - L(u)| over a grid-stride range of cells.
__global__ __launch_bounds__(NT) void k_mg_norm(const MgGeo G, const double *__restrict__ u,
                                                const double *__restrict__ f, const double *__restrict__ a,
                                                const double *__restrict__ a2, double *part) {
  double m = 0.0;
  for (long t = (long)blockIdx.x * NT + threadIdx.x; t < mg_cells(G); t += (long)gridDim.x * NT) {
    int i, j, k;
    mg_cell(G, t, i, j, k);
    const long o = mg_off(G, i, j, k);
    m = mg_absmax(m, f[o] - mg_L<false>(G, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, i, j, k, o, nullptr));
  }
  m = block_max(m);
  if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// Eight loads in flight per thread (16384 partials one by one took 22 us).
__global__ __launch_bounds__(NT) void k_mg_norm_finish(double *part, int nparts) {
  double m[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nparts; b += 8 * NT)
#pragma unroll
    for (int q = 0; q < 8; q++)
      if (b + q * NT < nparts) m[q] = fmax(m[q], part[b + q * NT]);
#pragma unroll
  for (int q = 1; q < 8; q++) m[0] = fmax(m[0], m[q]);
  const double r = block_max(m[0]);
  if (threadIdx.x == 0) part[kNormParts] = r;
}

// coarse = volume-weighted mean of the children (F: fine level, C: coarse).
__global__ __launch_bounds__(NT) void k_mg_restrict(const MgGeo F, const MgGeo C, const double *__restrict__ fine,
                                                    double *__restrict__ coarse) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(C)) return;
  int i, j, k;
  mg_cell(C, t, i, j, k);
  double s = 0.0, w = 0.0;
  const int nch = 1 << F.ndim;
  for (int ch = 0; ch < nch; ch++) {
    const int fi = 2 * i + (ch & 1);
    const int fj = F.ndim > 1 ? 2 * j + ((ch >> 1) & 1) : j;
    const int fk = F.ndim > 2 ? 2 * k + ((ch >> 2) & 1) : k;
    const double v = F.vol0[fi + F.g[0]] * F.vol1[fj + F.g[1]];
    s += v * fine[mg_off(F, fi, fj, fk)];
    w += v;
  }
  coarse[mg_off(C, i, j, k)] = s / w;
}

// FAS coarse problem: f_c = L_c(u_c) + r_c, and uo_c = u_c.
__global__ __launch_bounds__(NT) void k_mg_fas_rhs(const MgGeo C, const double *__restrict__ u,
                                                   const double *__restrict__ a, const double *__restrict__ a2,
                                                   const double *__restrict__ r, double *__restrict__ f,
                                                   double *__restrict__ uo) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(C)) return;
  int i, j, k;
  mg_cell(C, t, i, j, k);
  const long o = mg_off(C, i, j, k);
  f[o] = mg_L<false>(C, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, i, j, k, o, nullptr) + r[o];
  uo[o] = u[o];
}

// Coarse problem of a fine 1D level in one pass over the coarse cells: the
// residual f - L(u) of both children (boundary rule inline) and the
// volume-weighted means of u and of the residual into the coarse u and r.
// (Of 2D and 3D levels: k_mg_res.)
__global__ __launch_bounds__(NT) void k_mg_restrict_res(const MgGeo F, const MgGeo C, const double *__restrict__ u,
                                                        const double *__restrict__ f, const double *__restrict__ a,
                                                        const double *__restrict__ a2, double *__restrict__ uc,
                                                        double *__restrict__ rc) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(C)) return;
  double su = 0.0, sr = 0.0, w = 0.0;
#pragma unroll
  for (int ch = 0; ch < 2; ch++) {
    const int i = 2 * (int)t + ch;
    const double v = F.vol0[i + 1];
    const long o = mg_off(F, i, 0, 0);
    su += v * u[o];
    sr += v * (f[o] - mg_L<false>(F, u, a ? a[o] : 0.0, a2 ? a2[o] : 0.0, i, 0, 0, o, nullptr));
    w += v;
  }
  const long oc = mg_off(C, (int)t, 0, 0);
  uc[oc] = su / w;
  rc[oc] = sr / w;
}

// u_F += P (u_C - uo_C): Kwak prolongation of the coarse correction, whose
// values across the boundary follow the boundary rule (it is homogeneous,
// so the correction obeys it too); NC components back to back.
__device__ __forceinline__ double mg_corr(const MgGeo &C, const double *__restrict__ u,
                                          const double *__restrict__ uo, long o) {
  return u[o] - uo[o];
}

// One thread per coarse cell and component: the differences of the cell and its
// 2 ndim neighbours (boundary rule as a factor of its own) serve its 2^ndim
// children.  Bound by memory: 256^3 fine cells take 66 us (16 B per fine
// cell and a quarter of that again from the coarse level); one thread per
// child, with its neighbours' rules in branches, took 142.
template <int NC>
__global__ __launch_bounds__(NT) void k_mg_correct(const MgGeo C, const MgGeo F, const double *__restrict__ uc0,
                                                   const double *__restrict__ uoc0, double *__restrict__ fine0) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(C)) return;
  int cc[3];
  mg_cell(C, t, cc[0], cc[1], cc[2]);
  const int q = NC == 1 ? 0 : (int)blockIdx.y, nd = C.ndim;
  const double *uc = uc0 + q * C.nt, *uoc = uoc0 + q * C.nt;
  double *fine = fine0 + q * F.nt;
  const long oc = mg_off(C, cc[0], cc[1], cc[2]);
  const int S[3] = {1, (int)C.s1, (int)C.s2};
  int at[3][2];
  double fac[3][2];
#pragma unroll
  for (int a = 0; a < 3; a++)
#pragma unroll
    for (int d = 0; d < 2; d++) {
      at[a][d] = 0;
      fac[a][d] = 0.25;
      if (a >= nd) continue;
      const int n = C.n[a], kind = C.bc[a][d];
      const bool inside = d ? cc[a] < n - 1 : cc[a] > 0;
      const int step = inside ? S[a] : kind == GMUNU_MG_PERIODIC ? -(n - 1) * S[a] : 0;
      at[a][d] = d ? step : -step;
      if (!inside && kind != GMUNU_MG_PERIODIC) {
        if (NC == 3)  // vector components: their parity across the face
          fac[a][d] = (C.vodd[a][d] >> q) & 1 ? -0.25 : 0.25;
        else
          fac[a][d] = kind == GMUNU_MG_DIRICHLET ? -0.25
                      : kind == GMUNU_MG_NEUMANN ? 0.25
                                                 : 0.25 * mg_rob(C, cc[0], cc[1], cc[2], a, d);
      }
    }
  const double e0 = (nd == 1 ? 0.75 : nd == 2 ? 0.5 : 0.25) * mg_corr(C, uc, uoc, oc);
  double e[3][2];
#pragma unroll
  for (int a = 0; a < 3; a++)
#pragma unroll
    for (int d = 0; d < 2; d++) e[a][d] = a < nd ? fac[a][d] * mg_corr(C, uc, uoc, oc + at[a][d]) : 0.0;
  const long of = mg_off(F, 2 * cc[0], nd > 1 ? 2 * cc[1] : cc[1], nd > 2 ? 2 * cc[2] : cc[2]);
  double v[8];
#pragma unroll
  for (int ch = 0; ch < 8; ch++)
    if (ch >> nd == 0) v[ch] = fine[of + (ch & 1) + ((ch >> 1) & 1) * F.s1 + (ch >> 2) * F.s2];
#pragma unroll
  for (int ch = 0; ch < 8; ch++)
    if (ch >> nd == 0)
      fine[of + (ch & 1) + ((ch >> 1) & 1) * F.s1 + (ch >> 2) * F.s2] =
          v[ch] + (((e0 + e[0][ch & 1]) + e[1][(ch >> 1) & 1]) + e[2][ch >> 2]);
}

// ---- Tail of the hierarchy -------------------------------------------------
// A V-cycle (or the whole FMG cycle) over the coarse levels 0 .. top by one
// workgroup, on copies of the levels' arrays in LDS, every phase separated by
// a workgroup barrier (sweeps of at most one wavefront's cells run in one
// wavefront without one).  As launches these levels are latency alone: eleven
// launches of 3 to 5 us per level and cycle, whatever the level's size.  The
// phases are a program made on the host, so that each body is compiled once
// and the kernel stays small in registers and instruction cache (a version
// with the bodies inlined per level ran at the launches' speed).  A phase is
// bound by its chain of LDS reads and FP64 operations, about 1 us: on a
// 128 x 96 grid the levels 64 x 48 and below take 64 us per V-cycle (with ten
// coarsest sweeps) against about 160 us as launches, and the cleaning solve
// 1.14 instead of 2.05 ms; the limit of 4096 cells is the LDS that four
// arrays per level leave.

constexpr int kTailThreads = 1024;
constexpr int kTailLds = 20352;   // doubles of LDS (159 KB of the CU's 160)
constexpr int kTailCells = 4096;  // most cells of a tail level
constexpr int kTailLevels = 13;
constexpr int kTailSlots = 2;     // cells of one colour per thread, at most
enum { kOpSweep = 0, kOpCoarse = 1, kOpCorrect = 2 };

// One level of the tail: sizes, magic multipliers of the divisions by
// (n0 + 1) / 2, n0 and n1, and the places of its arrays in LDS (offsets in
// doubles, interior cells only, x fastest; -1: absent; tab: the 1D tables
// a0m, a0p, g1, g2, vol0 and a1m, a1p, s2t, vol1 of curvilinear levels).
struct MgLev {
  int n[3], s2, nc, cells;
  unsigned mh, mn0, mn1;
  int u, f, a, a2, uo, tab;
  int per[3];         // periodic axes
  unsigned rob;       // faces with a position-dependent Robin factor (bit 2 axis + side)
  double fac[3][2];   // boundary factor of the other faces
  double w[3];        // Cartesian weights 1 / h^2 (w[2] also of the others' axis 2)
  double x0[3], h[3];
};

struct MgTail {
  MgLev lev[kTailLevels];
  int ndim, coord, power, power2, top;
  double offset;
  int sweeps[3];                // pre, post, coarse
  int nprog[2];                 // V-cycle, FMG cycle
  int prog[2][512];             // op + 4 level + 64 (which of sweeps)
};

// u / d with the magic multiplier m of d (0: d = 1); exact for u d < 2^32.
__device__ __forceinline__ int mg_div(int u, unsigned m) { return m ? (int)__umulhi((unsigned)u, m) : u; }

// A tail cell's stencil: its offset, the steps to its neighbours (0 across a
// face of the domain, whose value is the boundary rule applied to the cell
// itself), the faces it lies on (bit 2 axis + side) and the rule's factor per
// axis (a level has at least two cells along an axis, so at most one face
// per axis).  CA: Cartesian weights (three scalars; else from the level's
// tables); ROB: faces whose Robin factor depends on the position exist; NL:
// power -1 or a second term.
struct MgCell {
  int o, dm[3], dp[3], i, j;
  unsigned edge;
  double fac[3];
};

template <bool ROB>
__device__ __forceinline__ MgCell mg_tail_stencil(const MgTail &T, const MgLev &V, int i, int j, int k) {
  MgCell c;
  const int x[3] = {i, j, k}, S[3] = {1, V.n[0], V.s2};
  c.i = i;
  c.j = j;
  c.o = i + V.n[0] * j + V.s2 * k;
  c.edge = 0;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const int n = V.n[a], wrap = V.per[a] ? (n - 1) * S[a] : 0;
    const bool lo = x[a] == 0, hi = x[a] == n - 1;
    c.dm[a] = lo ? wrap : -S[a];
    c.dp[a] = hi ? -wrap : S[a];
    if (!V.per[a]) c.edge |= (lo ? 1u : 0u) << (2 * a) | (hi ? 2u : 0u) << (2 * a);
    c.fac[a] = hi ? V.fac[a][1] : V.fac[a][0];
  }
  if (ROB && (c.edge & V.rob)) {
    // r_in / r_ghost
    double y[3], rr = 0.0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
      y[a] = V.x0[a] + (x[a] + 0.5) * V.h[a];
      if (a < T.ndim && (a < 2 || T.coord == GMUNU_CART)) rr += y[a] * y[a];
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
      if (!((c.edge & V.rob) >> (2 * a) & 3)) continue;
      const double g = (c.edge >> (2 * a)) & 2 ? y[a] + V.h[a] : y[a] - V.h[a];
      c.fac[a] = mg_dist_ratio(rr, rr - y[a] * y[a] + g * g);
    }
  }
  return c;
}

// L(u) and dL/du at a tail cell with coefficients av, a2v.
template <bool CA, bool NL>
__device__ __forceinline__ double mg_tail_L(const MgTail &T, const MgLev &V, const double *sm, const MgCell &c,
                                            double av, double a2v, double &dg) {
  const double *u = sm + V.u;
  const double uc = u[c.o];
  const int I = c.i + 1, J = c.j + (T.ndim > 1 ? 1 : 0), t0 = V.n[0] + 2, t1 = V.n[1] + (T.ndim > 1 ? 2 : 0);
  const double *p0 = sm + V.tab, *p1 = p0 + 5 * t0;
  double lap = 0.0, d = 0.0;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    if (a >= T.ndim) continue;
    double um = u[c.o + c.dm[a]], up = u[c.o + c.dp[a]];
    if ((c.edge >> (2 * a)) & 1) um *= c.fac[a];
    if ((c.edge >> (2 * a)) & 2) up *= c.fac[a];
    double wm, wp;
    if (CA) {
      wm = wp = V.w[a];
    } else if (a == 0) {
      wm = p0[I];
      wp = p0[t0 + I];
    } else if (a == 1) {
      wm = p0[2 * t0 + I] * p1[J];
      wp = p0[2 * t0 + I] * p1[t1 + J];
    } else {
      wm = wp = p0[3 * t0 + I] * p1[2 * t1 + J] * V.w[2];
    }
    lap += wp * (up - uc) - wm * (uc - um);
    d -= wm + wp;
  }
  if (NL) {
    double du;
    lap -= mg_nl_both(T.power, T.power2, T.offset, av, a2v, uc, du);
    dg = d - du;
  } else {
    const bool lin = T.power == 1;
    lap -= lin ? av * (uc + T.offset) : av;
    dg = lin ? d - av : d;
  }
  return lap;
}

__device__ __forceinline__ void mg_tail_cell(const MgLev &V, int t, int &i, int &j, int &k) {
  const int r = mg_div(t, V.mn0);
  i = t - r * V.n[0];
  k = mg_div(r, V.mn1);
  j = r - k * V.n[1];
}

// Sum over the 2^ndim lanes of one coarse cell.
__device__ __forceinline__ double mg_sum_children(double x, int ndim) {
  for (int o = 1; o < 1 << ndim; o <<= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Red-black sweeps of one level.  A thread keeps the stencils and coefficients
// of its cells (up to kTailSlots of each colour) in registers over the sweeps.
template <bool CA, bool ROB, bool NL>
__device__ __forceinline__ void mg_tail_sweeps(const MgTail &T, const MgLev &Vg, double *sm, int sweeps) {
  const MgLev V = Vg;  // in registers over the sweeps
  const int nc = V.nc, hrow = (V.n[0] + 1) >> 1, n0 = V.n[0], n1 = V.n[1];
  const bool one_wave = nc <= 64;
  if (!one_wave || threadIdx.x < 64) {
    MgCell c[kTailSlots][2];
    double f[kTailSlots][2], av[kTailSlots][2], a2v[kTailSlots][2];
    bool on[kTailSlots][2];
#pragma unroll
    for (int m = 0; m < kTailSlots; m++) {
      const int t = threadIdx.x + m * blockDim.x;
      const int row = mg_div(t, V.mh), k = mg_div(row, V.mn1), j = row - k * n1, h = 2 * (t - row * hrow);
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const int i = h + ((j + k + s) & 1);
        on[m][s] = t < nc && i < n0;
        if (!on[m][s]) continue;
        c[m][s] = mg_tail_stencil<ROB>(T, V, i, j, k);
        f[m][s] = sm[V.f + c[m][s].o];
        av[m][s] = V.a >= 0 ? sm[V.a + c[m][s].o] : 0.0;
        a2v[m][s] = NL && V.a2 >= 0 ? sm[V.a2 + c[m][s].o] : 0.0;
      }
    }
    for (int n = 0; n < sweeps; n++) {
#pragma unroll
      for (int s = 0; s < 2; s++) {
#pragma unroll
        for (int m = 0; m < kTailSlots; m++) {
          if (!on[m][s]) continue;
          double dg;
          const double L = mg_tail_L<CA, NL>(T, V, sm, c[m][s], av[m][s], a2v[m][s], dg);
          sm[V.u + c[m][s].o] -= (L - f[m][s]) * rcp(dg);
        }
        if (one_wave)
          wave_fence();
        else
          __syncthreads();
      }
    }
  }
  if (one_wave) __syncthreads();
}

// The coarse problem of level C below F, one lane per child in the restriction.
template <bool CA, bool ROB, bool NL>
__device__ __forceinline__ void mg_tail_coarse_problem(const MgTail &T, const MgLev &F, const MgLev &C, double *sm) {
  const int nc = C.cells, nd = T.ndim;
  // every lane of a wavefront takes part in the sums: rounds of whole blocks
  for (int t0 = 0; t0 < nc << nd; t0 += blockDim.x) {
    const int t = t0 + threadIdx.x, oc = t >> nd;
    double su = 0.0, sr = 0.0, w = 0.0;
    if (oc < nc) {
      int i, j, k;
      mg_tail_cell(C, oc, i, j, k);
      i = 2 * i + (t & 1);
      if (nd > 1) j = 2 * j + ((t >> 1) & 1);
      if (nd > 2) k = 2 * k + ((t >> 2) & 1);
      const MgCell c = mg_tail_stencil<ROB>(T, F, i, j, k);
      const double *v0 = sm + F.tab + 4 * (F.n[0] + 2), *v1 = v0 + F.n[0] + 2 + 3 * (F.n[1] + (nd > 1 ? 2 : 0));
      w = CA ? 1.0 : v0[i + 1] * v1[j + (nd > 1 ? 1 : 0)];
      double dg;
      const double L = mg_tail_L<CA, NL>(T, F, sm, c, F.a >= 0 ? sm[F.a + c.o] : 0.0,
                                         NL && F.a2 >= 0 ? sm[F.a2 + c.o] : 0.0, dg);
      su = w * sm[F.u + c.o];
      sr = w * (sm[F.f + c.o] - L);
    }
    su = mg_sum_children(su, nd);
    sr = mg_sum_children(sr, nd);
    w = CA ? (double)(1 << nd) : mg_sum_children(w, nd);
    if (oc < nc && (t & ((1 << nd) - 1)) == 0) {
      sm[C.u + oc] = sm[C.uo + oc] = su / w;
      sm[C.f + oc] = sr / w;
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nc; t += blockDim.x) {
    int i, j, k;
    mg_tail_cell(C, t, i, j, k);
    const MgCell c = mg_tail_stencil<ROB>(T, C, i, j, k);
    double dg;
    sm[C.f + t] += mg_tail_L<CA, NL>(T, C, sm, c, C.a >= 0 ? sm[C.a + t] : 0.0, NL && C.a2 >= 0 ? sm[C.a2 + t] : 0.0,
                                     dg);
  }
  __syncthreads();
}

// u_F += P(u_C - uo_C): k_mg_correct on the LDS arrays.
__device__ __forceinline__ void mg_tail_correct(const MgTail &T, const MgLev &F, const MgLev &C, double *sm) {
  const int nd = T.ndim;
  const double w0 = nd == 1 ? 0.75 : nd == 2 ? 0.5 : 0.25;
  const double *uc = sm + C.u, *uoc = sm + C.uo;
  const int S[3] = {1, C.n[0], C.s2};
  for (int t = threadIdx.x; t < F.cells; t += blockDim.x) {
    int fc[3];
    mg_tail_cell(F, t, fc[0], fc[1], fc[2]);
    const int cc[3] = {fc[0] >> 1, nd > 1 ? fc[1] >> 1 : fc[1], nd > 2 ? fc[2] >> 1 : fc[2]};
    const int oc = cc[0] + S[1] * cc[1] + S[2] * cc[2];
    const double e0 = uc[oc] - uoc[oc];
    double s = w0 * e0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
      if (a >= nd) continue;
      const bool up = fc[a] & 1;
      const int n = C.n[a];
      const bool inside = up ? cc[a] < n - 1 : cc[a] > 0;
      const int step = inside ? S[a] : C.per[a] ? -(n - 1) * S[a] : 0, on = up ? oc + step : oc - step;
      double e = uc[on] - uoc[on];
      if (!inside && !C.per[a]) {
        double fac = up ? C.fac[a][1] : C.fac[a][0];
        if ((C.rob >> (2 * a + (up ? 1 : 0))) & 1) {
          double ri = 0.0, rg = 0.0;
#pragma unroll
          for (int b = 0; b < 3; b++) {
            if (b >= nd || (b == 2 && T.coord != GMUNU_CART)) continue;
            const double x = C.x0[b] + (cc[b] + 0.5) * C.h[b], g = b == a ? (up ? x + C.h[b] : x - C.h[b]) : x;
            ri += x * x;
            rg += g * g;
          }
          fac = mg_dist_ratio(ri, rg);
        }
        e = fac * e0;
      }
      s += 0.25 * e;
    }
    sm[F.u + t] += s;
  }
  __syncthreads();
}

// The cells of a level between its global array (ghost layers as in the
// level's own geometry) and LDS.
template <bool OUT>
__device__ __forceinline__ void mg_tail_copy(const MgTail &T, const MgLev &V, double *glob, double *lds) {
  const int g1 = T.ndim > 1 ? 1 : 0, g2 = T.ndim > 2 ? 1 : 0;
  const int S1 = V.n[0] + 2, S2 = S1 * (V.n[1] + 2 * g1);
  for (int t = threadIdx.x; t < V.cells; t += blockDim.x) {
    int i, j, k;
    mg_tail_cell(V, t, i, j, k);
    const int o = (k + g2) * S2 + (j + g1) * S1 + i + 1;
    if (OUT)
      glob[o] = lds[t];
    else
      lds[t] = glob[o];
  }
}

// Tt: the plan; geo: the levels' geometries; u, f, a_top, a2_top: the top
// level's arrays; ptr: the a (then a2) arrays of the levels below (device
// memory).
template <bool CA, bool ROB, bool NL>
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(const MgTail *__restrict__ Tt, const MgGeo *__restrict__ geo,
                                                          double *u, const double *__restrict__ f,
                                                          const double *a_top, const double *a2_top,
                                                          double *const *__restrict__ ptr, int use_fmg) {
  __shared__ double sm[kTailLds];
  const MgTail &T = *Tt;
  mg_tail_copy<false>(T, T.lev[T.top], u, sm + T.lev[T.top].u);
  mg_tail_copy<false>(T, T.lev[T.top], const_cast<double *>(f), sm + T.lev[T.top].f);
  for (int l = 0; l <= T.top; l++) {
    const MgLev &V = T.lev[l];
    if (V.a >= 0) mg_tail_copy<false>(T, V, l == T.top ? const_cast<double *>(a_top) : ptr[l], sm + V.a);
    if (V.a2 >= 0)
      mg_tail_copy<false>(T, V, l == T.top ? const_cast<double *>(a2_top) : ptr[kTailLevels + l], sm + V.a2);
    if (!CA) {
      const MgGeo &g = geo[l];
      const int t0 = V.n[0] + 2, t1 = V.n[1] + (T.ndim > 1 ? 2 : 0);
      double *p = sm + V.tab;
      for (int t = threadIdx.x; t < t0; t += blockDim.x) {
        p[t] = g.a0m[t];
        p[t0 + t] = g.a0p[t];
        p[2 * t0 + t] = g.g1[t];
        p[3 * t0 + t] = g.g2[t];
        p[4 * t0 + t] = g.vol0[t];
      }
      p += 5 * t0;
      for (int t = threadIdx.x; t < t1; t += blockDim.x) {
        p[t] = g.a1m[t];
        p[t1 + t] = g.a1p[t];
        p[2 * t1 + t] = g.s2t[t];
        p[3 * t1 + t] = g.vol1[t];
      }
    }
  }
  __syncthreads();
  const int np = T.nprog[use_fmg];
  for (int pc = 0; pc < np; pc++) {
    const int op = T.prog[use_fmg][pc], l = (op >> 2) & 15;
    if ((op & 3) == kOpSweep)
      mg_tail_sweeps<CA, ROB, NL>(T, T.lev[l], sm, T.sweeps[op >> 6]);
    else if ((op & 3) == kOpCoarse)
      mg_tail_coarse_problem<CA, ROB, NL>(T, T.lev[l], T.lev[l - 1], sm);
    else
      mg_tail_correct(T, T.lev[l], T.lev[l - 1], sm);
  }
  mg_tail_copy<true>(T, T.lev[T.top], u, sm + T.lev[T.top].u);
}

// ---- Red-black sweeps out of place ------------------------------------------
// NS sweeps (2 NS colours) of a 2D or 3D level in one launch, from u to out.  A
// workgroup relaxes a 32 x 16 tile in x and y with a halo of H = 2 NS cells,
// the halo's cells redundantly; a thread owns one pair of x-neighbours (one
// cell of each colour in every plane).  In 3D it marches along z over a chunk
// of planes (H more below and above) through a ring of planes in LDS: at step
// p colour s is relaxed on plane p - (2 s - 1), which only needs the colour
// before it on planes relaxed in earlier steps, so a step has one barrier and
// 2 NS independent updates per thread; the planes of u, f, a and a2 are loaded
// two steps ahead, f, a and a2 once (kept in registers over the pipeline).  As launches per colour a pair of
// sweeps moves 96 bytes per cell (u four times, f and a in half lines); here
// 32.  Measured on 256^3 cells with a (u + c): 200 us per pair of sweeps against
// 474 as four launches (38 B per cell with the halo in flight: 3.2 TB/s; two
// wavefronts per SIMD in each of two workgroups, VALU and LDS about half busy
// each).  What it took: f and a fetched once (fetched per colour in half lines
// they missed the L2: 285 us), no branch in a step (the loads' waits cannot
// cross one: 295 us), faces folded into a factor of u (358 us).  Blocks of 32 x
// 8 x 8 cells staged at once, whose halo doubles the updates, took 558 us.

template <int ND, int NS>
struct RbTile {
  static constexpr int H = 2 * NS, TX = 32, TY = 16;
  static constexpr int HX = TX / 2 + H, RX = 2 * HX, RY = TY + 2 * H;  // pairs, cells and rows staged
  static constexpr int P = RX * RY;                                    // cells of a staged plane
  static constexpr int ring = ND > 2 ? 4 * NS + 2 : 1;
  static constexpr int threads = (HX * RY + 63) / 64 * 64;
};

// Index wrapped into [0, n).
__device__ __forceinline__ int mg_wrap(int i, int n) {
  if (i >= 0 && i < n) return i;
  i %= n;
  return i < 0 ? i + n : i;
}

// One cell of a thread's pair: place in a staged plane (even cells of a row,
// then odd ones, so that a colour's reads are contiguous) and of its
// neighbours there, place in a global plane, and what depends on (x, y) alone.
// Across a face of the domain the neighbour is the cell itself, whose
// difference vanishes, and the boundary rule u_ghost = s u adds (s - 1) times
// the face's weight to the factor cc of u: no branch in the update.  ROB:
// faces whose s depends on the position (their part of cc per update).
template <bool CA>
struct RbCell {
  int o, xm, xp, ym, yp;
  unsigned og;           // bytes
  int ow;                // o where the cell is relaxed, else the corner (0, 0), which no relaxed cell reads
  bool on;               // inside the domain (or a periodic image)
  unsigned rob;          // bits: such a face on the lower / upper side of axis 0, of axis 1
  double cc, x, y;       // x, y: centre
  double w[CA ? 1 : 5];  // curvilinear weights: a0m, a0p, g1 a1m, g1 a1p, g2 s2t / h2^2
};

// s - 1 of the boundary rule across face (a, side), 0 where it depends on the
// position.
__device__ __forceinline__ double mg_fold1(const MgGeo &G, int a, int side) {
  const int kind = G.bc[a][side];
  return kind == GMUNU_MG_DIRICHLET ? -2.0
         : kind == GMUNU_MG_ROBIN && G.coord == GMUNU_SPH ? (side ? G.rob_hi : G.rob_lo) - 1.0
                                                          : 0.0;
}
__device__ __forceinline__ bool mg_robin(const MgGeo &G, int a, int side) {
  return G.coord != GMUNU_SPH && G.bc[a][side] == GMUNU_MG_ROBIN;
}
// r_in / r_ghost - 1 for a cell at x along the face's axis (its ghost at g), rr
// its squared distance.
__device__ __forceinline__ double mg_robin1(double rr, double x, double g) {
  return mg_dist_ratio(rr, rr - x * x + g * g) - 1.0;
}

template <int ND, int NS, bool CA>
__device__ __forceinline__ RbCell<CA> mg_rb_cell(const MgGeo &G, int i0, int j0, int h, int y, int par) {
  using R = RbTile<ND, NS>;
  RbCell<CA> c;
  const int row = y * R::RX;
  int i = i0 - R::H + 2 * h + par, j = j0 - R::H + y;
  const bool px = G.bc[0][0] == GMUNU_MG_PERIODIC, py = G.bc[1][0] == GMUNU_MG_PERIODIC;
  c.on = y < R::RY && (px || (i >= 0 && i < G.n[0])) && (py || (j >= 0 && j < G.n[1]));
  if (px) i = mg_wrap(i, G.n[0]);
  if (py) j = mg_wrap(j, G.n[1]);
  const bool f0 = !px && i == 0, f1 = !px && i == G.n[0] - 1, f2 = !py && j == 0, f3 = !py && j == G.n[1] - 1;
  // threads without a cell, and rim cells without a neighbour, read places
  // that exist
  const bool in = y < R::RY;
  c.o = in ? row + (par ? R::HX : 0) + h : 0;
  c.xm = f0 || !in || (!par && h == 0) ? c.o : par ? row + h : row + R::HX + h - 1;
  c.xp = f1 || !in || (par && h + 1 == R::HX) ? c.o : par ? row + h + 1 : row + R::HX + h;
  c.ym = f2 || !in || y == 0 ? c.o : c.o - R::RX;
  c.yp = f3 || !in || y == R::RY - 1 ? c.o : c.o + R::RX;
  const int x = 2 * h + par;
  c.ow = c.on && x >= 1 && x < R::RX - 1 && y >= 1 && y < R::RY - 1 ? c.o : 0;
  c.x = G.x0[0] + (i + 0.5) * G.h[0];
  c.y = G.x0[1] + (j + 0.5) * G.h[1];
  c.og = c.on ? 8u * (unsigned)((j + 1) * (int)G.s1 + i + 1) : 0u;
  const int I = c.on ? i + 1 : 1, J = c.on ? j + 1 : 1;
  double wm0 = G.vih2[0], wp0 = wm0, wm1 = G.vih2[1], wp1 = wm1;
  if constexpr (!CA) {
    c.w[0] = wm0 = G.a0m[I];
    c.w[1] = wp0 = G.a0p[I];
    c.w[2] = wm1 = G.g1[I] * G.a1m[J];
    c.w[3] = wp1 = G.g1[I] * G.a1p[J];
    c.w[4] = ND > 2 ? G.g2[I] * G.s2t[J] * G.ih2_2 : 0.0;
  }
  c.cc = (f0 ? wm0 * mg_fold1(G, 0, 0) : 0.0) + (f1 ? wp0 * mg_fold1(G, 0, 1) : 0.0) +
         (f2 ? wm1 * mg_fold1(G, 1, 0) : 0.0) + (f3 ? wp1 * mg_fold1(G, 1, 1) : 0.0);
  c.rob = (f0 && mg_robin(G, 0, 0) ? 1u : 0u) | (f1 && mg_robin(G, 0, 1) ? 2u : 0u) |
          (f2 && mg_robin(G, 1, 0) ? 4u : 0u) | (f3 && mg_robin(G, 1, 1) ? 8u : 0u);
  return c;
}

// Newton update of cell c on the plane at sm + zc (neighbour planes at zm and
// zp; on a face of axis 2 the plane itself), zs: s - 1 of that face (0 off the
// faces), zr: bits of a face of axis 2 whose s depends on the position, k the
// index along axis 2 (of the cell itself where the plane is a periodic image).
// M: the terms (0: none, 1: a (u + c), 2: general).  Returns the new value.
template <int ND, bool CA, int M, bool ROB>
__device__ __forceinline__ double mg_rb_update(const MgGeo &G, const double *sm, const RbCell<CA> &c, int zc, int zm,
                                               int zp, double zs, unsigned zr, int k, double fv, double av,
                                               double a2v) {
  const double *u = sm + zc;
  const double uc = u[c.o], xm = u[c.xm], xp = u[c.xp], ym = u[c.ym], yp = u[c.yp];
  double lap, d, cc = c.cc, zw;
  if constexpr (CA) {
    lap = G.vih2[0] * ((xp - uc) - (uc - xm));
    lap += G.vih2[1] * ((yp - uc) - (uc - ym));
    zw = ND > 2 ? G.vih2[2] : 0.0;
    d = -2.0 * (G.vih2[0] + G.vih2[1] + zw);
  } else {
    lap = c.w[1] * (xp - uc) - c.w[0] * (uc - xm);
    lap += c.w[3] * (yp - uc) - c.w[2] * (uc - ym);
    zw = c.w[4];
    d = -(c.w[0] + c.w[1]) - (c.w[2] + c.w[3]) - 2.0 * zw;
  }
  if (ND > 2) {
    lap += zw * ((sm[zp + c.o] - uc) - (uc - sm[zm + c.o]));
    if (zs != 0.0) cc += zw * zs;
  }
  if (ROB && (c.rob || zr)) {
    double rr = c.x * c.x + c.y * c.y, z = 0.0;
    if (ND > 2 && G.coord == GMUNU_CART) {
      z = G.x0[2] + (k + 0.5) * G.h[2];
      rr += z * z;
    }
    const double wm0 = CA ? G.vih2[0] : c.w[0], wp0 = CA ? G.vih2[0] : c.w[CA ? 0 : 1];
    const double wm1 = CA ? G.vih2[1] : c.w[CA ? 0 : 2], wp1 = CA ? G.vih2[1] : c.w[CA ? 0 : 3];
    if (c.rob & 3u) cc += (c.rob & 1u ? wm0 : wp0) * mg_robin1(rr, c.x, c.rob & 1u ? c.x - G.h[0] : c.x + G.h[0]);
    if (c.rob & 12u) cc += (c.rob & 4u ? wm1 : wp1) * mg_robin1(rr, c.y, c.rob & 4u ? c.y - G.h[1] : c.y + G.h[1]);
    // (a level has two planes or more: a cell lies on one z face)
    if (zr) cc += zw * mg_robin1(rr, z, zr & 1u ? z - G.h[2] : z + G.h[2]);
  }
  lap += cc * uc;
  if constexpr (M == 2) {
    double du;
    lap -= mg_nl_both(G.power, G.power2, G.offset, av, a2v, uc, du);
    d -= du;
  } else if constexpr (M == 1) {
    lap -= av * (uc + G.offset);
    d -= av;
  }
  return uc - (lap - fv) * rcp(d);
}

// f, a and a2 of one update.
struct RbSrc {
  double f, a, a2;
};
// Entry at byte offset b of a plane (a uniform pointer and a 32-bit offset per
// lane: no address arithmetic in the VALU).
__device__ __forceinline__ double mg_rb_at(const double *plane, unsigned b) {
  return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(plane) + b);
}

template <int M>
__device__ __forceinline__ RbSrc mg_rb_src(const double *__restrict__ f, const double *__restrict__ a,
                                           const double *__restrict__ a2, long plane, unsigned b) {
  // M = 2: a or a2 may be absent (zero); f stands in for the address
  const double *pa = M == 2 && !a ? f : a, *pa2 = a2 ? a2 : f;
  RbSrc q;
  q.f = mg_rb_at(f + plane, b);
  q.a = M > 0 ? mg_rb_at(pa + plane, b) : 0.0;
  q.a2 = M == 2 ? mg_rb_at(pa2 + plane, b) : 0.0;
  if (M == 2 && !a) q.a = 0.0;
  if (M == 2 && !a2) q.a2 = 0.0;
  return q;
}

// 2D: the whole tile staged at once.
template <int NS, bool CA, int M, bool ROB>
__device__ __forceinline__ void mg_rb_tile(const MgGeo &G, const double *__restrict__ f, const double *__restrict__ a,
                                           const double *__restrict__ a2, double *__restrict__ out, double *sm,
                                           const RbCell<CA> *c, int h, int y) {
  using R = RbTile<2, NS>;
  RbSrc q[2];
#pragma unroll
  for (int m = 0; m < 2; m++) q[m] = mg_rb_src<M>(f, a, a2, 0, c[m].og);
#pragma unroll
  for (int s = 1; s <= 2 * NS; s++) {
    // x + y + colour even in tile coordinates (the tile and H start even)
    const bool par = (y + s - 1) & 1;
    const RbCell<CA> cc = par ? c[1] : c[0];
    const RbSrc qq = par ? q[1] : q[0];
    sm[cc.ow] = mg_rb_update<2, CA, M, ROB>(G, sm, cc, 0, 0, 0, 0.0, 0u, 0, qq.f, qq.a, qq.a2);
    __syncthreads();
  }
  if (y >= R::H && y < R::RY - R::H && h >= NS && h < R::HX - NS) {
#pragma unroll
    for (int m = 0; m < 2; m++)
      if (c[m].on) out[c[m].og / 8] = sm[c[m].o];
  }
}

// 3D: march over planes z0 .. z1 - 1.
template <int NS, bool CA, int M, bool ROB>
__device__ __forceinline__ void mg_rb_march(const MgGeo &G, const double *__restrict__ u, const double *__restrict__ f,
                                            const double *__restrict__ a, const double *__restrict__ a2,
                                            double *__restrict__ out, double *sm, const RbCell<CA> *c, int h, int y,
                                            int z0, int z1) {
  using R = RbTile<3, NS>;
  constexpr int S = 2 * NS;
  const int n2 = G.n[2];
  const bool pz = G.bc[2][0] == GMUNU_MG_PERIODIC;
  // planes that exist: all (periodic images) or 0 .. n2 - 1
  const int lo = pz ? z0 - R::H : (z0 - R::H > 0 ? z0 - R::H : 0);
  // offset of plane q in the arrays (planes that do not exist: the nearest,
  // whose values are loaded in vain)
  auto plane = [&](int q) { return (long)((pz ? mg_wrap(q, n2) : q < 0 ? 0 : q < n2 ? q : n2 - 1) + 1) * G.s2; };
  // At step p colour s updates, on plane q = p - (2 s - 1), the pair's member m
  // with m + y + q + s - 1 even, that is the parity of y + p - s: odd colours
  // one member, even ones the other, exchanged at every step.  Every cell that
  // has its neighbours in the staged planes is updated at every step: what a
  // colour makes of cells or planes its neighbours' colours have not reached
  // (the halo's rim, the pipeline's first steps) is not read by a cell that
  // is stored.
  const bool flip = (y + lo - 1 + R::H) & 1;
  const RbCell<CA> A = flip ? c[1] : c[0], B = flip ? c[0] : c[1];
  const bool store = y >= R::H && y < R::RY - R::H && h >= NS && h < R::HX - NS;
  const bool outA = store && A.on, outB = store && B.on;
  // po[m], sl[m]: offset in the arrays and place in LDS of plane p + 2 - m;
  // zi[m]: its index, a periodic image's that of its cell (for the Robin factor)
  constexpr int NP = 2 * S + 3;
  long po[NP];
  int sl[NP], zi[NP], top = 2;  // top: the ring's next slot, for plane lo + 2
#pragma unroll
  for (int m = 0; m < NP; m++) {
    po[m] = plane(lo + 2 - m);
    sl[m] = (2 - m + R::ring) % R::ring * R::P;
    if (ROB) zi[m] = pz ? mg_wrap(lo + 2 - m, n2) : lo + 2 - m;
  }
  const double zs0 = pz ? 0.0 : mg_fold1(G, 2, 0), zs1 = pz ? 0.0 : mg_fold1(G, 2, 1);
  const unsigned zr0 = ROB && mg_robin(G, 2, 0) ? 1u : 0u, zr1 = ROB && mg_robin(G, 2, 1) ? 2u : 0u;
  // u two planes ahead (by member), and the right-hand sides of planes p + 1,
  // p, .. that colours still need (member of the odd colours: up to plane
  // p - (2 S - 3); of the even ones: up to p - (2 S - 1)): each is read once,
  // as whole lines, and kept in registers
  constexpr int NO = 2 * S - 1, NE = 2 * S + 1;
  double ua[2], ub[2];
  RbSrc qo[NO], qe[NE];  // index m: plane p + 1 - m
  auto load_u = [&](int m, long o) {
    ua[m] = mg_rb_at(u + o, A.og);
    ub[m] = mg_rb_at(u + o, B.og);
  };
  int zn = pz ? mg_wrap(lo + 2, n2) : 0;  // index of the plane po[0] refers to (periodic)
  // one step: plane p is stored, the colours behind it run, u of plane p + 2
  // and the right-hand sides of p + 2 are fetched.  No branch but the stores':
  // the loads of a step stay in flight over the next one, and the updates of
  // the colours interleave.  X: member of the odd colours, Y: of the even
  // ones; face: one of the updated planes lies on a face of axis 2.
  auto step = [&](auto face, int p, int um, const RbCell<CA> &X, const RbCell<CA> &Y, bool outX, bool outY) {
    sm[sl[2] + A.o] = ua[um];
    sm[sl[2] + B.o] = ub[um];
    __syncthreads();
    double w[S + 1];
#pragma unroll
    for (int s = 1; s <= S; s++) {
      const int q = p - (2 * s - 1), m = 2 * s + 1;
      const bool zlo = face && q == 0, zhi = face && q == n2 - 1;
      const RbSrc &r = s & 1 ? qo[2 * s] : qe[2 * s];
      w[s] = mg_rb_update<3, CA, M, ROB>(G, sm, s & 1 ? X : Y, sl[m], zlo ? sl[m] : sl[m + 1], zhi ? sl[m] : sl[m - 1],
                                         zlo ? zs0 : zhi ? zs1 : 0.0, (zlo ? zr0 : 0u) | (zhi ? zr1 : 0u),
                                         ROB ? zi[m] : 0, r.f, r.a, r.a2);
    }
#pragma unroll
    for (int s = 1; s <= S; s++) sm[sl[2 * s + 1] + (s & 1 ? X : Y).ow] = w[s];
    // the last colour (even: member Y) was just done on plane q, X before
    const int q = p - (2 * S - 1);
    if (q >= z0 && q < z1) {
      char *po_ = reinterpret_cast<char *>(out + po[2 * S + 1]);
      if (outX) *reinterpret_cast<double *>(po_ + X.og) = sm[sl[2 * S + 1] + X.o];
      if (outY) *reinterpret_cast<double *>(po_ + Y.og) = w[S];
    }
    load_u(um, po[0]);
    // on to step p + 1
#pragma unroll
    for (int m = NO - 1; m > 0; m--) qo[m] = qo[m - 1];
#pragma unroll
    for (int m = NE - 1; m > 0; m--) qe[m] = qe[m - 1];
    // plane p + 2: its odd colours come at step p + 3, whose odd member is Y
    qo[0] = mg_rb_src<M>(f, a, a2, po[0], Y.og);
    qe[0] = mg_rb_src<M>(f, a, a2, po[0], X.og);
#pragma unroll
    for (int m = NP - 1; m > 0; m--) {
      po[m] = po[m - 1];
      sl[m] = sl[m - 1];
    }
    if constexpr (ROB) {
#pragma unroll
      for (int m = NP - 1; m > 0; m--) zi[m] = zi[m - 1];
      zi[0]++;
      if (pz && zi[0] == n2) zi[0] = 0;
      if (pz)
        po[0] = zi[0] ? po[1] + G.s2 : G.s2;
      else if (p + 3 < n2)
        po[0] = po[1] + G.s2;
    } else if (pz) {
      zn = zn + 1 == n2 ? 0 : zn + 1;
      po[0] = zn ? po[1] + G.s2 : G.s2;
    } else if (p + 3 < n2) {
      po[0] = po[1] + G.s2;
    }
    top = top + 1 == R::ring ? 0 : top + 1;
    sl[0] = top ? sl[1] + R::P : 0;
  };
  auto run = [&](int p, int um, const RbCell<CA> &X, const RbCell<CA> &Y, bool outX, bool outY) {
    if (!pz && (p <= 2 * S - 1 || p >= n2))
      step(std::true_type{}, p, um, X, Y, outX, outY);
    else
      step(std::false_type{}, p, um, X, Y, outX, outY);
  };
  load_u(0, po[2]);
  load_u(1, po[1]);
#pragma unroll
  for (int m = 0; m < NO; m++) qo[m] = RbSrc{0.0, 0.0, 0.0};
#pragma unroll
  for (int m = 0; m < NE; m++) qe[m] = RbSrc{0.0, 0.0, 0.0};
  // planes lo (odd member B, at step lo + 1) and lo + 1 (A)
  qo[1] = mg_rb_src<M>(f, a, a2, po[2], B.og);
  qe[1] = mg_rb_src<M>(f, a, a2, po[2], A.og);
  qo[0] = mg_rb_src<M>(f, a, a2, po[1], A.og);
  qe[0] = mg_rb_src<M>(f, a, a2, po[1], B.og);
  for (int p = lo; p - (2 * S - 1) < z1; p += 2) {
    run(p, 0, A, B, outA, outB);
    run(p + 1, 1, B, A, outB, outA);
  }
}

template <int ND, int NS, bool CA, int M, bool ROB>
__global__ __launch_bounds__((RbTile<ND, NS>::threads), (ND > 2 && CA && M < 2 && !ROB ? 4 : 2)) void k_mg_rb(const MgGeo G, const double *__restrict__ u,
                                                                     const double *__restrict__ f,
                                                                     const double *__restrict__ a,
                                                                     const double *__restrict__ a2,
                                                                     double *__restrict__ out, int chunk) {
  using R = RbTile<ND, NS>;
  __shared__ double sm[R::P * R::ring];
  // contiguous runs of tiles (x fastest, then y, then chunks of z) per XCD
  const int gx = (G.n[0] + R::TX - 1) / R::TX, gy = (G.n[1] + R::TY - 1) / R::TY;
  const int t = mg_xcd_run();
  const int i0 = t % gx * R::TX, j0 = t / gx % gy * R::TY;
  const int h = threadIdx.x % R::HX, y = threadIdx.x / R::HX;
  const RbCell<CA> c[2] = {mg_rb_cell<ND, NS, CA>(G, i0, j0, h, y, 0), mg_rb_cell<ND, NS, CA>(G, i0, j0, h, y, 1)};
  if constexpr (ND > 2) {
    const int z0 = t / (gx * gy) * chunk, z1 = z0 + chunk < G.n[2] ? z0 + chunk : G.n[2];
    mg_rb_march<NS, CA, M, ROB>(G, u, f, a, a2, out, sm, c, h, y, z0, z1);
  } else {
#pragma unroll
    for (int m = 0; m < 2; m++)
      if (c[m].on) sm[c[m].o] = mg_rb_at(u, c[m].og);
    __syncthreads();
    mg_rb_tile<NS, CA, M, ROB>(G, f, a, a2, out, sm, c, h, y);
  }
}

// ---- Residual passes ---------------------------------------------------------
// The residual f - L(u) of a 2D or 3D level reduced to its maximum (OP 0: one
// per workgroup, at part) or restricted (OP 1: volume-weighted means of u and of
// the residual over the 2^ndim children, to uc and rc).  A wavefront holds
// 32 x 2 cells, so the children of a coarse cell meet by two lane exchanges;
// a workgroup's four cover 32 x 8 and march along z, the column's two
// neighbours along z staying in registers.  What depends on (x, y) alone
// (offsets, weights, the faces folded into a factor of u as in k_mg_rb) is set
// up once per column.  Bound by memory: 256^3 cells with a (u + c) take
// 103 us for the norm and 112 us for the restriction (24 B per cell
// read); one thread per cell with the general operator took 167 us, one thread
// per coarse cell (eight children in turn) 190 us.
template <int ND, bool CA, int M, bool ROB, int OP>
__global__ __launch_bounds__(NT) void k_mg_res(const MgGeo G, const double *__restrict__ u,
                                               const double *__restrict__ f, const double *__restrict__ a,
                                               const double *__restrict__ a2, const MgGeo C, double *__restrict__ uc,
                                               double *__restrict__ rc, double *part, int zlen, int tiles) {
  const int n0 = G.n[0], n1 = G.n[1], n2 = ND > 2 ? G.n[2] : 1, lane = threadIdx.x & 63;
  const int gx = (n0 + 31) / 32, gy = (n1 + 7) / 8;
  const bool px = G.bc[0][0] == GMUNU_MG_PERIODIC, py = G.bc[1][0] == GMUNU_MG_PERIODIC,
             pz = ND > 2 && G.bc[2][0] == GMUNU_MG_PERIODIC;
  double mx = 0.0;
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int x = t % gx * 32 + (lane & 31), y = t / gx % gy * 8 + (int)(threadIdx.x >> 6) * 2 + (lane >> 5);
    const int z0 = t / (gx * gy) * zlen, z1 = z0 + zlen < n2 ? z0 + zlen : n2;
    const bool in = x < n0 && y < n1;
    const int i = x < n0 ? x : n0 - 1, j = y < n1 ? y : n1 - 1, I = i + 1, J = j + 1;
    const bool f0 = i == 0, f1 = i == n0 - 1, f2 = j == 0, f3 = j == n1 - 1;
    const int s1 = (int)G.s1;
    const long o = (long)(j + 1) * s1 + i + 1;
    const int xm = f0 ? (px ? n0 - 1 : 0) : -1, xp = f1 ? (px ? 1 - n0 : 0) : 1;
    const int ym = f2 ? (py ? (n1 - 1) * s1 : 0) : -s1, yp = f3 ? (py ? (1 - n1) * s1 : 0) : s1;
    const double wm0 = CA ? G.vih2[0] : G.a0m[I], wp0 = CA ? G.vih2[0] : G.a0p[I];
    const double wm1 = CA ? G.vih2[1] : G.g1[I] * G.a1m[J], wp1 = CA ? G.vih2[1] : G.g1[I] * G.a1p[J];
    const double w2 = ND < 3 ? 0.0 : CA ? G.vih2[2] : G.g2[I] * G.s2t[J] * G.ih2_2;
    const double vol = CA ? 1.0 : G.vol0[I] * G.vol1[J];
    const double cxy = (f0 && !px ? wm0 * mg_fold1(G, 0, 0) : 0.0) + (f1 && !px ? wp0 * mg_fold1(G, 0, 1) : 0.0) +
                       (f2 && !py ? wm1 * mg_fold1(G, 1, 0) : 0.0) + (f3 && !py ? wp1 * mg_fold1(G, 1, 1) : 0.0);
    const double xc = G.x0[0] + (i + 0.5) * G.h[0], yc = G.x0[1] + (j + 0.5) * G.h[1];
    const long g2 = ND > 2 ? 1 : 0;
    double um = 0.0, ucen = u[o + (z0 + g2) * G.s2], up = 0.0, su = 0.0, sr = 0.0;
    if (ND > 2) um = z0 > 0 ? u[o + z0 * G.s2] : pz ? u[o + n2 * G.s2] : ucen;
    for (int z = z0; z < z1; z++) {
      const long oz = o + (z + g2) * G.s2;
      const bool zlo = ND > 2 && !pz && z == 0, zhi = ND > 2 && !pz && z == n2 - 1;
      if (ND > 2) up = z < n2 - 1 ? u[oz + G.s2] : pz ? u[o + G.s2] : ucen;
      const double vxm = u[oz + xm], vxp = u[oz + xp], vym = u[oz + ym], vyp = u[oz + yp];
      const double fv = f[oz], av = M > 0 && a ? a[oz] : 0.0, a2v = M == 2 && a2 ? a2[oz] : 0.0;
      double lap = wp0 * (vxp - ucen) - wm0 * (ucen - vxm);
      lap += wp1 * (vyp - ucen) - wm1 * (ucen - vym);
      double cc = cxy;
      if (ND > 2) {
        lap += w2 * (up - ucen) - w2 * (ucen - um);
        if (zlo) cc += w2 * mg_fold1(G, 2, 0);
        if (zhi) cc += w2 * mg_fold1(G, 2, 1);
      }
      if (ROB) {
        double rr = xc * xc + yc * yc, zc = 0.0;
        if (ND > 2 && G.coord == GMUNU_CART) {
          zc = G.x0[2] + (z + 0.5) * G.h[2];
          rr += zc * zc;
        }
        if (f0 && !px && mg_robin(G, 0, 0)) cc += wm0 * mg_robin1(rr, xc, xc - G.h[0]);
        if (f1 && !px && mg_robin(G, 0, 1)) cc += wp0 * mg_robin1(rr, xc, xc + G.h[0]);
        if (f2 && !py && mg_robin(G, 1, 0)) cc += wm1 * mg_robin1(rr, yc, yc - G.h[1]);
        if (f3 && !py && mg_robin(G, 1, 1)) cc += wp1 * mg_robin1(rr, yc, yc + G.h[1]);
        if (zlo && mg_robin(G, 2, 0)) cc += w2 * mg_robin1(rr, zc, zc - G.h[2]);
        if (zhi && mg_robin(G, 2, 1)) cc += w2 * mg_robin1(rr, zc, zc + G.h[2]);
      }
      lap += cc * ucen;
      if (M == 2) {
        double du;
        lap -= mg_nl_both(G.power, G.power2, G.offset, av, a2v, ucen, du);
      } else if (M == 1) {
        lap -= av * (ucen + G.offset);
      }
      const double r = fv - lap;
      if (OP == 0) {
        if (in) mx = mg_absmax(mx, r);
      } else {
        su += vol * ucen;
        sr += vol * r;
        if (ND < 3 || (z & 1)) {
          double w = vol;
          su += __shfl_xor(su, 1, 64);
          sr += __shfl_xor(sr, 1, 64);
          su += __shfl_xor(su, 32, 64);
          sr += __shfl_xor(sr, 32, 64);
          if (!CA) {
            w += __shfl_xor(w, 1, 64);
            w += __shfl_xor(w, 32, 64);
          }
          const double iw = CA ? 1.0 / (1 << ND) : 1.0 / (ND > 2 ? 2.0 * w : w);
          if (in && !(x & 1) && !(y & 1)) {
            const long oc = mg_off(C, x >> 1, y >> 1, z >> 1);
            uc[oc] = su * iw;
            rc[oc] = sr * iw;
          }
          su = sr = 0.0;
        }
      }
      um = ucen;
      ucen = up;
    }
  }
  if (OP == 0) {
    mx = block_max(mx);
    if (threadIdx.x == 0) part[blockIdx.x] = mx;
  }
}

// Kwak prolongation of v (coarse, ghosts set) into the fine interior:
// fine = P v (add = 0) or fine += P v (add = 1).
__global__ __launch_bounds__(NT) void k_mg_prolong(const MgGeo C, const MgGeo F, const double *__restrict__ v,
                                                   double *__restrict__ fine, int add) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(F)) return;
  int fc[3];
  mg_cell(F, t, fc[0], fc[1], fc[2]);
  int cc[3];
#pragma unroll
  for (int a = 0; a < 3; a++) cc[a] = a < F.ndim ? fc[a] >> 1 : fc[a];
  const double w0 = F.ndim == 1 ? 0.75 : F.ndim == 2 ? 0.5 : 0.25;
  const long oc = mg_off(C, cc[0], cc[1], cc[2]);
  double s = w0 * v[oc];
  s += 0.25 * v[oc + ((fc[0] & 1) ? 1 : -1)];
  if (F.ndim > 1) s += 0.25 * v[oc + ((fc[1] & 1) ? C.s1 : -C.s1)];
  if (F.ndim > 2) s += 0.25 * v[oc + ((fc[2] & 1) ? C.s2 : -C.s2)];
  const long of = mg_off(F, fc[0], fc[1], fc[2]);
  fine[of] = add ? fine[of] + s : s;
}

// (1/sqrt g) d_i (sqrt g q^i), centred.
__global__ __launch_bounds__(NT) void k_mg_div(const MgGeo G, const double *__restrict__ q, double *__restrict__ out) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const int I = i + G.g[0], J = j + G.g[1];
  const long o = mg_off(G, i, j, k);
  const double sgc = G.sg0[I] * G.sg1[J];
  double s = (G.sg0[I + 1] * q[o + 1] - G.sg0[I - 1] * q[o - 1]) * G.sg1[J] / (2.0 * G.h[0]);
  if (G.ndim > 1)
    s += (G.sg1[J + 1] * q[G.nt + o + G.s1] - G.sg1[J - 1] * q[G.nt + o - G.s1]) * G.sg0[I] / (2.0 * G.h[1]);
  if (G.ndim > 2) s += (q[2 * G.nt + o + G.s2] - q[2 * G.nt + o - G.s2]) * sgc / (2.0 * G.h[2]);
  out[o] = s / sgc;
}

// q^i -= g^ii d_i phi, centred, on the interior.
__global__ __launch_bounds__(NT) void k_mg_subgrad(const MgGeo G, const double *__restrict__ phi,
                                                   double *__restrict__ q) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const int I = i + G.g[0], J = j + G.g[1];
  const long o = mg_off(G, i, j, k);
  q[o] -= (phi[o + 1] - phi[o - 1]) / (2.0 * G.h[0]);
  if (G.ndim > 1) q[G.nt + o] -= G.g1[I] * (phi[o + G.s1] - phi[o - G.s1]) / (2.0 * G.h[1]);
  if (G.ndim > 2) q[2 * G.nt + o] -= G.g2[I] * G.s2t[J] * (phi[o + G.s2] - phi[o - G.s2]) / (2.0 * G.h[2]);
}

// ------------------------------------------- vector equations of xCFC
//
// L(X)^i = Lap X^i + (1/3) d_i d_j X^j on Cartesian grids (section 2.6),
// second differences and the four-point mixed difference of section 2.7.
// The mixed stencil couples diagonal neighbours, so the Newton-Gauss-Seidel
// smoother visits 2^ndim colours (i mod 2, j mod 2, k mod 2), one launch
// each; cells of one colour are never neighbours, and the three components
// of a cell do not enter each other's diagonal, so a colour updates all its
// cells and components at once.  Across the boundary every axis applies its
// own rule (mirror times -1 or +1, periodic wrap): a step from a cell along
// an axis is an offset and a sign, and a diagonal neighbour takes the
// product of the two steps' signs.

__device__ __forceinline__ double mgv_flip(double v, unsigned bit) {
  return __hiloint2double(__double2hiint(v) ^ (int)(bit << 31), __double2loint(v));
}

struct VStep {
  int dm[3], dp[3];  // offsets of the minus / plus neighbour along each axis
  unsigned neg;      // bit 6 q + a: the minus step negates component q; 6 q + 3 + a: the plus step
};

__device__ __forceinline__ void mgv_axis(const MgGeo &G, int c, int a, int S, bool up, int &d, unsigned &neg) {
  const int n = G.n[a];
  if (up ? c < n - 1 : c > 0) {
    d = up ? S : -S;
    return;
  }
  if (G.bc[a][up ? 1 : 0] == GMUNU_MG_PERIODIC) {
    d = up ? -(n - 1) * S : (n - 1) * S;
    return;
  }
  d = 0;
  const unsigned odd = G.vodd[a][up ? 1 : 0];
#pragma unroll
  for (int q = 0; q < 3; q++)
    if ((odd >> q) & 1) neg |= 1u << (6 * q + (up ? 3 : 0) + a);
}

__device__ __forceinline__ VStep mgv_steps(const MgGeo &G, int i, int j, int k) {
  VStep s;
  s.neg = 0;
  const int c[3] = {i, j, k};
  const int S[3] = {1, (int)G.s1, (int)G.s2};
#pragma unroll
  for (int a = 0; a < 3; a++) {
    s.dm[a] = s.dp[a] = 0;
    if (a >= G.ndim) continue;
    mgv_axis(G, c[a], a, S[a], false, s.dm[a], s.neg);
    mgv_axis(G, c[a], a, S[a], true, s.dp[a], s.neg);
  }
  return s;
}

__device__ __forceinline__ double mgv_sgn(unsigned neg, int bits, double v) { return (neg >> bits) & 1 ? -v : v; }

// Component b at the diagonal neighbour (sq along axis qa, sb along axis
// ab; +1 or -1): the sign is the product of its two steps' signs.
__device__ __forceinline__ double mgv_corner(const double *__restrict__ ub, const VStep &s, long o, int b, int qa,
                                             int sq, int ab, int sb) {
  const unsigned n1 = s.neg >> (6 * b + (sq > 0 ? 3 : 0) + qa), n2 = s.neg >> (6 * b + (sb > 0 ? 3 : 0) + ab);
  return mgv_sgn(n1 ^ n2, 0, ub[o + (sq > 0 ? s.dp[qa] : s.dm[qa]) + (sb > 0 ? s.dp[ab] : s.dm[ab])]);
}

// L(X) at interior cell (i, j) (offset o) on a Cartesian level, all three
// components, and the inverse diagonals (level constants: 1/h_a^2,
// 1/(4 h_a h_b) and the inverse diagonals are precomputed in MgGeo).
__device__ __forceinline__ void mgv_L_cart(const MgGeo &G, const double *__restrict__ u, const VStep &s, long o,
                                           double L[3], double idg[3]) {
  const long nt = G.nt;
#pragma unroll
  for (int q = 0; q < 3; q++) {
    const double *uq = u + q * nt;
    const double u0 = uq[o];
    double lap = 0.0, self = 0.0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
      if (a >= G.ndim) continue;
      const double up = mgv_sgn(s.neg, 6 * q + 3 + a, uq[o + s.dp[a]]);
      const double um = mgv_sgn(s.neg, 6 * q + a, uq[o + s.dm[a]]);
      const double d2 = (up - 2.0 * u0 + um) * G.vih2[a];
      lap += d2;
      if (a == q) self = d2;
    }
    double gd = self;
#pragma unroll
    for (int b = 0; b < 3; b++) {
      if (q >= G.ndim || b == q || b >= G.ndim) continue;
      const double *ub = u + b * nt;
      const double pp = mgv_corner(ub, s, o, b, q, 1, b, 1), pm = mgv_corner(ub, s, o, b, q, 1, b, -1);
      const double mp = mgv_corner(ub, s, o, b, q, -1, b, 1), mm = mgv_corner(ub, s, o, b, q, -1, b, -1);
      gd += (pp - pm - mp + mm) * G.vmix[q + b - 1];
    }
    L[q] = lap + gd * (1.0 / 3.0);
    idg[q] = G.vidg[q];
  }
}

// The same on an axisymmetric cylindrical (R, z) or spherical (r, theta)
// level in orthonormal components: the flux-form Laplacian of each
// component (the scalar operator's tables), the connection terms of the
// vector Laplacian and of grad div, mixed differences by the four-point
// formula with signed corner coordinates; diagonals per cell.
__device__ __forceinline__ void mgv_L_curv(const MgGeo &G, const double *__restrict__ u, const VStep &s, long o,
                                           int i, int j, double L[3], double idg[3]) {
  const long nt = G.nt;
  const bool two = G.ndim > 1;
  const int I = i + G.g[0], J = j + G.g[1];
  const double h0 = G.h[0], h1 = G.h[1];
  const double r = G.x0[0] + (i + 0.5) * h0, ir2 = 1.0 / (r * r);
  const double wm0 = G.a0m[I], wp0 = G.a0p[I];
  const double wm1 = two ? G.g1[I] * G.a1m[J] : 0.0, wp1 = two ? G.g1[I] * G.a1p[J] : 0.0;
  const double i4h = two ? 1.0 / (4.0 * h0 * h1) : 0.0;
  double l0[3], l1[3], u0[3];
#pragma unroll
  for (int q = 0; q < 3; q++) {
    const double *uq = u + q * nt;
    u0[q] = uq[o];
    l0[q] = wp0 * (mgv_sgn(s.neg, 6 * q + 3, uq[o + s.dp[0]]) - u0[q]) -
            wm0 * (u0[q] - mgv_sgn(s.neg, 6 * q, uq[o + s.dm[0]]));
    l1[q] = two ? wp1 * (mgv_sgn(s.neg, 6 * q + 4, uq[o + s.dp[1]]) - u0[q]) -
                      wm1 * (u0[q] - mgv_sgn(s.neg, 6 * q + 1, uq[o + s.dm[1]]))
                : 0.0;
  }
  const double dl0 = -(wm0 + wp0), dl1 = -(wm1 + wp1), dlap = dl0 + dl1;
  const double *u0p = u, *u1p = u + nt;
  if (G.coord == GMUNU_CYL) {
    double mixz = 0.0, mixR = 0.0;
    if (two) {
#pragma unroll
      for (int di = -1; di <= 1; di += 2)
#pragma unroll
        for (int dj = -1; dj <= 1; dj += 2) {
          mixz += di * dj * mgv_corner(u1p, s, o, 1, 0, di, 1, dj);
          mixR += di * dj * (r + di * h0) * mgv_corner(u0p, s, o, 0, 0, di, 1, dj);
        }
      mixz *= i4h;
      mixR *= i4h / r;
    }
    L[0] = l0[0] + l1[0] - u0[0] * ir2 + (l0[0] - u0[0] * ir2 + mixz) * (1.0 / 3.0);
    idg[0] = 1.0 / (dlap - ir2 + (dl0 - ir2) * (1.0 / 3.0));
    L[1] = l0[1] + l1[1] + (mixR + l1[1]) * (1.0 / 3.0);
    idg[1] = 1.0 / (dlap + dl1 * (1.0 / 3.0));
    L[2] = l0[2] + l1[2] - u0[2] * ir2;
    idg[2] = 1.0 / (dlap - ir2);
  } else {
    const double sn = G.sg1[J], is2 = 1.0 / (sn * sn);
    double dth = 0.0, dr = 0.0, mixt = 0.0, mixr = 0.0;
    if (two) {
      dth = (G.sg1[J + 1] * mgv_sgn(s.neg, 6 + 4, u1p[o + s.dp[1]]) -
             G.sg1[J - 1] * mgv_sgn(s.neg, 6 + 1, u1p[o + s.dm[1]])) /
            (2.0 * h1);
      dr = (mgv_sgn(s.neg, 4, u0p[o + s.dp[1]]) - mgv_sgn(s.neg, 1, u0p[o + s.dm[1]])) / (2.0 * h1);
#pragma unroll
      for (int di = -1; di <= 1; di += 2)
#pragma unroll
        for (int dj = -1; dj <= 1; dj += 2) {
          const double rc = r + di * h0;
          mixt += di * dj * G.sg1[J + dj] * mgv_corner(u1p, s, o, 1, 0, di, 1, dj);
          mixr += di * dj * (rc * rc) * mgv_corner(u0p, s, o, 0, 0, di, 1, dj);
        }
      // (1/sin) d_r d_th (sin A_th / r) without dividing by a corner radius
      mixt = (mixt * i4h / r - dth * ir2) / sn;
      mixr *= i4h * ir2 / r;
    }
    L[0] = l0[0] + l1[0] - 2.0 * u0[0] * ir2 - 2.0 * ir2 / sn * dth +
           (l0[0] - 2.0 * u0[0] * ir2 + mixt) * (1.0 / 3.0);
    idg[0] = 1.0 / (dlap - 2.0 * ir2 + (dl0 - 2.0 * ir2) * (1.0 / 3.0));
    L[1] = l0[1] + l1[1] - u0[1] * ir2 * is2 + 2.0 * ir2 * dr + (mixr + l1[1] - u0[1] * ir2 * is2) * (1.0 / 3.0);
    idg[1] = 1.0 / (dlap - ir2 * is2 + (dl1 - ir2 * is2) * (1.0 / 3.0));
    L[2] = l0[2] + l1[2] - u0[2] * ir2 * is2;
    idg[2] = 1.0 / (dlap - ir2 * is2);
  }
}

__device__ __forceinline__ void mgv_L(const MgGeo &G, const double *__restrict__ u, long o, int i, int j, int k,
                                      double L[3], double idg[3]) {
  const VStep s = mgv_steps(G, i, j, k);
  if (G.coord == GMUNU_CART)
    mgv_L_cart(G, u, s, o, L, idg);
  else
    mgv_L_curv(G, u, s, o, i, j, L, idg);
}

// Cells of colour `colour` (bit a: parity along axis a) on a level.
__device__ __forceinline__ long mgv_colour_cells(const MgGeo &G, int colour) {
  long n = 1;
#pragma unroll
  for (int a = 0; a < 3; a++) n *= a < G.ndim ? (G.n[a] - ((colour >> a) & 1) + 1) >> 1 : G.n[a];
  return n;
}

__device__ __forceinline__ void mgv_smooth_one(const MgGeo &G, double *u, const double *__restrict__ f, int colour,
                                               long t) {
  const int ci = colour & 1, cj = (colour >> 1) & 1, ck = (colour >> 2) & 1;
  const unsigned hx = (unsigned)(G.n[0] - ci + 1) >> 1;
  const unsigned hy = G.ndim > 1 ? (unsigned)(G.n[1] - cj + 1) >> 1 : 1u;
  const unsigned hz = G.ndim > 2 ? (unsigned)(G.n[2] - ck + 1) >> 1 : 1u;
  if (t >= (long)hx * hy * hz) return;
  const unsigned tt = (unsigned)t, r = tt / hx;
  const int i = 2 * (int)(tt - r * hx) + ci;
  const unsigned kk = r / hy;
  const int j = G.ndim > 1 ? 2 * (int)(r - kk * hy) + cj : 0;
  const int k = G.ndim > 2 ? 2 * (int)kk + ck : 0;
  const long o = mg_off(G, i, j, k);
  double L[3], idg[3];
  mgv_L(G, u, o, i, j, k, L, idg);
#pragma unroll
  for (int q = 0; q < 3; q++) u[q * G.nt + o] -= (L[q] - f[q * G.nt + o]) * idg[q];
}

__global__ __launch_bounds__(NT) void k_mgv_smooth(const MgGeo G, double *u, const double *__restrict__ f,
                                                   int colour) {
  mgv_smooth_one(G, u, f, colour, (long)blockIdx.x * NT + threadIdx.x);
}

// Two consecutive colours in one launch: (i even, j, k parities of `pair`)
// then (i odd, same j, k parities).  Within such a pair a cell depends only
// on its x-neighbours in the same row (the other rows it reads have other
// j or k parities), so a workgroup owns whole rows (rpw of them) and
// separates the halves by a barrier.  Same order and arithmetic as two
// single-colour launches.
__global__ __launch_bounds__(NT) void k_mgv_smooth2(const MgGeo G, double *u, const double *__restrict__ f,
                                                    int pair, int rpw) {
  const int cj = pair & 1, ck = (pair >> 1) & 1;
  const unsigned hy = G.ndim > 1 ? (unsigned)(G.n[1] - cj + 1) >> 1 : 1u;
  const unsigned hz = G.ndim > 2 ? (unsigned)(G.n[2] - ck + 1) >> 1 : 1u;
  const unsigned rows = hy * hz, row0 = blockIdx.x * (unsigned)rpw;
  for (int ci = 0; ci < 2; ci++) {
    const unsigned hx = (unsigned)(G.n[0] - ci + 1) >> 1;
    for (unsigned idx = threadIdx.x; idx < (unsigned)rpw * hx; idx += NT) {
      const unsigned rr = idx / hx, row = row0 + rr;
      if (row >= rows) break;
      const int i = 2 * (int)(idx - rr * hx) + ci;
      const unsigned kk = row / hy;
      const int j = G.ndim > 1 ? 2 * (int)(row - kk * hy) + cj : 0;
      const int k = G.ndim > 2 ? 2 * (int)kk + ck : 0;
      const long o = mg_off(G, i, j, k);
      double L[3], idg[3];
      mgv_L(G, u, o, i, j, k, L, idg);
#pragma unroll
      for (int q = 0; q < 3; q++) u[q * G.nt + o] -= (L[q] - f[q * G.nt + o]) * idg[q];
    }
    __syncthreads();
  }
}

// The colours of one parity of k (in 2D all colours) on a Cartesian level, out
// of place: cells of planes k = kpar, kpar + 2, ... of out from planes k - 1
// and k + 1 of nb and plane k of u (out may not be u).  Two launches (nb = u, then nb = out) are
// one sweep.  A workgroup stages the three planes of a TX x TY tile and its
// halo in LDS, relaxes the four colours of plane k there and writes the
// tile.  The colours reach beyond the tile: colour (1, 1) at its upper edge
// needs (0, 1) at x = TX, which needs (1, 0) at TX + 1 and that (0, 0) at
// TX + 2 (and two cells below x = 0, one row above the tile), so those are
// relaxed redundantly, one 2 x 2 quad of cells per thread and component.  In LDS a row holds
// its even cells, then its odd ones: a colour's reads are contiguous.
// Against a launch per colour pair, which reads the whole field, this halves
// the launches and reads each plane from memory about once per parity.  Bound
// by the staged bytes (1.5 times the tile for its halo) on large levels and
// by one workgroup's chain of load, four colours and store on small ones:
// 51 us per launch at 128^3 (3.4 TB/s of staged, f and written bytes, 2.0 of
// those needed) and 7.5 us from 16^3 to 32^3 cells, against 30 and 7 us for each
// of the twice as many launches of a colour pair (one thread per quad and all
// components: 64 and 13 us).
constexpr int kPlX = 32, kPlY = 16;           // tile
constexpr int kPlRow = kPlX + 8, kPlRows = kPlY + 3;  // staged: x -3 .. TX + 3 (row of 40), y -1 .. TY + 1
constexpr int kPlQx = kPlX / 2 + 3, kPlQy = kPlY / 2 + 1;
constexpr int kPlCS = kPlRows * kPlRow;  // staged cells of a plane
constexpr int kPlQuads = 192;  // threads of one component
static_assert(kPlQx * kPlQy <= kPlQuads && kPlQuads % 64 == 0, "one quad per thread, whole wavefronts");

// Place of tile coordinate x (>= -4) in a staged row.
__device__ __forceinline__ constexpr int pl_x(int x) { return ((x + 4) & 1) * (kPlRow / 2) + ((x + 4) >> 1); }

// Component Q of the cell of colour (CI, CJ) whose centre in LDS is o (plane k,
// component 0): steps to its neighbours (EDGE: 0 across a face, with the
// flips of the components odd there) and L(X)^Q; u0: the component's value.
template <int ND, int CI, int CJ, bool EDGE, int Q>
__device__ __forceinline__ double mgv_plane_L(const MgGeo &G, const double *sm, int o, int zm, int zp, unsigned fzm,
                                              unsigned fzp, int gi, int gj, double &u0) {
  constexpr int XM = CI ? -(kPlRow / 2) : kPlRow / 2 - 1, XP = CI ? 1 - kPlRow / 2 : kPlRow / 2;
  int dm[3] = {XM, -kPlRow, zm}, dp[3] = {XP, kPlRow, zp};
  unsigned fm[3] = {0u, 0u, fzm}, fp[3] = {0u, 0u, fzp};
  if constexpr (EDGE) {
    const bool px = G.bc[0][0] == GMUNU_MG_PERIODIC, py = G.bc[1][0] == GMUNU_MG_PERIODIC;
    if (!px && gi == 0) dm[0] = 0, fm[0] = G.vodd[0][0];
    if (!px && gi == G.n[0] - 1) dp[0] = 0, fp[0] = G.vodd[0][1];
    if (!py && gj == 0) dm[1] = 0, fm[1] = G.vodd[1][0];
    if (!py && gj == G.n[1] - 1) dp[1] = 0, fp[1] = G.vodd[1][1];
  }
  auto at = [&](int c, int d, unsigned flip) -> double {
    const double v = sm[o + c * (3 * kPlCS) + d];
    return EDGE ? mgv_flip(v, flip >> c & 1u) : v;
  };
  u0 = sm[o + Q * (3 * kPlCS)];
  double lap = 0.0, gd = 0.0;
#pragma unroll
  for (int a = 0; a < ND; a++) {
    const double d2 = (at(Q, dp[a], fp[a]) - 2.0 * u0 + at(Q, dm[a], fm[a])) * G.vih2[a];
    lap += d2;
    if (a == Q) gd = d2;
  }
#pragma unroll
  for (int b = 0; b < ND; b++) {
    if (Q >= ND || b == Q) continue;
    const double pp = at(b, dp[Q] + dp[b], fp[Q] ^ fp[b]), pm = at(b, dp[Q] + dm[b], fp[Q] ^ fm[b]);
    const double mp = at(b, dm[Q] + dp[b], fm[Q] ^ fp[b]), mm = at(b, dm[Q] + dm[b], fm[Q] ^ fm[b]);
    gd += (pp - pm - mp + mm) * G.vmix[Q + b - 1];
  }
  return lap + gd * (1.0 / 3.0);
}

// The four colours, component Q.  The components of one cell are relaxed by
// three wavefronts; at a corner of the domain one reads the others of its
// own cell, so there (EDGE) a barrier separates the reads from the writes.
template <int ND, bool EDGE, int Q>
__device__ __forceinline__ void mgv_plane_colours(const MgGeo &G, double *sm, int i0, int j0, const bool *on,
                                                  const double *fv, int zm, int zp, unsigned fzm, unsigned fzp) {
  const int tq = threadIdx.x % kPlQuads, hx = tq % kPlQx, hy = tq / kPlQx, gi = i0 + 2 * hx - 2, gj = j0 + 2 * hy;
  const int o = kPlCS + (2 * hy + 1) * kPlRow + pl_x(0) + hx - 1;  // even cell of the quad's lower row, plane k
  double u0, L;
#define GM_PL(C)                                                                                                   \
  {                                                                                                                \
    const int oc = o + (C & 1) * (kPlRow / 2) + (C >> 1) * kPlRow;                                                 \
    if (on[C])                                                                                                     \
      L = mgv_plane_L<ND, C & 1, (C >> 1), EDGE, Q>(G, sm, oc, zm, zp, fzm, fzp, gi + (C & 1), gj + (C >> 1), u0); \
    if (EDGE) __syncthreads();                                                                                     \
    if (on[C]) sm[oc + Q * (3 * kPlCS)] = u0 - (L - fv[C]) * G.vidg[Q];                                            \
    __syncthreads();                                                                                               \
  }
  GM_PL(0)
  GM_PL(1)
  GM_PL(2)
  GM_PL(3)
#undef GM_PL
}

template <int ND, int Q>
__device__ __forceinline__ void mgv_plane_tile(const MgGeo &G, const double *u, const double *nb,
                                               const double *__restrict__ f, double *out, int i0, int j0, int k,
                                               double *sm) {
  const int n0 = G.n[0], n1 = G.n[1], n2 = G.n[2], tq = threadIdx.x % kPlQuads;
  const bool px = G.bc[0][0] == GMUNU_MG_PERIODIC, py = G.bc[1][0] == GMUNU_MG_PERIODIC,
             pz = ND > 2 && G.bc[2][0] == GMUNU_MG_PERIODIC;
  const bool lz = ND > 2 && !pz && k == 0, hz = ND > 2 && !pz && k == n2 - 1;
  const long q0 = Q * G.nt;
  const double *uk = u + q0 + k * G.s2, *um = nb + q0 + (k == 0 ? n2 - 1 : k - 1) * G.s2,
               *up = nb + q0 + (k == n2 - 1 ? 0 : k + 1) * G.s2;
  // every load of the tile before the first LDS write: one memory latency
  constexpr int NIT = (kPlCS + kPlQuads - 1) / kPlQuads;
  double v[NIT][3];
  bool in[NIT];
#pragma unroll
  for (int m = 0; m < NIT; m++) {
    const int e = tq + m * kPlQuads, r = e / kPlRow, xx = e % kPlRow;
    const int x = xx < kPlRow / 2 ? 2 * xx - 4 : 2 * (xx - kPlRow / 2) - 3;
    int i = i0 + x, j = j0 + r - 1;
    if (px) i = i < 0 ? i + (-i + n0 - 1) / n0 * n0 : i >= n0 ? i % n0 : i;
    if (py) j = j < 0 ? j + n1 : j >= n1 ? j % n1 : j;
    in[m] = e < kPlCS && i >= 0 && i < n0 && j >= 0 && j < n1 && x != -4;
    const long o = in[m] ? mg_off(G, i, j, 0) : 0;
    v[m][1] = in[m] ? uk[o] : 0.0;
    v[m][0] = in[m] && ND > 2 && !lz ? um[o] : 0.0;
    v[m][2] = in[m] && ND > 2 && !hz ? up[o] : 0.0;
  }
  // which cells of the thread's quad are relaxed, and their right-hand sides
  const int hx = tq % kPlQx, hy = tq / kPlQx, x = 2 * hx - 2, y = 2 * hy, gi = i0 + x, gj = j0 + y;
  bool on[4];
  double fv[4];
#pragma unroll
  for (int c = 0; c < 4; c++) {
    const int ci = c & 1, cj = c >> 1;
    int ii = gi + ci, jj = gj + cj;
    on[c] = hy < kPlQy && x + ci <= kPlX + 2 - c && (cj == 0 || (x + ci >= ci && hy < kPlQy - 1));
    on[c] = on[c] && (px || (ii >= 0 && ii < n0)) && (py || jj < n1);
    if (px) ii = ii < 0 ? ii + n0 : ii >= n0 ? ii % n0 : ii;
    if (py) jj = jj >= n1 ? jj % n1 : jj;
    fv[c] = on[c] ? f[q0 + mg_off(G, ii, jj, k)] : 0.0;
  }
#pragma unroll
  for (int m = 0; m < NIT; m++) {
    const int e = tq + m * kPlQuads;
    if (!in[m]) continue;
    double *d = sm + 3 * Q * kPlCS + e;
    d[kPlCS] = v[m][1];
    if (ND > 2) {
      d[0] = v[m][0];
      d[2 * kPlCS] = v[m][2];
    }
  }
  __syncthreads();
  const int zm = lz ? 0 : -kPlCS, zp = hz ? 0 : kPlCS;
  const unsigned fzm = lz ? G.vodd[2][0] : 0u, fzp = hz ? G.vodd[2][1] : 0u;
  const bool edge = (!px && (i0 == 0 || i0 + kPlX + 3 >= n0)) || (!py && (j0 == 0 || j0 + kPlY + 1 >= n1));
  if (edge || lz || hz)
    mgv_plane_colours<ND, true, Q>(G, sm, i0, j0, on, fv, zm, zp, fzm, fzp);
  else
    mgv_plane_colours<ND, false, Q>(G, sm, i0, j0, on, fv, zm, zp, fzm, fzp);
#pragma unroll
  for (int m = 0; m < (kPlX * kPlY + kPlQuads - 1) / kPlQuads; m++) {
    const int e = tq + m * kPlQuads, xe = e % kPlX, ye = e / kPlX;
    if (e < kPlX * kPlY && i0 + xe < n0 && j0 + ye < n1)
      out[q0 + mg_off(G, i0 + xe, j0 + ye, k)] = sm[(3 * Q + 1) * kPlCS + (ye + 1) * kPlRow + pl_x(xe)];
  }
}

template <int ND>
__global__ __launch_bounds__(3 * kPlQuads) void k_mgv_planes(const MgGeo G, const double *u, const double *nb,
                                                             const double *__restrict__ f, double *out, int kpar) {
  __shared__ double sm[9 * kPlCS];  // [component][plane k - 1, k, k + 1][row][x]
  // contiguous runs of tiles (x fastest, then y, then k) per XCD
  const int gx = (G.n[0] + kPlX - 1) / kPlX, gy = (G.n[1] + kPlY - 1) / kPlY;
  const int t = mg_xcd_run();
  const int i0 = (t % gx) * kPlX, j0 = (t / gx) % gy * kPlY, k = kpar + 2 * (t / (gx * gy));
  // one component per three wavefronts (the branch is uniform in each of them,
  // and its three sides pass the same barriers)
  const int q = threadIdx.x / kPlQuads;
  if (q == 0)
    mgv_plane_tile<ND, 0>(G, u, nb, f, out, i0, j0, k, sm);
  else if (q == 1)
    mgv_plane_tile<ND, 1>(G, u, nb, f, out, i0, j0, k, sm);
  else
    mgv_plane_tile<ND, 2>(G, u, nb, f, out, i0, j0, k, sm);
}

// ---- Tail of the hierarchy, vector equations (Cartesian) ----------------------
// As k_mg_tail, for levels of at most kVTailCells cells: one lane per cell and
// component, the components of a cell in one wavefront (at a corner of the
// domain a component's mixed difference reads the other components of the
// cell itself, so all must be read before one is written).  A colour is bound
// by the latency of its 15 LDS reads and their chain, 0.4 us on 8^3 cells
// against 5 us for the launch of a colour pair; above 1024 cells the LDS reads
// of one CU take longer than launches over many.

constexpr int kVTailCells = 1024;

struct MgvLev {
  int n[3], s2, cells;
  unsigned mn0, mn1;
  int u, f, uo;        // offsets of component 0 (component stride: cells)
  int per[3];
  unsigned odd[3][2];  // components odd across each non-periodic face
  double w[3], mix[3], idg[3];
};

struct MgvTail {
  MgvLev lev[kTailLevels];
  int ndim, top;
  int sweeps[3];
  int nprog[2];
  int prog[2][512];
};

// Component q of L(X) at cell (i, j, k) of a tail level.
__device__ __forceinline__ double mgv_tail_L(const MgvLev &V, const double *sm, int q, int i, int j, int k, int o) {
  const int x[3] = {i, j, k}, S[3] = {1, V.n[0], V.s2};
  int dm[3], dp[3];
  unsigned fm[3], fp[3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const int n = V.n[a], wrap = V.per[a] ? (n - 1) * S[a] : 0;
    const bool lo = x[a] == 0, hi = x[a] == n - 1;
    dm[a] = lo ? wrap : -S[a];
    dp[a] = hi ? -wrap : S[a];
    fm[a] = lo ? V.odd[a][0] : 0u;
    fp[a] = hi ? V.odd[a][1] : 0u;
  }
  const double *u = sm + V.u + o, *uq = u + q * V.cells;
  const double u0 = uq[0];
  double lap = 0.0, gd = 0.0;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const double up = mgv_flip(uq[dp[a]], fp[a] >> q & 1u), um = mgv_flip(uq[dm[a]], fm[a] >> q & 1u);
    const double d2 = (up - 2.0 * u0 + um) * V.w[a];
    lap += d2;
    if (a == q) gd = d2;
  }
  // mixed differences along q and each other axis b
  const int qm = q == 0 ? dm[0] : q == 1 ? dm[1] : dm[2], qp = q == 0 ? dp[0] : q == 1 ? dp[1] : dp[2];
  const unsigned gm = q == 0 ? fm[0] : q == 1 ? fm[1] : fm[2], gp = q == 0 ? fp[0] : q == 1 ? fp[1] : fp[2];
#pragma unroll
  for (int e = 0; e < 2; e++) {
    const bool first = e == 0 ? q == 0 : q == 2;  // the other axis is 1, else 0 (e = 0) or 2 (e = 1)
    const int b = first ? 1 : 2 * e;
    const int bm = first ? dm[1] : dm[2 * e], bp = first ? dp[1] : dp[2 * e];
    const unsigned hm = first ? fm[1] : fm[2 * e], hp = first ? fp[1] : fp[2 * e];
    const double *ub = u + b * V.cells;
    const double pp = mgv_flip(ub[qp + bp], (gp ^ hp) >> b & 1u), pm = mgv_flip(ub[qp + bm], (gp ^ hm) >> b & 1u);
    const double mp = mgv_flip(ub[qm + bp], (gm ^ hp) >> b & 1u), mm = mgv_flip(ub[qm + bm], (gm ^ hm) >> b & 1u);
    // pairs (0, 1), (0, 2), (1, 2): q + b - 1
    const double mix = e == 0 ? (q == 2 ? V.mix[1] : V.mix[0]) : (q == 0 ? V.mix[1] : V.mix[2]);
    gd += (pp - pm - mp + mm) * mix;
  }
  return lap + gd * (1.0 / 3.0);
}

__device__ __forceinline__ void mgv_tail_cell(const MgvLev &V, int t, int &i, int &j, int &k) {
  const int r = mg_div(t, V.mn0);
  i = t - r * V.n[0];
  k = mg_div(r, V.mn1);
  j = r - k * V.n[1];
}

__device__ __forceinline__ void mgv_tail_sweeps(const MgvTail &T, const MgvLev &Vg, double *sm, int sweeps) {
  const MgvLev V = Vg;  // in registers over the sweeps
  const int nd = T.ndim;
  // one lane per component of the 2^ndim cells that differ in their parities
  const int ln = threadIdx.x & 63, q = ln % 3, slot = (threadIdx.x >> 6) * 21 + ln / 3;
  const int hx = (V.n[0] + 1) >> 1, hy = (V.n[1] + 1) >> 1, hz = (V.n[2] + 1) >> 1;
  const int r = (int)((unsigned)slot / (unsigned)hx), kk = (int)((unsigned)r / (unsigned)hy);
  const int i0 = 2 * (slot - r * hx), j0 = 2 * (r - kk * hy), k0 = 2 * kk;
  const double idg = q == 0 ? V.idg[0] : q == 1 ? V.idg[1] : V.idg[2];
  const bool one_wave = hx * hy * hz <= 21, live = ln < 63 && kk < hz;
  if (!one_wave || threadIdx.x < 64) {
    for (int s = 0; s < sweeps; s++)
      for (int c = 0; c < 1 << nd; c++) {
        const int i = i0 + (c & 1), j = j0 + ((c >> 1) & 1), k = k0 + (c >> 2);
        if (live && i < V.n[0] && j < V.n[1] && k < V.n[2]) {
          const int o = i + V.n[0] * j + V.s2 * k;
          const double L = mgv_tail_L(V, sm, q, i, j, k, o);
          sm[V.u + q * V.cells + o] -= (L - sm[V.f + q * V.cells + o]) * idg;
        }
        if (one_wave)
          wave_fence();
        else
          __syncthreads();
      }
  }
  if (one_wave) __syncthreads();
}

__device__ __forceinline__ void mgv_tail_coarse_problem(const MgvTail &T, const MgvLev &F, const MgvLev &C,
                                                        double *sm) {
  const int nc = C.cells, nd = T.ndim;
  for (int t0 = 0; t0 < 3 * nc << nd; t0 += blockDim.x) {
    const int t = t0 + threadIdx.x, e = t >> nd;
    const int q = e >= 2 * nc ? 2 : e >= nc ? 1 : 0, oc = e - q * nc;
    double su = 0.0, sr = 0.0;
    if (e < 3 * nc) {
      int i, j, k;
      mgv_tail_cell(C, oc, i, j, k);
      i = 2 * i + (t & 1);
      if (nd > 1) j = 2 * j + ((t >> 1) & 1);
      if (nd > 2) k = 2 * k + ((t >> 2) & 1);
      const int o = i + F.n[0] * j + F.s2 * k;
      su = sm[F.u + q * F.cells + o];
      sr = sm[F.f + q * F.cells + o] - mgv_tail_L(F, sm, q, i, j, k, o);
    }
    su = mg_sum_children(su, nd);
    sr = mg_sum_children(sr, nd);
    if (e < 3 * nc && (t & ((1 << nd) - 1)) == 0) {
      const double iw = 1.0 / (1 << nd);
      sm[C.u + e] = sm[C.uo + e] = su * iw;
      sm[C.f + e] = sr * iw;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 3 * nc; e += blockDim.x) {
    const int q = e >= 2 * nc ? 2 : e >= nc ? 1 : 0;
    int i, j, k;
    mgv_tail_cell(C, e - q * nc, i, j, k);
    sm[C.f + e] += mgv_tail_L(C, sm, q, i, j, k, e - q * nc);
  }
  __syncthreads();
}

__device__ __forceinline__ void mgv_tail_correct(const MgvTail &T, const MgvLev &F, const MgvLev &C, double *sm) {
  const int nd = T.ndim;
  const double w0 = nd == 1 ? 0.75 : nd == 2 ? 0.5 : 0.25;
  const int S[3] = {1, C.n[0], C.s2};
  for (int e = threadIdx.x; e < 3 * F.cells; e += blockDim.x) {
    const int q = e >= 2 * F.cells ? 2 : e >= F.cells ? 1 : 0;
    int fc[3];
    mgv_tail_cell(F, e - q * F.cells, fc[0], fc[1], fc[2]);
    const int cc[3] = {fc[0] >> 1, nd > 1 ? fc[1] >> 1 : fc[1], nd > 2 ? fc[2] >> 1 : fc[2]};
    const int oc = cc[0] + S[1] * cc[1] + S[2] * cc[2] + q * C.cells;
    double s = w0 * (sm[C.u + oc] - sm[C.uo + oc]);
#pragma unroll
    for (int a = 0; a < 3; a++) {
      if (a >= nd) continue;
      const bool up = fc[a] & 1, inside = up ? cc[a] < C.n[a] - 1 : cc[a] > 0;
      const int step = inside ? S[a] : C.per[a] ? -(C.n[a] - 1) * S[a] : 0, on = up ? oc + step : oc - step;
      const unsigned odd = inside ? 0u : up ? C.odd[a][1] : C.odd[a][0];
      s += 0.25 * mgv_flip(sm[C.u + on] - sm[C.uo + on], odd >> q & 1u);
    }
    sm[F.u + e] += s;
  }
  __syncthreads();
}

template <bool OUT>
__device__ __forceinline__ void mgv_tail_copy(const MgvTail &T, const MgvLev &V, double *glob, double *lds) {
  const int g1 = T.ndim > 1 ? 1 : 0, g2 = T.ndim > 2 ? 1 : 0;
  const int S1 = V.n[0] + 2, S2 = S1 * (V.n[1] + 2 * g1), nt = S2 * (V.n[2] + 2 * g2);
  for (int e = threadIdx.x; e < 3 * V.cells; e += blockDim.x) {
    const int q = e >= 2 * V.cells ? 2 : e >= V.cells ? 1 : 0;
    int i, j, k;
    mgv_tail_cell(V, e - q * V.cells, i, j, k);
    const int o = q * nt + (k + g2) * S2 + (j + g1) * S1 + i + 1;
    if (OUT)
      glob[o] = lds[e];
    else
      lds[e] = glob[o];
  }
}

__global__ __launch_bounds__(kTailThreads) void k_mgv_tail(const MgvTail *__restrict__ Tt, double *u,
                                                           const double *__restrict__ f, int use_fmg) {
  __shared__ double sm[kVTailCells * 11 + 64];
  const MgvTail &T = *Tt;
  const MgvLev &P = T.lev[T.top];
  mgv_tail_copy<false>(T, P, u, sm + P.u);
  mgv_tail_copy<false>(T, P, const_cast<double *>(f), sm + P.f);
  __syncthreads();
  const int np = T.nprog[use_fmg];
  for (int pc = 0; pc < np; pc++) {
    const int op = T.prog[use_fmg][pc], l = (op >> 2) & 15;
    if ((op & 3) == kOpSweep)
      mgv_tail_sweeps(T, T.lev[l], sm, T.sweeps[op >> 6]);
    else if ((op & 3) == kOpCoarse)
      mgv_tail_coarse_problem(T, T.lev[l], T.lev[l - 1], sm);
    else
      mgv_tail_correct(T, T.lev[l], T.lev[l - 1], sm);
  }
  mgv_tail_copy<true>(T, P, u, sm + P.u);
}

// Coarsest level: all sweeps in one workgroup, colours separated by
// barriers; with lds != 0 on copies of X and f in dynamic LDS.
__global__ __launch_bounds__(NT) void k_mgv_coarse(const MgGeo G, double *u, const double *__restrict__ f,
                                                   int sweeps, int lds) {
  extern __shared__ double sm[];
  double *uu = u;
  const double *ff = f;
  const long n3 = 3 * G.nt;
  if (lds) {
    for (long e = threadIdx.x; e < n3; e += NT) {
      sm[e] = u[e];
      sm[n3 + e] = f[e];
    }
    __syncthreads();
    uu = sm;
    ff = sm + n3;
  }
  const int ncol = 1 << G.ndim;
  for (int s = 0; s < sweeps; s++)
    for (int c = 0; c < ncol; c++) {
      const long nc = mgv_colour_cells(G, c);
      for (long t = threadIdx.x; t < nc; t += NT) mgv_smooth_one(G, uu, ff, c, t);
      __syncthreads();
    }
  if (lds)
    for (long e = threadIdx.x; e < n3; e += NT) u[e] = uu[e];
}

// Row of component q's line system at cell cc: diagonal dg of the operator,
// residual r; over the diagonal with the boundary faces folded in.
__device__ __forceinline__ void mgv_line_row(const MgGeo &G, int ax, const int cc[3], int q, double dg, double r,
                                             double &wa, double &wc, double &d) {
  double wm, wp;
#pragma unroll
  for (int b = 0; b < 3; b++) {
    if (b >= G.ndim || G.bc[b][0] == GMUNU_MG_PERIODIC || (cc[b] > 0 && cc[b] < G.n[b] - 1)) continue;
    const double kb = b == q ? 4.0 / 3.0 : 1.0;
    mg_w(G, cc[0] + G.g[0], cc[1] + G.g[1], b, wm, wp);
    if (cc[b] == 0) dg += (G.vodd[b][0] >> q) & 1 ? -kb * wm : kb * wm;
    if (cc[b] == G.n[b] - 1) dg += (G.vodd[b][1] >> q) & 1 ? -kb * wp : kb * wp;
  }
  const double id = rcp(dg), ki = ax == q && q < G.ndim ? 4.0 / 3.0 * id : id;
  mg_w(G, cc[0] + G.g[0], cc[1] + G.g[1], ax, wm, wp);
  const int m = ax == 0 ? cc[0] : ax == 1 ? cc[1] : cc[2];
  wa = m == 0 ? 0.0 : wm * ki;
  wc = m == G.n[ax] - 1 ? 0.0 : wp * ki;
  d = r * id;
}

// Line relaxation of the vector equations, the line from cell c along
// axis ax by one wavefront (as mg_line_step): the components one after the
// other, each a Newton step of its own equation with its exact Jacobian
// with respect to that component on the line -- the couplings of the
// component's flux-form Laplacian, times 4/3 along the component's own
// axis through the grad-div term; on the diagonal the point smoother's
// plus, across each non-periodic boundary face, the weight toward the
// mirror ghost times the component's sign there -- and everything else
// (the other components included) at its current value.
__device__ __forceinline__ void mgv_line_step(const MgGeo &G, double *u, const double *__restrict__ f, int ax,
                                              const int c[3], bool live, double *sm, int m, bool one_wave) {
  const int n = G.n[ax];
  const bool on = live && m < n;
  const int cc[3] = {ax == 0 ? m : c[0], ax == 1 ? m : c[1], ax == 2 ? m : c[2]};
  const long o = on ? mg_off(G, cc[0], cc[1], cc[2]) : 0;
  for (int q = 0; q < 3; q++) {
    double wm = 0.0, wp = 0.0, d = 0.0;
    if (on) {
      double L[3], idg[3];
      mgv_L(G, u, o, cc[0], cc[1], cc[2], L, idg);
      mgv_line_row(G, ax, cc, q, rcp(idg[q]), f[q * G.nt + o] - L[q], wm, wp, d);
    }
    mg_pcr<1>(sm, n, m, on, one_wave, &wm, &wp, &d);
    if (on) u[q * G.nt + o] += d;
    mg_line_sync(one_wave);
  }
}

// The same on axisymmetric (2D cylindrical or spherical) levels.  There the
// third component enters no other's equation nor they its own, so that it is
// solved beside the first (PAIR; one after the other where the line's LDS
// would pass 64 KB: the results are the same), and a cell's operands (nine
// values of the first two components, five of the third) are loaded once and
// kept in registers: the second component's equation takes the first one's
// update, its neighbours' along the line from LDS.  A line otherwise waits
// three times for memory and computes all three operators per component:
// 320 lines of 64 cells 22.8 us, now 12.6; 32 lines of 640 cells 41.4 us,
// now 18.8.  sm: (PAIR ? 12 : 7) n doubles.
template <bool PAIR>
__device__ __forceinline__ void mgv_line_curv(const MgGeo &G, double *u, const double *__restrict__ f, int ax,
                                              const int c[3], bool live, double *sm, int m, bool one_wave) {
  constexpr int NS = PAIR ? 2 : 1;
  const int n = G.n[ax];
  const bool on = live && m < n;
  const int cc[3] = {ax == 0 ? m : c[0], ax == 0 ? c[1] : m, 0};
  const long nt = G.nt;
  double U0[3][3], U1[3][3], U2[3][3], fv[3] = {0.0, 0.0, 0.0};
  bool flip0[3][3];
  int along[3];           // step along the line of the neighbours m - 1, m, m + 1 (0 where the rule folds it)
  bool line[3];           // the transverse neighbour is on the line (the line itself, or folded onto it)
  VStep s;
  s.neg = 0;
  long o = 0;
  if (on) {
    o = mg_off(G, cc[0], cc[1], cc[2]);
    s = mgv_steps(G, cc[0], cc[1], 0);
  }
  const int d0[3] = {s.dm[0], 0, s.dp[0]}, d1[3] = {s.dm[1], 0, s.dp[1]};
#pragma unroll
  for (int e = 0; e < 3; e++) {
    const int da = ax == 0 ? d0[e] : d1[e], dt = ax == 0 ? d1[e] : d0[e];
    along[e] = da == 0 ? 0 : e - 1;
    line[e] = dt == 0;
  }
  if (on) {
#pragma unroll
    for (int x = 0; x < 3; x++)
#pragma unroll
      for (int y = 0; y < 3; y++) {
        const long at = o + d0[x] + d1[y];
        // signs of the two steps for components 0, 1, 2 (bit 6 q + a: minus, + 3: plus)
        const unsigned nx = x == 1 ? 0u : s.neg >> (x == 2 ? 3 : 0), ny = y == 1 ? 0u : s.neg >> (y == 2 ? 4 : 1);
        const unsigned neg = nx ^ ny;
        flip0[x][y] = neg & 1;
        U0[x][y] = mgv_flip(u[at], neg & 1);
        U1[x][y] = mgv_flip(u[nt + at], (neg >> 6) & 1);
        if (x == 1 || y == 1) U2[x][y] = mgv_flip(u[2 * nt + at], (neg >> 12) & 1);
      }
#pragma unroll
    for (int q = 0; q < 3; q++) fv[q] = f[q * nt + o];
  }
  const int I = cc[0] + G.g[0], J = cc[1] + G.g[1];
  const bool sph = G.coord == GMUNU_SPH;
  const double h0 = G.h[0], i2h1 = rcp(2.0 * G.h[1]), i4h = rcp(4.0 * h0 * G.h[1]);
  double w0m = 0.0, w0p = 0.0, w1m = 0.0, w1p = 0.0, sn = 1.0, sgm = 1.0, sgp = 1.0;
  if (on) {
    mg_w(G, I, J, 0, w0m, w0p);
    mg_w(G, I, J, 1, w1m, w1p);
    if (sph) {
      sn = G.sg1[J];
      sgm = G.sg1[J - 1];
      sgp = G.sg1[J + 1];
    }
  }
  const double r = G.x0[0] + (cc[0] + 0.5) * h0, ir = rcp(r), ir2 = ir * ir, rm = r - h0, rp = r + h0;
  const double is = sph ? rcp(sn) : 1.0, is2 = is * is;
  const double dl0 = -(w0m + w0p), dl1 = -(w1m + w1p), dlap = dl0 + dl1;
  double wa[NS], wc[NS], d[NS], xq[3];
  auto second = [&](const double (&U)[3][3], double &l0, double &l1) {
    l0 = w0p * (U[2][1] - U[1][1]) - w0m * (U[1][1] - U[0][1]);
    l1 = w1p * (U[1][2] - U[1][1]) - w1m * (U[1][1] - U[1][0]);
  };
  auto zero = [&](int k) { wa[k] = wc[k] = d[k] = 0.0; };
  auto row0 = [&](int k) {
    double l0, l1, L, dg;
    second(U0, l0, l1);
    const double u0 = U0[1][1];
    if (sph) {
      const double dth = (sgp * U1[1][2] - sgm * U1[1][0]) * i2h1;
      // (1/sin) d_r d_th (sin A_th / r) without dividing by a corner radius
      const double mix = ((sgp * (U1[2][2] - U1[0][2]) - sgm * (U1[2][0] - U1[0][0])) * (i4h * ir) - dth * ir2) * is;
      L = l0 + l1 - 2.0 * u0 * ir2 - 2.0 * ir2 * is * dth + (l0 - 2.0 * u0 * ir2 + mix) * (1.0 / 3.0);
      dg = dlap - 2.0 * ir2 + (dl0 - 2.0 * ir2) * (1.0 / 3.0);
    } else {
      const double mix = (U1[2][2] - U1[2][0] - U1[0][2] + U1[0][0]) * i4h;
      L = l0 + l1 - u0 * ir2 + (l0 - u0 * ir2 + mix) * (1.0 / 3.0);
      dg = dlap - ir2 + (dl0 - ir2) * (1.0 / 3.0);
    }
    mgv_line_row(G, ax, cc, 0, dg, fv[0] - L, wa[k], wc[k], d[k]);
  };
  auto row1 = [&](int k) {
    double l0, l1, L, dg;
    second(U1, l0, l1);
    const double u1 = U1[1][1];
    if (sph) {
      const double dr = (U0[1][2] - U0[1][0]) * i2h1;
      const double mix = (rp * rp * (U0[2][2] - U0[2][0]) - rm * rm * (U0[0][2] - U0[0][0])) * (i4h * ir2 * ir);
      L = l0 + l1 - u1 * ir2 * is2 + 2.0 * ir2 * dr + (mix + l1 - u1 * ir2 * is2) * (1.0 / 3.0);
      dg = dlap - ir2 * is2 + (dl1 - ir2 * is2) * (1.0 / 3.0);
    } else {
      const double mix = (rp * (U0[2][2] - U0[2][0]) - rm * (U0[0][2] - U0[0][0])) * (i4h * ir);
      L = l0 + l1 + (mix + l1) * (1.0 / 3.0);
      dg = dlap + dl1 * (1.0 / 3.0);
    }
    mgv_line_row(G, ax, cc, 1, dg, fv[1] - L, wa[k], wc[k], d[k]);
  };
  auto row2 = [&](int k) {
    double l0, l1;
    second(U2, l0, l1);
    mgv_line_row(G, ax, cc, 2, dlap - ir2 * is2, fv[2] - (l0 + l1 - U2[1][1] * ir2 * is2), wa[k], wc[k], d[k]);
  };
  if (!PAIR) {
    on ? row2(0) : zero(0);
    mg_pcr<NS>(sm, n, m, on, one_wave, wa, wc, d);
    xq[2] = d[0];
    mg_line_sync(one_wave);
  }
  on ? row0(0) : zero(0);
  if (PAIR) on ? row2(NS - 1) : zero(NS - 1);
  mg_pcr<NS>(sm, n, m, on, one_wave, wa, wc, d);
  xq[0] = d[0];
  if (PAIR) xq[2] = d[NS - 1];
  // the first component's update, for the neighbours: beyond the systems, or in
  // the last sixth of the copy that the last doubling did not read (the second
  // component's doublings reach it only after a barrier)
  const int doublings = 32 - __clz(n - 1);
  double *X = PAIR ? sm + ((doublings & 1) * 6 + 5) * n : sm + 6 * n;
  if (on) X[m] = xq[0];
  mg_line_sync(one_wave);
  double xa[1] = {0.0}, xc[1] = {0.0}, xd[1] = {0.0};
  if (on) {
    const double dx[3] = {X[m + along[0]], xq[0], X[m + along[2]]};
#pragma unroll
    for (int x = 0; x < 3; x++)
#pragma unroll
      for (int y = 0; y < 3; y++)
        if (line[ax == 0 ? y : x]) U0[x][y] += mgv_flip(dx[ax == 0 ? x : y], flip0[x][y]);
    row1(0);
    xa[0] = wa[0];
    xc[0] = wc[0];
    xd[0] = d[0];
  }
  mg_pcr<1>(sm, n, m, on, one_wave, xa, xc, xd);
  if (on) {
    u[o] += xq[0];
    u[nt + o] = U1[1][1] + xd[0];
    u[2 * nt + o] = U2[1][1] + xq[2];
  }
}

// KIND 0: any level; 1 and 2: axisymmetric levels, the third component
// apart or paired (mgv_line_curv).
template <int KIND>
__device__ __forceinline__ void mgv_line_any(const MgGeo &G, double *u, const double *__restrict__ f, int ax,
                                             const int c[3], bool live, double *sm, int m, bool one_wave) {
  if constexpr (KIND == 0)
    mgv_line_step(G, u, f, ax, c, live, sm, m, one_wave);
  else
    mgv_line_curv<KIND == 2>(G, u, f, ax, c, live, sm, m, one_wave);
}

template <int KIND, int THREADS>
__global__ __launch_bounds__(THREADS) void k_mgv_line(const MgGeo G, double *u, const double *__restrict__ f, int ax,
                                                      int colour) {
  extern __shared__ double sm[];
  int c[3];
  if (!mg_line(G, ax, colour, mg_xcd_run(), c)) return;
  mgv_line_any<KIND>(G, u, f, ax, c, true, sm, threadIdx.x, blockDim.x == kLineWave);
}

// Coarsest level of the vector equations (as k_mg_line_coarse): X and f
// staged in LDS, then 12 nmax doubles per line at work (52.9 us on 20x2 cells,
// 181 with the general step).
template <int KIND>
__global__ __launch_bounds__(KIND ? kCoarseLineThreads : 512) void k_mgv_line_coarse(const MgGeo G, double *u,
                                                                        const double *__restrict__ f, int sweeps,
                                                                        int nmax, int lanes) {
  extern __shared__ double sm[];
  const long n3 = 3 * G.nt;
  for (long e = threadIdx.x; e < n3; e += blockDim.x) {
    sm[e] = u[e];
    sm[n3 + e] = f[e];
  }
  __syncthreads();
  double *lines = sm + 2 * n3;
  const int w = threadIdx.x / lanes, ln = threadIdx.x % lanes, nw = blockDim.x / lanes;
  for (int s = 0; s < sweeps; s++)
    for (int ax = 0; ax < G.ndim; ax++) {
      if (G.bc[ax][0] == GMUNU_MG_PERIODIC) continue;
      for (int col = 0; col < 1 << (G.ndim - 1); col++) {
        const long nl = mg_line_count(G, ax, col);
        for (long t0 = 0; t0 < nl; t0 += nw) {
          int c[3] = {0, 0, 0};
          const bool live = mg_line(G, ax, col, t0 + w, c);
          mgv_line_any<KIND>(G, sm, sm + n3, ax, c, live, lines + (long)w * 12 * nmax, ln, lanes == kLineWave);
          __syncthreads();
        }
      }
    }
  for (long e = threadIdx.x; e < n3; e += blockDim.x) u[e] = sm[e];
}

__global__ __launch_bounds__(NT) void k_mgv_apply(const MgGeo G, const double *__restrict__ u,
                                                  double *__restrict__ out) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = mg_off(G, i, j, k);
  double L[3], idg[3];
  mgv_L(G, u, o, i, j, k, L, idg);
#pragma unroll
  for (int q = 0; q < 3; q++) out[q * G.nt + o] = L[q];
}

__global__ __launch_bounds__(NT) void k_mgv_norm(const MgGeo G, const double *__restrict__ u,
                                                 const double *__restrict__ f, double *part) {
  double m = 0.0;
  for (long t = (long)blockIdx.x * NT + threadIdx.x; t < mg_cells(G); t += (long)gridDim.x * NT) {
    int i, j, k;
    mg_cell(G, t, i, j, k);
    const long o = mg_off(G, i, j, k);
    double L[3], idg[3];
    mgv_L(G, u, o, i, j, k, L, idg);
#pragma unroll
    for (int q = 0; q < 3; q++) m = mg_absmax(m, f[q * G.nt + o] - L[q]);
  }
  m = block_max(m);
  if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// Coarse problem of a fine level for the vector equation: the children's
// residuals and values, volume-weighted means into the coarse r and u.  One
// thread per child, the 2^ndim of a coarse cell meeting by lane exchanges:
// bound by the latency of the operator's loads, which eight children in turn
// paid eight times (31 to 35 us from 64^3, 32^3 and 16^3 cells; now 13, 8 and 8; from 128^3 85, now 82).
__global__ __launch_bounds__(NT) void k_mgv_restrict_res(const MgGeo F, const MgGeo C, const double *__restrict__ u,
                                                         const double *__restrict__ f, double *__restrict__ uc,
                                                         double *__restrict__ rc) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  const int nd = F.ndim, ch = (int)(t & ((1 << nd) - 1));
  const bool live = t >> nd < mg_cells(C);
  double su[3] = {0.0, 0.0, 0.0}, sr[3] = {0.0, 0.0, 0.0}, w = 0.0;
  int i = 0, j = 0, k = 0;
  if (live) {
    mg_cell(C, t >> nd, i, j, k);
    const int fi = 2 * i + (ch & 1);
    const int fj = nd > 1 ? 2 * j + ((ch >> 1) & 1) : j;
    const int fk = nd > 2 ? 2 * k + ((ch >> 2) & 1) : k;
    const long o = mg_off(F, fi, fj, fk);
    w = F.vol0[fi + F.g[0]] * F.vol1[fj + F.g[1]];
    double L[3], idg[3];
    mgv_L(F, u, o, fi, fj, fk, L, idg);
#pragma unroll
    for (int q = 0; q < 3; q++) {
      su[q] = w * u[q * F.nt + o];
      sr[q] = w * (f[q * F.nt + o] - L[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < 3; q++) {
    su[q] = mg_sum_children(su[q], nd);
    sr[q] = mg_sum_children(sr[q], nd);
  }
  w = mg_sum_children(w, nd);
  if (!live || ch) return;
  const long oc = mg_off(C, i, j, k);
#pragma unroll
  for (int q = 0; q < 3; q++) {
    uc[q * C.nt + oc] = su[q] / w;
    rc[q * C.nt + oc] = sr[q] / w;
  }
}

// f_c = L_c(u_c) + r_c and uo_c = u_c.
__global__ __launch_bounds__(NT) void k_mgv_fas_rhs(const MgGeo C, const double *__restrict__ u,
                                                    const double *__restrict__ r, double *__restrict__ f,
                                                    double *__restrict__ uo) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(C)) return;
  int i, j, k;
  mg_cell(C, t, i, j, k);
  const long o = mg_off(C, i, j, k);
  double L[3], idg[3];
  mgv_L(C, u, o, i, j, k, L, idg);
#pragma unroll
  for (int q = 0; q < 3; q++) {
    f[q * C.nt + o] = L[q] + r[q * C.nt + o];
    uo[q * C.nt + o] = u[q * C.nt + o];
  }
}

// A~^ij = grad^i X^j + grad^j X^i - (2/3) delta^ij div X in orthonormal
// components (centred, boundary rule across the boundary; the connection
// terms of cylindrical and spherical coordinates, d/dphi = 0) as six
// components (xx yy zz xy xz yz in the order of the axes), and A~_ij A~^ij.
__global__ __launch_bounds__(NT) void k_mgv_aij(const MgGeo G, const double *__restrict__ X, double *__restrict__ A6,
                                                double *__restrict__ A2) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = mg_off(G, i, j, k);
  const VStep s = mgv_steps(G, i, j, k);
  double g[3][3];  // g[a][b] = grad_a X_b in orthonormal components
#pragma unroll
  for (int a = 0; a < 3; a++)
#pragma unroll
    for (int b = 0; b < 3; b++) {
      const double *xb = X + b * G.nt;
      g[a][b] = a < G.ndim ? (mgv_sgn(s.neg, 6 * b + 3 + a, xb[o + s.dp[a]]) -
                              mgv_sgn(s.neg, 6 * b + a, xb[o + s.dm[a]])) /
                                 (2.0 * G.h[a])
                           : 0.0;
    }
  // connection terms (d/dphi = 0)
  const double x0v = X[o], x1v = X[G.nt + o], x2v = X[2 * G.nt + o];
  if (G.coord == GMUNU_CYL) {
    const double R = G.x0[0] + (i + 0.5) * G.h[0];
    g[2][0] = -x2v / R;
    g[2][1] = 0.0;
    g[2][2] = x0v / R;
  } else if (G.coord == GMUNU_SPH) {
    const double r = G.x0[0] + (i + 0.5) * G.h[0], th = G.x0[1] + (j + 0.5) * G.h[1];
    const double ct = cos(th) / sin(th);
    g[1][0] = (g[1][0] - x1v) / r;
    g[1][1] = (g[1][1] + x0v) / r;
    g[1][2] = g[1][2] / r;
    g[2][0] = -x2v / r;
    g[2][1] = -ct * x2v / r;
    g[2][2] = (x0v + ct * x1v) / r;
  }
  const double dv = g[0][0] + g[1][1] + g[2][2];
  double A[3][3], a2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; a++)
#pragma unroll
    for (int b = 0; b < 3; b++) {
      A[a][b] = g[a][b] + g[b][a] - (a == b ? 2.0 / 3.0 * dv : 0.0);
      a2 += A[a][b] * A[a][b];
    }
  if (A6) {  // null: A2 alone (the residual check)
    A6[o] = A[0][0];
    A6[G.nt + o] = A[1][1];
    A6[2 * G.nt + o] = A[2][2];
    A6[3 * G.nt + o] = A[0][1];
    A6[4 * G.nt + o] = A[0][2];
    A6[5 * G.nt + o] = A[1][2];
  }
  A2[o] = a2;
}

// Source of the shift equation: 16 pi w S_i + 2 A~^ij grad_j w, w = alpha
// psi^-6 with its ghost entries as stored (centred orthonormal gradient).
__global__ __launch_bounds__(NT) void k_mgv_beta_rhs(const MgGeo G, const double *__restrict__ w,
                                                     const double *__restrict__ S, const double *__restrict__ A6,
                                                     double *__restrict__ out) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = mg_off(G, i, j, k);
  const long St[3] = {1, G.s1, G.s2};
  double gw[3];
#pragma unroll
  for (int a = 0; a < 3; a++) gw[a] = a < G.ndim ? (w[o + St[a]] - w[o - St[a]]) / (2.0 * G.h[a]) : 0.0;
  if (G.coord == GMUNU_SPH) gw[1] /= G.x0[0] + (i + 0.5) * G.h[0];  // orthonormal theta component
  const long nt = G.nt;
  const double axx = A6[o], ayy = A6[nt + o], azz = A6[2 * nt + o];
  const double axy = A6[3 * nt + o], axz = A6[4 * nt + o], ayz = A6[5 * nt + o];
  const double wc = 16.0 * M_PI * w[o];
  out[o] = wc * S[o] + 2.0 * (axx * gw[0] + axy * gw[1] + axz * gw[2]);
  out[nt + o] = wc * S[nt + o] + 2.0 * (axy * gw[0] + ayy * gw[1] + ayz * gw[2]);
  out[2 * nt + o] = wc * S[2 * nt + o] + 2.0 * (axz * gw[0] + ayz * gw[1] + azz * gw[2]);
}

// ------------------------------------------------- bridge to the GRMHD state

// Layout of a GRMHD state array (include/gmunu.h: [var][k][j][i], ng ghost
// layers on active axes) on the multigrid grid's interior.
struct Hydro {
  int ng[3];
  long T0, T1, nv;  // cells per row, per plane, per variable
  double gam;
};

__device__ __forceinline__ long hy_off(const Hydro &H, int i, int j, int k) {
  return (long)(k + H.ng[2]) * H.T1 + (long)(j + H.ng[1]) * H.T0 + (i + H.ng[0]);
}

// q_B of every entry of the multigrid vector layout (interior from q, the
// ghost layer from psi^6 times the primitive field, which the GRMHD ghost
// fill maintains).
__global__ __launch_bounds__(NT) void k_br_gather_qb(const MgGeo G, const Hydro H, const double *__restrict__ q,
                                                     const double *__restrict__ prim, const double *__restrict__ met,
                                                     double *__restrict__ qb) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= G.nt) return;
  const int I = (int)(t % G.s1), J = (int)((t / G.s1) % (G.s2 / G.s1)), K = (int)(t / G.s2);
  const int i = I - G.g[0], j = J - G.g[1], k = K - G.g[2];
  const long o = hy_off(H, i, j, k);
  const bool inside = i >= 0 && i < G.n[0] && j >= 0 && j < G.n[1] && k >= 0 && k < G.n[2];
  const double psi = met[o], psi2 = psi * psi, psi6 = psi2 * psi2 * psi2;
#pragma unroll
  for (int c = 0; c < 3; c++) qb[c * G.nt + t] = inside ? q[(5 + c) * H.nv + o] : psi6 * prim[(5 + c) * H.nv + o];
}

__global__ __launch_bounds__(NT) void k_br_scatter_qb(const MgGeo G, const Hydro H, const double *__restrict__ qb,
                                                      double *__restrict__ q) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = hy_off(H, i, j, k), m = mg_off(G, i, j, k);
#pragma unroll
  for (int c = 0; c < 3; c++) q[(5 + c) * H.nv + o] = qb[c * G.nt + m];
}

// Coefficients of the scalar CFC equations (section 2.6) on the interior:
// which 0 (conformal factor): a = -2 pi U~ with U~ = q_tau + q_D, and with
// A2 = A~_ij A~^ij given, a2 = -A2 / 8 (the term in psi^-7);
// which 1 (lapse): a = 2 pi (U~ + 2 S~) / psi^2 (+ (7/8) A2 psi^-8) with
// S~ = psi^6 (rho h W^2 v^2 + 3 p) from the primitives (fluid part) and psi
// from the metric.  u: the initial guess u = psi - 1, or alpha psi - 1, from
// the metric.
__global__ __launch_bounds__(NT) void k_br_cfc_coef(const MgGeo G, const Hydro H, const double *__restrict__ q,
                                                    const double *__restrict__ prim, const double *__restrict__ met,
                                                    int which, const double *__restrict__ A2, double *__restrict__ a,
                                                    double *__restrict__ a2, double *__restrict__ u) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = hy_off(H, i, j, k), m = mg_off(G, i, j, k);
  const double Ut = q[4 * H.nv + o] + q[o];
  const double psi = met[o];
  if (which == 0) {
    a[m] = -2.0 * M_PI * Ut;
    if (A2) a2[m] = -A2[m] / 8.0;
    u[m] = psi - 1.0;
    return;
  }
  const double psi2 = psi * psi, psi4 = psi2 * psi2;
  // gamma_ij = psi^4 gamma^_ij with the reference metric of the grid
  const int I = i + G.g[0], J = j + G.g[1];
  double g1 = 1.0, g2 = 1.0;
  if (G.coord == GMUNU_CYL) g2 = 1.0 / G.g2[I];
  if (G.coord == GMUNU_SPH) {
    g1 = 1.0 / G.g1[I];
    g2 = g1 / G.s2t[J];
  }
  const double u1 = prim[H.nv + o], u2 = prim[2 * H.nv + o], u3 = prim[3 * H.nv + o];
  const double w2v2 = psi4 * (u1 * u1 + g1 * u2 * u2 + g2 * u3 * u3);
  const double rho = prim[o], p = prim[4 * H.nv + o];
  const double rhoh = rho + H.gam / (H.gam - 1.0) * p;
  const double St = psi4 * psi2 * (rhoh * w2v2 + 3.0 * p);
  double av = 2.0 * M_PI * (Ut + 2.0 * St) / psi2;
  if (A2) av += 7.0 / 8.0 * A2[m] / (psi4 * psi4);
  a[m] = av;
  u[m] = met[H.nv + o] * psi - 1.0;
}

// Scale factors of the reference metric at signed cell-centre coordinates
// (x0, x1): orthonormal component = h_c times the contravariant one, and
// the covariant one divided by h_c.
__device__ __forceinline__ double mg_hscale(int coord, int c, double x0, double x1) {
  if (coord == GMUNU_CYL) return c == 2 ? x0 : 1.0;
  if (coord == GMUNU_SPH) return c == 0 ? 1.0 : c == 1 ? x0 : x0 * sin(x1);
  return 1.0;
}

// Momentum source of the vector equations in orthonormal components:
// S[c] = q_{S_c} / h_c (q_S = psi^6 S_c covariant, the rescaled S~_c of
// section 2.6) and fX = 8 pi S, on the interior.
__global__ __launch_bounds__(NT) void k_bx_src(const MgGeo G, const Hydro H, const double *__restrict__ q,
                                               double *__restrict__ S, double *__restrict__ fX) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = hy_off(H, i, j, k), m = mg_off(G, i, j, k);
  const double x0 = G.x0[0] + (i + 0.5) * G.h[0], x1 = G.x0[1] + (j + 0.5) * G.h[1];
#pragma unroll
  for (int c = 0; c < 3; c++) {
    const double v = q[(1 + c) * H.nv + o] / mg_hscale(G.coord, c, x0, x1);
    S[c * G.nt + m] = v;
    fX[c * G.nt + m] = 8.0 * M_PI * v;
  }
}

// w = alpha psi^-6 on every entry of the multigrid layout (its ghost layer
// from the metric's first ghost layer).
__global__ __launch_bounds__(NT) void k_bx_w(const MgGeo G, const Hydro H, const double *__restrict__ met,
                                             double *__restrict__ w) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= G.nt) return;
  const int I = (int)(t % G.s1), J = (int)((t / G.s1) % (G.s2 / G.s1)), K = (int)(t / G.s2);
  const long o = hy_off(H, I - G.g[0], J - G.g[1], K - G.g[2]);
  const double psi = met[o], psi2 = psi * psi;
  w[t] = met[H.nv + o] / (psi2 * psi2 * psi2);
}

// The metric's shift on the interior (orthonormal components) as the
// initial guess of its solve.
__global__ __launch_bounds__(NT) void k_bx_beta_in(const MgGeo G, const Hydro H, const double *__restrict__ met,
                                                   double *__restrict__ beta) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= mg_cells(G)) return;
  int i, j, k;
  mg_cell(G, t, i, j, k);
  const long o = hy_off(H, i, j, k), m = mg_off(G, i, j, k);
  const double x0 = G.x0[0] + (i + 0.5) * G.h[0], x1 = G.x0[1] + (j + 0.5) * G.h[1];
#pragma unroll
  for (int c = 0; c < 3; c++) beta[c * G.nt + m] = met[(2 + c) * H.nv + o] * mg_hscale(G.coord, c, x0, x1);
}

// Metric of every GRMHD cell (ng ghost layers included) from the solution u
// of level G, ghost layers extended by the multigrid boundary rule applied
// per layer (mirror about the face times -1, +1 or r_in / r_ghost; periodic
// wrap): which 0 writes psi = 1 + u, which 1 alpha = (1 + u) / psi, which
// 2..4 the shift component c = which - 2 from its orthonormal value u
// (mirrored with the component's parity, then divided by h_c at the
// cell's signed coordinates).
__global__ __launch_bounds__(NT) void k_br_store(const MgGeo G, const Hydro H, const double *__restrict__ u,
                                                 double xmin0, int which, double *__restrict__ met) {
  const long t = (long)blockIdx.x * NT + threadIdx.x;
  if (t >= H.nv) return;
  int c[3] = {(int)(t % H.T0) - H.ng[0], (int)((t / H.T0) % (H.T1 / H.T0)) - H.ng[1], (int)(t / H.T1) - H.ng[2]};
  const double xc0 = G.x0[0] + (c[0] + 0.5) * G.h[0], xc1 = G.x0[1] + (c[1] + 0.5) * G.h[1];
  double fac = 1.0;
  // axes from the last to the first: an edge or corner ghost takes the
  // factor of each axis at the other coordinates not yet mapped inside
#pragma unroll
  for (int a = 2; a >= 0; a--) {
    if (a >= G.ndim) continue;
    const int n = G.n[a];
    if (c[a] >= 0 && c[a] < n) continue;
    const int side = c[a] < 0 ? 0 : 1;
    const int kind = G.bc[a][side];
    if (kind == GMUNU_MG_PERIODIC) {
      c[a] = side == 0 ? c[a] + n : c[a] - n;
      continue;
    }
    const int in = side == 0 ? -1 - c[a] : 2 * n - 1 - c[a];
    if (which >= 2) {
      if ((G.vodd[a][side] >> (which - 2)) & 1) fac = -fac;
    } else if (kind == GMUNU_MG_DIRICHLET) {
      fac = -fac;
    }
    if (which < 2 && kind == GMUNU_MG_ROBIN) {
      if (G.coord == GMUNU_SPH) {
        fac *= (xmin0 + (in + 0.5) * G.h[0]) / (xmin0 + (c[a] + 0.5) * G.h[0]);
      } else {
        const int nb = G.coord == GMUNU_CYL ? 2 : 3;
        double ri = 0.0, rg = 0.0;
#pragma unroll
        for (int b = 0; b < 3; b++) {
          if (b >= G.ndim || b >= nb) continue;
          const double xg = G.x0[b] + (c[b] + 0.5) * G.h[b];
          const double xi = b == a ? G.x0[b] + (in + 0.5) * G.h[b] : xg;
          ri += xi * xi;
          rg += xg * xg;
        }
        fac *= sqrt(ri) / sqrt(rg);
      }
    }
    c[a] = in;
  }
  const double v = fac * u[mg_off(G, c[0], c[1], c[2])];
  if (which == 0)
    met[t] = 1.0 + v;
  else if (which == 1)
    met[H.nv + t] = (1.0 + v) / met[t];
  else
    met[which * H.nv + t] = v / mg_hscale(G.coord, which - 2, xc0, xc1);
}

}  // namespace

struct gmunu_mg {
  gmunu_mg_desc d;
  int levels;
  MgGeo geo[kMaxLevels];
  double *tab;  // geometry tables of all levels (device)
  // per level: u, f, a, r, uo (the finest level's u, f, a are the caller's;
  // a[l] is NULL when the equation has no a)
  double *u[kMaxLevels], *f[kMaxLevels], *a[kMaxLevels], *r[kMaxLevels], *uo[kMaxLevels];
  double *aown[kMaxLevels];  // coarse-level storage of a
  double *a2[kMaxLevels], *a2own[kMaxLevels];  // the same for a2 (allocated when power2 != 0)
  // second fields of the levels above the tail that k_mg_rb relaxes out of
  // place (the finest level's allocated by the first solve; null: in place)
  double *us[kMaxLevels];
  // the tail's plans by the terms present (bit 0: a, bit 1: a2): top level
  // (-1: none) and device copy; the levels' geometries and their own a and
  // a2 arrays on the device
  int ttop[4];
  MgTail *tplan;
  MgGeo *tgeo;
  double **tptr;
  int vtop;        // the vector equations' tail (Cartesian point smoother; -1: none)
  MgvTail *vplan;
  double *part;  // norm partials + result
  double *br;    // state bridge scratch (6 arrays of the finest level), allocated on first use
  // vector equations (Cartesian): per coarse level u, f, r, uo of three
  // components each, allocated on first use; xs: scratch of the xCFC
  // sequence (17 finest arrays), allocated on first use
  double *vu[kMaxLevels], *vf[kMaxLevels], *vr[kMaxLevels], *vuo[kMaxLevels];
  double *vs[kMaxLevels];  // second field of the levels that k_mgv_planes relaxes (null: none)
  bool vready;
  double *xs;
  std::vector<double *> owned;
  // V-cycles are replayed from graphs captured on a private stream, each for
  // the finest arrays it was captured with (two per kind of equation)
  hipStream_t gs;
  hipEvent_t ev;
  struct Slot {
    hipGraphExec_t exec;
    bool vec;
    const double *u, *f, *a, *a2;
  } slot[4];
  int next_slot;
};

namespace {

// Axis a after L halvings: divisible, at least two cells, and an even count
// on a periodic axis (an odd count would give the cells on either side of
// the wrap the same colour, and a colour's cells would not be independent).
bool coarsens(const gmunu_mg_desc &d, int a, int L) {
  const int n = d.n[a] >> L;
  return d.n[a] % (1 << L) == 0 && n >= 2 && (d.bc[a][0] != GMUNU_MG_PERIODIC || n % 2 == 0);
}

int auto_levels(const gmunu_mg_desc &d) {
  int L = 1;
  for (;;) {
    bool ok = L < kMaxLevels;
    for (int a = 0; a < d.ndim && ok; a++) ok = coarsens(d, a, L);
    if (!ok) return L;
    L++;
  }
}

int validate(const gmunu_mg_desc &d, int levels) {
  if (d.ndim < 1 || d.ndim > 3 || d.coord < GMUNU_CART || d.coord > GMUNU_SPH) return GMUNU_EINVAL;
  if (levels < 1 || levels > kMaxLevels) return GMUNU_EINVAL;
  for (int a = 0; a < 3; a++) {
    if (a >= d.ndim) {
      if (d.n[a] != 1) return GMUNU_EINVAL;
      continue;
    }
    if (d.n[a] < 1 || !(d.dx[a] > 0.0) || !coarsens(d, a, levels - 1)) return GMUNU_EINVAL;
    for (int s = 0; s < 2; s++) {
      const int b = d.bc[a][s];
      if (b < GMUNU_MG_DIRICHLET || b > GMUNU_MG_ROBIN) return GMUNU_EINVAL;
      if (b == GMUNU_MG_ROBIN && ((d.coord == GMUNU_SPH && a != 0) || (d.coord == GMUNU_CYL && a == 2)))
        return GMUNU_EINVAL;
      if ((b == GMUNU_MG_PERIODIC) != (d.bc[a][1 - s] == GMUNU_MG_PERIODIC)) return GMUNU_EINVAL;
    }
  }
  if (d.coord != GMUNU_CART && d.xmin[0] < 0.0) return GMUNU_EINVAL;
  if (d.coord == GMUNU_SPH && d.ndim > 1 && (d.xmin[1] < 0.0 || d.xmin[1] + d.n[1] * d.dx[1] > M_PI + 1e-12))
    return GMUNU_EINVAL;
  if (d.power < -1 || d.power > 1 || d.pre < 0 || d.post < 0 || d.coarse < 1) return GMUNU_EINVAL;
  if (d.power2 < -8 || d.power2 > 8) return GMUNU_EINVAL;
  if (d.smoother != GMUNU_MG_POINT && d.smoother != GMUNU_MG_LINE) return GMUNU_EINVAL;
  for (int a = 0; a < d.ndim; a++)
    if (d.smoother == GMUNU_MG_LINE && d.bc[a][0] != GMUNU_MG_PERIODIC && d.n[a] > kMaxLine) return GMUNU_EINVAL;
  // cell numbers of a level fit 32-bit kernel arithmetic
  if ((double)(d.n[0] + 2) * (d.n[1] + 2) * (d.n[2] + 2) >= 2147483647.0) return GMUNU_EINVAL;
  return GMUNU_OK;
}

// Host tables of one level: 6 per axis-0 index, 5 per axis-1 index.
void level_tables(const gmunu_mg_desc &d, int s, std::vector<double> &tab, size_t off[11], MgGeo &G) {
  for (int a = 0; a < 3; a++) {
    G.g[a] = a < d.ndim ? 1 : 0;
    G.n[a] = a < d.ndim ? d.n[a] >> s : 1;
    G.h[a] = a < d.ndim ? d.dx[a] * (double)(1 << s) : d.dx[a];
  }
  const int t0 = G.n[0] + 2 * G.g[0], t1 = G.n[1] + 2 * G.g[1], t2 = G.n[2] + 2 * G.g[2];
  G.s1 = t0;
  G.s2 = (long)t0 * t1;
  G.nt = G.s2 * t2;
  G.ndim = d.ndim;
  G.coord = d.coord;
  G.ih2_2 = 1.0 / (G.h[2] * G.h[2]);
  const bool cyl = d.coord == GMUNU_CYL, sph = d.coord == GMUNU_SPH;
  std::vector<double> a0m(t0), a0p(t0), g1(t0), g2(t0), vol0(t0), sg0(t0);
  const double h0 = G.h[0], h02 = h0 * h0;
  for (int I = 0; I < t0; I++) {
    const double x = d.xmin[0] + (I - G.g[0] + 0.5) * h0;
    const double fm = d.xmin[0] + (I - G.g[0]) * h0, fp = fm + h0;
    a0m[I] = a0p[I] = 1.0 / h02;
    g1[I] = g2[I] = vol0[I] = sg0[I] = 1.0;
    if (cyl) {
      a0m[I] = fm / (x * h02);
      a0p[I] = fp / (x * h02);
      g2[I] = 1.0 / (x * x);
      vol0[I] = sg0[I] = x;
    } else if (sph) {
      a0m[I] = fm * fm / (x * x * h02);
      a0p[I] = fp * fp / (x * x * h02);
      g1[I] = g2[I] = 1.0 / (x * x);
      vol0[I] = x * x + h02 / 12.0;
      sg0[I] = x * x;
    }
  }
  std::vector<double> a1m(t1), a1p(t1), s2t(t1), vol1(t1), sg1(t1);
  const double h1 = G.h[1], h12 = h1 * h1;
  for (int J = 0; J < t1; J++) {
    const double y = d.xmin[1] + (J - G.g[1] + 0.5) * h1;
    const double fm = d.xmin[1] + (J - G.g[1]) * h1, fp = fm + h1;
    a1m[J] = a1p[J] = 1.0 / h12;
    s2t[J] = vol1[J] = sg1[J] = 1.0;
    if (sph) {
      const double sy = std::sin(y);
      a1m[J] = std::sin(fm) / (sy * h12);
      a1p[J] = std::sin(fp) / (sy * h12);
      s2t[J] = 1.0 / (sy * sy);
      vol1[J] = d.ndim > 1 ? sy : 1.0;
      sg1[J] = sy;
    }
  }
  const std::vector<double> *all[11] = {&a0m, &a0p, &g1, &g2, &vol0, &sg0, &a1m, &a1p, &s2t, &vol1, &sg1};
  for (int q = 0; q < 11; q++) {
    while (tab.size() % 32) tab.push_back(0.0);
    off[q] = tab.size();
    tab.insert(tab.end(), all[q]->begin(), all[q]->end());
  }
  for (int a = 0; a < 3; a++)
    for (int sd = 0; sd < 2; sd++) G.bc[a][sd] = d.bc[a][sd];
  // Robin ghost factors: centre of the boundary cell / centre of its ghost
  const double xin_lo = d.xmin[0] + 0.5 * h0, xg_lo = d.xmin[0] - 0.5 * h0;
  const double xin_hi = d.xmin[0] + (G.n[0] - 0.5) * h0, xg_hi = d.xmin[0] + (G.n[0] + 0.5) * h0;
  G.rob_lo = xin_lo / xg_lo;
  G.rob_hi = xin_hi / xg_hi;
  for (int a = 0; a < 3; a++) G.x0[a] = d.xmin[a];
  // per-component parity across each non-periodic face for the vector
  // equations: Dirichlet all odd; Neumann a symmetry face (normal component
  // odd), plus phi at the cylindrical and polar axes and every component at
  // the spherical centre (equatorially symmetric grids)
  for (int a = 0; a < 3; a++)
    for (int sd = 0; sd < 2; sd++) {
      const double fpos = sd == 0 ? d.xmin[a] : d.xmin[a] + d.n[a] * d.dx[a];
      unsigned odd = d.bc[a][sd] == GMUNU_MG_DIRICHLET ? 7u : 1u << a;
      if (d.bc[a][sd] == GMUNU_MG_NEUMANN) {
        if (d.coord == GMUNU_CYL && a == 0 && std::fabs(fpos) < 1e-12) odd |= 4u;
        if (d.coord == GMUNU_SPH && a == 0 && std::fabs(fpos) < 1e-12) odd = 7u;
        if (d.coord == GMUNU_SPH && a == 1 && (std::fabs(fpos) < 1e-12 || std::fabs(fpos - M_PI) < 1e-12)) odd |= 4u;
      }
      G.vodd[a][sd] = odd;
    }
  G.power = d.power;
  G.power2 = d.power2;
  G.offset = d.offset;
  G.line = 0;
  for (int a = 0; a < d.ndim; a++)
    if (d.smoother == GMUNU_MG_LINE && d.bc[a][0] != GMUNU_MG_PERIODIC) G.line = 1;
  double dsum = 0.0;
  for (int a = 0; a < 3; a++) {
    G.vih2[a] = a < d.ndim ? 1.0 / (G.h[a] * G.h[a]) : 0.0;
    dsum -= 2.0 * G.vih2[a];
  }
  const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
  for (int q = 0; q < 3; q++) {
    G.vmix[q] = pb[q] < d.ndim ? 1.0 / (4.0 * G.h[pa[q]] * G.h[pb[q]]) : 0.0;
    G.vidg[q] = 1.0 / (q < d.ndim ? dsum - (2.0 / 3.0) * G.vih2[q] : dsum);
  }
}

long ghost_count(const MgGeo &G) {
  long s = 0;
  for (int a = 0; a < G.ndim; a++) {
    const int b1 = a == 0 ? 1 : 0, b2 = a == 2 ? 1 : 2;
    s += 2L * G.n[b1] * G.n[b2];
  }
  return s;
}

long cells(const MgGeo &G) { return (long)G.n[0] * G.n[1] * G.n[2]; }

void ghosts(const MgGeo &G, double *u, hipStream_t st) {
  const long gc = ghost_count(G);
  if (gc) hipLaunchKernelGGL(k_mg_ghosts<1>, dim3(nblocks(gc)), dim3(NT), 0, st, G, u);
}

// Threads per line workgroup: a lane per cell, whole wavefronts.
int line_threads(int n) { return (n + kLineWave - 1) / kLineWave * kLineWave; }

// Line sweeps: per sweep every non-periodic axis, per axis its colours.
void line_sweeps(const MgGeo &G, double *u, const double *f, const double *a, const double *a2, int sweeps,
                 hipStream_t st) {
  for (int s = 0; s < sweeps; s++)
    for (int ax = 0; ax < G.ndim; ax++) {
      if (G.bc[ax][0] == GMUNU_MG_PERIODIC) continue;
      const size_t lds = 6 * (size_t)G.n[ax] * sizeof(double);
      for (int c = 0; c < 1 << (G.ndim - 1); c++)
        hipLaunchKernelGGL(k_mg_line, dim3(mg_line_count(G, ax, c)), dim3(line_threads(G.n[ax])), lds, st, G, u, f,
                           a, a2, ax, c);
    }
}

// Longest line of a level.
int line_nmax(const MgGeo &G) {
  int nmax = 1;
  for (int ax = 0; ax < G.ndim; ax++)
    if (G.bc[ax][0] != GMUNU_MG_PERIODIC) nmax = G.n[ax] > nmax ? G.n[ax] : nmax;
  return nmax;
}

// A one-workgroup coarsest line solve staging `arrays` level arrays, with
// `per` doubles per cell of a line at work: lanes per line (a wavefront, or
// several for longer lines), as many lines at once as a colour has and as
// fit; lds = 0: does not fit.
struct LineCoarse {
  int lanes, threads;
  size_t lds;
};
LineCoarse line_coarse(const MgGeo &G, int arrays, int per, int max_threads = kCoarseLineThreads) {
  LineCoarse r{line_threads(line_nmax(G)), 0, 0};
  long lines = 1;
  for (int ax = 0; ax < G.ndim; ax++)
    if (G.bc[ax][0] != GMUNU_MG_PERIODIC) {
      const long c = mg_line_count(G, ax, 0);
      lines = c > lines ? c : lines;
    }
  const long most = max_threads / r.lanes;
  lines = lines < most ? lines : most;
  r.threads = (int)lines * r.lanes;
  const size_t b = ((size_t)arrays * G.nt + (size_t)lines * per * line_nmax(G)) * sizeof(double);
  r.lds = lines > 0 && b <= 64 * 1024 ? b : 0;
  return r;
}

// Smoothing sweeps in place (boundary rule inline: no ghost fill between
// colours): line sweeps for the line smoother, else red-black.
void sweeps_raw(const MgGeo &G, double *u, const double *f, const double *a, const double *a2, int sweeps,
                hipStream_t st) {
  if (G.line) {
    line_sweeps(G, u, f, a, a2, sweeps, st);
    return;
  }
  const long threads = (long)((G.n[0] + 1) / 2) * G.n[1] * G.n[2];
  for (int s = 0; s < sweeps; s++)
    for (int c = 0; c < 2; c++)
      hipLaunchKernelGGL(k_mg_smooth, dim3(nblocks(threads)), dim3(NT), 0, st, G, u, f, a, a2, c);
}

// Does a face have a position-dependent Robin factor?
bool rb_robin(const MgGeo &G) {
  bool rob = false;
  for (int q = 0; q < G.ndim; q++)
    rob = rob || (G.coord != GMUNU_SPH && (G.bc[q][0] == GMUNU_MG_ROBIN || G.bc[q][1] == GMUNU_MG_ROBIN));
  return rob;
}

// Levels that k_mg_rb relaxes.  Smaller 3D levels are faster in place: 64^3
// takes 24 us per pair of sweeps out of place (33 with Robin faces, 50 with the
// general term besides) against 16 as four launches; 128^3 45, 57 and 85 us
// against about 70.  In 2D the one tile pass beats the launches throughout.
bool rb_level(const MgGeo &G) {
  if (G.line || G.ndim < 2 || cells(G) <= kTailCells || G.s2 >= (1L << 29)) return false;  // 32-bit byte offsets
  const bool light = G.coord == GMUNU_CART && G.power != -1 && G.power2 == 0;
  return G.ndim == 2 || cells(G) >= (light ? 1L << 20 : 1L << 22);
}

// ns (1 or 2) sweeps out of place, u to out.
template <int ND, int NS>
void rb_launch(const MgGeo &G, const double *u, const double *f, const double *a, const double *a2, double *out,
               hipStream_t st) {
  using R = RbTile<ND, NS>;
  const int tiles = ((G.n[0] + R::TX - 1) / R::TX) * ((G.n[1] + R::TY - 1) / R::TY);
  const int terms = !a && !a2 ? 0 : a && !a2 && G.power == 1 ? 1 : 2;
  const bool rob = rb_robin(G);
  // 3D: planes per workgroup.  A chunk of L planes takes L + 4 H - 1 steps (halo
  // and pipeline).  With at most 256 workgroups a step takes about 1.05 us;
  // two workgroups fit a CU where the registers allow (no position-dependent
  // factor, no general term), a step of both 1.5 times as long (256^3: 190 us
  // in chunks of 64 planes, 240 in chunks of 128; 128^3: 49 in 8, 45 in 16).
  const bool two = G.coord == GMUNU_CART && terms < 2 && !rob;
  int chunk = 1;
  if (ND > 2) {
    double best = -1.0;
    for (int n = 1; n <= G.n[2]; n++) {
      const int len = (G.n[2] + n - 1) / n;
      if (n > 1 && len < 4) break;
      const long wg = (long)tiles * ((G.n[2] + len - 1) / len), steps = len + 4 * R::H - 1;
      const double cost = two && wg > 256 ? 1.5 * steps * ((wg + 511) / 512) : (double)steps * ((wg + 255) / 256);
      if (best < 0.0 || cost < best) {
        best = cost;
        chunk = len;
      }
    }
  }
  const dim3 grid(tiles * ((G.n[2] + chunk - 1) / chunk));
  auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(R::threads), 0, st, G, u, f, a, a2, out, chunk); };
  if (G.coord != GMUNU_CART)
    rob ? run(k_mg_rb<ND, NS, false, 2, true>) : run(k_mg_rb<ND, NS, false, 2, false>);
  else if (rob)
    terms == 1 ? run(k_mg_rb<ND, NS, true, 1, true>) : run(k_mg_rb<ND, NS, true, 2, true>);
  else
    terms == 0   ? run(k_mg_rb<ND, NS, true, 0, false>)
    : terms == 1 ? run(k_mg_rb<ND, NS, true, 1, false>)
                 : run(k_mg_rb<ND, NS, true, 2, false>);
}

void rb(const MgGeo &G, int ns, const double *u, const double *f, const double *a, const double *a2, double *out,
        hipStream_t st) {
  if (G.ndim == 2)
    ns == 2 ? rb_launch<2, 2>(G, u, f, a, a2, out, st) : rb_launch<2, 1>(G, u, f, a, a2, out, st);
  else
    ns == 2 ? rb_launch<3, 2>(G, u, f, a, a2, out, st) : rb_launch<3, 1>(G, u, f, a, a2, out, st);
}

// `sweeps` sweeps of field u, alternating with the second field s, in pairs;
// *cur: the field that holds the current values, u or s.  flips: how many
// launches, at least (sweeps + 1) / 2 and at most `sweeps`.
void rb_sweeps(const MgGeo &G, double *u, double *s, double **cur, const double *f, const double *a, const double *a2,
               int sweeps, int flips, hipStream_t st) {
  for (; sweeps > 0; flips--) {
    const int ns = sweeps > flips ? 2 : 1;
    double *next = *cur == u ? s : u;
    rb(G, ns, *cur, f, a, a2, next, st);
    *cur = next;
    sweeps -= ns;
  }
}

// `sweeps` sweeps whose result is in u again: an even number of launches (a
// single sweep in place).
void rb_sweeps_back(const MgGeo &G, double *u, double *s, const double *f, const double *a, const double *a2,
                    int sweeps, hipStream_t st) {
  if (sweeps == 1 || !s) {
    sweeps_raw(G, u, f, a, a2, sweeps, st);
    return;
  }
  const int least = (sweeps + 1) / 2;
  double *cur = u;
  rb_sweeps(G, u, s, &cur, f, a, a2, sweeps, least + (least & 1), st);
}

// The residual of a 2D or 3D level: its maxima (OP 0, at part) or restricted
// to level C (OP 1).  Returns the workgroups launched.
template <int ND, int OP>
int residual_nd(const MgGeo &G, const double *u, const double *f, const double *a, const double *a2, const MgGeo &C,
                double *uc, double *rc, double *part, hipStream_t st) {
  const long cols = (long)((G.n[0] + 31) / 32) * ((G.n[1] + 7) / 8);
  // planes per workgroup: as many as leave about eight workgroups per CU (even:
  // a coarse cell's planes stay together)
  long len = 1;
  if (ND > 2)
    for (len = 2; len < 16 && cols * (G.n[2] / (2 * len)) >= 2048;) len *= 2;
  const long tiles = ND > 2 ? cols * ((G.n[2] + len - 1) / len) : cols;
  const int grid = OP == 0 && tiles > kNormParts ? kNormParts : (int)tiles;
  const int terms = !a && !a2 ? 0 : a && !a2 && G.power == 1 ? 1 : 2;
  const bool rob = rb_robin(G);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(NT), 0, st, G, u, f, a, a2, C, uc, rc, part, (int)len, (int)tiles);
  };
  if (G.coord != GMUNU_CART)
    rob ? run(k_mg_res<ND, false, 2, true, OP>) : run(k_mg_res<ND, false, 2, false, OP>);
  else if (rob)
    terms == 1 ? run(k_mg_res<ND, true, 1, true, OP>) : run(k_mg_res<ND, true, 2, true, OP>);
  else
    terms == 0   ? run(k_mg_res<ND, true, 0, false, OP>)
    : terms == 1 ? run(k_mg_res<ND, true, 1, false, OP>)
                 : run(k_mg_res<ND, true, 2, false, OP>);
  return grid;
}
template <int OP>
int residual(const MgGeo &G, const double *u, const double *f, const double *a, const double *a2, const MgGeo &C,
             double *uc, double *rc, double *part, hipStream_t st) {
  return G.ndim == 2 ? residual_nd<2, OP>(G, u, f, a, a2, C, uc, rc, part, st)
                     : residual_nd<3, OP>(G, u, f, a, a2, C, uc, rc, part, st);
}

// Coarse problem of level l: u_{l-1} = R u_l (kept in uo_{l-1}),
// f_{l-1} = L_{l-1}(R u_l) + R (f_l - L_l(u_l)).
void coarse_problem(gmunu_mg *m, int l, hipStream_t st) {
  const MgGeo &F = m->geo[l], &C = m->geo[l - 1];
  if (F.ndim > 1)
    residual<1>(F, m->u[l], m->f[l], m->a[l], m->a2[l], C, m->u[l - 1], m->r[l - 1], nullptr, st);
  else
    hipLaunchKernelGGL(k_mg_restrict_res, dim3(nblocks(cells(C))), dim3(NT), 0, st, F, C, m->u[l], m->f[l], m->a[l],
                       m->a2[l], m->u[l - 1], m->r[l - 1]);
  hipLaunchKernelGGL(k_mg_fas_rhs, dim3(nblocks(cells(C))), dim3(NT), 0, st, C, m->u[l - 1], m->a[l - 1],
                     m->a2[l - 1], m->r[l - 1], m->f[l - 1], m->uo[l - 1]);
}

// u_l += P(u_{l-1} - uo_{l-1})
void correct(gmunu_mg *m, int l, hipStream_t st) {
  const MgGeo &F = m->geo[l], &C = m->geo[l - 1];
  hipLaunchKernelGGL(k_mg_correct<1>, dim3(nblocks(cells(C))), dim3(NT), 0, st, C, F, m->u[l - 1], m->uo[l - 1],
                     m->u[l]);
}

// Dynamic LDS a one-workgroup coarsest solve may stage (bytes).
constexpr long kCoarseLds = 64L * 1024;

// Which of the tail's plans serves the bound equation.
int tail_kind(const gmunu_mg *m) { return (m->a[0] ? 1 : 0) | (m->a2[0] ? 2 : 0); }

// A V-cycle (the whole FMG cycle) of the tail's levels, u and f of its top
// level in place.
void launch_tail(gmunu_mg *m, bool use_fmg, hipStream_t st) {
  const int kind = tail_kind(m), top = m->ttop[kind];
  const MgGeo &G = m->geo[top];
  const long nc = (long)((G.n[0] + 1) / 2) * G.n[1] * G.n[2], th = (nc + 63) / 64 * 64;
  const dim3 block(th < kTailThreads ? th : kTailThreads);
  bool rob = G.coord != GMUNU_CART;
  for (int a = 0; a < G.ndim; a++) rob = rob || G.bc[a][0] == GMUNU_MG_ROBIN || G.bc[a][1] == GMUNU_MG_ROBIN;
  const bool nl = m->d.power == -1 || m->a2[top];
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), block, 0, st, m->tplan + kind, m->tgeo, m->u[top], m->f[top], m->a[top],
                       m->a2[top], m->tptr, use_fmg ? 1 : 0);
  };
  if (G.coord != GMUNU_CART)
    run(k_mg_tail<false, true, true>);
  else if (rob)
    nl ? run(k_mg_tail<true, true, true>) : run(k_mg_tail<true, true, false>);
  else
    nl ? run(k_mg_tail<true, false, true>) : run(k_mg_tail<true, false, false>);
}

// The coarsest level beyond the tail: launches (the line smoother's own
// one-workgroup solve when it is small).
void coarse_solve(gmunu_mg *m, hipStream_t st) {
  const MgGeo &G = m->geo[0];
  if (G.line) {
    const LineCoarse p = line_coarse(G, 2 + (m->a[0] ? 1 : 0) + (m->a2[0] ? 1 : 0), 6);
    if (cells(G) <= 64L * NT && p.lds)
      hipLaunchKernelGGL(k_mg_line_coarse, dim3(1), dim3(p.threads), p.lds, st, G, m->u[0], m->f[0], m->a[0],
                         m->a2[0], m->d.coarse, line_nmax(G), p.lanes);
    else
      line_sweeps(G, m->u[0], m->f[0], m->a[0], m->a2[0], m->d.coarse, st);
    return;
  }
  sweeps_raw(G, m->u[0], m->f[0], m->a[0], m->a2[0], m->d.coarse, st);
}

void vcycle(gmunu_mg *m, int l, hipStream_t st) {
  if (l == m->ttop[tail_kind(m)]) {
    launch_tail(m, false, st);
    return;
  }
  if (l == 0) {
    coarse_solve(m, st);
    return;
  }
  const MgGeo &G = m->geo[l];
  double *u = m->u[l], *s = m->us[l];
  const double *f = m->f[l], *a = m->a[l], *a2 = m->a2[l];
  const int pre = m->d.pre, post = m->d.post, h0 = (pre + 1) / 2, h1 = (post + 1) / 2;
  if (!s || pre + post < 2) {
    sweeps_raw(G, u, f, a, a2, pre, st);
    coarse_problem(m, l, st);
    vcycle(m, l - 1, st);
    correct(m, l, st);
    sweeps_raw(G, u, f, a, a2, post, st);
    return;
  }
  // an even number of launches in all, so that the field ends where it began:
  // if need be, one pair of sweeps as two launches
  const int odd = (h0 + h1) & 1, more0 = odd && pre >= 2, more1 = odd && !more0;
  rb_sweeps(G, u, s, &m->u[l], f, a, a2, pre, h0 + more0, st);
  coarse_problem(m, l, st);
  vcycle(m, l - 1, st);
  correct(m, l, st);
  rb_sweeps(G, u, s, &m->u[l], f, a, a2, post, h1 + more1, st);
}

void fmg(gmunu_mg *m, hipStream_t st) {
  const int top = m->levels - 1;
  const int tail = m->ttop[tail_kind(m)], bottom = tail < 0 ? 0 : tail;
  for (int l = top; l > bottom; l--) coarse_problem(m, l, st);
  if (tail >= 0)
    launch_tail(m, true, st);
  else
    coarse_solve(m, st);
  for (int l = bottom + 1; l <= top; l++) {
    correct(m, l, st);
    vcycle(m, l, st);
  }
}

// The finest-level residual norm's kernels: the result lands in
// part[kNormParts].
void norm_enqueue(gmunu_mg *m, hipStream_t st) {
  const int top = m->levels - 1;
  const MgGeo &G = m->geo[top];
  const long nb = nblocks(cells(G));
  int np = (int)(nb < kNormParts ? nb : kNormParts);
  if (G.ndim > 1)
    np = residual<0>(G, m->u[top], m->f[top], m->a[top], m->a2[top], G, nullptr, nullptr, m->part, st);
  else
    hipLaunchKernelGGL(k_mg_norm, dim3(np), dim3(NT), 0, st, G, m->u[top], m->f[top], m->a[top], m->a2[top],
                       m->part);
  hipLaunchKernelGGL(k_mg_norm_finish, dim3(1), dim3(NT), 0, st, m->part, np);
}

int norm(gmunu_mg *m, double *out, hipStream_t st) {
  norm_enqueue(m, st);
  if (hipMemcpyAsync(out, m->part + kNormParts, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return GMUNU_EHIP;
  return launch_status();
}

// Bind the caller's finest-level arrays and restrict a and a2 to the coarse
// levels.
void bind(gmunu_mg *m, double *u, const double *f, const double *a, const double *a2, hipStream_t st) {
  const int top = m->levels - 1;
  m->u[top] = u;
  m->f[top] = const_cast<double *>(f);
  m->a[top] = const_cast<double *>(a);
  m->a2[top] = const_cast<double *>(a2);
  for (int l = top; l > 0; l--) {
    m->a[l - 1] = a ? m->aown[l - 1] : nullptr;
    m->a2[l - 1] = a2 ? m->a2own[l - 1] : nullptr;
    if (a)
      hipLaunchKernelGGL(k_mg_restrict, dim3(nblocks(cells(m->geo[l - 1]))), dim3(NT), 0, st, m->geo[l],
                         m->geo[l - 1], m->a[l], m->a[l - 1]);
    if (a2)
      hipLaunchKernelGGL(k_mg_restrict, dim3(nblocks(cells(m->geo[l - 1]))), dim3(NT), 0, st, m->geo[l],
                         m->geo[l - 1], m->a2[l], m->a2[l - 1]);
  }
}

// n doubles of device memory.  A refusal is the caller's to answer: it does not
// stay behind as the error that the next launch_status reports.
bool try_alloc(size_t n, double **out) {
  if (hipMalloc(out, n * sizeof(double)) == hipSuccess) return true;
  (void)hipGetLastError();
  *out = nullptr;
  return false;
}

// The second field of the finest level (without memory for it the level is
// relaxed in place).
void second_field(gmunu_mg *m) {
  const int top = m->levels - 1;
  const MgGeo &G = m->geo[top];
  double *p = nullptr;
  if (m->us[top] || !rb_level(G) || !try_alloc(G.nt, &p)) return;
  m->owned.push_back(p);
  m->us[top] = p;
}

// a2 is accepted only by a hierarchy whose equation has the second term.
bool a2_ok(const gmunu_mg *m, const double *a2) { return !a2 || (m->d.power2 != 0 && aligned8(a2)); }

bool ok_ptr(const void *p) { return p && aligned8(p); }

// The vector equations: Cartesian grids, or axisymmetric cylindrical and
// spherical ones (at most two active axes), faces Dirichlet, Neumann or
// periodic; a spherical grid reaching r = 0 must end at theta = pi/2.
bool vector_ok(const gmunu_mg *m) {
  const gmunu_mg_desc &d = m->d;
  for (int a = 0; a < 3; a++)
    for (int sd = 0; sd < 2; sd++)
      if (d.bc[a][sd] == GMUNU_MG_ROBIN) return false;
  if (d.coord != GMUNU_CART && d.ndim > 2) return false;
  if (d.coord == GMUNU_SPH && std::fabs(d.xmin[0]) < 1e-12 &&
      (d.ndim < 2 || std::fabs(d.xmin[1] + d.n[1] * d.dx[1] - M_PI / 2) > 1e-12))
    return false;
  return true;
}

// ----------------------------------------------- vector-equation cycles

long colour_cells(const MgGeo &G, int c) {
  long n = 1;
  for (int a = 0; a < 3; a++) n *= a < G.ndim ? (G.n[a] - ((c >> a) & 1) + 1) >> 1 : G.n[a];
  return n;
}

// Levels whose vector lines take mgv_line_curv.
bool axisymmetric(const MgGeo &G) { return G.ndim == 2 && G.coord != GMUNU_CART; }

// Sweeps over the 2^ndim colours: two colours per launch (k_mgv_smooth2)
// when a row's half fits in 4 passes of a workgroup, else one per launch.
void vsweeps(const MgGeo &G, double *u, const double *f, int sweeps, hipStream_t st) {
  if (G.line) {
    for (int s = 0; s < sweeps; s++)
      for (int ax = 0; ax < G.ndim; ax++) {
        if (G.bc[ax][0] == GMUNU_MG_PERIODIC) continue;
        // 12 doubles per cell in 64 KB: lines of at most 682 cells pair
        // two components
        const int kind = !axisymmetric(G) ? 0 : G.n[ax] <= 682 ? 2 : 1;
        const size_t lds = (kind == 0 ? 6 : kind == 1 ? 7 : 12) * (size_t)G.n[ax] * sizeof(double);
        auto run = [&](auto kernel, int c) {
          hipLaunchKernelGGL(kernel, dim3(mg_line_count(G, ax, c)), dim3(line_threads(G.n[ax])), lds, st, G, u, f, ax,
                             c);
        };
        for (int c = 0; c < 1 << (G.ndim - 1); c++)
          if (kind == 2)
            run(k_mgv_line<2, 704>, c);
          else if (kind == 1)
            run(k_mgv_line<1, kMaxLine>, c);
          else  // (the general operator's registers spill under the longest lines' bound)
            G.n[ax] <= 512 ? run(k_mgv_line<0, 512>, c) : run(k_mgv_line<0, kMaxLine>, c);
      }
    return;
  }
  const int ncol = 1 << G.ndim;
  const long hx0 = (G.n[0] + 1) >> 1;
  const bool paired = hx0 <= 4L * NT;
  const int rpw = hx0 >= NT ? 1 : (int)(NT / hx0);
  for (int s = 0; s < sweeps; s++)
    for (int c = 0; c < ncol; c += paired ? 2 : 1) {
      if (paired) {
        const long rows = colour_cells(G, c) / ((G.n[0] + 1) >> 1);
        hipLaunchKernelGGL(k_mgv_smooth2, dim3((rows + rpw - 1) / rpw), dim3(NT), 0, st, G, u, f, c >> 1, rpw);
      } else {
        hipLaunchKernelGGL(k_mgv_smooth, dim3(nblocks(colour_cells(G, c))), dim3(NT), 0, st, G, u, f, c);
      }
    }
}

// One sweep out of place (k_mgv_planes): u to out.
void vsweep_planes(const MgGeo &G, const double *u, double *out, const double *f, hipStream_t st) {
  const int tiles = ((G.n[0] + kPlX - 1) / kPlX) * ((G.n[1] + kPlY - 1) / kPlY);
  if (G.ndim == 2) {
    hipLaunchKernelGGL(k_mgv_planes<2>, dim3(tiles), dim3(3 * kPlQuads), 0, st, G, u, u, f, out, 0);
    return;
  }
  hipLaunchKernelGGL(k_mgv_planes<3>, dim3(tiles * ((G.n[2] + 1) / 2)), dim3(3 * kPlQuads), 0, st, G, u, u, f, out, 0);
  if (G.n[2] > 1)
    hipLaunchKernelGGL(k_mgv_planes<3>, dim3(tiles * (G.n[2] / 2)), dim3(3 * kPlQuads), 0, st, G, u, out, f, out, 1);
}

// `sweeps` sweeps of field u, alternating with the second field s (null: in
// place); *cur: the field that holds the current values, u or s.
void vsweeps_alt(const MgGeo &G, double *u, double *s, double **cur, const double *f, int sweeps, hipStream_t st) {
  if (!s) {
    vsweeps(G, u, f, sweeps, st);
    return;
  }
  for (int n = 0; n < sweeps; n++) {
    double *next = *cur == u ? s : u;
    vsweep_planes(G, *cur, next, f, st);
    *cur = next;
  }
}

void vghosts(const MgGeo &G, double *u, hipStream_t st) {
  const long gc = ghost_count(G);
  if (gc) hipLaunchKernelGGL(k_mg_ghosts<3>, dim3(nblocks(gc)), dim3(NT), 0, st, G, u);
}

void vcoarse_problem(gmunu_mg *m, int l, hipStream_t st) {
  const MgGeo &F = m->geo[l], &C = m->geo[l - 1];
  hipLaunchKernelGGL(k_mgv_restrict_res, dim3(nblocks(cells(C) << F.ndim)), dim3(NT), 0, st, F, C, m->vu[l], m->vf[l],
                     m->vu[l - 1], m->vr[l - 1]);
  hipLaunchKernelGGL(k_mgv_fas_rhs, dim3(nblocks(cells(C))), dim3(NT), 0, st, C, m->vu[l - 1], m->vr[l - 1],
                     m->vf[l - 1], m->vuo[l - 1]);
}

void vcorrect(gmunu_mg *m, int l, hipStream_t st) {
  const MgGeo &F = m->geo[l], &C = m->geo[l - 1];
  hipLaunchKernelGGL(k_mg_correct<3>, dim3(nblocks(cells(C)), 3), dim3(NT), 0, st, C, F, m->vu[l - 1], m->vuo[l - 1],
                     m->vu[l]);
}

void vcoarse_solve(gmunu_mg *m, hipStream_t st) {
  const MgGeo &G = m->geo[0];
  if (G.line) {
    const LineCoarse p = line_coarse(G, 6, 12, axisymmetric(G) ? kCoarseLineThreads : 512);
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(1), dim3(p.threads), p.lds, st, G, m->vu[0], m->vf[0], m->d.coarse,
                         line_nmax(G), p.lanes);
    };
    if (cells(G) <= 64L * NT && p.lds)
      axisymmetric(G) ? run(k_mgv_line_coarse<2>) : run(k_mgv_line_coarse<0>);
    else
      vsweeps(G, m->vu[0], m->vf[0], m->d.coarse, st);
    return;
  }
  if (cells(G) <= 64L * NT) {
    const long bytes = 6 * G.nt * (long)sizeof(double);
    const int lds = bytes <= kCoarseLds;
    hipLaunchKernelGGL(k_mgv_coarse, dim3(1), dim3(NT), lds ? bytes : 0, st, G, m->vu[0], m->vf[0], m->d.coarse,
                       lds);
  } else
    vsweeps(G, m->vu[0], m->vf[0], m->d.coarse, st);
}

void launch_vtail(gmunu_mg *m, bool use_fmg, hipStream_t st) {
  const MgGeo &G = m->geo[m->vtop];
  const long waves = (colour_cells(G, 0) + 20) / 21;  // 21 cells of one colour per wavefront
  hipLaunchKernelGGL(k_mgv_tail, dim3(1), dim3(64 * waves), 0, st, m->vplan, m->vu[m->vtop], m->vf[m->vtop],
                     use_fmg ? 1 : 0);
}

void vvcycle(gmunu_mg *m, int l, hipStream_t st) {
  if (l == m->vtop) {
    launch_vtail(m, false, st);
    return;
  }
  if (l == 0) {
    vcoarse_solve(m, st);
    return;
  }
  // an odd number of sweeps: one in place, so that the field ends where it began
  const MgGeo &G = m->geo[l];
  double *u = m->vu[l], *s = m->vs[l];
  const int odd = s && ((m->d.pre + m->d.post) & 1) ? 1 : 0, in_pre = odd && m->d.pre > 0;
  vsweeps(G, u, m->vf[l], in_pre, st);
  vsweeps_alt(G, u, s, &m->vu[l], m->vf[l], m->d.pre - in_pre, st);
  vcoarse_problem(m, l, st);
  vvcycle(m, l - 1, st);
  vcorrect(m, l, st);
  if (odd && !in_pre) vsweeps(G, m->vu[l], m->vf[l], 1, st);
  vsweeps_alt(G, u, s, &m->vu[l], m->vf[l], m->d.post - (odd && !in_pre), st);
}

void vfmg(gmunu_mg *m, hipStream_t st) {
  const int top = m->levels - 1, bottom = m->vtop < 0 ? 0 : m->vtop;
  for (int l = top; l > bottom; l--) vcoarse_problem(m, l, st);
  if (m->vtop >= 0)
    launch_vtail(m, true, st);
  else
    vcoarse_solve(m, st);
  for (int l = bottom + 1; l <= top; l++) {
    vcorrect(m, l, st);
    vvcycle(m, l, st);
  }
}

int vnorm(gmunu_mg *m, double *out, hipStream_t st) {
  const int top = m->levels - 1;
  const MgGeo &G = m->geo[top];
  const long nb = nblocks(cells(G));
  const int np = (int)(nb < kNormParts ? nb : kNormParts);
  hipLaunchKernelGGL(k_mgv_norm, dim3(np), dim3(NT), 0, st, G, m->vu[top], m->vf[top], m->part);
  hipLaunchKernelGGL(k_mg_norm_finish, dim3(1), dim3(NT), 0, st, m->part, np);
  if (hipMemcpyAsync(out, m->part + kNormParts, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return GMUNU_EHIP;
  return launch_status();
}

bool alloc_zeroed(gmunu_mg *m, size_t n, double **out) {
  double *p = nullptr;
  if (!try_alloc(n, &p)) return false;
  if (hipMemset(p, 0, n * sizeof(double)) != hipSuccess) {
    (void)hipFree(p);
    return false;
  }
  m->owned.push_back(p);
  *out = p;
  return true;
}

bool vector_storage(gmunu_mg *m) {
  if (m->vready) return true;
  for (int l = 0; l < m->levels - 1; l++) {
    const size_t n = 3 * (size_t)m->geo[l].nt;
    // (after a failure the next call goes on where this one stopped)
    for (double **p : {&m->vu[l], &m->vf[l], &m->vr[l], &m->vuo[l]})
      if (!*p && !alloc_zeroed(m, n, p)) return false;
  }
  // second fields of the levels above the tail; without memory for one the
  // level is relaxed in place
  for (int l = m->vtop + 1; l < m->levels; l++)
    if (m->d.coord == GMUNU_CART && m->d.ndim > 1 && !m->geo[l].line && !m->vs[l])
      (void)alloc_zeroed(m, 3 * (size_t)m->geo[l].nt, &m->vs[l]);
  m->vready = true;
  return true;
}

// Magic multiplier of the division by v (mg_div).
unsigned magic_of(int v) { return v == 1 ? 0u : (unsigned)(0x100000000ull / (unsigned)v) + 1u; }

// The programs of a tail up to level `top`: a V-cycle, and the FMG cycle.
template <typename Tail>
void tail_program(const gmunu_mg_desc &d, Tail &T) {
  enum { kPre, kPost, kCoarse };
  T.sweeps[kPre] = d.pre;
  T.sweeps[kPost] = d.post;
  T.sweeps[kCoarse] = d.coarse;
  auto put = [&](int f, int op, int l, int which) {
    if (op != kOpSweep || T.sweeps[which]) T.prog[f][T.nprog[f]++] = op + 4 * l + 64 * which;
  };
  auto vcycle_at = [&](int f, int lt) {
    for (int l = lt; l > 0; l--) {
      put(f, kOpSweep, l, kPre);
      put(f, kOpCoarse, l, 0);
    }
    put(f, kOpSweep, 0, kCoarse);
    for (int l = 1; l <= lt; l++) {
      put(f, kOpCorrect, l, 0);
      put(f, kOpSweep, l, kPost);
    }
  };
  vcycle_at(0, T.top);
  for (int l = T.top; l > 0; l--) put(1, kOpCoarse, l, 0);
  put(1, kOpSweep, 0, kCoarse);
  for (int l = 1; l <= T.top; l++) {
    put(1, kOpCorrect, l, 0);
    vcycle_at(1, l);
  }
}

// The plan of the tail for an equation with (kind bit 0) a and (bit 1) a2:
// the largest level whose tail fits the LDS, -1 if none does.
int tail_plan(const gmunu_mg *m, int kind, MgTail &T) {
  std::memset(&T, 0, sizeof T);
  const gmunu_mg_desc &d = m->d;
  T.ndim = d.ndim;
  T.coord = d.coord;
  T.power = d.power;
  T.power2 = d.power2;
  T.offset = d.offset;
  // u, f, a, a2 of every level and uo below the top, small levels first
  long at = 0;
  T.top = -1;
  for (int l = 0; l < m->levels && l < kTailLevels && cells(m->geo[l]) <= kTailCells; l++) {
    const MgGeo &G = m->geo[l];
    if ((long)((G.n[0] + 1) / 2) * G.n[1] * G.n[2] > kTailSlots * kTailThreads) break;
    MgLev &V = T.lev[l];
    const int nc = (int)cells(G);
    for (int a = 0; a < 3; a++) {
      V.n[a] = G.n[a];
      V.per[a] = a < G.ndim && G.bc[a][0] == GMUNU_MG_PERIODIC;
      V.w[a] = G.coord == GMUNU_CART ? G.vih2[a] : G.ih2_2;
      V.x0[a] = G.x0[a];
      V.h[a] = G.h[a];
      for (int sd = 0; sd < 2 && a < G.ndim; sd++) {
        V.fac[a][sd] = G.bc[a][sd] == GMUNU_MG_DIRICHLET ? -1.0 : 1.0;
        if (G.bc[a][sd] != GMUNU_MG_ROBIN) continue;
        if (G.coord == GMUNU_SPH)
          V.fac[a][sd] = sd ? G.rob_hi : G.rob_lo;
        else
          V.rob |= 1u << (2 * a + sd);
      }
    }
    V.s2 = G.n[0] * G.n[1];
    V.nc = (G.n[0] + 1) / 2 * G.n[1] * G.n[2];
    V.cells = nc;
    V.mh = magic_of((G.n[0] + 1) / 2);
    V.mn0 = magic_of(G.n[0]);
    V.mn1 = magic_of(G.n[1]);
    long p = at;
    auto take = [&p](long n) {
      p += n;
      return (int)(p - n);
    };
    V.u = take(nc);
    V.f = take(nc);
    V.a = kind & 1 ? take(nc) : -1;
    V.a2 = kind & 2 ? take(nc) : -1;
    V.tab = G.coord == GMUNU_CART ? 0 : take(5 * (G.n[0] + 2) + 4 * (G.n[1] + 2));
    if (p > kTailLds) break;
    T.top = l;
    V.uo = take(nc);  // used when a level above belongs to the tail too
    at = p;
  }
  if (T.top >= 0) tail_program(d, T);
  return T.top;
}

// The vector equations' plan (-1: the coarsest level is too large).
int vtail_plan(const gmunu_mg *m, MgvTail &T) {
  std::memset(&T, 0, sizeof T);
  T.ndim = m->d.ndim;
  T.top = -1;
  int at = 0;
  for (int l = 0; l < m->levels && l < kTailLevels && cells(m->geo[l]) <= kVTailCells; l++) {
    const MgGeo &G = m->geo[l];
    const int nc = (int)cells(G);
    // 21 cells of one colour per wavefront; u, f and uo of three components
    if ((colour_cells(G, 0) + 20) / 21 > kTailThreads / 64 || at + 6 * nc > kVTailCells * 11) break;
    MgvLev &V = T.lev[l];
    for (int a = 0; a < 3; a++) {
      V.n[a] = G.n[a];
      V.per[a] = a < G.ndim && G.bc[a][0] == GMUNU_MG_PERIODIC;
      for (int sd = 0; sd < 2; sd++) V.odd[a][sd] = a < G.ndim && !V.per[a] ? G.vodd[a][sd] : 0u;
      V.w[a] = G.vih2[a];
      V.mix[a] = G.vmix[a];
      V.idg[a] = G.vidg[a];
    }
    V.s2 = G.n[0] * G.n[1];
    V.cells = nc;
    V.mn0 = magic_of(G.n[0]);
    V.mn1 = magic_of(G.n[1]);
    V.u = at;
    V.f = at + 3 * nc;
    V.uo = at + 6 * nc;  // used when a level above belongs to the tail too
    at += 9 * nc;
    T.top = l;
  }
  if (T.top >= 0) tail_program(m->d, T);
  return T.top;
}

// The tail's plans, geometries and array pointers, uploaded once.
bool tail_plans(gmunu_mg *m) {
  std::vector<MgTail> T(4);
  int top = -1;
  for (int k = 0; k < 4; k++) {
    if ((k & 2) && !m->d.power2) continue;
    m->ttop[k] = tail_plan(m, k, T[k]);
    top = m->ttop[k] > top ? m->ttop[k] : top;
  }
  MgvTail V;
  std::memset(&V, 0, sizeof V);
  if (m->d.coord == GMUNU_CART) m->vtop = vtail_plan(m, V);
  if (top < 0) return true;
  std::vector<double *> ptr(2 * kTailLevels, nullptr);
  for (int l = 0; l <= top && l < m->levels - 1; l++) {
    ptr[l] = m->aown[l];
    ptr[kTailLevels + l] = m->a2own[l];
  }
  // one upload: the plans, the levels' geometries, the array pointers
  const size_t b0 = T.size() * sizeof(MgTail), b1 = b0 + sizeof(MgvTail), b2 = b1 + (top + 1) * sizeof(MgGeo);
  std::vector<char> buf(b2 + ptr.size() * sizeof(double *));
  std::memcpy(buf.data(), T.data(), b0);
  std::memcpy(buf.data() + b0, &V, sizeof V);
  std::memcpy(buf.data() + b1, m->geo, (top + 1) * sizeof(MgGeo));
  std::memcpy(buf.data() + b2, ptr.data(), ptr.size() * sizeof(double *));
  char *p = nullptr;
  if (hipMalloc(&p, buf.size()) != hipSuccess) return false;
  m->owned.push_back(reinterpret_cast<double *>(p));
  if (hipMemcpy(p, buf.data(), buf.size(), hipMemcpyHostToDevice) != hipSuccess) return false;
  m->tplan = reinterpret_cast<MgTail *>(p);
  m->vplan = reinterpret_cast<MgvTail *>(p + b0);
  m->tgeo = reinterpret_cast<MgGeo *>(p + b1);
  m->tptr = reinterpret_cast<double **>(p + b2);
  return true;
}

// ------------------------------------------------- solve driver

// The private stream is ordered after the caller's work on entry and the
// caller's stream after the private one on exit.
int enter(gmunu_mg *m, hipStream_t cst) {
  if (!m->gs && hipStreamCreateWithFlags(&m->gs, hipStreamNonBlocking) != hipSuccess) return GMUNU_EHIP;
  if (!m->ev && hipEventCreateWithFlags(&m->ev, hipEventDisableTiming) != hipSuccess) return GMUNU_EHIP;
  if (hipEventRecord(m->ev, cst) != hipSuccess || hipStreamWaitEvent(m->gs, m->ev, 0) != hipSuccess)
    return GMUNU_EHIP;
  return GMUNU_OK;
}

int leave(gmunu_mg *m, hipStream_t cst) {
  if (hipEventRecord(m->ev, m->gs) != hipSuccess || hipStreamWaitEvent(cst, m->ev, 0) != hipSuccess)
    return GMUNU_EHIP;
  return launch_status();
}

// The graph of one V-cycle over the bound arrays: a cached one, else
// captured now into the least recently made slot (launches only: no
// memset, no host synchronisation inside).
hipGraphExec_t cycle_graph(gmunu_mg *m, bool vec, const double *u, const double *f, const double *a,
                           const double *a2) {
  for (auto &sl : m->slot)
    if (sl.exec && sl.vec == vec && sl.u == u && sl.f == f && sl.a == a && sl.a2 == a2) return sl.exec;
  auto &sl = m->slot[m->next_slot];
  m->next_slot = (m->next_slot + 1) % 4;
  if (sl.exec) {
    (void)hipGraphExecDestroy(sl.exec);
    sl.exec = nullptr;
  }
  hipStream_t st = m->gs;
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) return nullptr;
  if (vec)
    vvcycle(m, m->levels - 1, st);
  else
    vcycle(m, m->levels - 1, st);
  if (hipStreamEndCapture(st, &g) != hipSuccess) return nullptr;
  const bool ok = hipGraphInstantiate(&sl.exec, g, nullptr, nullptr, 0) == hipSuccess;
  (void)hipGraphDestroy(g);
  if (!ok) {
    sl.exec = nullptr;
    return nullptr;
  }
  sl.vec = vec;
  sl.u = u;
  sl.f = f;
  sl.a = a;
  sl.a2 = a2;
  return sl.exec;
}

// Cycles until the norm is at most tol (arrays bound); the first one an FMG
// cycle when use_fmg.
int cycles(gmunu_mg *m, bool vec, hipGraphExec_t exec, double tol, int max_cycles, int use_fmg, double *res_host,
           int *cycles_out) {
  hipStream_t st = m->gs;
  double r;
  int rc = vec ? vnorm(m, &r, st) : norm(m, &r, st);
  if (rc) return rc;
  if (res_host) res_host[0] = r;
  int c = 0;
  while (c < max_cycles && r > tol) {
    if (c == 0 && use_fmg) {
      if (vec)
        vfmg(m, st);
      else
        fmg(m, st);
    } else if (hipGraphLaunch(exec, st) != hipSuccess) {
      return GMUNU_EHIP;
    }
    c++;
    rc = vec ? vnorm(m, &r, st) : norm(m, &r, st);
    if (rc) return rc;
    if (res_host) res_host[c] = r;
  }
  if (cycles_out) *cycles_out = c;
  return GMUNU_OK;
}

}  // namespace

// --------------------------------------------------------------------- API

extern "C" {

int gmunu_mg_create(const gmunu_mg_desc *desc, gmunu_mg **out) {
  if (!desc || !out) return GMUNU_ENULL;
  const int levels = desc->levels > 0 ? desc->levels : auto_levels(*desc);
  int rc = validate(*desc, levels);
  if (rc) return rc;
  gmunu_mg *m = new (std::nothrow) gmunu_mg();
  if (!m) return GMUNU_ENOMEM;
  m->d = *desc;
  m->levels = levels;
  std::vector<double> tab;
  size_t off[kMaxLevels][11];
  for (int l = 0; l < levels; l++) level_tables(*desc, levels - 1 - l, tab, off[l], m->geo[l]);
  m->br = nullptr;
  m->xs = nullptr;
  for (auto v : {m->vu, m->vf, m->vr, m->vuo})
    for (int l = 0; l < kMaxLevels; l++) v[l] = nullptr;
  for (int &t : m->ttop) t = -1;
  m->tplan = nullptr;
  m->tgeo = nullptr;
  m->tptr = nullptr;
  m->vtop = -1;
  m->vplan = nullptr;
  for (double *&v : m->us) v = nullptr;
  m->vready = false;
  for (double *&v : m->vs) v = nullptr;
  m->gs = nullptr;
  m->ev = nullptr;
  for (auto &sl : m->slot) sl = gmunu_mg::Slot{nullptr, false, nullptr, nullptr, nullptr, nullptr};
  m->next_slot = 0;
  // one allocation: the tables, the norm's partials, then the zeroed level
  // arrays (ghosts of coarse arrays are then defined): u, f, a, r (restricted
  // residual), uo (restricted u), a2 and second field of the coarse levels, uo of the finest
  // (the cleaning's divergence when the caller passes none)
  size_t at = 0;
  auto take = [&at](size_t n) {
    at = (at + 31) / 32 * 32;
    at += n;
    return at - n;
  };
  const size_t tab_at = take(tab.size()), part_at = take(kNormParts + 1 + kGateSlots), zero_at = take(0);
  size_t arr_at[kMaxLevels][7];
  for (int l = 0; l < levels; l++)
    for (int q = 0; q < 6; q++) {
      if (q == 0 || (l < levels - 1 && (q < 5 || desc->power2 != 0)))
        arr_at[l][q] = take(m->geo[l].nt);
      else
        arr_at[l][q] = SIZE_MAX;
    }
  const size_t without = at;
  for (int l = 0; l < levels; l++)
    arr_at[l][6] = l < levels - 1 && rb_level(m->geo[l]) ? take(m->geo[l].nt) : SIZE_MAX;
  double *p = nullptr;
  bool ok = try_alloc(at, &p);
  if (!ok && at > without) {  // without memory for the second fields their levels are relaxed in place
    at = without;
    for (int l = 0; l < levels; l++) arr_at[l][6] = SIZE_MAX;
    ok = try_alloc(at, &p);
  }
  if (ok) m->owned.push_back(p);
  m->tab = p + tab_at;
  m->part = p + part_at;
  for (int l = 0; l < levels; l++) {
    const bool coarse = l < levels - 1;
    m->uo[l] = p + arr_at[l][0];
    m->u[l] = coarse ? p + arr_at[l][1] : nullptr;
    m->f[l] = coarse ? p + arr_at[l][2] : nullptr;
    m->aown[l] = coarse ? p + arr_at[l][3] : nullptr;
    m->r[l] = coarse ? p + arr_at[l][4] : nullptr;
    m->a2own[l] = coarse && desc->power2 != 0 ? p + arr_at[l][5] : nullptr;
    m->us[l] = arr_at[l][6] != SIZE_MAX ? p + arr_at[l][6] : nullptr;
  }
  ok = ok && hipMemcpy(m->tab, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice) == hipSuccess &&
       hipMemset(p + zero_at, 0, (at - zero_at) * sizeof(double)) == hipSuccess &&
       hipDeviceSynchronize() == hipSuccess;
  if (!ok) {
    for (double *q : m->owned) (void)hipFree(q);
    delete m;
    return GMUNU_ENOMEM;
  }
  for (int l = 0; l < levels; l++) {
    MgGeo &G = m->geo[l];
    const double *b = m->tab;
    G.a0m = b + off[l][0];
    G.a0p = b + off[l][1];
    G.g1 = b + off[l][2];
    G.g2 = b + off[l][3];
    G.vol0 = b + off[l][4];
    G.sg0 = b + off[l][5];
    G.a1m = b + off[l][6];
    G.a1p = b + off[l][7];
    G.s2t = b + off[l][8];
    G.vol1 = b + off[l][9];
    G.sg1 = b + off[l][10];
  }
  if (!m->geo[levels - 1].line && !tail_plans(m)) {
    for (double *p : m->owned) (void)hipFree(p);
    delete m;
    return GMUNU_ENOMEM;
  }
  *out = m;
  return GMUNU_OK;
}

int gmunu_mg_destroy(gmunu_mg *m) {
  if (!m) return GMUNU_ENULL;
  int rc = GMUNU_OK;
  for (auto &sl : m->slot)
    if (sl.exec && hipGraphExecDestroy(sl.exec) != hipSuccess) rc = GMUNU_EHIP;
  if (m->ev && hipEventDestroy(m->ev) != hipSuccess) rc = GMUNU_EHIP;
  if (m->gs && hipStreamDestroy(m->gs) != hipSuccess) rc = GMUNU_EHIP;
  for (double *p : m->owned)
    if (hipFree(p) != hipSuccess) rc = GMUNU_EHIP;
  delete m;
  return rc;
}

int gmunu_mg_levels(const gmunu_mg *m) { return m ? m->levels : GMUNU_ENULL; }

long gmunu_mg_size(const gmunu_mg *m, int level) {
  if (!m || level < 0 || level >= m->levels) return -1;
  return m->geo[level].nt;
}

int gmunu_mg_solve(gmunu_mg *m, double *u, const double *f, const double *a, const double *a2, double tol,
                   int max_cycles, int use_fmg, double *res_host, int *cycles_out, void *stream) {
  if (!m || !u || !f) return GMUNU_ENULL;
  if (!ok_ptr(u) || !ok_ptr(f) || (a && !aligned8(a))) return GMUNU_EALIGN;
  if (max_cycles < 0 || !(tol >= 0.0) || !a2_ok(m, a2)) return GMUNU_EINVAL;
  // the cycles run on the context's stream, ordered after the caller's work
  hipStream_t cst = as_stream(stream);
  int rc = enter(m, cst);
  if (rc) return rc;
  second_field(m);
  bind(m, u, f, a, a2, m->gs);
  hipGraphExec_t exec = cycle_graph(m, false, u, f, a, a2);
  if (!exec) return GMUNU_EHIP;
  rc = cycles(m, false, exec, tol, max_cycles, use_fmg, res_host, cycles_out);
  if (rc) return rc;
  ghosts(m->geo[m->levels - 1], u, m->gs);
  return leave(m, cst);
}

int gmunu_mg_residual_norm(gmunu_mg *m, double *u, const double *f, const double *a, const double *a2,
                           double *norm_out, void *stream) {
  if (!m || !u || !f || !norm_out) return GMUNU_ENULL;
  if (!ok_ptr(u) || !ok_ptr(f) || (a && !aligned8(a))) return GMUNU_EALIGN;
  if (!a2_ok(m, a2)) return GMUNU_EINVAL;
  hipStream_t st = as_stream(stream);
  const int top = m->levels - 1;
  m->u[top] = u;
  m->f[top] = const_cast<double *>(f);
  m->a[top] = const_cast<double *>(a);
  m->a2[top] = const_cast<double *>(a2);
  return norm(m, norm_out, st);
}

int gmunu_mg_apply(gmunu_mg *m, const double *u, const double *a, const double *a2, double *out, void *stream) {
  if (!m || !u || !out) return GMUNU_ENULL;
  if (!ok_ptr(u) || !ok_ptr(out) || (a && !aligned8(a))) return GMUNU_EALIGN;
  if (!a2_ok(m, a2)) return GMUNU_EINVAL;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mg_apply, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, u, a, a2, out);
  return launch_status();
}

int gmunu_mg_fill_ghosts(gmunu_mg *m, int level, double *u, void *stream) {
  if (!m || !u) return GMUNU_ENULL;
  if (!aligned8(u)) return GMUNU_EALIGN;
  if (level < 0 || level >= m->levels) return GMUNU_EINVAL;
  ghosts(m->geo[level], u, as_stream(stream));
  return launch_status();
}

int gmunu_mg_smooth(gmunu_mg *m, double *u, const double *f, const double *a, const double *a2, int sweeps,
                    void *stream) {
  if (!m || !u || !f) return GMUNU_ENULL;
  if (!ok_ptr(u) || !ok_ptr(f) || (a && !aligned8(a))) return GMUNU_EALIGN;
  if (sweeps < 0 || !a2_ok(m, a2)) return GMUNU_EINVAL;
  hipStream_t st = as_stream(stream);
  const MgGeo &G = m->geo[m->levels - 1];
  // out of place only on large levels: smaller ones are relaxed on the caller's
  // arrays alone, so that calls on different arrays may overlap
  const bool large = cells(G) >= 32768 && G.n[0] >= 16;
  if (large) second_field(m);
  rb_sweeps_back(G, u, large ? m->us[m->levels - 1] : nullptr, f, a, a2, sweeps, st);
  ghosts(G, u, st);
  return launch_status();
}

int gmunu_mg_restrict(gmunu_mg *m, int level, const double *fine, double *coarse, void *stream) {
  if (!m || !fine || !coarse) return GMUNU_ENULL;
  if (!ok_ptr(fine) || !ok_ptr(coarse)) return GMUNU_EALIGN;
  if (level < 1 || level >= m->levels) return GMUNU_EINVAL;
  const MgGeo &C = m->geo[level - 1];
  hipLaunchKernelGGL(k_mg_restrict, dim3(nblocks(cells(C))), dim3(NT), 0, as_stream(stream), m->geo[level], C, fine,
                     coarse);
  return launch_status();
}

int gmunu_mg_prolong(gmunu_mg *m, int level, const double *coarse, double *fine, void *stream) {
  if (!m || !fine || !coarse) return GMUNU_ENULL;
  if (!ok_ptr(fine) || !ok_ptr(coarse)) return GMUNU_EALIGN;
  if (level < 1 || level >= m->levels) return GMUNU_EINVAL;
  const MgGeo &F = m->geo[level];
  hipLaunchKernelGGL(k_mg_prolong, dim3(nblocks(cells(F))), dim3(NT), 0, as_stream(stream), m->geo[level - 1], F,
                     coarse, fine, 0);
  return launch_status();
}

int gmunu_mg_divergence(gmunu_mg *m, const double *q, double *div, void *stream) {
  if (!m || !q || !div) return GMUNU_ENULL;
  if (!ok_ptr(q) || !ok_ptr(div)) return GMUNU_EALIGN;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mg_div, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, q, div);
  return launch_status();
}

int gmunu_mg_subtract_gradient(gmunu_mg *m, const double *phi, double *q, void *stream) {
  if (!m || !q || !phi) return GMUNU_ENULL;
  if (!ok_ptr(q) || !ok_ptr(phi)) return GMUNU_EALIGN;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mg_subgrad, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, phi, q);
  return launch_status();
}

int gmunu_mg_clean(gmunu_mg *m, double *q, double *phi, double *div, double tol, int max_cycles, double *res_host,
                   int *cycles_out, void *stream) {
  if (!m || !q || !phi) return GMUNU_ENULL;
  if (m->d.power != 0) return GMUNU_EINVAL;
  if (!ok_ptr(q) || !ok_ptr(phi) || (div && !aligned8(div))) return GMUNU_EALIGN;
  const int top = m->levels - 1;
  // the divergence goes into the caller's div, else into the finest uo buffer
  double *f = div ? div : m->uo[top];
  int rc = gmunu_mg_divergence(m, q, f, stream);
  if (rc) return rc;
  rc = gmunu_mg_solve(m, phi, f, nullptr, nullptr, tol, max_cycles, 1, res_host, cycles_out, stream);
  if (rc) return rc;
  ghosts(m->geo[top], phi, as_stream(stream));
  return gmunu_mg_subtract_gradient(m, phi, q, stream);
}

// ------------------------------------------------ vector equations (xCFC)

int gmunu_mg_vapply(gmunu_mg *m, const double *X, double *out, void *stream) {
  if (!m || !X || !out) return GMUNU_ENULL;
  if (!ok_ptr(X) || !ok_ptr(out)) return GMUNU_EALIGN;
  if (!vector_ok(m)) return GMUNU_EINVAL;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mgv_apply, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, X, out);
  return launch_status();
}

int gmunu_mg_vsmooth(gmunu_mg *m, double *X, const double *f, int sweeps, void *stream) {
  if (!m || !X || !f) return GMUNU_ENULL;
  if (!ok_ptr(X) || !ok_ptr(f)) return GMUNU_EALIGN;
  if (!vector_ok(m) || sweeps < 0) return GMUNU_EINVAL;
  const MgGeo &G = m->geo[m->levels - 1];
  hipStream_t st = as_stream(stream);
  vsweeps(G, X, f, sweeps, st);
  vghosts(G, X, st);
  return launch_status();
}

int gmunu_mg_vsolve(gmunu_mg *m, double *X, const double *f, double tol, int max_cycles, int use_fmg,
                    double *res_host, int *cycles_out, void *stream) {
  if (!m || !X || !f) return GMUNU_ENULL;
  if (!ok_ptr(X) || !ok_ptr(f)) return GMUNU_EALIGN;
  if (!vector_ok(m) || max_cycles < 0 || !(tol >= 0.0)) return GMUNU_EINVAL;
  if (!vector_storage(m)) return GMUNU_ENOMEM;
  hipStream_t cst = as_stream(stream);
  int rc = enter(m, cst);
  if (rc) return rc;
  const int top = m->levels - 1;
  m->vu[top] = X;
  m->vf[top] = const_cast<double *>(f);
  hipGraphExec_t exec = cycle_graph(m, true, X, f, nullptr, nullptr);
  if (!exec) return GMUNU_EHIP;
  rc = cycles(m, true, exec, tol, max_cycles, use_fmg, res_host, cycles_out);
  if (rc) return rc;
  vghosts(m->geo[top], X, m->gs);
  return leave(m, cst);
}

int gmunu_mg_xcfc_aij(gmunu_mg *m, const double *X, double *A6, double *A2, void *stream) {
  if (!m || !X || !A6 || !A2) return GMUNU_ENULL;
  if (!ok_ptr(X) || !ok_ptr(A6) || !ok_ptr(A2)) return GMUNU_EALIGN;
  if (!vector_ok(m)) return GMUNU_EINVAL;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mgv_aij, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, X, A6, A2);
  return launch_status();
}

int gmunu_mg_xcfc_beta_rhs(gmunu_mg *m, const double *w, const double *S, const double *A6, double *out,
                           void *stream) {
  if (!m || !w || !S || !A6 || !out) return GMUNU_ENULL;
  if (!ok_ptr(w) || !ok_ptr(S) || !ok_ptr(A6) || !ok_ptr(out)) return GMUNU_EALIGN;
  if (!vector_ok(m)) return GMUNU_EINVAL;
  const MgGeo &G = m->geo[m->levels - 1];
  hipLaunchKernelGGL(k_mgv_beta_rhs, dim3(nblocks(cells(G))), dim3(NT), 0, as_stream(stream), G, w, S, A6, out);
  return launch_status();
}

}  // extern "C"

namespace {

// The GRMHD layout of a descriptor whose interior is the multigrid's finest
// grid (same dimensions, coordinates, spacing and origin), else EINVAL.
int hydro_of(const gmunu_mg *m, const gmunu_grid_desc *hd, Hydro &H) {
  const gmunu_mg_desc &d = m->d;
  if (hd->ndim != d.ndim || hd->coord != d.coord || hd->ng < 1) return GMUNU_EINVAL;
  long T[3];
  for (int a = 0; a < 3; a++) {
    if (hd->n[a] != d.n[a]) return GMUNU_EINVAL;
    if (a < d.ndim && (std::fabs(hd->dx[a] - d.dx[a]) > 1e-12 * d.dx[a] ||
                       std::fabs(hd->xmin[a] - d.xmin[a]) > 1e-12 * (std::fabs(d.xmin[a]) + d.dx[a])))
      return GMUNU_EINVAL;
    H.ng[a] = a < d.ndim ? hd->ng : 0;
    T[a] = d.n[a] + 2 * H.ng[a];
  }
  H.T0 = T[0];
  H.T1 = T[0] * T[1];
  H.nv = H.T1 * T[2];
  H.gam = hd->gamma;
  return GMUNU_OK;
}

bool bridge_scratch(gmunu_mg *m);

// Steps 3 to 5 of the xCFC sequence (A2 = A~_ij A~^ij, or NULL for the
// scalar CFC equations alone): psi from its equation, S~ with the new psi,
// then alpha psi; psi and alpha written to the metric.  cyc: 2 ints.
int scalar_cfc(gmunu_mg *mpsi, gmunu_mg *malpha, const Hydro &H, const double *q, const double *prim,
               double *metric, const double *A2, double tol, int max_cycles, int *cyc, hipStream_t st) {
  gmunu_mg *ms[2] = {mpsi, malpha};
  const MgGeo &G0 = mpsi->geo[mpsi->levels - 1];
  double *u = mpsi->br, *a = mpsi->br + G0.nt, *f = mpsi->br + 2 * G0.nt, *a2 = mpsi->br + 3 * G0.nt;
  for (int w = 0; w < 2; w++) {
    gmunu_mg *m = ms[w];
    const MgGeo &G = m->geo[m->levels - 1];
    if (hipMemsetAsync(f, 0, (size_t)G0.nt * sizeof(double), st) != hipSuccess) return GMUNU_EHIP;
    hipLaunchKernelGGL(k_br_cfc_coef, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, H, q, prim, metric, w, A2, a, a2,
                       u);
    const int rc = gmunu_mg_solve(m, u, f, a, w == 0 && A2 ? a2 : nullptr, tol, max_cycles, 1, nullptr, &cyc[w],
                                  (void *)st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_br_store, dim3(nblocks(H.nv)), dim3(NT), 0, st, G, H, u, m->d.xmin[0], w, metric);
  }
  return launch_status();
}

bool bridge_scratch(gmunu_mg *m) {
  if (m->br) return true;
  double *p = nullptr;
  if (hipMalloc(&p, 6 * (size_t)m->geo[m->levels - 1].nt * sizeof(double)) != hipSuccess) return false;
  if (hipMemset(p, 0, 6 * (size_t)m->geo[m->levels - 1].nt * sizeof(double)) != hipSuccess) {
    (void)hipFree(p);
    return false;
  }
  m->owned.push_back(p);
  m->br = p;
  return true;
}

}  // namespace

extern "C" {

int gmunu_mg_clean_state(gmunu_mg *m, const gmunu_grid_desc *hydro, double *q, const double *prim,
                         const double *metric, double tol, int max_cycles, double *res_host, int *cycles_out,
                         void *stream) {
  if (!m || !hydro || !q || !prim || !metric) return GMUNU_ENULL;
  if (!aligned8(q) || !aligned8(prim) || !aligned8(metric)) return GMUNU_EALIGN;
  Hydro H;
  int rc = hydro_of(m, hydro, H);
  if (rc) return rc;
  if (m->d.power != 0) return GMUNU_EINVAL;
  if (!bridge_scratch(m)) return GMUNU_ENOMEM;
  const MgGeo &G = m->geo[m->levels - 1];
  hipStream_t st = as_stream(stream);
  double *qb = m->br, *phi = m->br + 3 * G.nt, *div = m->br + 4 * G.nt;
  hipLaunchKernelGGL(k_br_gather_qb, dim3(nblocks(G.nt)), dim3(NT), 0, st, G, H, q, prim, metric, qb);
  if (hipMemsetAsync(phi, 0, (size_t)G.nt * sizeof(double), st) != hipSuccess) return GMUNU_EHIP;
  rc = gmunu_mg_clean(m, qb, phi, div, tol, max_cycles, res_host, cycles_out, stream);
  if (rc) return rc;
  hipLaunchKernelGGL(k_br_scatter_qb, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, H, qb, q);
  return launch_status();
}

int gmunu_mg_cfc_solve(gmunu_mg *mpsi, gmunu_mg *malpha, const gmunu_grid_desc *hydro, const double *q,
                       const double *prim, double *metric, double tol, int max_cycles, int *cycles_out,
                       void *stream) {
  if (!mpsi || !malpha || !hydro || !q || !prim || !metric) return GMUNU_ENULL;
  if (!aligned8(q) || !aligned8(prim) || !aligned8(metric)) return GMUNU_EALIGN;
  Hydro H, H2;
  int rc = hydro_of(mpsi, hydro, H);
  if (!rc) rc = hydro_of(malpha, hydro, H2);
  if (rc) return rc;
  if (mpsi->d.power != -1 || mpsi->d.offset != 1.0 || malpha->d.power != 1 || malpha->d.offset != 1.0)
    return GMUNU_EINVAL;
  if (!bridge_scratch(mpsi)) return GMUNU_ENOMEM;
  int cyc[2] = {0, 0};
  rc = scalar_cfc(mpsi, malpha, H, q, prim, metric, nullptr, tol, max_cycles, cyc, as_stream(stream));
  if (!rc && cycles_out) {
    cycles_out[0] = cyc[0];
    cycles_out[1] = cyc[1];
  }
  return rc;
}

int gmunu_mg_xcfc_solve(gmunu_mg *mvec, gmunu_mg *mpsi, gmunu_mg *malpha, const gmunu_grid_desc *hydro,
                        const double *q, const double *prim, double *metric, double *X, double tol, int max_cycles,
                        int *cycles_out, void *stream) {
  if (!mvec || !mpsi || !malpha || !hydro || !q || !prim || !metric || !X) return GMUNU_ENULL;
  if (!aligned8(q) || !aligned8(prim) || !aligned8(metric) || !aligned8(X)) return GMUNU_EALIGN;
  Hydro H, H2, H3;
  int rc = hydro_of(mpsi, hydro, H);
  if (!rc) rc = hydro_of(malpha, hydro, H2);
  if (!rc) rc = hydro_of(mvec, hydro, H3);
  if (rc) return rc;
  if (!vector_ok(mvec) || mpsi->d.power != -1 || mpsi->d.offset != 1.0 || mpsi->d.power2 != -7 ||
      malpha->d.power != 1 || malpha->d.offset != 1.0)
    return GMUNU_EINVAL;
  if (!bridge_scratch(mpsi) || !vector_storage(mvec)) return GMUNU_ENOMEM;
  const MgGeo &G = mvec->geo[mvec->levels - 1];
  if (!mvec->xs && !alloc_zeroed(mvec, 17 * (size_t)G.nt, &mvec->xs)) return GMUNU_ENOMEM;
  hipStream_t st = as_stream(stream);
  double *S = mvec->xs, *fv = S + 3 * G.nt, *beta = S + 6 * G.nt, *A6 = S + 9 * G.nt, *A2 = S + 15 * G.nt,
         *w = S + 16 * G.nt;
  int cyc[4] = {0, 0, 0, 0};
  // step 1: the vector potential
  hipLaunchKernelGGL(k_bx_src, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, H, q, S, fv);
  rc = gmunu_mg_vsolve(mvec, X, fv, tol, max_cycles, 1, nullptr, &cyc[0], stream);
  if (rc) return rc;
  // step 2: A~^ij
  hipLaunchKernelGGL(k_mgv_aij, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, X, A6, A2);
  // steps 3 to 5: conformal factor and lapse
  rc = scalar_cfc(mpsi, malpha, H, q, prim, metric, A2, tol, max_cycles, &cyc[1], st);
  if (rc) return rc;
  // step 6: the shift
  hipLaunchKernelGGL(k_bx_w, dim3(nblocks(G.nt)), dim3(NT), 0, st, G, H, metric, w);
  hipLaunchKernelGGL(k_mgv_beta_rhs, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, w, S, A6, fv);
  hipLaunchKernelGGL(k_bx_beta_in, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, H, metric, beta);
  rc = gmunu_mg_vsolve(mvec, beta, fv, tol, max_cycles, 1, nullptr, &cyc[3], stream);
  if (rc) return rc;
  for (int c = 0; c < 3; c++)
    hipLaunchKernelGGL(k_br_store, dim3(nblocks(H.nv)), dim3(NT), 0, st, G, H, beta + c * G.nt, mvec->d.xmin[0],
                       2 + c, metric);
  if (cycles_out)
    for (int c = 0; c < 4; c++) cycles_out[c] = cyc[c];
  return launch_status();
}

}  // extern "C"

namespace {

// The kernels of gmunu_mg_psi_residual: the residual lands in
// mpsi->part[kNormParts].
int psi_residual_enqueue(gmunu_mg *mvec, gmunu_mg *mpsi, const gmunu_grid_desc *hydro, const double *q,
                         const double *metric, const double *X, hipStream_t st) {
  if (!mpsi || !hydro || !q || !metric || (mvec && !X)) return GMUNU_ENULL;
  if (!aligned8(q) || !aligned8(metric) || (X && !aligned8(X))) return GMUNU_EALIGN;
  Hydro H;
  int rc = hydro_of(mpsi, hydro, H);
  if (!rc && mvec) rc = hydro_of(mvec, hydro, H);
  if (rc) return rc;
  if (mpsi->d.power != -1 || mpsi->d.offset != 1.0 || (mvec && (!vector_ok(mvec) || mpsi->d.power2 != -7)))
    return GMUNU_EINVAL;
  if (!bridge_scratch(mpsi)) return GMUNU_ENOMEM;
  if (mvec && !mvec->xs && !alloc_zeroed(mvec, 17 * (size_t)mvec->geo[mvec->levels - 1].nt, &mvec->xs))
    return GMUNU_ENOMEM;
  const MgGeo &G = mpsi->geo[mpsi->levels - 1];
  double *u = mpsi->br, *a = mpsi->br + G.nt, *f = mpsi->br + 2 * G.nt, *a2 = mpsi->br + 3 * G.nt;
  const double *A2 = nullptr;
  if (mvec) {
    const MgGeo &V = mvec->geo[mvec->levels - 1];
    double *A2v = mvec->xs + 15 * V.nt;
    hipLaunchKernelGGL(k_mgv_aij, dim3(nblocks(cells(V))), dim3(NT), 0, st, V, X, nullptr, A2v);
    A2 = A2v;
  }
  if (hipMemsetAsync(f, 0, (size_t)G.nt * sizeof(double), st) != hipSuccess) return GMUNU_EHIP;
  // which 0 (the conformal factor) reads no primitives
  hipLaunchKernelGGL(k_br_cfc_coef, dim3(nblocks(cells(G))), dim3(NT), 0, st, G, H, q, nullptr, metric, 0, A2, a, a2,
                     u);
  const int top = mpsi->levels - 1;
  mpsi->u[top] = u;
  mpsi->f[top] = f;
  mpsi->a[top] = a;
  mpsi->a2[top] = A2 ? a2 : nullptr;
  norm_enqueue(mpsi, st);
  return launch_status();
}

__global__ void k_dyn_reset(double *g) {
  g[0] = 0.0;
  g[1] = 0.0;
}

// After step `step` of a chunk: the first step whose residual exceeds eps
// is recorded (g[0]) with the time after it (g[1]), and t becomes +inf, so
// that every later step of the chunk computes dt = 0 (its cap t_end - t,
// t_end finite, is negative) and changes nothing.
__global__ void k_dyn_gate(const double *res, double eps, double step, double *t, double *g) {
  if (g[0] == 0.0 && *res > eps) {
    g[0] = step;
    g[1] = *t;
    *t = INFINITY;
  }
}

__global__ void k_dyn_restore(double *t, const double *g) {
  if (g[0] != 0.0) *t = g[1];
}

}  // namespace

extern "C" {

int gmunu_mg_psi_residual(gmunu_mg *mvec, gmunu_mg *mpsi, const gmunu_grid_desc *hydro, const double *q,
                          const double *metric, const double *X, double *norm_out, void *stream) {
  if (!norm_out) return GMUNU_ENULL;
  hipStream_t st = as_stream(stream);
  const int rc = psi_residual_enqueue(mvec, mpsi, hydro, q, metric, X, st);
  if (rc) return rc;
  if (hipMemcpyAsync(norm_out, mpsi->part + kNormParts, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return GMUNU_EHIP;
  return launch_status();
}

int gmunu_mg_dynamical_steps(gmunu_mg *mvec, gmunu_mg *mpsi, gmunu_ctx *ctx, const gmunu_grid_desc *hydro,
                             double *q_n, double *q_s, double *prim, const double *metric, const double *X,
                             double cfl, double t_end, double *t_dev, double *dt_dev, uint8_t *flags,
                             unsigned int *nfatal_dev, int nsteps, double eps, int *steps_out, int *triggered_out,
                             void *stream) {
  if (!ctx || !mpsi || !hydro || !t_dev || !dt_dev || !steps_out || !triggered_out) return GMUNU_ENULL;
  if (nsteps < 1 || !std::isfinite(t_end)) return GMUNU_EINVAL;
  hipStream_t st = as_stream(stream);
  double *g = mpsi->part + kNormParts + 1;
  hipLaunchKernelGGL(k_dyn_reset, dim3(1), dim3(1), 0, st, g);
  for (int s = 1; s <= nsteps; s++) {
    int rc = gmunu_step(ctx, q_n, q_s, prim, metric, nullptr, cfl, t_end, t_dev, dt_dev, flags, nfatal_dev, stream);
    if (!rc) rc = psi_residual_enqueue(mvec, mpsi, hydro, q_n, metric, X, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_dyn_gate, dim3(1), dim3(1), 0, st, mpsi->part + kNormParts, eps, (double)s, t_dev, g);
  }
  hipLaunchKernelGGL(k_dyn_restore, dim3(1), dim3(1), 0, st, t_dev, g);
  double h[2];
  if (hipMemcpyAsync(h, g, sizeof h, hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
    return GMUNU_EHIP;
  *triggered_out = h[0] != 0.0;
  *steps_out = h[0] != 0.0 ? (int)h[0] : nsteps;
  return launch_status();
}

int gmunu_mg_metric_update(gmunu_mg *mvec, gmunu_mg *mpsi, gmunu_mg *malpha, gmunu_ctx *ctx,
                           const gmunu_grid_desc *hydro, double *q, double *prim, double *metric, double *X,
                           uint8_t *flags, unsigned int *nfatal_dev, double tol, int max_cycles, int *cycles_out,
                           void *stream) {
  if (!ctx || (mvec && !X)) return GMUNU_ENULL;
  int cyc[4] = {0, 0, 0, 0};
  int rc = mvec ? gmunu_mg_xcfc_solve(mvec, mpsi, malpha, hydro, q, prim, metric, X, tol, max_cycles, cyc, stream)
                : gmunu_mg_cfc_solve(mpsi, malpha, hydro, q, prim, metric, tol, max_cycles, cyc + 1, stream);
  if (rc) return rc;
  rc = gmunu_c2p(ctx, q, metric, prim, flags, nfatal_dev, stream);
  if (rc) return rc;
  rc = gmunu_fill_ghosts(ctx, prim, stream);
  if (rc) return rc;
  if (cycles_out)
    for (int c = 0; c < 4; c++) cycles_out[c] = cyc[c];
  return GMUNU_OK;
}

}  // extern "C"
