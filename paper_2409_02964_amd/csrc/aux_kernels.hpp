// aux_kernels.hpp -- set-up and read-out kernels around the fused step:
// field uploads, initial populations, population I/O, macroscopic fields and
// FP64 observables.  None of these is on the per-step path.
//
// Storage convention (see step_kernel.hpp): buffer slot s_i(y) holds the
// post-collision population that the next pull delivers to node y + e_i as
// f_i, or -- when y + e_i lies beyond a wall -- back to node y as f_opp(i).
// Values are f (plain storage) or deviations g = f - f^rest (shifted storage,
// times a power-of-two scale).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "step_kernel.hpp"

namespace vanse_dev {

// Directions of Eq. (5) and their opposites, as constant expressions for
// loops that are unrolled in full: an index that the compiler does not know
// would put the populations of a node into scratch memory.
__device__ constexpr int ex_of(int i) { return int(i == 1 || i == 5 || i == 8) - int(i == 3 || i == 6 || i == 7); }
__device__ constexpr int ey_of(int i) { return int(i == 2 || i == 5 || i == 6) - int(i == 4 || i == 7 || i == 8); }
__device__ constexpr int opp_of(int i) { return i == 0 ? 0 : i < 5 ? (i + 1) % 4 + 1 : (i - 3) % 4 + 5; }

struct Geo {
  int nx, ny, pitch, walls;
  int xwalls;  // half-way walls at x = -1/2 and x = nx - 1/2 as well
  long long plane;
  int nee_lo, nee_hi;  // velocity boundary rows (first / last row), see StepPhys
  double un_lo, un_hi;
};

// Kind of row y: 1 (2) when it is the lower (upper) velocity boundary row.
__device__ __forceinline__ int vel_row_kind(const Geo& G, int y) {
  if (!G.walls) return 0;
  if (G.nee_lo && y == 0) return 1;
  if (G.nee_hi && y == G.ny - 1) return 2;
  return 0;
}

constexpr int NOBS = 5;  // observables per reduction record

// Rest-state population f^rest_i = f^eq_i(rho0, 0) of Eq. (14) at a node
// of void fraction phi.
template <typename T>
__device__ __forceinline__ T rest_pop(int i, T phi, const StepPhys<T>& ph) {
  if (i == 0) return phi * ph.rho0 - ph.rest0_k;
  return (i < 5) ? ph.rest_axis : ph.rest_diag;
}

// Adjusted equilibrium of Eq. (14), written with cs^2 = 1/3 and X = kappa/phi:
// the third-order factor is (3 - X)/2 on the axes and X on the diagonals; 1
// for the second-order equilibrium of Eq. (B1) (eq2).
__device__ inline double feq_pop(int i, double phi, double rho, double ux, double uy,
                                 double kappa, int eq2) {
  const double uu = ux * ux + uy * uy;
  if (i == 0) return phi * rho - 5.0 / 9.0 * kappa * rho - 2.0 / 3.0 * phi * rho * uu;
  const double X = kappa / phi;
  const double eu = ex_of(i) * ux + ey_of(i) * uy;
  const bool axis = i < 5;
  const double w = axis ? 1.0 / 9.0 : 1.0 / 36.0;
  const double h3 = eq2 ? 1.0 : (axis ? 0.5 * (3.0 - X) : X);
  return w * (kappa * rho + phi * rho * (3.0 * eu * h3 + 4.5 * eu * eu - 1.5 * uu));
}

// Moving-wall correction of a population f+_i that crossed the wall at
// y = -1/2 (lo) or y = ny - 1/2 (hi): it returns as f_opp(i) = f+_i - delta,
// delta = f^eq_i - f^eq_opp(i) at (phi, rho0, u_w).
template <typename T>
__device__ inline double wall_delta(int i, T phi, bool lo, const StepPhys<T>& ph) {
  const double uw = double(lo ? ph.uw_lo : ph.uw_hi);
  if (uw == 0.0) return 0.0;
  return feq_pop(i, double(phi), double(ph.rho0), uw, 0.0, double(ph.kappa), ph.eq2) -
         feq_pop(opp_of(i), double(phi), double(ph.rho0), uw, 0.0, double(ph.kappa), ph.eq2);
}

template <typename S, typename T, bool SHIFT>
__device__ __forceinline__ S encode(double f, T phi, int i, const StepPhys<T>& ph) {
  if (SHIFT) return static_cast<S>((static_cast<T>(f - double(rest_pop(i, phi, ph)))) * ph.scale);
  return static_cast<S>(f);
}

template <typename S, typename T, bool SHIFT>
__device__ __forceinline__ double decode(S s, T phi, int i, const StepPhys<T>& ph) {
  if (SHIFT) return double(static_cast<T>(s) * ph.inv_scale) + double(rest_pop(i, phi, ph));
  return double(static_cast<T>(s));
}

// Solid flags of a node (0 without a mask); bit layout as FEAT_MASK.
__device__ __forceinline__ unsigned nbr_at(const Geo& G, const uint16_t* __restrict__ nbr, int x,
                                           int y) {
  return nbr ? unsigned(nbr[(long long)y * G.pitch + x]) : 0u;
}

// Solid flags (FEAT_MASK layout) from a dense uint8 mask, nonzero = solid:
// bit 0 the node, bit i the node standing in for x + e_i, which across a wall
// is its mirror image in the first or last row (or column).  A solid node
// keeps bit 0 alone: nothing it computes is used, and without neighbour bits
// the step's bounce-back and stand-in paths pass over solid regions.  Counts
// solid nodes.
__global__ void build_nbr(Geo G, const uint8_t* __restrict__ mask, uint16_t* __restrict__ nbr,
                          unsigned long long* __restrict__ nsolid) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  unsigned b = mask[(long long)y * G.nx + x] ? 1u : 0u;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    int xn = x + ex_of(i), yn = y + ey_of(i);
    if (G.xwalls) xn = xn < 0 ? -1 - xn : (xn >= G.nx ? 2 * G.nx - 1 - xn : xn);
    else xn = xn < 0 ? xn + G.nx : (xn >= G.nx ? xn - G.nx : xn);
    if (G.walls) yn = yn < 0 ? -1 - yn : (yn >= G.ny ? 2 * G.ny - 1 - yn : yn);
    else yn = yn < 0 ? yn + G.ny : (yn >= G.ny ? yn - G.ny : yn);
    if (mask[(long long)yn * G.nx + xn]) b |= 1u << i;
  }
  if (b & 1u) b = 1u;
  nbr[(long long)y * G.pitch + x] = (uint16_t)b;
  if (b & 1u) atomicAdd(nsolid, 1ull);
}

// phi = 1 on solid nodes (a finite placeholder; never enters a fluid node).
template <typename T>
__global__ void phi_on_solids(Geo G, T* __restrict__ phi, const uint16_t* __restrict__ nbr) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  if (nbr[(long long)y * G.pitch + x] & 1u) phi[(long long)y * G.pitch + x] = T(1);
}

// Uploads of dense float64 fields into pitched planes of T, up to five in one
// launch (grid z).  check: a void fraction, whose values must lie in (0, 1]
// (solid nodes excepted, which take the placeholder phi = 1): *bad, host
// memory that the device can write, becomes nonzero where one does not.
// Bound by HBM: each field read and written once, and on small lattices by the
// launch and the synchronization.  A void fraction with the call around it: 62
// us on 4096 x 4096 FP64, 17 on 64 x 64; checked in a pass of its own, with the
// counter cleared before and copied after, 147 and 33.
struct UploadJob {
  const double* in;
  void* out;
  int check;
};
struct UploadJobs {
  UploadJob job[5];
};
template <typename T>
__global__ void __launch_bounds__(256) upload_fields(UploadJobs J, int nx, int ny, int pitch,
                                                     const uint16_t* __restrict__ nbr, int* __restrict__ bad) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  const UploadJob j = J.job[blockIdx.z];
  if (x >= nx || y >= ny) return;
  double v = j.in[(long long)y * nx + x];
  const long long o = (long long)y * pitch + x;
  if (j.check) {
    const bool solid = nbr && (nbr[o] & 1u);
    if (solid) v = 1.0;
    const bool wrong = !(v > 0.0 && v <= 1.0);
    const unsigned long long m = __ballot(wrong);  // (one write a wave)
    if (wrong && (m & ((1ull << (threadIdx.x & 63)) - 1)) == 0) *bad = 1;
  }
  static_cast<T*>(j.out)[o] = static_cast<T>(v);
}

// For the error message: count entries of a dense field outside (0, 1] (or
// non-finite), solid
// nodes (flag bit 0 of nbr, when given) excepted.
__global__ void count_bad_phi(const double* __restrict__ in, int nx, long long n,
                              const uint16_t* __restrict__ nbr, int pitch,
                              unsigned long long* __restrict__ bad) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  unsigned long long cnt = 0;
  for (; i < n; i += stride) {
    if (nbr && (nbr[(i / nx) * pitch + i % nx] & 1u)) continue;
    const double v = in[i];
    if (!(v > 0.0 && v <= 1.0)) ++cnt;
  }
  if (cnt) atomicAdd(bad, cnt);
}

// The slot that the pull of f_i at node (x, y) reads, as a byte offset into
// the population buffer: slot i of x - e_i, or slot opp(i) of the node itself
// when x - e_i lies beyond a wall or is solid (flag bit opp(i)); *crossed:
// beyond a wall in y.
template <typename S>
__device__ __forceinline__ unsigned slot_offset(const Geo& G, int x, int y, int i, unsigned nb, bool* crossed) {
  const unsigned pb = unsigned(G.plane) * unsigned(sizeof(S)), rb = unsigned(G.pitch) * unsigned(sizeof(S));
  const int ex = ex_of(i), ey = ey_of(i), o = opp_of(i);
  const int xs = ex == 1 ? (x == 0 ? G.nx - 1 : x - 1) : ex == -1 ? (x == G.nx - 1 ? 0 : x + 1) : x;
  const int ys = ey == 1 ? (y == 0 ? G.ny - 1 : y - 1) : ey == -1 ? (y == G.ny - 1 ? 0 : y + 1) : y;
  *crossed = G.walls && ((ey == 1 && y == 0) || (ey == -1 && y == G.ny - 1));
  const bool back = *crossed || (i > 0 && solid_bit(nb, o)) ||
                    (G.xwalls && ((ex == 1 && x == 0) || (ex == -1 && x == G.nx - 1)));
  return back ? unsigned(o) * pb + unsigned(y) * rb + unsigned(x) * unsigned(sizeof(S))
              : unsigned(i) * pb + unsigned(ys) * rb + unsigned(xs) * unsigned(sizeof(S));
}

// Fill the stored slots so that the next pull yields f(0): either the
// equilibrium of Eq. (14) at (rho0, u0), or given dense populations.  Each
// node writes the nine slots that its pull reads (every slot of a fluid node
// is read by exactly one pull), so its phi is read and divided by once;
// solid nodes write the rest state into their own slots, which no pull reads.
// Bound by HBM, the writes above all.  Forming a slot's value at the slot
// (nine receivers' phi and divisions per node, directions looked up at run
// time) took 340 us on 4096 x 4096 in FP32, this 233.
template <typename S, typename T, bool SHIFT>
__global__ void fill_state(Geo G, S* __restrict__ buf, const T* __restrict__ phi, StepPhys<T> ph,
                           const double* __restrict__ fin, double rho_init, double ux0, double uy0,
                           double kappa, const uint16_t* __restrict__ nbr) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const long long N = (long long)G.nx * G.ny;
  const unsigned nb = nbr_at(G, nbr, x, y);
  const T ph_x = phi[y * G.pitch + x];
  const rsrc_t dst = make_rsrc(buf, 9u * unsigned(G.plane) * unsigned(sizeof(S)));
  if (nb & 1u) {  // solid node: the rest state (never pulled by a fluid node)
    const unsigned own = (unsigned(y) * unsigned(G.pitch) + unsigned(x)) * unsigned(sizeof(S));
#pragma unroll
    for (int i = 0; i < 9; ++i)
      bstore(encode<S, T, SHIFT>(double(rest_pop(i, ph_x, ph)), ph_x, i, ph), dst,
             unsigned(i) * unsigned(G.plane) * unsigned(sizeof(S)) + own, 0u);
    return;
  }
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    bool crossed;
    const unsigned off = slot_offset<S>(G, x, y, j, nb, &crossed);
    double f = fin ? fin[j * N + (long long)y * G.nx + x]
                   : feq_pop(j, double(ph_x), rho_init, ux0, uy0, kappa, ph.eq2);
    if (crossed)  // the pull subtracts it again
      f += wall_delta(opp_of(j), ph_x, ey_of(j) == 1, ph);
    bstore(encode<S, T, SHIFT>(f, ph_x, j, ph), dst, off, 0u);
  }
}

// Populations f_i(x, t); zero on solid nodes.
template <typename S, typename T, bool SHIFT>
__global__ void read_pops(Geo G, const S* __restrict__ buf, const T* __restrict__ phi,
                          StepPhys<T> ph, double* __restrict__ out,
                          const uint16_t* __restrict__ nbr) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const long long N = (long long)G.nx * G.ny;
  const T ph_x = phi[y * G.pitch + x];
  const unsigned nb = nbr_at(G, nbr, x, y);
  const rsrc_t src = make_rsrc(buf, 9u * unsigned(G.plane) * unsigned(sizeof(S)));
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    bool crossed;
    const S s = bload<S>(src, slot_offset<S>(G, x, y, i, nb, &crossed), 0u);
    double f = decode<S, T, SHIFT>(s, ph_x, i, ph);
    if (crossed) f -= wall_delta(opp_of(i), ph_x, ey_of(i) == 1, ph);
    out[i * N + (long long)y * G.nx + x] = (nb & 1u) ? 0.0 : f;
  }
}

// The nine stored values that the pull of node (x, y) delivers (see
// slot_offset).  y is uniform over the workgroup; xm and xp are the neighbour
// columns.  GEN: with solid nodes or walls in x, where the slot is a choice
// per lane.
template <typename S, bool GEN>
__device__ __forceinline__ void pull_slots(const Geo& G, rsrc_t src, int x, int xm, int xp, int y,
                                           unsigned nb, S (&s)[9]) {
  const unsigned pb = unsigned(G.plane) * unsigned(sizeof(S)), rb = unsigned(G.pitch) * unsigned(sizeof(S));
  const unsigned c = unsigned(x) * unsigned(sizeof(S)), m = unsigned(xm) * unsigned(sizeof(S)),
                 p = unsigned(xp) * unsigned(sizeof(S));
  const bool lo = G.walls && y == 0, hi = G.walls && y == G.ny - 1;
  const int ys = y == 0 ? G.ny - 1 : y - 1, yn = y == G.ny - 1 ? 0 : y + 1;
  if constexpr (GEN) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      bool crossed;
      s[i] = bload<S>(src, slot_offset<S>(G, x, y, i, nb, &crossed), 0u);
    }
  } else {
    const unsigned r = unsigned(y) * rb, rs = unsigned(ys) * rb, rn = unsigned(yn) * rb;
    s[0] = bload<S>(src, c, r);
    s[1] = bload<S>(src, m, pb + r);
    s[3] = bload<S>(src, p, 3u * pb + r);
    s[2] = bload<S>(src, c, lo ? 4u * pb + r : 2u * pb + rs);
    s[5] = bload<S>(src, lo ? c : m, lo ? 7u * pb + r : 5u * pb + rs);
    s[6] = bload<S>(src, lo ? c : p, lo ? 8u * pb + r : 6u * pb + rs);
    s[4] = bload<S>(src, c, hi ? 2u * pb + r : 4u * pb + rn);
    s[7] = bload<S>(src, hi ? c : p, hi ? 5u * pb + r : 7u * pb + rn);
    s[8] = bload<S>(src, hi ? c : m, hi ? 6u * pb + r : 8u * pb + rn);
  }
}

// Columns a read-out workgroup of 256 lanes outputs (one halo column on
// either side)
constexpr int READ_W = 254;

// What a lane of the read-out keeps of a row until the row above it is there
template <typename T>
struct ReadRow {
  double m0;
  T dm0, jx, jy, phi, drho, fx, fy, beta, ux0, uy0;
  unsigned nb;
};

// Macroscopic read-out: rho, u, p (Eq. 7, with grad rho of Eq. 10 by mirror
// images at walls and centre values for solid neighbours), each output
// optional, and with `partials` the FP64 observables, one record per
// workgroup.  Solid nodes report zeros; they and the velocity rows are left
// out of the partials.  uprev: the velocity kept for the next residual.
//
// Bound by HBM: the populations, phi and the outputs once each.  A workgroup
// sweeps `rows` rows of a strip of READ_W columns; each row's moments are
// formed once, its delta rho goes to the neighbours through an LDS ring of
// four rows (one barrier a row: the slot written next was last read two
// barriers ago), and the row below it is output; the next row's loads are in
// flight meanwhile.  GEN: solid nodes, walls in x, moving walls or velocity
// rows; the other lattices take loads without per-lane choices.
// Measured, a call that reads rho, u and p of the 4096 x 4096 FP32 channel: 283 us
// (4.3 TB/s of the bytes above) against 2570 for two passes through a delta rho plane
// whose loops over the directions were not unrolled (their populations lived
// in scratch memory), the observables alone 195 against 2500; 2048 x 2048 FP64 107
// against 1013, and 109 against 984.
template <typename S, typename T, bool SHIFT, bool GEN>
__global__ void __launch_bounds__(256) read_out(
    Geo G, const S* __restrict__ buf, const T* __restrict__ phi, StepPhys<T> ph,
    const T* __restrict__ fxf, const T* __restrict__ fyf, const T* __restrict__ beta,
    double* __restrict__ rho_o, double* __restrict__ ux_o, double* __restrict__ uy_o,
    double* __restrict__ p_o, double* __restrict__ partials, T* __restrict__ uprev, int uprev_valid,
    const uint16_t* __restrict__ nbr, int strips, int rows) {
  __shared__ T s_rho[4][256];
  const int t = threadIdx.x;
  const int tile = xcd_tile(int(blockIdx.x), int(gridDim.x));
  const int x0 = (tile % strips) * READ_W, y0 = (tile / strips) * rows;
  const int w = min(READ_W, G.nx - x0), y1 = min(y0 + rows, G.ny);
  const bool out = t >= 1 && t <= w;
  const int xg = x0 - 1 + t;
  const int x = (GEN && G.xwalls) ? min(max(xg, 0), G.nx - 1) : wrap_index(xg, G.nx);
  const int xm = x == 0 ? G.nx - 1 : x - 1, xp = x == G.nx - 1 ? 0 : x + 1;
  const int tl = max(t - 1, 0), tr = min(t + 1, 255);
  const rsrc_t src = make_rsrc(buf, 9u * unsigned(G.plane) * unsigned(sizeof(S)));
  double mass = 0.0, u2 = 0.0, umax = 0.0, bad = 0.0, du2 = 0.0;

  // the row that stands for row yy: wrapped, or the wall's own row beyond it
  // (the mirror image); a velocity row takes the density of the fluid row
  // next to it
  auto row_of = [&](int yy) { return G.walls ? min(max(yy, 0), G.ny - 1) : wrap_index(yy, G.ny); };
  auto source_row = [&](int y) {
    if (!GEN) return y;
    const int kind = vel_row_kind(G, y);
    return kind == 1 ? 1 : (kind == 2 ? G.ny - 2 : y);
  };
  struct In {
    S s[9];
    T phi, fx, fy, beta, ux0, uy0;
    unsigned nb;
  };
  auto load = [&](int yy, In& in) {
    const int y = source_row(row_of(yy));
    const int o = y * G.pitch + x;
    in.nb = GEN ? nbr_at(G, nbr, x, y) : 0u;
    in.phi = phi[o];
    in.fx = fxf ? fxf[o] : T(0);
    in.fy = fyf ? fyf[o] : T(0);
    in.beta = beta ? beta[o] : T(0);
    in.ux0 = (uprev && uprev_valid) ? uprev[o] : T(0);
    in.uy0 = (uprev && uprev_valid) ? uprev[G.plane + o] : T(0);
    pull_slots<S, GEN>(G, src, x, xm, xp, y, in.nb, in.s);
  };

  // moments of row yy, then the output of row yy - 1 (held in R)
  auto body = [&](int yy, const In& in, ReadRow<T>& R) {
    ReadRow<T> N;
    N.phi = in.phi; N.fx = in.fx; N.fy = in.fy; N.beta = in.beta;
    N.ux0 = in.ux0; N.uy0 = in.uy0; N.nb = in.nb;
    T f[9];
    N.m0 = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      double fi = decode<S, T, SHIFT>(in.s[i], N.phi, i, ph);
      if constexpr (GEN) {  // moving walls: less the odd part of the equilibrium
        const int y = source_row(row_of(yy));
        if (G.walls && ey_of(i) == 1 && y == 0) fi -= wall_delta(opp_of(i), N.phi, true, ph);
        if (G.walls && ey_of(i) == -1 && y == G.ny - 1) fi -= wall_delta(opp_of(i), N.phi, false, ph);
      }
      f[i] = static_cast<T>(fi - double(rest_pop(i, N.phi, ph)));
      N.m0 += fi;
    }
    N.dm0 = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) N.dm0 += f[i];
    N.jx = (f[1] - f[3]) + ((f[5] - f[6]) + (f[8] - f[7]));
    N.jy = (f[2] - f[4]) + ((f[5] + f[6]) - (f[7] + f[8]));
    N.drho = (N.nb & 1u) ? T(0) : N.dm0 / N.phi;
    s_rho[yy & 3][t] = N.drho;
    __syncthreads();
    const int y = yy - 1;
    if (y >= y0 && out) {
      const long long o = (long long)y * G.nx + x;
      const int kind = GEN ? vel_row_kind(G, y) : 0;
      if (GEN && kind == 0 && (R.nb & 1u)) {
        if (rho_o) rho_o[o] = 0.0;
        if (ux_o) ux_o[o] = 0.0;
        if (uy_o) uy_o[o] = 0.0;
        if (p_o) p_o[o] = 0.0;
      } else if (GEN && kind) {
        // velocity row: the wall velocity and the fluid neighbour's density
        const double rho = double(ph.rho0 + R.drho);
        if (rho_o) rho_o[o] = rho;
        if (ux_o) ux_o[o] = kind == 1 ? G.un_lo : G.un_hi;
        if (uy_o) uy_o[o] = 0.0;
        if (p_o) p_o[o] = rho / 3.0;
      } else {
        const int sc = y & 3, sn = (y + 1) & 3, ss = (y - 1) & 3;
        T rE = s_rho[sc][tr], rW = s_rho[sc][tl], rN = s_rho[sn][t], rS = s_rho[ss][t];
        T rNE = s_rho[sn][tr], rNW = s_rho[sn][tl], rSE = s_rho[ss][tr], rSW = s_rho[ss][tl];
        if constexpr (GEN) {  // solid neighbour: the centre value
          const unsigned nb = R.nb;
          rE = solid_bit(nb, 1) ? R.drho : rE;
          rN = solid_bit(nb, 2) ? R.drho : rN;
          rW = solid_bit(nb, 3) ? R.drho : rW;
          rS = solid_bit(nb, 4) ? R.drho : rS;
          rNE = solid_bit(nb, 5) ? R.drho : rNE;
          rNW = solid_bit(nb, 6) ? R.drho : rNW;
          rSW = solid_bit(nb, 7) ? R.drho : rSW;
          rSE = solid_bit(nb, 8) ? R.drho : rSE;
        }
        const T grx = stencil_dx(rE, rW, rNE, rSE, rNW, rSW);
        const T gry = stencil_dy(rN, rS, rNE, rNW, rSE, rSW);
        const T kp = (ph.kappa - (ph.model_b ? T(1) : R.phi)) * T(1.0 / 3.0);  // Eq. (13) / model B
        const T sg = ph.scale_by_phi ? R.phi : T(1);
        T Fx = kp * grx + sg * ph.gx;
        T Fy = kp * gry + sg * ph.gy;
        if (fxf) {
          Fx += R.fx;
          Fy += R.fy;
        }
        const T m0 = R.phi * ph.rho0 + R.dm0;
        T ux, uy;
        if (beta) {  // u of Eq. (7) with the drag solved in closed form
          const T d = R.phi * R.beta;
          ux = (R.jx + T(0.5) * (Fx + d * ph.usx)) / (m0 + T(0.5) * d);
          uy = (R.jy + T(0.5) * (Fy + d * ph.usy)) / (m0 + T(0.5) * d);
        } else {
          ux = (R.jx + T(0.5) * Fx) / m0;
          uy = (R.jy + T(0.5) * Fy) / m0;
        }
        const T rho = ph.rho0 + R.drho;
        if (rho_o) rho_o[o] = double(rho);
        if (ux_o) ux_o[o] = double(ux);
        if (uy_o) uy_o[o] = double(uy);
        if (p_o) p_o[o] = double(rho) / 3.0;
        if (uprev) {
          T* const px = uprev + (long long)y * G.pitch + x;
          px[0] = ux;
          px[G.plane] = uy;
        }
        if (partials) {
          const bool finite = isfinite(R.m0) && isfinite(double(ux)) && isfinite(double(uy)) &&
                              isfinite(double(R.jx)) && isfinite(double(R.jy));
          if (finite) {
            const double v2 = double(ux) * double(ux) + double(uy) * double(uy);
            mass += R.m0;
            u2 += v2;
            umax = fmax(umax, v2);
            if (uprev && uprev_valid) {  // |u(t) - u(t')|^2
              const double dx = double(ux) - double(R.ux0), dy = double(uy) - double(R.uy0);
              du2 += dx * dx + dy * dy;
            }
          } else {
            bad += 1.0;
          }
        }
      }
    }
    R = N;
  };

  ReadRow<T> R{};
  In a, b;
  load(y0 - 1, a);
  for (int yy = y0 - 1; yy <= y1; yy += 2) {
    if (yy + 1 <= y1) load(yy + 1, b);
    body(yy, a, R);
    if (yy + 1 > y1) break;
    if (yy + 2 <= y1) load(yy + 2, a);
    body(yy + 1, b, R);
  }

  if (partials) {
    // workgroup reduction in a fixed order: wavefront shuffles, then LDS
    // (the square root is monotonic: taken once, of the largest |u|^2)
    __shared__ double red[NOBS][4];
    umax = sqrt(umax);
    for (int off = 32; off > 0; off >>= 1) {
      mass += __shfl_down(mass, off, 64);
      u2 += __shfl_down(u2, off, 64);
      umax = fmax(umax, __shfl_down(umax, off, 64));
      bad += __shfl_down(bad, off, 64);
      du2 += __shfl_down(du2, off, 64);
    }
    const int lane = t & 63, wv = t >> 6;
    if (lane == 0) {
      red[0][wv] = mass; red[1][wv] = u2; red[2][wv] = umax; red[3][wv] = bad; red[4][wv] = du2;
    }
    __syncthreads();
    if (t == 0) {
      double a5[NOBS] = {0, 0, 0, 0, 0};
      for (int k = 0; k < 4; ++k) {
        a5[0] += red[0][k]; a5[1] += red[1][k]; a5[2] = fmax(a5[2], red[2][k]); a5[3] += red[3][k];
        a5[4] += red[4][k];
      }
      for (int q = 0; q < NOBS; ++q) partials[(long long)tile * NOBS + q] = a5[q];
    }
  }
}

// Fixed-order reduction of block partials, in two levels: reduce_partials
// folds contiguous chunks (one workgroup per chunk) and is applied again to
// the chunk results until one record is left.  Record fields: mass, sum |u|^2,
// max |u|, non-finite count, sum |u - u_prev|^2.
__global__ void reduce_partials(const double* __restrict__ partials, long long nblk,
                                long long chunk, double* __restrict__ out) {
  __shared__ double red[NOBS][256];
  const long long beg = (long long)blockIdx.x * chunk;
  const long long end = min(beg + chunk, nblk);
  double a[NOBS] = {0, 0, 0, 0, 0};
  for (long long k = beg + threadIdx.x; k < end; k += blockDim.x) {
    a[0] += partials[k * NOBS + 0];
    a[1] += partials[k * NOBS + 1];
    a[2] = fmax(a[2], partials[k * NOBS + 2]);
    a[3] += partials[k * NOBS + 3];
    a[4] += partials[k * NOBS + 4];
  }
  for (int q = 0; q < NOBS; ++q) red[q][threadIdx.x] = a[q];
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
      red[2][threadIdx.x] = fmax(red[2][threadIdx.x], red[2][threadIdx.x + s]);
      red[3][threadIdx.x] += red[3][threadIdx.x + s];
      red[4][threadIdx.x] += red[4][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int q = 0; q < NOBS; ++q) out[(long long)blockIdx.x * NOBS + q] = red[q][0];
}

// In-step divergence check: reset the flag (first time a non-finite node was
// seen, -1 for none) ...
__global__ void set_flag(long long* __restrict__ flag, long long v) {
  if (threadIdx.x == 0) *flag = v;
}

// ... and record time t in it when the reduced observables (record field 3,
// the non-finite count) show a non-finite node and no earlier check did.
__global__ void note_nonfinite(const double* __restrict__ rec, long long t,
                               long long* __restrict__ flag) {
  if (threadIdx.x == 0 && rec[3] > 0.0 && *flag < 0) *flag = t;
}

// Speed-of-light reference with the step's memory pattern: every node pulls
// its nine populations from the same shifted positions (with the same
// bounce-back at walls) and writes them back unchanged to the other buffer.
// No arithmetic: 9 reads + 9 writes per node, the step's HBM traffic minus
// the phi plane.
template <typename S>
__global__ void __launch_bounds__(256) stream_copy(Geo G, const S* __restrict__ src,
                                                   S* __restrict__ dst) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const long long P = G.plane;
  const int xm = x == 0 ? G.nx - 1 : x - 1, xp = x == G.nx - 1 ? 0 : x + 1;
  const int o = y * G.pitch;
  S f[9];
  f[0] = src[o + x];
  f[1] = src[P + o + xm];
  f[3] = src[3 * P + o + xp];
  if (G.walls && y == 0) {
    f[2] = src[4 * P + o + x]; f[5] = src[7 * P + o + x]; f[6] = src[8 * P + o + x];
  } else {
    const int os = (y == 0 ? G.ny - 1 : y - 1) * G.pitch;
    f[2] = src[2 * P + os + x]; f[5] = src[5 * P + os + xm]; f[6] = src[6 * P + os + xp];
  }
  if (G.walls && y == G.ny - 1) {
    f[4] = src[2 * P + o + x]; f[7] = src[5 * P + o + x]; f[8] = src[6 * P + o + x];
  } else {
    const int on = (y == G.ny - 1 ? 0 : y + 1) * G.pitch;
    f[4] = src[4 * P + on + x]; f[7] = src[7 * P + on + xp]; f[8] = src[8 * P + on + xm];
  }
#pragma unroll
  for (int i = 0; i < 9; ++i) dst[i * P + o + x] = f[i];
}

}  // namespace vanse_dev
