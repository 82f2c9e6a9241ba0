// tile_kernel.hpp -- the one-step scheme for lattices too small to fill the
// GPU: a tile of nodes per workgroup, one node per lane, several time steps
// per launch.
//
// Such lattices are bound by latency: a launch with its loads and stores
// takes 2.6 us (a copy of 64 x 64 nodes), and the row sweep of
// step_kernel.hpp adds about half a microsecond a row with little else to
// run, 5.7 us a step on 64 x 64 FP64 nodes however few rows a workgroup has.
// Here all rows of a
// tile go through the three stages (A moments, B velocity, C collision) at
// once, and `steps` time steps run one after the other on a tile that shrinks
// by three nodes a side per step: the post-collision populations go to the
// neighbours through LDS, and only the last step's reach memory.  A step
// therefore costs three barriers, and a launch one round of loads, whatever
// the number of steps.  The node arithmetic is step_kernel.hpp's, and the
// values between the steps are rounded to the storage type as a store would
// round them, so the results are bitwise those of single steps.
// Measured (us per step; sweep, then tiles with the steps per launch that the
// host picks): 64 x 64 FP64 5.7, 2.66 (4), FP32 4.8, 2.19 (4); 129 x 129 FP64
// with a force field 6.9, 3.26 (3), FP32 5.7, 2.47 (4); 256 x 256 FP64 9.2,
// 5.75 (2), FP32 7.45, 3.22 (3); 512 x 512 FP64 16.7, 14.3 (2), FP32 10.8, 9.6
// (2).  There and beyond the recomputed halo costs more than the sweep's
// latency: 1003 x 777 FP32 18.5, 21.8 (2).  Pairs of steps against the two-step
// sweep: 64 x 64 FP64 11.6, 2.65, FP32 9.5, 2.2; 256 x 256 FP64 12.0, 5.8, FP32
// 9.9, 4.4; 512 x 512 FP64 15.9, 14.7, FP32 11.6, 9.8, with solid nodes 15.6,
// 10.3; a moving phi with drag on 256 x 256 FP64 14.2, 5.8.
//
// Lane (lx, ly) is node (x0 - h + lx, y0 - h + ly), h = 3 steps - 1: a step
// needs two nodes around its output (delta-rho, then the velocity) and its
// pull one more, which the first step takes from memory.  Step s computes
// valid delta-rho on lanes 3 s from the tile's edge, velocities 3 s + 1 and
// collisions 3 s + 2; the other lanes compute values that nothing reads.
// Walls: lanes beyond a face do nothing, and the face's own lanes write their
// image (delta-rho alike, velocity-like fields negated) there.
#pragma once

#include "step2_kernel.hpp"
#include "step_kernel.hpp"

namespace vanse_dev {

// Tile sides in lanes.  In FP32 arithmetic (93-116 registers) 32 x 32 lanes,
// the largest workgroup; in FP64 (158-168 registers) 32 x 24, the largest
// that three waves per SIMD and their 168 registers allow (32 x 32 spills 112
// bytes a lane and takes 4.1 us a step on 64 x 64 nodes against 2.7).  Smaller
// tiles recompute more: 32 x 16 lanes at two steps 3.6 us a step on 129 x 129
// FP64, 32 x 24 at three 3.3.
constexpr int TILE_X = 32;
constexpr int tile_y(int tbytes) { return tbytes == 8 ? 24 : 32; }
// Nodes a side that a tile of `lanes` lanes outputs after `steps` steps
constexpr int tile_out(int lanes, int steps) { return lanes - 2 * (3 * steps - 1); }

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

template <typename T, int NT>
struct TileLds {
  T rho[NT];
  Pair<T> u[NT], mr[NT], mr2[NT];  // (u_x, u_y), (phi rho, rho) u_x and (phi rho, rho) u_y
  T pop[9][NT];  // stored values between two steps, widened to T (or deviations)
};

// FEAT: FEAT_FORCE, FEAT_DRAG, FEAT_MASK (with walls in x or not) and
// FEAT_DYNPHI (one launch per hand-over of phi); absent planes read as zero,
// which leaves the results as they are.
// PAIRS: the arithmetic of two-step launches (step2_kernel.hpp): the separable
// form of Eq. (10), and the state between the two steps of a pair kept as
// deviations in T; the launch takes one or more pairs.  The scheme is the
// same, and so are the results, bit for bit, as those of the two-step sweep.
// walls: bit 0 in y, bit 1 in x.
template <typename S, typename T, bool SHIFT, int FEAT, bool PAIRS, int TY>
__global__ void __launch_bounds__(TILE_X * TY)
__attribute__((amdgpu_waves_per_eu(TILE_X * TY / 256)))
vanse_tile_kernel(StepGeom g, StepPhys<T> ph, int walls, int steps) {
  constexpr int TX = TILE_X, NT = TX * TY;
  constexpr bool DYN = (FEAT & FEAT_DYNPHI) != 0, MASK = (FEAT & FEAT_MASK) != 0;
  const int out_x = tile_out(TX, steps), out_y = tile_out(TY, steps);
  __shared__ TileLds<T, NT> L;
  const int t0 = threadIdx.x;
  const int lx = t0 % TX, ly = t0 / TX;
  const int h = 3 * steps - 1;
  const int x0 = int(blockIdx.x % unsigned(g.strips)) * out_x, y0 = int(blockIdx.x / unsigned(g.strips)) * out_y;
  const int xg = x0 - h + lx, yg = y0 - h + ly;
  const bool wy = (walls & 1) != 0, wx = (walls & 2) != 0;
  const int x = wx ? min(max(xg, 0), g.nx - 1) : wrap_index(xg, g.nx);
  const int y = wy ? min(max(yg, 0), g.ny - 1) : wrap_index(yg, g.ny);
  const bool live = (!wx || (xg >= 0 && xg < g.nx)) && (!wy || (yg >= 0 && yg < g.ny));
  // a face's lanes, where the lane beyond them is in the tile
  const bool xlo = wx && x == 0, xhi = wx && x == g.nx - 1, ylo = wy && y == 0, yhi = wy && y == g.ny - 1;
  const int gx = live ? (xlo && lx > 0 ? -1 : (xhi && lx < TX - 1 ? 1 : 0)) : 0;
  const int gy = live ? (ylo && ly > 0 ? -TX : (yhi && ly < TY - 1 ? TX : 0)) : 0;
  // neighbours in the tile
  const int dw = lx > 0 ? -1 : 0, de = lx < TX - 1 ? 1 : 0;
  const int n = ly < TY - 1 ? TX : 0, s = ly > 0 ? -TX : 0;

  constexpr unsigned SB = sizeof(S), TB = sizeof(T);
  const unsigned plane = unsigned(g.plane), own = unsigned(y) * unsigned(g.pitch) + unsigned(x);
  const rsrc_t srcr = make_rsrc(g.src, 9u * plane * SB);
  const rsrc_t dstr = make_rsrc(g.dst, 9u * plane * SB);
  const rsrc_t phir = make_rsrc(g.phi, plane * TB);
  const rsrc_t betar = make_rsrc(g.beta, ((FEAT & FEAT_DRAG) && g.beta) ? plane * TB : 0u);
  const rsrc_t fxr = make_rsrc(g.fxf, ((FEAT & FEAT_FORCE) && g.fxf) ? plane * TB : 0u);
  const rsrc_t fyr = make_rsrc(g.fyf, ((FEAT & FEAT_FORCE) && g.fyf) ? plane * TB : 0u);
  const rsrc_t nbrr = make_rsrc(g.nbr, ((FEAT & FEAT_MASK) && g.nbr) ? plane * 2u : 0u);

  RowState<T> r{};
  r.nb = (FEAT & FEAT_MASK) ? bload_u16(nbrr, own * 2u, 0u) : 0u;
  const T phi = bload<T>(phir, own * TB, 0u);
  r.beta = (FEAT & FEAT_DRAG) ? bload<T>(betar, own * TB, 0u) : T(0);
  T ffx = (FEAT & FEAT_FORCE) ? bload<T>(fxr, own * TB, 0u) : T(0);
  T ffy = (FEAT & FEAT_FORCE) ? bload<T>(fyr, own * TB, 0u) : T(0);
  const rsrc_t phinr = make_rsrc(g.phin, DYN ? plane * TB : 0u);
  r.phi = phi;
  r.dphi = DYN ? bload<T>(phinr, own * TB, 0u) - phi : T(0);
  // directions whose source lies beyond a wall or is solid: half-way
  // bounce-back, the node's own opposite slot
  unsigned back = 0;
  if (FEAT & FEAT_MASK) {  // bit i of the flags: x + e_i is solid
    back = ((r.nb >> 2) & 0x6u) | ((r.nb << 2) & 0x18u) | ((r.nb >> 2) & 0x60u) | ((r.nb << 2) & 0x180u);
  }
  back |= (xlo ? (1u << 1) | (1u << 5) | (1u << 8) : 0u) | (xhi ? (1u << 3) | (1u << 6) | (1u << 7) : 0u) |
          (ylo ? (1u << 2) | (1u << 5) | (1u << 6) : 0u) | (yhi ? (1u << 4) | (1u << 7) | (1u << 8) : 0u);
  auto bounced = [&](int i) { return ((back >> i) & 1u) != 0u; };

  // the pull of the first step, from memory
  S f[9];
  {
    const unsigned xm = unsigned(x == 0 ? g.nx - 1 : x - 1), xp = unsigned(x == g.nx - 1 ? 0 : x + 1);
    const unsigned row = unsigned(y) * unsigned(g.pitch);
    const unsigned rs = unsigned(y == 0 ? g.ny - 1 : y - 1) * unsigned(g.pitch);
    const unsigned rn = unsigned(y == g.ny - 1 ? 0 : y + 1) * unsigned(g.pitch);
    auto pull = [&](int i, int o, unsigned from) {
      return bload<S>(srcr, (bounced(i) ? unsigned(o) * plane + own : unsigned(i) * plane + from) * SB, 0u);
    };
    f[0] = bload<S>(srcr, own * SB, 0u);
    f[1] = pull(1, 3, row + xm);
    f[2] = pull(2, 4, rs + unsigned(x));
    f[3] = pull(3, 1, row + xp);
    f[4] = pull(4, 2, rn + unsigned(x));
    f[5] = pull(5, 7, rs + xm);
    f[6] = pull(6, 8, rs + xp);
    f[7] = pull(7, 5, rn + xp);
    f[8] = pull(8, 6, rn + xm);
  }
  T q[9];
  deviations<S, T, SHIFT>(f, phi, ph, q);

  for (int step = 1;; ++step) {
    // rows that still matter: a wave whose rows all lie outside has nothing to
    // do but meet the barriers
    const int m = 3 * (step - 1);
    // (opaque in FP64 pairs: addresses formed from it are formed anew each step
    // rather than held in registers through the loop, where they would spill;
    // the others have the registers, and holding them is 3% faster)
    int t = t0;
    if (PAIRS && sizeof(T) == 8) __asm__ volatile("" : "+v"(t));
    const int e = t + de, w = t + dw;
    const bool liveA = live && ly >= m && ly < TY - m;
    const bool liveB = live && ly > m && ly < TY - 1 - m;
    const bool liveC = live && ly > m + 1 && ly < TY - 2 - m;
    // ---------------- stage A ----------------
    if (liveA) {
      if (PAIRS) moments2_of(q, r);
      else moments_of(q, r);
      r.rphi = recip(r.phi);
      r.drho = r.dm0 * r.rphi;
      // (PAIRS: solid nodes are left out of the separable sums)
      const T dr = (PAIRS && MASK && solid_bit(r.nb, 0)) ? T(0) : r.drho;
      L.rho[t] = dr;
      if (gx) L.rho[t + gx] = dr;
      if (gy) L.rho[t + gy] = dr;
      if (gx && gy) L.rho[t + gx + gy] = dr;
    }
    __syncthreads();

    // ---------------- stage B ----------------
    T Fx, Fy;
    if (liveB) {
      RhoAround<T> a;
      a.E = L.rho[e]; a.W = L.rho[w]; a.N = L.rho[t + n]; a.S = L.rho[t + s];
      a.NE = L.rho[e + n]; a.NW = L.rho[w + n]; a.SE = L.rho[e + s]; a.SW = L.rho[w + s];
      U4<T> u;
      U2<T> v;
      if constexpr (PAIRS) {
        // D and S of the rows below (m), here (c) and above (n), as in
        // step2_kernel.hpp
        const T dm = a.SE - a.SW, dc = a.E - a.W, dn = a.NE - a.NW;
        const T sm = (a.SE + a.SW) + T(4) * a.S, sn = (a.NE + a.NW) + T(4) * a.N;
        T grx = T(4) * dc + (dm + dn);
        T gry = sn - sm;
        if constexpr (MASK) {
          if (wave_any((r.nb & 0x1FEu) != 0)) {  // solid neighbours: the centre value
            grx += T(solid_kx(r.nb)) * r.drho;
            gry += T(solid_ky(r.nb)) * r.drho;
          }
        }
        velocity2_of<FEAT>(grx, gry, r, ffx, ffy, false, ph, u, v, Fx, Fy);
        if (MASK && solid_bit(r.nb, 0)) {
          u.ux = u.uy = u.mux = u.rux = T(0);
          v.muy = v.ruy = T(0);
        }
      } else {
        T m0, rho;
        velocity_of<FEAT>(a, r, [&](T& fx, T& fy) { fx = ffx; fy = ffy; }, ph, u, v, Fx, Fy, m0, rho);
      }
      auto put = [&](int at, T sg) {
        L.u[at] = {sg * u.ux, sg * u.uy};
        L.mr[at] = {sg * u.mux, sg * u.rux};
        L.mr2[at] = {sg * v.muy, sg * v.ruy};
      };
      put(t, T(1));
      if (gx) put(t + gx, T(-1));  // the images beyond the walls
      if (gy) put(t + gy, T(-1));
      if (gx && gy) put(t + gx + gy, T(-1));
    }
    __syncthreads();

    // ---------------- stage C ----------------
    const bool second = PAIRS && (step & 1) == 0;
    S out[9];
    T o9[9];
    if (liveC) {
      // The neighbours' records one pair of fields after the other, so that
      // few are held at a time (all at once take a third more registers).
      if constexpr (PAIRS) {
        // (rows below m, here c and above n, as derivs2_of; in FP64 row by row)
        auto part = [] { if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0); };
        Derivs2<T> d;
        const Pair<T> uc = L.u[t];
        {
          const Pair<T> cE = L.u[e], cW = L.u[w];
          const T cx = cE.a - cW.a, cy = cE.b - cW.b;
          part();
          const Pair<T> mE = L.u[e + s], mW = L.u[w + s], m0 = L.u[t + s];
          const T mx = mE.a - mW.a, my = mE.b - mW.b;
          const T msx = (mE.a + mW.a) + T(4) * m0.a, msy = (mE.b + mW.b) + T(4) * m0.b;
          part();
          const Pair<T> nE = L.u[e + n], nW = L.u[w + n], n0 = L.u[t + n];
          const T nx = nE.a - nW.a, ny = nE.b - nW.b;
          const T nsx = (nE.a + nW.a) + T(4) * n0.a, nsy = (nE.b + nW.b) + T(4) * n0.b;
          d.ux_x = T(4) * cx + (mx + nx);
          d.uy_x = T(4) * cy + (my + ny);
          d.ux_y = nsx - msx;
          d.uy_y = nsy - msy;
        }
        __builtin_amdgcn_sched_barrier(0);
        {
          const Pair<T> cE = L.mr[e], cW = L.mr[w], mE = L.mr[e + s], mW = L.mr[w + s], nE = L.mr[e + n],
                        nW = L.mr[w + n];
          const T cm = cE.a - cW.a, mm = mE.a - mW.a, nm = nE.a - nW.a;
          const T cr = cE.b - cW.b, mr = mE.b - mW.b, nr = nE.b - nW.b;
          d.mux_x = T(4) * cm + (mm + nm);
          d.rux_x = T(4) * cr + (mr + nr);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
          const Pair<T> mE = L.mr2[e + s], mW = L.mr2[w + s], m0 = L.mr2[t + s], nE = L.mr2[e + n],
                        nW = L.mr2[w + n], n0 = L.mr2[t + n];
          const T mm = (mE.a + mW.a) + T(4) * m0.a, mr = (mE.b + mW.b) + T(4) * m0.b;
          const T nm = (nE.a + nW.a) + T(4) * n0.a, nr = (nE.b + nW.b) + T(4) * n0.b;
          d.muy_y = nm - mm;
          d.ruy_y = nr - mr;
        }
        __builtin_amdgcn_sched_barrier(0);
        collide2_of<FEAT>(d, r, r.nb, uc.a, uc.b, Fx, Fy, false, SHIFT && second, ph, o9);
        if (MASK && solid_bit(r.nb, 0)) {  // solid node: keep the rest state
#pragma unroll
          for (int i = 0; i < 9; ++i) o9[i] = T(0);
        }
        const T drest = DYN ? ph.rho0 * r.dphi : T(0);
        if (DYN && !second) o9[0] -= drest;
        if (second && SHIFT) {  // already scaled
          out[0] = DYN ? less_scaled<S>(o9[0], ph.scale, drest) : static_cast<S>(o9[0]);
#pragma unroll
          for (int i = 1; i < 9; ++i) out[i] = static_cast<S>(o9[i]);
        } else if (second) {
          stored<S, T, false, 0>(o9, r.phi, T(0), ph, [&](int i, S x) { out[i] = x; });
        }
      } else {
        // a solid neighbour stands in with the centre's, negated
        auto at = [&](const Pair<T>* L2, int k, int i, const Pair<T>& c) {
          Pair<T> p = L2[k];
          if constexpr ((FEAT & FEAT_MASK) != 0) {
            p.a = solid_bit(r.nb, i) ? -c.a : p.a;
            p.b = solid_bit(r.nb, i) ? -c.b : p.b;
          }
          return p;
        };
        Derivs<T> d;
        const Pair<T> uc = L.u[t];
        {
          const Pair<T> pE = at(L.u, e, 1, uc), pN = at(L.u, t + n, 2, uc), pW = at(L.u, w, 3, uc),
                        pS = at(L.u, t + s, 4, uc), pNE = at(L.u, e + n, 5, uc), pNW = at(L.u, w + n, 6, uc),
                        pSW = at(L.u, w + s, 7, uc), pSE = at(L.u, e + s, 8, uc);
          d.ux_x = stencil_dx(pE.a, pW.a, pNE.a, pSE.a, pNW.a, pSW.a);
          d.uy_y = stencil_dy(pN.b, pS.b, pNE.b, pNW.b, pSE.b, pSW.b);
          d.uy_x = stencil_dx(pE.b, pW.b, pNE.b, pSE.b, pNW.b, pSW.b);
          d.ux_y = stencil_dy(pN.a, pS.a, pNE.a, pNW.a, pSE.a, pSW.a);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
          const Pair<T> c = (FEAT & FEAT_MASK) ? L.mr[t] : Pair<T>{};
          const Pair<T> pE = at(L.mr, e, 1, c), pW = at(L.mr, w, 3, c), pNE = at(L.mr, e + n, 5, c),
                        pNW = at(L.mr, w + n, 6, c), pSW = at(L.mr, w + s, 7, c), pSE = at(L.mr, e + s, 8, c);
          d.mux_x = stencil_dx(pE.a, pW.a, pNE.a, pSE.a, pNW.a, pSW.a);
          d.rux_x = stencil_dx(pE.b, pW.b, pNE.b, pSE.b, pNW.b, pSW.b);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
          const Pair<T> c = (FEAT & FEAT_MASK) ? L.mr2[t] : Pair<T>{};
          const Pair<T> pN = at(L.mr2, t + n, 2, c), pS = at(L.mr2, t + s, 4, c), pNE = at(L.mr2, e + n, 5, c),
                        pNW = at(L.mr2, w + n, 6, c), pSW = at(L.mr2, w + s, 7, c), pSE = at(L.mr2, e + s, 8, c);
          d.muy_y = stencil_dy(pN.a, pS.a, pNE.a, pNW.a, pSE.a, pSW.a);
          d.ruy_y = stencil_dy(pN.b, pS.b, pNE.b, pNW.b, pSE.b, pSW.b);
        }
        __builtin_amdgcn_sched_barrier(0);
        T Ca, Cb, Cc;
        const T rho = ph.rho0 + r.drho, X = ph.kappa * r.rphi;
        penalty20(d, ph.kappa, ph.kappa - r.phi, rho, X, Ca, Cb, Cc);
        if (DYN) Ca -= T(2) * X * rho * r.dphi;
        collide_of<FEAT>(Ca, Cb, Cc, r, uc.a, uc.b, Fx, Fy, ph, o9);
        stored<S, T, SHIFT, FEAT>(o9, phi, r.dphi, ph, [&](int i, S x) { out[i] = x; });
      }
    }
    if (step == steps) {
      if (live && lx >= h && ly >= h && lx < TX - h && ly < TY - h && xg < min(x0 + out_x, g.nx) &&
          yg < min(y0 + out_y, g.ny)) {
#pragma unroll
        for (int i = 0; i < 9; ++i) bstore(out[i], dstr, own * SB, unsigned(i) * plane * SB);
      }
      break;
    }
    // into LDS, rounded as stored (between the steps of a pair as they are),
    // and pulled from there
    if (liveC) {
#pragma unroll
      for (int i = 0; i < 9; ++i) L.pop[i][t] = (PAIRS && !second) ? o9[i] : static_cast<T>(out[i]);
    }
    // a moving phi: the second step's phi(t+1), phi(t+2), drag coefficient and
    // force field, loaded only here (held from the start they would spill)
    T phi1 = T(0), phi2 = T(0);
    if (DYN && PAIRS) {
      phi1 = bload<T>(phinr, own * TB, 0u);
      phi2 = bload<T>(make_rsrc(g.phin2, plane * TB), own * TB, 0u);
      r.beta = bload<T>(make_rsrc(g.beta2, g.beta2 ? plane * TB : 0u), own * TB, 0u);
      ffx = bload<T>(make_rsrc(g.fxf2, g.fxf2 ? plane * TB : 0u), own * TB, 0u);
      ffy = bload<T>(make_rsrc(g.fyf2, g.fyf2 ? plane * TB : 0u), own * TB, 0u);
    }
    __syncthreads();
    T p[9];
    p[0] = L.pop[0][t];
    p[1] = bounced(1) ? L.pop[3][t] : L.pop[1][w];
    p[2] = bounced(2) ? L.pop[4][t] : L.pop[2][t + s];
    p[3] = bounced(3) ? L.pop[1][t] : L.pop[3][e];
    p[4] = bounced(4) ? L.pop[2][t] : L.pop[4][t + n];
    p[5] = bounced(5) ? L.pop[7][t] : L.pop[5][w + s];
    p[6] = bounced(6) ? L.pop[8][t] : L.pop[6][e + s];
    p[7] = bounced(7) ? L.pop[5][t] : L.pop[7][e + n];
    p[8] = bounced(8) ? L.pop[6][t] : L.pop[8][w + n];
    if (PAIRS && !second) {
#pragma unroll
      for (int i = 0; i < 9; ++i) q[i] = p[i];
      if (DYN) {  // the second step of the hand-over
        r.phi = phi1;
        r.dphi = phi2 - phi1;
      }
    } else {
      deviations<S, T, SHIFT>(p, phi, ph, q);
    }
  }
}

}  // namespace vanse_dev
