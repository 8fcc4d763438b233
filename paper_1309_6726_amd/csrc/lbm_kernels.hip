// Device kernels of the reactive two-component lattice Boltzmann step for
// gfx950 (MI355X).  The step follows the model of Sergi, Grossi, Leidi &
// Ortona (section "LB models"): D2Q9 BGK for both fluid components with
// bounce-back at solids, cohesion and adhesion forces, D2Q5 BGK solute lattice
// advected by the flow, first-order precipitation at wall-adjacent nodes and
// threshold growth of the solid phase.
//
// Memory layout in HBM (structure of arrays, plane stride P >= nx*ny, P a
// multiple of 64 so every plane starts 256-byte aligned):
//   f  float[18][P]  populations, component-major, link order
//                    (0,0),(1,0),(0,1),(-1,0),(0,-1),(1,1),(-1,1),(-1,-1),(1,-1);
//                    in the moment scheme planes 0..5 hold instead the
//                    post-collision moments rho1, v1x, v1y, rho2, v2x, v2y
//   g  float[5][P]   solute populations (first five links)
//   mask uint8[P]    bit0 solid; bits 1..3 growth pending (see pending_bit)
//   m  double[P]     precipitated mass (touched only at wall-adjacent nodes)
//   sstep int32[P]   state index at which the node turned solid (-1 fluid)
//   drop float[3][P] populations a node carried when it turned solid
// f and g are double-buffered (A/B); a step reads one buffer and writes the
// other.
//
// Population step (any tau), one kernel per time step (pop_rows).  A workgroup
// owns 62 consecutive columns (one lane each, plus one halo column on each
// side) and up to POP_ROWS rows, one wavefront per row and one more below and
// above.  A wavefront loads its row's populations (coalesced along x), forms the
// densities and momenta, publishes the densities in LDS, and collides its row
// with the cohesion/adhesion stencil read from there, applies the reaction, and
// pushes the post-collision populations to the neighbours (or back into the
// node's own opposite link at a solid neighbour).
//
// Moment step (tau = 1).  With full relaxation the post-collision populations
// of a component are its equilibria at (rho_s, v_s), so a node stores those
// three numbers per component (24 bytes instead of 72) and the next step
// rebuilds the populations that arrive at x by evaluating the equilibrium of
// each upstream neighbour (halfway bounce-back: the node's own moments with
// the velocity reversed when the upstream node is solid).  A tile then owns 60
// columns: the gathered densities feed the force stencil, which reaches two
// columns and two rows out.  Two kernels run it (moment_kind chooses): mom_rows,
// one wavefront per row of the tile with the links exchanged through LDS, and
// mom_wave, one wavefront that marches up its tile.  Per-node arithmetic is
// independent of the kernel and of the launch shape in both steps, so every tile
// shape gives bit-identical results.
//
// Growth timing.  In the step n -> n+1 a node whose precipitate exceeds the
// threshold still streams as fluid (the step uses the solid set of state n);
// it is marked with pending_bit(n).  Step n+1 reads it as solid and books the
// populations it carried into `drop`; step n+2 folds the mark into bit0.  A
// node being marked in the current step is read as fluid by its neighbours,
// so concurrent workgroups never disagree on the solid sets of states n-1
// and n, which the moment step needs both of.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lbm_dev.h"

// Multiply-adds are fused only where one source expression states them: the
// compiler may peel or duplicate loop iterations, and fusion chosen per copy
// would make the rounding of a node depend on which copy computes it (and so
// on the launch shape).
#pragma clang fp contract(on)

namespace lbmdev {

template <typename R>
__device__ __forceinline__ R feq(R w, R rho, R eu, R uu) {
  return w * rho * (R(1) + R(3) * eu + R(4.5) * eu * eu - R(1.5) * uu);
}

template <typename R>
__device__ __forceinline__ R sum9(const float* v) {
  return (((R)v[0] + (R)v[1]) + ((R)v[2] + (R)v[3])) + (((R)v[4] + (R)v[5]) + ((R)v[6] + (R)v[7])) +
         (R)v[8];
}

// s_waitcnt immediate for vmcnt(0) with expcnt and lgkmcnt left open (gfx9
// encoding: vmcnt[3:0] and [15:14], expcnt[6:4], lgkmcnt[11:8]).
#define VMCNT0 0x0F70

typedef unsigned v2u __attribute__((ext_vector_type(2)));

// Cache-policy operand of the buffer builtins: the non-temporal bit (nt).
#define CPOL_NT 2

// Raw buffer descriptor (stride 0, no format conversion) over bytes [0, extent)
// of base.  Word 3 is the value the gfx9-family buffer instructions take for
// untyped dword access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned extent) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)extent, 0x00020000);
}

// One dword per lane at byte offset voff + soff, with the non-temporal hint if NT.
template <bool NT>
__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __uint_as_float(
      (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, NT ? CPOL_NT : 0));
}

// Workgroup-wide LDS barrier that leaves outstanding global memory operations
// in flight (only LDS traffic is ordered).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// 1/x from the hardware estimate refined by two Newton steps (a few ulp; the
// correctly rounded division sequence costs twice the instructions).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ double fmar(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmar(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return __builtin_fmaf(r, __builtin_fmaf(-x, r, 1.0f), r);
}

// Shan-Chen interaction forces plus the body force at a fluid node (section
// "LB models": cohesion between the two components and adhesion to the solid,
// each a weight-normalised sum over the eight neighbours).  n1, n2: the
// neighbours' densities (zero at solid nodes), index = link, 1..8 = E, N, W, S,
// NE, NW, SW, SE (index 0 unused); (csx, csy): the weighted sum of the links to
// solid neighbours (wall_links).
template <typename R>
__device__ __forceinline__ void sc_forces(const StepArgs& a, const R* n1, const R* n2, R csx, R csy,
                                          R rho1, R rho2, R& F1x, R& F1y, R& F2x, R& F2y) {
  const R WA = R(1) / R(9), WD = R(1) / R(36);
  const R c2x = WA * (n2[1] - n2[3]) + WD * ((n2[5] - n2[6]) + (n2[8] - n2[7]));
  const R c2y = WA * (n2[2] - n2[4]) + WD * ((n2[5] + n2[6]) - (n2[8] + n2[7]));
  const R c1x = WA * (n1[1] - n1[3]) + WD * ((n1[5] - n1[6]) + (n1[8] - n1[7]));
  const R c1y = WA * (n1[2] - n1[4]) + WD * ((n1[5] + n1[6]) - (n1[8] + n1[7]));
  const R G = (R)a.G, Ga1 = (R)a.Gads1, Ga2 = (R)a.Gads2, ax = (R)a.ax, ay = (R)a.ay;
  F1x = -G * rho1 * c2x - Ga1 * rho1 * csx + rho1 * ax;
  F1y = -G * rho1 * c2y - Ga1 * rho1 * csy + rho1 * ay;
  F2x = -G * rho2 * c1x - Ga2 * rho2 * csx + rho2 * ax;
  F2y = -G * rho2 * c1y - Ga2 * rho2 * csy + rho2 * ay;
}

// Equilibrium velocities of the two components (common velocity shifted by
// tau F_s / rho_s) and the physical velocity (j + F/2) / rho that advects the
// solute; irt = 1 / (rho1 + rho2).
template <typename R>
__device__ __forceinline__ void sc_velocities(R tau, R rho1, R rho2, R j1x, R j1y, R j2x, R j2y,
                                              R F1x, R F1y, R F2x, R F2y, R& v1x, R& v1y,
                                              R& v2x, R& v2y, R& ux, R& uy, R& irt) {
  const R rt = rho1 + rho2;
  irt = recip(rt);
  const R upx = (j1x + j2x) * irt, upy = (j1y + j2y) * irt;
  v1x = upx; v1y = upy; v2x = upx; v2y = upy;
  if (rho1 > R(0)) { const R s = tau * recip(rho1); v1x += s * F1x; v1y += s * F1y; }
  if (rho2 > R(0)) { const R s = tau * recip(rho2); v2x += s * F2x; v2y += s * F2y; }
  ux = (j1x + j2x + R(0.5) * (F1x + F2x)) * irt;
  uy = (j1y + j2y + R(0.5) * (F1y + F2y)) * irt;
}

// Solute collision (BGK on D2Q5, or on D2Q4 with weights 1/4 and no rest
// link, advected by u), first-order precipitation at a node with ns > 0 solid
// axis neighbours (rate k_r ns phi, phi the wetting fraction; with a
// saturation concentration c_eq > 0 only the excess C - c_eq precipitates),
// the held source (post-collision solute of a node with x < hold_x set to the
// equilibrium at c_hold), threshold test, and push of the solute populations
// (bounce-back at solid axis neighbours).  wall: solid flags of the axis
// neighbours 1..4.
// What solute_step leaves for memory every step: the five pushed populations
// with their element offsets in gout, and the new precipitate of the node
// (wm: the node is next to a wall, so m changed).
struct SoluteOut {
  float g[5];
  unsigned off[5];
  double m;
  bool wm;
};

template <bool REACT, bool VAR, typename R>
__device__ __forceinline__ void solute_step(const StepArgs& a, const float* g, R ux, R uy, R rho1,
                                            R rho2, R irt, const bool* wall, double m_cur, unsigned P,
                                            unsigned idx, unsigned iE, unsigned iN, unsigned iW,
                                            unsigned iS, int xc, bool& ev, SoluteOut& so) {
  so.wm = false;
  so.m = 0.0;
  // VAR = false: the plain model (D2Q5, c_eq = 0, no held source)
  const bool q4 = VAR && a.q4 != 0;
  const R C = (((R)g[0] + (R)g[1]) + ((R)g[2] + (R)g[3])) + (R)g[4];
  const R WQ = q4 ? R(0.25) : R(1) / R(6), CQ = q4 ? R(2) : R(3);
  const R og = (R)a.omega_g;
  R gs[5];
  gs[1] = (R)g[1] + og * (WQ * C * (R(1) + CQ * ux) - (R)g[1]);
  gs[2] = (R)g[2] + og * (WQ * C * (R(1) + CQ * uy) - (R)g[2]);
  gs[3] = (R)g[3] + og * (WQ * C * (R(1) - CQ * ux) - (R)g[3]);
  gs[4] = (R)g[4] + og * (WQ * C * (R(1) - CQ * uy) - (R)g[4]);
  gs[0] = q4 ? R(0) : C - ((gs[1] + gs[2]) + (gs[3] + gs[4]));
  if (REACT) {
    const int ns = (int)wall[1] + (int)wall[2] + (int)wall[3] + (int)wall[4];
    if (ns > 0) {
      // rho1 / (rho1 + rho2) from the reciprocal, corrected by its residual
      const double q = (double)rho1 * (double)irt;
      const double phi = __builtin_fma(__builtin_fma(-q, (double)rho1 + (double)rho2, (double)rho1), (double)irt, q);
      const double rr = a.k_r * (double)ns * phi;
      double dm, keep;
      if (VAR && a.c_eq > 0.0) {
        const double excess = (double)C > a.c_eq ? (double)C - a.c_eq : 0.0;
        dm = rr * excess;
        keep = dm > 0.0 ? 1.0 - dm / (double)C : 1.0;
      } else {
        dm = rr * (double)C;
        keep = 1.0 - rr;
      }
      const double mm = m_cur + dm;
      so.m = mm;
      so.wm = true;
#pragma unroll
      for (int q = 0; q < 5; ++q) gs[q] *= (R)keep;
      if (mm > a.threshold) {
        a.mask[idx] = (uint8_t)a.bit_cur;
        a.sstep[idx] = (int32_t)(a.step + 1);
        ev = true;
      }
    }
  }
  if (VAR && xc < a.hold_x) {
    const R Ch = (R)a.c_hold;
    gs[1] = WQ * Ch * (R(1) + CQ * ux);
    gs[2] = WQ * Ch * (R(1) + CQ * uy);
    gs[3] = WQ * Ch * (R(1) - CQ * ux);
    gs[4] = WQ * Ch * (R(1) - CQ * uy);
    gs[0] = q4 ? R(0) : (R(1) - R(4) * WQ) * Ch;
  }
  // push; at a solid axis neighbour the value bounces into the opposite link
#pragma unroll
  for (int q = 0; q < 5; ++q) so.g[q] = (float)gs[q];
  so.off[0] = idx;
  so.off[1] = wall[1] ? 3 * P + idx : 1 * P + iE;
  so.off[2] = wall[2] ? 4 * P + idx : 2 * P + iN;
  so.off[3] = wall[3] ? 1 * P + idx : 3 * P + iW;
  so.off[4] = wall[4] ? 2 * P + idx : 4 * P + iS;
}

// Stores what solute_step leaves: descriptors of the outgoing solute and the
// precipitate.
template <bool REACT>
__device__ __forceinline__ void store_solute(const SoluteOut& o, __amdgpu_buffer_rsrc_t rg,
                                             __amdgpu_buffer_rsrc_t rm, unsigned idx) {
#pragma unroll
  for (int q = 0; q < 5; ++q)
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o.g[q]), rg, (int)(4u * o.off[q]), 0, 0);
  if (REACT && o.wm) {
    const v2u mb = {(unsigned)__double2loint(o.m), (unsigned)__double2hiint(o.m)};
    __builtin_amdgcn_raw_buffer_store_b64(mb, rm, (int)(8u * idx), 0, 0);
  }
}

// One lane per wavefront reserves event-log slots for every lane that marked
// a node in this row, with a single atomic.
__device__ __forceinline__ void log_events(const StepArgs& a, bool ev, int x, int y) {
  const int lane = __lane_id();
  const unsigned long long bal = __ballot(ev);
  if (bal) {
    const int leader = __ffsll((unsigned long long)bal) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd(a.ev_count, (unsigned long long)__popcll(bal));
    base = __shfl(base, leader);
    if (ev) {
      // events of lower lanes in this row come first
      const unsigned below = __builtin_amdgcn_mbcnt_hi(
          (unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
      const unsigned long long e = base + below;
      if ((long long)e < a.ev_cap) {
        a.ev[e].x = x;
        a.ev[e].y = y;
        a.ev[e].step = a.step + 1;
      }
    }
  }
}

// Incoming populations of a node in state n rebuilt from stored moments
// (moment scheme, tau = 1).  r, vx, vy: the node's own post-collision moments
// (index 0) and those of the upstream node x - e_i of link i (index i); up[i]:
// that upstream node was fluid in state n-1.  A link whose upstream node was
// solid carries the node's own equilibrium on the opposite link (halfway
// bounce-back), i.e. the same expression with the node's velocity reversed.
// f[0] is the node's own rest equilibrium.
template <typename R>
__device__ __forceinline__ void gather_links(const float* r, const float* vx, const float* vy,
                                             const bool* up, R* f) {
  const R WA = R(1) / R(9), WD = R(1) / R(36), W0 = R(4) / R(9);
  const R r0 = (R)r[0], x0 = (R)vx[0], y0 = (R)vy[0];
  const R uu0 = x0 * x0 + y0 * y0;
  f[0] = feq<R>(W0, r0, R(0), uu0);
#define GL(i, w, EU)                                                  \
  do {                                                                \
    const R rr = up[i] ? (R)r[i] : r0;                                \
    const R ux = up[i] ? (R)vx[i] : -x0;                              \
    const R uy = up[i] ? (R)vy[i] : -y0;                              \
    const R uu = up[i] ? ux * ux + uy * uy : uu0;                     \
    f[i] = feq<R>(w, rr, EU, uu);                                     \
  } while (0)
  GL(1, WA, ux);
  GL(2, WA, uy);
  GL(3, WA, -ux);
  GL(4, WA, -uy);
  GL(5, WD, ux + uy);
  GL(6, WD, -ux + uy);
  GL(7, WD, -ux - uy);
  GL(8, WD, ux - uy);
#undef GL
}

// Density and momentum of nine populations (the summation order of the
// population step).
template <typename R>
__device__ __forceinline__ void moments9(const R* f, R& rho, R& jx, R& jy) {
  rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
  jx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]);
  jy = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
}

// Cross-lane moves within one wavefront (DPP wave shifts): from_left(v) in
// lane t is v of lane t-1, from_right(v) is v of lane t+1; the end lane
// without a source reads 0.  Called with every lane active.
__device__ __forceinline__ int from_left_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x138, 0xF, 0xF, true);  // wave_shr:1
}
__device__ __forceinline__ int from_right_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x130, 0xF, 0xF, true);  // wave_shl:1
}
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(from_left_i(__float_as_int(v)));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(from_right_i(__float_as_int(v)));
}
__device__ __forceinline__ double from_left(double v) {
  return __hiloint2double(from_left_i(__double2hiint(v)), from_left_i(__double2loint(v)));
}
__device__ __forceinline__ double from_right(double v) {
  return __hiloint2double(from_right_i(__double2hiint(v)), from_right_i(__double2loint(v)));
}

// Solid nodes of a row as lane masks: bit t is lane t.  A neighbour row's or
// column's solidity is then a scalar shift of a mask, and a 0/1 value per lane
// one select (on_lane).
typedef unsigned long long lanes_t;
__device__ __forceinline__ bool on_lane(lanes_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// The eight neighbours of every lane's node from the masks of the row below,
// the row itself and the row above; index = link, E, N, W, S, NE, NW, SW, SE.
struct Neighbours {
  lanes_t n[9];
  __device__ __forceinline__ Neighbours(lanes_t dn, lanes_t own, lanes_t up)
      : n{0, own >> 1, up, own << 1, dn, up >> 1, up << 1, dn << 1, dn >> 1} {}
  __device__ __forceinline__ lanes_t any() const {
    return ((n[1] | n[2]) | (n[3] | n[4])) | ((n[5] | n[6]) | (n[7] | n[8]));
  }
};

// Weighted sum of the links to solid neighbours.
template <typename R>
__device__ __forceinline__ void wall_links(const Neighbours& solid, R& csx, R& csy) {
  const R WA = R(1) / R(9), WD = R(1) / R(36);
  csx = R(0);
  csy = R(0);
  if (solid.any()) {  // the same for all lanes
    auto w = [&](int i) { return on_lane(solid.n[i]) ? 1 : 0; };
    const int ne_sw = w(5) - w(7), se_nw = w(8) - w(6);
    csx = WA * R(w(1) - w(3)) + WD * R(ne_sw + se_nw);
    csy = WA * R(w(2) - w(4)) + WD * R(ne_sw - se_nw);
  }
}

// Which links of every lane's node lead to a solid node, as factors 0 and 1;
// any: some link of some fluid lane does (a node solid itself sends nothing).
template <typename R>
struct Bounce {
  bool any;   // the same for all lanes
  bool none;  // no lane is fluid: the row sends nothing
  R s[9];
  __device__ __forceinline__ Bounce(const Neighbours& solid, lanes_t row)
      : any((solid.any() & ~row) != 0), none(~row == 0) {
#pragma unroll
    for (int i = 0; i < 9; ++i) s[i] = R(0);
    if (any) {
#pragma unroll
      for (int i = 1; i < 9; ++i) s[i] = on_lane(solid.n[i]) ? R(1) : R(0);
    }
  }
};

// One component's outgoing equilibria of every lane's node from its stored
// moments (zero moments: nothing goes out), handed to `to`: to.up(o2, o5, o6)
// gets the links into the row above, to.down(o4, o7, o8) those into the row
// below, to.own(r, x) what adds (r, x, 0) to the accumulators (rho, jx, jy) of
// the row itself (the rest and horizontal links, streamed along the row by DPP
// wave shifts) and to.bounced(r, x, y) what bounces back (to.unbounced() where
// nothing does on any lane).  Called with every lane active.
// With u3 = 3 v: w rho (1 + 3 e.v + 9/2 (e.v)^2 - 3/2 v^2)
//              = w rho (cc + e3 (1 + e3 / 2)), e3 = e . u3, cc = 1 - u3^2 / 6.
template <typename R, typename To>
__device__ __forceinline__ void stream_row(float rho_s, float vx, float vy, const Bounce<R>& bounce,
                                           To&& to) {
  if (bounce.none) {  // inside a wall: a sixth of a sweep's rows
    to.up(R(0), R(0), R(0));
    to.down(R(0), R(0), R(0));
    to.own(R(0), R(0));
    to.unbounced();
    return;
  }
  const R WA = R(1) / R(9), WD = R(1) / R(36), WR = R(4) / R(9);
  const R rho = (R)rho_s;
  const R ux = R(3) * (R)vx, uy = R(3) * (R)vy;
  const R cc = fmar(ux * ux + uy * uy, R(-1) / R(6), R(1));
  const R ra = WA * rho, rd = WD * rho;
  auto out = [&](R r, R e3) { return r * fmar(e3, fmar(e3, R(0.5), R(1)), cc); };
  const R o0 = WR * rho * cc;
  const R o1 = out(ra, ux), o2 = out(ra, uy), o3 = out(ra, -ux), o4 = out(ra, -uy);
  const R o5 = out(rd, ux + uy), o6 = out(rd, uy - ux), o7 = out(rd, -ux - uy),
          o8 = out(rd, ux - uy);
  to.up(o2, o5, o6);
  to.down(o4, o7, o8);
  // rest and horizontal links (1, 3)
  const R a1 = from_left(o1), a3 = from_right(o3);
  to.own((o0 + a1) + a3, a1 - a3);
  // a value streaming into a solid node bounces back into the sender's
  // opposite link: rho += o_i, j -= e_i o_i
  if (bounce.any) {
    const R* s = bounce.s;
    R br = s[1] * o1, bx = s[3] * o3, by = s[4] * o4;
    br = fmar(s[2], o2, br); br = fmar(s[3], o3, br);
    br = fmar(s[4], o4, br); br = fmar(s[5], o5, br);
    br = fmar(s[6], o6, br); br = fmar(s[7], o7, br);
    br = fmar(s[8], o8, br);
    bx = fmar(-s[1], o1, bx); bx = fmar(-s[5], o5, bx);
    bx = fmar(s[6], o6, bx); bx = fmar(s[7], o7, bx);
    bx = fmar(-s[8], o8, bx);
    by = fmar(-s[2], o2, by); by = fmar(-s[5], o5, by);
    by = fmar(-s[6], o6, by); by = fmar(s[7], o7, by);
    by = fmar(s[8], o8, by);
    to.bounced(br, bx, by);
  } else {
    to.unbounced();
  }
}

// stream_row into the accumulators of the rows above (started by it), own and
// below (completed by it).
template <typename R>
struct RowSums {
  R *above, *row, *below;
  __device__ __forceinline__ void up(R o2, R o5, R o6) const {
    const R a5 = from_left(o5), a6 = from_right(o6);
    above[0] = above[2] = (o2 + a5) + a6;
    above[1] = a5 - a6;
  }
  __device__ __forceinline__ void own(R r, R x) const {
    row[0] += r;
    row[1] += x;
  }
  __device__ __forceinline__ void bounced(R r, R x, R y) const {
    row[0] += r;
    row[1] += x;
    row[2] += y;
  }
  __device__ __forceinline__ void unbounced() const {}
  __device__ __forceinline__ void down(R o4, R o7, R o8) const {
    const R a7 = from_right(o7), a8 = from_left(o8);
    const R v = (o4 + a7) + a8;
    below[0] += v;
    below[1] += a8 - a7;
    below[2] -= v;
  }
};

// Where a collided row goes: buffer descriptors of the outgoing moments, the
// outgoing solute and the precipitate, and the byte stride of a plane.
struct MomentOut {
  __amdgpu_buffer_rsrc_t m, g, prec;
  unsigned PB;
};

// Collision of the node (xc, y) of a complete row in the moment scheme: forces
// from the density window (rows W0 above, W1 own, W2 below, each centre, left
// and right of both components, zero at solids), new moments, solute,
// reaction and growth, and all stores.  rC: the node's (rho, jx, jy) per
// component; own: its mask byte; solid: its neighbours solid in state n; gv:
// its solute populations; prec(): its precipitate.
template <bool SOLUTE, bool REACT, bool VAR, typename R, typename Prec>
__device__ __forceinline__ void collide_moments(const StepArgs& a, const MomentOut& o, const R* rC,
                                                const R* W0, const R* W1, const R* W2,
                                                unsigned own, const Neighbours& solid,
                                                unsigned SCUR, const float* gv, Prec&& prec, int xc,
                                                int xl, int xr, int y, unsigned idx, bool& ev) {
  const int nx = a.nx, ny = a.ny;
  const unsigned P = (unsigned)a.P;
  // outgoing moments; zero at a node solid in state n, which no reader of
  // the next state takes as fluid.  Every owned lane stores, so each plane
  // is written as whole rows rather than lines with holes at solids.
  float mo[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  if (own & SCUR) {
    if (REACT) {
      if (own & a.bit_p1) {
        // turned solid at the end of the previous step: book what it carried
        a.drop[idx] = (float)rC[0];
        a.drop[P + idx] = (float)rC[3];
        a.drop[2 * P + idx] =
            SOLUTE ? (float)((((R)gv[0] + (R)gv[1]) + ((R)gv[2] + (R)gv[3])) + (R)gv[4]) : 0.0f;
      } else if (own & a.bit_p2) {
        a.mask[idx] = 1;  // booked one step ago: fold the mark into bit0
      }
    }
  } else {
    // neighbours x + e_i, link order 1..8 = E, N, W, S, NE, NW, SW, SE
    const R n1[9] = {R(0), W1[4], W0[0], W1[2], W2[0], W0[4], W0[2], W2[2], W2[4]};
    const R n2[9] = {R(0), W1[5], W0[1], W1[3], W2[1], W0[5], W0[3], W2[3], W2[5]};
    R csx, csy;
    wall_links<R>(solid, csx, csy);
    R F1x, F1y, F2x, F2y;
    sc_forces<R>(a, n1, n2, csx, csy, rC[0], rC[3], F1x, F1y, F2x, F2y);
    R v1x, v1y, v2x, v2y, ux, uy, irt;
    // tau = 1 in the moment scheme
    sc_velocities<R>(R(1), rC[0], rC[3], rC[1], rC[2], rC[4], rC[5], F1x, F1y, F2x, F2y, v1x, v1y,
                     v2x, v2y, ux, uy, irt);
    mo[0] = (float)rC[0];
    mo[1] = (float)v1x;
    mo[2] = (float)v1y;
    mo[3] = (float)rC[3];
    mo[4] = (float)v2x;
    mo[5] = (float)v2y;
    if (SOLUTE) {
      const int yd = y == 0 ? ny - 1 : y - 1;
      const int yu = y == ny - 1 ? 0 : y + 1;
      const unsigned iE = (unsigned)y * nx + xr, iW = (unsigned)y * nx + xl;
      const unsigned iN = (unsigned)yu * nx + xc, iS = (unsigned)yd * nx + xc;
      const double mC = REACT ? prec() : 0.0;
      SoluteOut so;
      const bool wall[5] = {false, on_lane(solid.n[1]), on_lane(solid.n[2]), on_lane(solid.n[3]),
                            on_lane(solid.n[4])};
      solute_step<REACT, VAR, R>(a, gv, ux, uy, rC[0], rC[3], irt, wall, mC, P, idx, iE, iN, iW, iS, xc, ev,
                                 so);
      store_solute<REACT>(so, o.g, o.prec, idx);
    }
  }
#pragma unroll
  for (int q = 0; q < 6; ++q)
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(mo[q]), o.m, (int)(4u * idx),
                                          (int)((unsigned)q * o.PB), 0);
}

// Moment step (tau = 1), one wavefront per workgroup: lane t holds column
// x0 - 2 + t and the workgroup owns the 60 columns of lanes 2..61.  At
// iteration k the lanes take the stored moments of row k (ys - 2 + k) and
// evaluate the eight outgoing equilibria of their node (zero at nodes solid
// in state n-1).  Each value is added to the accumulator (rho_s, j_s) of the
// node it streams to: same lane for vertical links, the neighbouring lane
// (DPP wave shift) for the others; a value streaming into a solid node is
// bounced back into the sender's own accumulator on the opposite link.  Row
// k-1 is then complete; its densities (zero at solids in state n) join a
// three-row window held in registers, from which row k-2 is collided: forces,
// new moments, solute, reaction and growth.
//
// Memory: the moments of row k+1 and the solute populations and precipitate
// of row k-1 are copied from HBM straight into an LDS double buffer (no
// registers held while in flight) before row k is computed, and the mask two
// rows ahead into a register, so one iteration's arithmetic covers the next
// iteration's memory latency.  The summation order of every node is fixed,
// so results do not depend on the tile shape.
//
// NT: the copies of data that only this wavefront reads in the step carry
// the non-temporal cache hint: the moments of the tile's own rows and the
// solute populations.  The two halo rows at each end (rows of the
// neighbouring segments, which read them too) and the precipitate (read here
// and rewritten by the same wavefront an iteration later) keep the normal
// policy.  Whether the hint pays depends on how the step's footprint meets
// the caches, so the single-lattice step takes it as an autotuned choice.
//
// BATCH: rows that are nothing but wall (a sixth of a capillary sweep's) are
// skipped.  A single lattice streams them: there the branch costs more than it
// saves, on a preform that has no such rows (2048^2 with the hint, 12 rows: 100.1
// us with it, 97.8 without) and on a capillary a third of which is wall (16384x256
// with the hint, 9 rows: 96.4, 94.6; without the hint 96.0, 95.8).
template <bool SOLUTE, bool REACT, bool VAR, typename R, bool NT, bool BATCH>
__device__ __forceinline__ void mom_wave(const StepArgs& a, int strip, int seg) {
  // prefetch slots per buffer: 0..5 moments, 6..10 solute, 11..12 precipitate
  __shared__ float pf[2][13][64];
  const int t = threadIdx.x;
  const int nx = a.nx, ny = a.ny;
  const unsigned P = (unsigned)a.P;
  const int x0 = strip * a.tx_owned;
  const int nown = min(a.tx_owned, nx - x0);
  const bool active = t <= nown + 3;
  const bool owner = t >= 2 && t <= nown + 1;
  int xc = x0 - 2 + t;
  if (xc < 0) xc += nx;
  if (xc >= nx) xc -= nx;
  const int xl = xc == 0 ? nx - 1 : xc - 1;
  const int xr = xc == nx - 1 ? 0 : xc + 1;
  const int ys = seg * a.sy;
  const int ye = min(ys + a.sy, ny);
  const int nrows = ye - ys + 4;
  const unsigned SPREV = 1u | a.bit_p2;    // solid in state n-1
  const unsigned SCUR = SPREV | a.bit_p1;  // solid in state n
  // Buffer descriptors: one per array, plane q at scalar offset q * P * 4
  // bytes, so an access costs one 32-bit lane offset per row instead of a
  // 64-bit address per plane.  The extent covers every plane the kernel
  // touches: the hardware checks lane offset plus scalar offset against it,
  // and a lane beyond it reads 0 and drops its store.
  const unsigned PB = P * 4u;
  const auto rMin = make_rsrc(a.fin, 6u * PB);
  const auto rGin = make_rsrc(a.gin, SOLUTE ? 5u * PB : 0u);
  const auto rMask = make_rsrc(a.mask, P);
  const auto rPrec = make_rsrc(a.m, REACT ? 2u * PB : 0u);
  const MomentOut o{make_rsrc(a.fout, 6u * PB), make_rsrc(a.gout, SOLUTE ? 5u * PB : 0u), rPrec, PB};

  auto row_y = [&](int k) {
    int yr = ys - 2 + k;
    if (yr < 0) yr += ny;
    if (yr >= ny) yr -= ny;
    return yr;
  };
  auto mask_at = [&](int k) -> unsigned {
    return (active && k < nrows)
               ? (unsigned)__builtin_amdgcn_raw_buffer_load_b8(
                     rMask, (int)((unsigned)row_y(k) * (unsigned)nx + (unsigned)xc), 0, 0)
               : 1u;
  };
  using lds_ptr = __attribute__((address_space(3))) void*;
  // One dword per lane at byte offset voff + soff into prefetch slot
  // (buf, slot), with the normal cache policy (to_lds) or the non-temporal
  // one (to_lds_nt).
  auto to_lds = [&](__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, int buf, int slot) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)&pf[buf][slot][0], 4, (int)voff, (int)soff,
                                             0, 0);
  };
  auto to_lds_nt = [&](__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, int buf, int slot) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)&pf[buf][slot][0], 4, (int)voff, (int)soff,
                                             0, CPOL_NT);
  };
  // Copy row k's moments (fluid nodes of state n-1) and row k-2's solute
  // and precipitate (fluid owned nodes, precipitate only next to a wall of
  // state n) into buffer buf.  Every lane issues every load; a lane with
  // nothing to copy gives a lane offset past every extent (such an offset
  // stays out of range whatever scalar offset is added), so the hardware
  // writes 0 to its slot without touching memory, and the reader needs no
  // select.
  constexpr unsigned NONE = 0xFFFFFFF0u;
  auto prefetch = [&](int buf, int k, unsigned m_k, unsigned mm3, unsigned mm2, unsigned mm1) {
    if (k >= nrows) return;
    const bool got_m = active && !(m_k & SPREV);
    const unsigned vm = got_m ? 4u * ((unsigned)row_y(k) * (unsigned)nx + (unsigned)xc) : NONE;
    if (NT && k >= 2 && k < nrows - 2) {
#pragma unroll
      for (int q = 0; q < 6; ++q) to_lds_nt(rMin, vm, (unsigned)q * PB, buf, q);
    } else {
#pragma unroll
      for (int q = 0; q < 6; ++q) to_lds(rMin, vm, (unsigned)q * PB, buf, q);
    }
    if (SOLUTE && k >= 4) {
      const unsigned i = (unsigned)(ys + k - 4) * (unsigned)nx + (unsigned)xc;
      const bool got_g = owner && !(mm2 & SPREV);
      const unsigned vg = got_g ? 4u * i : NONE;
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        if (NT) to_lds_nt(rGin, vg, (unsigned)q * PB, buf, 6 + q);
        else to_lds(rGin, vg, (unsigned)q * PB, buf, 6 + q);
      }
      if (REACT) {
        const lanes_t row = __ballot(mm2 & SCUR);
        const lanes_t wall = (row >> 1) | (row << 1) | __ballot(mm1 & SCUR) | __ballot(mm3 & SCUR);
        const bool got_p = owner && on_lane(wall & ~row);
        const unsigned vp = got_p ? 8u * i : NONE;
        to_lds(rPrec, vp, 0u, buf, 11);
        to_lds(rPrec, vp, 4u, buf, 12);
      }
    }
  };

  // mask bytes of rows k-3 .. k+1 (rows outside the tile read as solid)
  unsigned m_m3 = 1, m_m2 = 1, m_m1 = 1;
  unsigned m_0 = mask_at(0);
  unsigned m_ahead = mask_at(1);  // of row k+1 (then k+2)
  prefetch(0, 0, m_0, m_m3, m_m2, m_m1);

  R acc0[6], acc1[6];  // (rho1, j1x, j1y, rho2, j2x, j2y) of rows k and k-1
#pragma unroll
  for (int q = 0; q < 6; ++q) { acc0[q] = R(0); acc1[q] = R(0); }
  R rC[6];  // complete (rho, j) of row k-2
#pragma unroll
  for (int q = 0; q < 6; ++q) rC[q] = R(0);
  // density window (zero at solids of state n): centre, from left, from right
  R W1[6], W2[6];  // rows k-2, k-3: (c1, c2, l1, l2, r1, r2)
#pragma unroll
  for (int q = 0; q < 6; ++q) { W1[q] = R(0); W2[q] = R(0); }

  for (int k = 0; k < nrows; ++k) {
    const int buf = k & 1;
    // everything requested during the previous iteration has arrived
    __builtin_amdgcn_s_waitcnt(VMCNT0);
    const unsigned m_p1 = m_ahead;
    // buffer buf holds row k's moments and row k-2's solute and precipitate
    // (0 where nothing was copied)
    auto take = [&](int slot) { return pf[buf][slot][t]; };
    // requests for the next iteration: row k+1's moments, row k-1's solute,
    // the mask of row k+2
    prefetch(buf ^ 1, k + 1, m_p1, m_m2, m_m1, m_0);
    m_ahead = mask_at(k + 2);

    const bool crow = k >= 4 && owner;
    const int yC = ys + k - 4;
    const unsigned idxC = (unsigned)(crow ? yC : 0) * (unsigned)nx + (unsigned)xc;

    // neighbours solid in state n-1, from which values bounce back
    const lanes_t row0 = __ballot(m_0 & SPREV);
    const Neighbours prev(__ballot(m_m1 & SPREV), row0, __ballot(m_p1 & SPREV));
    Bounce<R> bounce(prev, row0);
    if (!BATCH) bounce.none = false;

    // ---- sources of row k: outgoing equilibria, streamed -----------------
    R accN[6];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      stream_row<R>(take(3 * c), take(3 * c + 1), take(3 * c + 2), bounce,
                    RowSums<R>{accN + 3 * c, acc0 + 3 * c, acc1 + 3 * c});

    // ---- row k-1 complete: density window --------------------------------
    R W0[6];
    {
      const bool s1 = (m_m1 & SCUR) != 0u;
      const R d1 = s1 ? R(0) : acc1[0], d2 = s1 ? R(0) : acc1[3];
      W0[0] = d1; W0[1] = d2;
      W0[2] = from_left(d1); W0[3] = from_left(d2);
      W0[4] = from_right(d1); W0[5] = from_right(d2);
    }

    // ---- collide row k-2 ---------------------------------------------------
    bool ev = false;
    const Neighbours cur(__ballot(m_m3 & SCUR), __ballot(m_m2 & SCUR), __ballot(m_m1 & SCUR));
    if (crow) {
      float gv[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) gv[q] = take(6 + q);
      auto prec = [&]() {
        return __hiloint2double(__float_as_int(pf[buf][12][t]), __float_as_int(pf[buf][11][t]));
      };
      collide_moments<SOLUTE, REACT, VAR, R>(a, o, rC, W0, W1, W2, m_m2, cur, SCUR, gv, prec, xc, xl, xr,
                                             yC, idxC, ev);
    }
    if (REACT) log_events(a, ev, xc, yC);

    // ---- rotate ------------------------------------------------------------
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      rC[q] = acc1[q];
      acc1[q] = acc0[q];
      acc0[q] = accN[q];
      W2[q] = W1[q];
      W1[q] = W0[q];
    }
    m_m3 = m_m2;
    m_m2 = m_m1;
    m_m1 = m_0;
    m_0 = m_p1;
  }
  // drain: no request may still be writing this wavefront's LDS at exit
  __builtin_amdgcn_s_waitcnt(VMCNT0);
}

// Short tiles of the moment step: one wavefront per row.  A tile of sy owned
// rows takes sy + 4 wavefronts; wavefront k holds row ys - 2 + k.  All loads of
// the tile are issued at once, every wavefront streams its row's equilibria
// (vertical and diagonal links through LDS), completes its row, publishes its
// densities in LDS and collides it.  The additions to a node happen in the
// order of mom_wave (from below, own row, from above), so the results are
// bit-identical to it.
//
// What bounds it: on a small lattice latency.  A few hundred rows of 64 nodes
// leave most SIMDs idle, and there mom_wave's sy + 4 row iterations in series
// (1.1-1.9 us each) are the step; here a step is one memory round trip, two
// LDS exchanges and one row's arithmetic (256x32 without solute: 3.65 us a
// step against 6.6 for mom_wave's best height).  On one that fills the chip
// arithmetic: it does (sy + 4) / sy times the streaming work, 577 vector
// instructions per owned row of 60 nodes at eight rows (counted; they keep the
// SIMDs busy for 70% of a step at 1448^2), but with 24 wavefronts per CU
// resident (72 VGPRs, 74 KB LDS) instead of mom_wave's 12: 1024^2 preform 26.7
// us against 35.2, 700x500 11.1 against 16.1.  Eight rows because two workgroups of
// 12 wavefronts share a CU's LDS; nine to twelve leave one (launch_rows).
static_assert(SHORT_TILE + 4 <= 16, "one wavefront per row within a workgroup");

// stream_row with the vertical links into LDS rows of LROW values (lane t at
// t + 1, so a diagonal link is read from the neighbouring column), the rest
// kept.
constexpr int LROW = 66;
template <typename R>
struct RowShares {
  R *s_up, *s_dn;  // [3][LROW]
  bool has_up, has_dn;
  R r, x, b[3];
  __device__ __forceinline__ void up(R o2, R o5, R o6) {
    if (has_up) { s_up[0] = o2; s_up[LROW] = o5; s_up[2 * LROW] = o6; }
  }
  __device__ __forceinline__ void own(R r_, R x_) { r = r_; x = x_; }
  __device__ __forceinline__ void bounced(R r_, R x_, R y_) { b[0] = r_; b[1] = x_; b[2] = y_; }
  __device__ __forceinline__ void unbounced() { bounced(R(0), R(0), R(0)); }
  __device__ __forceinline__ void down(R o4, R o7, R o8) {
    if (has_dn) { s_dn[0] = o4; s_dn[LROW] = o7; s_dn[2 * LROW] = o8; }
  }
};

template <bool SOLUTE, bool REACT, bool VAR, typename R>
__device__ __forceinline__ void mom_rows(const StepArgs& a, int strip, int seg, char* lds_raw) {
  // links of both components out of rows 0 .. nrows-3 (up) and 2 .. nrows-1
  // (down), densities of rows 1 .. nrows-2
  const int nin = a.sy + 2;
  R(*s_up)[2][3 * LROW] = (R(*)[2][3 * LROW])lds_raw;
  R(*s_dn)[2][3 * LROW] = s_up + nin;
  R(*s_rho)[2][LROW] = (R(*)[2][LROW])(s_dn + nin);
  const int t = threadIdx.x & 63;
  const int k = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nx = a.nx, ny = a.ny;
  const unsigned PB = (unsigned)a.P * 4u;
  const int x0 = strip * a.tx_owned;
  const int nown = min(a.tx_owned, nx - x0);
  const bool active = t <= nown + 3;
  const bool owner = t >= 2 && t <= nown + 1;
  int xc = x0 - 2 + t;
  if (xc < 0) xc += nx;
  if (xc >= nx) xc -= nx;
  const int xl = xc == 0 ? nx - 1 : xc - 1;
  const int xr = xc == nx - 1 ? 0 : xc + 1;
  const int ys = seg * a.sy;
  const int nrows = min(a.sy, ny - ys) + 4;
  const bool live = k < nrows;                     // the last tile may be shorter
  const bool inner = k >= 1 && k < nrows - 1;      // rows whose sums are complete
  const bool crow = k >= 2 && k < nrows - 2;       // owned rows
  int y = ys - 2 + k;
  if (y < 0) y += ny;
  if (y >= ny) y -= ny;
  const unsigned SPREV = 1u | a.bit_p2;    // solid in state n-1
  const unsigned SCUR = SPREV | a.bit_p1;  // solid in state n
  constexpr unsigned NONE = 0xFFFFFFF0u;   // past every extent: reads 0
  const auto rMin = make_rsrc(a.fin, 6u * PB);
  const auto rGin = make_rsrc(a.gin, SOLUTE ? 5u * PB : 0u);
  const auto rMask = make_rsrc(a.mask, (unsigned)a.P);
  const auto rPrec = make_rsrc(a.m, REACT ? 2u * PB : 0u);
  const MomentOut o{make_rsrc(a.fout, 6u * PB), make_rsrc(a.gout, SOLUTE ? 5u * PB : 0u), rPrec, PB};

  const unsigned idx = (unsigned)y * (unsigned)nx + (unsigned)xc;
  float mo[6], gv[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  unsigned m0 = 1, md = 1, mu = 1;
  v2u pr = {0u, 0u};
  RowShares<R> sh[2];
  if (live) {
    const unsigned yd = y == 0 ? ny - 1 : y - 1, yu = y == ny - 1 ? 0 : y + 1;
    auto mask_of = [&](unsigned row) -> unsigned {
      const unsigned v = (unsigned)__builtin_amdgcn_raw_buffer_load_b8(
          rMask, (int)(active ? row * (unsigned)nx + (unsigned)xc : NONE), 0, 0);
      return active ? v : 1u;
    };
    m0 = mask_of((unsigned)y);
    md = mask_of(yd);
    mu = mask_of(yu);
    auto load_moments = [&](unsigned vm) {
#pragma unroll
      for (int q = 0; q < 6; ++q) mo[q] = load_f32<false>(rMin, vm, (unsigned)q * PB);
    };
    // a node solid in state n-1 holds zeros (every step that stores moments
    // writes them there), so the loads need not wait for the mask (written in
    // place instead of called, they are scheduled otherwise: 1024^2 at five rows
    // 36.2 us instead of 33.0)
    load_moments(active ? 4u * idx : NONE);
    const lanes_t row = __ballot(m0 & SPREV);
    const Neighbours prev(__ballot(md & SPREV), row, __ballot(mu & SPREV));
    const bool fluid = on_lane(~row);
    if (crow) {
      if (SOLUTE) {
        const unsigned vg = owner && fluid ? 4u * idx : NONE;
#pragma unroll
        for (int q = 0; q < 5; ++q)
          gv[q] = load_f32<false>(rGin, vg, (unsigned)q * PB);
      }
      if (REACT) {
        const lanes_t here = __ballot(m0 & SCUR);
        const lanes_t wall = (here >> 1) | (here << 1) | __ballot(md & SCUR) | __ballot(mu & SCUR);
        pr = __builtin_amdgcn_raw_buffer_load_b64(
            rPrec, (int)(owner && on_lane(wall & ~here) ? 8u * idx : NONE), 0, 0);
      }
    }
    const Bounce<R> bounce(prev, row);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      sh[c].has_up = k < nrows - 2;
      sh[c].has_dn = k >= 2;
      sh[c].s_up = &s_up[k < nrows - 2 ? k : 0][c][t + 1];
      sh[c].s_dn = &s_dn[k >= 2 ? k - 2 : 0][c][t + 1];
      stream_row<R>(mo[3 * c], mo[3 * c + 1], mo[3 * c + 2], bounce, sh[c]);
    }
  }
  lds_barrier();

  R acc[6], W1[6];
  if (inner) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const R* su = &s_up[k - 1][c][t + 1];
      const R* sd = &s_dn[k - 1][c][t + 1];
      const R a5 = su[LROW - 1], a6 = su[2 * LROW + 1];
      const R u = (su[0] + a5) + a6;
      acc[3 * c] = (u + sh[c].r) + sh[c].b[0];
      acc[3 * c + 1] = ((a5 - a6) + sh[c].x) + sh[c].b[1];
      acc[3 * c + 2] = u + sh[c].b[2];
      const R a7 = sd[LROW + 1], a8 = sd[2 * LROW - 1];
      const R d = (sd[0] + a7) + a8;
      acc[3 * c] += d;
      acc[3 * c + 1] += a8 - a7;
      acc[3 * c + 2] -= d;
    }
    const bool s1 = (m0 & SCUR) != 0u;
    W1[0] = s1 ? R(0) : acc[0];
    W1[1] = s1 ? R(0) : acc[3];
    s_rho[k - 1][0][t + 1] = W1[0];
    s_rho[k - 1][1][t + 1] = W1[1];
  }
  lds_barrier();

  if (!crow) return;
  bool ev = false;
  const Neighbours cur(__ballot(md & SCUR), __ballot(m0 & SCUR), __ballot(mu & SCUR));
  if (owner) {
    R W0[6], W2[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const int at = t + (q < 2 ? 1 : q < 4 ? 0 : 2);
      if (q >= 2) W1[q] = s_rho[k - 1][q & 1][at];
      W0[q] = s_rho[k][q & 1][at];
      W2[q] = s_rho[k - 2][q & 1][at];
    }
    auto prec = [&]() { return __hiloint2double((int)pr.y, (int)pr.x); };
    collide_moments<SOLUTE, REACT, VAR, R>(a, o, acc, W0, W1, W2, m0, cur, SCUR, gv, prec, xc, xl, xr, y,
                                           idx, ev);
  }
  if (REACT) log_events(a, ev, xc, y);
}

// Population step (any tau), one wavefront per row: lane t holds column
// x0 - 1 + t, and a workgroup owns at most the 62 columns of lanes 1..62 and at
// most POP_ROWS rows (blockIdx.y counts them in taller tiles, see launch_rows):
// wavefront k holds the row below them (k = 0), one of them, or the row above.
// Every wavefront loads its row's populations at once, publishes the densities in
// LDS, and collides and pushes its row (the two halo rows only publish).  The rest
// population is rho minus the moving ones, so the collision conserves mass exactly.
// OUTM (tau = 1 only): store the moments (rho_s, v_s) of the collided node, zero at
// solids, instead of pushing populations.
//
// What bounds it: the round trips and the bandwidth of 23 planes read and
// written.  Rows in parallel put a tile's loads in flight together.  The
// densities and momenta are summed as the populations arrive, and the
// populations then wait in LDS until the collision takes them one by one: 78
// VGPRs and no spill keep 24 wavefronts per CU (held in registers they spilled:
// 1023x1024 41.0 us per step against 34.2 at six rows, 700x500 16.5 against
// 14.6, 2048^2 258 against 245).  us per step, against workgroups that marched
// up their rows (best shape): 1023x1024 preform 34.2 against 42.0, 2048^2 237
// against 250 (hint), 1024x64 capillary 6.2 against 7.2.

// What a wavefront of pop_rows keeps in LDS: its row's densities, lane t at
// t + 1, for the neighbouring rows, and its own lanes' populations.
struct PopRow {
  double rho[2][LROW];
  float f[18][64];
};
template <bool SOLUTE, bool REACT, bool VAR, typename R, bool OUTM, bool NT>
__device__ __forceinline__ void pop_rows(const StepArgs& a, int strip, int seg, char* lds_raw) {
  const int t = threadIdx.x & 63;
  const int k = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  PopRow* const row = (PopRow*)lds_raw + k;
  const int nx = a.nx, ny = a.ny;
  const unsigned P = (unsigned)a.P;
  const int x0 = strip * a.tx_owned;
  const int nown = min(a.tx_owned, nx - x0);
  const bool active = t <= nown + 1;
  const bool owner = t >= 1 && t <= nown;
  int xc = x0 - 1 + t;
  if (xc < 0) xc += nx;
  if (xc >= nx) xc -= nx;
  const int xl = xc == 0 ? nx - 1 : xc - 1;
  const int xr = xc == nx - 1 ? 0 : xc + 1;
  const int ys = seg * a.sy + POP_ROWS * (int)blockIdx.y;
  const int ye = min((seg + 1) * a.sy, ny);
  if (ys >= ye) return;  // the whole workgroup
  const int nrows = min(POP_ROWS, ye - ys) + 2;
  const bool live = k < nrows;
  const bool crow = k >= 1 && k < nrows - 1;
  int y = ys - 1 + k;
  if (y < 0) y += ny;
  if (y >= ny) y -= ny;
  const int yd = y == 0 ? ny - 1 : y - 1, yu = y == ny - 1 ? 0 : y + 1;
  const unsigned SPREV = 1u | a.bit_p2;    // solid in state n-1
  const unsigned SCUR = SPREV | a.bit_p1;  // solid in state n
  const unsigned idx = (unsigned)y * (unsigned)nx + (unsigned)xc;
  constexpr unsigned NONE = 0xFFFFFFF0u;   // past every extent: reads 0, stores nothing
  const unsigned PB = P * 4u;
  // one descriptor per component: nine planes stay below 2^32 bytes
  const auto rF1 = make_rsrc(a.fin, 9u * PB), rF2 = make_rsrc(a.fin + 9ll * P, 9u * PB);
  const auto rO1 = make_rsrc(a.fout, 9u * PB), rO2 = make_rsrc(a.fout + 9ll * P, 9u * PB);
  const auto rGin = make_rsrc(a.gin, SOLUTE ? 5u * PB : 0u);
  const auto rGout = make_rsrc(a.gout, SOLUTE ? 5u * PB : 0u);
  const auto rMask = make_rsrc(a.mask, P);
  const auto rPrec = make_rsrc(a.m, REACT ? 2u * PB : 0u);
  auto store = [](__amdgpu_buffer_rsrc_t r, R v, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)v), r, (int)voff, (int)soff, 0);
  };

  float g[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) g[q] = 0.0f;
  v2u pr = {0u, 0u};
  unsigned m0 = 1, md = 1, mu = 1;
  R rho1 = R(0), rho2 = R(0), j1x = R(0), j1y = R(0), j2x = R(0), j2y = R(0);
  if (live) {
    float f[18];
    auto mask_of = [&](unsigned yr) -> unsigned {
      const unsigned v = (unsigned)__builtin_amdgcn_raw_buffer_load_b8(
          rMask, (int)(active ? yr * (unsigned)nx + (unsigned)xc : NONE), 0, 0);
      return active ? v : 1u;
    };
    m0 = mask_of((unsigned)y);
    if (crow) {
      md = mask_of((unsigned)yd);
      mu = mask_of((unsigned)yu);
    }
    const unsigned vf = m0 & SPREV ? NONE : 4u * idx;
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = load_f32<NT>(rF1, vf, (unsigned)q * PB);
#pragma unroll
    for (int q = 0; q < 9; ++q) f[9 + q] = load_f32<NT>(rF2, vf, (unsigned)q * PB);
    if (crow) {
      if (SOLUTE) {
        const unsigned vg = owner ? vf : NONE;
#pragma unroll
        for (int q = 0; q < 5; ++q) g[q] = load_f32<NT>(rGin, vg, (unsigned)q * PB);
      }
      if (REACT) {
        const lanes_t here = __ballot(m0 & SCUR);
        const lanes_t wall = (here >> 1) | (here << 1) | __ballot(md & SCUR) | __ballot(mu & SCUR);
        pr = __builtin_amdgcn_raw_buffer_load_b64(
            rPrec, (int)(owner && on_lane(wall & ~here) ? 8u * idx : NONE), 0, 0);
      }
    }
    if (!(m0 & SCUR)) {
      rho1 = sum9<R>(f);
      rho2 = sum9<R>(f + 9);
    }
    row->rho[0][t + 1] = rho1;
    row->rho[1][t + 1] = rho2;
    if (crow) {
      j1x = ((R)f[1] - (R)f[3]) + ((R)f[5] - (R)f[6]) + ((R)f[8] - (R)f[7]);
      j1y = ((R)f[2] - (R)f[4]) + ((R)f[5] + (R)f[6]) - ((R)f[7] + (R)f[8]);
      j2x = ((R)f[10] - (R)f[12]) + ((R)f[14] - (R)f[15]) + ((R)f[17] - (R)f[16]);
      j2y = ((R)f[11] - (R)f[13]) + ((R)f[14] + (R)f[15]) - ((R)f[16] + (R)f[17]);
#pragma unroll
      for (int q = 0; q < 18; ++q) row->f[q][t] = f[q];
    }
  }
  lds_barrier();
  if (!crow) return;
  auto pop = [&](int q) { return (R)row->f[q][t]; };

  bool ev = false;
  const Neighbours cur(__ballot(md & SCUR), __ballot(m0 & SCUR), __ballot(mu & SCUR));
  if (owner) {
    if (m0 & SCUR) {
      if (REACT) {
        if (m0 & a.bit_p1) {
          // turned solid at the end of the previous step: book its populations
          float f[18];
#pragma unroll
          for (int q = 0; q < 18; ++q) f[q] = row->f[q][t];
          a.drop[idx] = (float)sum9<R>(f);
          a.drop[P + idx] = (float)sum9<R>(f + 9);
          a.drop[2 * P + idx] =
              SOLUTE ? (float)((((R)g[0] + (R)g[1]) + ((R)g[2] + (R)g[3])) + (R)g[4]) : 0.0f;
        } else if (m0 & a.bit_p2) {
          a.mask[idx] = 1;  // booked one step ago: fold the mark into bit0
        }
      }
      if (OUTM) {
#pragma unroll
        for (int q = 0; q < 6; ++q) store(rO1, R(0), 4u * idx, (unsigned)q * PB);
      }
    } else {
      const R* up = &row[1].rho[0][t + 1];
      const R* at = &row[0].rho[0][t + 1];
      const R* dn = &row[-1].rho[0][t + 1];
      const R n1[9] = {R(0), at[1], up[0], at[-1], dn[0], up[1], up[-1], dn[-1], dn[1]};
      const R n2[9] = {R(0), at[LROW + 1], up[LROW], at[LROW - 1], dn[LROW], up[LROW + 1],
                       up[LROW - 1], dn[LROW - 1], dn[LROW + 1]};
      bool wall[9];
#pragma unroll
      for (int i = 1; i < 9; ++i) wall[i] = on_lane(cur.n[i]);
      R csx, csy;
      wall_links<R>(cur, csx, csy);
      R F1x, F1y, F2x, F2y;
      sc_forces<R>(a, n1, n2, csx, csy, rho1, rho2, F1x, F1y, F2x, F2y);
      R v1x, v1y, v2x, v2y, ux, uy, irt;
      sc_velocities<R>((R)a.tau, rho1, rho2, j1x, j1y, j2x, j2y, F1x, F1y, F2x, F2y, v1x, v1y, v2x,
                       v2y, ux, uy, irt);
      const unsigned iE = (unsigned)y * nx + xr, iW = (unsigned)y * nx + xl;
      const unsigned iN = (unsigned)yu * nx + xc, iS = (unsigned)yd * nx + xc;
      if (SOLUTE) {
        SoluteOut so;
        solute_step<REACT, VAR, R>(a, g, ux, uy, rho1, rho2, irt, wall,
                                   __hiloint2double((int)pr.y, (int)pr.x), P, idx, iE, iN, iW, iS, xc, ev,
                                   so);
        store_solute<REACT>(so, rGout, rPrec, idx);
      }
      if (OUTM) {
        const R mo[6] = {rho1, v1x, v1y, rho2, v2x, v2y};
#pragma unroll
        for (int q = 0; q < 6; ++q) store(rO1, mo[q], 4u * idx, (unsigned)q * PB);
      } else {
        const unsigned iNE = (unsigned)yu * nx + xr, iNW = (unsigned)yu * nx + xl;
        const unsigned iSW = (unsigned)yd * nx + xl, iSE = (unsigned)yd * nx + xr;
        const R om = (R)a.omega;
        // collide one component and push each moving population as soon as
        // it is formed (halfway bounce-back into the node's own opposite
        // link at a solid neighbour); the rest population closes the mass
        // balance exactly (the moving-link weights are not exact binary
        // fractions)
        auto collide_push = [&](int q0, __amdgpu_buffer_rsrc_t r, R rho, R vx, R vy) {
          const R uu = vx * vx + vy * vy;
          R sum = R(0);
#define CP(i, opp, w, eu, tgt)                                              \
  do {                                                                      \
    const R fi = pop(q0 + i);                                                \
    const R v = fi + om * (feq<R>(w, rho, eu, uu) - fi);                    \
    sum += v;                                                               \
    store(r, v, wall[i] ? (opp) * PB + 4u * idx : (i) * PB + 4u * (tgt), 0);  \
  } while (0)
          const R WA = R(1) / R(9), WD = R(1) / R(36);
          CP(1, 3, WA, vx, iE);
          CP(2, 4, WA, vy, iN);
          CP(3, 1, WA, -vx, iW);
          CP(4, 2, WA, -vy, iS);
          CP(5, 7, WD, vx + vy, iNE);
          CP(6, 8, WD, -vx + vy, iNW);
          CP(7, 5, WD, -vx - vy, iSW);
          CP(8, 6, WD, vx - vy, iSE);
#undef CP
          store(r, rho - sum, 4u * idx, 0);
        };
        collide_push(0, rO1, rho1, v1x, v1y);
        collide_push(9, rO2, rho2, v2x, v2y);
      }
    }
  }
  if (REACT) log_events(a, ev, xc, y);
}

// XCD-aware order: the hardware hands block b to XCD b mod 8, so XCD x
// receives q + (x < r) of T blocks (q = T / 8, r = T mod 8).  Give each XCD a
// contiguous run of tiles.  Tiles are numbered segment-major, so a run is a
// horizontal band of full rows: the waves resident on one XCD read whole
// rows together (DRAM pages stay open), and both halo directions are shared
// in one L2 except at the band's edges.
__host__ __device__ inline int xcd_tile(int b, int T) {
  const int q = T >> 3, r = T & 7, x = b & 7, j = b >> 3;
  return (x < r) ? x * (q + 1) + j : r * (q + 1) + (x - r) * q + j;
}

template <bool SOLUTE, bool REACT, bool VAR, typename R, int KIND, bool NT, bool BATCH>
__device__ __forceinline__ void run_tile(const StepArgs& a, int strip, int seg, char* lds_raw) {
  if constexpr (KIND == KIND_MM)
    mom_wave<SOLUTE, REACT, VAR, R, NT, BATCH>(a, strip, seg);
  else if constexpr (KIND == KIND_MM_SHORT)
    mom_rows<SOLUTE, REACT, VAR, R>(a, strip, seg, lds_raw);
  else
    pop_rows<SOLUTE, REACT, VAR, R, KIND == KIND_PM, NT>(a, strip, seg, lds_raw);
}

// Largest workgroup and register budget (waves per SIMD) of each kind.
template <int KIND>
constexpr int max_threads() { return KIND == KIND_MM ? 64 : 64 * 16; }
template <int KIND>
constexpr int min_waves() { return KIND == KIND_MM ? 3 : 6; }

template <bool SOLUTE, bool REACT, bool VAR, typename R, int KIND, bool NT>
__global__ void __launch_bounds__(max_threads<KIND>()) __attribute__((amdgpu_waves_per_eu(min_waves<KIND>(), 8)))
k_step(const StepArgs a) {
  extern __shared__ char lds_raw[];
  const int T = a.nstrips * a.nsegs;
  const int tile = a.remap ? xcd_tile(blockIdx.x, T) : (int)blockIdx.x;
  const int seg = tile / a.nstrips;
  run_tile<SOLUTE, REACT, VAR, R, KIND, NT, false>(a, tile - seg * a.nstrips, seg, lds_raw);
}

// Batched step: one launch advances every instance of a batch by one step.
// Block b takes tile tiles[b] (instance, strip, segment; the host orders the
// list per XCD); the instance's arguments for the current parity come from
// device memory, and the step index is the device counter *stepc plus the
// launch's offset j within its sequence.  A sequence of n launches (offsets
// 0..n-1) is followed by k_tick(stepc, n), so a captured sequence replays
// from where the last one ended.
template <bool SOLUTE, bool REACT, bool VAR, typename R, int KIND>
__global__ void __launch_bounds__(max_threads<KIND>()) __attribute__((amdgpu_waves_per_eu(min_waves<KIND>(), 8)))
k_step_batch(const StepArgs* __restrict__ insts, const int4* __restrict__ tiles,
             const long long* __restrict__ stepc, int j) {
  extern __shared__ char lds_raw[];
  const long long step = *stepc + j;
  const int4 e = tiles[blockIdx.x];
  StepArgs a = insts[2 * e.x + (int)(step & 1)];
  a.step = step;
  a.bit_p1 = pending_bit(step - 1);
  a.bit_p2 = pending_bit(step - 2);
  a.bit_cur = pending_bit(step);
  run_tile<SOLUTE, REACT, VAR, R, KIND, false, true>(a, e.y, e.z, lds_raw);
}

// Advances the device step counter by n (one lane).
__global__ void k_tick(long long* stepc, int n) {
  if (threadIdx.x == 0) *stepc += n;
}

// Rest-state populations from the FP64 densities (rounded once to FP32).
__global__ void k_init(const double* __restrict__ rho1, const double* __restrict__ rho2,
                       const double* __restrict__ conc, const uint8_t* __restrict__ mask,
                       float* __restrict__ f, float* __restrict__ g, double* __restrict__ m,
                       int32_t* __restrict__ sstep, float* __restrict__ drop, long long N,
                       long long P, int solute, int react, int q4) {
  const float w9[9] = {4.0f / 9.0f, 1.0f / 9.0f, 1.0f / 9.0f, 1.0f / 9.0f, 1.0f / 9.0f,
                       1.0f / 36.0f, 1.0f / 36.0f, 1.0f / 36.0f, 1.0f / 36.0f};
  const float w5[5] = {q4 ? 0.0f : 1.0f / 3.0f, q4 ? 0.25f : 1.0f / 6.0f, q4 ? 0.25f : 1.0f / 6.0f,
                       q4 ? 0.25f : 1.0f / 6.0f, q4 ? 0.25f : 1.0f / 6.0f};
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const bool s = mask[i] != 0;
    const float r1 = s ? 0.0f : (float)rho1[i];
    const float r2 = s ? 0.0f : (float)rho2[i];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      f[q * P + i] = w9[q] * r1;
      f[(9 + q) * P + i] = w9[q] * r2;
    }
    if (solute) {
      const float c = s ? 0.0f : (float)conc[i];
#pragma unroll
      for (int q = 0; q < 5; ++q) g[q * P + i] = w5[q] * c;
    }
    if (react) {
      m[i] = 0.0;
      sstep[i] = s ? 0 : -1;
      drop[i] = 0.0f;
      drop[P + i] = 0.0f;
      drop[2 * P + i] = 0.0f;
    }
  }
}

// ---- observers -------------------------------------------------------------
// Node densities and momenta of state n, from stored populations or, in the
// moment scheme, gathered from the stored moments of the node and its
// upstream neighbours (the same arithmetic as the moment step, in FP64).
struct PopSrc {
  const float* __restrict__ f;
  long long P;
  __device__ void rho(long long i, int, int, double& r1, double& r2) const {
    double a = 0, b = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      a += (double)f[q * P + i];
      b += (double)f[(9 + q) * P + i];
    }
    r1 = a;
    r2 = b;
  }
  __device__ void full(long long i, int, int, double* o) const {
    const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    double r1 = 0, r2 = 0, j1x = 0, j1y = 0, j2x = 0, j2y = 0;
    for (int q = 0; q < 9; ++q) {
      const double a = f[q * P + i], b = f[(9 + q) * P + i];
      r1 += a; r2 += b;
      j1x += a * ex[q]; j1y += a * ey[q];
      j2x += b * ex[q]; j2y += b * ey[q];
    }
    o[0] = r1; o[1] = r2; o[2] = j1x; o[3] = j1y; o[4] = j2x; o[5] = j2y;
  }
};

struct MomSrc {
  const float* __restrict__ M;
  const uint8_t* __restrict__ mask;
  long long P;
  int nx, ny;
  unsigned sprev;  // solid bits of state n-1
  __device__ void links(int x, int y, int comp, double* fl) const {
    const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    float r[9], vx[9], vy[9];
    bool up[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      int xs = x - ex[q], ysrc = y - ey[q];
      xs = xs < 0 ? xs + nx : (xs >= nx ? xs - nx : xs);
      ysrc = ysrc < 0 ? ysrc + ny : (ysrc >= ny ? ysrc - ny : ysrc);
      const long long k = (long long)ysrc * nx + xs;
      up[q] = !(mask[k] & sprev);
      r[q] = M[(3 * comp) * P + k];
      vx[q] = M[(3 * comp + 1) * P + k];
      vy[q] = M[(3 * comp + 2) * P + k];
    }
    gather_links<double>(r, vx, vy, up, fl);
  }
  __device__ void full(long long, int x, int y, double* o) const {
    double fl[9];
    links(x, y, 0, fl);
    moments9<double>(fl, o[0], o[2], o[3]);
    links(x, y, 1, fl);
    moments9<double>(fl, o[1], o[4], o[5]);
  }
  __device__ void rho(long long i, int x, int y, double& r1, double& r2) const {
    double o[6];
    full(i, x, y, o);
    r1 = o[0];
    r2 = o[1];
  }
};

constexpr int OBS_THREADS = 512;

// Sum over a wavefront, in a fixed order; the result is in lane 0.
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
  return v;
}

// One block's FP64 partial sums over its nodes.  Slots: 0 mass1, 1 mass2,
// 2 solute, 3 precipitate, 4 removed1, 5 removed2, 6 removed solute, 7 solid
// count, 8 non-finite count.
template <typename Src>
__device__ void partial_sums(const Src& src, const float* __restrict__ g,
                             const uint8_t* __restrict__ mask, const double* __restrict__ m,
                             const float* __restrict__ drop, int nx, long long N, long long P,
                             unsigned p1, unsigned p2, int solute, int react, int block,
                             int nblocks, double* __restrict__ partial) {
  __shared__ double red[OBS_SLOTS][OBS_THREADS / 64];
  const unsigned sprev = 1u | p2, scur = sprev | p1;
  double acc[OBS_SLOTS];
#pragma unroll
  for (int j = 0; j < OBS_SLOTS; ++j) acc[j] = 0.0;
  for (long long i = block * (long long)OBS_THREADS + threadIdx.x; i < N;
       i += (long long)nblocks * OBS_THREADS) {
    const unsigned b = mask[i];
    double s1 = 0, s2 = 0, sc = 0;
    if (!(b & sprev)) {
      src.rho(i, (int)(i % nx), (int)(i / nx), s1, s2);
      if (solute) {
#pragma unroll
        for (int q = 0; q < 5; ++q) sc += (double)g[q * P + i];
      }
    }
    if (b & scur) {
      acc[7] += 1.0;
      if (b & p1) {  // turned solid at the end of the last step, not yet booked
        acc[4] += s1;
        acc[5] += s2;
        acc[6] += sc;
      }
    } else {
      acc[0] += s1;
      acc[1] += s2;
      acc[2] += sc;
      if (!isfinite(s1) || !isfinite(s2) || !isfinite(sc)) acc[8] += 1.0;
    }
    if (react) {
      acc[3] += m[i];
      acc[4] += (double)drop[i];
      acc[5] += (double)drop[P + i];
      acc[6] += (double)drop[2 * P + i];
    }
  }
#pragma unroll
  for (int j = 0; j < OBS_SLOTS; ++j) {
    const double v = wave_sum(acc[j]);
    if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < OBS_SLOTS) {
    double v = 0.0;
    for (int w = 0; w < OBS_THREADS / 64; ++w) v += red[threadIdx.x][w];
    partial[block * OBS_SLOTS + threadIdx.x] = v;
  }
}

// Capillary observables computed by one workgroup of OBS_THREADS threads, one
// column per thread and pass: the centreline front and, with FULL, largest
// grown width, first closure, and the sums behind the radii of Fig. 4.  out:
// [0] z, [1] delta_e, [2] closure step (-1 if none), [3] open area A (fluid
// nodes between the walls), [4] narrowest open column, [5] sum over
// neighbouring columns of |h(x+1) - h(x)|, h the growth on the lower wall.
// sb: solid bits of state n.
//
// What bounds it: round trips to memory.  Each column's wetting fraction is
// formed once and its neighbour's taken from LDS, and a column's mask bytes
// are read in one pass with independent loads; the front alone stops at the
// pass that holds it.  A 1024-column capillary took 51 us with 256 threads
// that evaluated every column twice and followed each wall by dependent loads
// (the fronts of 34 runs 105 us), and takes 15 us with the sums beside it (9.3 us).
template <bool FULL, typename Src>
__device__ void capillary_obs(const Src& src, const uint8_t* __restrict__ mask,
                              const int32_t* __restrict__ sstep, int nx, unsigned sb, int x_in,
                              int x_out, int y0, int W, int react, double* __restrict__ out) {
  constexpr int T = OBS_THREADS;
  __shared__ double s_phi[T];
  __shared__ int s_blocked[T], s_db[T];
  __shared__ int s_x[T], s_area[T], s_wmin[T], s_steps[T];
  __shared__ double s_z[T], s_de[T];
  __shared__ long long s_cl[T];
  const int t = threadIdx.x;
  const int nr = (W % 2 == 0) ? 2 : 1;
  const int row0 = (W % 2 == 0) ? (y0 + W / 2 - 1) : (y0 + (W - 1) / 2);
  int best = x_out;  // this thread's first x where the scan stops, and z there
  double z = (double)(x_out - x_in);
  double de = 0.0;
  long long cl = -1;
  int area = 0, wmin = W, steps = 0;
  // each pass decides the columns of T - 1 threads; the last one's only serves
  // as a neighbour, and is the next pass's first
  for (int xb = x_in; xb < x_out; xb += T - 1) {
    const int x = xb + t;
    bool blocked = false;
    double phi = 0;
    int db = 0, dt = 0, w = 0;
    if (x < x_out) {
      for (int r = 0; r < nr; ++r) {
        const long long i = (long long)(row0 + r) * nx + x;
        if (mask[i] & sb) blocked = true;
        else { double a, b; src.rho(i, x, row0 + r, a, b); phi += a / (a + b); }
      }
      phi /= nr;
      if (FULL) {  // growth from the two walls and fluid nodes of this column
        int lo = W, hi = -1;  // lowest and highest fluid node
#pragma unroll 8
        for (int y = 0; y < W; ++y) {
          const bool fluid = !(mask[(long long)(y0 + y) * nx + x] & sb);
          w += fluid ? 1 : 0;
          lo = fluid && lo == W ? y : lo;
          hi = fluid ? y : hi;
        }
        db = lo;
        dt = hi < 0 ? W : W - 1 - hi;
      }
    }
    s_phi[t] = phi;
    s_blocked[t] = blocked;
    if (FULL) s_db[t] = db;
    __syncthreads();
    const bool next = x + 1 < x_out;
    if (x < x_out && t < T - 1) {
      const double phin = next ? s_phi[t + 1] : 0.0;
      const bool crossing = next && !s_blocked[t + 1] && phi >= 0.5 && phin < 0.5;
      const bool dry = x == x_in && phi < 0.5;
      if ((blocked || dry || crossing) && x < best) {
        best = x;
        z = blocked ? (double)(x - x_in) : dry ? 0.0 : (double)x + (phi - 0.5) / (phi - phin) - x_in;
      }
      if (FULL) {
        area += w;
        wmin = min(wmin, w);
        if (next) steps += abs(s_db[t + 1] - db);
        double col;
        if (db >= W) {
          col = 0.5 * W;
          long long last = 0;
          if (react)
            for (int y = y0; y < y0 + W; ++y) {
              const long long st = sstep[(long long)y * nx + x];
              if (st > last) last = st;
            }
          if (cl < 0 || last < cl) cl = last;
        } else {
          col = (double)(db > dt ? db : dt);
        }
        if (col > de) de = col;
      }
    }
    // (also orders the reads above before the next pass's writes)
    const int found = __syncthreads_or(best < x_out);
    if (!FULL && found) break;
  }
  s_x[t] = best;
  s_z[t] = z;
  if (FULL) {
    s_de[t] = de;
    s_cl[t] = cl;
    s_area[t] = area;
    s_wmin[t] = wmin;
    s_steps[t] = steps;
  }
  __syncthreads();
  for (int s = T / 2; s > 0; s >>= 1) {
    if (t < s) {
      if (s_x[t + s] < s_x[t]) {
        s_x[t] = s_x[t + s];
        s_z[t] = s_z[t + s];
      }
      if (FULL) {
        s_area[t] += s_area[t + s];
        s_wmin[t] = min(s_wmin[t], s_wmin[t + s]);
        s_steps[t] += s_steps[t + s];
        s_de[t] = fmax(s_de[t], s_de[t + s]);
        const long long o = s_cl[t + s];
        if (o >= 0 && (s_cl[t] < 0 || o < s_cl[t])) s_cl[t] = o;
      }
    }
    __syncthreads();
  }
  if (t == 0) {
    out[0] = s_z[0];
    if (FULL) {
      out[1] = s_de[0];
      out[2] = (double)s_cl[0];
      out[3] = (double)s_area[0];
      out[4] = (double)s_wmin[0];
      out[5] = (double)s_steps[0];
    }
  }
}

// Observe, pass 1: block 0 the capillary (W > 0), the others partial sums.
template <typename Src>
__global__ void __launch_bounds__(OBS_THREADS)
k_observe(Src src, const float* __restrict__ g, const uint8_t* __restrict__ mask,
          const double* __restrict__ m, const float* __restrict__ drop,
          const int32_t* __restrict__ sstep, int nx, long long N, long long P, unsigned p1,
          unsigned p2, int solute, int react, int nblocks, int x_in, int x_out, int y0, int W,
          double* __restrict__ partial, double* __restrict__ out) {
  const int first = W > 0 ? 1 : 0;
  if ((int)blockIdx.x < first)
    capillary_obs<true>(src, mask, sstep, nx, 1u | p1 | p2, x_in, x_out, y0, W, react, out + OBS_SLOTS);
  else
    partial_sums(src, g, mask, m, drop, nx, N, P, p1, p2, solute, react, (int)blockIdx.x - first,
                 nblocks, partial);
}

// Observe, pass 2: fixed-order sum of the partials (deterministic; one
// wavefront per slot, 42-164 us when one lane added a slot's 256-1024 values
// in series) and the event count.
__global__ void __launch_bounds__(64 * OBS_SLOTS)
k_obs_final(const double* __restrict__ partial, int nblocks,
            const unsigned long long* __restrict__ ev_count, double* __restrict__ out) {
  const int j = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double s = 0.0;
  for (int b = lane; b < nblocks; b += 64) s += partial[b * OBS_SLOTS + j];
  s = wave_sum(s);
  if (lane == 0) out[j] = s;
  if (threadIdx.x == 0) out[OBS_OUT - 1] = __longlong_as_double((long long)*ev_count);
}

// Front of every instance of a batch (workgroup i -> instance i) into column
// `slot` of the n x nslots table; queued without synchronisation.
__global__ void __launch_bounds__(OBS_THREADS)
k_front_batch(const StepArgs* __restrict__ insts, const int4* __restrict__ capi,
              const long long* __restrict__ stepc, int slot, int nslots, int mom,
              double* __restrict__ table) {
  const long long step = *stepc;
  const int i = blockIdx.x;
  const StepArgs& a = insts[2 * i + (int)(step & 1)];
  const int4 c = capi[i];  // x_in, x_out, y0, W
  double* z = table + (long long)i * nslots + slot;
  if (c.w <= 0) {
    if (threadIdx.x == 0) *z = __builtin_nan("");
    return;
  }
  const unsigned p1 = pending_bit(step - 1), p2 = pending_bit(step - 2);
  const unsigned sb = 1u | p1 | p2;
  if (mom) {
    const MomSrc src{a.fin, a.mask, a.P, a.nx, a.ny, 1u | p2};
    capillary_obs<false>(src, a.mask, a.sstep, a.nx, sb, c.x, c.y, c.z, c.w, a.react, z);
  } else {
    const PopSrc src{a.fin, a.P};
    capillary_obs<false>(src, a.mask, a.sstep, a.nx, sb, c.x, c.y, c.z, c.w, a.react, z);
  }
}

// Macroscopic fields of the current state as FP64 planes, the selected ones
// (bits of sel: 0 rho1, 1 rho2, 2 ux, 3 uy, 4 conc, 5 precipitate, 6 solid)
// one after another in `out`.  The velocities need the neighbours' densities:
// with a velocity selected this pass also leaves both densities in planes 7
// and 8 of `out`, and k_velocity fills in ux and uy from them.
template <typename Src>
__global__ void k_fields(Src src, const float* __restrict__ g, const uint8_t* __restrict__ mask,
                         const double* __restrict__ m, int nx, long long N, long long P, unsigned sb,
                         int solute, int react, unsigned sel, double* __restrict__ out) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const bool s = (mask[i] & sb) != 0;
    double r1 = 0, r2 = 0, c = 0;
    if (!s && (sel & 0xFu)) src.rho(i, (int)(i % nx), (int)(i / nx), r1, r2);
    if (!s && solute && (sel & 16u))
#pragma unroll
      for (int q = 0; q < 5; ++q) c += g[q * P + i];
    const double v[7] = {r1, r2, 0.0, 0.0, c, react && (sel & 32u) ? m[i] : 0.0, s ? 1.0 : 0.0};
    double* o = out + i;
#pragma unroll
    for (int b = 0; b < 7; ++b) {
      if (!(sel & (1u << b))) continue;
      if (b != 2 && b != 3) *o = v[b];
      o += N;
    }
    if (sel & 0xCu) {
      out[7 * N + i] = r1;
      out[8 * N + i] = r2;
    }
  }
}

template <typename Src>
__global__ void k_velocity(Src src, const uint8_t* __restrict__ mask, int nx, int ny, unsigned sb,
                           double G, double Gads1, double Gads2, double ax, double ay,
                           const double* __restrict__ rho1, const double* __restrict__ rho2,
                           double* __restrict__ out_x, double* __restrict__ out_y) {
  const long long N = (long long)nx * ny;
  const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  const double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    double ux = 0, uy = 0;
    if (!(mask[i] & sb)) {
      const int x = (int)(i % nx), y = (int)(i / nx);
      double o[6];
      src.full(i, x, y, o);
      const double r1 = o[0], r2 = o[1];
      double c1x = 0, c1y = 0, c2x = 0, c2y = 0, sx = 0, sy = 0;
#pragma unroll
      for (int q = 1; q < 9; ++q) {
        int xn = x + ex[q], yn = y + ey[q];
        xn = xn < 0 ? xn + nx : (xn >= nx ? xn - nx : xn);
        yn = yn < 0 ? yn + ny : (yn >= ny ? yn - ny : yn);
        const long long k = (long long)yn * nx + xn;
        const double f = (mask[k] & sb) ? 1.0 : 0.0;
        sx += w[q] * f * ex[q]; sy += w[q] * f * ey[q];
        const double a = rho1[k], b = rho2[k];  // zero at solids
        c1x += w[q] * a * ex[q]; c1y += w[q] * a * ey[q];
        c2x += w[q] * b * ex[q]; c2y += w[q] * b * ey[q];
      }
      const double F1x = -G * r1 * c2x - Gads1 * r1 * sx + r1 * ax;
      const double F1y = -G * r1 * c2y - Gads1 * r1 * sy + r1 * ay;
      const double F2x = -G * r2 * c1x - Gads2 * r2 * sx + r2 * ax;
      const double F2y = -G * r2 * c1y - Gads2 * r2 * sy + r2 * ay;
      ux = (o[2] + o[4] + 0.5 * (F1x + F2x)) / (r1 + r2);
      uy = (o[3] + o[5] + 0.5 * (F1y + F2y)) / (r1 + r2);
    }
    if (out_x) out_x[i] = ux;
    if (out_y) out_y[i] = uy;
  }
}

// Populations of state n rebuilt from the stored moments (zero at nodes that
// were solid in state n-1, which carry none).
__global__ void k_unpack(MomSrc src, float* __restrict__ fout) {
  const long long N = (long long)src.nx * src.ny;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N;
       i += (long long)gridDim.x * blockDim.x) {
    const int x = (int)(i % src.nx), y = (int)(i / src.nx);
    const bool fluid = !(src.mask[i] & src.sprev);
    for (int comp = 0; comp < 2; ++comp) {
      double fl[9];
      if (fluid) src.links(x, y, comp, fl);
#pragma unroll
      for (int q = 0; q < 9; ++q) fout[(9 * comp + q) * src.P + i] = fluid ? (float)fl[q] : 0.0f;
    }
  }
}

// ---- launchers ------------------------------------------------------------
// Threads per workgroup: one wavefront per tile in the moment step, one per
// row (halo rows included) otherwise.
static int step_threads(int kind, int sy) {
  return kind == KIND_MM ? 64 : 64 * (kind == KIND_MM_SHORT ? sy + 4 : (sy < POP_ROWS ? sy : POP_ROWS) + 2);
}

// LDS beyond the static part: see mom_rows and pop_rows.
static size_t step_lds_bytes(int kind, int threads) {
  if (kind == KIND_MM) return 0;
  const size_t rows = threads / 64;
  return kind == KIND_MM_SHORT ? (rows - 2) * (2 * 6 + 2) * LROW * sizeof(double) : rows * sizeof(PopRow);
}

// Workgroups of T tiles: a population tile taller than POP_ROWS takes several.
static dim3 step_grid(int kind, int sy, int T) {
  return dim3(T, kind == KIND_POP || kind == KIND_PM ? (sy + POP_ROWS - 1) / POP_ROWS : 1);
}

// Runs that use a reaction or solute-lattice variant (saturation, held
// source, D2Q4) take their own instantiation, so the plain model keeps its
// instruction stream.
inline bool uses_variants(const StepArgs& a) { return a.c_eq > 0.0 || a.hold_x > 0 || a.q4; }

template <typename R, int KIND, bool NT>
void launch_step_t(const StepArgs& a, int T, int tx, size_t lds, hipStream_t st) {
  if (a.solute && a.react && uses_variants(a))
    hipLaunchKernelGGL((k_step<true, true, true, R, KIND, NT>), step_grid(KIND, a.sy, T), dim3(tx), lds, st, a);
  else if (a.solute && a.react)
    hipLaunchKernelGGL((k_step<true, true, false, R, KIND, NT>), step_grid(KIND, a.sy, T), dim3(tx), lds, st, a);
  else if (a.solute && uses_variants(a))
    hipLaunchKernelGGL((k_step<true, false, true, R, KIND, NT>), step_grid(KIND, a.sy, T), dim3(tx), lds, st, a);
  else if (a.solute)
    hipLaunchKernelGGL((k_step<true, false, false, R, KIND, NT>), step_grid(KIND, a.sy, T), dim3(tx), lds, st, a);
  else
    hipLaunchKernelGGL((k_step<false, false, false, R, KIND, NT>), step_grid(KIND, a.sy, T), dim3(tx), lds, st, a);
}

// nt: the non-temporal load hint, compiled for the marching moment step and the
// population step (moment_kind says why not for short tiles; the one-off PM step
// ignores it too).  The arithmetic is FP64 throughout.
hipError_t launch_step(const StepArgs& a, int kind, int nt, hipStream_t st) {
  const int T = a.nstrips * a.nsegs;
  const int tx = step_threads(kind, a.sy);
  const size_t lds = step_lds_bytes(kind, tx);
  switch (kind + (nt ? 8 : 0)) {
    case KIND_MM: launch_step_t<double, KIND_MM, false>(a, T, tx, lds, st); break;
    case KIND_MM + 8: launch_step_t<double, KIND_MM, true>(a, T, tx, lds, st); break;
    case KIND_MM_SHORT:
    case KIND_MM_SHORT + 8: launch_step_t<double, KIND_MM_SHORT, false>(a, T, tx, lds, st); break;
    case KIND_POP: launch_step_t<double, KIND_POP, false>(a, T, tx, lds, st); break;
    case KIND_POP + 8: launch_step_t<double, KIND_POP, true>(a, T, tx, lds, st); break;
    default: launch_step_t<double, KIND_PM, false>(a, T, tx, lds, st);
  }
  return hipGetLastError();
}

template <typename R, int KIND>
void launch_batch_t(const StepArgs* insts, const int4* tiles, int ntiles, const long long* stepc,
                    int j, int sy, int tx, int solute, int react, int var, size_t lds, hipStream_t st) {
  if (solute && react && var)
    hipLaunchKernelGGL((k_step_batch<true, true, true, R, KIND>), step_grid(KIND, sy, ntiles), dim3(tx), lds, st, insts, tiles, stepc, j);
  else if (solute && react)
    hipLaunchKernelGGL((k_step_batch<true, true, false, R, KIND>), step_grid(KIND, sy, ntiles), dim3(tx), lds, st, insts, tiles, stepc, j);
  else if (solute && var)
    hipLaunchKernelGGL((k_step_batch<true, false, true, R, KIND>), step_grid(KIND, sy, ntiles), dim3(tx), lds, st, insts, tiles, stepc, j);
  else if (solute)
    hipLaunchKernelGGL((k_step_batch<true, false, false, R, KIND>), step_grid(KIND, sy, ntiles), dim3(tx), lds, st, insts, tiles, stepc, j);
  else
    hipLaunchKernelGGL((k_step_batch<false, false, false, R, KIND>), step_grid(KIND, sy, ntiles), dim3(tx), lds, st, insts, tiles, stepc, j);
}

hipError_t launch_step_batch(const StepArgs* insts, const int4* tiles, int ntiles,
                             const long long* stepc, int j, int sy, int solute, int react, int var,
                             int kind, hipStream_t st) {
  const int tx = step_threads(kind, sy);
  const size_t lds = step_lds_bytes(kind, tx);
  if (kind == KIND_MM_SHORT) launch_batch_t<double, KIND_MM_SHORT>(insts, tiles, ntiles, stepc, j, sy, tx, solute, react, var, lds, st);
  else if (kind == KIND_MM) launch_batch_t<double, KIND_MM>(insts, tiles, ntiles, stepc, j, sy, tx, solute, react, var, lds, st);
  else if (kind == KIND_PM) launch_batch_t<double, KIND_PM>(insts, tiles, ntiles, stepc, j, sy, tx, solute, react, var, lds, st);
  else launch_batch_t<double, KIND_POP>(insts, tiles, ntiles, stepc, j, sy, tx, solute, react, var, lds, st);
  return hipGetLastError();
}

hipError_t launch_tick(long long* stepc, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, st, stepc, n);
  return hipGetLastError();
}

hipError_t launch_front_batch(const StepArgs* insts, const int4* capi, const long long* stepc,
                              int n, int slot, int nslots, int mom, double* table, hipStream_t st) {
  hipLaunchKernelGGL(k_front_batch, dim3(n), dim3(OBS_THREADS), 0, st, insts, capi, stepc, slot, nslots,
                     mom, table);
  return hipGetLastError();
}

int host_xcd_tile(int b, int T) { return xcd_tile(b, T); }

static int grid_for(long long N) { return (int)((N + 255) / 256 < 8192 ? (N + 255) / 256 : 8192); }

hipError_t launch_init(const double* r1, const double* r2, const double* c, const uint8_t* mask,
                       float* f, float* g, double* m, int32_t* sstep, float* drop, long long N,
                       long long P, int solute, int react, int q4, hipStream_t st) {
  hipLaunchKernelGGL(k_init, dim3(grid_for(N)), dim3(256), 0, st, r1, r2, c, mask, f, g, m, sstep,
                     drop, N, P, solute, react, q4);
  return hipGetLastError();
}

hipError_t launch_unpack(const float* M, const uint8_t* mask, int nx, int ny, long long P,
                         unsigned sprev, float* fout, hipStream_t st) {
  const MomSrc src{M, mask, P, nx, ny, sprev};
  hipLaunchKernelGGL(k_unpack, dim3(grid_for((long long)nx * ny)), dim3(256), 0, st, src, fout);
  return hipGetLastError();
}

hipError_t launch_observe(const float* f, const float* g, const uint8_t* mask, const double* m,
                          const float* drop, const int32_t* sstep, int nx, int ny, long long P,
                          unsigned p1, unsigned p2, int mom, int solute, int react, int max_blocks,
                          double* partial, double* out, const unsigned long long* ev_count, int x_in,
                          int x_out, int y0, int W, hipStream_t st) {
  const long long N = (long long)nx * ny;
  const int nblocks = (int)((N + OBS_THREADS - 1) / OBS_THREADS < max_blocks
                                ? (N + OBS_THREADS - 1) / OBS_THREADS : max_blocks);
  auto go = [&](const auto& src) {
    hipLaunchKernelGGL(k_observe, dim3(nblocks + (W > 0 ? 1 : 0)), dim3(OBS_THREADS), 0, st, src, g, mask,
                       m, drop, sstep, nx, N, P, p1, p2, solute, react, nblocks, x_in, x_out, y0, W,
                       partial, out);
  };
  if (mom) go(MomSrc{f, mask, P, nx, ny, 1u | p2});
  else go(PopSrc{f, P});
  hipLaunchKernelGGL(k_obs_final, dim3(1), dim3(64 * OBS_SLOTS), 0, st, partial, nblocks, ev_count, out);
  return hipGetLastError();
}

hipError_t launch_fields(const float* f, const float* g, const uint8_t* mask, const double* m,
                         int nx, int ny, long long P, unsigned p1, unsigned p2, int mom,
                         int solute, int react, double G, double Gads1, double Gads2, double ax,
                         double ay, unsigned sel, double* out, hipStream_t st) {
  const long long N = (long long)nx * ny;
  const int blocks = grid_for(N);
  const unsigned sb = 1u | p1 | p2;
  double* vx = sel & 4u ? out + N * __builtin_popcount(sel & 3u) : nullptr;
  double* vy = sel & 8u ? out + N * __builtin_popcount(sel & 7u) : nullptr;
  auto go = [&](const auto& src) {
    hipLaunchKernelGGL(k_fields, dim3(blocks), dim3(256), 0, st, src, g, mask, m, nx, N, P, sb, solute,
                       react, sel, out);
    if (vx || vy)
      hipLaunchKernelGGL(k_velocity, dim3(blocks), dim3(256), 0, st, src, mask, nx, ny, sb, G, Gads1,
                         Gads2, ax, ay, out + 7 * N, out + 8 * N, vx, vy);
  };
  if (mom) go(MomSrc{f, mask, P, nx, ny, 1u | p2});
  else go(PopSrc{f, P});
  return hipGetLastError();
}

}  // namespace lbmdev
