// Private declarations shared by the kernels and the host layer of the HIP
// library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm.h"

namespace lbmdev {

constexpr int OBS_SLOTS = 9;   // per-block partial sums of the observe reduction
constexpr int OBS_OUT = OBS_SLOTS + 7;  // + capillary: z, delta_e, closure, area, min width, steps;
                                        // last: the event count (bits of an int64)

struct StepArgs {
  const float* fin;
  float* fout;
  const float* gin;
  float* gout;
  uint8_t* mask;
  double* m;
  int32_t* sstep;
  float* drop;
  lbm_event* ev;
  unsigned long long* ev_count;
  long long ev_cap;
  long long P;        // plane stride in elements
  long long step;     // index n of the state being advanced (n -> n+1)
  int nx, ny;
  int tx_owned;       // columns owned per workgroup: 62 of 64 lanes, or 60 in the
                      // moment step, whose stencil reaches two columns out
  int sy;             // rows owned per workgroup
  int nstrips, nsegs;
  int remap;          // XCD-aware tile order (tile count divisible by 8)
  int solute, react;
  unsigned bit_p1;    // pending bit written by step n-1 (solid in state n)
  unsigned bit_p2;    // pending bit written by step n-2 (folded into bit0 now)
  unsigned bit_cur;   // pending bit this step writes
  // model parameters in FP64 (kernel arguments stay in scalar registers)
  double omega;       // 1/tau
  double tau;
  double G, Gads1, Gads2, ax, ay;
  double omega_g;     // 1/tau_g
  double k_r, threshold;
  double c_eq;        // saturation concentration of the reaction (0: plain first order)
  double c_hold;      // held concentration of the source region x < hold_x
  int hold_x;         // 0: no held source
  int q4;             // 1: D2Q4 solute lattice, 0: D2Q5
};

// The model parameters of p (solute: it has a solute lattice).
inline void set_model(StepArgs& a, const lbm_params& p, bool solute) {
  a.omega = 1.0 / p.tau;
  a.tau = p.tau;
  a.G = p.G;
  a.Gads1 = p.G_ads[0];
  a.Gads2 = p.G_ads[1];
  a.ax = p.accel[0];
  a.ay = p.accel[1];
  a.omega_g = solute ? 1.0 / p.tau_g : 0.0;
  a.k_r = p.k_r;
  a.threshold = p.threshold;
  a.c_eq = p.c_eq;
  a.c_hold = p.c_hold;
  a.hold_x = p.hold_x;
  a.q4 = p.solute_q == 4;
}

// Growth marks rotate over three pending bits: step n marks a node with
// pending_bit(n); step n+1 books the populations it carried; step n+2 folds
// the mark into bit0.  In state n the solid set of state n-1 is
// bit0 | pending(n-2) and that of state n adds pending(n-1); both stay
// readable while a step runs, whatever order its workgroups take.
__host__ __device__ inline unsigned pending_bit(long long n) {
  return 2u << (unsigned)(((n % 3) + 3) % 3);
}

// Kinds of step kernel.  POP: populations in, populations out.  At tau = 1
// the post-collision populations are the equilibria of (rho_s, v_s) of each
// component, so the state can be kept as six moments per node: PM collides
// populations and stores moments, MM reads moments (rebuilding the incoming
// populations by gathering from the neighbours) and stores moments.
enum StepKind { KIND_POP = 0, KIND_PM = 1, KIND_MM = 2, KIND_MM_SHORT = 3 };

// Which moment step runs `tiles` tiles of sy rows when the lattices it advances
// together hold `nodes` nodes: one wavefront per row (short tiles) or one marching
// up each tile.
//
// Short tiles while the step's two buffers fit the 256 MB memory-side cache.
// Measured on square preforms, us per step (best height of each): 1024^2 (92 MB)
// 26.7 against 35.2, 1448^2 (184 MB) 46.7 against 48.4, 1600^2 (225 MB) 55.6
// against 60.6, 1700^2 (254 MB) 76.8 against 77.7, 2048^2 (369 MB) 117 against 104.
// Once the reads come from HBM, the short tiles' loads (one round trip per
// workgroup, two workgroups per CU) are not covered.
//
// That is the best height's line; a set height has its own.  Eight rows and up to
// four fill a CU with two and three workgroups (24 wavefronts), five and six leave
// places empty (18 and 20) and repeat half as much again.  us per step, short
// against marching, without solute in brackets: five rows 1150^2 39.9, 40.9,
// 1600^2 71.2, 67.5 (52.3, 52.1), 2100^2 (86.5, 82.5); six rows 1250^2 44.5, 45.6
// (33.3, 35.6), 1448^2 59.2, 53.9 (43.8, 41.4), 2100^2 (84.7, 76.4).  More than
// eight are launched as eight (launch_rows): ten rows 1024^2 26.1, 33.4, twelve rows
// 1150^2 31.6, 38.3, but 34 capillaries (2.0 million nodes) 50.0, 48.3, 2100^2 (71.0,
// 67.9).
//
// Marching needs a wavefront for every SIMD: with fewer tiles than that the step
// is one wavefront's chain of rows, and tiles are short on a lattice of any size.
// us per step, marching against eight short rows: 256x32 at 16 rows 32, 5.4, 1024^2
// at 24 rows 50.5, 25.9, 1448^2 at 64 rows 122, 45.9, 2500^2 at 128 rows 260, 177.
//
// nt: the non-temporal load hint is set.  Short tiles, whose neighbours read their
// halo rows at the same time, are slower with it and run without; where there are
// many of them (low ones on large lattices) a marching wavefront with it is faster
// still.  us per step with the hint set, marching against short without it: 800^2 at
// one row (11200 tiles) 33.8, 37.3, 1024^2 at two rows (9216) 38.2, 39.7, 2100^2
// without solute at four rows (18375) 79.5, 83.7; 1024^2 at three rows (6156) 36.7,
// 34.1, at eight 37.1, 25.6, 1600^2 at eight (5400) 67.6, 55.0 (72.2 with the hint).
constexpr int SHORT_TILE = 12, SHORT_ROWS = 8, SIMDS = 1024;
inline int moment_kind(long long nodes, bool solute, int sy, long long tiles, int nt) {
  constexpr long long SHORT_BYTES = 240ll << 20, SHARED_NODES = 1400000, LOOSE_NODES = 2000000,
                      HINTED_TILES = 9000;
  if (tiles < SIMDS) return KIND_MM_SHORT;
  if (nodes * (solute ? 88 : 48) > SHORT_BYTES || (nt && tiles > HINTED_TILES)) return KIND_MM;
  if (sy > SHORT_ROWS) return nodes <= SHARED_NODES ? KIND_MM_SHORT : KIND_MM;
  return (sy == 5 || sy == 6) && nodes > LOOSE_NODES ? KIND_MM : KIND_MM_SHORT;
}

// Rows of the tiles that a step of this kind is launched with where `tiles` tiles of
// sy rows are set: several workgroups share a tall tile, which is launched as lower
// ones.
//
// Population tiles, at most POP_ROWS rows a workgroup, in parts as even as may be:
// 16 rows as 8 and 8 against 14 and 2, us per step: 1024^2 38.6, 54.1; 2048x1100 with
// the hint 113, 130; 2500^2 397, 425.
//
// Short moment tiles: nine rows and more leave a CU one workgroup with fewer rows than
// two of SHORT_ROWS have, which pays while there are hardly two for each CU.  Whole
// against eight rows, us per step, without solute in brackets: 2048x76 at 12 rows
// (245 tiles) 6.9, 7.6, 800^2 at 10 rows (1120 tiles) 25.0, 18.2, 1024^2 at 9 rows
// 33.3, 25.6 (23.9, 20.5), at 10 rows 38.0, 26.1 (30.3, 20.7).
constexpr int POP_ROWS = 14;
inline int launch_rows(int kind, int sy, long long tiles) {
  if (kind == KIND_MM) return sy;
  if (kind == KIND_MM_SHORT) return sy <= (tiles <= 512 ? SHORT_TILE : SHORT_ROWS) ? sy : SHORT_ROWS;
  const int parts = (sy + POP_ROWS - 1) / POP_ROWS;
  return (sy + parts - 1) / parts;
}

// Records a message for lbm_last_error() and returns s.
lbm_status fail(lbm_status s, const char* fmt, ...);

// nt: non-temporal load hint
hipError_t launch_step(const StepArgs& a, int kind, int nt, hipStream_t st);
// var: some instance uses a reaction or solute-lattice variant
// One batched step at index *stepc + j; a sequence of n such launches
// (j = 0..n-1) is followed by launch_tick(stepc, n).
hipError_t launch_step_batch(const StepArgs* insts, const int4* tiles, int ntiles,
                             const long long* stepc, int j, int sy, int solute, int react, int var,
                             int kind, hipStream_t st);
hipError_t launch_tick(long long* stepc, int n, hipStream_t st);
hipError_t launch_front_batch(const StepArgs* insts, const int4* capi, const long long* stepc,
                              int n, int slot, int nslots, int mom, double* table, hipStream_t st);
// Populations of state n rebuilt from stored moments (zero at nodes solid in
// state n-1) into fout[18][P].
hipError_t launch_unpack(const float* M, const uint8_t* mask, int nx, int ny, long long P,
                         unsigned sprev, float* fout, hipStream_t st);
int host_xcd_tile(int b, int T);
hipError_t launch_init(const double* r1, const double* r2, const double* c, const uint8_t* mask,
                       float* f, float* g, double* m, int32_t* sstep, float* drop, long long N,
                       long long P, int solute, int react, int q4, hipStream_t st);
// Observers of state n.  f holds populations (mom = 0) or the moments of the
// last step (mom = 1); p1, p2 are pending(n-1), pending(n-2).
hipError_t launch_observe(const float* f, const float* g, const uint8_t* mask, const double* m,
                          const float* drop, const int32_t* sstep, int nx, int ny, long long P,
                          unsigned p1, unsigned p2, int mom, int solute, int react, int max_blocks,
                          double* partial, double* out, const unsigned long long* ev_count, int x_in,
                          int x_out, int y0, int W, hipStream_t st);
// The selected fields (bits of sel) one after another; out holds nine planes.
hipError_t launch_fields(const float* f, const float* g, const uint8_t* mask, const double* m,
                         int nx, int ny, long long P, unsigned p1, unsigned p2, int mom,
                         int solute, int react, double G, double Gads1, double Gads2, double ax,
                         double ay, unsigned sel, double* out, hipStream_t st);

}  // namespace lbmdev
