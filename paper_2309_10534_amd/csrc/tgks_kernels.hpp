// tgks_kernels.hpp -- HIP kernels of one S2O4 step of the TENO-D GKS (gfx950).
//
// Per stage and direction a face kernel produces, for every face, the
// Gauss-point averaged time-integrated fluxes combined as the S2O4 update
// needs them (Sec. 2.2):
//   stage 1:  FA = F(W^n, dt/2),  FB = 8/3 F(W^n, dt/2) - 1/3 F(W^n, dt)
//   stage 2:  FA = 4/3 F(W*, dt) - 8/3 F(W*, dt/2)
// so that  W* = W^n - sum_d D_d FA / dx_d,  P = W^n - sum_d D_d FB / dx_d,
// W^{n+1} = P - sum_d D_d FA* / dx_d, algebraically the update of Sec. 2.2.
// The update kernels apply the flux differences; the stage-2 update also
// reduces the CFL time step of the new state (Sec. 5 preamble).
#pragma once
#include "tgks_flux_face.hpp"

namespace tgks {

struct Geom {
  int D;
  int n[3];
  double dx[3];
  int bclo[3], bchi[3];
  long long ncell;
};

// Prescribed sides of 1-D and 2-D grids: a ghost cell centred at s along
// the other axis (0 in 1-D) and r along the side's axis holds A where
// s < (s0 + s_n r) + s_t t, beyond the line B (far == BC_PRESCRIBED) or the
// transmissive / reflective image (far == 1 / 2).
struct Prescribed {
  int on;               // some side is prescribed
  int far[2][2];        // [axis][end]
  double A[4], B[4];    // global component order
  double line[2][2][3]; // [axis][end]: s0, s_n, s_t
};

// value of lane (lane ^ MASK), MASK = 1 or 2, by a DPP quad permute (a
// VALU move; no LDS instruction, unlike a general lane shuffle)
template <int MASK>
__device__ __forceinline__ int lane_xor(int v) {
  static_assert(MASK == 1 || MASK == 2, "quad permutes only");
  return __builtin_amdgcn_mov_dpp(v, MASK == 1 ? 0xB1 : 0x4E, 0xF, 0xF, false);
}
template <int MASK>
__device__ __forceinline__ double lane_xor(double v) {
  const int lo = lane_xor<MASK>(__double2loint(v)), hi = lane_xor<MASK>(__double2hiint(v));
  return __hiloint2double(hi, lo);
}

// value of lane 7 - i within the lane's group of eight (DPP half-row
// mirror): for a value that is the same in the four lanes of each quad, the
// other quad's value, as lane ^ 4 would give
__device__ __forceinline__ double other_quad(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x141, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x141, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// The clock {t, dt} of a step taken from the step before: t += dt, the new dt
// from the partial minima that its stage 2 left (cfl > 0; else the same dt).
// Every wavefront of the new step's stage 1 evaluates it for itself (few
// partial minima) and the grid's first writes it down, in another place than
// the old one: no kernel of its own between the steps.
//
// Up to 256 partial minima, four loads per lane, issued together: eight steps
// of 400 cells 135 us with a kernel between the steps, 119 without; of 14,000
// cells (242 partial minima) 128 and 117; of 64 x 64 291 and 277; of 256 x 256
// (256 partial minima) 624 and 615, where reading them in every block takes up
// most of the gain.
constexpr int CLOCK_NBLK = 256;

struct StepClock {
  const double* prev;     // the clock of the step before; null: none, dt is given
  double* next;
  const double* partial;
  long long* steps;       // counts the steps taken (null: not counted)
  int nblk;
  double cfl, t_end;
};

struct StageArgs {
  Geom g;
  FluxCfg fc;
  TenoCfg tn;  // normal reconstruction
  TenoCfg tt;  // tangential reconstruction
  SchemeCfg sc;  // constants of the comparison schemes (WENO-AO, TENO5, WENO-Z)
  const double* W;
  double* FA;
  double* FB;
  const double* dt;
  unsigned long long* fail;
  uint8_t* nflags;  // normal flags [D][nc][cells] or null
  uint8_t* tflags;  // tangential flags of this direction or null
  const double* R;  // 3-D: normal reconstruction of this direction
  double* Rout;
  double gamma;     // ratio of specific heats (characteristic variables)
  Prescribed pb;    // prescribed sides
  double t0;        // time of W (prescribed states) is t0 + *tclk (tclk may be null)
  const double* tclk;
  int fallback;     // 1: first-order fallback at non-physical Gauss-point states
  unsigned long long* fbc;  // fallback counter, or null (not counted)
  StepClock ck;     // stage 1 in 1-D and 2-D: the step's clock from the step before (or dt and tclk as given)
};

__device__ __forceinline__ long long face_count(const Geom& g, int ax) {
  long long c = 1;
  for (int d = 0; d < 3; ++d) c *= (long long)(d == ax ? g.n[d] + 1 : g.n[d]);
  return c;
}

// offset of the cell (i, j, k) within a component plane, ghost cells by the
// boundary index map; f0..f2 receive the mirror kinds along each axis
__device__ __forceinline__ long long cell_offset(const Geom& g, int i, int j, int k, int& f0, int& f1, int& f2) {
  f0 = f1 = f2 = 0;
  const int ii = map_index(i, g.n[0], g.bclo[0], g.bchi[0], f0);
  const int jj = g.D >= 2 ? map_index(j, g.n[1], g.bclo[1], g.bchi[1], f1) : 0;
  const int kk = g.D >= 3 ? map_index(k, g.n[2], g.bclo[2], g.bchi[2], f2) : 0;
  return ((long long)kk * g.n[1] + jj) * g.n[0] + ii;
}

// whether component c (global order) changes sign at a mirrored cell: a
// reflective wall negates the momentum normal to it, a no-slip wall every
// momentum component
__device__ __forceinline__ bool cell_flip(const Geom& g, int c, int f0, int f1, int f2) {
  if (c < 1 || c > g.D) return false;
  const int fo = c == 1 ? f0 : (c == 2 ? f1 : f2);
  return (fo == 1) ^ (f0 == 2) ^ (f1 == 2) ^ (f2 == 2);
}

// value of component c (global order) of the cell (i, j, k), ghost cells by
// the boundary index map
__device__ __forceinline__ double load_cell(const Geom& g, const double* W, int c, int i, int j, int k) {
  int f0, f1, f2;
  const long long off = cell_offset(g, i, j, k, f0, f1, f2);
  const double v = W[(long long)c * g.ncell + off];
  return cell_flip(g, c, f0, f1, f2) ? -v : v;
}

// stage 2 works on W*, the state at the half step
__device__ __forceinline__ double stage2_time(double t, double dt) {
#pragma clang fp contract(off)
  return t + 0.5 * dt;
}

// time of the prescribed states in stage STAGE of a step of length dt
__device__ __forceinline__ double boundary_time(const StageArgs& a, int stage, double dt) {
#pragma clang fp contract(off)
  if (!a.pb.on) return 0.0;
  const double t = a.t0 + (a.tclk ? *a.tclk : 0.0);
  return stage == 2 ? stage2_time(t, dt) : t;
}

// load_cell with prescribed sides resolved first (x side, then y side): the
// given state at the ghost cell's centre, or the far kind's image
__device__ __forceinline__ double cell_value(const Geom& g, const Prescribed& pb, const double* W, int c, int i,
                                             int j, double tb) {
#pragma clang fp contract(off)
  if (!pb.on) return load_cell(g, W, c, i, j, 0);
  int lo0 = g.bclo[0], hi0 = g.bchi[0], lo1 = g.bclo[1], hi1 = g.bchi[1];
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    if (d >= g.D) break;
    const int id = d == 0 ? i : j;
    const int n = g.n[d];
    if (id >= 0 && id < n) continue;
    const bool low = id < 0;
    const int kind = d == 0 ? (low ? lo0 : hi0) : (low ? lo1 : hi1);
    if (kind != BC_PRESCRIBED) continue;
    const double s = g.D == 2 ? ((double)(d == 0 ? j : i) + 0.5) * g.dx[1 - d] : 0.0;
    const double r = ((double)id + 0.5) * g.dx[d];
    const double* L = low ? pb.line[d][0] : pb.line[d][1];
    if (s < (L[0] + L[1] * r) + L[2] * tb) return pb.A[c];
    const int far = low ? pb.far[d][0] : pb.far[d][1];
    if (far == BC_PRESCRIBED) return pb.B[c];
    if (d == 0) {
      if (low) lo0 = far; else hi0 = far;
    } else {
      if (low) lo1 = far; else hi1 = far;
    }
  }
  int f0 = 0, f1 = 0;
  const int ii = map_index(i, g.n[0], lo0, hi0, f0);
  const int jj = g.D >= 2 ? map_index(j, g.n[1], lo1, hi1, f1) : 0;
  double v = W[(long long)c * g.ncell + (long long)jj * g.n[0] + ii];
  if (c >= 1 && c <= g.D) {
    const int fo = c == 1 ? f0 : f1;
    if ((fo == 1) ^ (f0 == 2) ^ (f1 == 2)) v = -v;
  }
  return v;
}

// density and pressure of a frame-ordered Gauss-point state positive and
// finite, in one fixed operation order (the fallback's test)
template <int NC>
__device__ __forceinline__ bool physical_state(const double* w, double gamma) {
#pragma clang fp contract(off)
  double ke = 0.0;
#pragma unroll
  for (int q = 1; q < NC - 1; ++q) ke = ke + w[q] * w[q];
  const double pr = (gamma - 1.0) * (w[NC - 1] - 0.5 * ke / w[0]);
  return w[0] > 0.0 && pr > 0.0 && isfinite(w[0]) && isfinite(pr);
}

// first-order fallback: a non-physical side state becomes the side's cell
// average C with zero slopes; returns 1 if it did
template <int NC, int ND>
__device__ __forceinline__ int fallback_side(double* w, double (*dw)[NC], const double* C, double gamma) {
  if (physical_state<NC>(w, gamma)) return 0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    w[q] = C[q];
#pragma unroll
    for (int d = 0; d < ND; ++d) dw[d][q] = 0.0;
  }
  return 1;
}

// The selection of five values and the selected polynomial at the Gauss
// points; returns the flag (unused: not evaluated).
//   SEL_SMOOTH: the large stencil; sure becomes false where the data is not
//     smooth for certain (teno_smooth).  About 30 instructions against 135: a
//     wavefront whose lanes are all smooth, or hold equal values, takes its
//     selections in this form, and the others give up at the first that is
//     not.  Where both forms apply they agree to the bit, so a result does
//     not depend on the lanes beside it.  2-D four-quadrant problem 1024^2,
//     20 steps: 15.6 -> 12.3 ms; double Mach reflection, 8 steps: 1.76 ->
//     1.51 ms; a 97 x 61 grid with waves everywhere: 366 -> 367 us.  The same
//     test in the 2-D normal step gained nothing there and cost the small
//     grid 13 % (three short passes, one branch more in each).
//   SEL_FILTER: sure becomes false where the exact weights have to decide.
//     The caller then takes those selections in a loop of its own
//     (exact_flags: one copy of the exact code, four bits per selection) and
//     evaluates everything again with
//   SEL_GIVEN: the flag given.
constexpr int SEL_GIVEN = 3, SEL_SMOOTH = 4;

// EQ: five equal values count as smooth (their flag is then not the
// selection's).
template <int MODE, bool EQ = true>
__device__ __forceinline__ unsigned select_poly(const double* Q, const TenoCfg& c, TenoPoly<double>& o, bool& sure,
                                                unsigned given) {
  TenoParts<double> p;
  teno_parts(Q, p);
  if constexpr (MODE == SEL_SMOOTH) {
    sure &= teno_smooth<EQ>(p);
    teno_poly_large(p, o);
    return 1u;
  } else {
    TenoSel s;
    if constexpr (MODE == SEL_GIVEN)
      s = teno_sel(given);
    else
      sure &= teno_certain<MODE>(Q, p, c, s);
    teno_poly(p, s, o);
    return s.flag();
  }
}

// flags of n <= 8 selections from the exact weights, four bits each; load(i,
// Q) fills the i-th one's values
template <class F>
__device__ __forceinline__ unsigned exact_flags(int n, const TenoCfg& c, F load) {
  unsigned fl = 0;
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    double Q[5];
    load(i, Q);
    fl |= teno_exact(Q, c) << (4 * i);
  }
  return fl;
}

// the combination of F(dt), F(dt/2) that stage STAGE's update needs
__host__ __device__ constexpr int flux_out(int stage) { return stage == 1 ? FLUX_STAGE1 : FLUX_STAGE2; }

// A no-slip adiabatic wall is impermeable and, at rest, does no work and
// conducts no heat: the mass and energy fluxes of its faces are zero (frame
// components 0 and NC-1); f: face index along the normal axis ax.
template <int NC>
__device__ __forceinline__ void wall_fluxes(const Geom& g, int ax, int f, double* accA, double* accB) {
  if ((f == 0 && g.bclo[ax] == BC_NOSLIP) || (f == g.n[ax] && g.bchi[ax] == BC_NOSLIP)) {
    accA[0] = accA[NC - 1] = 0.0;
    accB[0] = accB[NC - 1] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// CFL time step (Sec. 5 preamble).
// ---------------------------------------------------------------------------
// value of another lane of the row by a DPP control, and of lane k
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                          __builtin_amdgcn_readlane(__double2loint(v), k));
}

// minimum over the wavefront (all lanes active, no NaN), in every lane: the
// rows of sixteen lanes by DPP moves, then the four rows (six steps through
// the LDS lane shuffle took 800 cycles of a small grid's kernel)
__device__ __forceinline__ double wave_min(double v) {
  v = fmin(v, dpp_move<0xB1>(v));   // quad: lane ^ 1
  v = fmin(v, dpp_move<0x4E>(v));   // quad: lane ^ 2
  v = fmin(v, dpp_move<0x141>(v));  // half row mirrored
  v = fmin(v, dpp_move<0x140>(v));  // row mirrored
  return fmin(fmin(lane_value(v, 0), lane_value(v, 16)), fmin(lane_value(v, 32), lane_value(v, 48)));
}

// minimum over the block (blockDim.x a multiple of 64, at most 1024);
// valid in thread 0
__device__ __forceinline__ double block_min(double v, double* red) {
  v = wave_min(v);
  if (blockDim.x == 64) return v;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) v = fmin(v, red[i]);
  }
  return v;
}

// local CFL limit of one cell (Sec. 5 preamble); NaN for a non-physical state
template <int D>
__device__ __forceinline__ double cell_dt(const double* w, double gamma, double mu, double dxm) {
  const double rho = w[0];
  double ke = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const double u = w[d + 1] / rho;
    ke += u * u;
  }
  const double p = (gamma - 1.0) * (w[D + 1] - 0.5 * rho * ke);
  if (!(rho > 0.0) || !(p > 0.0)) return NAN;
  double v = dxm / (sqrt(ke) + sqrt(gamma * p / rho));
  if (mu > 0.0) v = fmin(v, dxm * dxm * rho / (4.0 * mu));
  return v;
}

// the block's CFL minimum over its live cells' states w, to *partial
template <int D>
__device__ __forceinline__ void block_cfl(bool live, const double* w, double gamma, double mu, double dxm,
                                          double* partial) {
  __shared__ double red[16];  // one entry per wave, up to 1024 threads
  double v = live ? cell_dt<D>(w, gamma, mu, dxm) : INFINITY;
  // NaN (non-physical cell) wins the reduction
  const bool nan = live && !(v == v);
  v = block_min(nan ? -INFINITY : v, red);
  if (threadIdx.x == 0) *partial = v == -INFINITY ? NAN : v;
}

// the time step after the minimum v of the cells' limits (-inf: a
// non-physical cell), clipped to t_end - t
__device__ __forceinline__ double next_dt(double v, double cfl, double t, double t_end) {
#pragma clang fp contract(off)
  double dt = v == -INFINITY ? NAN : cfl * v;
  if (t_end > 0.0) {
    if (t >= t_end * (1.0 - 1e-14))
      dt = 0.0;
    else if (t + dt > t_end)
      dt = t_end - t;
  }
  return dt;
}

__device__ __forceinline__ void step_clock(const StepClock& k, bool write, double& t, double& dt) {
  double v = INFINITY;
  bool nan = false;
  if (k.cfl > 0.0) {
    double p[CLOCK_NBLK / 64];  // loaded together: one latency
#pragma unroll
    for (int r = 0; r < CLOCK_NBLK / 64; ++r) {
      const int i = (threadIdx.x & 63) + 64 * r;
      p[r] = i < k.nblk ? k.partial[i] : INFINITY;
    }
#pragma unroll
    for (int r = 0; r < CLOCK_NBLK / 64; ++r) {
      nan = nan || !(p[r] == p[r]);
      v = fmin(v, p[r]);
    }
  }
  t = k.prev[0];
  const double used = k.prev[1];
  if (used > 0.0) t += used;
  dt = k.cfl > 0.0 ? next_dt(wave_min(nan ? -INFINITY : v), k.cfl, t, k.t_end) : used;
  t = lane_value(t, 0);  // in scalar registers, as a clock that is loaded
  dt = lane_value(dt, 0);
  if (write && (threadIdx.x & 63) == 0) {
    k.next[0] = t;
    k.next[1] = dt;
    if (k.steps && used > 0.0) *k.steps += 1;
  }
}

// ---------------------------------------------------------------------------
// 1-D: one stage of a step in one kernel, faces and update together.  A
// wavefront owns LINE_CELLS = 58 consecutive cells: lane i loads cell c =
// first - 3 + i (ghost cells by the index map), takes its neighbours' values
// from the lanes beside it, reconstructs its cell and evaluates the flux of
// the face below it, with the left state from the lane below; lanes 3..60 then
// update their cells with the upper face's flux from the lane above.  What
// bounds a single small grid is latency: dependent loads and one lane's chain
// of arithmetic.  Hence one cell's loads and index map per lane, the three
// selections and both kinds of face values as one straight line of code, and
// every load issued before the first wait.  50 steps of 400 cells: 0.74 ms
// (0.82 with all six cells loaded by each lane, the selections in turn and a
// clock kernel between the steps; 1.42 with separate face and update kernels).
// ---------------------------------------------------------------------------
constexpr int LINE_CELLS = 58;

struct LineArgs {
  StageArgs s;
  const double* base;  // what the stage's flux differences are subtracted from: stage 1: s.W; stage 2: P
  double* out1;        // stage 1: W*; stage 2: W^{n+1}
  double* out2;        // stage 1: P
  double mu, idx;      // viscosity; 1 / dx
};

// value of the lane below (UP = false) or above (UP = true)
template <bool UP>
__device__ __forceinline__ double lane_shift(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), UP ? 0x130 : 0x138, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), UP ? 0x130 : 0x138, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// EX: prescribed sides or the first-order fallback may be on (a separate
// instantiation, so that grids without them run the plain code)
// SCHEME: the reconstruction (SCHEME_TENO_D, the paper's scheme, or one of
// its comparison schemes)
// first: the wavefront's first cell; partial (CFL): where the block's minimum
// over its cells goes.  A step of dt <= 0 or NaN leaves the state as it is:
// decided at the end, so that no load waits for dt.
template <int STAGE, bool NS, bool FLAGS, bool CFL, bool CHAR = false, bool EX = false, int SCHEME = SCHEME_TENO_D>
__device__ __forceinline__ void line_body(const LineArgs& l, int first, double* partial) {
  const StageArgs& a = l.s;
  const int n = a.g.n[0], i = threadIdx.x & 63;
  const int f = first - 3 + i;  // the lane's cell and the face below it
  const bool own = i >= 3 && i < 3 + LINE_CELLS && f < n;  // the lane updates its cell
  const bool face = i >= 3 && i <= 3 + LINE_CELLS && f <= n;
  const bool counts = own || (face && f == n && first < n);  // (a face between two wavefronts: the upper one)
  // the constants, loaded together before the first wait (one latency of the
  // scalar cache instead of one where each group is used)
  asm volatile("" ::"s"(l.idx), "s"(a.g.bclo[0]), "s"(a.g.bchi[0]), "s"(a.fc.N), "s"(a.fc.mu), "s"(a.fc.c1),
               "s"(a.fc.c2), "s"(a.fc.tau_mode), "s"(a.tn.fast), "s"(a.tn.eps4), "s"(a.tn.ct1_up), "s"(a.tn.ct1_dn),
               "s"(a.tn.ct2_up), "s"(a.tn.ct2_dn), "s"(a.W), "s"(a.dt), "s"(l.base), "s"(l.out1));
  double C[6][3], w[3];  // cells f-3 .. f+2 (the lane's own: C[3])
  const int fc = f < 0 ? 0 : (f >= n ? n - 1 : f);
  if (!EX)
#pragma unroll
    for (int c = 0; c < 3; ++c) C[3][c] = load_cell(a.g, a.W, c, f, 0, 0);
#pragma unroll
  for (int c = 0; c < 3; ++c) w[c] = l.base[(long long)c * n + fc];
  double dt, t = 0.0;
  if (STAGE == 1 && a.ck.prev) {
    step_clock(a.ck, first == 0, t, dt);
    t += a.t0;
  } else {
    dt = *a.dt;
    if (EX && a.pb.on) t = a.t0 + (a.tclk ? *a.tclk : 0.0);
  }
  if (EX) {
    const double tb = STAGE == 2 ? stage2_time(t, dt) : t;  // of the prescribed states
#pragma unroll
    for (int c = 0; c < 3; ++c) C[3][c] = cell_value(a.g, a.pb, a.W, c, f, 0, tb);
  }
  if (!(dt > 0.0)) {
    // at the end time: the state stays, without the fluxes
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (own) {
        l.out1[(long long)c * n + f] = w[c];
        if (STAGE == 1) l.out2[(long long)c * n + f] = w[c];
      }
    if (CFL) block_cfl<1>(own, w, a.gamma, l.mu, a.g.dx[0], partial);
    return;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    C[4][c] = lane_shift<true>(C[3][c]);
    C[5][c] = lane_shift<true>(C[4][c]);
    C[2][c] = lane_shift<false>(C[3][c]);
    C[1][c] = lane_shift<false>(C[2][c]);
    C[0][c] = lane_shift<false>(C[1][c]);
  }
  double A[3] = {0, 0, 0}, B[3] = {0, 0, 0};
  double Wl[3], Wr[3], dWl[1][3], dWr[1][3], dW0[1][3];
  const double idx = l.idx;  // normal slopes per unit length
  if (CHAR) {
    unsigned fr[3];
    char_recon_face<1>(a.gamma, C, a.tn, idx, Wl, dWl[0], Wr, dWr[0], fr);
    if (FLAGS && own)
#pragma unroll
      for (int k = 0; k < 3; ++k) a.nflags[(long long)k * n + f] = (uint8_t)fr[k];
  } else {
    double Q[3][5];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int r = 0; r < 5; ++r) Q[c][r] = C[1 + r][c];
    TenoSel sel[3];
    if (SCHEME == SCHEME_TENO_D) {
      bool sure = (a.tn.fast & TENO_FILTER_OK) != 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        TenoParts<double> p;
        teno_parts(Q[c], p);
        sure &= teno_certain<SEL_FILTER>(Q[c], p, a.tn, sel[c]);
      }
      if (!sure) {
#pragma unroll
        for (int c = 0; c < 3; ++c) sel[c] = teno_sel(teno_exact_cold(Q[c], a.tn));
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double o[4];
      unsigned fl;
      if (SCHEME == SCHEME_TENO_D) {
        teno_face_both(Q[c], sel[c], o);
        fl = sel[c].flag();
      } else {
        fl = scheme_face<SCHEME>(Q[c], a.sc, o);
        // separately reconstructed equilibrium slope (Eq. 3.12)
        if (SCHEME >= SCHEME_TENO5) dW0[0][c] = sealed(eq_slope(C[1][c], C[2][c], C[3][c], C[4][c]) * idx);
      }
      // (sealed: the flux of every variant of the kernel is compiled from the
      // same inputs, hence with the same contractions and to the same bits)
      Wr[c] = sealed(o[0]);
      dWr[0][c] = sealed(o[1] * idx);
      Wl[c] = sealed(lane_shift<false>(o[2]));
      dWl[0][c] = sealed(lane_shift<false>(o[3] * idx));
      if (FLAGS && own) a.nflags[(long long)c * n + f] = (uint8_t)fl;
    }
  }
  if (face) {
    if (EX && a.fallback) {
      const int nfb =
          fallback_side<3, 1>(Wl, dWl, C[2], a.gamma) + fallback_side<3, 1>(Wr, dWr, C[3], a.gamma);
      if (nfb && a.fbc && counts) atomicAdd(a.fbc, (unsigned long long)nfb);
    }
    const bool ok = SCHEME >= SCHEME_TENO5 ? gp_flux_eq<1, NS, flux_out(STAGE)>(
                                                 Wl, Wr, dWl, dWr, (const double*)nullptr, dW0, a.fc, dt, A, B)
                                           : gp_flux<1, NS, flux_out(STAGE)>(Wl, Wr, dWl, dWr, a.fc, dt, A, B);
    if (!ok && counts) atomicAdd(a.fail, 1ull);
    wall_fluxes<3>(a.g, 0, f, A, B);
  }
  double w1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double Ah = lane_shift<true>(A[c]), Bh = lane_shift<true>(B[c]);
    w1[c] = w[c] - (Ah - A[c]) * idx;
    if (own) {
      l.out1[(long long)c * n + f] = w1[c];
      if (STAGE == 1) l.out2[(long long)c * n + f] = w[c] - (Bh - B[c]) * idx;
    }
  }
  if (CFL) block_cfl<1>(own, w1, a.gamma, l.mu, a.g.dx[0], partial);
}

template <int STAGE, bool NS, bool FLAGS, bool CFL, bool CHAR = false, bool EX = false, int SCHEME = SCHEME_TENO_D>
__global__ __launch_bounds__(256) void line_kernel(LineArgs l, double* partial) {
  const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  line_body<STAGE, NS, FLAGS, CFL, CHAR, EX, SCHEME>(l, wave * LINE_CELLS, partial + blockIdx.x);
}

// ---------------------------------------------------------------------------
// 2-D: fused face kernel.  A block owns TN faces along the normal axis AX by
// TT rows along the tangential axis.  It stages the cells of the tile with a
// halo of 3 (normal) and 2 (tangential) in LDS, reconstructs every needed
// cell once along AX into LDS (values and normal slopes on both faces), and
// then each thread reconstructs its face's left and right states along the
// face at the two Gauss points and evaluates the two Gauss-point fluxes.
// ---------------------------------------------------------------------------
// Tile shapes (faces along the normal x faces along the tangential axis),
// two lanes per face; chosen per grid by the autotuner.
constexpr int NTILE2 = 3;
constexpr int CHAR_TILE2 = 2;  // the one tile shape of the characteristic path
__host__ __device__ constexpr int tile2_tn(int k) { return k == 0 ? 16 : (k == 1 ? 16 : 8); }
__host__ __device__ constexpr int tile2_tt(int k) { return k == 0 ? 8 : (k == 1 ? 16 : 16); }

// LDS doubles of one 2-D face tile: the staged cells and their normal
// reconstruction
__host__ __device__ constexpr int tile2_lds(int k) {
  return 4 * (tile2_tt(k) + 4) * (tile2_tn(k) + 5) + 4 * (tile2_tt(k) + 4) * (tile2_tn(k) + 1) * 4;
}

// ... plus, with characteristic variables, the per-face field values of both
// sides and the right eigenvectors of every staged face row
__host__ __device__ constexpr int tile2_lds_char(int k) {
  return tile2_lds(k) + 4 * (tile2_tt(k) + 4) * tile2_tn(k) * 4 + (tile2_tt(k) + 4) * tile2_tn(k) * 16;
}

// ... plus, with a separately reconstructed equilibrium (WENO-Z, TENO5),
// the equilibrium state and its normal slope of every staged face segment
__host__ __device__ constexpr int tile2_lds_eq(int k) {
  return tile2_lds(k) + 2 * 4 * (tile2_tt(k) + 4) * tile2_tn(k);
}

// (bx, by): tile index along the normal and the tangential axis; lds: the
// block's tile2_lds(TILE) (CHAR: tile2_lds_char(TILE); SCHEME_TENO5 and
// SCHEME_WENO_Z: tile2_lds_eq(TILE)) doubles of shared memory.  CHAR:
// reconstruction in characteristic variables (steps 2 and 3 below project
// onto the fields of each face and back).  SCHEME: the reconstruction
// (SCHEME_TENO_D or a comparison scheme; conservative variables).
template <int AX, int STAGE, bool NS, bool FLAGS, int TILE, bool CHAR = false, bool EX = false,
          int SCHEME = SCHEME_TENO_D>
__device__ __forceinline__ void face2d_tile(const StageArgs& a, int bx, int by, double* lds) {
  constexpr int TN = tile2_tn(TILE), TT = tile2_tt(TILE), NT = 2 * TN * TT;
  constexpr int NC = 4;
  constexpr int LN = TN + 5, LT = TT + 4, RN = TN + 1;
  double(*sW)[LT][LN] = reinterpret_cast<double(*)[LT][LN]>(lds);
  double(*sR)[LT][RN][4] = reinterpret_cast<double(*)[LT][RN][4]>(lds + NC * LT * LN);
  double dt, t_prev = 0.0;
  const bool clocked = STAGE == 1 && a.ck.prev != nullptr;
  if (clocked)  // (written by the launch's first block: a tile of the x faces)
    step_clock(a.ck, AX == 0 && blockIdx.x == 0 && threadIdx.x < 64, t_prev, dt);
  else
    dt = *a.dt;
  if (!(dt > 0.0)) return;
  const Geom& g = a.g;
  const int TA = 1 - AX;  // tangential axis
  const int nN = g.n[AX], nT = g.n[TA];
  const int f0 = bx * TN, t0 = by * TT;
  const int tid = threadIdx.x;
  const double tb = !EX ? 0.0 : clocked ? a.t0 + t_prev : boundary_time(a, STAGE, dt);

  // 1. cells of the tile, ghost cells by the index map or prescribed states;
  //    without prescribed sides one thread per cell maps it once and loads
  //    its four components
  if (EX) {
    for (int L = tid; L < NC * LN * LT; L += NT) {
      int nl, tl;
      if (AX == 0) {
        nl = L % LN;
        tl = (L / LN) % LT;
      } else {
        tl = L % LT;
        nl = (L / LT) % LN;
      }
      const int c = L / (LN * LT);
      const int pn = f0 - 3 + nl, pt = t0 - 2 + tl;
      sW[c][tl][nl] = cell_value(g, a.pb, a.W, c, AX == 0 ? pn : pt, AX == 0 ? pt : pn, tb);
    }
  } else {
    for (int L = tid; L < LN * LT; L += NT) {
      int nl, tl;
      if (AX == 0) {
        nl = L % LN;
        tl = L / LN;
      } else {
        tl = L % LT;
        nl = L / LT;
      }
      const int pn = f0 - 3 + nl, pt = t0 - 2 + tl;
      int m0, m1, m2;
      const long long off = cell_offset(g, AX == 0 ? pn : pt, AX == 0 ? pt : pn, 0, m0, m1, m2);
      double v[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) v[c] = a.W[(long long)c * g.ncell + off];
#pragma unroll
      for (int c = 0; c < NC; ++c) sW[c][tl][nl] = cell_flip(g, c, m0, m1, m2) ? -v[c] : v[c];
    }
  }
  __syncthreads();

  // 2. normal reconstruction of cells f0-1 .. f0+TN-1 on every staged row
  const double idn = 1.0 / g.dx[AX];  // normal slopes per unit length
  const int perm[NC] = {0, 1 + AX, 1 + TA, 3};
  if (CHAR) {
    // per face and row: the fields of the face's normal basis.  (a) one
    // thread per (side, row, face) projects the side's five cells, selects
    // and reconstructs every field; the left-side thread also keeps the
    // right eigenvectors.  (b) one thread per (component, row, face) projects
    // back.  Same slots of sR as the conservative path: face fn's left state
    // in cell slot fn (high face), its right state in slot fn + 1 (low face).
    double(*sV)[LT][TN][4] = reinterpret_cast<double(*)[LT][TN][4]>(lds + tile2_lds(TILE));
    double(*sM)[TN][16] = reinterpret_cast<double(*)[TN][16]>(lds + tile2_lds(TILE) + NC * LT * TN * 4);
    auto project = [&](int L, auto mode) {
      constexpr int MODE = decltype(mode)::value;
      const int fn = L % TN;
      const int tl = (L / TN) % LT;
      const int sd = L / (TN * LT);
      double C[6][NC];
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int q = 0; q < NC; ++q) C[r][q] = sW[perm[q]][tl][fn + r];
      double Wb[NC], Lm[NC][NC], Rm[NC][NC];
      {
#pragma clang fp contract(off)
#pragma unroll
        for (int q = 0; q < NC; ++q) Wb[q] = 0.5 * (C[2][q] + C[3][q]);
      }
      char_basis<2, 0>(a.gamma, Wb, Lm, Rm);
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        double V[5];
#pragma unroll
        for (int r = 0; r < 5; ++r) V[r] = char_dot<NC>(Lm[k], sd == 0 ? C[r] : C[r + 1]);
        const unsigned fl = teno_flag<MODE, true>(V, a.tn);
        double o[4];
        teno_face(V, fl, o);
        if (sd == 0) {
          sV[k][tl][fn][0] = o[2];
          sV[k][tl][fn][1] = o[3];
        } else {
          sV[k][tl][fn][2] = o[0];
          sV[k][tl][fn][3] = o[1];
          if (FLAGS) {
            const int cell = f0 + fn, row = t0 - 2 + tl;
            if (cell < nN && tl >= 2 && tl < TT + 2 && row < nT) {
              const long long lin = AX == 0 ? (long long)row * g.n[0] + cell : (long long)cell * g.n[0] + row;
              a.nflags[((long long)AX * NC + k) * g.ncell + lin] = (uint8_t)fl;
            }
          }
        }
      }
      if (sd == 0)
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
          for (int k = 0; k < NC; ++k) sM[tl][fn][q * NC + k] = Rm[q][k];
    };
    // (the exact weights alone where the certain decisions are off: a form of
    // its own, so that they share the values' sums and nothing is formed twice)
    if (a.tn.fast & TENO_FILTER_OK)
      for (int L = tid; L < 2 * LT * TN; L += NT) project(L, std::integral_constant<int, SEL_FILTER>());
    else
      for (int L = tid; L < 2 * LT * TN; L += NT) project(L, std::integral_constant<int, SEL_EXACT>());
    __syncthreads();
    for (int L = tid; L < NC * LT * TN; L += NT) {
      const int fn = L % TN;
      const int tl = (L / TN) % LT;
      const int q = L / (TN * LT);
      const double* rq = &sM[tl][fn][q * NC];
      double x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double v[NC] = {sV[0][tl][fn][j], sV[1][tl][fn][j], sV[2][tl][fn][j], sV[3][tl][fn][j]};
        x[j] = char_dot<NC>(rq, v);
      }
      const int c = q == 0 ? perm[0] : (q == 1 ? perm[1] : (q == 2 ? perm[2] : perm[3]));
      sR[c][tl][fn][2] = x[0];
      sR[c][tl][fn][3] = x[1] * idn;
      sR[c][tl][fn + 1][0] = x[2];
      sR[c][tl][fn + 1][1] = x[3] * idn;
    }
  } else {
    for (int L = tid; L < NC * LT * RN; L += NT) {
      const int nr = L % RN;
      const int tl = (L / RN) % LT;
      const int c = L / (RN * LT);
      const double* Q = &sW[c][tl][nr];
      double o[4];
      unsigned fl;
      if (SCHEME == SCHEME_TENO_D) {
        fl = teno_flag<SEL_FILTER, true>(Q, a.tn);
        teno_face(Q, fl, o);
      } else {
        fl = scheme_face<SCHEME>(Q, a.sc, o);
      }
      sR[c][tl][nr][0] = o[0];
      sR[c][tl][nr][1] = o[1] * idn;
      sR[c][tl][nr][2] = o[2];
      sR[c][tl][nr][3] = o[3] * idn;
      if (FLAGS) {
        const int cell = f0 - 1 + nr, row = t0 - 2 + tl;
        if (nr >= 1 && cell < nN && tl >= 2 && tl < TT + 2 && row < nT) {
          const long long lin = AX == 0 ? (long long)row * g.n[0] + cell : (long long)cell * g.n[0] + row;
          a.nflags[((long long)AX * NC + c) * g.ncell + lin] = (uint8_t)fl;
        }
      }
    }
  }
  __syncthreads();

  // 2b. WENO-Z / TENO5: the equilibrium state of every staged face segment,
  //     the kinetic weighting of its two line-averaged interface states
  //     (Eq. 2.6), and its normal slope from the cells (Eq. 3.12), frame
  //     order; reconstructed along the face at the Gauss points in step 3
  double(*sE)[2][LT][TN] = reinterpret_cast<double(*)[2][LT][TN]>(lds + tile2_lds(TILE));
  if (SCHEME >= SCHEME_TENO5) {
    for (int L = tid; L < LT * TN; L += NT) {
      const int fn = L % TN, tl = L / TN;
      double wl[NC], wr[NC], sl[NC], sr[NC], h0, h1, k0, k1;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        wl[q] = sR[perm[q]][tl][fn][2];
        wr[q] = sR[perm[q]][tl][fn + 1][0];
      }
      Gas<2, double> gl, gr;
      side_w0<2>(wl, a.fc, 1.0, gl, h0, h1, sl);
      side_w0<2>(wr, a.fc, -1.0, gr, k0, k1, sr);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = perm[q];
        sE[q][0][tl][fn] = sl[q] + sr[q];
        sE[q][1][tl][fn] = eq_slope(sW[c][tl][fn + 1], sW[c][tl][fn + 2], sW[c][tl][fn + 3], sW[c][tl][fn + 4]) * idn;
      }
    }
    __syncthreads();
  }

  // 3. lanes 2k and 2k+1 share face k.  Lane m reconstructs side m (left: 0,
  //    right: 1) along the face at both Gauss points, keeps Gauss point m and
  //    hands Gauss point 1-m to its partner; each lane then evaluates the
  //    flux at its Gauss point m and the pair sums the two.  The flux takes
  //    the lane's own side first, with its sign (+1 left, -1 right): the two
  //    sides' shares are added in either order with the same result, so no
  //    lane has to sort them (CHAR: left side first, see gp_flux_face).
  const int m = tid & 1;
  const int fi = tid >> 1;
  const int fn = fi % TN, ft = fi / TN;
  const int f = f0 + fn, t = t0 + ft;
  const bool live = f <= nN && t < nT;
  const long long nf = face_count(g, AX);
  const long long fidx = AX == 0 ? (long long)t * (g.n[0] + 1) + f : (long long)f * g.n[0] + t;
  const double idt = 1.0 / g.dx[TA];
  double Wo[NC], Do[2][NC], Wp[NC], Dp[2][NC];  // own and partner's side (CHAR: left and right); slopes [axis n/t][q]
  const double sg = m ? 1.0 : -1.0;             // sign of the lane's Gauss point; -sg: of its side
  const int nr = m == 0 ? fn : fn + 1;
  const int vo = m == 0 ? 2 : 0;
  // value, derivative along the face and normal slope of the lane's side at
  // its own Gauss point (index 0) and at its partner's (1); false where a
  // selection needs the exact weights
  double gV[NC][2], gD[NC][2], gN[NC][2];
  unsigned given = 0;  // flags of W (bits 8 q) and W_n (8 q + 4) of frame component or field q
  auto tangential = [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
    bool sure = true;
    if (CHAR) {
      // fields of the basis along the face at this face's reference state
      // (cells f-1 and f of row t); each field of W and of W_n is selected,
      // evaluated and projected back.  MODE: SEL_FILTER, or SEL_EXACT where
      // the certain decisions are off
#pragma unroll
      for (int q = 0; q < NC; ++q) gV[q][0] = gV[q][1] = gD[q][0] = gD[q][1] = gN[q][0] = gN[q][1] = 0.0;
      double Wb[NC], Lt[NC][NC], Rt[NC][NC];
      {
#pragma clang fp contract(off)
#pragma unroll
        for (int q = 0; q < NC; ++q) Wb[q] = 0.5 * (sW[perm[q]][ft + 2][fn + 2] + sW[perm[q]][ft + 2][fn + 3]);
      }
      char_basis<2, 1>(a.gamma, Wb, Lt, Rt);
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        double Qw[5], Qn[5];
#pragma unroll
        for (int r = 0; r < 5; ++r) {
          double xw[NC], xn[NC];
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            xw[q] = sR[perm[q]][ft + r][nr][vo];
            xn[q] = sR[perm[q]][ft + r][nr][vo + 1];
          }
          Qw[r] = char_dot<NC>(Lt[k], xw);
          Qn[r] = char_dot<NC>(Lt[k], xn);
        }
        const unsigned fw = teno_flag<MODE, true>(Qw, a.tt), fq = teno_flag<MODE, true>(Qn, a.tt);
        if (FLAGS) {
          a.tflags[((long long)(0 * 2 + m) * NC + k) * nf + fidx] = (uint8_t)fw;
          a.tflags[((long long)(1 * 2 + m) * NC + k) * nf + fidx] = (uint8_t)fq;
        }
        double pv[2], pd[2], qv[2], qd[2], v[2], dv[2], vn[2];
        teno_gauss_powers(Qw, fw, pv, pd);
        teno_gauss_powers(Qn, fq, qv, qd);
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          v[gp] = m ^ gp ? pv[1] : pv[0];
          dv[gp] = m ^ gp ? pd[1] : pd[0];
          vn[gp] = m ^ gp ? qv[1] : qv[0];
        }
        {
          // back-projection: dense sums in field order, no contraction
#pragma clang fp contract(off)
#pragma unroll
          for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int gp = 0; gp < 2; ++gp) {
              gV[q][gp] = gV[q][gp] + Rt[q][k] * v[gp];
              gD[q][gp] = gD[q][gp] + Rt[q][k] * dv[gp];
              gN[q][gp] = gN[q][gp] + Rt[q][k] * vn[gp];
            }
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int c = perm[q];
        double Qw[5], Qn[5];
#pragma unroll
        for (int r = 0; r < 5; ++r) {
          Qw[r] = sR[c][ft + r][nr][vo];
          Qn[r] = sR[c][ft + r][nr][vo + 1];
        }
        unsigned fw, fq;
        if (SCHEME == SCHEME_TENO_D) {
          TenoPoly<double> w, n;
          fw = select_poly<MODE>(Qw, a.tt, w, sure, (given >> (8 * q)) & 15u);
          fq = select_poly<MODE>(Qn, a.tt, n, sure, (given >> (8 * q + 4)) & 15u);
          if (MODE == SEL_SMOOTH && !all_lanes(sure)) return false;
#pragma unroll
          for (int gp = 0; gp < 2; ++gp) {
            const double x = gp == 0 ? sg : -sg;
            gV[q][gp] = fma(x, w.odd, w.base);
            gD[q][gp] = fma(x, w.od, w.ev);
            gN[q][gp] = fma(x, n.odd, n.base);
            if (MODE == SEL_SMOOTH) {  // evaluated here, not after the last early exit
              gV[q][gp] = opaque(gV[q][gp]);
              gD[q][gp] = opaque(gD[q][gp]);
              gN[q][gp] = opaque(gN[q][gp]);
            }
          }
        } else {
          double v[2], dv[2], vn[2], dvn[2];
          fw = scheme_gauss<SCHEME>(Qw, a.sc, v, dv);
          fq = scheme_gauss<SCHEME>(Qn, a.sc, vn, dvn);
#pragma unroll
          for (int gp = 0; gp < 2; ++gp) {
            gV[q][gp] = m ^ gp ? v[1] : v[0];
            gD[q][gp] = m ^ gp ? dv[1] : dv[0];
            gN[q][gp] = m ^ gp ? vn[1] : vn[0];
          }
        }
        if (FLAGS) {
          a.tflags[((long long)(0 * 2 + m) * NC + c) * nf + fidx] = (uint8_t)fw;
          a.tflags[((long long)(1 * 2 + m) * NC + c) * nf + fidx] = (uint8_t)fq;
        }
      }
    }
    return sure;
  };
  if (live) {
    if (CHAR) {
      if (a.tt.fast & TENO_FILTER_OK)
        tangential(std::integral_constant<int, SEL_FILTER>());
      else
        tangential(std::integral_constant<int, SEL_EXACT>());
    } else if (SCHEME != SCHEME_TENO_D) {
      tangential(std::integral_constant<int, SEL_GIVEN>());
    } else {
      bool sure = false;
      if (!FLAGS && (a.tt.fast & TENO_RATIO_OK)) sure = tangential(std::integral_constant<int, SEL_SMOOTH>());
      if (!sure && (a.tt.fast & TENO_FILTER_OK)) sure = tangential(std::integral_constant<int, SEL_FILTER>());
      if (!sure) {
        given = exact_flags(2 * NC, a.tt, [&](int i, double* Q) {
          const int q = i >> 1, c = q == 1 ? perm[1] : q == 2 ? perm[2] : q;  // mass and energy in place
#pragma unroll
          for (int r = 0; r < 5; ++r) Q[r] = sR[c][ft + r][nr][vo + (i & 1)];
        });
        tangential(std::integral_constant<int, SEL_GIVEN>());
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < NC; ++q) gV[q][0] = gV[q][1] = gD[q][0] = gD[q][1] = gN[q][0] = gN[q][1] = 0.0;
  }
  const bool sw = CHAR && m;  // the face frame's flux takes the left side first
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const double pv = lane_xor<1>(gV[q][1]), pd = lane_xor<1>(gD[q][1]), pn = lane_xor<1>(gN[q][1]);
    Wo[q] = sw ? pv : gV[q][0];
    Do[0][q] = sw ? pn : gN[q][0];
    Do[1][q] = (sw ? pd : gD[q][0]) * idt;
    Wp[q] = sw ? gV[q][0] : pv;
    Dp[0][q] = sw ? gN[q][0] : pn;
    Dp[1][q] = (sw ? gD[q][0] : pd) * idt;
  }
  double A[NC] = {0, 0, 0, 0}, B[NC] = {0, 0, 0, 0};
  if (EX && live && a.fallback) {
    double Co[NC], Cp[NC];  // the cells of the lane's own and of its partner's side
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      Co[q] = sW[perm[q]][ft + 2][fn + 2 + (CHAR ? 0 : m)];
      Cp[q] = sW[perm[q]][ft + 2][fn + 3 - (CHAR ? 0 : m)];
    }
    const int nfb = fallback_side<NC, 2>(Wo, Do, Co, a.gamma) + fallback_side<NC, 2>(Wp, Dp, Cp, a.gamma);
    if (nfb && a.fbc) atomicAdd(a.fbc, (unsigned long long)nfb);
  }
  if (live) {
    bool ok;
    if (SCHEME >= SCHEME_TENO5) {
      // the equilibrium at this lane's Gauss point: the five face segments'
      // states reconstructed with the cut-off of Sec. 4.1 (TENO5, q = 6;
      // the linear quartic where they are smooth, Sec. 3.1 Step 4), value
      // and derivatives
      SchemeCfg se = a.sc;
      se.q = 6;
      // (the pair shares the work: lane m reconstructs the components 2 m and
      // 2 m + 1 at both Gauss points and they swap)
      double W0e[NC], dW0e[2][NC];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int q = 2 * m + j;
        double Qe[5], Qx[5], v[2], d[2], vx[2], dx[2];
#pragma unroll
        for (int r = 0; r < 5; ++r) {
          Qe[r] = sE[q][0][ft + r][fn];
          Qx[r] = sE[q][1][ft + r][fn];
        }
        scheme_gauss<SCHEME_TENO5>(Qe, se, v, d);
        scheme_gauss<SCHEME_TENO5>(Qx, se, vx, dx);
        const double own[3] = {m ? v[1] : v[0], m ? d[1] : d[0], m ? vx[1] : vx[0]};
        const double got[3] = {lane_xor<1>(m ? v[0] : v[1]), lane_xor<1>(m ? d[0] : d[1]),
                               lane_xor<1>(m ? vx[0] : vx[1])};
        W0e[j] = m ? got[0] : own[0];
        W0e[2 + j] = m ? own[0] : got[0];
        dW0e[1][j] = (m ? got[1] : own[1]) * idt;
        dW0e[1][2 + j] = (m ? own[1] : got[1]) * idt;
        dW0e[0][j] = m ? got[2] : own[2];
        dW0e[0][2 + j] = m ? own[2] : got[2];
      }
      ok = gp_flux_eq<2, NS, flux_out(STAGE)>(Wo, Wp, Do, Dp, W0e, dW0e, a.fc, dt, A, B, 0.5, -sg);
    } else if constexpr (CHAR) {
      double Fdt[NC], Fh[NC];
      ok = gp_flux_face<2, NS>(Wo, Wp, Do, Dp, a.fc, dt, Fdt, Fh);
      combine_times<STAGE, NC>(Fdt, Fh, 0.5, A, B);
    } else {
      ok = gp_flux<2, NS, flux_out(STAGE)>(Wo, Wp, Do, Dp, a.fc, dt, A, B, 0.5, -sg);
    }
    if (!ok) atomicAdd(a.fail, 1ull);
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    A[q] += lane_xor<1>(A[q]);
    if (STAGE == 1) B[q] += lane_xor<1>(B[q]);
  }
  wall_fluxes<NC>(g, AX, f, A, B);
  if (live && m == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      a.FA[(long long)perm[q] * nf + fidx] = A[q];
      if (STAGE == 1) a.FB[(long long)perm[q] * nf + fidx] = B[q];
    }
  }
}

// Both directions in one launch: the first blocks take the x-face tiles,
// the rest the y-face tiles (one shared LDS tile), so that neither
// direction waits for the other's tail.
template <int STAGE, bool NS, bool FLAGS, int TILE, bool CHAR = false, bool EX = false, int SCHEME = SCHEME_TENO_D>
__global__ __launch_bounds__(2 * tile2_tn(TILE) * tile2_tt(TILE), 2) void face2d_xy_kernel(StageArgs ax,
                                                                                           StageArgs ay) {
  constexpr int TN = tile2_tn(TILE);
  __shared__ double lds[CHAR ? tile2_lds_char(TILE) : (SCHEME >= SCHEME_TENO5 ? tile2_lds_eq(TILE) : tile2_lds(TILE))];
  const int nbx = (ax.g.n[0] + 1 + TN - 1) / TN;          // x faces: tiles along x
  const int nx = nbx * ((ax.g.n[1] + tile2_tt(TILE) - 1) / tile2_tt(TILE));
  // XCD-aware order: workgroups are dealt to the 8 XCDs in turn; the tiles
  // are renumbered so that each XCD walks a contiguous range of them (a
  // bijection for any grid size), where neighbouring tiles, which stage
  // common halo cells and write common cache lines of the face fluxes,
  // meet in one L2 (HBM reads per launch fall 2.7-3.0x, writes to the
  // algorithmic bytes).
  const int nbt = gridDim.x, x8 = blockIdx.x & 7, per = nbt >> 3, rem = nbt & 7;
  const int b = x8 * per + min(x8, rem) + (int)(blockIdx.x >> 3);
  if (b < nx) {
    face2d_tile<0, STAGE, NS, FLAGS, TILE, CHAR, EX, SCHEME>(ax, b % nbx, b / nbx, lds);
  } else {
    const int nby = (ay.g.n[1] + 1 + TN - 1) / TN;        // y faces: tiles along y
    face2d_tile<1, STAGE, NS, FLAGS, TILE, CHAR, EX, SCHEME>(ay, (b - nx) % nby, (b - nx) / nby, lds);
  }
}

// ---------------------------------------------------------------------------
// 3-D.  (a) normal reconstruction along AX of every cell with AX index in
// [-1, n] (interior in the other axes): R[c][4][k][j][i'] with the AX index
// shifted by one, values and slopes on both faces.
// ---------------------------------------------------------------------------
template <int AX, bool FLAGS>
__global__ __launch_bounds__(256) void recon3d_kernel(StageArgs a) {
  const Geom& g = a.g;
  int ext[3] = {g.n[0], g.n[1], g.n[2]};
  ext[AX] += 2;
  const long long nr = (long long)ext[0] * ext[1] * ext[2];
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= nr * 5) return;
  const int c = (int)(id / nr);
  long long r = id % nr;
  int p[3];
  p[0] = (int)(r % ext[0]);
  r /= ext[0];
  p[1] = (int)(r % ext[1]);
  p[2] = (int)(r / ext[1]);
  p[AX] -= 1;
  // the stencil runs along AX only (the other indices are interior): one
  // base offset, and the index map along AX for each of its five cells
  const long long sax = AX == 0 ? 1 : (AX == 1 ? (long long)g.n[0] : (long long)g.n[0] * g.n[1]);
  int pz[3] = {p[0], p[1], p[2]};
  pz[AX] = 0;
  const double* Wc = a.W + (long long)c * g.ncell + ((long long)pz[2] * g.n[1] + pz[1]) * g.n[0] + pz[0];
  double Q[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    int f[3] = {0, 0, 0};
    const int m = map_index(p[AX] + s - 2, g.n[AX], g.bclo[AX], g.bchi[AX], f[AX]);
    const double v = Wc[m * sax];
    Q[s] = cell_flip(g, c, f[0], f[1], f[2]) ? -v : v;
  }
  double o[4];
  const unsigned fl = teno_flag<SEL_RATIO>(Q, a.tn);
  teno_face(Q, fl, o);
  const double idn = 1.0 / g.dx[AX];
  const long long base = (long long)c * 4 * nr + (id % nr);
  a.Rout[base] = o[0];
  a.Rout[base + nr] = o[1] * idn;
  a.Rout[base + 2 * nr] = o[2];
  a.Rout[base + 3 * nr] = o[3] * idn;
  if (FLAGS && p[AX] >= 0 && p[AX] < g.n[AX])
    a.nflags[((long long)AX * 5 + c) * g.ncell + ((long long)p[2] * g.n[1] + p[1]) * g.n[0] + p[0]] = (uint8_t)fl;
}

// (b) face kernel.  A block owns one plane of faces (fixed index along AX)
// and a B1 x B2 tile of it along the tangential axes T1, T2 (cyclic order:
// x-faces y, z; y-faces z, x; z-faces x, y).  It stages the normal
// reconstruction of both sides (from recon3d_kernel) with a halo of two in
// LDS (ghost positions by the index map, mirrored momenta negated),
// reconstructs every face line of the tile and its T2 halo once along T1
// (sweep 1, both T1 Gauss points), and then eight lanes share a face: lane
// (m1, m3, m2) owns side m2 at Gauss point (m1, m3).
//   * Sweep 2: the pair (m3 = 0, 1) of a side and T1 point splits the
//     fifteen T2 reconstructions of that side (five components of the value,
//     its T1 derivative and its normal slope) and swaps the results at each
//     other's T2 point.
//   * Flux: each lane evaluates its side's share of the equilibrium state
//     and of the non-equilibrium moments (side_w0, side_part); the pair
//     (m2 = 0, 1) adds the shares (a + b is exact-order independent), and
//     both lanes evaluate the equilibrium part (flux_combine).
// Three wavefronts per SIMD (168 registers, 4 to 30 of them spilled for a
// short while) instead of two keep the vector units busier: 128^3
// Taylor-Green vortex, 2 steps: 19.3 -> 18.6 ms.
// Tiles are dealt to the 8 XCDs in contiguous ranges.
// FLAGS: record the tangential selections (stage 1), per face of this
// direction: sweep 1 of the face's own line as [(q*2 + side)*5 + c] (q = 0:
// W, 1: W_n), then sweep 2 as [20 + ((m1*3 + kind)*2 + side)*5 + c] (kind 0:
// W, 1: dW/dt1, 2: W_n at T1 Gauss point m1), c the global component, each a
// plane of faces indexed like a state whose axis AX has n + 1 entries.
//
// Tile shapes (faces along T1 x T2, 32 faces in 256 threads): 0 = 2 x 16, 1 =
// 4 x 8.  Shape 0 has the smaller halo in sweep 1 (400 items against 480) and
// is 0.7 % faster where both fill their tiles (128^3: 18.8 and 18.95 ms for two
// steps); shape 1 fills planes better whose T2 extent is small or just above a
// multiple of 16.  The shape with fewer blocks is taken, shape 1 if it saves
// more than one block in 32: 29 x 35 x 22, Euler, four steps, 1096 us with shape 0
// alone, 1009 with shape 1 alone, 997 by the rule.
constexpr int L3 = 8;
__host__ __device__ constexpr int tile3_1(int k) { return k == 0 ? 2 : 4; }
__host__ __device__ constexpr int tile3_2(int k) { return k == 0 ? 16 : 8; }

template <int AX, int STAGE, bool NS, bool EX = false, bool FLAGS = false, int TILE = 0>
__global__ __launch_bounds__(L3 * tile3_1(TILE) * tile3_2(TILE), 3) void face3d_kernel(StageArgs a) {
  constexpr int NC = 5, B1 = tile3_1(TILE), B2 = tile3_2(TILE), NT = L3 * B1 * B2;
  constexpr int L1 = B1 + 4, L2 = B2 + 4;
  constexpr int T1 = (AX + 1) % 3, T2 = (AX + 2) % 3;
  __shared__ double sR[2][NC][2][L2][L1];      // [side][c][value, normal slope][t2][t1]
  __shared__ double sS[2][NC][L2][B1][6];      // sweep 1: v(m1), d_t1 v(m1), v_n(m1)
  const double dt = *a.dt;
  if (!(dt > 0.0)) return;
  const Geom& g = a.g;
  // XCD-aware order: workgroups are dealt to the 8 XCDs in turn; the
  // logical tiles are renumbered so that each XCD walks a contiguous range
  // in which tiles that share cache lines of the normal reconstruction
  // (x fastest in memory) follow each other and meet in one L2: for the
  // x faces the face plane is fastest (neighbouring planes share the lines
  // along x), for the y and z faces the T1 tile (the z-rows of the y faces'
  // tiles overlap by four of six, the z faces' tiles cover the x-lines two
  // cells at a time), then the plane, then the T2 tile.
  const int nb1 = (g.n[T1] + B1 - 1) / B1, nb2 = (g.n[T2] + B2 - 1) / B2;
  const int np = g.n[AX] + 1;
  const int nbl = np * nb1 * nb2;
  const int per = (nbl + 7) / 8;
  const int lb = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (lb >= nbl) return;
  const int fa = AX == 0 ? lb % np : (lb / nb1) % np;
  const int t10 = (AX == 0 ? (lb / np) % nb1 : lb % nb1) * B1, t20 = (lb / (np * nb1)) * B2;
  const int tid = threadIdx.x;
  int ext[3] = {g.n[0], g.n[1], g.n[2]};
  ext[AX] += 2;
  const long long nr = (long long)ext[0] * ext[1] * ext[2];

  // 1. normal reconstruction of the two cells beside each face position:
  //    thread (position, k) maps its tangential position once and loads
  //    both sides' five components of the value (k = 0) or the normal slope
  //    (k = 1); x, the fastest axis in memory, runs fastest over threads
  static_assert(2 * L1 * L2 <= NT, "one thread per position and kind");
  if (tid < 2 * L1 * L2) {
    const int p = tid % (L1 * L2), k = tid / (L1 * L2);
    const int i1 = AX == 1 ? p / L2 : p % L1;
    const int i2 = AX == 1 ? p % L2 : p / L1;
    int f1 = 0, f2 = 0;
    int e[3];
    e[AX] = fa;  // cell fa - 1 along AX, shifted by one; the right side is the next
    e[T1] = map_index(t10 - 2 + i1, g.n[T1], g.bclo[T1], g.bchi[T1], f1);
    e[T2] = map_index(t20 - 2 + i2, g.n[T2], g.bclo[T2], g.bchi[T2], f2);
    const long long off = ((long long)e[2] * ext[1] + e[1]) * ext[0] + e[0];
    const long long sax = AX == 0 ? 1 : (AX == 1 ? (long long)ext[0] : (long long)ext[0] * ext[1]);
    double v[2][NC];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c) v[s][c] = a.R[(long long)(c * 4 + (s == 0 ? 2 : 0) + k) * nr + off + s * sax];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bool mom = c >= 1 && c <= 3;
      const bool neg = (c == 1 + T1 && f1 == 1) ^ (c == 1 + T2 && f2 == 1) ^ (mom && f1 == 2) ^ (mom && f2 == 2);
#pragma unroll
      for (int s = 0; s < 2; ++s) sR[s][c][k][i2][i1] = neg ? -v[s][c] : v[s][c];
    }
  }
  __syncthreads();

  // 2. sweep 1 along T1 of every face line of the tile and its T2 halo
  const double i1d = 1.0 / g.dx[T1], i2d = 1.0 / g.dx[T2];
  int nfa[3] = {g.n[0], g.n[1], g.n[2]};
  nfa[AX] += 1;
  const long long nf = (long long)nfa[0] * nfa[1] * nfa[2];
  for (int L = tid; L < 2 * NC * L2 * B1; L += NT) {
    const int j1 = L % B1;
    const int i2 = (L / B1) % L2;
    const int c = (L / (B1 * L2)) % NC;
    const int s = L / (NC * B1 * L2);
    double Qw[5], Qn[5];
#pragma unroll
    for (int r = 0; r < 5; ++r) {
      Qw[r] = sR[s][c][0][i2][j1 + r];
      Qn[r] = sR[s][c][1][i2][j1 + r];
    }
    double v[2], dv[2], vn[2], dvn[2];
    unsigned fw = 1u, fq = 1u;
    bool smooth = false;
    if (a.tt.fast & TENO_RATIO_OK) {
      TenoParts<double> pw, pn;
      teno_parts(Qw, pw);
      teno_parts(Qn, pn);
      smooth = all_lanes(teno_smooth<false>(pw) & teno_smooth<false>(pn));
    }
    if (!smooth) {
      fw = teno_flag<SEL_RATIO, true>(Qw, a.tt);
      fq = teno_flag<SEL_RATIO, true>(Qn, a.tt);
    }
    // the inputs of the second sweep's selections: one fixed evaluation order
    teno_gauss_exact(Qw, fw, v, dv);
    teno_gauss_exact(Qn, fq, vn, dvn);
    if (FLAGS && i2 >= 2 && i2 < B2 + 2) {
      int q3[3];
      q3[AX] = fa;
      q3[T1] = t10 + j1;
      q3[T2] = t20 + i2 - 2;
      if (q3[T1] < g.n[T1] && q3[T2] < g.n[T2]) {
        const long long fid = ((long long)q3[2] * nfa[1] + q3[1]) * nfa[0] + q3[0];
        a.tflags[((long long)(0 * 2 + s) * NC + c) * nf + fid] = (uint8_t)fw;
        a.tflags[((long long)(1 * 2 + s) * NC + c) * nf + fid] = (uint8_t)fq;
      }
    }
    double* o = sS[s][c][i2][j1];
    o[0] = v[0];
    o[1] = v[1];
    o[2] = dv[0] * i1d;
    o[3] = dv[1] * i1d;
    o[4] = vn[0];
    o[5] = vn[1];
  }
  __syncthreads();

  // 3. sweep 2 along T2, split over the pair m3 = 0, 1.  Item it = 3 q + kind
  //    (kind 0: value, 1: T1 derivative, 2: normal slope of component perm[q]);
  //    in round r lane m3 reconstructs item 2 r + m3 at both T2 points and
  //    hands its partner the value (and T2 derivative) at the partner's point.
  const int m2 = tid & 1, m3 = (tid >> 1) & 1, m1 = (tid >> 2) & 1, fi = tid >> 3;
  const int j1 = fi % B1, j2 = fi / B1;
  int fp[3];
  fp[AX] = fa;
  fp[T1] = t10 + j1;
  fp[T2] = t20 + j2;
  const bool live = fp[T1] < g.n[T1] && fp[T2] < g.n[T2];
  const long long fid = ((long long)fp[2] * nfa[1] + fp[1]) * nfa[0] + fp[0];
  const int perm[NC] = {0, 1 + AX, 1 + T1, 1 + T2, 4};
  const double sg = m3 ? 1.0 : -1.0;  // sign of the lane's T2 point
  // (cell units) at this lane's T2 point [r][0] and at its partner's [r][1];
  // false where a selection needs the exact weights
  double sv[8][2], sd[8][2];
  unsigned given = 0;  // flags of the lane's items, four bits each
  auto item_values = [&](int it, int& kind, int& c, double* Q) {
    const int q = it / 3;
    kind = it - 3 * q;
    c = q == 0 ? perm[0] : q == 1 ? perm[1] : q == 2 ? perm[2] : q == 3 ? perm[3] : perm[4];
#pragma unroll
    for (int k = 0; k < 5; ++k) Q[k] = sS[m2][c][j2 + k][j1][2 * kind + m1];
  };
  auto sweep2 = [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
    bool sure = true;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int it = 2 * r + m3;
      if (it < 15) {
        int kind, c;
        double Q[5];
        item_values(it, kind, c, Q);
        TenoPoly<double> w;
        const unsigned fl = select_poly<MODE>(Q, a.tt, w, sure, (given >> (4 * r)) & 15u);
        if (MODE == SEL_SMOOTH && !all_lanes(sure)) return false;
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          const double x = gp == 0 ? sg : -sg;
          sv[r][gp] = fma(x, w.odd, w.base);
          sd[r][gp] = fma(x, w.od, w.ev);
          if (MODE == SEL_SMOOTH) {
            sv[r][gp] = opaque(sv[r][gp]);
            if (r != 2 && r != 5) sd[r][gp] = opaque(sd[r][gp]);  // (their derivatives are not used)
          }
        }
        if (FLAGS) a.tflags[((long long)4 * NC + ((m1 * 3 + kind) * 2 + m2) * NC + c) * nf + fid] = (uint8_t)fl;
      } else {
        sv[r][0] = sv[r][1] = sd[r][0] = sd[r][1] = 0.0;
      }
    }
    return sure;
  };
  if (live) {
    bool sure = false;
    if (!FLAGS && (a.tt.fast & TENO_RATIO_OK)) sure = sweep2(std::integral_constant<int, SEL_SMOOTH>());
    if (!sure && (a.tt.fast & TENO_FILTER_OK)) sure = sweep2(std::integral_constant<int, SEL_FILTER>());
    if (!sure) {
      given = exact_flags(8 - m3, a.tt, [&](int r, double* Q) {
        int kind, c;
        item_values(2 * r + m3, kind, c, Q);
      });
      sweep2(std::integral_constant<int, SEL_GIVEN>());
    }
  } else {
#pragma unroll
    for (int r = 0; r < 8; ++r) sv[r][0] = sv[r][1] = sd[r][0] = sd[r][1] = 0.0;
  }
  double item[15], item_d[15];  // at this lane's T2 point: value, T2 derivative (cell units)
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const double own = sv[r][0], own_d = sd[r][0];
    const double rcv = lane_xor<2>(sv[r][1]), rcv_d = lane_xor<2>(sd[r][1]);
    // item 2 r is lane m3 = 0's, item 2 r + 1 lane m3 = 1's
    item[2 * r] = m3 ? rcv : own;
    item_d[2 * r] = m3 ? rcv_d : own_d;
    if (2 * r + 1 < 15) {
      item[2 * r + 1] = m3 ? own : rcv;
      item_d[2 * r + 1] = m3 ? own_d : rcv_d;
    }
  }
  double Ws[NC], dWs[3][NC];  // this lane's side at its Gauss point, face frame
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    Ws[q] = item[3 * q];
    dWs[2][q] = item_d[3 * q] * i2d;
    dWs[1][q] = item[3 * q + 1];
    dWs[0][q] = item[3 * q + 2];
  }
  if (EX && live && a.fallback) {
    // first-order fallback: this side's cell (fa - 1 + m2 along AX), frame order
    int cp[3] = {fp[0], fp[1], fp[2]};
    cp[AX] = fa - 1 + m2;
    double C[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) C[q] = load_cell(g, a.W, perm[q], cp[0], cp[1], cp[2]);
    if (fallback_side<NC, 3>(Ws, dWs, C, a.gamma) && a.fbc) atomicAdd(a.fbc, 1ull);
  }

  // 4. the Gauss-point flux, one side per lane
  Gas<3, double> gs, g0;
  double h0 = 0.0, h1 = 0.0, w0[NC] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (live) side_w0<3>(Ws, a.fc, m2 ? -1.0 : 1.0, gs, h0, h1, w0);
  double W0[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) W0[q] = w0[q] + lane_xor<1>(w0[q]);
  SidePart<3, double> P, T;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
#pragma unroll
    for (int d = 0; d < 3; ++d) P.dW0[d][q] = 0.0;
    P.S1[q] = P.S2[q] = P.S3[q] = 0.0;
  }
  P.H1 = P.H2 = P.H3 = 0.0;
  bool ok = true;
  const double ps = live ? gs.rho * gs.h : 0.0, pp = lane_xor<1>(ps);
  FluxTime<double> ftm{0.0, 0.0};
  if (live) {
    make_gas<3>(W0, a.fc.N, g0);
    ftm = flux_time<3>(g0, ps, pp, a.fc, dt);
    side_part<3, NS>(gs, h0, h1, dWs, a.fc, g0, P);
    ok = gs.ok && g0.ok;
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
#pragma unroll
    for (int d = 0; d < 3; ++d) T.dW0[d][q] = P.dW0[d][q] + lane_xor<1>(P.dW0[d][q]);
    T.S1[q] = P.S1[q] + lane_xor<1>(P.S1[q]);
    T.S2[q] = P.S2[q] + lane_xor<1>(P.S2[q]);
    T.S3[q] = P.S3[q] + lane_xor<1>(P.S3[q]);
  }
  if (NS) {
    T.H1 = P.H1 + lane_xor<1>(P.H1);
    T.H2 = P.H2 + lane_xor<1>(P.H2);
    T.H3 = P.H3 + lane_xor<1>(P.H3);
  } else {
    T.H1 = T.H2 = T.H3 = 0.0;
  }
  ok = ok && (lane_xor<1>((int)ok) != 0);
  double A[NC] = {0, 0, 0, 0, 0}, B[NC] = {0, 0, 0, 0, 0};
  if (live) {
    flux_combine<3, NS, flux_out(STAGE)>(W0, g0, T, ftm, a.fc, dt, 0.25, A, B);
    if (!ok && m2 == 0) atomicAdd(a.fail, 1ull);
  }
  // sum over the four Gauss points (m3, m1); both lanes of a pair hold the
  // same flux
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    A[q] += lane_xor<2>(A[q]);
    A[q] += other_quad(A[q]);  // quads hold their sums after the two steps above
    if (STAGE == 1) {
      B[q] += lane_xor<2>(B[q]);
      B[q] += other_quad(B[q]);
    }
  }
  wall_fluxes<NC>(g, AX, fa, A, B);
  if (live && (tid & 7) == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      a.FA[(long long)perm[q] * nf + fid] = A[q];
      if (STAGE == 1) a.FB[(long long)perm[q] * nf + fid] = B[q];
    }
  }
}

// ---------------------------------------------------------------------------
// Updates.  Face arrays of direction d: [nc][faces_d] with the face index of
// cell (i,j,k)'s low face equal to the cell index in a grid whose axis d has
// n[d] + 1 entries.
// ---------------------------------------------------------------------------
struct UpdateArgs {
  Geom g;
  const double* W;    // stage 1: W^n; stage 2: P
  double* out1;       // stage 1: W*; stage 2: W^{n+1}
  double* out2;       // stage 1: P
  const double* FA[3];
  const double* FB[3];
  const double* dt;
  double gamma, mu;
  double* partial;    // stage 2 with CFL: one minimum per block, or null
};

// cell id of this thread; the block's CFL minimum goes to *partial.  Large grids
// move the face fluxes at 5 TB/s, the rate of a copy; a small grid waits:
// hence 32-bit index arithmetic (a 64-bit quotient takes some hundred
// instructions) and loads that do not wait for the time step (97 x 61, one
// update: 4.6 -> 4.1 us).  STOP: the fluxes are read only where the step
// advances: batches, in which instances stop, and single grids beyond
// CLOCK_NBLK blocks, where other wavefronts hide the wait and a step after the
// end time costs its traffic (1000 x 1000, 20 such steps: 1.77 ms, 2.60 with
// the fluxes read; four steps that advance 2.46 and 2.47 ms; at 256 x 256, below
// the line, 0.37 and 0.32 ms either way).
template <int D, int STAGE, bool CFL, bool STOP = false>
__device__ __forceinline__ void update_body(const UpdateArgs& u, long long id, double* partial) {
  constexpr int NC = D + 2;
  const Geom& g = u.g;
  const bool live = id < g.ncell;
  const double dt = *u.dt;
  const bool adv = dt > 0.0;
  double w1[NC];
  if (live) {
    int i, j, k;
    if (g.ncell <= 0x7fffffffLL) {
      const unsigned n0 = (unsigned)g.n[0], q = (unsigned)id / n0;
      i = (int)((unsigned)id - q * n0);
      k = D >= 3 ? (int)(q / (unsigned)g.n[1]) : 0;
      j = (int)q - k * g.n[1];
    } else {
      const long long q = id / g.n[0];
      i = (int)(id - q * g.n[0]);
      k = D >= 3 ? (int)(q / g.n[1]) : 0;
      j = (int)(q - (long long)k * g.n[1]);
    }
    long long lo[3], hi[3], nf[3];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int e0 = g.n[0] + (d == 0), e1 = g.n[1] + (d == 1);
      nf[d] = (long long)e0 * e1 * (g.n[2] + (d == 2));
      lo[d] = ((long long)k * e1 + j) * e0 + i;
      hi[d] = lo[d] + (d == 0 ? 1 : d == 1 ? (long long)e0 : (long long)e0 * e1);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double w = u.W[(long long)c * g.ncell + id];
      double a = w, b = w;
      if (adv || !STOP) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const double* FA = u.FA[d] + (long long)c * nf[d];
          a -= (FA[hi[d]] - FA[lo[d]]) / g.dx[d];
          if (STAGE == 1) {
            const double* FB = u.FB[d] + (long long)c * nf[d];
            b -= (FB[hi[d]] - FB[lo[d]]) / g.dx[d];
          }
        }
      }
      a = adv ? a : w;
      u.out1[(long long)c * g.ncell + id] = a;
      if (STAGE == 1) u.out2[(long long)c * g.ncell + id] = adv ? b : w;
      w1[c] = a;
    }
  }
  if (CFL) {
    double dxm = g.dx[0];
    for (int d = 1; d < D; ++d) dxm = fmin(dxm, g.dx[d]);
    block_cfl<D>(live, w1, u.gamma, u.mu, dxm, partial);
  }
}

template <int D, int STAGE, bool CFL, bool STOP>
__global__ __launch_bounds__(256) void update_kernel(UpdateArgs u) {
  update_body<D, STAGE, CFL, STOP>(u, (long long)blockIdx.x * blockDim.x + threadIdx.x,
                                   CFL ? u.partial + blockIdx.x : nullptr);
}

// CFL partial minima of a state (no update); id: the thread's cell, if live
template <int D>
__device__ __forceinline__ void cfl_partial_body(const Geom& g, const double* W, double gamma, double mu,
                                                 long long id, bool live, double* partial) {
  constexpr int NC = D + 2;
  double dxm = g.dx[0];
  for (int d = 1; d < D; ++d) dxm = fmin(dxm, g.dx[d]);
  live = live && id < g.ncell;
  double w[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) w[c] = live ? W[(long long)c * g.ncell + id] : 1.0;
  block_cfl<D>(live, w, gamma, mu, dxm, partial);
}

// per: cells per block (one partial minimum each), at most the block's threads
template <int D>
__global__ __launch_bounds__(256) void cfl_partial_kernel(Geom g, const double* W, double gamma, double mu, int per,
                                                          double* partial) {
  cfl_partial_body<D>(g, W, gamma, mu, (long long)blockIdx.x * per + threadIdx.x, (int)threadIdx.x < per,
                      partial + blockIdx.x);
}

// Final reduction.  clock = {t, dt}.  mode 0: dt_out = cfl * min (clipped to
// t_end - t_in); mode 1 (after a step): t += dt, then the next dt as mode 0;
// mode 2: fixed step, t += dt only.
__device__ __forceinline__ void finalize_body(const double* partial, int nblk, double cfl, double t_in,
                                              double t_end, double* clock, double* dt_out, int mode) {
  __shared__ double red[16];  // one entry per wave, up to 1024 threads
  double v = INFINITY;
  bool nan = false;
  if (mode != 2)
    for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
      const double p = partial[i];
      if (!(p == p)) nan = true;
      v = fmin(v, p);
    }
  v = block_min(nan ? -INFINITY : v, red);
  if (threadIdx.x == 0) {
    double t = t_in;
    if (mode >= 1) {
      t = clock[0];
      const double used = clock[1];
      if (used > 0.0) t += used;
    }
    if (clock) clock[0] = t;
    if (mode != 2) {
      const double dt = next_dt(v, cfl, t, t_end);
      if (clock) clock[1] = dt;
      if (dt_out) *dt_out = dt;
    }
  }
}

// The whole CFL step of a small state in one block: one launch instead of two
// as long as the block's threads pass over few cells.  400 cells 5.5 us (7.7 in
// two launches), 4,096 cells 6.5 (7.6), 14,000 cells 13.9 (7.8).
constexpr int CFL_ONE = 4096;

template <int D>
__global__ __launch_bounds__(1024) void cfl_one_kernel(Geom g, const double* W, double gamma, double mu, double cfl,
                                                       double t_in, double t_end, double* clock, double* dt_out) {
  constexpr int NC = D + 2;
  __shared__ double red[16];  // one entry per wave
  double dxm = g.dx[0];
  for (int d = 1; d < D; ++d) dxm = fmin(dxm, g.dx[d]);
  double v = INFINITY;
  bool nan = false;
  for (int id = threadIdx.x; id < (int)g.ncell; id += blockDim.x) {
    double w[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) w[c] = W[(long long)c * g.ncell + id];
    const double x = cell_dt<D>(w, gamma, mu, dxm);
    nan = nan || !(x == x);
    v = fmin(v, x);
  }
  v = block_min(nan ? -INFINITY : v, red);
  if (threadIdx.x == 0) {
    const double dt = next_dt(v, cfl, t_in, t_end);
    if (clock) {
      clock[0] = t_in;
      clock[1] = dt;
    }
    if (dt_out) *dt_out = dt;
  }
}

static __global__ __launch_bounds__(256) void cfl_finalize_kernel(const double* partial, int nblk, double cfl,
                                                           double t_in, double t_end, double* clock,
                                                           double* dt_out, int mode) {
  finalize_body(partial, nblk, cfl, t_in, t_end, clock, dt_out, mode);
}

// clears n counters (a kernel rather than a memset, so that a caller may
// capture it into a graph)
static __global__ __launch_bounds__(256) void zero_counters_kernel(unsigned long long* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

static __global__ void set_clock_kernel(double* clock, double t, double dt) {
  clock[0] = t;
  clock[1] = dt;
}

}  // namespace tgks
