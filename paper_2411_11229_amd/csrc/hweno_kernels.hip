// HIP kernels and C ABI of the HWENO-I hot path for gfx950.
//
// Forward stage kernel ("marcher"): one wavefront per block. The 64 lanes
// hold 64 consecutive cells of a row (60 output columns plus a 2-cell halo
// on each side); x-neighbours are read across lanes. The wavefront marches
// up a strip of rows, keeping in registers (and, for the pointwise y-fluxes
// and pending updates, in LDS) what the y-stencil still needs, in a tile
// order that keeps neighbouring tiles behind one XCD's L2, so every cell's
// HWENO interpolation is done once per direction and
// every input value is read from memory once per strip (plus halos).
// Per output cell and stage it does: the x-sweep (HWENO, pointwise fluxes,
// central correction, LF flux, mixed flux, flux difference), the y-sweep
// likewise, the residual (odeH)/(ode2H) and the SSP-RK3 combination
// (fully-hweno)/(2Dfully-hweno), and the max wave speed of the new state for
// the next stage's Lax-Friedrichs alpha (after stage 3: the next step's).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <atomic>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "../../include/hweno.h"
#include "hweno_adjoint_diff.h"
#include "hweno_device.h"

namespace hweno {

enum Mode { kRhs = 0, kStage1 = 1, kStage2 = 2, kStage3 = 3 };

// A split y side (see hweno_split): ghost (x, y) follows kind[0] where
// x < x0 + slope y + speed t, else kind[1].
struct SplitRule {
  double x0, slope, speed;
  int kind[2];
  double state[2][4];
};

// Workspace scalars of a time step.
struct StepScalars {
  double dt;
  double t0;                      // the step's start time
  double tnew;                    // its end time (t0 + dt, or t_end when clipped)
  int active;
  unsigned flags;
};

// Accumulators of the Lax-Friedrichs alphas, behind the scalars: kSlots slots,
// in each one (x, y) pair per set, holding the non-negative doubles' bit
// patterns (atomic max). A stage's blocks spread over the slots, the next stage
// takes the maximum over them: a thousand blocks' atomics on one pair of
// addresses serialise (512^2 FP64: 50 us a stage with one slot, 34 with 32; 33
// without the atomics). Up to kOneSlotBlocks blocks use one slot, which costs
// the next stage no reduction (0.5 us a launch: 1D, N = 2000, 34 blocks).
// Sets: kSet2 the stage-2 alphas (written by stage 1), kSet3 the stage-3 alphas
// (by stage 2), kSetNext the next step's stage-1 alphas, i.e. those of the
// step's result (by stage 3), kSetSeed the stage-1 alphas of a call's first step
// (by the pass over its initial state). Between calls kSet2 and kSetSeed are
// zero, also after a call that returned an error (alpha_clear_kernel).
constexpr int kSlots = 32, kSets = 4, kOneSlotBlocks = 64;
enum AlphaSet { kSet2 = 0, kSet3 = 1, kSetNext = 2, kSetSeed = 3 };
constexpr size_t kSlotOffset = 2048;   // from the scalars, in bytes
struct AlphaSlots {
  unsigned long long v[kSlots][kSets][2];
};
__host__ __device__ inline AlphaSlots* alpha_slots(StepScalars* sc) {
  return (AlphaSlots*)((char*)sc + kSlotOffset);
}
// Behind the accumulators: the blocks of a speed_kernel launch that are done, per
// slot, each count in a line of its own, and the slots whose blocks all are. Zero
// between launches.
struct SpeedTickets {
  unsigned slot[kSlots][16];
  unsigned slots;
};
constexpr size_t kTicketOffset = kSlotOffset + sizeof(AlphaSlots);
__host__ __device__ inline SpeedTickets* speed_tickets(StepScalars* sc) {
  return (SpeedTickets*)((char*)sc + kTicketOffset);
}

// Time-step control of a stage-1 launch that computes dt itself (flux-LF): from
// its alphas by `rule` (production cfl / (ax/hx + ay/hy) with hx, hy = dx, dy;
// accuracy the same with dx^(5/3), dy^(5/3); fixed dt_fixed), clipped so that
// t + dt does not pass t_end. sc null: dt is given (frozen steps, adjoint).
struct StepCtl {
  StepScalars* sc;
  double* t;                      // the caller's time (read by stage 1, advanced by stage 2)
  double* dt_used;                // or null
  int rule, dim;
  double cfl, dt_fixed, t_end, hx, hy;
};

// Scales between what the stage kernels carry and the scheme's quantities: a
// row's derivatives are multiplied by lx = lam dx, ly = lam dy when it is
// loaded (Carried); ilx, ily their inverses; vtx, vty times the modified
// derivatives of the interpolation give v~, w~; xu, xv, xw times the
// differences F_{i-1/2} - F_{i+1/2} of the scaled interface fluxes
// (interface_flux) along x give L of the three equations, yu, yv, yw along y.
struct FluxK {
  double lx, ly, ilx, ily, vtx, vty, xu, xv, xw, yu, yv, yw;
};

template <typename T>
struct StageArgs {
  const T* U;  const T* V;  const T* W;   // stage state X (W null in 1D)
  const T* Ub; const T* Vb; const T* Wb;  // RK base B^n = (U^n, V~^n, W~^n), stages 2-3
  T* Uo; T* Vo; T* Wo;                    // new state (stages) or L^1..L^3 (rhs)
  T* Vt; T* Wt;                           // stage 1: V~^n, W~^n; rhs: modified derivatives
  const double* alpha;                    // [2] LF alphas of this stage, or null: set alpha_set
  int alpha_set, next_set;                // of ctl.sc: read from, written to (next_set -1: no)
  int nslots;                             // accumulator slots in use: 1 or kSlots
  const double* dt;                       // stages 2-3, frozen steps: time step
  const int* active;                      // stages 2-3: 0 = the step is skipped
  double* alpha_rec;                      // [2] record of the alphas used, or null
  int nx, ny, rows;                       // rows: output rows per block (2D)
  int plane;                              // nx * ny
  int bc[4];
  int iface;                              // host side: interface characteristic basis
  double gs[4][4];                        // fixed (Dirichlet) ghost states per side
  double gravity;                         // g of the (euler2d-s) source
  SplitRule sp[2];                        // split y sides (low, high)
  const double* t0;                       // step start time (device), null: t = 0
  double tc;                              // this stage's time: t0 + tc dt
  StepCtl ctl;                            // stage 1 computing dt, stages 2-3 of such a step
  Scheme s;
  PointK pk;                              // HWENO point constants (difference form)
  FluxK fk;
};

// Maximum over the wavefront's lanes of a non-negative double, in scalar
// registers: DPP row shifts, then the row broadcasts (absent lanes give 0).
template <int CTRL>
__device__ __forceinline__ double dpp_max_step(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return fmax(v, __hiloint2double(hi, lo));
}
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max_step<0x111>(v);   // row_shr:1, 2, 4, 8
  v = dpp_max_step<0x112>(v);
  v = dpp_max_step<0x114>(v);
  v = dpp_max_step<0x118>(v);
  v = dpp_max_step<0x142>(v);   // row_bcast:15, 31
  v = dpp_max_step<0x143>(v);
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), kWave - 1),
                          __builtin_amdgcn_readlane(__double2loint(v), kWave - 1));
}
__device__ __forceinline__ unsigned wave_or(unsigned v) {
  unsigned r = 0;
#pragma unroll
  for (int b = 0; b < 2; ++b) r |= __ballot((v >> b) & 1u) ? 1u << b : 0u;
  return r;
}
// Atomic max of non-negative doubles through their bit patterns (ordered
// like unsigned integers); order-independent, hence deterministic.
__device__ __forceinline__ unsigned long long atomic_max_pos(unsigned long long* p, double v) {
  return atomicMax(p, (unsigned long long)__double_as_longlong(v));
}
// One lane adds its block's maxima and state flags to the accumulators.
template <int DIM>
__device__ __forceinline__ void raise_alphas(StepScalars* sc, int nslots, int set, int block, double ax,
                                             double ay, unsigned flag) {
  unsigned long long* p = alpha_slots(sc)->v[nslots == 1 ? 0 : block % kSlots][set];
  atomic_max_pos(p, ax);
  if (DIM == 2) atomic_max_pos(p + 1, ay);
  if (flag) atomicOr(&sc->flags, flag);
}

// Touches the whole 64-byte lines of a kernel's first argument, all in flight at
// once: the code's own reads of them, spread over the kernel's start, then find
// them in the scalar cache instead of waiting for one line after the other. (us a
// pass: 60x240 with walls, 24 stage launches, 244 -> 218; 1D Euler N = 2000, 96,
// 556 -> 514; 512^2, 12, 377 -> 369.) The line begun last, with the end of that
// argument and the system's constants, is left to those reads: with it too the
// adjoint and small scalar grids gain 1-2%, stages with walls lose up to 0.8%.
template <class Args>
__device__ __forceinline__ void touch_args() {
  const volatile __attribute__((address_space(4))) unsigned* p =
      (const volatile __attribute__((address_space(4))) unsigned*)__builtin_amdgcn_kernarg_segment_ptr();
  unsigned x[sizeof(Args) / 64];
#pragma unroll
  for (unsigned i = 0; i < sizeof(Args) / 64; ++i) x[i] = p[16 * i];
#pragma unroll
  for (unsigned i = 1; i < sizeof(Args) / 64; ++i) x[0] |= x[i];
  asm volatile("" ::"s"(x[0]));   // (waits here, once)
}

// What a stage launch starts from, read before its rows so that both are in
// flight together: the alphas (with kSlots slots one pair a lane, to be reduced),
// and the step's start time, dt and activity where the launch is given them.
// (1D Euler, N = 2000, launches back to back: 6.6 -> 6.1 us a stage; a 2D stage
// gains 0.1 us or less.)
struct StageIn {
  double ax, ay, t, dt;
  int active;
};
template <int MODE, typename T>
__device__ __forceinline__ StageIn stage_read(const StageArgs<T>& A) {
  StageIn in{0.0, 0.0, 0.0, 0.0, 1};
  const int lane = threadIdx.x & (kWave - 1);
  if (A.alpha) {
    in.ax = A.alpha[0];
    in.ay = A.alpha[1];
  } else if (lane < A.nslots || A.nslots == 1) {
    const unsigned long long* p = alpha_slots(A.ctl.sc)->v[A.nslots == 1 ? 0 : lane][A.alpha_set];
    in.ax = __longlong_as_double((long long)p[0]);
    in.ay = __longlong_as_double((long long)p[1]);
  }
  if (MODE == kStage1 && A.ctl.sc) {
    in.t = *A.ctl.t;
  } else if (MODE != kRhs) {
    if (A.active) in.active = *A.active;
    in.dt = *A.dt;
    if (A.t0) in.t = *A.t0;
  }
  return in;
}

// dt of a step that starts at t0, from its alphas, and its end time; false (dt 0)
// if t_end is reached.
__device__ __forceinline__ bool step_size(const StepCtl& c, double t0, double ax, double ay, double& d,
                                          double& tn) {
  d = c.rule == HWENO_DT_FIXED ? c.dt_fixed
                               : c.cfl / (c.dim == 2 ? ax / c.hx + ay / c.hy : ax / c.hx);
  tn = t0 + d;
  if (!(t0 < c.t_end)) {
    d = 0.0;
    tn = t0;
    return false;
  }
  if (tn >= c.t_end) {
    d = c.t_end - t0;
    tn = c.t_end;
  }
  return true;
}

// Start of a stage launch, by every wavefront: the stage's alphas, dt and time,
// and whether the step is active. A stage 1 with time-step control computes dt
// itself from its alphas (every block alike); the first wavefront of the first
// block (`leader`) also publishes dt, the step's times and the record of the
// alphas, and clears the stage-3 accumulators. Stage 2 of such a step advances
// the caller's time and clears the next-step and seed accumulators (read by
// stage 1; the former written again by stage 3); stage 3 clears the stage-2
// accumulators. Each clear comes after the last read of those accumulators and
// before their next writer, one kernel boundary apart. A skipped step leaves
// all but the seed set as they are.
template <int MODE, typename T>
__device__ __forceinline__ bool stage_begin(const StageArgs<T>& A, const StageIn& in, bool leader,
                                            double& ax, double& ay, double& dt, double& tstage) {
  dt = 0.0;
  tstage = 0.0;
  const StepCtl& c = A.ctl;
  const int lane = threadIdx.x & (kWave - 1);
  const bool first = leader && lane == 0;
  auto clear = [&](int set) {
    if (lane < kSlots) {
      unsigned long long* p = alpha_slots(c.sc)->v[lane][set];
      p[0] = p[1] = 0ull;
    }
  };
  const bool reduce = !A.alpha && A.nslots != 1;
  ax = reduce ? wave_max(in.ax) : in.ax;
  ay = reduce ? wave_max(in.ay) : in.ay;
  if (MODE == kRhs) return true;
  if (MODE == kStage1 && c.sc) {
    if (c.dim == 1) ay = 0.0;
    const double t0 = in.t;
    double d, tn;
    const bool active = step_size(c, t0, ax, ay, d, tn);
    if (leader) clear(kSet3);
    if (leader && !active && A.alpha_set == kSetSeed && lane < kSlots) {
      // nothing was stepped: the seed stays the next step's alphas
      AlphaSlots* a = alpha_slots(c.sc);
      a->v[lane][kSetNext][0] = a->v[lane][kSetSeed][0];
      a->v[lane][kSetNext][1] = a->v[lane][kSetSeed][1];
    }
    if (first) {
      c.sc->dt = d;
      c.sc->t0 = t0;
      c.sc->tnew = tn;
      c.sc->active = active ? 1 : 0;
      if (c.dt_used) *c.dt_used = d;
      if (A.alpha_rec) {
        A.alpha_rec[0] = ax;
        A.alpha_rec[1] = ay;
      }
    }
    dt = d;
    tstage = t0;
    return active;
  }
  if (MODE == kStage2 && c.sc && leader) clear(kSetSeed);
  if (in.active == 0) return false;
  dt = in.dt;
  tstage = A.t0 ? in.t + A.tc * dt : 0.0;
  if (first) {
    if (A.alpha_rec) {
      A.alpha_rec[0] = ax;
      A.alpha_rec[1] = A.ctl.dim == 1 ? 0.0 : ay;
    }
    if (c.sc && MODE == kStage2) *c.t = c.sc->tnew;
  }
  if (leader && c.sc) {
    if (MODE == kStage2) clear(kSetNext);
    if (MODE == kStage3) clear(kSet2);
  }
  return true;
}

// ---------------------------------------------------------------- helpers
// Element idx of a state array through a 32-bit byte offset from the uniform
// base pointer: the loads and stores then take the scalar-base form (base in
// SGPRs, offset in one VGPR) instead of a 64-bit address per lane. The host
// guarantees ncomp * plane * sizeof(T) < 2^32.
template <typename T>
__device__ __forceinline__ T ld32(const T* base, unsigned idx) {
  return *(const T*)((const char*)base + idx * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void st32(T* base, unsigned idx, T v) {
  *(T*)((char*)base + idx * (unsigned)sizeof(T)) = v;
}
// Asynchronous copies of kWave consecutive elements of a row (from column
// col0, columns outside [0, nx) clamped to the edge) straight from global memory into
// LDS (dst[0..kWave)), with no VGPR in between: each 4-byte load of a wave
// writes lane i's word at byte 4i of its 256-byte part. The caller orders
// them with LDS reads of dst: wait_copies() before reading the copy,
// wait_lds_reads() after the last read of dst's previous contents. The lanes'
// byte offsets in a row are formed once (one VALU instruction a load is left).
template <typename T>
struct RowCopy {
  static constexpr int P = sizeof(T) / 4;
  unsigned off[P];
  __device__ __forceinline__ RowCopy(int col0, int nx, int lane) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int col = max(0, min(col0 + j * (kWave / P) + lane / P, nx - 1));
      off[j] = (unsigned)col * (unsigned)sizeof(T) + 4u * (unsigned)(lane % P);
    }
  }
  __device__ __forceinline__ void operator()(const T* base, unsigned row_off, T* dst) const {
#pragma unroll
    for (int j = 0; j < P; ++j)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)((const char*)base +
                                                          (row_off * (unsigned)sizeof(T) + off[j])),
          (__attribute__((address_space(3))) void*)((char*)dst + 256 * j), 4, 0, 0);
  }
};
// Waits that are also compiler barriers for memory accesses (the compiler's
// own wait insertion does not order every LDS read after a pending copy)
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// ------------------------------------------------------ x-direction sweep
// The numerical fluxes (flux-1d), (flux-LF) with the central correction
// (Cd-1)-(DfDh) at one interface x_{i+1/2}, from the pointwise fluxes as f0 =
// f_i and the differences d0 = f_i - f_{i-1}, d1, d2 (FP64) or the values fm,
// f0, f1, f2 at i-1 .. i+2 (FP32, d unused), the pointwise derivative fluxes
// hm = h'_{i-1}, hp = h'_{i+2} (h' = lam h f'(u) v), and the sums sF, sH of
// the LF terms f + a u of the two sides (those of the derivative equation
// carry mu besides). In FP64 scaled so that every term costs one FMA or none:
//   F = -960 lam / 19 f_{i+1/2},   H = 864 / 37 (lam h) h_{i+1/2};
// in FP32 (kFluxScaled false) F = f_{i+1/2}, H = h h_{i+1/2}.
template <typename T>
constexpr bool kFluxScaled = sizeof(T) == 8;
template <typename T>
__device__ __forceinline__ void interface_flux(T d0, T d1, T d2, T hm, T hp, T sF, T sH, T& F, T& H) {
  constexpr double lam = Carried<T>::lam, mu = Carried<T>::mu;
  F = fma(T(-480.0 / 19.0 * lam), sF, fma(T(97.0 / 38.0 * lam), d2 - d0, hm - hp));
  H = fma(T(432.0 / 37.0 / mu), sH,
          fma(T(475.0 / 111.0 * lam), d1, fma(T(-697.0 / 222.0 * lam), d0 + d2, hm + hp)));
}
template <typename T>
__device__ __forceinline__ void interface_flux_plain(T fm, T f0, T f1, T f2, T hm, T hp, T sF, T sH,
                                                     T& F, T& H) {
  const T s4 = (fm + f2) - (f0 + f1);
  const T Df = fma(T(-97.0 / 1920.0), s4, T(-19.0 / 960.0) * (hm - hp));
  const T Dh = fma(T(697.0 / 5184.0), fm - f2, fma(T(-61.0 / 192.0), f0 - f1, T(37.0 / 864.0) * (hm + hp)));
  F = fma(T(0.5), sF, Df);
  H = fma(T(0.5), sH, Dh);
}

// Steps 1-4 of section 2 along x for the row held by the wavefront (one cell
// per lane). Inputs: this lane's U, V' = lam dx u_x and, with NF == 3,
// W' = lam dy u_y (carried derivatives, see hweno_cell_diff), and the cell's
// characteristic basis and primitives `ce`. Outputs: the differences
// F_{i-1/2} - F_{i+1/2} of the scaled fluxes of the u-, v- and w-equations
// (the last 12 times the mixed flux of eta = f'(u) w'), formed in double, and
// the modified derivative as hweno_cell_diff scales it. Valid on lanes 2..61.
template <int NF, bool IFACE, class Sys, typename T>
__device__ __forceinline__ void sweep_x(const Sys& sy, const Scheme& s, const PointK& pk,
                                        double alpha,
                                        const typename Sys::template CellEig<T>& ce,
                                        const T (&U)[Sys::NC], const T (&V)[Sys::NC],
                                        const T (&W)[Sys::NC], double (&RU)[Sys::NC],
                                        double (&RV)[Sys::NC], double (&RW)[Sys::NC],
                                        T (&vt)[Sys::NC]) {
  constexpr int NC = Sys::NC;
  // Step 1: HWENO once per cell -> u at both faces, v~ at the centre, and the
  // face derivatives of (P'xi)
  T uR[NC], uL[NC], vR[NC], vL[NC];
  if constexpr (IFACE && sizeof(T) == 4) {
    T Um[NC], Up[NC], Vm[NC], Vp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Um[c] = from_prev(U[c]);
      Up[c] = from_next(U[c]);
      Vm[c] = from_prev(V[c]);
      Vp[c] = from_next(V[c]);
    }
    // mesh width 1 for the scaled derivatives
    hweno_cell_b<0, true>(sy, s, 1.0, 1.0, ce.q, Um, U, Up, Vm, Vp, uR, uL, vt);
#pragma unroll
    for (int c = 0; c < NC; ++c) face_derivs(Um[c], U[c], Up[c], Vm[c], Vp[c], T(1), vR[c], vL[c]);
  } else {
    // the stencil as differences: E1 = U_i - U_{i-1}, E2 = U_{i+1} - U_i
    // (E1 of the next lane), S and D the sum and difference of V'_{i-1}, V'_{i+1}
    T E1[NC], E2[NC], Sv[NC], Dv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) E1[c] = U[c] - from_prev(U[c]);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      E2[c] = from_next(E1[c]);
      const T vm = from_prev(V[c]), vp = from_next(V[c]);
      Sv[c] = vm + vp;
      Dv[c] = vm - vp;
    }
    if constexpr (IFACE) {
      T Um[NC], Up[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        Um[c] = from_prev(U[c]);
        Up[c] = from_next(U[c]);
      }
      hweno_cell_diff_iface<0>(sy, pk, ce, Um, U, Up, E1, E2, Sv, Dv, uR, uL, vt, vR, vL);
    } else {
      hweno_cell_diff<0>(sy, pk, ce, U, E1, E2, Sv, Dv, uR, uL, vt, vR, vL);
    }
  }
  // pointwise f, h' = f'(u) v', eta' = f'(u) w' at the cell centre
  T f[NC], hf[NC], e[NC] = {};
  sy.template flux<0>(U, ce.q, f);
  sy.template jac<0>(U, ce.q, V, hf);
  if constexpr (NF == 3) sy.template jac<0>(U, ce.q, W, e);
  round_all(f);
  round_all(hf);
  round_all(e);
  // Lax-Friedrichs sums of this cell's faces (flux-LF), halved at the
  // interface: f(u^-) + a u^- at x_{i+1/2}, f(u^+) - a u^+ at x_{i-1/2}
  T mF[NC], mH[NC], pF[NC], pH[NC];
  {
    const T a = T(alpha);
    T fr[NC], hr[NC], fl[NC], hl[NC];
    const auto qr = prim_rounded(sy, uR);
    sy.template flux<0>(uR, qr, fr);
    sy.template jac<0>(uR, qr, vR, hr);
    const auto ql = prim_rounded(sy, uL);
    sy.template flux<0>(uL, ql, fl);
    sy.template jac<0>(uL, ql, vL, hl);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      mF[c] = fma(a, uR[c], fr[c]);
      mH[c] = fma(a, vR[c], hr[c]);
      pF[c] = fma(-a, uL[c], fl[c]);
      pH[c] = fma(-a, vL[c], hl[c]);
    }
  }
  // Steps 2-3 at x_{i+1/2}, then the differences of Step 4
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    T Fi, Hi;
    const T sF = mF[c] + from_next(pF[c]), sH = mH[c] + from_next(pH[c]);
    if constexpr (kFluxScaled<T>) {
      const T d0 = f[c] - from_prev(f[c]), d1 = from_next(d0), d2 = from_next(d1);
      interface_flux(d0, d1, d2, from_prev(hf[c]), from_next2(hf[c]), sF, sH, Fi, Hi);
    } else {
      const T fp = from_next(f[c]);
      interface_flux_plain(from_prev(f[c]), f[c], fp, from_next(fp), from_prev(hf[c]),
                           from_next2(hf[c]), sF, sH, Fi, Hi);
    }
    RU[c] = (double)from_prev(Fi) - (double)Fi;
    RV[c] = (double)from_prev(Hi) - (double)Hi;
    if constexpr (NF == 3) {
      // (mixed) times 12: 7 (e_i + e_{i+1}) - (e_{i-1} + e_{i+2})
      const T em1 = from_prev(e[c]), ep1 = from_next(e[c]), ep2 = from_next(ep1);
      const T Ei = fma(T(7), e[c] + ep1, -(em1 + ep2));
      RW[c] = (double)from_prev(Ei) - (double)Ei;
    }
  }
}

// The Runge-Kutta combination (fully-hweno)/(2Dfully-hweno) of one value, in
// two parts: X_new = rk_base + rk_wl dt L, with
//   stage 1: X + dt L,  stage 2: 3/4 B + 1/4 (X + dt L),
//   stage 3: 1/3 B + 2/3 (X + dt L),  operator only (rhs): L.
// X is x times `scale` (1, or the scale of a modified derivative). All in
// double, one rounding at the store. The stage-3 weights multiply (an FP64
// division would cost about ten instructions per value).
template <int MODE>
__device__ __forceinline__ double rk_x(double scale) {
  return MODE == kStage2 ? 0.25 * scale : (MODE == kStage3 ? (2.0 / 3.0) * scale : scale);
}
template <int MODE>
__device__ __forceinline__ double rk_base(double x, double wx, double base) {
  if constexpr (MODE == kStage1) return wx * x;
  else if constexpr (MODE == kStage2) return fma(wx, x, 0.75 * base);
  else if constexpr (MODE == kStage3) return fma(wx, x, (1.0 / 3.0) * base);
  else return 0.0;
}
template <int MODE>
__device__ __forceinline__ double rk_wl(double dt) {
  if constexpr (MODE == kStage1) return dt;
  else if constexpr (MODE == kStage2) return 0.25 * dt;
  else if constexpr (MODE == kStage3) return (2.0 / 3.0) * dt;
  else return 1.0;
}

// ------------------------------------------------------------ 1D stage kernels
// One stage on a line of 64 cells, one a lane (column col, mapped to g): from
// the loaded U, V the new state, the modified derivative and the weighted RK
// combination with the base Bu, Bv (stages 2-3). Halo lanes' results are void.
template <int MODE, bool IFACE, class Sys, typename T>
__device__ __forceinline__ void stage1d_line(const StageArgs<T>& A, const Sys& sy, int col, double ax,
                                             double dt, T (&U)[Sys::NC], T (&V)[Sys::NC],
                                             const T (&Bu)[Sys::NC], const T (&Bv)[Sys::NC],
                                             T (&Un)[Sys::NC], T (&Vn)[Sys::NC], T (&Vt)[Sys::NC]) {
  constexpr int NC = Sys::NC;
  const bool m = mirrored(col, A.nx, A.bc[0], A.bc[1]);
  mirror_state<Sys, 0>(m, U);
  mirror_normal_derivative<Sys, 0>(m, V);
  const int fs = fixed_side(col, A.nx, A.bc[0], A.bc[1]);
  if (fs >= 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      U[c] = T(A.gs[fs][c]);
      V[c] = T(0);
    }
  }
  // the carried derivatives (see sweep_x)
#pragma unroll
  for (int c = 0; c < NC; ++c) V[c] = T(A.fk.lx) * V[c];
  double RU[NC], RV[NC], RW[NC];
  T W[NC], vt[NC];
  const auto ce = sy.cell_eig(U);
  sweep_x<2, IFACE>(sy, A.s, A.pk, ax, ce, U, V, W, RU, RV, RW, vt);
  const double wl = rk_wl<MODE>(dt), wu = wl * A.fk.xu, wv = wl * A.fk.xv;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double ub = MODE >= kStage2 ? (double)Bu[c] : 0.0;
    const double vb = MODE >= kStage2 ? (double)Bv[c] : 0.0;
    Un[c] = (T)fma(wu, RU[c], rk_base<MODE>((double)U[c], rk_x<MODE>(1.0), ub));
    Vn[c] = (T)fma(wv, RV[c], rk_base<MODE>((double)vt[c], rk_x<MODE>(A.fk.vtx), vb));
    Vt[c] = (T)((double)vt[c] * A.fk.vtx);
  }
}

template <class Sys, typename T, int MODE, bool IFACE>
__global__ __launch_bounds__(64) void stage1d_kernel(StageArgs<T> A, Sys sy) {
  constexpr int NC = Sys::NC;
  const int lane = threadIdx.x;
  touch_args<StageArgs<T>>();
  const StageIn in = stage_read<MODE>(A);
  const int col = blockIdx.x * kXOut - kHalo + lane;
  const int g = map_index(col, A.nx, A.bc[0], A.bc[1]);
  const bool out = lane >= kHalo && lane < kWave - kHalo && col < A.nx;
  T U[NC], V[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    U[c] = A.U[c * A.plane + g];
    V[c] = A.V[c * A.plane + g];
  }
  T Bu[NC], Bv[NC];                      // RK base (stages 2-3)
  if constexpr (MODE >= kStage2) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Bu[c] = A.Ub[c * A.plane + g];
      Bv[c] = A.Vb[c * A.plane + g];
    }
  }
  double ax, ay, dt, tstage;
  if (!stage_begin<MODE>(A, in, blockIdx.x == 0, ax, ay, dt, tstage)) return;
  T Un[NC], Vn[NC], Vt[NC];
  stage1d_line<MODE, IFACE>(A, sy, col, ax, dt, U, V, Bu, Bv, Un, Vn, Vt);
  double smax = 0.0;
  unsigned flag = 0;
  if (out) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int o = c * A.plane + col;
      A.Uo[o] = Un[c];
      A.Vo[o] = Vn[c];
      if (MODE == kStage1 || MODE == kRhs) A.Vt[o] = Vt[c];
    }
    if (A.next_set >= 0) {
      double sy_;
      flag = sy.speeds(Un, smax, sy_);
    }
  }
  if (A.next_set >= 0) {
    smax = wave_max(smax);
    flag = wave_or(flag);
    if (lane == 0) raise_alphas<1>(A.ctl.sc, A.nslots, A.next_set, blockIdx.x, smax, 0.0, flag);
  }
}

// Whole steps of a short line in one block ("line"): wavefront w holds the cells
// 60 w .. 60 w + 59 (with the halo, as a block of stage1d_kernel), the state
// stays in LDS, in two copies that the stages read and write in turn, and so do
// the wavefronts' maxima for the alphas; one barrier a stage. The arithmetic and
// the step control are those of the stage kernels. A launch of those is bound by
// latency and the launch itself, not by its work; here a stage costs its
// arithmetic, the wavefronts of one CU sharing it, and a barrier. FP64 only (see
// rounded()). Measured at the rule (line_fits).
constexpr int kLineSteps = 64;                     // most steps of a launch
constexpr int line_waves(bool iface) { return iface ? 8 : 16; }
template <int NC, typename T>
constexpr size_t line_lds(int nx) {
  return (size_t)4 * NC * nx * sizeof(T) + 2 * line_waves(false) * sizeof(double);
}
template <class Sys, typename T, bool IFACE>
__global__ __launch_bounds__(line_waves(IFACE) * kWave) void steps1d_kernel(StageArgs<T> A, Sys sy,
                                                                           int nsteps) {
  constexpr int NC = Sys::NC;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nw = blockDim.x / kWave;
  touch_args<StageArgs<T>>();
  const StepCtl& ctl = A.ctl;
  const int col = wv * kXOut - kHalo + lane;
  const int g = map_index(col, A.nx, A.bc[0], A.bc[1]);
  const bool out = lane >= kHalo && lane < kWave - kHalo && col < A.nx;
  const bool first = threadIdx.x == 0;
  extern __shared__ __align__(16) char line_smem[];
  double* const peak = (double*)line_smem;         // [copy][wavefront]
  T* const state = (T*)(peak + 2 * line_waves(false));   // [copy][u, v][NC][nx]
  auto at = [&](int p, int f, int c, int i) -> T& { return state[((p * 2 + f) * NC + c) * A.nx + i]; };
  double smax = 0.0;
  unsigned flag = 0;
  if (out) {
    T u[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      u[c] = A.Uo[c * A.plane + col];
      at(0, 0, c, col) = u[c];
      at(0, 1, c, col) = A.Vo[c * A.plane + col];
    }
    double sy_;
    flag = sy.speeds(u, smax, sy_);
  }
  double t = *ctl.t;
  int p = 0;                                       // the copy that holds the state
  smax = wave_max(smax);
  if (lane == 0) peak[wv] = smax;
  __syncthreads();
  auto alpha = [&]() { return wave_max(lane < nw ? peak[p * line_waves(false) + lane] : 0.0); };
  T Bu[NC], Bv[NC];                                // RK base
#pragma unroll
  for (int c = 0; c < NC; ++c) Bu[c] = Bv[c] = T(0);
  auto stage = [&](auto mode, double ax, double dt) {
    constexpr int MODE = decltype(mode)::value;
    T U[NC], V[NC], Un[NC], Vn[NC], Vt[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      U[c] = at(p, 0, c, g);
      V[c] = at(p, 1, c, g);
      if (MODE == kStage1) Bu[c] = U[c];
    }
    stage1d_line<MODE, IFACE>(A, sy, col, ax, dt, U, V, Bu, Bv, Un, Vn, Vt);
    p ^= 1;
    double sx = 0.0;
    if (out) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        at(p, 0, c, col) = Un[c];
        at(p, 1, c, col) = Vn[c];
        if (MODE == kStage1) Bv[c] = Vt[c];
      }
      double sy_;
      flag |= sy.speeds(Un, sx, sy_);
    }
    sx = wave_max(sx);
    if (lane == 0) peak[p * line_waves(false) + wv] = sx;
    __syncthreads();
  };
  for (int k = 0; k < nsteps; ++k) {
    double ax = alpha(), tn;
    double* rec = A.alpha_rec ? A.alpha_rec + 6 * k : nullptr;
    auto record = [&](int j) {
      if (rec && first) {
        rec[2 * j] = ax;
        rec[2 * j + 1] = 0.0;
      }
    };
    double dt;
    const bool active = step_size(ctl, t, ax, 0.0, dt, tn);
    if (first && ctl.dt_used) ctl.dt_used[k] = dt;
    record(0);
    if (!active) continue;                         // (alike in every wavefront)
    stage(std::integral_constant<int, kStage1>{}, ax, dt);
    ax = alpha();
    record(1);
    stage(std::integral_constant<int, kStage2>{}, ax, dt);
    ax = alpha();
    record(2);
    stage(std::integral_constant<int, kStage3>{}, ax, dt);
    t = tn;
  }
  if (out) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      A.Uo[c * A.plane + col] = at(p, 0, c, col);
      A.Vo[c * A.plane + col] = at(p, 1, c, col);
    }
  }
  flag = wave_or(flag);
  if (lane == 0 && flag) atomicOr(&ctl.sc->flags, flag);
  if (first) *ctl.t = t;
}

// ------------------------------------------------------------ 2D stage kernel
// Loads row r of column gcol (ghost rows and columns by index map). With
// WALLS (some boundary is reflective or fixed): xm, this lane is a ghost
// column behind a reflective wall; xf, the fixed side whose state this ghost
// lane holds (or -1); xwall, some lane of the wavefront is either
// (wave-uniform, so unaffected blocks skip this code). Problems with neither
// use the kernel without this code, whose register allocation it would
// disturb.
template <class Sys, bool WALLS, typename T>
__device__ __forceinline__ void load_row(const StageArgs<T>& A, double tstage, int r, int col,
                                         int gcol, T (&U)[Sys::NC], T (&V)[Sys::NC],
                                         T (&W)[Sys::NC], int& split_rule) {
  int gr = map_index(r, A.ny, A.bc[2], A.bc[3]);
  // split side: this lane's rule from its x, the ghost row's y and the
  // stage time (0: transmissive, 1: reflective, 2 + k: fixed state k)
  split_rule = -1;
  if constexpr (WALLS) {
    const int yside = r < 0 ? 0 : (r >= A.ny ? 1 : -1);
    if (yside >= 0 && A.bc[2 + yside] == kBcSplit) {
      const SplitRule& sr = A.sp[yside];
      const double xs = sr.x0 + sr.slope * ((r + 0.5) * A.s.dy) + sr.speed * tstage;
      const int k = (col + 0.5) * A.s.dx < xs ? 0 : 1;
      const int kind = sr.kind[k];
      split_rule = kind == kBcReflective ? 1 : (kind == kBcDirichlet ? 2 + k : 0);
      if (split_rule == 1) gr = map_index(r, A.ny, kBcReflective, kBcReflective);
    }
  }
  const unsigned off = (unsigned)(gr * A.nx + gcol);
#pragma unroll
  for (int c = 0; c < Sys::NC; ++c) {
    const unsigned i = (unsigned)(c * A.plane) + off;
    U[c] = ld32(A.U, i);
    V[c] = ld32(A.V, i);
    W[c] = ld32(A.W, i);
  }
}

// What load_row leaves to the row's first use (so that the loads stay in
// flight until then): the ghost rules of walls, fixed states and split sides,
// and the scales of the carried derivatives (see sweep_x).
template <class Sys, bool WALLS, typename T>
__device__ __forceinline__ void finish_row(const StageArgs<T>& A, int r, bool xwall, bool xm,
                                           int xf, int split_rule, T (&U)[Sys::NC],
                                           T (&V)[Sys::NC], T (&W)[Sys::NC]) {
  if constexpr (WALLS) {
    auto fix = [&](int side) {
#pragma unroll
      for (int c = 0; c < Sys::NC; ++c) {
        U[c] = T(A.gs[side][c]);
        V[c] = T(0);
        W[c] = T(0);
      }
    };
    if (xwall) {
      mirror_state<Sys, 0>(xm, U);
      mirror_normal_derivative<Sys, 0>(xm, V);
      mirror_state<Sys, 0>(xm, W);
      if (xf >= 0) fix(xf);
    }
    if (mirrored(r, A.ny, A.bc[2], A.bc[3]) || split_rule == 1) {
      mirror_state<Sys, 1>(true, U);
      mirror_state<Sys, 1>(true, V);
      mirror_normal_derivative<Sys, 1>(true, W);
    }
    const int yf = fixed_side(r, A.ny, A.bc[2], A.bc[3]);
    if (yf >= 0) fix(2 + yf);
    if (split_rule >= 2) {
      const SplitRule& sr = A.sp[r < 0 ? 0 : 1];
#pragma unroll
      for (int c = 0; c < Sys::NC; ++c) {
        U[c] = T(sr.state[split_rule - 2][c]);
        V[c] = T(0);
        W[c] = T(0);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < Sys::NC; ++c) {
    V[c] = rounded(T(A.fk.lx) * V[c]);
    W[c] = rounded(T(A.fk.ly) * W[c]);
  }
}

// VAR: kVarWalls (some boundary is reflective or fixed), kVarIface (interface
// basis), kVarSource (the gravity source of (euler2d-s)); each combination is
// its own instantiation, so the common one carries no code of the others.
constexpr int kVarWalls = 1, kVarIface = 2, kVarSource = 4;

// Tile of a workgroup in a 2D grid of tiles (row-major, gridDim.x tiles a
// row). Workgroups go to the eight XCDs (each with its own L2) in turn by
// linear id; this gives every XCD one contiguous run of tiles, so that
// horizontally adjacent tiles, which re-read each other's halo columns and
// share the cache lines at their edges, mostly sit behind the same L2.
constexpr int kXcds = 8;
__device__ __forceinline__ void xcd_tile(int& bx, int& by) {
  const int nbx = gridDim.x, n = nbx * gridDim.y;
  const int h = blockIdx.x + nbx * blockIdx.y;
  const int q = n / kXcds, rem = n % kXcds;   // XCDs below rem take q + 1 tiles
  const int x = h % kXcds;
  const int L = x * q + min(x, rem) + h / kXcds;
  by = L / nbx;
  bx = L - by * nbx;
}

// (FP32 with walls and source: stages 2 and 3 would take 258 registers, two more
// than leave room for a second wavefront a SIMD; within 256 one pair of them waits
// in scratch, outside the row loop but for a split side's rows. 2048^2, two steps:
// 1471 -> 1341 us.)
template <class Sys, typename T, int MODE, int VAR>
__global__ __launch_bounds__(64, sizeof(T) == 4 && VAR == (kVarWalls | kVarSource) ? 2 : 1) void stage2d_kernel(StageArgs<T> A, Sys sy) {
  constexpr bool WALLS = (VAR & kVarWalls) != 0;
  constexpr bool IFACE = (VAR & kVarIface) != 0;
  constexpr bool SOURCE = (VAR & kVarSource) != 0 && Sys::kChar && Sys::NC == 4;
  constexpr int NC = Sys::NC;
  const Scheme& s = A.s;
  const int lane = threadIdx.x;
  int bx, by;
  touch_args<StageArgs<T>>();
  xcd_tile(bx, by);
  const StageIn in = stage_read<MODE>(A);
  const int col = bx * kXOut - kHalo + lane;
  const int gcol = map_index(col, A.nx, A.bc[0], A.bc[1]);
  const bool out_col = lane >= kHalo && lane < kWave - kHalo && col < A.nx;
  const bool xm = mirrored(col, A.nx, A.bc[0], A.bc[1]);
  const int xf = fixed_side(col, A.nx, A.bc[0], A.bc[1]);
  const int col0 = bx * kXOut - kHalo;   // the wavefront's first column
  auto special = [](int b) { return b == kBcReflective || b == kBcDirichlet; };
  const bool xwall = (special(A.bc[0]) && col0 < 0) || (special(A.bc[1]) && col0 + kWave > A.nx);
  const int y0 = by * A.rows;
  const int y1 = min(y0 + A.rows, A.ny);
  // FP64: rows y0-2 and y0-1 are taken before the loop, which starts at y0
  // (FP32: at y0-2, which leaves its results as they were, see rounded())
  constexpr bool kAhead = sizeof(T) == 8;
  const int r0 = kAhead ? y0 : y0 - 2;
  // the first rows are in flight while the stage's alphas and dt are formed
  // (a split side's rows depend on the time)
  T Un[NC], Vn[NC], Wn[NC], Up[NC], Vp[NC], Wp[NC];
  int rule_n, rule_p;
  double ax, ay, dt, tstage = 0.0;
  auto first_rows = [&]() {
    load_row<Sys, WALLS>(A, tstage, y0 - 2, col, gcol, Un, Vn, Wn, rule_n);
    if constexpr (kAhead) load_row<Sys, WALLS>(A, tstage, y0 - 1, col, gcol, Up, Vp, Wp, rule_p);
  };
  const bool split = WALLS && (A.bc[2] == kBcSplit || A.bc[3] == kBcSplit);
  if (!split) first_rows();
  if (!stage_begin<MODE>(A, in, bx == 0 && by == 0, ax, ay, dt, tstage)) return;
  if (split) first_rows();
  const T a_y = T(ay);
  // weights of the flux differences (F_{i-1/2} - F_{i+1/2}) of the three
  // equations in the new state, along x and y, and of the modified derivatives
  const double wl = rk_wl<MODE>(dt);
  const double wxu = wl * A.fk.xu, wxv = wl * A.fk.xv, wxw = wl * A.fk.xw;
  const double wyu = wl * A.fk.yu, wyv = wl * A.fk.yv, wyw = wl * A.fk.yw;
  const double wvt = rk_x<MODE>(A.fk.vtx), wwt = rk_x<MODE>(A.fk.vty);

  // Rows march upwards; at iteration r the rows r-2, r-1 and r (just loaded)
  // are present. Iteration r does: the pointwise y-fluxes of
  // row r; the HWENO of row r-1 in y, then in x with the same
  // characteristic basis; the y-interface (r-2)+1/2 and with it the output
  // row r-2; the x-sweep of row r-1, whose flux difference and RK
  // combination wait in LDS (pend) until the next iteration adds the
  // y-part. U, W of rows r-2, r-1 and V of row r-1 stay in registers.
  T Ub[NC], Wb[NC], Vb[NC];
  // U, W of row r-2 and the pointwise g of row r-1: in LDS in FP64 (4 blocks
  // of 40 KB a CU; in registers their moves to AGPRs cost more than the LDS
  // accesses), in registers in FP32 (8 blocks of 20 KB)
  constexpr bool kRowLds = sizeof(T) == 8 && !IFACE && !SOURCE;
  __shared__ T rowl[kRowLds ? 3 : 1][kRowLds ? NC : 1][kWave];
  T rowr[kRowLds ? 1 : 3][kRowLds ? 1 : NC];
  auto prev_row = [&](int f, int c) -> T& {
    if constexpr (kRowLds) return rowl[f][c][lane];
    else return rowr[f][c];
  };
  // pointwise g (FP64: the difference g_k - g_{k-1}), theta, xi of rows k =
  // r-3, r-2, r-1, slot (row mod 3); each lane only touches its own column
  __shared__ T ring[3][3][NC][kWave];
  int slot = (r0 % 3 + 3) % 3;           // slot of row r (and of row r-3)
  // Lax-Friedrichs sums g(u) + a u, theta + a w at the top face of row r-2
  __shared__ T topr[2][NC][kWave];
  // y-interface fluxes of the u-, w- and v-equation at (r-3)+1/2, scaled as
  // interface_flux does (the mixed one times 12)
  __shared__ T fprev[3][NC][kWave];
  // RK combination of row r-2 (u, v, w) without its y flux difference
  __shared__ double pend[3][NC][kWave];
  double smx = 0.0, smy = 0.0;
  unsigned flag = 0;

  T Bu[NC], Bv[NC], Bw[NC];              // RK base of row r-1 (stages 2-3)
  if constexpr (kAhead) {
    // they enter as stencil rows only: their pointwise y-fluxes, both rows'
    // loads in flight together. (512^2: 33.1 -> 30.5 us a stage, 60x240 14.6 ->
    // 11.8, against two iterations of the loop with its unused y-HWENO.)
    finish_row<Sys, WALLS>(A, y0 - 2, xwall, xm, xf, rule_n, Un, Vn, Wn);
    finish_row<Sys, WALLS>(A, y0 - 1, xwall, xm, xf, rule_p, Up, Vp, Wp);
    auto pointwise = [&](int sl, const T (&U)[NC], const T (&V)[NC], const T (&W)[NC], T (&g)[NC]) {
      T th[NC], xi[NC];
      const auto q = prim_rounded(sy, U);
      sy.template flux<1>(U, q, g);
      sy.template jac<1>(U, q, W, th);
      sy.template jac<1>(U, q, V, xi);
      round_all(g);
      round_all(th);
      round_all(xi);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        ring[sl][0][c][lane] = g[c];
        ring[sl][1][c][lane] = th[c];
        ring[sl][2][c][lane] = xi[c];
      }
    };
    const int s2 = slot == 2 ? 0 : slot + 1, s1 = slot == 0 ? 2 : slot - 1;
    T g2[NC], g1[NC];
    pointwise(s2, Un, Vn, Wn, g2);
    pointwise(s1, Up, Vp, Wp, g1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      prev_row(0, c) = Un[c];
      prev_row(1, c) = Wn[c];
      ring[s1][0][c][lane] = g1[c] - g2[c];
      prev_row(2, c) = g1[c];
      Ub[c] = Up[c];
      Vb[c] = Vp[c];
      Wb[c] = Wp[c];
    }
  } else {
    // start from an admissible state
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Ub[c] = T(c == 0 ? 1.0 : (c == NC - 1 ? 2.0 : 0.0));
      Wb[c] = Vb[c] = T(0);
      prev_row(0, c) = Ub[c];
      prev_row(1, c) = prev_row(2, c) = T(0);
    }
  }
  if constexpr (kAhead) load_row<Sys, WALLS>(A, tstage, r0, col, gcol, Un, Vn, Wn, rule_n);
  // The y-work below runs in every iteration, also in the first ones, whose
  // interface and output row are never used (so that it forms one block of
  // straight-line code the compiler can schedule across).
  for (int r = r0; r < y1 + 2; ++r) {
    T Uc[NC], Vc[NC], Wc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) { Uc[c] = Un[c]; Vc[c] = Vn[c]; Wc[c] = Wn[c]; }
    finish_row<Sys, WALLS>(A, r, xwall, xm, xf, rule_n, Uc, Vc, Wc);
    if (r + 1 < y1 + 2) load_row<Sys, WALLS>(A, tstage, r + 1, col, gcol, Un, Vn, Wn, rule_n);  // prefetch
    // RK base of row r, for the x-sweep of the next iteration (rows and
    // columns clamped into the array: the values outside are never used)
    T Bun[NC], Bvn[NC], Bwn[NC];
    if constexpr (MODE >= kStage2) {
      const int rr = min(max(r, 0), A.ny - 1);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned idx = (unsigned)(c * A.plane + rr * A.nx + gcol);
        Bun[c] = ld32(A.Ub, idx);
        Bvn[c] = ld32(A.Vb, idx);
        Bwn[c] = ld32(A.Wb, idx);
      }
    }
    // pointwise g, theta = g'(u) w, xi = g'(u) v of row r
    T gc[NC], tc[NC], xc[NC];
    {
      const auto q = prim_rounded(sy, Uc);
      sy.template flux<1>(Uc, q, gc);
      sy.template jac<1>(Uc, q, Wc, tc);
      sy.template jac<1>(Uc, q, Vc, xc);
      round_all(gc);
      round_all(tc);
      round_all(xc);
    }
    // HWENO in y of row r-1: u at its top and bottom faces, w~, and the LF
    // sums there
    typename Sys::template CellEig<T> ce;
    T mG[NC], mT[NC], pG[NC], pT[NC], wt[NC];
    {
      ce = sy.cell_eig(Ub);
      T uT[NC], uB[NC], wT[NC], wB[NC];
      T Ua[NC], Wa[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        Ua[c] = prev_row(0, c);
        Wa[c] = prev_row(1, c);
        prev_row(0, c) = Ub[c];
        prev_row(1, c) = Wb[c];
      }
      if constexpr (IFACE && sizeof(T) == 4) {
        // mesh width 1 for the scaled derivatives
        hweno_cell_b<1, true>(sy, s, 1.0, 1.0, ce.q, Ua, Ub, Uc, Wa, Wc, uT, uB, wt);
#pragma unroll
        for (int c = 0; c < NC; ++c) face_derivs(Ua[c], Ub[c], Uc[c], Wa[c], Wc[c], T(1), wT[c], wB[c]);
      } else {
        T E1[NC], E2[NC], Sw[NC], Dw[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          E1[c] = Ub[c] - Ua[c];
          E2[c] = Uc[c] - Ub[c];
          Sw[c] = Wa[c] + Wc[c];
          Dw[c] = Wa[c] - Wc[c];
        }
        if constexpr (IFACE)
          hweno_cell_diff_iface<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, Sw, Dw, uT, uB, wt, wT, wB);
        else
          hweno_cell_diff<1>(sy, A.pk, ce, Ub, E1, E2, Sw, Dw, uT, uB, wt, wT, wB);
      }
      T gt[NC], tt[NC], gb[NC], tb[NC];
      const auto qt = prim_rounded(sy, uT);
      sy.template flux<1>(uT, qt, gt);
      sy.template jac<1>(uT, qt, wT, tt);
      const auto qb = prim_rounded(sy, uB);
      sy.template flux<1>(uB, qb, gb);
      sy.template jac<1>(uB, qb, wB, tb);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        mG[c] = fma(a_y, uT[c], gt[c]);
        mT[c] = fma(a_y, wT[c], tt[c]);
        pG[c] = fma(-a_y, uB[c], gb[c]);
        pT[c] = fma(-a_y, wB[c], tb[c]);
      }
    }
    // y-interface (r-2)+1/2: minus side = top face of row r-2, plus side =
    // bottom face of row r-1; central correction from rows r-3..r
    T Gn[NC], Tn[NC], Xn[NC];
    {
      const int s3 = slot, s2 = slot == 2 ? 0 : slot + 1, s1 = slot == 0 ? 2 : slot - 1;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const T t3 = ring[s3][1][c][lane];
        const T x3 = ring[s3][2][c][lane], x2 = ring[s2][2][c][lane], x1 = ring[s1][2][c][lane];
        const T sG = topr[0][c][lane] + pG[c], sT = topr[1][c][lane] + pT[c];
        const T g2 = ring[s2][0][c][lane], g1 = ring[s1][0][c][lane];
        if constexpr (kFluxScaled<T>) {
          const T d0 = gc[c] - prev_row(2, c);
          interface_flux(g2, g1, d0, t3, tc[c], sG, sT, Gn[c], Tn[c]);
          prev_row(2, c) = gc[c];
          gc[c] = d0;
        } else {
          interface_flux_plain(ring[s3][0][c][lane], g2, g1, gc[c], t3, tc[c], sG, sT, Gn[c], Tn[c]);
        }
        Xn[c] = fma(T(7), x2 + x1, -(x3 + xc[c]));
      }
    }
    // row r takes the ring slot of row r-3; row r-1's top-face sums replace
    // row r-2's
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      ring[slot][0][c][lane] = gc[c];
      ring[slot][1][c][lane] = tc[c];
      ring[slot][2][c][lane] = xc[c];
      topr[0][c][lane] = mG[c];
      topr[1][c][lane] = mT[c];
    }
    // output row o = r - 2: the pending combination plus its y flux
    // difference (odeH)/(ode2H), Step 4
    T Unew[NC], Vnew[NC], Wnew[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Unew[c] = (T)fma(wyu, (double)fprev[0][c][lane] - (double)Gn[c], pend[0][c][lane]);
      Vnew[c] = (T)fma(wyv, (double)fprev[2][c][lane] - (double)Xn[c], pend[1][c][lane]);
      Wnew[c] = (T)fma(wyw, (double)fprev[1][c][lane] - (double)Tn[c], pend[2][c][lane]);
      fprev[0][c][lane] = Gn[c];
      fprev[1][c][lane] = Tn[c];
      fprev[2][c][lane] = Xn[c];
    }
    if (r >= y0 + 2 && out_col) {
      const unsigned row = (unsigned)((r - 2) * A.nx + col);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned idx = (unsigned)(c * A.plane) + row;
        st32(A.Uo, idx, Unew[c]);
        st32(A.Vo, idx, Vnew[c]);
        st32(A.Wo, idx, Wnew[c]);
      }
      if (A.next_set >= 0) {
        double sx_, sy_;
        flag |= sy.speeds(Unew, sx_, sy_);
        smx = fmax(smx, sx_);
        smy = fmax(smy, sy_);
      }
    }
    if (r >= y0 + 1 && r <= y1) {
      // x-sweep of row r-1 and its RK combination without the y part.
      // Keep the scheduler from interleaving it with the y-work above:
      // both working sets live at once would spill.
      __builtin_amdgcn_sched_barrier(0);
      double RU[NC], RV[NC], RW[NC];
      T vt[NC];
      sweep_x<3, IFACE>(sy, s, A.pk, ax, ce, Ub, Vb, Wb, RU, RV, RW, vt);
      if (out_col) {
        const unsigned row = (unsigned)((r - 1) * A.nx + col);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const double ub = MODE >= kStage2 ? (double)Bu[c] : 0.0;
          const double vb = MODE >= kStage2 ? (double)Bv[c] : 0.0;
          const double wb = MODE >= kStage2 ? (double)Bw[c] : 0.0;
          double pu = fma(wxu, RU[c], rk_base<MODE>((double)Ub[c], rk_x<MODE>(1.0), ub));
          double pv = fma(wxv, RV[c], rk_base<MODE>((double)vt[c], wvt, vb));
          double pw = fma(wxw, RW[c], rk_base<MODE>((double)wt[c], wwt, wb));
          if constexpr (SOURCE) {
            // S(X) = g (0, 0, X_0, X_2) for X = u, v, w of the stage state
            if (c >= 2) {
              const int k = c == 2 ? 0 : 2;
              const double g = wl * A.gravity;
              pu = fma(g, (double)Ub[k], pu);
              pv = fma(g * A.fk.ilx, (double)Vb[k], pv);
              pw = fma(g * A.fk.ily, (double)Wb[k], pw);
            }
          }
          pend[0][c][lane] = pu;
          pend[1][c][lane] = pv;
          pend[2][c][lane] = pw;
          if (MODE == kStage1 || MODE == kRhs) {
            const unsigned idx = (unsigned)(c * A.plane) + row;
            st32(A.Vt, idx, (T)((double)vt[c] * A.fk.vtx));
            st32(A.Wt, idx, (T)((double)wt[c] * A.fk.vty));
          }
        }
      }
    }
    // rotate the registers
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Ub[c] = Uc[c];
      Wb[c] = Wc[c];
      Vb[c] = Vc[c];
      if (MODE >= kStage2) { Bu[c] = Bun[c]; Bv[c] = Bvn[c]; Bw[c] = Bwn[c]; }
    }
    slot = slot == 2 ? 0 : slot + 1;
  }
  if (A.next_set >= 0) {
    smx = wave_max(smx);
    smy = wave_max(smy);
    flag = wave_or(flag);
    if (lane == 0)
      raise_alphas<2>(A.ctl.sc, A.nslots, A.next_set, blockIdx.x + gridDim.x * blockIdx.y, smx, smy, flag);
  }
}

// Shared-memory barrier of a block: orders LDS accesses only.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The same stage for short strips ("tile"): one wavefront per row. A block of
// H + 2 wavefronts takes H output rows of 60 columns; wavefront w does row
// q = y0 - 1 + w: the y-HWENO and the pointwise y-fluxes of its row go to LDS,
// then, in the H inner wavefronts, the x-sweep; after one barrier each of them
// forms the two y-interfaces of its row from LDS and stores it. The marcher's
// warm-up (two rows of y-work on each side of every strip, one after the other
// in one wavefront) becomes two wavefronts beside the others, so that a strip
// of a few rows takes the time of one row instead of H + 4. The arithmetic of
// every row is the marcher's, so the results are the same bit for bit. It is
// bound by latency: the start, one row's loads (2.6 us) and a row's serial
// arithmetic (3.5 us). FP64 only (in FP32 a row's bits depend on the loop it is
// compiled into, see rounded()). Measured times at the rule (tile_rows).
// MOST: the most output rows of a block, up to kTileFew with two wavefronts a
// SIMD, beyond (and at most kTileRows, which a CU's LDS holds) with three, whose
// smaller share of the registers costs the shorter blocks 0.8-1.0 us a stage.
constexpr int kTileFew = 6, kTileRows = 8;
// LDS of a block: per row y0-2 .. y0+H+1 the pointwise g, theta, xi; per row
// y0-1 .. y0+H the LF sums of its top and bottom face for g and theta
template <int NC, typename T>
constexpr size_t tile_lds(int H) {
  return ((size_t)(H + 4) * 3 + (size_t)(H + 2) * 4) * NC * kWave * sizeof(T);
}

template <class Sys, typename T, int MODE, int VAR, int MOST>
__global__ __launch_bounds__((MOST + 2) * kWave, MOST > kTileFew ? 3 : 2) void stage2d_tile_kernel(StageArgs<T> A, Sys sy) {
  static_assert(sizeof(T) == 8);
  constexpr bool WALLS = (VAR & kVarWalls) != 0;
  constexpr bool IFACE = (VAR & kVarIface) != 0;
  constexpr bool SOURCE = (VAR & kVarSource) != 0 && Sys::kChar && Sys::NC == 4;
  constexpr int NC = Sys::NC;
  constexpr int R = NC * kWave;                    // values of one field of one row
  const Scheme& s = A.s;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int bx, by;
  touch_args<StageArgs<T>>();
  xcd_tile(bx, by);
  const StageIn in = stage_read<MODE>(A);
  const int col0 = bx * kXOut - kHalo;
  const int col = col0 + lane;
  const int gcol = map_index(col, A.nx, A.bc[0], A.bc[1]);
  const bool xm = mirrored(col, A.nx, A.bc[0], A.bc[1]);
  const int xf = fixed_side(col, A.nx, A.bc[0], A.bc[1]);
  auto special = [](int b) { return b == kBcReflective || b == kBcDirichlet; };
  const bool xwall = (special(A.bc[0]) && col0 < 0) || (special(A.bc[1]) && col0 + kWave > A.nx);
  const int y0 = by * A.rows;
  const int H = min(A.rows, A.ny - y0);            // output rows of this block
  const int q = y0 - 1 + wv;
  const bool run = wv < H + 2;                     // (fewer rows in the last strip)
  const bool inner = wv >= 1 && wv <= H;
  const bool out = inner && lane >= kHalo && lane < kWave - kHalo && col < A.nx;
  extern __shared__ __align__(16) char tile_smem[];
  T* const rowsF = (T*)tile_smem;                  // row q is slot wv + 1
  T* const rowsM = rowsF + (A.rows + 4) * 3 * R;   // row q is slot wv: mG, mT, pG, pT

  T Ub[NC], Vb[NC], Wb[NC], wt[NC];
  typename Sys::template CellEig<T> ce;
  T Ua[NC], Va[NC], Wa[NC], Uc[NC], Vc[NC], Wc[NC];
  int ra, rb, rc;
  double ax, ay, dt, tstage = 0.0;
  auto rows = [&]() {                              // (row indices are mapped: any q is safe)
    load_row<Sys, WALLS>(A, tstage, q, col, gcol, Ub, Vb, Wb, rb);
    load_row<Sys, WALLS>(A, tstage, q - 1, col, gcol, Ua, Va, Wa, ra);
    load_row<Sys, WALLS>(A, tstage, q + 1, col, gcol, Uc, Vc, Wc, rc);
  };
  const bool split = WALLS && (A.bc[2] == kBcSplit || A.bc[3] == kBcSplit);
  if (!split) rows();
  if (!stage_begin<MODE>(A, in, bx == 0 && by == 0 && wv == 0, ax, ay, dt, tstage)) return;
  if (split) rows();
  if (run) {
    finish_row<Sys, WALLS>(A, q, xwall, xm, xf, rb, Ub, Vb, Wb);
    finish_row<Sys, WALLS>(A, q - 1, xwall, xm, xf, ra, Ua, Va, Wa);
    finish_row<Sys, WALLS>(A, q + 1, xwall, xm, xf, rc, Uc, Vc, Wc);
    // pointwise g, theta = g'(u) w, xi = g'(u) v of a row, to its slot
    auto pointwise = [&](int slot, const T (&U)[NC], const T (&V)[NC], const T (&W)[NC]) {
      T g[NC], th[NC], xi[NC];
      const auto pr = prim_rounded(sy, U);
      sy.template flux<1>(U, pr, g);
      sy.template jac<1>(U, pr, W, th);
      sy.template jac<1>(U, pr, V, xi);
      round_all(g);
      round_all(th);
      round_all(xi);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        rowsF[(slot * 3 + 0) * R + c * kWave + lane] = g[c];
        rowsF[(slot * 3 + 1) * R + c * kWave + lane] = th[c];
        rowsF[(slot * 3 + 2) * R + c * kWave + lane] = xi[c];
      }
    };
    pointwise(wv + 1, Ub, Vb, Wb);
    if (wv == 0) pointwise(0, Ua, Va, Wa);
    if (wv == H + 1) pointwise(H + 3, Uc, Vc, Wc);
    // HWENO in y of row q: u at its top and bottom faces, w~, the LF sums there
    ce = sy.cell_eig(Ub);
    T uT[NC], uB[NC], wT[NC], wB[NC];
    T E1[NC], E2[NC], Sw[NC], Dw[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      E1[c] = Ub[c] - Ua[c];
      E2[c] = Uc[c] - Ub[c];
      Sw[c] = Wa[c] + Wc[c];
      Dw[c] = Wa[c] - Wc[c];
    }
    if constexpr (IFACE)
      hweno_cell_diff_iface<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, Sw, Dw, uT, uB, wt, wT, wB);
    else
      hweno_cell_diff<1>(sy, A.pk, ce, Ub, E1, E2, Sw, Dw, uT, uB, wt, wT, wB);
    T gt[NC], tt[NC], gb[NC], tb[NC];
    const T a_y = T(ay);
    const auto qt = prim_rounded(sy, uT);
    sy.template flux<1>(uT, qt, gt);
    sy.template jac<1>(uT, qt, wT, tt);
    const auto qb = prim_rounded(sy, uB);
    sy.template flux<1>(uB, qb, gb);
    sy.template jac<1>(uB, qb, wB, tb);
    T* m = rowsM + wv * 4 * R + lane;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      m[c * kWave] = fma(a_y, uT[c], gt[c]);
      m[R + c * kWave] = fma(a_y, wT[c], tt[c]);
      m[2 * R + c * kWave] = fma(-a_y, uB[c], gb[c]);
      m[3 * R + c * kWave] = fma(-a_y, wB[c], tb[c]);
    }
  }
  const double wl = rk_wl<MODE>(dt);
  double PU[NC], PV[NC], PW[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) PU[c] = PV[c] = PW[c] = 0.0;
  if (inner) {
    // x-sweep and the RK combination without the y part; the scheduler must
    // not interleave it with the y-work (both working sets would spill)
    __builtin_amdgcn_sched_barrier(0);
    T Bu[NC], Bv[NC], Bw[NC];
    if constexpr (MODE >= kStage2) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned idx = (unsigned)(c * A.plane + q * A.nx + gcol);
        Bu[c] = ld32(A.Ub, idx);
        Bv[c] = ld32(A.Vb, idx);
        Bw[c] = ld32(A.Wb, idx);
      }
    }
    double RU[NC], RV[NC], RW[NC];
    T vt[NC];
    sweep_x<3, IFACE>(sy, s, A.pk, ax, ce, Ub, Vb, Wb, RU, RV, RW, vt);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double ub = MODE >= kStage2 ? (double)Bu[c] : 0.0;
      const double vb = MODE >= kStage2 ? (double)Bv[c] : 0.0;
      const double wb = MODE >= kStage2 ? (double)Bw[c] : 0.0;
      PU[c] = fma(wl * A.fk.xu, RU[c], rk_base<MODE>((double)Ub[c], rk_x<MODE>(1.0), ub));
      PV[c] = fma(wl * A.fk.xv, RV[c], rk_base<MODE>((double)vt[c], rk_x<MODE>(A.fk.vtx), vb));
      PW[c] = fma(wl * A.fk.xw, RW[c], rk_base<MODE>((double)wt[c], rk_x<MODE>(A.fk.vty), wb));
      if constexpr (SOURCE) {
        // S(X) = g (0, 0, X_0, X_2) for X = u, v, w of the stage state
        if (c >= 2) {
          const int k = c == 2 ? 0 : 2;
          const double g = wl * A.gravity;
          PU[c] = fma(g, (double)Ub[k], PU[c]);
          PV[c] = fma(g * A.fk.ilx, (double)Vb[k], PV[c]);
          PW[c] = fma(g * A.fk.ily, (double)Wb[k], PW[c]);
        }
      }
      if (MODE == kStage1 || MODE == kRhs) {
        const unsigned idx = (unsigned)(c * A.plane + q * A.nx + col);
        if (out) {
          st32(A.Vt, idx, (T)((double)vt[c] * A.fk.vtx));
          st32(A.Wt, idx, (T)((double)wt[c] * A.fk.vty));
        }
      }
    }
  }
  lds_barrier();
  double smx = 0.0, smy = 0.0;
  unsigned flag = 0;
  if (out) {
    // y-interfaces q-1/2 and q+1/2: minus side = top face of the row below,
    // plus side = bottom face of the row above; central correction from two
    // rows on either side
    const double wyu = wl * A.fk.yu, wyv = wl * A.fk.yv, wyw = wl * A.fk.yw;
    T Un[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      auto F = [&](int j, int f) -> T { return rowsF[((wv + 1 + j) * 3 + f) * R + c * kWave + lane]; };
      auto M = [&](int j, int f) -> T { return rowsM[((wv + j) * 4 + f) * R + c * kWave + lane]; };
      T G[2], Tn[2], X[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {                // interface q + k - 1/2
        const T sG = M(k - 1, 0) + M(k, 2), sT = M(k - 1, 1) + M(k, 3);
        const T hm = F(k - 2, 1), hp = F(k + 1, 1);
        const T g0 = F(k - 2, 0), g1 = F(k - 1, 0), g2 = F(k, 0), g3 = F(k + 1, 0);
        interface_flux(g1 - g0, g2 - g1, g3 - g2, hm, hp, sG, sT, G[k], Tn[k]);
        X[k] = fma(T(7), F(k - 1, 2) + F(k, 2), -(F(k - 2, 2) + F(k + 1, 2)));
      }
      const unsigned idx = (unsigned)(c * A.plane + q * A.nx + col);
      Un[c] = (T)fma(wyu, (double)G[0] - (double)G[1], PU[c]);
      st32(A.Uo, idx, Un[c]);
      st32(A.Vo, idx, (T)fma(wyv, (double)X[0] - (double)X[1], PV[c]));
      st32(A.Wo, idx, (T)fma(wyw, (double)Tn[0] - (double)Tn[1], PW[c]));
    }
    if (A.next_set >= 0) flag = sy.speeds(Un, smx, smy);
  }
  if (A.next_set >= 0 && inner) {
    smx = wave_max(smx);
    smy = wave_max(smy);
    flag = wave_or(flag);
    if (lane == 0)
      raise_alphas<2>(A.ctl.sc, A.nslots, A.next_set, (blockIdx.x + gridDim.x * blockIdx.y) * MOST + wv,
                      smx, smy, flag);
  }
}

// -------------------------------------------- wave-speed reduction (flux-LF)
// The maxima of the spectral radius over interior cells, in x and y, into the
// accumulators kSetSeed, for a run's first step (alpha null); also raises the
// state flags. With `alpha` the maxima are the result: the block that is done
// last takes them from the accumulators (leaving zeros) and writes them; nobody
// waits. A block counts itself as done once its atomic maxima have returned, that
// is once they stand where every block's atomics meet; the maxima and the counts
// are only ever accessed by such atomics, so that no cache has to be written back
// or invalidated. The blocks are counted per slot, then the slots. Measured (FP64
// Euler, us a launch, this | with a device-wide fence a block, one count | two
// launches): 128^2 4.3 | 4.3 | 5.3, 385x250 4.4 | 9.5 | 5.5, 512^2 5.0 | 22.0 | 5.3,
// 1000x777 6.1 | 22.5 | 6.0, 2000^2 21.2 | 39.7 | 21.4; the second launch also
// costs 4 us of the host's time.
template <class Sys, typename T, int DIM>
__global__ __launch_bounds__(256) void speed_kernel(const T* U, int plane, Sys sy, StepScalars* sc,
                                                    int nslots, double* alpha) {
  constexpr int NC = Sys::NC;
  double mx = 0.0, my = 0.0;
  unsigned flag = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < plane; i += gridDim.x * blockDim.x) {
    T u[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) u[c] = U[c * plane + i];
    double sx_, sy_;
    flag |= sy.speeds(u, sx_, sy_);
    mx = fmax(mx, sx_);
    if (DIM == 2) my = fmax(my, sy_);
  }
  __shared__ double sx[4], sy_[4];
  __shared__ unsigned sf[4];
  mx = wave_max(mx);
  my = wave_max(my);
  flag = wave_or(flag);
  const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  if (lane == 0) { sx[w] = mx; sy_[w] = my; sf[w] = flag; }
  __syncthreads();
  if (w != 0) return;
  bool last = false;
  if (lane == 0) {
    const int nw = blockDim.x / kWave;
    for (int k = 1; k < nw; ++k) { mx = fmax(mx, sx[k]); my = fmax(my, sy_[k]); flag |= sf[k]; }
    if (!alpha) {
      raise_alphas<DIM>(sc, nslots, kSetSeed, blockIdx.x, mx, my, flag);
    } else {
      const unsigned slot = blockIdx.x % kSlots, nb = gridDim.x;
      unsigned long long* p = alpha_slots(sc)->v[slot][kSetSeed];
      SpeedTickets* done = speed_tickets(sc);
      const unsigned long long ox = atomic_max_pos(p, mx), oy = DIM == 2 ? atomic_max_pos(p + 1, my) : 0ull;
      if (flag) atomicOr(&sc->flags, flag);
      // the old values are here: both maxima stand (nothing moves above this)
      asm volatile("s_waitcnt vmcnt(0)" ::"v"((unsigned)ox), "v"((unsigned)oy) : "memory");
      if (atomicAdd(&done->slot[slot][0], 1u) == (nb - slot + kSlots - 1) / kSlots - 1) {
        asm volatile("" ::: "memory");
        last = atomicAdd(&done->slots, 1u) == (nb < kSlots ? nb : kSlots) - 1;
      }
    }
  }
  if (!__any(last)) return;
  double x = 0.0, y = 0.0;
  if (lane < kSlots) {
    unsigned long long* p = alpha_slots(sc)->v[lane][kSetSeed];
    x = __longlong_as_double((long long)atomicExch(p, 0ull));
    if (DIM == 2) y = __longlong_as_double((long long)atomicExch(p + 1, 0ull));
    atomicExch(&speed_tickets(sc)->slot[lane][0], 0u);
  }
  x = wave_max(x);
  y = wave_max(y);
  if (lane == 0) {
    alpha[0] = x;
    alpha[1] = y;
    atomicExch(&speed_tickets(sc)->slots, 0u);
  }
}

__device__ __forceinline__ void clear_alphas(StepScalars* sc) {
  const int lane = threadIdx.x;
  if (lane < kSlots)
    for (int k = 0; k < kSets; ++k) alpha_slots(sc)->v[lane][k][0] = alpha_slots(sc)->v[lane][k][1] = 0ull;
}
// After a step that returns an error between its launches: the maxima that its
// later stages would have cleared (the sticky flags stay).
__global__ __launch_bounds__(kWave) void alpha_clear_kernel(StepScalars* sc) { clear_alphas(sc); }
__global__ __launch_bounds__(kWave) void ws_init_kernel(StepScalars* sc) {
  clear_alphas(sc);
  if (threadIdx.x < kSlots) speed_tickets(sc)->slot[threadIdx.x][0] = 0u;
  if (threadIdx.x != 0) return;
  sc->dt = sc->t0 = sc->tnew = 0.0;
  sc->active = 0;
  sc->flags = 0u;
  speed_tickets(sc)->slots = 0u;
}

// ================================================================ adjoint
// Vector-Jacobian product of one stage for the x direction, on lines laid
// out along memory rows (1D, or each row of a 2D field). Given the
// state X = (u, a, o) -- a the derivative along the line, o the other one --
// and cotangents a_B of B(X) = (u, a~, ...) and b of L(X), it writes
//   G = (dB/dX)^T a_B + (dL_dir/dX)^T b
// restricted to this direction's terms (in 2D it adds that to G, which
// holds the y-direction terms). Lanes hold "virtual" cells (ghost cells
// included). Along a periodic line these are images of cells like any other,
// and the cells [0, n) are the output; otherwise [-2, n+2) is, every cell an
// output lane of exactly one block, and what a ghost cell receives goes to the
// cell it is an image of (the transpose of the ghost index map) within the
// wavefront: the blocks divide the line evenly, so that a ghost cell and its
// image, at most two cells from the line's end, share one.
//
// The along-derivative is carried multiplied by lam h as in the stage kernels
// (Carried), the cotangents with the inverse factors, which leaves no mesh
// constant in the arithmetic; the scales are part of VjpScales. Bound by the
// number of instructions and, the wavefronts of a SIMD starting together, by the
// latency of the loads at each start; the difference form and its recomputed
// interpolation (hweno_adjoint_diff.h) leave room for two wavefronts a SIMD.
// FP64 2D Euler at 512^2, one a set: 44.7 -> 32.1 us a launch (three: 46.4 ->
// 34.1), and the 5.5 us of a second kernel that added the ghost columns' terms
// are gone.
struct VjpScales {
  double lamh;            // lam h: of the carried derivative
  double u, a, o;         // of the cotangent b (u, along, other), over dt
  double vt;              // of the modified derivative (FluxK::vtx)
};
template <typename T>
VjpScales vjp_scales(const Scheme& s, double h, double cb) {
  const double lam = Carried<T>::lam, mu = Carried<T>::mu;
  VjpScales k;
  k.lamh = lam * h;
  k.u = 0.5 * cb / h;                    // the two halves of the LF flux
  k.a = 0.5 * cb / (h * (mu * lam * h));
  k.o = cb / (12.0 * h);                 // (mixed)
  k.vt = point_vt_scale<T>(s) / h;
  return k;
}
template <typename T>
struct VjpArgs {
  const T* X[3];          // u, along-derivative, other derivative (null in 1D)
  const T* b[3];          // b = cb dt lam_b: the one cotangent state L sees
  const T* a[3][2];       // a_B = sum_k ca_k lam_k (u and along fields)
  double ca[3];
  const double* dt;
  const double* alpha;    // [2]; this pass uses alpha[0]
  int accumulate;         // 2D: add the result and the y-pass's folds to G (else overwrite G)
  T* G[3];                // outputs (u, along, other)
  // with accumulate: the y-pass's strip halos [strip][2 sides][u, w][NC][n]
  // and ghost rows [4][3][NC][n], its strip height and count, the y sides
  // ghost row k (-2, -1, ny, ny+1): the row it folds into (-1: none), whether
  // the wall's sign rules apply, the strip (-1: none) and side of the halo
  // term aimed at it
  const T* yhalo;
  const T* yghost;
  int yR, ystrips;
  int yimg[4], yflip[4], yqj[4], yqs[4];
  int n, rows, plane;
  int bc_lo, bc_hi;
  double gs[2][4];        // fixed ghost states of the low and high side
  VjpScales sc;
  PointK pk;
};

// The y-pass strip whose halo term is aimed at virtual row q: strip j (rows
// [-2 + jR, -2 + (j+1)R)) sends side 0 to its row o0 - 1 and side 1 to its
// row o1. Returns j (side in `side`), or -1.
HWENO_HD int halo_source(int q, int R, int nstrips, int& side) {
  if ((q + 3) % R == 0) {
    const int j = (q + 3) / R;
    if (j >= 1 && j <= nstrips - 1) {
      side = 0;
      return j;
    }
  }
  if ((q + 2) % R == 0) {
    const int j = (q + 2) / R - 1;
    if (j >= 0 && j <= nstrips - 2) {
      side = 1;
      return j;
    }
  }
  return -1;
}

// Cotangents of the pointwise fluxes of a cell from those of the interfaces
// i-3/2 .. i+3/2 (F: of the flux, halved, H: of the along-derivative flux,
// halved and scaled, E: of the mixed one, over 12): the transpose of the central
// correction (Cd-1)-(DfDh) and of (mixed).
template <typename T>
__device__ __forceinline__ void point_cotangents(T F1, T F0, T Fm1, T Fm2, T H1, T H0, T Hm1, T Hm2,
                                                 T& gf, T& gh) {
  constexpr double lam = Carried<T>::lam, mu = Carried<T>::mu;
  const T s = (F0 + Fm1) - (F1 + Fm2);
  gf = fma(T(97.0 / 960.0), s,
           fma(T(2.0 * mu * lam * 697.0 / 5184.0), H1 - Hm2, T(2.0 * mu * lam * 61.0 / 192.0) * (Hm1 - H0)));
  gh = fma(T(2.0 * 19.0 / (960.0 * lam)), Fm2 - F1, T(2.0 * mu * 37.0 / 864.0) * (H1 + Hm2));
}
template <typename T>
__device__ __forceinline__ T point_cotangent_mixed(T E1, T E0, T Em1, T Em2) {
  return fma(T(7), E0 + Em1, -(E1 + Em2));
}
// Reverse of one side of the LF flux at a face: f(u) + a u, f'(u) v + a v with
// cotangents gF, gH (a of either sign) -> those of u and v.
template <int D, class Sys, typename T>
__device__ __forceinline__ void face_vjp(const Sys& sy, T a, const T (&u)[Sys::NC],
                                         const T (&v)[Sys::NC], const T (&gF)[Sys::NC],
                                         const T (&gH)[Sys::NC], T (&gu)[Sys::NC], T (&gv)[Sys::NC]) {
#pragma unroll
  for (int c = 0; c < Sys::NC; ++c) {
    gu[c] = a * gF[c];
    gv[c] = a * gH[c];
  }
  const auto q = sy.prim(u);
  typename StateBarOf<Sys, T>::type b{};
  flux_vjp<D>(sy, u, q, gF, b, gu);
  jac_vjp<D>(sy, u, q, v, gH, b, gu, gv);
  prim_vjp(sy, u, q, b, gu);
}

template <class Sys, typename T, int NF, int NA, bool WALLS, bool IFACE = false>
__global__ __launch_bounds__(64, IFACE ? 1 : 2) void vjp_row_kernel(VjpArgs<T> A, Sys sy) {
  // WALLS: some side of this direction is reflective or fixed
  constexpr int NC = Sys::NC;
  touch_args<VjpArgs<T>>();
  const int lane = threadIdx.x;
  int bx, row;
  xcd_tile(bx, row);
  const bool periodic = A.bc_lo == kBcPeriodic;
  const int lo = periodic ? 0 : -2, total = periodic ? A.n : A.n + 4;
  const int nb = gridDim.x, wq = total / nb, wr = total % nb;
  const int start = lo + bx * wq + min(bx, wr), end = start + wq + (bx < wr ? 1 : 0);
  const int col0 = start - kHalo;
  const int v = col0 + lane;
  const int g = map_index(v, A.n, A.bc_lo, A.bc_hi);
  const bool interior = v >= 0 && v < A.n;
  const bool out = lane >= kHalo && v < end;
  const int base = row * A.n;
  const double dtv = A.dt ? *A.dt : 0.0;
  const T alpha = T(A.alpha[0]);

  // with A.accumulate, the values this pass adds to, and the y-pass halo
  // term aimed at this row (u, w), copied into LDS while the lane works
  __shared__ T gin[NF][NC][kWave];
  __shared__ T yh[2][NC][kWave];
  __shared__ T fold[4][3][NC];   // what the ghost cells -2, -1, n, n+1 received
  const RowCopy<T> copy(col0, A.n, lane);
  int hside = 0;
  const int hj = A.accumulate ? halo_source(row, A.yR, A.ystrips, hside) : -1;
  if (A.accumulate) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int f = 0; f < NF; ++f)
        copy(A.G[f], (unsigned)(c * A.plane + base), &gin[f][c][0]);
    if (hj >= 0) {
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int c = 0; c < NC; ++c)
          copy(A.yhalo, (unsigned)(((hj * 4 + hside * 2 + hf) * NC + c) * A.n), &yh[hf][c][0]);
    }
  }
  T U[NC], Av[NC], Ov[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const unsigned i = (unsigned)(c * A.plane + base + g);
    U[c] = ld32(A.X[0], i);
    Av[c] = T(A.sc.lamh) * ld32(A.X[1], i);
    Ov[c] = NF == 3 ? ld32(A.X[2], i) : T(0);
  }
  // cotangents; zero at ghost cells that are no images (L and B are defined on
  // interior cells)
  T aU[NC], aA[NC], bU[NC], bA[NC], bO[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) { aU[c] = T(0); aA[c] = T(0); bU[c] = T(0); bA[c] = T(0); bO[c] = T(0); }
  if (interior || periodic) {
    const T su = T(A.sc.u * dtv), sa = T(A.sc.a * dtv), so = T(A.sc.o * dtv);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const unsigned idx = (unsigned)(c * A.plane + base + g);
      bU[c] = su * ld32(A.b[0], idx);
      bA[c] = sa * ld32(A.b[1], idx);
      if (NF == 3) bO[c] = so * ld32(A.b[2], idx);
#pragma unroll
      for (int k = 0; k < NA; ++k) {
        aU[c] += T(A.ca[k]) * ld32(A.a[k][0], idx);
        aA[c] += T(A.ca[k] * A.sc.vt) * ld32(A.a[k][1], idx);
      }
    }
  }
  if constexpr (WALLS) {
    const bool m = mirrored(v, A.n, A.bc_lo, A.bc_hi);
    mirror_state<Sys, 0>(m, U);
    mirror_normal_derivative<Sys, 0>(m, Av);
    mirror_state<Sys, 0>(m, Ov);
    const int fs = fixed_side(v, A.n, A.bc_lo, A.bc_hi);
    if (fs >= 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        U[c] = T(A.gs[fs][c]);
        Av[c] = T(0);
        Ov[c] = T(0);
      }
    }
  }
  // ---- interface cotangents: L_i = -(F_{i+1/2} - F_{i-1/2}) / h
  T lF[NC], lH[NC], lE[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    lF[c] = from_next(bU[c]) - bU[c];
    lH[c] = from_next(bA[c]) - bA[c];
    lE[c] = NF == 3 ? from_next(bO[c]) - bO[c] : T(0);
  }
  // ---- the pointwise fluxes f, f'(u) a, f'(u) o of the cell: gather from the
  // interfaces v-3/2 .. v+3/2
  T gU[NC], gA[NC], gO[NC], pF[NC], pH[NC];
  const auto ce = sy.cell_eig(U);
  typename StateBarOf<Sys, T>::type sb{};
  {
    T gf[NC], gh[NC], ge[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      pF[c] = from_prev(lF[c]);
      pH[c] = from_prev(lH[c]);
      point_cotangents(from_next(lF[c]), lF[c], pF[c], from_prev(pF[c]), from_next(lH[c]), lH[c],
                       pH[c], from_prev(pH[c]), gf[c], gh[c]);
      ge[c] = T(0);
      if constexpr (NF == 3) {
        const T Em1 = from_prev(lE[c]);
        ge[c] = point_cotangent_mixed(from_next(lE[c]), lE[c], Em1, from_prev(Em1));
      }
      gU[c] = aU[c];
      gA[c] = T(0);
      gO[c] = T(0);
    }
    flux_vjp<0>(sy, U, ce.q, gf, sb, gU);
    jac_vjp<0>(sy, U, ce.q, Av, gh, sb, gU, gA);
    if constexpr (NF == 3) jac_vjp<0>(sy, U, ce.q, Ov, ge, sb, gU, gO);
  }
  // ---- this cell's face values, the LF halves (minus side of x_{v+1/2}, plus
  // side of x_{v-1/2}) and the reverse of its HWENO and face derivatives
  {
    T E1[NC], E2[NC], S[NC], Dd[NC];
    T Um[NC], Up[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Um[c] = from_prev(U[c]);
      Up[c] = from_next(U[c]);
      const T Am = from_prev(Av[c]), Ap = from_next(Av[c]);
      E1[c] = U[c] - Um[c];
      E2[c] = Up[c] - U[c];
      S[c] = Am + Ap;
      Dd[c] = Am - Ap;
    }
    T guR[NC], guL[NC], g1[NC], g2[NC], gS[NC], gD[NC];
    {
      T uR[NC], uL[NC], at[NC], vR[NC], vL[NC], gvR[NC], gvL[NC];
      if constexpr (IFACE)
        hweno_cell_diff_iface<0>(sy, A.pk, ce, Um, U, Up, E1, E2, S, Dd, uR, uL, at, vR, vL);
      else
        hweno_cell_diff<0>(sy, A.pk, ce, U, E1, E2, S, Dd, uR, uL, at, vR, vL);
      face_vjp<0>(sy, alpha, uR, vR, lF, lH, guR, gvR);
      face_vjp<0>(sy, -alpha, uL, vL, pF, pH, guL, gvL);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        face_derivs_diff_vjp(gvR[c], gvL[c], g1[c], g2[c], gS[c], gD[c]);
    }
    T tm[NC], tp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) tm[c] = tp[c] = T(0);
    if constexpr (IFACE && Sys::kChar)
      hweno_cell_diff_iface_vjp<0>(sy, A.pk, ce, Um, U, Up, E1, E2, S, Dd, guR, guL, aA, g1, g2, gS, gD,
                                   tm, gU, tp, sb);
    else
      hweno_cell_diff_vjp<0>(sy, A.pk, ce, E1, E2, S, Dd, guR, guL, aA, g1, g2, gS, gD, sb);
    cell_state_vjp(sy, U, ce, sb, gU);
    // gather: own + right-neighbour part of the left lane + left part of the right lane
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      tm[c] -= g1[c];
      tp[c] += g2[c];
      gU[c] += ((guR[c] + guL[c]) + (g1[c] - g2[c])) + (from_prev(tp[c]) + from_next(tm[c]));
      gA[c] += from_prev(gS[c] - gD[c]) + from_next(gS[c] + gD[c]);
      gA[c] *= T(A.sc.lamh);
    }
  }
  if (!periodic && (start < 0 || end > A.n)) {
    auto ghost_cell = [&](int k) { return k < 2 ? k - 2 : A.n + k - 2; };
    if (out && !interior) {
      const int k = v < 0 ? v + 2 : v - A.n + 2;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        fold[k][0][c] = gU[c];
        fold[k][1][c] = gA[c];
        if (NF == 3) fold[k][2][c] = gO[c];
      }
    }
    wait_lds_reads();
    if (out && interior) {
      for (int k = 0; k < 4; ++k) {
        const int w = ghost_cell(k);
        if (w < start || w >= end || fixed_side(w, A.n, A.bc_lo, A.bc_hi) >= 0) continue;
        if (map_index(w, A.n, A.bc_lo, A.bc_hi) != v) continue;
        const bool mir = mirrored(w, A.n, A.bc_lo, A.bc_hi);
        auto add = [&](int f, T (&G)[NC]) {
#pragma unroll
          for (int c = 0; c < NC; ++c) G[c] += mir && mirror_flips(0, f, c) ? -fold[k][f][c] : fold[k][f][c];
        };
        add(0, gU);
        add(1, gA);
        if (NF == 3) add(2, gO);
      }
    }
  }
  unsigned gmask = 0;   // y ghost rows folding into this row
  if (A.accumulate) {
    wait_copies();
#pragma unroll
    for (int k = 0; k < 4; ++k) gmask |= A.yimg[k] == row ? 1u << k : 0u;
  }
  if (out && interior) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const unsigned idx = (unsigned)(c * A.plane + base + v);
      if (A.accumulate) {
        gU[c] += gin[0][c][lane];
        gA[c] += gin[1][c][lane];
        if (NF == 3) gO[c] += gin[NF - 1][c][lane];
        if (hj >= 0) {
          gU[c] += yh[0][c][lane];
          if (NF == 3) gO[c] += yh[1][c][lane];
        }
        // the y ghost rows whose image is this row (edge rows only), each
        // with the halo term aimed at it, with the y walls' sign rules
        if (gmask) {
#pragma unroll 1
          for (int k = 0; k < 4; ++k) {
            if (!((gmask >> k) & 1u)) continue;
            const int qj = A.yqj[k], qs = A.yqs[k];
            T gv[3];
#pragma unroll
            for (int f = 0; f < 3; ++f) {
              gv[f] = A.yghost[((size_t)(k * 3 + f) * NC + c) * A.n + v];
              if (qj >= 0 && f != 1)
                gv[f] += A.yhalo[((size_t)(qj * 4 + qs * 2 + (f == 0 ? 0 : 1)) * NC + c) * A.n + v];
              if (A.yflip[k] && mirror_flips(1, f, c)) gv[f] = -gv[f];
            }
            gU[c] += gv[0];
            gA[c] += gv[1];
            if (NF == 3) gO[c] += gv[2];
          }
        }
      }
      st32(A.G[0], idx, gU[c]);
      st32(A.G[1], idx, gA[c]);
      if (NF == 3) st32(A.G[2], idx, gO[c]);
    }
  }
}

// y-direction VJP by marching up strips of rows (2D; natural layout, no
// transposes). Each lane owns one column and needs no neighbour lane. Strip k
// owns the virtual rows [o0, o1) of [-2, ny+2) and reverses the HWENO of its
// own cells only: the contributions of cell o0 to row o0-1 and of cell o1-1
// to row o1 go to a halo buffer, and the x-pass (vjp_row_kernel) adds them,
// and the ghost rows kept in a side buffer, to the rows they belong to. At iteration r (row r
// loaded): the interface cotangents of (r-1)+1/2, the reverse of cell r-1's
// HWENO and face values if the strip owns it (contributions to rows r-2..r),
// and the reverse of row r-2's pointwise fluxes; row r-2 is then complete up
// to the halo terms and is stored to G (the x-pass, which runs next, adds
// its own result). The next row's inputs are copied into LDS while a row is
// computed, so a row's loads wait on memory only once per strip.
// Bound by the number of instructions (an iteration of the FP64 Euler kernel:
// 1855 VALU instructions, with the term-by-term reverse 2770): 512^2 49.5 -> 38.7
// us a launch.
template <typename T>
struct VjpYArgs {
  const T* X[3];          // u, v, w
  const T* b[3];          // b = cb dt lam_b (u, v, w)
  const T* aw[3];         // w fields of the a sets: a_w = sum_k ca_k lam_k,w
  double ca[3];
  int na;                 // number of a sets (1 or 3)
  const double* dt;
  const double* alpha;    // [2]; uses alpha[1]
  T* G[3];                // out (overwritten): u, v, w
  T* ghost;               // [4][3][NC][nx]: rows -2, -1, ny, ny+1
  T* halo;                // [strip][2: to row o0-1, to row o1][2: u, w][NC][nx]
  int nx, ny, rows, plane;
  int bc_lo, bc_hi;
  double gs[2][4];        // fixed ghost states of the low and high side (y)
  VjpScales sc;           // along y
  PointK pk;
};

template <class Sys, typename T, bool WALLS, bool IFACE = false>
__global__ __launch_bounds__(64) void vjp_y_kernel(VjpYArgs<T> A, Sys sy) {
  constexpr int NC = Sys::NC;
  touch_args<VjpYArgs<T>>();
  const int lane = threadIdx.x;
  const int x = blockIdx.x * kWave + lane;
  const bool colok = x < A.nx;
  const int o0 = -2 + blockIdx.y * A.rows;
  const int o1 = min(o0 + A.rows, A.ny + 2);
  const double dtv = A.dt ? *A.dt : 0.0;
  const T alpha = T(A.alpha[1]);
  const T su = T(A.sc.u * dtv), sv = T(A.sc.o * dtv), sw = T(A.sc.a * dtv), lamh = T(A.sc.lamh);
  // interface cotangents (G, theta, xi) of the 3 previous interfaces, slot k mod 3
  __shared__ T lring[3][3][NC][kWave];
  // the next row's inputs, copied in while the current row is computed:
  // u, v, w, b_u, b_v, b_w, then the a_w sets
  __shared__ T stage[9][NC][kWave];
  const RowCopy<T> copy(blockIdx.x * kWave, A.nx, lane);
  // (v of row rr - 2 and the a_w of row rr - 1, which is when they are used)
  auto fetch = [&](int rr) {
    const int g = map_index(rr, A.ny, A.bc_lo, A.bc_hi);
    const int g2 = map_index(rr - 2, A.ny, A.bc_lo, A.bc_hi);
    const bool in = rr >= 0 && rr < A.ny, in1 = rr >= 1 && rr <= A.ny;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const unsigned off = (unsigned)(c * A.plane + g * A.nx);
      copy(A.X[0], off, &stage[0][c][0]);
      copy(A.X[1], (unsigned)(c * A.plane + g2 * A.nx), &stage[1][c][0]);
      copy(A.X[2], off, &stage[2][c][0]);
      if (in) {
#pragma unroll
        for (int f = 0; f < 3; ++f) copy(A.b[f], off, &stage[3 + f][c][0]);
      }
    }
    if (in1) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < A.na) {
#pragma unroll
          for (int c = 0; c < NC; ++c)
            copy(A.aw[k], (unsigned)(c * A.plane + (rr - 1) * A.nx), &stage[6 + k][c][0]);
        }
    }
  };
  T Ua[NC], Ub[NC], Wa[NC], Wb[NC];      // rows r-2, r-1
  T bU1[NC], bV1[NC], bW1[NC];           // cotangents of row r-1
  T accUa[NC], accWa[NC], accUb[NC], accWb[NC];      // HWENO-reverse sums of rows r-2, r-1
#pragma unroll
  for (int c = 0; c < NC; ++c) { accUa[c] = T(0); accWa[c] = T(0); accUb[c] = T(0); accWb[c] = T(0); }
  fetch(o0 - 2);
  for (int r = o0 - 2; r < o1 + 2; ++r) {
    const bool inrow = r >= 0 && r < A.ny, inrow1 = r >= 1 && r <= A.ny;
    wait_copies();
    T Uc[NC], Va[NC], Wc[NC], bUc[NC], bVc[NC], bWc[NC], aW1[NC];   // v of row r-2, a_w of row r-1
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Uc[c] = stage[0][c][lane];
      Va[c] = stage[1][c][lane];
      Wc[c] = lamh * stage[2][c][lane];
      bUc[c] = T(0); bVc[c] = T(0); bWc[c] = T(0); aW1[c] = T(0);
      if (inrow) {
        bUc[c] = su * stage[3][c][lane];
        bVc[c] = sv * stage[4][c][lane];
        bWc[c] = sw * stage[5][c][lane];
      }
    }
    if (inrow1) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < A.na) {
          const T ca = T(A.ca[k] * A.sc.vt);
#pragma unroll
          for (int c = 0; c < NC; ++c) aW1[c] += ca * stage[6 + k][c][lane];
        }
    }
    wait_lds_reads();
    if (r + 1 < o1 + 2) fetch(r + 1);
    if constexpr (WALLS) {
      if (mirrored(r, A.ny, A.bc_lo, A.bc_hi)) {
        mirror_state<Sys, 1>(true, Uc);
        mirror_normal_derivative<Sys, 1>(true, Wc);
      }
      if (mirrored(r - 2, A.ny, A.bc_lo, A.bc_hi)) mirror_state<Sys, 1>(true, Va);
      const int fs = fixed_side(r, A.ny, A.bc_lo, A.bc_hi);
      if (fs >= 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          Uc[c] = T(A.gs[fs][c]);
          Wc[c] = T(0);
        }
      }
      if (fixed_side(r - 2, A.ny, A.bc_lo, A.bc_hi) >= 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) Va[c] = T(0);
      }
    }
    // interface (r-1)+1/2: L_j = -(F_{j+1/2} - F_{j-1/2}) / dy
    T lG[NC], lT[NC], lX[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lG[c] = bUc[c] - bU1[c];
      lT[c] = bWc[c] - bW1[c];
      lX[c] = bVc[c] - bV1[c];
    }
    const int s1 = ((r - 1) % 3 + 3) % 3;        // slot of interface r-1 (and r-4)
    const int s2 = s1 == 0 ? 2 : s1 - 1;          // interface r-2
    const int s3 = s2 == 0 ? 2 : s2 - 1;          // interface r-3
    T accUc[NC], accWc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) { accUc[c] = T(0); accWc[c] = T(0); }
    if (r >= o0 + 1 && r <= o1) {
      // reverse of cell r-1's faces: top face -> interface (r-1)+1/2 (minus
      // side), bottom face -> interface (r-2)+1/2 (plus side)
      const auto ce = sy.cell_eig(Ub);
      typename StateBarOf<Sys, T>::type sb{};
      T E1[NC], E2[NC], S[NC], Dd[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        E1[c] = Ub[c] - Ua[c];
        E2[c] = Uc[c] - Ub[c];
        S[c] = Wa[c] + Wc[c];
        Dd[c] = Wa[c] - Wc[c];
      }
      T guT[NC], guB[NC], g1[NC], g2[NC], gS[NC], gD[NC];
      {
        T uT[NC], uB[NC], wt_[NC], wT[NC], wB[NC], gwT[NC], gwB[NC], pG[NC], pT[NC];
        if constexpr (IFACE)
          hweno_cell_diff_iface<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, S, Dd, uT, uB, wt_, wT, wB);
        else
          hweno_cell_diff<1>(sy, A.pk, ce, Ub, E1, E2, S, Dd, uT, uB, wt_, wT, wB);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          pG[c] = lring[s2][0][c][lane];
          pT[c] = lring[s2][1][c][lane];
        }
        face_vjp<1>(sy, alpha, uT, wT, lG, lT, guT, gwT);
        face_vjp<1>(sy, -alpha, uB, wB, pG, pT, guB, gwB);
#pragma unroll
        for (int c = 0; c < NC; ++c)
          face_derivs_diff_vjp(gwT[c], gwB[c], g1[c], g2[c], gS[c], gD[c]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (IFACE && Sys::kChar)
        hweno_cell_diff_iface_vjp<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, S, Dd, guT, guB, aW1, g1, g2, gS,
                                     gD, accUa, accUb, accUc, sb);
      else
        hweno_cell_diff_vjp<1>(sy, A.pk, ce, E1, E2, S, Dd, guT, guB, aW1, g1, g2, gS, gD, sb);
      cell_state_vjp(sy, Ub, ce, sb, accUb);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        accUa[c] -= g1[c];
        accUb[c] += (guT[c] + guB[c]) + (g1[c] - g2[c]);
        accUc[c] += g2[c];
        accWa[c] += gS[c] + gD[c];
        accWc[c] += gS[c] - gD[c];
      }
    }
    if (r == o0 + 1 && colok) {
      // row r-2 = o0-1 belongs to the strip below: its sums (from cell o0
      // alone) leave through the halo buffer
      T* hb = A.halo + (size_t)blockIdx.y * 4 * NC * A.nx + x;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        hb[(0 * NC + c) * A.nx] = accUa[c];
        hb[(1 * NC + c) * A.nx] = lamh * accWa[c];
      }
    }
    if (r >= o0 + 2) {
      // reverse of row r-2's pointwise g, theta, xi (interfaces r-4..r-1)
      const int o = r - 2;
      T gg[NC], gt[NC], gx[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const T G1 = lG[c], G0 = lring[s2][0][c][lane], Gm1 = lring[s3][0][c][lane], Gm2 = lring[s1][0][c][lane];
        const T T1 = lT[c], T0 = lring[s2][1][c][lane], Tm1 = lring[s3][1][c][lane], Tm2 = lring[s1][1][c][lane];
        const T X1 = lX[c], X0 = lring[s2][2][c][lane], Xm1 = lring[s3][2][c][lane], Xm2 = lring[s1][2][c][lane];
        point_cotangents(G1, G0, Gm1, Gm2, T1, T0, Tm1, Tm2, gg[c], gt[c]);
        gx[c] = point_cotangent_mixed(X1, X0, Xm1, Xm2);
      }
      T gU[NC], gV[NC], gW[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) { gU[c] = accUa[c]; gW[c] = accWa[c]; gV[c] = T(0); }
      const auto q = sy.prim(Ua);
      typename StateBarOf<Sys, T>::type bq{};
      flux_vjp<1>(sy, Ua, q, gg, bq, gU);
      jac_vjp<1>(sy, Ua, q, Wa, gt, bq, gU, gW);
      jac_vjp<1>(sy, Ua, q, Va, gx, bq, gU, gV);
      prim_vjp(sy, Ua, q, bq, gU);
#pragma unroll
      for (int c = 0; c < NC; ++c) gW[c] *= lamh;
      if (colok) {
        if (o >= 0 && o < A.ny) {
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const unsigned idx = (unsigned)(c * A.plane + o * A.nx + x);
            st32(A.G[0], idx, gU[c]);
            st32(A.G[1], idx, gV[c]);
            st32(A.G[2], idx, gW[c]);
          }
        } else {
          const int slot = o < 0 ? o + 2 : o - A.ny + 2;
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            T* gp = A.ghost + ((size_t)slot * 3 * NC) * A.nx + x;
            gp[(0 * NC + c) * A.nx] = gU[c];
            gp[(1 * NC + c) * A.nx] = gV[c];
            gp[(2 * NC + c) * A.nx] = gW[c];
          }
        }
      }
    }
    // interface (r-1)+1/2 replaces (r-4)+1/2; rotate rows
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lring[s1][0][c][lane] = lG[c];
      lring[s1][1][c][lane] = lT[c];
      lring[s1][2][c][lane] = lX[c];
      Ua[c] = Ub[c]; Ub[c] = Uc[c];
      Wa[c] = Wb[c]; Wb[c] = Wc[c];
      bU1[c] = bUc[c]; bV1[c] = bVc[c]; bW1[c] = bWc[c];
      accUa[c] = accUb[c]; accWa[c] = accWb[c];
      accUb[c] = accUc[c]; accWb[c] = accWc[c];
    }
  }
  // row o1 belongs to the strip above: its sums (from cell o1-1 alone) leave
  // through the halo buffer
  if (colok) {
    T* hb = A.halo + (size_t)blockIdx.y * 4 * NC * A.nx + x;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      hb[(2 * NC + c) * A.nx] = accUa[c];
      hb[(3 * NC + c) * A.nx] = lamh * accWa[c];
    }
  }
}

// The same for small grids: one wavefront per row, as in the stage's tile kernel.
// A block of H + 2 wavefronts takes the H virtual rows [o0, o0 + H); wavefront w
// reverses the HWENO of row q = o0 - 1 + w and, in the inner ones, the pointwise
// fluxes of the row. The scaled cotangents b of the rows meet in LDS before,
// what the cells add to the rows below and above them after the work. A row's
// sums are complete within the block: no halo terms. Bound by latency (the start,
// the loads, one row's serial arithmetic) in place of the marcher's H + 4 rows
// one after the other; measured at the rule (tile_rows). Two wavefronts a SIMD at
// six rows leave 256 registers: FP64 Euler waits with 32 B a lane in scratch, in
// the interface basis with 500 B (the marcher, with 512 registers, 0 and 52 B).
constexpr int kVjpTileRows = 6;
constexpr int kVjpTileThreads = (kVjpTileRows + 2) * kWave;
template <int NC, typename T>
constexpr size_t vjp_tile_lds(int H) {
  return ((size_t)(H + 4) * 3 + (size_t)(H + 2) * 4) * NC * kWave * sizeof(T);
}
template <class Sys, typename T, bool WALLS, bool IFACE = false>
__global__ __launch_bounds__(kVjpTileThreads, 2) void vjp_y_tile_kernel(VjpYArgs<T> A, Sys sy) {
  constexpr int NC = Sys::NC;
  constexpr int R = NC * kWave;                    // values of one field of one row
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int bx, by;
  touch_args<VjpYArgs<T>>();
  xcd_tile(bx, by);
  const int x = bx * kWave + lane;
  const bool colok = x < A.nx;
  const int col = min(x, A.nx - 1);
  const int o0 = -2 + by * A.rows;
  const int H = min(A.rows, A.ny + 2 - o0);        // output rows of this block
  const int q = o0 - 1 + wv;
  const bool run = wv < H + 2;                     // (fewer rows in the last strip)
  const bool inner = wv >= 1 && wv <= H;
  const double dtv = A.dt ? *A.dt : 0.0;
  const T alpha = T(A.alpha[1]);
  const T lamh = T(A.sc.lamh);
  extern __shared__ __align__(16) char tile_smem[];
  T* const bs = (T*)tile_smem;                     // b of row q: slot wv + 1
  T* const cs = bs + (A.rows + 4) * 3 * R;         // to rows q - 1 and q + 1 (u, w): slot wv

  T Ua[NC], Wa[NC], Ub[NC], Wb[NC], Uc[NC], Wc[NC], Va[NC], aW[NC];
  if (run) {
    auto load = [&](int r, T (&U)[NC], T (&W)[NC]) {
      const unsigned off = (unsigned)(map_index(r, A.ny, A.bc_lo, A.bc_hi) * A.nx + col);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        U[c] = ld32(A.X[0], (unsigned)(c * A.plane) + off);
        W[c] = lamh * ld32(A.X[2], (unsigned)(c * A.plane) + off);
      }
      if constexpr (WALLS) {
        if (mirrored(r, A.ny, A.bc_lo, A.bc_hi)) {
          mirror_state<Sys, 1>(true, U);
          mirror_normal_derivative<Sys, 1>(true, W);
        }
        const int fs = fixed_side(r, A.ny, A.bc_lo, A.bc_hi);
        if (fs >= 0) {
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            U[c] = T(A.gs[fs][c]);
            W[c] = T(0);
          }
        }
      }
    };
    // b of a row to its slot (zero at ghost rows: L is defined on interior cells)
    auto load_b = [&](int r, int slot) {
      const T su = T(A.sc.u * dtv), sv = T(A.sc.o * dtv), sw = T(A.sc.a * dtv);
      const bool in = r >= 0 && r < A.ny;
      T* d = bs + slot * 3 * R + lane;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned idx = (unsigned)(c * A.plane + (in ? r : 0) * A.nx + col);
        d[c * kWave] = in ? su * ld32(A.b[0], idx) : T(0);
        d[R + c * kWave] = in ? sw * ld32(A.b[2], idx) : T(0);
        d[2 * R + c * kWave] = in ? sv * ld32(A.b[1], idx) : T(0);
      }
    };
    load_b(q, wv + 1);
    if (wv == 0) load_b(q - 1, 0);
    if (wv == H + 1) load_b(q + 1, H + 3);
    load(q - 1, Ua, Wa);
    load(q, Ub, Wb);
    load(q + 1, Uc, Wc);
    const unsigned off = (unsigned)(map_index(q, A.ny, A.bc_lo, A.bc_hi) * A.nx + col);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Va[c] = ld32(A.X[1], (unsigned)(c * A.plane) + off);
      aW[c] = T(0);
    }
    if constexpr (WALLS) {
      if (mirrored(q, A.ny, A.bc_lo, A.bc_hi)) mirror_state<Sys, 1>(true, Va);
      if (fixed_side(q, A.ny, A.bc_lo, A.bc_hi) >= 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) Va[c] = T(0);
      }
    }
    if (q >= 0 && q < A.ny) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < A.na) {
          const T ca = T(A.ca[k] * A.sc.vt);
#pragma unroll
          for (int c = 0; c < NC; ++c) aW[c] += ca * ld32(A.aw[k], (unsigned)(c * A.plane) + off);
        }
    }
  }
  lds_barrier();
  T gU[NC], gV[NC], gW[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) gU[c] = gV[c] = gW[c] = T(0);
  if (run) {
    auto B = [&](int j, int f, int c) -> T { return bs[((wv + 1 + j) * 3 + f) * R + c * kWave + lane]; };
    const auto ce = sy.cell_eig(Ub);
    typename StateBarOf<Sys, T>::type sb{};
    if (inner) {
      // reverse of the row's pointwise g, theta, xi (interfaces q-3/2..q+3/2)
      T gg[NC], gt[NC], gx[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        T l[3][4];                                 // [field][interface q+3/2 .. q-3/2]
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          const T p2 = B(2, f, c), p1 = B(1, f, c), z = B(0, f, c), m1 = B(-1, f, c), m2 = B(-2, f, c);
          l[f][0] = p2 - p1;
          l[f][1] = p1 - z;
          l[f][2] = z - m1;
          l[f][3] = m1 - m2;
        }
        point_cotangents(l[0][0], l[0][1], l[0][2], l[0][3], l[1][0], l[1][1], l[1][2], l[1][3], gg[c], gt[c]);
        gx[c] = point_cotangent_mixed(l[2][0], l[2][1], l[2][2], l[2][3]);
      }
      flux_vjp<1>(sy, Ub, ce.q, gg, sb, gU);
      jac_vjp<1>(sy, Ub, ce.q, Wb, gt, sb, gU, gW);
      jac_vjp<1>(sy, Ub, ce.q, Va, gx, sb, gU, gV);
    }
    __builtin_amdgcn_sched_barrier(0);
    // reverse of the row's faces and HWENO
    T E1[NC], E2[NC], S[NC], Dd[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      E1[c] = Ub[c] - Ua[c];
      E2[c] = Uc[c] - Ub[c];
      S[c] = Wa[c] + Wc[c];
      Dd[c] = Wa[c] - Wc[c];
    }
    T guT[NC], guB[NC], g1[NC], g2[NC], gS[NC], gD[NC];
    {
      T uT[NC], uB[NC], wt_[NC], wT[NC], wB[NC], gwT[NC], gwB[NC], tG[NC], tT[NC], pG[NC], pT[NC];
      if constexpr (IFACE)
        hweno_cell_diff_iface<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, S, Dd, uT, uB, wt_, wT, wB);
      else
        hweno_cell_diff<1>(sy, A.pk, ce, Ub, E1, E2, S, Dd, uT, uB, wt_, wT, wB);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const T g0 = B(0, 0, c), t0 = B(0, 1, c);
        tG[c] = B(1, 0, c) - g0;
        tT[c] = B(1, 1, c) - t0;
        pG[c] = g0 - B(-1, 0, c);
        pT[c] = t0 - B(-1, 1, c);
      }
      face_vjp<1>(sy, alpha, uT, wT, tG, tT, guT, gwT);
      face_vjp<1>(sy, -alpha, uB, wB, pG, pT, guB, gwB);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        face_derivs_diff_vjp(gwT[c], gwB[c], g1[c], g2[c], gS[c], gD[c]);
    }
    __builtin_amdgcn_sched_barrier(0);
    T tm[NC], tp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) tm[c] = tp[c] = T(0);
    if constexpr (IFACE && Sys::kChar)
      hweno_cell_diff_iface_vjp<1>(sy, A.pk, ce, Ua, Ub, Uc, E1, E2, S, Dd, guT, guB, aW, g1, g2, gS, gD,
                                   tm, gU, tp, sb);
    else
      hweno_cell_diff_vjp<1>(sy, A.pk, ce, E1, E2, S, Dd, guT, guB, aW, g1, g2, gS, gD, sb);
    cell_state_vjp(sy, Ub, ce, sb, gU);
    T* d = cs + wv * 4 * R + lane;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      gU[c] += (guT[c] + guB[c]) + (g1[c] - g2[c]);
      d[c * kWave] = tm[c] - g1[c];
      d[R + c * kWave] = gS[c] + gD[c];
      d[2 * R + c * kWave] = tp[c] + g2[c];
      d[3 * R + c * kWave] = gS[c] - gD[c];
    }
  }
  lds_barrier();
  if (inner && colok) {
    const T* up = cs + (wv + 1) * 4 * R + lane;    // from the cell above to this row
    const T* dn = cs + (wv - 1) * 4 * R + 2 * R + lane;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      gU[c] += up[c * kWave] + dn[c * kWave];
      gW[c] = lamh * (gW[c] + (up[R + c * kWave] + dn[R + c * kWave]));
    }
    if (q >= 0 && q < A.ny) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const unsigned idx = (unsigned)(c * A.plane + q * A.nx + x);
        st32(A.G[0], idx, gU[c]);
        st32(A.G[1], idx, gV[c]);
        st32(A.G[2], idx, gW[c]);
      }
    } else {
      T* gp = A.ghost + (size_t)((q < 0 ? q + 2 : q - A.ny + 2) * 3 * NC) * A.nx + x;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        gp[(0 * NC + c) * A.nx] = gU[c];
        gp[(1 * NC + c) * A.nx] = gV[c];
        gp[(2 * NC + c) * A.nx] = gW[c];
      }
    }
  }
}

// Transpose of the gravity source (euler2d-s) of one stage:
// G_f += S^T (c dt b_f) for the fields f = u, v, w, where S(X) = g (0, 0,
// X_0, X_2): G_f[0] += g c dt b_f[2], G_f[2] += g c dt b_f[3].
template <typename T>
__global__ __launch_bounds__(256) void source_vjp_kernel(T* __restrict__ G0, T* __restrict__ G1,
                                                         T* __restrict__ G2, const T* __restrict__ b0,
                                                         const T* __restrict__ b1,
                                                         const T* __restrict__ b2, double cb,
                                                         const double* dt, double g, int plane) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= plane) return;
  const T k = T(g * cb * *dt);
  T* Gs[3] = {G0, G1, G2};
  const T* bs[3] = {b0, b1, b2};
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    Gs[f][i] += k * bs[f][2 * plane + i];
    Gs[f][2 * plane + i] += k * bs[f][3 * plane + i];
  }
}

}  // namespace hweno

// The device scratch of hweno_step_noalloc: the workspace of a step (step
// scalars, per-block maxima, the stage states and the RK base derivatives)
// for callers that cannot allocate. One copy per GPU, held while the process
// lives. Host code must not pass `scratch` itself to a kernel (in host code it
// names a host-side stand-in): it uses the device address that
// hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchBytes = size_t(128) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// =================================================================== host side
using namespace hweno;

namespace {

// StepScalars, AlphaSlots and SpeedTickets. (Larger than they need: with the stage states this
// decides which problems hweno_step_noalloc's scratch holds.)
constexpr size_t kScalarBytes = 20480;
static_assert(sizeof(StepScalars) <= kSlotOffset && kTicketOffset + sizeof(SpeedTickets) <= kScalarBytes);
constexpr int kSpeedBlocks = 1024;
constexpr int kRowsPerBlock = 32;

// Strip height of the 2D forward stage kernels set by hweno_set_strip_rows
// (0: chosen by the occupancy model).
std::atomic<int> g_strip_rows{0};

struct Geometry {
  int nc, nf;           // components; fields per state (2 in 1D: u, v; 3 in 2D)
  size_t esize;         // element size
  size_t plane;         // cells
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A finite Euler state (rho, momenta..., E) with rho > 0 and P > 0.
bool admissible_state(const double* q, int nc, double gas) {
  for (int c = 0; c < nc; ++c)
    if (!std::isfinite(q[c])) return false;
  double m2 = 0.0;
  for (int c = 1; c < nc - 1; ++c) m2 += q[c] * q[c];
  return q[0] > 0.0 && (gas - 1.0) * (q[nc - 1] - 0.5 * m2 / q[0]) > 0.0;
}

bool has_split(const hweno_problem* p) {
  return p->bc[2] == HWENO_SPLIT || p->bc[3] == HWENO_SPLIT;
}

hweno_status validate(const hweno_problem* p) {
  if (!p) return HWENO_EINVAL;
  if (p->dim != 1 && p->dim != 2) return HWENO_EINVAL;
  if (p->nx < 5) return HWENO_EINVAL;
  if (p->dim == 2 && p->ny < 5) return HWENO_EINVAL;
  if (p->dim == 1 && p->ny != 1) return HWENO_EINVAL;
  if (!(p->dx > 0.0) || !std::isfinite(p->dx)) return HWENO_EINVAL;
  if (p->dim == 2 && (!(p->dy > 0.0) || !std::isfinite(p->dy))) return HWENO_EINVAL;
  if (p->system < HWENO_ADVECTION || p->system > HWENO_EULER) return HWENO_EINVAL;
  if (p->system == HWENO_EULER && !(p->gas_gamma > 1.0)) return HWENO_EINVAL;
  if (p->system == HWENO_ADVECTION && (!std::isfinite(p->adv_a) || !std::isfinite(p->adv_b)))
    return HWENO_EINVAL;
  if (!(p->gamma0 > 0.0 && p->gamma0 < 1.0)) return HWENO_EINVAL;
  if (!(p->d0 > 0.0 && p->d0 < 1.0)) return HWENO_EINVAL;
  if (!(p->eps > 0.0) || !std::isfinite(p->eps)) return HWENO_EINVAL;
  for (int k = 0; k < 4; ++k) {
    if (p->bc[k] != HWENO_PERIODIC && p->bc[k] != HWENO_TRANSMISSIVE &&
        p->bc[k] != HWENO_REFLECTIVE && p->bc[k] != HWENO_DIRICHLET && p->bc[k] != HWENO_SPLIT)
      return HWENO_EINVAL;
    if (p->bc[k] == HWENO_SPLIT) {
      if (k < 2 || p->dim != 2 || p->system != HWENO_EULER) return HWENO_EINVAL;
      const hweno_split& sp = p->split[k - 2];
      if (!std::isfinite(sp.x0) || !std::isfinite(sp.slope) || !std::isfinite(sp.speed))
        return HWENO_EINVAL;
      for (int j = 0; j < 2; ++j) {
        const int kind = sp.kind[j];
        if (kind != HWENO_TRANSMISSIVE && kind != HWENO_REFLECTIVE && kind != HWENO_DIRICHLET)
          return HWENO_EINVAL;
        if (kind == HWENO_DIRICHLET && !admissible_state(sp.state[j], 4, p->gas_gamma))
          return HWENO_EINVAL;
      }
    }
    // reflective walls are defined for the Euler equations only
    if (p->bc[k] == HWENO_REFLECTIVE && p->system != HWENO_EULER) return HWENO_EINVAL;
    if (p->bc[k] == HWENO_DIRICHLET && (k < 2 || p->dim == 2)) {
      const double* q = p->bc_state[k];
      const int nc = p->system == HWENO_EULER ? p->dim + 2 : 1;
      if (p->system == HWENO_EULER) {
        if (!admissible_state(q, nc, p->gas_gamma)) return HWENO_EINVAL;
      } else if (!std::isfinite(q[0])) {
        return HWENO_EINVAL;
      }
    }
  }
  if (!std::isfinite(p->gravity)) return HWENO_EINVAL;
  if (p->gravity != 0.0 && !(p->system == HWENO_EULER && p->dim == 2)) return HWENO_EINVAL;
  if ((p->bc[0] == HWENO_PERIODIC) != (p->bc[1] == HWENO_PERIODIC)) return HWENO_EINVAL;
  if (p->dim == 2 && (p->bc[2] == HWENO_PERIODIC) != (p->bc[3] == HWENO_PERIODIC))
    return HWENO_EINVAL;
  if (p->precision != HWENO_F64 && p->precision != HWENO_F32) return HWENO_EINVAL;
  if (p->char_basis != HWENO_BASIS_CELL && p->char_basis != HWENO_BASIS_INTERFACE)
    return HWENO_EINVAL;
  const int nc = p->system == HWENO_EULER ? p->dim + 2 : 1;
  // 32-bit element offsets inside a state array, and 32-bit byte offsets in
  // the stage kernels
  if ((double)nc * (double)p->nx * (double)p->ny >= 2147483647.0) return HWENO_EINVAL;
  const double esize = p->precision == HWENO_F64 ? 8.0 : 4.0;
  if ((double)nc * (double)p->nx * (double)p->ny * esize >= 4294967296.0) return HWENO_EINVAL;
  return HWENO_OK;
}

Geometry geometry(const hweno_problem* p) {
  Geometry g;
  g.nc = p->system == HWENO_EULER ? p->dim + 2 : 1;
  g.nf = p->dim == 1 ? 2 : 3;
  g.esize = p->precision == HWENO_F64 ? 8 : 4;
  g.plane = (size_t)p->nx * (size_t)p->ny;
  return g;
}

// Workspace: scalars | states | adjoint scratch.
// States are stored densely ([field][comp][ny][nx]); each region starts on a
// 256-byte boundary. Regions: X^(1), X^(2), the RK base derivatives
// (V~^n[, W~^n]), and for the adjoint: lambda^(2), lambda^(1) and, in 2D, the
// y-pass's ghost rows and strip halo terms.
struct WsLayout {
  StepScalars* sc;
  char* x1;
  char* x2;
  char* base;
  char* lam2;
  char* lam1;
  char* ghost_y;   // y-pass ghost rows [4][3][NC][nx]
  char* halo;      // y-pass strip halo terms [strips][2][2][NC][nx]
  size_t state_bytes;
};

size_t state_bytes(const Geometry& g) { return align_up((size_t)g.nf * g.nc * g.plane * g.esize, 256); }
size_t base_bytes(const Geometry& g) { return align_up((size_t)(g.nf - 1) * g.nc * g.plane * g.esize, 256); }
size_t ghost_y_bytes(const hweno_problem* p, const Geometry& g) {
  return p->dim == 2 ? align_up((size_t)p->nx * 4 * 3 * g.nc * g.esize, 256) : 0;
}
// y-VJP strips have at least kMinStripRows of the ny + 4 virtual rows
constexpr int kMinStripRows = 4;
size_t halo_bytes(const hweno_problem* p, const Geometry& g) {
  if (p->dim != 2) return 0;
  const size_t strips = (size_t)(p->ny + 4 + kMinStripRows - 1) / kMinStripRows;
  return align_up(strips * 4 * g.nc * (size_t)p->nx * g.esize, 256);
}
size_t ghost_bytes(const hweno_problem* p, const Geometry& g) {
  return ghost_y_bytes(p, g) + halo_bytes(p, g);
}
size_t ws_total(const hweno_problem* p, const Geometry& g) {
  return kScalarBytes + 4 * state_bytes(g) + base_bytes(g) + ghost_bytes(p, g);
}

// The part of the workspace a forward step uses (ws_layout puts it first):
// scalars, X^(1), X^(2), the RK base derivatives.
size_t ws_step_bytes(const Geometry& g) {
  return kScalarBytes + 2 * state_bytes(g) + base_bytes(g);
}

// Device address of `scratch` on the current device, looked up once per
// device (hipGetSymbolAddress with that device current) and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

hweno_status scratch_on_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HWENO_EDEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return HWENO_EDEVICE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return HWENO_OK;
}

WsLayout ws_layout(const hweno_problem* p, void* ws, const Geometry& g) {
  WsLayout w;
  char* b = (char*)ws;
  w.sc = (StepScalars*)b;
  w.state_bytes = state_bytes(g);
  w.x1 = b + kScalarBytes;
  w.x2 = w.x1 + w.state_bytes;
  w.base = w.x2 + w.state_bytes;
  w.lam2 = w.base + base_bytes(g);
  w.lam1 = w.lam2 + w.state_bytes;
  w.ghost_y = w.lam1 + w.state_bytes;
  w.halo = w.ghost_y + ghost_y_bytes(p, g);
  return w;
}

Scheme make_scheme(const hweno_problem* p) {
  Scheme s;
  s.dx = p->dx;
  s.dy = p->dim == 2 ? p->dy : 1.0;
  s.idx = 1.0 / s.dx;
  s.idy = 1.0 / s.dy;
  s.gamma0 = p->gamma0;
  s.g1 = 0.5 * (1.0 - p->gamma0);
  s.d0 = p->d0;
  s.d1 = 0.5 * (1.0 - p->d0);
  s.eps = p->eps;
  s.gas = p->gas_gamma;
  s.adv_a = p->adv_a;
  s.adv_b = p->adv_b;
  return s;
}

inline hweno_status check_launch() {
  return hipGetLastError() == hipSuccess ? HWENO_OK : HWENO_EDEVICE;
}

// Calls f(Sys{}, T{}, DIM) for the problem's system, element type and dimension.
template <class F>
hweno_status dispatch(const hweno_problem* p, F&& f) {
  auto by_type = [&](auto tag) -> hweno_status {
    using T = decltype(tag);
    if (p->dim == 1) {
      switch (p->system) {
        case HWENO_ADVECTION: return f(Advection{p->adv_a, p->adv_b}, T{}, std::integral_constant<int, 1>{});
        case HWENO_BURGERS: return f(Burgers{}, T{}, std::integral_constant<int, 1>{});
        default: return f(Euler<1>{p->gas_gamma}, T{}, std::integral_constant<int, 1>{});
      }
    }
    switch (p->system) {
      case HWENO_ADVECTION: return f(Advection{p->adv_a, p->adv_b}, T{}, std::integral_constant<int, 2>{});
      case HWENO_BURGERS: return f(Burgers{}, T{}, std::integral_constant<int, 2>{});
      default: return f(Euler<2>{p->gas_gamma}, T{}, std::integral_constant<int, 2>{});
    }
  };
  return p->precision == HWENO_F64 ? by_type(double{}) : by_type(float{});
}

// A kernel as a type.
template <auto K>
struct Kernel {
  static constexpr auto fn = K;
};
// Occupancy of the kernel K (block size BLOCK) on the current device: blocks per
// CU from the occupancy query (cached per kernel instance) and the CU count (asked
// each time). False if unknown.
template <auto K, int BLOCK>
bool occupancy(int* per_cu, int* cus) {
  static std::atomic<int> per_cu_cache{0};
  int pc = per_cu_cache.load(std::memory_order_relaxed);
  if (pc <= 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&pc, K, BLOCK, 0) != hipSuccess || pc <= 0)
      return false;
    per_cu_cache.store(pc, std::memory_order_relaxed);
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || *cus <= 0)
    return false;
  *per_cu = pc;
  return true;
}

// Strip height R of a one-wavefront-per-block marcher: col_blocks blocks side
// by side, each marching strips of R of `rows` rows. A strip costs R +
// overhead row units (its warm-up rows). With k of its blocks per SIMD a
// round of 4 CUs k blocks takes k (R + overhead) / g(k), g(1) = 1 and g(k>1)
// = 1.1 (the measured gain of a second wavefront on a SIMD in these
// VALU-bound kernels); R minimises the total over rounds. `fallback` if the
// occupancy is unknown.
int balanced_rows(long col_blocks, int rows, bool known, int per_cu, int cus, double overhead,
                  int fallback, int rmin = 1) {
  if (!known) return fallback < rmin ? rmin : fallback;
  const long simds = 4L * cus;
  const long lanes = per_cu >= 4 ? simds : (long)cus * per_cu;   // blocks at one per SIMD
  const long kmax = per_cu >= 4 ? per_cu / 4 : 1;
  int best = rows > rmin ? rows : rmin;
  double best_cost = 1e300;
  for (int r = rmin; r <= rows; ++r) {
    const long blocks = col_blocks * ((rows + r - 1) / r);
    long k = (blocks + lanes - 1) / lanes;
    if (k > kmax) k = kmax;
    const long rounds = (blocks + lanes * k - 1) / (lanes * k);
    const double cost = (double)rounds * k * (r + overhead) / (k > 1 ? 1.1 : 1.0);
    if (cost < best_cost) {
      best_cost = cost;
      best = r;
    }
  }
  return best;
}

// Rows of a block of the tile kernel, 0 for the marcher: the fewest (of at most
// `most`) with which the blocks are at most one a CU, so that every row of the
// grid is under way at once. A stage then takes about the time of one row; with
// more blocks a second round follows (a block's LDS leaves room for one a CU, at
// one or two rows for two) and the marcher, whose blocks share rows' warm-up over
// more rows, is as fast. Measured (FP64 Euler, us a stage, marcher | tile): 60x60
// 11.2 | 7.6, 60x240 11.5 | 7.9, 240x240 13.7 | 11.0, 256x256 17.4 | 12.5, 320x256
// 17.6 | 14.6, 385x250 18.3 | 15.2, 480x256 19.0 | 16.9; in two rounds 385x250 |
// 18.6; Burgers, the marcher at its best height: 60x60 6.2 | 5.5, 240x240 7.2 |
// 6.5, 256x256 7.4 | 6.9, 320x256 7.4 | 7.5, 480x256 8.1 | 8.2. The y-pass of the adjoint follows the same rule, in both precisions (FP64 Euler, us for
// the adjoint of a step, three y-passes in it): 64x64 105 | 56, 128x128 109 | 57,
// 256x256 126 | 88, 320x256 131 | 93, interface basis 209 | 172, FP32 105 | 74;
// beyond the line 384x384 161 | 151, interface basis 254 | 281, 512x512 214 | 230.
int tile_rows(long col_blocks, int ny, int cus, int most) {
  for (int h = 1; h <= most; ++h)
    if (col_blocks * ((ny + h - 1) / h) <= cus) return h;
  return 0;
}

// The tile kernel of a stage (FP64; nullptr for FP32, which has none).
template <class Sys, typename T, int MODE, int VAR>
auto tile_kernel(int rows) {
  if constexpr (sizeof(T) == 8)
    return rows > kTileFew ? stage2d_tile_kernel<Sys, T, MODE, VAR, kTileRows>
                           : stage2d_tile_kernel<Sys, T, MODE, VAR, kTileFew>;
  else return nullptr;
}

template <class Sys, typename T, int DIM>
hweno_status launch_stage(int mode, const StageArgs<T>& A0, const Sys& sy, hipStream_t st) {
  StageArgs<T> A = A0;
  if constexpr (DIM == 1) {
    dim3 grid((A.nx + kXOut - 1) / kXOut);
    auto modes = [&](auto iface) {
      constexpr bool I = decltype(iface)::value;
      switch (mode) {
        case kRhs: stage1d_kernel<Sys, T, kRhs, I><<<grid, kWave, 0, st>>>(A, sy); break;
        case kStage1: stage1d_kernel<Sys, T, kStage1, I><<<grid, kWave, 0, st>>>(A, sy); break;
        case kStage2: stage1d_kernel<Sys, T, kStage2, I><<<grid, kWave, 0, st>>>(A, sy); break;
        default: stage1d_kernel<Sys, T, kStage3, I><<<grid, kWave, 0, st>>>(A, sy); break;
      }
    };
    if constexpr (Sys::kChar) {
      if (A.iface)
        modes(std::true_type{});
      else
        modes(std::false_type{});
    } else {
      modes(std::false_type{});
    }
  } else {
    const int col_blocks = (A.nx + kXOut - 1) / kXOut;
    auto go = [&](auto kernel, auto tile) {
      constexpr auto fn = decltype(kernel)::fn;
      int per_cu = 0, cus = 0;
      const bool known = occupancy<fn, kWave>(&per_cu, &cus);
      const int forced = g_strip_rows.load(std::memory_order_relaxed);
      if constexpr (sizeof(T) == 8) {
        A.rows = known && forced <= 0 ? tile_rows(col_blocks, A.ny, cus, kTileRows) : 0;
        if (A.rows > 0) {
          const dim3 grid(col_blocks, (A.ny + A.rows - 1) / A.rows);
          tile(A.rows)<<<grid, (A.rows + 2) * kWave, tile_lds<Sys::NC, T>(A.rows), st>>>(A, sy);
          return;
        }
      }
      // warm-up: two rows of loads and y-pointwise fluxes, two of y-HWENO,
      // about one full row in all
      A.rows = forced > 0 ? forced : balanced_rows(col_blocks, A.ny, known, per_cu, cus, 1.0, 32);
      dim3 grid(col_blocks, (A.ny + A.rows - 1) / A.rows);
      fn<<<grid, kWave, 0, st>>>(A, sy);
    };
    auto modes = [&](auto var) {
      constexpr int V = decltype(var)::value;
      switch (mode) {
        case kRhs: go(Kernel<stage2d_kernel<Sys, T, kRhs, V>>{}, [](int h) { return tile_kernel<Sys, T, kRhs, V>(h); }); break;
        case kStage1: go(Kernel<stage2d_kernel<Sys, T, kStage1, V>>{}, [](int h) { return tile_kernel<Sys, T, kStage1, V>(h); }); break;
        case kStage2: go(Kernel<stage2d_kernel<Sys, T, kStage2, V>>{}, [](int h) { return tile_kernel<Sys, T, kStage2, V>(h); }); break;
        default: go(Kernel<stage2d_kernel<Sys, T, kStage3, V>>{}, [](int h) { return tile_kernel<Sys, T, kStage3, V>(h); }); break;
      }
    };
    bool walls = false;
    for (int k = 0; k < 4; ++k)
      walls = walls || A.bc[k] == kBcReflective || A.bc[k] == kBcDirichlet || A.bc[k] == kBcSplit;
    const int var = (walls ? kVarWalls : 0) | (Sys::kChar && A.iface ? kVarIface : 0) |
                    (Sys::kChar && A.gravity != 0.0 ? kVarSource : 0);
    if constexpr (Sys::kChar) {
      switch (var) {
        case 0: modes(std::integral_constant<int, 0>{}); break;
        case 1: modes(std::integral_constant<int, 1>{}); break;
        case 2: modes(std::integral_constant<int, 2>{}); break;
        case 3: modes(std::integral_constant<int, 3>{}); break;
        case 4: modes(std::integral_constant<int, 4>{}); break;
        case 5: modes(std::integral_constant<int, 5>{}); break;
        case 6: modes(std::integral_constant<int, 6>{}); break;
        default: modes(std::integral_constant<int, 7>{}); break;
      }
    } else if (walls) {
      modes(std::integral_constant<int, kVarWalls>{});
    } else {
      modes(std::integral_constant<int, 0>{});
    }
  }
  return check_launch();
}

template <typename T>
StageArgs<T> base_args(const hweno_problem* p) {
  StageArgs<T> A;
  std::memset(&A, 0, sizeof(A));
  A.nx = p->nx;
  A.ny = p->ny;
  A.rows = kRowsPerBlock;
  A.plane = p->nx * p->ny;
  for (int k = 0; k < 4; ++k) A.bc[k] = p->bc[k];
  A.iface = p->char_basis == HWENO_BASIS_INTERFACE;
  for (int k = 0; k < 4; ++k)
    for (int c = 0; c < 4; ++c) A.gs[k][c] = p->bc_state[k][c];
  A.gravity = p->system == HWENO_EULER && p->dim == 2 ? p->gravity : 0.0;
  for (int k = 0; k < 2; ++k) {
    A.sp[k].x0 = p->split[k].x0;
    A.sp[k].slope = p->split[k].slope;
    A.sp[k].speed = p->split[k].speed;
    for (int j = 0; j < 2; ++j) {
      A.sp[k].kind[j] = p->split[k].kind[j];
      for (int c = 0; c < 4; ++c) A.sp[k].state[j][c] = p->split[k].state[j][c];
    }
  }
  A.t0 = nullptr;
  A.tc = 0.0;
  A.ctl.dim = p->dim;
  A.next_set = -1;
  A.s = make_scheme(p);
  const double lam = Carried<T>::lam;
  const double vt = point_vt_scale<T>(A.s);
  A.pk = point_k(A.s, lam, vt);
  const double F = kFluxScaled<T> ? -19.0 / (960.0 * lam) : 1.0;
  const double H = kFluxScaled<T> ? 37.0 / (864.0 * lam) : 1.0;
  FluxK& k = A.fk;
  k.lx = lam * A.s.dx;
  k.ly = lam * A.s.dy;
  k.ilx = A.s.idx / lam;
  k.ily = A.s.idy / lam;
  k.vtx = vt * A.s.idx;
  k.vty = vt * A.s.idy;
  k.xu = F * A.s.idx;
  k.yu = F * A.s.idy;
  k.xv = H * A.s.idx * A.s.idx;
  k.yw = H * A.s.idy * A.s.idy;
  k.xw = k.yv = A.s.idx * A.s.idy / (12.0 * lam);
  return A;
}

// alpha: null for the seed of a run's first step (see speed_kernel).
template <class Sys, typename T, int DIM>
hweno_status launch_speed(const hweno_problem* p, const T* U, const Sys& sy, StepScalars* sc, int nslots,
                          double* alpha, hipStream_t st) {
  const size_t plane = (size_t)p->nx * p->ny, b = (plane + 255) / 256;
  const int nb = (int)(b < (size_t)kSpeedBlocks ? b : (size_t)kSpeedBlocks);
  speed_kernel<Sys, T, DIM><<<nb, 256, 0, st>>>(U, (int)plane, sy, sc, nslots, alpha);
  return check_launch();
}

// One VJP of a stage: in 2D the y-pass marches up column strips and writes
// out[], then the x-pass adds its terms and the y-pass's strip halos and ghost
// rows; in 1D the x-pass alone writes it.
struct Cot {
  const void* b[3];       // the flux cotangent state (u, v, w; w null in 1D), scaled by cb dt
  double cb;
  const void* a[3][3];    // the a sets (u, v, w each)
  double ca[3];
  int na;                 // 1 or 3
};

template <class Sys, typename T, int DIM>
hweno_status launch_vjp(const hweno_problem* p, const Sys& sy, const Geometry& g,
                        const WsLayout& wl, const T* X[3], const Cot& cot,
                        const double* alpha, const double* dt, T* out[3], hipStream_t st) {
  constexpr int NC = Sys::NC;
  const Scheme sc = make_scheme(p);
  const PointK pk = point_k(sc, Carried<T>::lam, point_vt_scale<T>(sc));
  const int nx = p->nx, ny = p->ny, plane = nx * ny;
  // the interface basis changes only the per-cell reverse (three bases)
  const bool iface = Sys::kChar && p->char_basis == HWENO_BASIS_INTERFACE;
  // y-pass (2D): overwrites out; its strip halos and ghost rows are folded
  // in by the x-pass
  int ystrip_rows = 0, ystrips = 0;
  if constexpr (DIM == 2) {
    VjpYArgs<T> A;
    std::memset(&A, 0, sizeof(A));
    for (int f = 0; f < 3; ++f) {
      A.X[f] = X[f];
      A.b[f] = (const T*)cot.b[f];
    }
    for (int k = 0; k < cot.na; ++k) {
      A.aw[k] = (const T*)cot.a[k][2];
      A.ca[k] = cot.ca[k];
    }
    A.na = cot.na;
    A.dt = dt;
    A.alpha = alpha;
    for (int f = 0; f < 3; ++f) A.G[f] = out[f];
    A.ghost = (T*)wl.ghost_y;
    A.halo = (T*)wl.halo;
    A.nx = nx;
    A.ny = ny;
    A.plane = plane;
    A.bc_lo = p->bc[2];
    A.bc_hi = p->bc[3];
    for (int c = 0; c < 4; ++c) {
      A.gs[0][c] = p->bc_state[2][c];
      A.gs[1][c] = p->bc_state[3][c];
    }
    A.sc = vjp_scales<T>(sc, sc.dy, cot.cb);
    A.pk = pk;
    // strips of at least kMinStripRows rows (the halo buffer is sized for
    // that); warm-up: four rows of loads
    bool walls = false;
    for (int k = 0; k < 4; ++k) walls = walls || p->bc[k] == HWENO_REFLECTIVE || p->bc[k] == HWENO_DIRICHLET;
    int nstrips = 0;
    const int col_blocks = (nx + kWave - 1) / kWave;
    auto go = [&](auto kernel, auto tile) {
      constexpr auto fn = decltype(kernel)::fn;
      int per_cu = 0, cus = 0;
      const bool known = occupancy<fn, kWave>(&per_cu, &cus);
      A.rows = known ? tile_rows(col_blocks, ny + 4, cus, kVjpTileRows) : 0;
      if (A.rows > 0) {   // no strip halos
        const dim3 grid(col_blocks, (ny + 4 + A.rows - 1) / A.rows);
        tile<<<grid, (A.rows + 2) * kWave, vjp_tile_lds<NC, T>(A.rows), st>>>(A, sy);
        return;
      }
      A.rows = balanced_rows(col_blocks, ny + 4, known, per_cu, cus, 1.0, 16, kMinStripRows);
      nstrips = (ny + 4 + A.rows - 1) / A.rows;
      fn<<<dim3(col_blocks, nstrips), kWave, 0, st>>>(A, sy);
    };
    if (iface) {
      if constexpr (Sys::kChar) {
        if (walls)
          go(Kernel<vjp_y_kernel<Sys, T, true, true>>{}, vjp_y_tile_kernel<Sys, T, true, true>);
        else
          go(Kernel<vjp_y_kernel<Sys, T, false, true>>{}, vjp_y_tile_kernel<Sys, T, false, true>);
      }
    } else if (walls) {
      go(Kernel<vjp_y_kernel<Sys, T, true>>{}, vjp_y_tile_kernel<Sys, T, true>);
    } else {
      go(Kernel<vjp_y_kernel<Sys, T, false>>{}, vjp_y_tile_kernel<Sys, T, false>);
    }
    if (check_launch() != HWENO_OK) return HWENO_EDEVICE;
    ystrip_rows = A.rows;
    ystrips = nstrips;
  }
  // x-pass (in 2D after the y-pass, adding to its result)
  {
    VjpArgs<T> A;
    std::memset(&A, 0, sizeof(A));
    for (int f = 0; f < 3; ++f) {
      A.X[f] = X[f];
      A.b[f] = (const T*)cot.b[f];
    }
    for (int k = 0; k < cot.na; ++k) {
      A.a[k][0] = (const T*)cot.a[k][0];
      A.a[k][1] = (const T*)cot.a[k][1];
      A.ca[k] = cot.ca[k];
    }
    A.dt = dt;
    A.alpha = alpha;
    A.accumulate = DIM == 2;   // in 2D the y-pass has written out
    if (DIM == 2) {
      A.yhalo = (const T*)wl.halo;
      A.yghost = (const T*)wl.ghost_y;
      A.yR = ystrip_rows;
      A.ystrips = ystrips;
      for (int k = 0; k < 4; ++k) {
        const int q = k < 2 ? k - 2 : ny + k - 2;
        const bool fixed = fixed_side(q, ny, p->bc[2], p->bc[3]) >= 0;
        A.yimg[k] = fixed ? -1 : map_index(q, ny, p->bc[2], p->bc[3]);
        A.yflip[k] = mirrored(q, ny, p->bc[2], p->bc[3]);
        A.yqj[k] = halo_source(q, ystrip_rows, ystrips, A.yqs[k]);
      }
    }
    for (int f = 0; f < 3; ++f) A.G[f] = out[f];
    A.n = nx;
    A.rows = ny;
    A.plane = plane;
    A.bc_lo = p->bc[0];
    A.bc_hi = p->bc[1];
    for (int c = 0; c < 4; ++c) {
      A.gs[0][c] = p->bc_state[0][c];
      A.gs[1][c] = p->bc_state[1][c];
    }
    A.sc = vjp_scales<T>(sc, sc.dx, cot.cb);
    A.pk = pk;
    const int total = p->bc[0] == HWENO_PERIODIC ? nx : nx + 4;
    dim3 grid((total + kXOut - 1) / kXOut, ny);
    auto special = [](int b) { return b == HWENO_REFLECTIVE || b == HWENO_DIRICHLET; };
    const bool xwalls = special(p->bc[0]) || special(p->bc[1]);
    auto go = [&](auto walls, auto ifc) {
      constexpr bool W = decltype(walls)::value, I = decltype(ifc)::value;
      if (cot.na == 1)
        vjp_row_kernel<Sys, T, DIM + 1, 1, W, I><<<grid, kWave, 0, st>>>(A, sy);
      else
        vjp_row_kernel<Sys, T, DIM + 1, 3, W, I><<<grid, kWave, 0, st>>>(A, sy);
    };
    auto go_w = [&](auto ifc) {
      if (xwalls)
        go(std::true_type{}, ifc);
      else
        go(std::false_type{}, ifc);
    };
    if constexpr (Sys::kChar) {
      if (iface)
        go_w(std::true_type{});
      else
        go_w(std::false_type{});
    } else {
      go_w(std::false_type{});
    }
    if (check_launch() != HWENO_OK) return HWENO_EDEVICE;
  }
  if constexpr (DIM == 2) {
    if (Sys::kChar && NC == 4 && p->gravity != 0.0) {
      source_vjp_kernel<T><<<(plane + 255) / 256, 256, 0, st>>>(
          out[0], out[1], out[2], (const T*)cot.b[0], (const T*)cot.b[1], (const T*)cot.b[2], cot.cb,
          dt, p->gravity, plane);
      if (check_launch() != HWENO_OK) return HWENO_EDEVICE;
    }
  }
  return HWENO_OK;
}

// Whether a 1D problem's steps run in one block: as long as a block holds the
// line (16 wavefronts, with the interface basis 8, which its registers allow).
// There one CU's share of the arithmetic still takes less than a launch per
// stage. Measured (us for 32 steps, launches | one block): Burgers N = 60 351 |
// 60, 480 392 | 90, 960 386 | 152; Euler N = 60 431 | 144, 480 479 | 236, 960
// 476 | 422; interface basis N = 60 499 | 214, 480 548 | 376. One step alone:
// 19-24 | 11-18.
template <class Sys>
bool line_fits(const hweno_problem* p) {
  const bool iface = Sys::kChar && p->char_basis == HWENO_BASIS_INTERFACE;
  return p->nx <= line_waves(iface) * kXOut;
}
template <class Sys, typename T>
void launch_line(const StageArgs<T>& A, const Sys& sy, int nsteps, hipStream_t st) {
  const int waves = (A.nx + kXOut - 1) / kXOut;
  auto go = [&](auto kernel) {
    kernel<<<1, waves * kWave, line_lds<Sys::NC, T>(A.nx), st>>>(A, sy, nsteps);
  };
  if constexpr (Sys::kChar) {
    if (A.iface) return go(steps1d_kernel<Sys, T, true>);
  }
  go(steps1d_kernel<Sys, T, false>);
}

// Time-stepping loop of hweno_step(s) ((fully-hweno), (2Dfully-hweno)). Short 1D
// lines (line_fits): one launch for up to kLineSteps steps. Else one
// seeding pass (the maxima of the spectral radii of the initial state, into the
// accumulators of the stage-1 alphas), then three stage launches per step. Stage 1 computes the
// step's dt from its alphas, stage 3 reduces the next step's stage-1 alphas
// in its epilogue, so steady-state steps launch the three stage kernels only.
hweno_status run_steps(const hweno_problem* p, void* u, void* v, void* w, int32_t nsteps,
                       int32_t dt_rule, double cfl, double dt_fixed, double t_end, double* t,
                       double* dt_used, double* alpha_rec, void* stages, void* ws,
                       hipStream_t stream, hipEvent_t* events) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!u || !v || !t || !ws || nsteps < 1) return HWENO_EINVAL;
  if (p->dim == 2 && !w) return HWENO_EINVAL;
  if (p->dim == 1 && w) return HWENO_EINVAL;
  if (dt_rule < HWENO_DT_PRODUCTION || dt_rule > HWENO_DT_FIXED) return HWENO_EINVAL;
  if (dt_rule == HWENO_DT_FIXED ? !(dt_fixed > 0.0) : !(cfl > 0.0)) return HWENO_EINVAL;
  if (std::isnan(t_end)) return HWENO_EINVAL;
  if (stages && nsteps != 1) return HWENO_EINVAL;
  const Geometry g = geometry(p);
  WsLayout wl = ws_layout(p, ws, g);
  return dispatch(p, [&](auto sy, auto tag, auto dimc) -> hweno_status {
    using T = decltype(tag);
    using Sys = decltype(sy);
    constexpr int DIM = decltype(dimc)::value;
    const size_t P = g.plane;
    // stage states: the caller's `stages` buffer when given, else the workspace
    char* x1 = stages ? (char*)stages : wl.x1;
    char* x2 = stages ? (char*)stages + (size_t)g.nf * g.nc * P * sizeof(T) : wl.x2;
    T* Vt = (T*)wl.base;
    T* Wt = DIM == 2 ? Vt + (size_t)g.nc * P : nullptr;
    auto F = [&](char* b, int f) { return (T*)(b + (size_t)f * g.nc * P * sizeof(T)); };
    // (a 1D stage has a block per kXOut cells; in 2D a small grid has more)
    const int nslots = DIM == 1 && (p->nx + kXOut - 1) / kXOut <= kOneSlotBlocks ? 1 : kSlots;
    StageArgs<T> A = base_args<T>(p);
    A.dt = &wl.sc->dt;
    A.active = &wl.sc->active;
    A.alpha = nullptr;
    A.nslots = nslots;
    A.t0 = &wl.sc->t0;            // stage times t0, t0 + dt, t0 + dt/2
    A.ctl.sc = wl.sc;
    A.ctl.t = t;
    A.ctl.rule = dt_rule;
    A.ctl.cfl = cfl;
    A.ctl.dt_fixed = dt_fixed;
    A.ctl.t_end = t_end;
    if (dt_rule == HWENO_DT_ACCURACY) {
      A.ctl.hx = std::pow(p->dx, 5.0 / 3.0);
      A.ctl.hy = DIM == 2 ? std::pow(p->dy, 5.0 / 3.0) : 1.0;
    } else {
      A.ctl.hx = p->dx;
      A.ctl.hy = DIM == 2 ? p->dy : 1.0;
    }
    if constexpr (DIM == 1 && sizeof(T) == 8) {
      if (!stages && !events && line_fits<Sys>(p)) {
        A.Uo = (T*)u;
        A.Vo = (T*)v;
        for (int k = 0; k < nsteps; k += kLineSteps) {
          A.alpha_rec = alpha_rec ? alpha_rec + 6 * k : nullptr;
          A.ctl.dt_used = dt_used ? dt_used + k : nullptr;
          const int n = nsteps - k < kLineSteps ? nsteps - k : kLineSteps;
          launch_line<Sys, T>(A, sy, n, stream);
          if (check_launch() != HWENO_OK) return HWENO_EDEVICE;
        }
        return HWENO_OK;
      }
    }
    // an error between the launches: what they raised must not reach a later call
    auto failed = [&](hweno_status s) {
      alpha_clear_kernel<<<1, kWave, 0, stream>>>(wl.sc);
      (void)hipGetLastError();
      return s;
    };
    hweno_status s2 = launch_speed<Sys, T, DIM>(p, (const T*)u, sy, wl.sc, nslots, nullptr, stream);
    if (s2 != HWENO_OK) return failed(s2);
    for (int k = 0; k < nsteps; ++k) {
      hipEvent_t* ev = events ? events + 4 * k : nullptr;
      auto mark = [&](int j) -> bool { return !ev || hipEventRecord(ev[j], stream) == hipSuccess; };
      double* rec = alpha_rec ? alpha_rec + 6 * k : nullptr;
      A.ctl.dt_used = dt_used ? dt_used + k : nullptr;
      // stage 1: X^n -> X^(1), V~^n, W~^n; computes dt
      if (!mark(0)) return failed(HWENO_EDEVICE);
      A.U = (const T*)u; A.V = (const T*)v; A.W = (const T*)w;
      A.Ub = nullptr; A.Vb = nullptr; A.Wb = nullptr;
      A.Uo = F(x1, 0); A.Vo = F(x1, 1); A.Wo = DIM == 2 ? F(x1, 2) : nullptr;
      A.Vt = Vt; A.Wt = Wt;
      A.alpha_set = k == 0 ? kSetSeed : kSetNext;
      A.next_set = kSet2;
      A.alpha_rec = rec;
      A.tc = 0.0;
      if ((s2 = launch_stage<Sys, T, DIM>(kStage1, A, sy, stream)) != HWENO_OK) return failed(s2);
      if (!mark(1)) return failed(HWENO_EDEVICE);
      // stage 2: X^(1) -> X^(2) with base (U^n, V~^n, W~^n)
      A.U = F(x1, 0); A.V = F(x1, 1); A.W = DIM == 2 ? F(x1, 2) : nullptr;
      A.Ub = (const T*)u; A.Vb = Vt; A.Wb = Wt;
      A.Uo = F(x2, 0); A.Vo = F(x2, 1); A.Wo = DIM == 2 ? F(x2, 2) : nullptr;
      A.Vt = nullptr; A.Wt = nullptr;
      A.alpha_set = kSet2;
      A.next_set = kSet3;
      A.alpha_rec = rec ? rec + 2 : nullptr;
      A.tc = 1.0;
      if ((s2 = launch_stage<Sys, T, DIM>(kStage2, A, sy, stream)) != HWENO_OK) return failed(s2);
      if (!mark(2)) return failed(HWENO_EDEVICE);
      // stage 3: X^(2) -> X^{n+1}, in place on (u, v, w); the result's alphas
      // are the next step's stage-1 alphas
      A.U = F(x2, 0); A.V = F(x2, 1); A.W = DIM == 2 ? F(x2, 2) : nullptr;
      A.Uo = (T*)u; A.Vo = (T*)v; A.Wo = (T*)w;
      A.alpha_set = kSet3;
      A.next_set = kSetNext;
      A.alpha_rec = rec ? rec + 4 : nullptr;
      A.tc = 0.5;
      if ((s2 = launch_stage<Sys, T, DIM>(kStage3, A, sy, stream)) != HWENO_OK) return failed(s2);
      if (!mark(3)) return failed(HWENO_EDEVICE);
    }
    return HWENO_OK;
  });
}

}  // namespace

// =================================================================== C ABI
extern "C" {

const char* hweno_status_string(hweno_status s) {
  switch (s) {
    case HWENO_OK: return "ok";
    case HWENO_EINVAL: return "invalid argument";
    case HWENO_EUNSUPPORTED: return "unsupported";
    case HWENO_EDEVICE: return "HIP runtime error";
    case HWENO_ENONFINITE: return "non-finite state";
    case HWENO_ENONPHYSICAL: return "non-physical state (density or pressure <= 0)";
    case HWENO_ESCRATCH: return "problem exceeds the static scratch of hweno_step_noalloc";
  }
  return "unknown status";
}

hweno_status hweno_workspace_bytes(const hweno_problem* p, size_t* bytes) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!bytes) return HWENO_EINVAL;
  const Geometry g = geometry(p);
  *bytes = ws_total(p, g);
  return HWENO_OK;
}

hweno_status hweno_workspace_init(const hweno_problem* p, void* ws, hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!ws) return HWENO_EINVAL;
  ws_init_kernel<<<1, kWave, 0, stream>>>((StepScalars*)ws);
  return check_launch();
}

hweno_status hweno_max_wavespeed(const hweno_problem* p, const void* u, double* alpha, void* ws,
                                 hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!u || !alpha || !ws) return HWENO_EINVAL;
  const Geometry g = geometry(p);
  WsLayout w = ws_layout(p, ws, g);
  return dispatch(p, [&](auto sy, auto tag, auto dimc) -> hweno_status {
    using T = decltype(tag);
    using Sys = decltype(sy);
    constexpr int DIM = decltype(dimc)::value;
    return launch_speed<Sys, T, DIM>(p, (const T*)u, sy, w.sc, kSlots, alpha, stream);
  });
}

hweno_status hweno_rhs(const hweno_problem* p, const void* u, const void* v, const void* w,
                       const double* alpha, void* Lu, void* Lv, void* Lw, void* vtilde,
                       void* wtilde, void* ws, hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!u || !v || !alpha || !Lu || !Lv || !vtilde || !ws) return HWENO_EINVAL;
  if (p->dim == 2 && (!w || !Lw || !wtilde)) return HWENO_EINVAL;
  if (p->dim == 1 && (w || Lw || wtilde)) return HWENO_EINVAL;
  const void* ins[3] = {u, v, w};
  void* outs[5] = {Lu, Lv, Lw, vtilde, wtilde};
  for (auto o : outs)
    for (auto i : ins)
      if (o && i && o == i) return HWENO_EINVAL;
  return dispatch(p, [&](auto sy, auto tag, auto dimc) -> hweno_status {
    using T = decltype(tag);
    using Sys = decltype(sy);
    constexpr int DIM = decltype(dimc)::value;
    StageArgs<T> A = base_args<T>(p);
    A.U = (const T*)u; A.V = (const T*)v; A.W = (const T*)w;
    A.Uo = (T*)Lu; A.Vo = (T*)Lv; A.Wo = (T*)Lw;
    A.Vt = (T*)vtilde; A.Wt = (T*)wtilde;
    A.alpha = alpha;
    return launch_stage<Sys, T, DIM>(kRhs, A, sy, stream);
  });
}

hweno_status hweno_step(const hweno_problem* p, void* u, void* v, void* w, int32_t dt_rule,
                        double cfl, double dt_fixed, double t_end, double* t, double* dt_used,
                        double* alpha_rec, void* stages, void* ws, hipStream_t stream) {
  return run_steps(p, u, v, w, 1, dt_rule, cfl, dt_fixed, t_end, t, dt_used, alpha_rec, stages, ws,
                   stream, nullptr);
}

hweno_status hweno_step_profiled(const hweno_problem* p, void* u, void* v, void* w,
                                 int32_t dt_rule, double cfl, double dt_fixed, double t_end,
                                 double* t, double* dt_used, double* alpha_rec, void* stages,
                                 void* ws, hipStream_t stream, hipEvent_t* events) {
  return run_steps(p, u, v, w, 1, dt_rule, cfl, dt_fixed, t_end, t, dt_used, alpha_rec, stages, ws,
                   stream, events);
}

hweno_status hweno_steps(const hweno_problem* p, void* u, void* v, void* w, int32_t nsteps,
                         int32_t dt_rule, double cfl, double dt_fixed, double t_end, double* t,
                         double* dt_used, double* alpha_rec, void* ws, hipStream_t stream,
                         hipEvent_t* events) {
  return run_steps(p, u, v, w, nsteps, dt_rule, cfl, dt_fixed, t_end, t, dt_used, alpha_rec,
                   nullptr, ws, stream, events);
}

hweno_status hweno_step_noalloc(const hweno_problem* p, void* u, void* v, void* w,
                                int32_t dt_rule, double cfl, double dt_fixed, double t_end,
                                double* t, double* dt_used, double* alpha_rec,
                                hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (ws_step_bytes(geometry(p)) > kScratchBytes) return HWENO_ESCRATCH;
  if (!u || !v || !t) return HWENO_EINVAL;
  void* ws = nullptr;
  if ((st = scratch_on_current_device(&ws)) != HWENO_OK) return st;
  // the scratch keeps the previous call's contents: clear the step scalars
  // (flags, alpha accumulators) with a kernel, before the step's launches
  ws_init_kernel<<<1, kWave, 0, stream>>>((StepScalars*)ws);
  if ((st = check_launch()) != HWENO_OK) return st;
  return run_steps(p, u, v, w, 1, dt_rule, cfl, dt_fixed, t_end, t, dt_used, alpha_rec, nullptr,
                   ws, stream, nullptr);
}

hweno_status hweno_set_strip_rows(int32_t rows) {
  if (rows < 0) return HWENO_EINVAL;
  g_strip_rows.store(rows, std::memory_order_relaxed);
  return HWENO_OK;
}

hweno_status hweno_step_frozen(const hweno_problem* p, void* u, void* v, void* w, void* u_out,
                               void* v_out, void* w_out, const double* dt, const double* alpha_rec,
                               void* stages, void* ws, hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!u || !v || !dt || !alpha_rec || !ws) return HWENO_EINVAL;
  if (p->dim == 2 && !w) return HWENO_EINVAL;
  if (p->dim == 1 && w) return HWENO_EINVAL;
  if (has_split(p)) return HWENO_EUNSUPPORTED;   // no step time here
  if (u_out) {
    if (!v_out || (p->dim == 2) != (w_out != nullptr)) return HWENO_EINVAL;
    const void* ins[4] = {u, v, w, stages};
    for (const void* o : {(const void*)u_out, (const void*)v_out, (const void*)w_out})
      for (const void* i : ins)
        if (o && i && o == i) return HWENO_EINVAL;
  } else if (v_out || w_out) {
    return HWENO_EINVAL;
  }
  const Geometry g = geometry(p);
  WsLayout wl = ws_layout(p, ws, g);
  return dispatch(p, [&](auto sy, auto tag, auto dimc) -> hweno_status {
    using T = decltype(tag);
    using Sys = decltype(sy);
    constexpr int DIM = decltype(dimc)::value;
    const size_t fs = (size_t)g.nc * g.plane;
    char* x1 = stages ? (char*)stages : wl.x1;
    char* x2 = stages ? (char*)stages + (size_t)g.nf * fs * sizeof(T) : wl.x2;
    auto F = [&](char* b, int f) { return (T*)(b + (size_t)f * fs * sizeof(T)); };
    T* Vt = (T*)wl.base;
    T* Wt = DIM == 2 ? Vt + fs : nullptr;
    StageArgs<T> A = base_args<T>(p);
    A.dt = dt;
    hweno_status s2;
    A.U = (const T*)u; A.V = (const T*)v; A.W = (const T*)w;
    A.Uo = F(x1, 0); A.Vo = F(x1, 1); A.Wo = DIM == 2 ? F(x1, 2) : nullptr;
    A.Vt = Vt; A.Wt = Wt;
    A.alpha = alpha_rec;
    if ((s2 = launch_stage<Sys, T, DIM>(kStage1, A, sy, stream)) != HWENO_OK) return s2;
    A.U = F(x1, 0); A.V = F(x1, 1); A.W = DIM == 2 ? F(x1, 2) : nullptr;
    A.Ub = (const T*)u; A.Vb = Vt; A.Wb = Wt;
    A.Uo = F(x2, 0); A.Vo = F(x2, 1); A.Wo = DIM == 2 ? F(x2, 2) : nullptr;
    A.Vt = nullptr; A.Wt = nullptr;
    A.alpha = alpha_rec + 2;
    if ((s2 = launch_stage<Sys, T, DIM>(kStage2, A, sy, stream)) != HWENO_OK) return s2;
    A.U = F(x2, 0); A.V = F(x2, 1); A.W = DIM == 2 ? F(x2, 2) : nullptr;
    if (u_out) {
      A.Uo = (T*)u_out; A.Vo = (T*)v_out; A.Wo = (T*)w_out;
    } else {
      A.Uo = (T*)u; A.Vo = (T*)v; A.Wo = (T*)w;
    }
    A.alpha = alpha_rec + 4;
    return launch_stage<Sys, T, DIM>(kStage3, A, sy, stream);
  });
}

hweno_status hweno_adjoint_step(const hweno_problem* p, const void* u_n, const void* v_n,
                                const void* w_n, const void* stages, const double* dt,
                                const double* alpha_rec, const void* lam_u_in,
                                const void* lam_v_in, const void* lam_w_in, void* lam_u_out,
                                void* lam_v_out, void* lam_w_out, void* ws, hipStream_t stream) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  const bool two = p->dim == 2;
  if (!u_n || !v_n || !dt || !alpha_rec || !lam_u_in || !lam_v_in || !lam_u_out || !lam_v_out || !ws)
    return HWENO_EINVAL;
  if (has_split(p)) return HWENO_EUNSUPPORTED;
  if (two && (!w_n || !lam_w_in || !lam_w_out)) return HWENO_EINVAL;
  if (!two && (w_n || lam_w_in || lam_w_out)) return HWENO_EINVAL;
  const void* ins[8] = {u_n, v_n, w_n, stages, lam_u_in, lam_v_in, lam_w_in, nullptr};
  void* outs[3] = {lam_u_out, lam_v_out, lam_w_out};
  for (auto o : outs)
    for (auto i : ins)
      if (o && i && o == i) return HWENO_EINVAL;
  const Geometry g = geometry(p);
  WsLayout wl = ws_layout(p, ws, g);
  return dispatch(p, [&](auto sy, auto tag, auto dimc) -> hweno_status {
    using T = decltype(tag);
    using Sys = decltype(sy);
    constexpr int DIM = decltype(dimc)::value;
    const size_t P = g.plane;
    const size_t fs = (size_t)g.nc * P;        // elements per field
    char* x1 = stages ? (char*)stages : wl.x1;
    char* x2 = stages ? (char*)stages + (size_t)g.nf * fs * sizeof(T) : wl.x2;
    auto F = [&](char* b, int f) { return (T*)(b + (size_t)f * fs * sizeof(T)); };
    hweno_status s2;
    if (!stages) {
      // recompute X^(1), X^(2) with the recorded alphas and dt
      T* Vt = (T*)wl.base;
      T* Wt = DIM == 2 ? Vt + fs : nullptr;
      StageArgs<T> A = base_args<T>(p);
      A.dt = dt;
      A.U = (const T*)u_n; A.V = (const T*)v_n; A.W = (const T*)w_n;
      A.Uo = F(x1, 0); A.Vo = F(x1, 1); A.Wo = DIM == 2 ? F(x1, 2) : nullptr;
      A.Vt = Vt; A.Wt = Wt;
      A.alpha = alpha_rec;
      if ((s2 = launch_stage<Sys, T, DIM>(kStage1, A, sy, stream)) != HWENO_OK) return s2;
      A.U = F(x1, 0); A.V = F(x1, 1); A.W = DIM == 2 ? F(x1, 2) : nullptr;
      A.Ub = (const T*)u_n; A.Vb = Vt; A.Wb = Wt;
      A.Uo = F(x2, 0); A.Vo = F(x2, 1); A.Wo = DIM == 2 ? F(x2, 2) : nullptr;
      A.Vt = nullptr; A.Wt = nullptr;
      A.alpha = alpha_rec + 2;
      if ((s2 = launch_stage<Sys, T, DIM>(kStage2, A, sy, stream)) != HWENO_OK) return s2;
    }
    T* l2[3] = {F(wl.lam2, 0), F(wl.lam2, 1), DIM == 2 ? F(wl.lam2, 2) : nullptr};
    T* l1[3] = {F(wl.lam1, 0), F(wl.lam1, 1), DIM == 2 ? F(wl.lam1, 2) : nullptr};
    T* lo[3] = {(T*)lam_u_out, (T*)lam_v_out, (T*)lam_w_out};
    const T* X2[3] = {F(x2, 0), F(x2, 1), DIM == 2 ? F(x2, 2) : nullptr};
    const T* X1[3] = {F(x1, 0), F(x1, 1), DIM == 2 ? F(x1, 2) : nullptr};
    const T* X0[3] = {(const T*)u_n, (const T*)v_n, (const T*)w_n};
    // lambda^(2) = vjp(X^(2); 2/3 lambda, 2/3 dt lambda)
    const void* lin[3] = {lam_u_in, lam_v_in, lam_w_in};
    Cot c3{};
    for (int f = 0; f < 3; ++f) c3.b[f] = c3.a[0][f] = lin[f];
    c3.cb = 2.0 / 3.0;
    c3.ca[0] = 2.0 / 3.0;
    c3.na = 1;
    if ((s2 = launch_vjp<Sys, T, DIM>(p, sy, g, wl, X2, c3, alpha_rec + 4, dt, l2, stream)) != HWENO_OK)
      return s2;
    // lambda^(1) = vjp(X^(1); 1/4 lambda^(2), 1/4 dt lambda^(2))
    Cot c2{};
    for (int f = 0; f < 3; ++f) c2.b[f] = c2.a[0][f] = l2[f];
    c2.cb = 0.25;
    c2.ca[0] = 0.25;
    c2.na = 1;
    if ((s2 = launch_vjp<Sys, T, DIM>(p, sy, g, wl, X1, c2, alpha_rec + 2, dt, l1, stream)) != HWENO_OK)
      return s2;
    // lambda^n = vjp(X^n; lambda^(1) + 3/4 lambda^(2) + 1/3 lambda, dt lambda^(1))
    Cot c1{};
    for (int f = 0; f < 3; ++f) {
      c1.b[f] = c1.a[0][f] = l1[f];
      c1.a[1][f] = l2[f];
      c1.a[2][f] = lin[f];
    }
    c1.cb = 1.0;
    c1.ca[0] = 1.0;
    c1.ca[1] = 0.75;
    c1.ca[2] = 1.0 / 3.0;
    c1.na = 3;
    return launch_vjp<Sys, T, DIM>(p, sy, g, wl, X0, c1, alpha_rec, dt, lo, stream);
  });
}

hweno_status hweno_health(const hweno_problem* p, void* ws, hipStream_t stream, int32_t clear) {
  hweno_status st = validate(p);
  if (st != HWENO_OK) return st;
  if (!ws) return HWENO_EINVAL;
  unsigned flags = 0;
  StepScalars* sc = (StepScalars*)ws;
  if (hipMemcpyAsync(&flags, &sc->flags, sizeof(unsigned), hipMemcpyDeviceToHost, stream) != hipSuccess)
    return HWENO_EDEVICE;
  if (hipStreamSynchronize(stream) != hipSuccess) return HWENO_EDEVICE;
  if (clear) {
    ws_init_kernel<<<1, kWave, 0, stream>>>(sc);
    if (check_launch() != HWENO_OK) return HWENO_EDEVICE;
    if (hipStreamSynchronize(stream) != hipSuccess) return HWENO_EDEVICE;
  }
  if (flags & 1u) return HWENO_ENONFINITE;
  if (flags & 2u) return HWENO_ENONPHYSICAL;
  return HWENO_OK;
}

}  // extern "C"
