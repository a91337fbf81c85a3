// Host-side launch interface of the gfx950 Kadanoff-Baym kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kbe_device.hpp"

#define KBE_DEV_INT_HUBBARD 0
#define KBE_DEV_INT_INTERBAND 1
#define KBE_DEV_NOBS 17
#define KBE_DEV_OBS_NORB 9
#define KBE_DEV_OBS_NBAND 13

#define KBE_ROW_PREDICT 0
#define KBE_ROW_CORRECT 1
#define KBE_ROW_EVAL 2
#define KBE_ROW_EVAL_NEXT 3   // EVAL of row m, then PREDICT of row m + 1

namespace kbe {

// Device pointers and scalars a launch needs (the roles *_prev / *_cur are resolved by
// the caller for the current step).
struct LaunchArgs {
  void* hist;      // packed history, FP64 (cplx) or FP32 (float2) elements
  cplx* row64;     // FP64 working copies of history rows m-1 and m
  cplx* sig;
  cplx* I_prev;
  cplx* I_cur;
  cplx* col0;
  cplx* diag;
  cplx* colpart;   // column sums of the history sums, per row segment: [k][cseg][C][Tp]
  cplx* rowpart;
  cplx* rho_prev;
  cplx* rho_cur;
  cplx* D_prev;
  cplx* D_cur;
  cplx* props;
  cplx* hfbuf;
  cplx* hop;
  double* eig_w;
  cplx* eig_U;
  double* mu;
  double* obs;
  int commit;      // 0: the row kernel writes only the FP64 working row (recomputation)
  double* chg;     // if set, the corrector row kernel writes max |G_new - G_old| of each of its blocks here
  cplx* gR;        // interband self-energy: real-space lines of row m, [t_j][comp][ab][R] (else null)
  QuadW quad;      // quadrature weights of eq. (CI)
  double Ax, Ay;  // A(t) * pol for the launch at hand
  double polx, poly;  // pulse polarisation
  double dt, U, UU, temp, target, spin;
  int interaction, hf, corr;
};

// The observables of one time slice: its index, time, pulse amplitude, density matrices and
// collision row.
struct ObsStep {
  int m;
  double t, A;
  const cplx *rho, *Icur;
};
// whether the observables of a step ride in the next step's first history pass (else in its
// propagator launch)
inline bool obs_in_pass(const Dims& d) { return d.nb <= 2; }

hipError_t launch_fill_zero(double* p, int64_t n, hipStream_t st);
hipError_t launch_init(const Dims& d, const LaunchArgs& a, hipStream_t st);
// mean field (into hfbuf) and propagators for the density (1 - wb) rho_prev + wb rho_cur; o (nb >= 3
// only): also the observables of that slice
hipError_t launch_props(const Dims& d, const LaunchArgs& a, double wb, const ObsStep* o, hipStream_t st);
hipError_t launch_sigma(const Dims& d, const LaunchArgs& a, int m, hipStream_t st);
// the paper's direct-sum self-energy (interband preset, chain with even n <= 1024)
hipError_t launch_sigma_direct(const Dims& d, const LaunchArgs& a, int m, hipStream_t st);
// the dipole kick on the completed slice m (nb = 2): the row's copies and rho_cur (and rho_other)
hipError_t launch_kick(const Dims& d, const LaunchArgs& a, int m, double kc, double ks, cplx* rho_other,
                       hipStream_t st);
// history sums of row m and the equal-time integral I(t_m, t_m), D_m; props: also what
// launch_props(d, *props, wb, nullptr, st) does; o (nb <= 2 only): also the observables of that slice
// (independent work in the same launch)
hipError_t launch_collide(const Dims& d, const LaunchArgs& a, int m, const LaunchArgs* props, double wb,
                          const ObsStep* o, hipStream_t st);
hipError_t launch_row(const Dims& d, const LaunchArgs& a, int m, int mode, hipStream_t st);
// launch_row(d, a, m, KBE_ROW_EVAL, st) and launch_row(d, next, m + 1, KBE_ROW_PREDICT, st) in one, m >= 1;
// next: I_prev and D_prev are a's I_cur and D_cur, the working rows the same
inline bool row_next_fused(const Dims& d) { return d.nb <= 2 && d.qp == 1; }
hipError_t launch_row_next(const Dims& d, const LaunchArgs& a, const LaunchArgs& next, int m, hipStream_t st);
// out[0] = max of the row kernel's per-block changes at row m (one block, deterministic)
hipError_t launch_change_max(const Dims& d, const double* chg, int m, double* out, hipStream_t st);
hipError_t launch_obs(const Dims& d, const LaunchArgs& a, const ObsStep& o, hipStream_t st);
hipError_t launch_aux(const Dims& d, const LaunchArgs& a, int m, hipStream_t st);

}  // namespace kbe
