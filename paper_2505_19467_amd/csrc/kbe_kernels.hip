// HIP kernels (gfx950) of the Kadanoff-Baym propagation step.
//
//   k_init_*        uncorrelated initial state (Fermi-Dirac density of h0, mu by bisection)
//   k_props         mean-field (first-order) self-energy from the local density matrix, and the
//                   per-k propagators V, Vh, Phi of the midpoint Hamiltonian
//   k_kick_row      the dipole kick of eq. (dipole) on the completed slice nearest t0
//   k_sigma         second-Born self-energy of a time slice, eq. (2BSE), by k <-> R transforms
//                   (Hubbard preset)
//   k_sigma_fwd/ib  the same for the interband preset: lines to real space, then products
//                   and back
//   k_sigma_direct  the paper's direct momentum sums for the interband preset (comparison)
//   k_hist_pair, k_hist_bulk(_split) and their FP32 forms
//                   the history sums of eq. (CI): stream the packed triangle of rows 0..m-1
//                   once, every stored block feeding its column and its row; in front of them
//                   the equal-time collision integral I^<(t_m, t_m) and D_m (and, in a corrector
//                   pass, the propagators), k_extras where there is no history yet
//   k_row           end-point terms (trapezoid or Gregory), collision row assembly,
//                   predictor/corrector update
//   k_change_max    the corrector's row change (stopping rule)
//   k_obs           observables of one time slice
//   k_aux           refresh the column / diagonal / recent-row copies of the history
#include "kbe_device.hpp"
#include "kbe_kernels.hpp"

namespace kbe {

// ------------------------------------------------------------------ utility
__global__ void k_fill_zero(double* __restrict__ p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0.0;
}

// Write one element of the packed history in its storage precision.
__device__ __forceinline__ void commit_store(const Dims& d, void* hist, int k, int c, int j, int tp, cplx v) {
  if (d.fp32)
    reinterpret_cast<float2*>(hist)[hist_idx(d, k, c, j, tp)] = make_float2((float)v.x, (float)v.y);
  else
    reinterpret_cast<cplx*>(hist)[hist_idx(d, k, c, j, tp)] = v;
}
__device__ __forceinline__ cplx history_load(const Dims& d, const void* hist, int k, int c, int j, int tp) {
  if (d.fp32) {
    float2 v = reinterpret_cast<const float2*>(hist)[hist_idx(d, k, c, j, tp)];
    return make_double2((double)v.x, (double)v.y);
  }
  return reinterpret_cast<const cplx*>(hist)[hist_idx(d, k, c, j, tp)];
}

// ------------------------------------------------------------------ initial state
// Eigen-decomposition of h0(k - A(0)) per k (one thread per k).
template <int NB>
__global__ __launch_bounds__(64) void k_init_eig(Dims d, const cplx* __restrict__ hop, double Ax, double Ay,
                                                 double* __restrict__ w, cplx* __restrict__ U) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.nk) return;
  cplx h[NB * NB], V[NB * NB];
  double ev[NB];
  bloch_h0<NB>(hop, d.nkx, d.nky, k, Ax, Ay, h);
  jacobi_eigh<NB>(h, ev, V);
#pragma unroll
  for (int b = 0; b < NB; ++b) w[k * NB + b] = ev[b];
#pragma unroll
  for (int i = 0; i < NB * NB; ++i) U[(int64_t)k * NB * NB + i] = V[i];
}

// Chemical potential by bisection: N_k^{-1} sum_{k,b} f((w - mu)/T) = target (one block).
__global__ __launch_bounds__(256) void k_init_mu(int n, const double* __restrict__ w, double temp,
                                                 double target, double* __restrict__ mu_out) {
  __shared__ double red[256];
  __shared__ double lohi[2], sum[1];
  int t = threadIdx.x;
  double lo = 1e300, hi = -1e300;
  for (int i = t; i < n; i += 256) {
    lo = fmin(lo, w[i]);
    hi = fmax(hi, w[i]);
  }
  red[t] = lo;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) red[t] = fmin(red[t], red[t + s]);
    __syncthreads();
  }
  if (t == 0) lohi[0] = red[0] - 50.0 * temp - 1.0;
  __syncthreads();
  red[t] = hi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) red[t] = fmax(red[t], red[t + s]);
    __syncthreads();
  }
  if (t == 0) lohi[1] = red[0] + 50.0 * temp + 1.0;
  __syncthreads();
  for (int it = 0; it < 200; ++it) {
    double mid = 0.5 * (lohi[0] + lohi[1]);
    double acc = 0.0;
    for (int i = t; i < n; i += 256) acc += 1.0 / (1.0 + exp((w[i] - mid) / temp));
    block_sum_once<1>(&acc, red, sum);
    if (t == 0) {
      if (sum[0] < target) lohi[0] = mid;
      else lohi[1] = mid;
    }
    __syncthreads();
    if (lohi[1] - lohi[0] < 1e-15 * fmax(1.0, fabs(mid))) break;
  }
  if (t == 0) *mu_out = 0.5 * (lohi[0] + lohi[1]);
}

// rho0 = U f(w - mu) U^dag; row 0 of the history (G^< = i rho, G^> = -i (1 - rho)).
template <int NB>
__global__ __launch_bounds__(64) void k_init_rho(Dims d, const double* __restrict__ w, const cplx* __restrict__ U,
                                                 const double* __restrict__ mu, double temp,
                                                 cplx* __restrict__ rhoA, cplx* __restrict__ rhoB,
                                                 void* __restrict__ hist, cplx* __restrict__ row64,
                                                 cplx* __restrict__ col0, cplx* __restrict__ diag) {
  constexpr int NBB = NB * NB;
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.nk) return;
  double f[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) f[b] = 1.0 / (1.0 + exp((w[k * NB + b] - *mu) / temp));
  const cplx* Uk = U + (int64_t)k * NBB;
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      cplx s = czero();
#pragma unroll
      for (int c = 0; c < NB; ++c) s = cadd(s, cscal(cmul(Uk[a * NB + c], cconj(Uk[b * NB + c])), f[c]));
      int e = a * NB + b;
      rhoA[(int64_t)k * NBB + e] = s;
      rhoB[(int64_t)k * NBB + e] = s;
      cplx g[2];
      g[0] = cmuli(s);
      g[1] = cneg(cmuli(csub(cmk(a == b ? 1.0 : 0.0, 0.0), s)));
#pragma unroll
      for (int sc = 0; sc < 2; ++sc) {
        int c = sc * NBB + e;
        commit_store(d, hist, k, c, 0, 0, g[sc]);
        row64[row64_idx(d, 0, k, c, 0)] = g[sc];
        col0[colq_idx(d, k, c, 0, 0)] = g[sc];
        diag[band_idx(d, k, c, 0, 0)] = g[sc];
      }
    }
}

// ------------------------------------------------------------------ observables
// One block of at least 256 threads. Bound by latency (the Bloch Hamiltonian, its velocities and a
// Jacobi diagonalisation per k, at most four k per thread); sums by wavefront, then over the four
// wavefronts in LDS. Inside kbe_step the block of step m rides in the next step's first history pass
// (nb <= 2) or propagator launch (nb = 3, 4, whose register need the history kernels should not have):
// alone it held the stream up 8 us (16 points) to 18 us (576 points, nb = 2) per step.
struct ObsArgs {
  const cplx *hop, *rho, *Icur;
  double* obs;
  double t, A, Ax, Ay, U, spin;
  int m, interaction, hf;
};
template <int N>
__device__ __forceinline__ void block_sum_waves(const double* v, double* lds /* [N][4] */, double* out) {
  const int t = threadIdx.x, w = t >> 6;
  double rt[1][N];
#pragma unroll
  for (int i = 0; i < N; ++i) rt[0][i] = v[i];
  reduce_rows<1>(rt);
  if ((t & 63) == 0 && w < 4)
#pragma unroll
    for (int i = 0; i < N; ++i) lds[4 * i + w] = rt[0][i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = (lds[4 * i] + lds[4 * i + 1]) + (lds[4 * i + 2] + lds[4 * i + 3]);
  __syncthreads();
}
template <int NB>
constexpr int obs_lds() {
  return 4 * (6 + 2 * NB);
}
template <int NB>
__device__ __forceinline__ void obs_block(const Dims& d, const ObsArgs& o, double* lds) {
  constexpr int NBB = NB * NB;
  constexpr int NV = 6 + 2 * NB;  // N, Ekin, Ehf, Ecorr, Jx, Jy, n_orb[NB], n_band[NB]
  const cplx* __restrict__ rho = o.rho;
  const int tid = threadIdx.x;
  const double inv = 1.0 / d.nk, U = o.U;
  // mean field of the local density matrix
  cplx hfm[NBB], ob[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) hfm[e] = ob[e] = czero();
  if (o.interaction == KBE_DEV_INT_HUBBARD) {
    double v[NB], loc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) v[a] = 0.0;
    for (int k = tid; k < d.nk && tid < 256; k += 256)
#pragma unroll
      for (int a = 0; a < NB; ++a) v[a] += rho[(int64_t)k * NBB + a * (NB + 1)].x;
    block_sum_waves<NB>(v, lds, loc);
    if (o.hf)
#pragma unroll
      for (int a = 0; a < NB; ++a) hfm[a * (NB + 1)] = cmk(U * (loc[a] * inv), 0.0);
  } else if constexpr (NB == 2) {
    double v[8], loc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.0;
    for (int k = tid; k < d.nk && tid < 256; k += 256)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const cplx r = rho[(int64_t)k * 4 + e];
        v[2 * e] += r.x;
        v[2 * e + 1] += r.y;
      }
    block_sum_waves<8>(v, lds, loc);
    ob[3] = cmk(-U, 0.0);
    if (o.hf) {
      hfm[0] = cmk(U * (loc[6] * inv), 0.0);
      hfm[3] = cmk(U * (loc[0] * inv), 0.0);
      hfm[1] = cscal(cmk(loc[2] * inv, loc[3] * inv), -U);
      hfm[2] = cscal(cmk(loc[4] * inv, loc[5] * inv), -U);
    }
  }
  double acc[NV], tot[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  for (int k = tid; k < d.nk && tid < 256; k += 256) {
    cplx r[NBB], h[NBB], v[NBB], Vv[NBB];
    double w[NB];
#pragma unroll
    for (int e = 0; e < NBB; ++e) r[e] = rho[(int64_t)k * NBB + e];
    bloch_h0<NB>(o.hop, d.nkx, d.nky, k, o.Ax, o.Ay, h);
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      acc[0] += r[a * NB + a].x;
      acc[6 + a] += r[a * NB + a].x;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        acc[1] += cmul(cadd(h[a * NB + b], ob[a * NB + b]), r[b * NB + a]).x;
        acc[2] += cmul(hfm[a * NB + b], r[b * NB + a]).x;
      }
      acc[3] += 0.5 * o.Icur[rowbuf_idx(d, k, a * NB + a, o.m)].y;  // Re(-i/2 I) = Im(I)/2
    }
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      bloch_vel<NB>(o.hop, d.nkx, d.nky, k, o.Ax, o.Ay, dir, v);
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[4 + dir] += cmul(v[a * NB + b], r[b * NB + a]).x;
    }
    jacobi_eigh<NB>(h, w, Vv);
#pragma unroll
    for (int bnd = 0; bnd < NB; ++bnd) {
      double sacc = 0.0;
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          sacc += cmul(cmul(cconj(Vv[a * NB + bnd]), r[a * NB + b]), Vv[b * NB + bnd]).x;
      acc[6 + NB + bnd] += sacc;
    }
  }
  block_sum_waves<NV>(acc, lds, tot);
  if (tid == 0) {
    double* out = o.obs + (int64_t)o.m * KBE_DEV_NOBS;
    for (int i = 0; i < KBE_DEV_NOBS; ++i) out[i] = 0.0;
    out[0] = o.t;
    out[1] = o.spin * tot[0] * inv;
    out[2] = o.spin * tot[1] * inv;
    out[3] = 0.5 * o.spin * tot[2] * inv;
    out[4] = o.spin * tot[3] * inv;
    out[5] = out[2] + out[3] + out[4];
    out[6] = o.spin * tot[4] * inv;
    out[7] = o.spin * tot[5] * inv;
    out[8] = o.A;
    for (int a = 0; a < NB; ++a) out[9 + a] = tot[6 + a] * inv;
    for (int b = 0; b < NB; ++b) out[13 + b] = tot[6 + NB + b] * inv;
  }
}
template <int NB>
__global__ __launch_bounds__(256) void k_obs(Dims d, ObsArgs o) {
  __shared__ double lds[obs_lds<NB>() > 32 ? obs_lds<NB>() : 32];
  obs_block<NB>(d, o, lds);
}

// ------------------------------------------------------------------ propagators
// Mean field and propagators of the midpoint Hamiltonian hbar = h0(k - A) + Sigma^HF[rho_loc],
// rho = (1 - wb) rhoA + wb rhoB. Bound by latency (a chain of 13 dependent matrix-vector products on
// nb x nb matrices); one lane carries one column of one k, so that the chain needs no exchange
// between lanes, and every block sums the local density by itself (N_k nb^2 numbers from the L2)
// instead of a launch of its own: 16 points 11.2 -> 4.0 us, 576 points 20.9 -> 6.6 us (nb = 2) for both,
// against one wavefront per k on the augmented 2nb x 2nb matrix with every product through LDS.
//
// Phi = -i dt phi1(X), V = exp(X), Vh = exp(X/2), X = -i hbar dt. phi1(X / 2^s) by its Taylor
// polynomial of degree 13 (||X / 2^s||_F <= 1/4: the rest is below 2e-19), exp = 1 + X phi1, then s >= 1
// squarings E(2X) = E^2, phi1(2X) = (E + 1) phi1 / 2; the square before the last gives Vh. nb = 1 keeps
// the augmented matrix's own recurrence of degree 16 (its two nontrivial entries).
//
// The one-body term beside h0 and the first-order self-energy of the local density sum loc:
// (loc: the real diagonal in the Hubbard preset, all (re, im) in the interband one)
template <int NB>
__device__ __forceinline__ cplx hf_element(const double* loc, int e, double inv, int interaction, int hf, double U) {
  cplx out = czero();
  if (interaction == KBE_DEV_INT_HUBBARD) {
    if (hf && e % (NB + 1) == 0) out = cmk(U * loc[e / (NB + 1)] * inv, 0.0);
  } else {
    // eq. (ham): -U c_c^dag c_c one-body term; Hartree U n_c / U n_v, Fock -U rho_vc
    if (e == NB * NB - 1) out = cmk(-U, 0.0);
    if constexpr (NB == 2) {
      if (hf) {
        if (e == 0 || e == 3) out.x += U * loc[2 * (3 - e)] * inv;
        else out = cscal(cmk(loc[2 * e], loc[2 * e + 1]), -U * inv);
      }
    }
  }
  return out;
}
template <int NB>
struct PropsShape {
  static constexpr int LPK = NB == 3 ? 4 : NB;   // lanes per k
  static constexpr int KPB = 256 / LPK;          // k per block
};
struct PropsArgs {
  const cplx *hop, *rhoA, *rhoB;
  cplx *hf_out, *props;
  double wb, U, Ax, Ay, dt;
  int interaction, hf;
};
// Block blk of the propagator blocks, any block of at least 256 threads; red: props_lds<NB>() doubles.
template <int NB>
constexpr int props_lds() {
  constexpr int sums = (NB == 2 ? 8 : NB) * 256, mats = 2 * NB * NB * PropsShape<NB>::KPB;
  return (NB == 1 || sums > mats ? sums : mats) + 4 * NB * NB;
}
template <int NB>
__device__ __forceinline__ void props_block(const Dims& d, const PropsArgs& x, int blk, double* red) {
  constexpr int NBB = NB * NB, LPK = PropsShape<NB>::LPK, KPB = PropsShape<NB>::KPB;
  double* loc = red + props_lds<NB>() - 4 * NBB;
  cplx* hfm = reinterpret_cast<cplx*>(loc + 2 * NBB);
  const cplx* __restrict__ rhoA = x.rhoA;
  const cplx* __restrict__ rhoB = x.rhoB;
  const double wb = x.wb, U = x.U, dt = x.dt;
  const int interaction = x.interaction, hf = x.hf;
  const int t = threadIdx.x;
  {
    // local density: the Hubbard field needs the real diagonal only; N_k <= 1024
    auto rho = [&](int i, int e) {
      const int k = t + 256 * i;
      if (k >= d.nk || t >= 256) return czero();
      const cplx a = rhoA[(int64_t)k * NBB + e];
      if (wb == 0.0) return a;
      return cadd(cscal(a, 1.0 - wb), cscal(rhoB[(int64_t)k * NBB + e], wb));
    };
    if (interaction == KBE_DEV_INT_HUBBARD) {
      double v[NB];
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        v[a] = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[a] += rho(i, a * (NB + 1)).x;
      }
      block_sum_once<NB>(v, red, loc);
    } else if constexpr (NB == 2) {
      double v[2 * NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        v[2 * e] = v[2 * e + 1] = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const cplx r = rho(i, e);
          v[2 * e] += r.x;
          v[2 * e + 1] += r.y;
        }
      }
      block_sum_once<2 * NBB>(v, red, loc);
    }
    if (t < NBB) {
      hfm[t] = hf_element<NB>(loc, t, 1.0 / d.nk, interaction, hf, U);
      if (blk == 0) x.hf_out[t] = hfm[t];
    }
    __syncthreads();
  }
  const int kl = t / LPK, c = t - kl * LPK;
  const int k = blk * KPB + kl;
  const bool act = t < 256 && k < d.nk && c < NB;
  cplx X[NBB];
  {
    cplx h[NBB];
    bloch_h0<NB>(x.hop, d.nkx, d.nky, act ? k : 0, x.Ax, x.Ay, h);
#pragma unroll
    for (int e = 0; e < NBB; ++e) X[e] = cscal(cmuli(cadd(h[e], hfm[e])), -dt);  // -i hbar dt
  }
  cplx* P = x.props + (int64_t)(act ? k : 0) * 3 * NBB;
  double nrm2 = 0.0;
#pragma unroll
  for (int e = 0; e < NBB; ++e) nrm2 += cabs2(X[e]);
  int s = 1;
  if constexpr (NB == 1) {
    // E = exp(M), M = [[X, dt], [0, 0]]: entries (0, 0) and (0, 1) of the Horner steps 1 + M E / n
    // and of the squarings
    double nrm = sqrt(nrm2 + dt * dt);
    while (nrm > ldexp(0.25, s) && s < 60) ++s;
    const double scale = ldexp(1.0, -s);
    const cplx xs = cscal(X[0], scale), y = cmk(dt * scale, 0.0), one = cmk(1.0, 0.0);
    cplx e0 = one, e1 = czero();
    for (int n = 16; n >= 1; --n) {
      cplx a0 = czero(), a1 = czero();
      cmac(a0, xs, e0);
      cmac(a1, xs, e1);
      cmac(a1, y, one);
      e0 = cadd(one, cscal(a0, 1.0 / n));
      e1 = cscal(a1, 1.0 / n);
    }
    cplx half = czero();
    for (int q = 0; q < s; ++q) {
      if (q == s - 1) half = e0;
      cplx a0 = czero(), a1 = czero();
      cmac(a0, e0, e0);
      cmac(a1, e0, e1);
      cmac(a1, e1, one);
      e0 = a0;
      e1 = a1;
    }
    if (act) {
      P[0] = e0;
      P[1] = half;
      P[2] = cneg(cmuli(e1));
    }
  } else {
    double nrm = sqrt(nrm2);
    while (nrm > ldexp(0.25, s) && s < 60) ++s;
    const double scale = ldexp(1.0, -s);
#pragma unroll
    for (int e = 0; e < NBB; ++e) X[e] = cscal(X[e], scale);
    cplx f[NB], E[NB];   // column c of phi1 and of exp
    auto mulX = [&](const cplx* v, cplx* out) {
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        out[r] = czero();
#pragma unroll
        for (int l = 0; l < NB; ++l) cmac(out[r], X[r * NB + l], v[l]);
      }
    };
#pragma unroll
    for (int r = 0; r < NB; ++r) f[r] = cmk(r == c ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int n = 13; n >= 1; --n) {
      cplx u[NB];
      mulX(f, u);
#pragma unroll
      for (int r = 0; r < NB; ++r) f[r] = cadd(cmk(r == c ? 1.0 : 0.0, 0.0), cscal(u[r], 1.0 / (n + 1)));
    }
    mulX(f, E);
#pragma unroll
    for (int r = 0; r < NB; ++r) E[r].x += r == c ? 1.0 : 0.0;
    cplx* sE = reinterpret_cast<cplx*>(red) + kl * NBB;   // exp of this k, columns from its lanes (one wavefront)
    const int smax = wave_max(act ? s : 0);
    for (int q = 0; q < smax; ++q) {
      if (act)
#pragma unroll
        for (int r = 0; r < NB; ++r) sE[r * NB + c] = E[r];
      wave_sync();
      if (act && q < s) {
        if (q == s - 1)
#pragma unroll
          for (int r = 0; r < NB; ++r) P[NBB + r * NB + c] = E[r];   // Vh
        cplx e2[NB], f2[NB];
#pragma unroll
        for (int r = 0; r < NB; ++r) {
          e2[r] = f2[r] = czero();
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            const cplx el = sE[r * NB + l];
            cmac(e2[r], el, E[l]);
            cmac(f2[r], el, f[l]);
          }
        }
#pragma unroll
        for (int r = 0; r < NB; ++r) {
          E[r] = e2[r];
          f[r] = cscal(cadd(f2[r], f[r]), 0.5);
        }
      }
      wave_sync();
    }
    if (act)
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        P[r * NB + c] = E[r];                                          // V
        P[2 * NBB + r * NB + c] = cneg(cmuli(cscal(f[r], dt)));        // Phi
      }
  }
}
// the last block (nobs = 1): the observables of the step before (nb >= 3)
template <int NB>
__global__ __launch_bounds__(256) void k_props(Dims d, PropsArgs x, ObsArgs o, int nobs) {
  __shared__ double red[props_lds<NB>()];
  if constexpr (NB >= 3)
    if (nobs && blockIdx.x + 1 == gridDim.x) {
      obs_block<NB>(d, o, red);
      return;
    }
  props_block<NB>(d, x, blockIdx.x, red);
}

// ------------------------------------------------------------------ self-energy
// One block per (t_j, orbital pair ab) of row m. With plain index transforms
//   g(R) = N_k^{-1} sum_j e^{+2 pi i j.R / n} G(k_j),   S(k_j) = sum_R e^{-2 pi i j.R / n} S(R),
// the -pi offset of eq. (kj) cancels in the product of two forward lines and one backward
// line, and the backward line is g_ba(-R; t_j, t_m) = -conj(g_ab(R; t_m, t_j)), so
//   Hubbard:  Sigma^<_ab(R) = -U^2 g^<_ab(R)^2 conj(g^>_ab(R)),  Sigma^> with < and > swapped.
// Block-to-work mapping gives each XCD a contiguous range of t_j, so the cache lines of
// row m that several t_j share stay in one L2. NX, NY > 0: the grid size is fixed at compile
// time (unrolled transforms, 1.8x faster on 24 x 24); NX = NY = 0: any grid, sizes from d.
// Dynamic LDS: four lines of N_k points and the nx + ny roots of unity.
// Threads per block: 256, or as many as the larger stage of a compile-time transform has items where
// that is more (24 x 24: 288 -> 320 threads, 24.2 -> 22.9 us at m <= 300; with fewer than 256 on the small
// grids the loads have too few wavefronts: 12 x 12 10.2 -> 10.9 us with 128). Any other grid takes 512
// threads from 512 points on (a block's LDS leaves room for one to three such blocks per CU: at 1024
// points 105 -> 58 and 118 -> 69 us for the two interband kernels with the in-place transform), else 256.
template <int NX, int NY>
constexpr int sigma_threads() {
  if (NX == 0) return 512;
  int items = 2 * NY * (NX / fft_split_ct(NX > 0 ? NX : 4));
  if (NY > 1 && 2 * NX * (NY / fft_split_ct(NY)) > items) items = 2 * NX * (NY / fft_split_ct(NY));
  return items > 256 ? (items + 63) / 64 * 64 : 256;
}
// U (run-time grids): terms of a chain whose LDS reads are in flight, 4 or 2. Four take 116 registers (four
// wavefronts per SIMD), two take 90 (five): the launch takes two where that saves it a round of the chip
// (1025..1280 blocks of 256 threads and so on: 9 x 7, m = 280 17.2 -> 12.8 us, 128 points 13.8 -> 11.1), else
// four (64 points, m = 255 / 400 12.1 -> 11.5, 22.2 -> 20.3 us).
template <int NB, int NX, int NY, int U = 4>
__global__ __launch_bounds__((sigma_threads<NX, NY>())) void k_sigma(Dims d, const cplx* __restrict__ row64, cplx* __restrict__ sig,
                                               int m, double UU, int corr) {
  constexpr int NBB = NB * NB;
  extern __shared__ cplx lds[];
  const int nk = NX > 0 ? NX * NY : d.nk;
  const int nx = NX > 0 ? NX : d.nkx, ny = NX > 0 ? NY : d.nky;
  cplx* gl = lds;
  cplx* gg = lds + nk;
  // two lines and their scratch (a long power-of-two chain needs none)
  const int lines = NX == 0 && pow2_chain(nx, ny) ? 2 : 4;
  cplx* tl = lds + (lines - 2) * nk;
  cplx* tg = lds + (lines - 1) * nk;
  cplx* twx = lds + lines * nk;  // roots of unity, nx and ny entries
  cplx* twy = twx + nx;
  int total = (m + 1) * NBB;
  int per = (total + 7) >> 3;
  int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (item >= total) return;
  int j = item / NBB, ab = item - (item / NBB) * NBB;
  const int t = threadIdx.x, nt = NX > 0 ? sigma_threads<NX, NY>() : blockDim.x;
  // at most two points a thread; the roots are made while the loads are in flight
  cplx vl[2], vg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = t + i * nt < nk ? t + i * nt : nk - 1;
    vl[i] = row64[row64_idx(d, m, k, ab, j)];
    vg[i] = row64[row64_idx(d, m, k, NBB + ab, j)];
  }
  fill_roots(twx, nx);
  fill_roots(twy, ny);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (t + i * nt < nk) {
      gl[t + i * nt] = vl[i];
      gg[t + i * nt] = vg[i];
    }
  __syncthreads();
  // k -> R (1/N_k)
  if constexpr (NX > 0)
    grid_dft_ct<NX, NY, sigma_threads<NX, NY>()>(gl, gg, tl, tg, twx, twy, +1, 1.0 / nk);
  else
    grid_dft<U>(d, gl, gg, tl, tg, twx, twy, +1, 1.0 / nk);
  for (int o = t; o < nk; o += nt) {
    cplx al = gl[o], ag = gg[o];
    cplx sl = czero(), sg = czero();
    if (corr) {
      sl = cscal(cmul(cmul(al, al), cconj(ag)), -UU);
      sg = cscal(cmul(cmul(ag, ag), cconj(al)), -UU);
    }
    gl[o] = sl;
    gg[o] = sg;
  }
  __syncthreads();
  // R -> k
  if constexpr (NX > 0)
    grid_dft_ct<NX, NY, sigma_threads<NX, NY>()>(gl, gg, tl, tg, twx, twy, -1, 1.0);
  else
    grid_dft<U>(d, gl, gg, tl, tg, twx, twy, -1, 1.0);
  for (int o = t; o < nk; o += nt) {
    cplx al = gl[o], ag = gg[o];
    sig[sig_idx(d, o, 0, ab, j)] = al;
    sig[sig_idx(d, o, 1, ab, j)] = ag;
    sig[sig_idx(d, o, 2, ab, j)] = csub(ag, al);
  }
}

// Interband preset (nb = 2, the paper's eq. (2BSE)): with jbar the other band,
//   Sigma^<_ab(R) = -U^2 (-1)^(a+b) det g^<(R) conj(g^>_{abar bbar}(R)),  Sigma^> with < and > swapped,
// (the direct minus the exchange term of eq. (2BSE): g_{abar bbar} g_ab - g_{a bbar} g_{abar b} is
// (-1)^(a+b) det g; the backward line is -conj of the forward one, as for the Hubbard preset).
// Each output needs all four orbital pairs of both components at R, so the transforms are split
// around a real-space buffer gR[t_j][comp][ab][R]: k_sigma_fwd takes the lines of row m to R,
// k_sigma_ib forms the products and takes them back to k. Both: one block per (t_j, ab), the
// same XCD-aware mapping and LDS tile as k_sigma.
__device__ __forceinline__ int64_t gr_idx(const Dims& d, int j, int comp, int ab, int R) {
  return (((int64_t)j * 2 + comp) * 4 + ab) * d.nk + R;
}
template <int NX, int NY, int U = 4>
__global__ __launch_bounds__((sigma_threads<NX, NY>())) void k_sigma_fwd(Dims d, const cplx* __restrict__ row64, cplx* __restrict__ gR,
                                                   int m) {
  extern __shared__ cplx lds[];
  const int nk = NX > 0 ? NX * NY : d.nk;
  const int nx = NX > 0 ? NX : d.nkx, ny = NX > 0 ? NY : d.nky;
  cplx* gl = lds;
  cplx* gg = lds + nk;
  // two lines and their scratch (a long power-of-two chain needs none)
  const int lines = NX == 0 && pow2_chain(nx, ny) ? 2 : 4;
  cplx* tl = lds + (lines - 2) * nk;
  cplx* tg = lds + (lines - 1) * nk;
  cplx* twx = lds + lines * nk;
  cplx* twy = twx + nx;
  int total = (m + 1) * 4;
  int per = (total + 7) >> 3;
  int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (item >= total) return;
  int j = item >> 2, ab = item & 3;
  const int t = threadIdx.x, nt = NX > 0 ? sigma_threads<NX, NY>() : blockDim.x;
  // at most two points a thread; the roots are made while the loads are in flight
  cplx vl[2], vg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = t + i * nt < nk ? t + i * nt : nk - 1;
    vl[i] = row64[row64_idx(d, m, k, ab, j)];
    vg[i] = row64[row64_idx(d, m, k, 4 + ab, j)];
  }
  fill_roots(twx, nx);
  fill_roots(twy, ny);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (t + i * nt < nk) {
      gl[t + i * nt] = vl[i];
      gg[t + i * nt] = vg[i];
    }
  __syncthreads();
  if constexpr (NX > 0)
    grid_dft_ct<NX, NY, sigma_threads<NX, NY>()>(gl, gg, tl, tg, twx, twy, +1, 1.0 / nk);
  else
    grid_dft<U>(d, gl, gg, tl, tg, twx, twy, +1, 1.0 / nk);
  for (int o = t; o < nk; o += nt) {
    gR[gr_idx(d, j, 0, ab, o)] = gl[o];
    gR[gr_idx(d, j, 1, ab, o)] = gg[o];
  }
}
template <int NX, int NY, int U = 4>
__global__ __launch_bounds__((sigma_threads<NX, NY>())) void k_sigma_ib(Dims d, const cplx* __restrict__ gR, cplx* __restrict__ sig,
                                                  int m, double UU, int corr) {
  extern __shared__ cplx lds[];
  const int nk = NX > 0 ? NX * NY : d.nk;
  const int nx = NX > 0 ? NX : d.nkx, ny = NX > 0 ? NY : d.nky;
  cplx* sl = lds;
  cplx* sg = lds + nk;
  // two lines and their scratch (a long power-of-two chain needs none)
  const int lines = NX == 0 && pow2_chain(nx, ny) ? 2 : 4;
  cplx* tl = lds + (lines - 2) * nk;
  cplx* tg = lds + (lines - 1) * nk;
  cplx* twx = lds + lines * nk;
  cplx* twy = twx + nx;
  int total = (m + 1) * 4;
  int per = (total + 7) >> 3;
  int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (item >= total) return;
  int j = item >> 2, ab = item & 3;
  int a = ab >> 1, b = ab & 1;
  int cross = (1 - a) * 2 + (1 - b);                 // orbital pair (abar, bbar)
  double pre = ((a + b) & 1) ? UU : -UU;             // -U^2 (-1)^(a+b)
  const int t = threadIdx.x, nt = NX > 0 ? sigma_threads<NX, NY>() : blockDim.x;
  fill_roots(twx, nx);
  fill_roots(twy, ny);
  for (int o = t; o < nk; o += nt) {
    cplx l00 = gR[gr_idx(d, j, 0, 0, o)], l01 = gR[gr_idx(d, j, 0, 1, o)];
    cplx l10 = gR[gr_idx(d, j, 0, 2, o)], l11 = gR[gr_idx(d, j, 0, 3, o)];
    cplx g00 = gR[gr_idx(d, j, 1, 0, o)], g01 = gR[gr_idx(d, j, 1, 1, o)];
    cplx g10 = gR[gr_idx(d, j, 1, 2, o)], g11 = gR[gr_idx(d, j, 1, 3, o)];
    cplx dl = csub(cmul(l00, l11), cmul(l01, l10));
    cplx dg = csub(cmul(g00, g11), cmul(g01, g10));
    cplx lx = gR[gr_idx(d, j, 0, cross, o)], gx = gR[gr_idx(d, j, 1, cross, o)];
    sl[o] = corr ? cscal(cmul(dl, cconj(gx)), pre) : czero();
    sg[o] = corr ? cscal(cmul(dg, cconj(lx)), pre) : czero();
  }
  __syncthreads();
  if constexpr (NX > 0)
    grid_dft_ct<NX, NY, sigma_threads<NX, NY>()>(sl, sg, tl, tg, twx, twy, -1, 1.0);
  else
    grid_dft<U>(d, sl, sg, tl, tg, twx, twy, -1, 1.0);
  for (int o = t; o < nk; o += nt) {
    cplx vl = sl[o], vg = sg[o];
    sig[sig_idx(d, o, 0, ab, j)] = vl;
    sig[sig_idx(d, o, 1, ab, j)] = vg;
    sig[sig_idx(d, o, 2, ab, j)] = csub(vg, vl);
  }
}

// The paper's own evaluation of eq. (2BSE) for the interband preset on a chain (n divisible by
// 8): the direct term through the polarizability of eq. (polarizability)/(kernel2), O(n^2) per
// (t_j, jm), and the exchange term by the nested momentum sums of Alg. "contraction2",
// O(n^3) per (t_j, jm); kept beside the transform route to time the paper's algorithm on this
// hardware (same output). Momenta on the -pi-offset grid of eq. (kj): k_a + k_b has index
// a + b - n/2 and k_a - k_b index a - b + n/2 (mod n), so k' + q - k has index k' + q - k.
// One block per (t_j, jm) of row m, both components in turn; 512 threads in 4 groups that split
// the q range (8 waves per CU: the 96 KB of LDS leave room for one block). In a group thread i
// owns the KD = 8 outputs k = 8i .. 8i+7 (n <= 1024) and slides a window of KD backward-line
// values along k', so one LDS read feeds KD complex multiply-adds; neighbouring lanes then read
// the backward line 8 elements apart, so it is stored with one pad element after every 8 (lane
// stride 36 banks). The groups' partial sums are added in LDS in a fixed order.
// Dynamic LDS: the four forward lines of the component, P, the padded backward line:
// 6n + n/8 complex.
constexpr int KD = 8, DG = 4;
__device__ __forceinline__ int wrap_n(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }
__device__ __forceinline__ int padded(int x) { return x + (x >> 3); }
__global__ __launch_bounds__(512) void k_sigma_direct(Dims d, const cplx* __restrict__ row64, cplx* __restrict__ sig,
                                                      int m, double UU, int corr) {
  extern __shared__ cplx lds[];
  const int n = d.nk, h = n / 2;
  cplx* Ajm = lds;           // G^s_{j m}     (t_m, t_j)
  cplx* Abb = lds + n;       // G^s_{jb mb}
  cplx* Ajb = lds + 2 * n;   // G^s_{j mb}
  cplx* Abm = lds + 3 * n;   // G^s_{jb m}
  cplx* P = lds + 4 * n;
  cplx* Bk = lds + 5 * n;    // G^{s'}_{mb jb}(k; t_j, t_m) = -conj(G^{s'}_{jb mb}(k; t_m, t_j)), padded
  int item = blockIdx.x;     // (t_j, jm)
  int j = item >> 2, ab = item & 3;
  int a = ab >> 1, b = ab & 1, ja = 1 - a, mb = 1 - b;
  int t = threadIdx.x;
  int g = t >> 7, k0 = (t & 127) * KD;
  int q0 = g * (n / DG), q1 = q0 + n / DG;
  cplx outv[2][KD];
  const double pre = UU / ((double)n * (double)n);
  for (int s = 0; s < 2; ++s) {
    __syncthreads();
    for (int k = t; k < n; k += 512) {
      Ajm[k] = row64[row64_idx(d, m, k, s * 4 + a * 2 + b, j)];
      Abb[k] = row64[row64_idx(d, m, k, s * 4 + ja * 2 + mb, j)];
      Ajb[k] = row64[row64_idx(d, m, k, s * 4 + a * 2 + mb, j)];
      Abm[k] = row64[row64_idx(d, m, k, s * 4 + ja * 2 + b, j)];
      Bk[padded(k)] = cneg(cconj(row64[row64_idx(d, m, k, (1 - s) * 4 + ja * 2 + mb, j)]));
    }
    __syncthreads();
    // polarizability P(q) = sum_k' G_{jb mb}(k' + q) G_{mb jb}(k'; t_j, t_m)
    for (int q = t; q < n; q += 512) {
      cplx acc = czero();
      int idx = wrap_n(q - h, n);
      for (int kp = 0; kp < n; ++kp) {
        cmac(acc, Abb[idx], Bk[padded(kp)]);
        idx = idx + 1 == n ? 0 : idx + 1;
      }
      P[q] = acc;
    }
    __syncthreads();
    cplx part[KD];
#pragma unroll
    for (int r = 0; r < KD; ++r) part[r] = czero();
    if (k0 < n) {
      cplx dir[KD], ex[KD];
#pragma unroll
      for (int r = 0; r < KD; ++r) dir[r] = ex[r] = czero();
      // direct: sum_q G_{jm}(k - q) P(q), this group's q
      for (int q = q0; q < q1; ++q) {
        cplx pq = P[q];
#pragma unroll
        for (int r = 0; r < KD; ++r)
          if (k0 + r < n) cmac(dir[r], Ajm[wrap_n(k0 + r - q + h, n)], pq);
      }
      // exchange: sum_q G_{jb m}(q) sum_k' G_{j mb}(k') G_{mb jb}(k' + q - k; t_j, t_m)
      for (int q = q0; q < q1; ++q) {
        cplx acc[KD], w[KD];
        int base = q - k0;  // window element r at k' is Bk[k' + base - r]
#pragma unroll
        for (int r = 0; r < KD; ++r) {
          acc[r] = czero();
          w[r] = Bk[padded(wrap_n(base - r, n))];
        }
        int idx = wrap_n(base, n);
        for (int kp = 0; kp < n; kp += KD) {  // unrolled by the window length: the shifts are renames
#pragma unroll
          for (int u = 0; u < KD; ++u) {
            cplx av = Ajb[kp + u];
#pragma unroll
            for (int r = 0; r < KD; ++r) cmac(acc[r], av, w[r]);
#pragma unroll
            for (int r = KD - 1; r > 0; --r) w[r] = w[r - 1];
            idx = idx + 1 == n ? 0 : idx + 1;
            w[0] = Bk[padded(idx)];
          }
        }
        cplx cq = Abm[q];
#pragma unroll
        for (int r = 0; r < KD; ++r) cmac(ex[r], cq, acc[r]);
      }
#pragma unroll
      for (int r = 0; r < KD; ++r) part[r] = csub(dir[r], ex[r]);
    }
    // add the 4 groups' partial sums (in the forward-line area, no longer read)
    __syncthreads();
    if (k0 < n) {
#pragma unroll
      for (int r = 0; r < KD; ++r)
        if (k0 + r < n) lds[g * n + k0 + r] = part[r];
    }
    __syncthreads();
    if (g == 0 && k0 < n) {
#pragma unroll
      for (int r = 0; r < KD; ++r) {
        int k = k0 + r;
        cplx v = czero();
        if (k < n) v = cadd(cadd(lds[k], lds[n + k]), cadd(lds[2 * n + k], lds[3 * n + k]));
        outv[s][r] = corr ? cscal(v, pre) : czero();
      }
    }
  }
  if (g == 0 && k0 < n) {
#pragma unroll
    for (int r = 0; r < KD; ++r) {
      int k = k0 + r;
      if (k < n) {
        sig[sig_idx(d, k, 0, ab, j)] = outv[0][r];
        sig[sig_idx(d, k, 1, ab, j)] = outv[1][r];
        sig[sig_idx(d, k, 2, ab, j)] = csub(outv[1][r], outv[0][r]);
      }
    }
  }
}

// ------------------------------------------------------------------ equal-time collision
// I^<(t_m, t_m) = dt sum_j a_j [Sigma^>_mj G^<_jm - Sigma^<_mj G^>_jm],  G_jm = -(G_mj)^dag
// for j < m, a_j the quadrature weights on [0, t_m] (trapezoid, or with Gregory end
// corrections); I^>(t_m, t_m) is the same matrix (both integrals of eq. (CI) run over
// [0, t_m] and combine term by term). One block of at least 256 threads per k.
// Thread (row a, j) of 256: NB complex sums of one row each.
template <int NB>
constexpr int diag_lds() {
  return 2 * NB * 256;
}
template <int NB>
__device__ __forceinline__ void diag_block(const Dims& d, const cplx* __restrict__ row64, const cplx* __restrict__ sig,
                                           cplx* __restrict__ Icur, cplx* __restrict__ Dcur, int m, double dt,
                                           const QuadW& Q, int k, double* lds) {
  constexpr int NBB = NB * NB, RP = PropsShape<NB>::LPK, JT = 256 / RP;   // rows (padded), j per round
  const int t = threadIdx.x, a = t / JT;
  cplx acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = czero();
  if (m > 0 && a < NB && t < 256) {
    for (int j = t - a * JT; j <= m; j += JT) {
      const double wgt = quad_w(Q, j, m);
      cplx u[NB], v[NB], Sl[NB], Sg[NB];
#pragma unroll
      for (int l = 0; l < NB; ++l) {
        Sl[l] = sig[sig_idx(d, k, 0, a * NB + l, j)];
        Sg[l] = sig[sig_idx(d, k, 1, a * NB + l, j)];
        u[l] = v[l] = czero();
      }
      // j < m: G_jm = -G_mj^dag, so Sg G^<_jm - Sl G^>_jm = Sl Gg^dag - Sg Gl^dag;
      // j = m: the stored equal-time block, Sg Gl - Sl Gg.
      if (j < m) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            cmacc(u[b], Sl[l], row64[row64_idx(d, m, k, NBB + b * NB + l, j)]);
            cmacc(v[b], Sg[l], row64[row64_idx(d, m, k, b * NB + l, j)]);
          }
      } else {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            cmac(u[b], Sg[l], row64[row64_idx(d, m, k, l * NB + b, j)]);
            cmac(v[b], Sl[l], row64[row64_idx(d, m, k, NBB + l * NB + b, j)]);
          }
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[b] = cadd(acc[b], cscal(csub(u[b], v[b]), wgt));
    }
  }
  // sums over the JT threads of a row
  if (t < 256)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      lds[(2 * b) * 256 + t] = acc[b].x;
      lds[(2 * b + 1) * 256 + t] = acc[b].y;
    }
  __syncthreads();
  const int lane = t & 63;
  for (int i = t >> 6; i < 2 * NBB; i += blockDim.x >> 6) {
    const int r = i / (2 * NB), q = i - r * 2 * NB;   // row, real/imaginary part of column q / 2
    const double* x = lds + q * 256 + r * JT + lane;
    double v;
    if constexpr (JT == 256) v = (x[0] + x[128]) + (x[64] + x[192]);
    else if constexpr (JT == 128) v = x[0] + x[64];
    else v = x[0];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    // the sum's own place in LDS is read by no other wavefront
    if (lane == 0) lds[q * 256 + r * JT] = v;
  }
  __syncthreads();
  if (t < NBB) {
    const int r = t / NB, b = t - r * NB;
    auto sum = [&](int i, int j) { return cmk(lds[2 * j * 256 + i * JT], lds[(2 * j + 1) * 256 + i * JT]); };
    const cplx I = cscal(sum(r, b), dt);
    Icur[rowbuf_idx(d, k, t, m)] = I;
    Icur[rowbuf_idx(d, k, NBB + t, m)] = I;
    Dcur[(int64_t)k * NBB + t] = cadd(I, cconj(cscal(sum(b, r), dt)));
  }
}

// Blocks that ride in front of a history pass's own, on work that is independent of it: the
// equal-time integral of each k, in a corrector pass the propagators of the iterate, in an evaluation
// pass those of the next step's predictor (from the row's own density, final by then), and in a
// step's first pass the observables of the step before. They are a few microseconds of latency and
// N_k, N_k nb / 256 (propagators) and one block; in launches of their own they held up the stream
// 5 and 4-7 us per pass and 8-18 us per step.
struct PassExtras {
  const cplx *row64, *sig;
  cplx *Icur, *Dcur;
  double dt;
  QuadW Q;
  int m, nprops;      // nprops: propagator blocks (0: none)
  PropsArgs props;
  int nobs;           // 1: the observables of the step before (nb <= 2)
  ObsArgs obs;
  __host__ __device__ int blocks(const Dims& d) const { return nobs + nprops + d.nk; }
};
template <int NB>
constexpr int extras_lds() {
  return props_lds<NB>() > diag_lds<NB>() ? props_lds<NB>() : diag_lds<NB>();
}
template <int NB>
__device__ __forceinline__ void extras_block(const Dims& d, const PassExtras& x, int blk, void* lds) {
  double* w = reinterpret_cast<double*>(lds);
  if constexpr (NB <= 2) {
    if (blk < x.nobs) {
      obs_block<NB>(d, x.obs, w);
      return;
    }
    blk -= x.nobs;
  }
  if (blk < x.nprops) props_block<NB>(d, x.props, blk, w);
  else diag_block<NB>(d, x.row64, x.sig, x.Icur, x.Dcur, x.m, x.dt, x.Q, blk - x.nprops, w);
}
template <int NB>
__global__ __launch_bounds__(256) void k_extras(Dims d, PassExtras x) {
  __shared__ double lds[extras_lds<NB>()];
  extras_block<NB>(d, x, blockIdx.x, lds);
}

// ------------------------------------------------------------------ history sums (hot loop)
typedef float kbe_f4v __attribute__((ext_vector_type(4)));
// two complex64 values (a component pair of one column) in one 16-byte load
__device__ __forceinline__ void load_stream32x2(const float2* p, float2& a, float2& b) {
  kbe_f4v v = __builtin_nontemporal_load(reinterpret_cast<const kbe_f4v*>(p));
  a = make_float2(v.x, v.y);
  b = make_float2(v.z, v.w);
}

typedef float2 cplx32;
__device__ __forceinline__ void cmac32(cplx32& acc, cplx32 a, cplx32 b) {
  acc.x = fmaf(a.x, b.x, acc.x);
  acc.x = fmaf(-a.y, b.y, acc.x);
  acc.y = fmaf(a.x, b.y, acc.y);
  acc.y = fmaf(a.y, b.x, acc.y);
}
__device__ __forceinline__ void cmacc32(cplx32& acc, cplx32 a, cplx32 b) {  // acc += a conj(b)
  acc.x = fmaf(a.x, b.x, acc.x);
  acc.x = fmaf(a.y, b.y, acc.x);
  acc.y = fmaf(a.y, b.x, acc.y);
  acc.y = fmaf(-a.x, b.y, acc.y);
}
__device__ __forceinline__ cplx32 to32(cplx v) { return make_float2((float)v.x, (float)v.y); }
__device__ __forceinline__ float rs_half32(float a, float b) {
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                            false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float rs_row32(float a, float b) {
  auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                            false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_sum32(float x) {
  x += dpp_f<0xB1>(x);
  x += dpp_f<0x4E>(x);
  x += dpp_f<0x141>(x);
  x += dpp_f<0x140>(x);
  return x;
}

template <int R, int Q>
__device__ __forceinline__ void reduce_rows32(float (&rt)[R][Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    float y;
    if constexpr (R == 4) {
      y = rs_row32(rs_half32(rt[0][q], rt[1][q]), rs_half32(rt[2][q], rt[3][q]));
    } else if constexpr (R == 2) {
      float x = rs_half32(rt[0][q], rt[1][q]);
      y = rs_row32(x, x);
    } else {
      float x = rs_half32(rt[0][q], rt[0][q]);
      y = rs_row32(x, x);
    }
    rt[0][q] = row16_sum32(y);
  }
}
// The FP64 nb = 4 kernel's two component halves stage the row partials of the same 16 rows;
// after a block barrier each of the two wavefronts stores half of the nb^2 components of their sum
// (st0 + st1, a fixed order) to rows rb .. rb + 15 of the strip's slot, 256-byte runs.
template <int NBB>
__device__ __forceinline__ void flush_rows_fold(const cplx* st0, const cplx* st1, cplx* rp, int Tp, int rb, int m,
                                                int lane, int h) {
#pragma unroll
  for (int q = lane; q < NBB * 8; q += 64) {
    int e = h * (NBB / 2) + (q >> 4), r = q & 15;
    int row = rb + r;
    if (row < m) store_stream(rp + (int64_t)e * Tp + row, cadd(st0[e * 16 + r], st1[e * 16 + r]));
  }
}
// The FP32 nb = 4 kernel's two component halves stage the row partials of a 32-row chunk (rows
// cb .. cb + 31, both wave pairs); after a block barrier the whole block stores their sum
// (st0 + st1, a fixed order) to the strip's slot, one 512-byte run per component.
template <int NBB>
__device__ __forceinline__ void flush_chunk_fold(const cplx* st0, const cplx* st1, cplx* rp, int Tp, int cb, int m) {
  for (int q = threadIdx.x; q < NBB * 32; q += 256) {
    const int e = q >> 5, r = q & 31, row = cb + r;
    if (row < m) store_stream(rp + (int64_t)e * Tp + row, cadd(st0[e * 32 + r], st1[e * 32 + r]));
  }
}

// Bulk of the collision integrals at row m over the stored blocks (j, t'), t' <= j <= m-1,
// each with weight 1 (end-point weights are corrected in k_row):
//   column term -> output t':  SR_j G^{<,>}_{j t'}                    (SR = Sigma^> - Sigma^<)
//   row term    -> output j:   -Sigma^>_{t'} (G^<_{j t'})^dag + Sigma^<_{t'} (G^>_{j t'})^dag,
//                               t' < j, shared by I^< and I^>    (G_{t' j} = -G_{j t'}^dag)
// nb <= 2, FP64. Block = (pair of 64-column strips 2 sp, 2 sp + 1; k), the pairs with the
// most rows launched first, and a segment of their rows. Lane l owns columns 128 sp + l and
// 128 sp + 64 + l and keeps both column sums in registers; the Sigma of its two columns (row term)
// sits in LDS. Of the WAVES wavefronts w takes rows w, w + WAVES, ... of every 64-row chunk (so a
// chunk cut short by m leaves no wavefront idle while the others finish), R rows per iteration (R = 1 at nb = 2: 2 x 8 loads
// of 1 KB-contiguous data in flight; R = 4 at nb = 1), so every stored block is read from HBM
// once. The row terms of the two strips are added before the 64-lane
// reduce-scatter (at nb = 2 the four components of the row term share one reduce-scatter as
// four groups), so one row partial covers 128 columns: the writes that interleave with the
// read stream are half of what one strip per block would produce, and they leave in long runs
// (the block's rows of four 64-row chunks staged in LDS, then stored by all its threads as
// contiguous 4 KB runs per component, streaming stores). Both measures keep the read stream
// from stalling on scattered write-backs. Row partials go to slot sp; the wavefronts' column
// sums are combined in LDS, a share of the components by each. Deterministic: no atomics.
template <int NB, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_hist_pair(Dims d, const cplx* __restrict__ hist,
                                                   const cplx* __restrict__ sig, cplx* __restrict__ colpart,
                                                   cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr int R = NB == 1 ? 4 : 1;
  // row partials of the last ROWS_ST rows (4 chunks of 64), stored by the whole block at once
  constexpr int ROWS_ST = 256;
  constexpr int RSTEP = WAVES;              // a wavefront's rows are RSTEP apart
  constexpr int RPC = 64 / WAVES;           // its rows per 64-row chunk
  struct Rows {
    cplx stg[NBB][ROWS_ST];
    cplx sS[2][2][NBB][64];  // [strip of the pair][Sigma^<, Sigma^>][e][lane]
  };
  union Shared {
    Rows r;
    cplx red[WAVES][C][64];  // column sums of one strip, after the row loop
  };
  __shared__ __align__(16) unsigned char shraw[sizeof(Shared) > 8 * extras_lds<NB>() ? sizeof(Shared) : 8 * extras_lds<NB>()];
  auto& stg = reinterpret_cast<Shared*>(shraw)->r.stg;
  auto& sS = reinterpret_cast<Shared*>(shraw)->r.sS;
  auto& red = reinterpret_cast<Shared*>(shraw)->red;
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, shraw);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<128>(task, m, lgL);
  const int sp = ht.s, r0 = ht.r0, r1 = ht.r1;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // rows and Sigma^R wavefront-uniform
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  for (int q = threadIdx.x; q < 4 * NBB * 64; q += 64 * WAVES) {
    int l = q & 63, e = (q >> 6) % NBB, x = (q >> 6) / NBB;
    int t = 64 * (2 * sp + (x >> 1)) + l;
    sS[x >> 1][x & 1][e][l] = t < m ? sk[((x & 1) * NBB + e) * d.Tp + t] : czero();
  }
  __syncthreads();
  // the pair's second strip exists only if its first column is below m
  const bool two = 64 * (2 * sp + 1) < m;
  int tp[2];
  bool colv[2];
  const cplx* hk[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    tp[h] = 64 * (2 * sp + h) + lane;
    colv[h] = tp[h] < m;
    hk[h] = hist + strip_lane_base(d, k, (h && two) ? 2 * sp + 1 : 2 * sp, lane);
  }
  cplx acc[2][C];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[h][c] = czero();
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, sp));
  for (int cb = r0; cb < r1; cb += 64) {
    const int rb = cb + wv;   // the wavefront's rows of the chunk: rb, rb + RSTEP, ... (RPC of them)
    const int cslot = ((cb - r0) >> 6) % (ROWS_ST / 64);   // chunk's place in the staging
    cplx* st = &stg[0][64 * cslot];                                // st[e * ROWS_ST + (row - cb)]
    for (int i = 0; i < RPC;) {
      const int jb = rb + RSTEP * i;
      if (jb >= r1) break;
      // rows past the pair's first 128 (and below the segment's end) need no masks (as in k_hist_pair32)
      auto iteration = [&](auto tag, auto nh, auto nr) {
        constexpr int RR = decltype(nr)::value;   // rows in this iteration
        constexpr int MM = decltype(tag)::value;   // masks: 0 none, 1 the second strip's only, 2 all
        constexpr bool MASKED = MM == 2;
        constexpr int NH = decltype(nh)::value;   // strips of the pair with work in these rows
        cplx G[RR][2][C];
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            int j = jb + RSTEP * r;
            bool v = (MM == 2 || (MM == 1 && h == 1)) ? (colv[h] && tp[h] <= j && j < r1) : true;
            const cplx* row = hk[h] + 64 * (int64_t)C * j;
#pragma unroll
            for (int c = 0; c < C; ++c) G[r][h][c] = v ? load_stream(row + 64 * c) : czero();
          }
        double rt[RR][2 * NBB];
#pragma unroll
        for (int r = 0; r < RR; ++r) {
          int j = jb + RSTEP * r;
          int jc = MASKED ? (j < r1 ? j : r1 - 1) : j;
          cplx SR[NBB];
#pragma unroll
          for (int e = 0; e < NBB; ++e) SR[e] = sk[(2 * NBB + e) * d.Tp + jc];
#pragma unroll
          for (int e = 0; e < 2 * NBB; ++e) rt[r][e] = 0.0;
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            mm_acc<NB>(acc[h], SR, G[r][h]);
            mm_acc<NB>(acc[h] + NBB, SR, G[r][h] + NBB);
            cplx Sl[NBB], Sg[NBB], a[NBB], u[NBB];
#pragma unroll
            for (int e = 0; e < NBB; ++e) {
              Sl[e] = sS[h][0][e][lane];
              Sg[e] = sS[h][1][e][lane];
            }
            mat_zero<NB>(a);
            mat_zero<NB>(u);
            mm_acc_bdag<NB>(a, Sl, G[r][h] + NBB);
            mm_acc_bdag<NB>(u, Sg, G[r][h]);
            bool rv = (MM == 2 || (MM == 1 && h == 1)) ? tp[h] < j : true;
#pragma unroll
            for (int e = 0; e < NBB; ++e) {
              rt[r][2 * e] += rv ? a[e].x - u[e].x : 0.0;
              rt[r][2 * e + 1] += rv ? a[e].y - u[e].y : 0.0;
            }
          }
        }
        if constexpr (RR == 1 && NBB == 4) {
          // one row, four components: each component's (re, im) is one group of a 4-group
          // reduce-scatter (2 lane reductions instead of 8)
          double xg[4][2];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            xg[e][0] = rt[0][2 * e];
            xg[e][1] = rt[0][2 * e + 1];
          }
          reduce_rows<4>(xg);
          int e = reduced_row<4>(lane);
          if (e >= 0) st[e * ROWS_ST + (jb - cb)] = cmk(xg[0][0], xg[0][1]);
        } else {
          reduce_rows<RR>(rt);
          int rr = reduced_row<RR>(lane);
          if (rr >= 0) {
#pragma unroll
            for (int e = 0; e < NBB; ++e) st[e * ROWS_ST + (jb - cb) + RSTEP * rr] = cmk(rt[0][2 * e], rt[0][2 * e + 1]);
          }
        }
      };
      // rows of the pair's first 64 lie above every column of its second strip: one strip's
      // work; in its next 64 rows every column of the first strip lies below the row: masks for
      // the second strip only
      // (an iteration's rows jb, jb + RSTEP, ..., jb + RSTEP (RR - 1) lie in one 64-row chunk)
      if (jb >= 128 * sp + 128 && jb + RSTEP * (R - 1) < r1) {
        iteration(IntTag<0>{}, IntTag<2>{}, IntTag<R>{});
        i += R;
      } else if (R == 1 && jb + RSTEP < 128 * sp + 64 && jb + RSTEP < r1) {
        // two rows at a time where only the first strip has work: its loads of both rows in
        // flight together (one row would keep half the loads of a full iteration in flight)
        iteration(IntTag<2>{}, IntTag<1>{}, IntTag<2>{});
        i += 2;
      } else if (jb + RSTEP * (R - 1) < 128 * sp + 64) {
        iteration(IntTag<2>{}, IntTag<1>{}, IntTag<R>{});
        i += R;
      } else if (jb >= 128 * sp + 64 && jb + RSTEP * (R - 1) < r1 && jb + RSTEP * (R - 1) < 128 * sp + 128) {
        iteration(IntTag<1>{}, IntTag<2>{}, IntTag<R>{});
        i += R;
      } else {
        iteration(IntTag<2>{}, IntTag<2>{}, IntTag<R>{});
        i += R;
      }
    }
    // every fourth chunk (and the last): the staged rows of all the wavefronts leave as one
    // contiguous run of up to 256 rows per component (4 KB), streaming stores
    if (cslot == ROWS_ST / 64 - 1 || cb + 64 >= r1) {
      __syncthreads();
      const int base = cb - 64 * cslot;
      const int nrows = (cb + 64 < r1 ? cb + 64 : r1) - base;
      for (int q = threadIdx.x; q < NBB * nrows; q += 64 * WAVES) {
        const int e = q / nrows, row = q - e * nrows;
        store_stream(rp + (int64_t)e * d.Tp + base + row, stg[e][row]);
      }
      __syncthreads();
    }
  }
  // combine the wavefronts' column sums, strip by strip: every wavefront adds up its share of the
  // components, in the order of the wavefronts
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int c = 0; c < C; ++c) red[wv][c][lane] = acc[h][c];
    __syncthreads();
    if (colv[h])
      for (int c = wv; c < C; c += WAVES) {
        cplx a = red[0][c][lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) a = cadd(a, red[w][c][lane]);
        colpart[colpart_idx(d, k, ht.g, c, tp[h])] = a;
      }
    if (h == 0) __syncthreads();
  }
}

// ------------------------------------------------------------------ history sums, FP32 form
// Same structure as k_hist_pair over an FP32-stored history (complex64, half the bytes, a
// column's component pairs in one 16-byte load): R = 2 rows per iteration at nb = 2 (2 rows x
// 2 strips x 4 loads in flight per wavefront), R = 4 at nb = 1. Products and the 64-lane row
// reductions in FP32; the column sums accumulate in FP32 over each wavefront's 16 rows of a
// 64-row chunk and are then added into FP64 registers; row partials and column sums leave the
// kernel in FP64 (the cross-strip reduction, the end points, the update and the density matrix
// stay FP64).
template <int NB>
__global__ __launch_bounds__(256) void k_hist_pair32(Dims d, const cplx32* __restrict__ hist,
                                                     const cplx* __restrict__ sig, cplx* __restrict__ colpart,
                                                     cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr int R = NB == 1 ? 4 : 2;
  __shared__ cplx red[3][C][64];
  constexpr int ROWS_ST = 256;   // row partials staged over four 64-row chunks, as in k_hist_pair
  __shared__ cplx stg[NBB][ROWS_ST];
  __shared__ cplx32 sS[2][2][NBB][64];
  static_assert(sizeof(red) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, red);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<128>(task, m, lgL);
  const int sp = ht.s, r0 = ht.r0, r1 = ht.r1;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  for (int q = threadIdx.x; q < 4 * NBB * 64; q += 256) {
    int l = q & 63, e = (q >> 6) % NBB, x = (q >> 6) / NBB;
    int t = 64 * (2 * sp + (x >> 1)) + l;
    sS[x >> 1][x & 1][e][l] = to32(t < m ? sk[((x & 1) * NBB + e) * d.Tp + t] : czero());
  }
  __syncthreads();
  const bool two = 64 * (2 * sp + 1) < m;
  int tp[2];
  bool colv[2];
  const cplx32* hk[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    tp[h] = 64 * (2 * sp + h) + lane;
    colv[h] = tp[h] < m;
    hk[h] = hist + strip_lane_base(d, k, (h && two) ? 2 * sp + 1 : 2 * sp, lane);
  }
  cplx acc[2][C];
  cplx32 acc32[2][C];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < C; ++c) {
      acc[h][c] = czero();
      acc32[h][c] = make_float2(0.f, 0.f);
    }
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, sp));
  for (int cb = r0; cb < r1; cb += 64) {
    const int rb = cb + wv;   // the wavefront's rows of the chunk: rb, rb + 4, ..., rb + 60
    const int cslot = ((cb - r0) >> 6) % (ROWS_ST / 64);
    cplx* st = &stg[0][64 * cslot];   // st[e * ROWS_ST + (row - cb)]
    for (int i = 0; i < 16 / R; ++i) {
      const int jb = rb + 4 * R * i;
      if (jb >= r1) break;
      // rows past the pair's first 128 (and below the segment's end) need no masks: every lane's columns lie
      // below the row, so that common case runs without the bounds selects
      auto iteration = [&](auto tag, auto nh) {
        constexpr int MM = decltype(tag)::value;   // masks: 0 none, 1 the second strip's only, 2 all
        constexpr bool MASKED = MM == 2;
        constexpr int NH = decltype(nh)::value;   // strips of the pair with work in these rows
        cplx32 G[R][2][C];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            int j = jb + 4 * r;
            bool v = (MM == 2 || (MM == 1 && h == 1)) ? (colv[h] && tp[h] <= j && j < r1) : true;
            const cplx32* row = hk[h] + 64 * (int64_t)C * j;
#pragma unroll
            for (int c2 = 0; c2 < C / 2; ++c2) {
              if (v) {
                load_stream32x2(row + 128 * c2, G[r][h][2 * c2], G[r][h][2 * c2 + 1]);
              } else {
                G[r][h][2 * c2] = make_float2(0.f, 0.f);
                G[r][h][2 * c2 + 1] = make_float2(0.f, 0.f);
              }
            }
          }
        float rt[R][2 * NBB];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          int j = jb + 4 * r;
          int jc = MASKED ? (j < r1 ? j : r1 - 1) : j;
          cplx32 SR[NBB];
#pragma unroll
          for (int e = 0; e < NBB; ++e) SR[e] = to32(sk[(2 * NBB + e) * d.Tp + jc]);
#pragma unroll
          for (int e = 0; e < 2 * NBB; ++e) rt[r][e] = 0.f;
#pragma unroll
          for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int sc = 0; sc < 2; ++sc)
#pragma unroll
              for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                  for (int l = 0; l < NB; ++l)
                    cmac32(acc32[h][sc * NBB + a * NB + b], SR[a * NB + l], G[r][h][sc * NBB + l * NB + b]);
            bool rv = (MM == 2 || (MM == 1 && h == 1)) ? tp[h] < j : true;
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
              for (int b = 0; b < NB; ++b) {
                cplx32 x = make_float2(0.f, 0.f), u = make_float2(0.f, 0.f);
#pragma unroll
                for (int l = 0; l < NB; ++l) {
                  cmacc32(x, sS[h][0][a * NB + l][lane], G[r][h][NBB + b * NB + l]);
                  cmacc32(u, sS[h][1][a * NB + l][lane], G[r][h][b * NB + l]);
                }
                int e = a * NB + b;
                rt[r][2 * e] += rv ? x.x - u.x : 0.f;
                rt[r][2 * e + 1] += rv ? x.y - u.y : 0.f;
              }
          }
        }
        if constexpr (R == 2 && NBB == 4) {
          // two rows, four components: groups (row, component pair) of a 4-group reduce-scatter
          // (4 lane reductions instead of 8); group g = 2 r + p holds components 2 p, 2 p + 1
          float xg[4][4];
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int p2 = 0; p2 < 2; ++p2)
#pragma unroll
              for (int q = 0; q < 4; ++q) xg[2 * r + p2][q] = rt[r][4 * p2 + q];
          reduce_rows32<4>(xg);
          int g = reduced_row<4>(lane);
          if (g >= 0) {
            int r = g >> 1, p2 = g & 1;
#pragma unroll
            for (int c = 0; c < 2; ++c)
              st[(2 * p2 + c) * ROWS_ST + (jb - cb) + 4 * r] = cmk((double)xg[0][2 * c], (double)xg[0][2 * c + 1]);
          }
        } else {
          reduce_rows32<R>(rt);
          int rr = reduced_row<R>(lane);
          if (rr >= 0) {
#pragma unroll
            for (int e = 0; e < NBB; ++e)
              st[e * ROWS_ST + (jb - cb) + 4 * rr] = cmk((double)rt[0][2 * e], (double)rt[0][2 * e + 1]);
          }
        }
      };
      // rows of the pair's first 64 lie above every column of its second strip: one strip's
      // work; in its next 64 rows every column of the first strip lies below the row: masks for
      // the second strip only
      // (an iteration's rows jb, jb + 4, ..., jb + 4 (R - 1) lie in one 64-row chunk)
      if (jb >= 128 * sp + 128 && jb + 4 * (R - 1) < r1)
        iteration(IntTag<0>{}, IntTag<2>{});
      else if (jb + 4 * (R - 1) < 128 * sp + 64)
        iteration(IntTag<2>{}, IntTag<1>{});
      else if (jb >= 128 * sp + 64 && jb + 4 * (R - 1) < r1 && jb + 4 * (R - 1) < 128 * sp + 128)
        iteration(IntTag<1>{}, IntTag<2>{});
      else
        iteration(IntTag<2>{}, IntTag<2>{});
    }
    // the group's FP32 column sums into the FP64 accumulators
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        acc[h][c].x += (double)acc32[h][c].x;
        acc[h][c].y += (double)acc32[h][c].y;
        acc32[h][c] = make_float2(0.f, 0.f);
      }
    if (cslot == ROWS_ST / 64 - 1 || cb + 64 >= r1) {
      __syncthreads();
      const int base = cb - 64 * cslot;
      const int nrows = (cb + 64 < r1 ? cb + 64 : r1) - base;
      for (int q = threadIdx.x; q < NBB * nrows; q += 256) {
        const int e = q / nrows, row = q - e * nrows;
        store_stream(rp + (int64_t)e * d.Tp + base + row, stg[e][row]);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (wv > 0) {
#pragma unroll
      for (int c = 0; c < C; ++c) red[wv - 1][c][lane] = acc[h][c];
    }
    __syncthreads();
    if (wv == 0 && colv[h]) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        cplx a = acc[h][c];
        a = cadd(a, red[0][c][lane]);
        a = cadd(a, red[1][c][lane]);
        a = cadd(a, red[2][c][lane]);
        colpart[colpart_idx(d, k, ht.g, c, tp[h])] = a;
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ history sums, nb = 3
// FP64: one 64-column strip per block (row partials in slot s; the 18 components of a block leave no
// registers for a second strip), wavefront w on rows w, w + 4, ... of every 64-row chunk, one row (18
// loads of 1 KB) per iteration, the strip's triangular first 64 rows in a masked copy of the loop body,
// the per-column Sigma of the row term in LDS. The 18 numbers of a row term go through one 64-lane
// reduce-scatter as four groups of five (5 lane reductions instead of 18); row partials are staged over
// four chunks and stored as 4 KB runs. 2 wavefronts per SIMD (with 18 reductions live the kernel held
// 294 registers, one wavefront per SIMD): 38.5 -> 28.5 us on average at 63 points, m <= 150.
template <int NB>
__global__ __launch_bounds__(256) void k_hist_bulk(Dims d, const cplx* __restrict__ hist,
                                                   const cplx* __restrict__ sig, cplx* __restrict__ colpart,
                                                   cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  static_assert(NB == 3, "five numbers per group");
  constexpr int ROWS_ST = 256, Q = 5;
  struct Rows {
    cplx stg[NBB][ROWS_ST];
    cplx sS[2][NBB][64];
  };
  union Shared {
    Rows r;
    cplx red[4][NBB][64];   // column sums of one component half, after the row loop
  };
  __shared__ __align__(16) unsigned char shraw[sizeof(Shared)];
  static_assert(sizeof(Shared) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  auto& stg = reinterpret_cast<Shared*>(shraw)->r.stg;
  auto& sS = reinterpret_cast<Shared*>(shraw)->r.sS;
  auto& red = reinterpret_cast<Shared*>(shraw)->red;
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, shraw);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<64>(task, m, lgL);
  const int s = ht.s, r0 = ht.r0, r1 = ht.r1;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tp = 64 * s + lane;
  const bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  for (int i = threadIdx.x; i < 2 * NBB * 64; i += 256) {
    int y = i / (NBB * 64), e = (i / 64) % NBB, l = i % 64;
    int t = 64 * s + l;
    sS[y][e][l] = t < m ? sk[(y * NBB + e) * d.Tp + t] : czero();
  }
  __syncthreads();
  cplx acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = czero();
  const cplx* hk = hist + strip_lane_base(d, k, s, lane);
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, s));
  for (int cb = r0; cb < r1; cb += 64) {
    const int cslot = ((cb - r0) >> 6) % (ROWS_ST / 64);
    for (int i = 0; i < 16; ++i) {
      const int j = cb + wv + 4 * i;
      if (j >= r1) break;
      auto row = [&](auto tag) {
        constexpr bool MASKED = decltype(tag)::value;
        const bool v = MASKED ? (colv && tp <= j) : true;
        const cplx* g = hk + 64 * (int64_t)C * j;
        cplx G[C];
#pragma unroll
        for (int c = 0; c < C; ++c) G[c] = v ? load_stream(g + 64 * c) : czero();
        cplx SR[NBB];
#pragma unroll
        for (int e = 0; e < NBB; ++e) SR[e] = sk[(2 * NBB + e) * d.Tp + j];
        mm_acc<NB>(acc, SR, G);
        mm_acc<NB>(acc + NBB, SR, G + NBB);
        const bool rv = MASKED ? tp < j : true;
        double xg[4][Q];   // numbers 5 g + q of (e, re/im)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
          for (int q = 0; q < Q; ++q) xg[g4][q] = 0.0;
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            cplx y = czero(), u = czero();
#pragma unroll
            for (int l = 0; l < NB; ++l) {
              cmacc(y, sS[0][a * NB + l][lane], G[NBB + b * NB + l]);
              cmacc(u, sS[1][a * NB + l][lane], G[b * NB + l]);
            }
            const int e = a * NB + b;
            xg[(2 * e) / Q][(2 * e) % Q] = rv ? y.x - u.x : 0.0;
            xg[(2 * e + 1) / Q][(2 * e + 1) % Q] = rv ? y.y - u.y : 0.0;
          }
        reduce_rows<4>(xg);
        const int g4 = reduced_row<4>(lane);
        if (g4 >= 0) {
          double* st = reinterpret_cast<double*>(&stg[0][64 * cslot + (j - cb)]);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int n = Q * g4 + q;
            if (n < 2 * NBB) st[2 * ROWS_ST * (n >> 1) + (n & 1)] = xg[0][q];
          }
        }
      };
      if (j >= 64 * s + 64)
        row(BoolTag<false>{});
      else
        row(BoolTag<true>{});
    }
    if (cslot == ROWS_ST / 64 - 1 || cb + 64 >= r1) {
      __syncthreads();
      const int base = cb - 64 * cslot;
      const int nrows = (cb + 64 < r1 ? cb + 64 : r1) - base;
      for (int q = threadIdx.x; q < NBB * nrows; q += 256) {
        const int e = q / nrows, r = q - e * nrows;
        store_stream(rp + (int64_t)e * d.Tp + base + r, stg[e][r]);
      }
      __syncthreads();
    }
  }
  // the wavefronts' column sums, one component half at a time, a share of the components by each
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) red[wv][e][lane] = acc[h * NBB + e];
    __syncthreads();
    if (colv)
      for (int e = wv; e < NBB; e += 4)
        colpart[colpart_idx(d, k, ht.g, h * NBB + e, tp)] =
            cadd(cadd(cadd(red[0][e][lane], red[1][e][lane]), red[2][e][lane]), red[3][e][lane]);
    if (h == 0) __syncthreads();
  }
}

// FP32 form at nb = 3: two rows per iteration, Sigma of the row term in registers; FP32 tiles
// of 16 rows per wavefront added into FP64 accumulators.
template <int NB>
__global__ __launch_bounds__(256) void k_hist_bulk32(Dims d, const cplx32* __restrict__ hist,
                                                     const cplx* __restrict__ sig, cplx* __restrict__ colpart,
                                                     cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr int CH = (C < 8) ? C : 8;
  constexpr int R = 2;
  constexpr int FLUSH = 16 / R;  // iterations per FP32 accumulation tile (16 rows)
  __shared__ cplx red[3][CH][64];
  static_assert(sizeof(red) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, red);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<64>(task, m, lgL);
  const int s = ht.s, r0 = ht.r0, r1 = ht.r1;
  int lane = threadIdx.x & 63;
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tp = 64 * s + lane;
  bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  cplx32 Sl[NBB], Sg[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    Sl[e] = to32(colv ? sk[(0 * NBB + e) * d.Tp + tp] : czero());
    Sg[e] = to32(colv ? sk[(1 * NBB + e) * d.Tp + tp] : czero());
  }
  cplx acc[C];
  cplx32 acc32[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    acc[c] = czero();
    acc32[c] = make_float2(0.f, 0.f);
  }
  const cplx32* hk = hist + strip_lane_base(d, k, s, lane);
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, s));
  int it = 0;
  for (int jb = r0 + R * wv; jb < r1; jb += 4 * R) {
    cplx32 G[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int j = jb + r;
      bool v = colv && tp <= j && j < r1;
      const cplx32* row = hk + 64 * (int64_t)C * j;
#pragma unroll
      for (int c2 = 0; c2 < C / 2; ++c2) {
        if (v) {
          load_stream32x2(row + 128 * c2, G[r][2 * c2], G[r][2 * c2 + 1]);
        } else {
          G[r][2 * c2] = make_float2(0.f, 0.f);
          G[r][2 * c2 + 1] = make_float2(0.f, 0.f);
        }
      }
    }
    float rt[R][2 * NBB];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int j = jb + r;
      int jc = j < r1 ? j : r1 - 1;
      cplx32 SR[NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) SR[e] = to32(sk[(2 * NBB + e) * d.Tp + jc]);
#pragma unroll
      for (int sc = 0; sc < 2; ++sc)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int jj = 0; jj < NB; ++jj)
#pragma unroll
            for (int l = 0; l < NB; ++l) cmac32(acc32[sc * NBB + i * NB + jj], SR[i * NB + l], G[r][sc * NBB + l * NB + jj]);
      bool rv = tp < j;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int jj = 0; jj < NB; ++jj) {
          cplx32 a = make_float2(0.f, 0.f), u = make_float2(0.f, 0.f);
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            cmacc32(a, Sl[i * NB + l], G[r][NBB + jj * NB + l]);
            cmacc32(u, Sg[i * NB + l], G[r][jj * NB + l]);
          }
          int e = i * NB + jj;
          rt[r][2 * e] = rv ? a.x - u.x : 0.f;
          rt[r][2 * e + 1] = rv ? a.y - u.y : 0.f;
        }
    }
    if (++it == FLUSH) {
      it = 0;
#pragma unroll
      for (int c = 0; c < C; ++c) {
        acc[c].x += (double)acc32[c].x;
        acc[c].y += (double)acc32[c].y;
        acc32[c] = make_float2(0.f, 0.f);
      }
    }
    reduce_rows32<R>(rt);
    int rsel = reduced_row<R>(lane);
    if (rsel >= 0 && jb + rsel < r1) {
#pragma unroll
      for (int e = 0; e < NBB; ++e)
        rp[(int64_t)e * d.Tp + jb + rsel] = cmk((double)rt[0][2 * e], (double)rt[0][2 * e + 1]);
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    acc[c].x += (double)acc32[c].x;
    acc[c].y += (double)acc32[c].y;
  }
#pragma unroll
  for (int c0 = 0; c0 < C; c0 += CH) {
    if (wv > 0) {
#pragma unroll
      for (int c = 0; c < CH; ++c) red[wv - 1][c][lane] = acc[c0 + c];
    }
    __syncthreads();
    if (wv == 0) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        cplx a = acc[c0 + c];
        a = cadd(a, red[0][c][lane]);
        a = cadd(a, red[1][c][lane]);
        a = cadd(a, red[2][c][lane]);
        if (colv) colpart[colpart_idx(d, k, ht.g, c0 + c, tp)] = a;
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ history sums, nb = 4
// With nb = 4 a stored block has 2 nb^2 = 32 components, too many for one wavefront's
// registers next to its column sums. The block's components are split by half: waves 0 and 2
// stream G^< (components 0..15), waves 1 and 3 stream G^> (16..31); the row pair (0, 1) takes
// rows 0-15 of every 32-row chunk of the strip, the pair (2, 3) rows 16-31 (16 contiguous 1 KB
// segments in flight per wavefront). Half 0 contributes -Sigma^>_{t'} (G^<_{j t'})^dag to the
// row term, half 1 +Sigma^<_{t'} (G^>_{j t'})^dag. The four block rows of a row term go through
// one 64-lane reduce-scatter together (4 quantities for the instructions of one); a
// wavefront's 16 row partials are staged in LDS (two buffers, alternating by chunk), and after
// one block barrier per 32-row chunk the two halves' partials are added and stored as 256-byte
// runs with streaming stores, one row-partial slot per strip. The per-column Sigma of the row
// term is read from LDS. FP64 storage; 2 waves per SIMD.
template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_hist_bulk_split(
    Dims d, const cplx* __restrict__ hist, const cplx* __restrict__ sig, cplx* __restrict__ colpart,
    cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  static_assert(NB == 4, "the four block rows share one reduce-scatter");
  __shared__ cplx sS[2][NBB][64];  // [half][e][lane]: half 0 needs Sigma^>, half 1 Sigma^<;
                                   // reused for the column-sum combine after the row loop
  __shared__ cplx stg[2][2][2][NBB * 16];  // [buffer][row pair][half][e * 16 + row]
  static_assert(sizeof(sS) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, sS);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<64>(task, m, lgL);
  const int s = ht.s, r0 = ht.r0, r1 = ht.r1;
  int lane = threadIdx.x & 63;
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront-uniform: rows and Sigma^R in SGPRs
  int h = wv & 1, rg = wv >> 1;
  int tp = 64 * s + lane;
  bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  for (int i = threadIdx.x; i < 2 * NBB * 64; i += 256) {
    int x = i / (NBB * 64), e = (i / 64) % NBB, l = i % 64;
    int t = 64 * s + l;
    sS[x][e][l] = t < m ? sk[((1 - x) * NBB + e) * d.Tp + t] : czero();
  }
  __syncthreads();
  cplx acc[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) acc[e] = czero();
  const cplx* hk = hist + strip_lane_base(d, k, s, lane) + 64 * NBB * h;
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, s));
  const double sgn = h ? 1.0 : -1.0;
  int buf = 0;
  for (int cb = r0; cb < r1; cb += 32) {  // the same chunks in every wavefront
    const int rb = cb + 16 * rg;
    cplx* st = stg[buf][rg][h];
    for (int i = 0; i < 16; ++i) {
      const int j = rb + i;
      if (j >= r1) break;
      bool v = colv && tp <= j;
      const cplx* row = hk + 64 * (int64_t)C * j;
      cplx G[NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) G[e] = v ? load_stream(row + 64 * e) : czero();
      bool rv = tp < j;
      double x[NB][2 * NB];  // row term of block row a, column b: x[a][2 b], x[a][2 b + 1]
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        cplx SRa[NB];
#pragma unroll
        for (int l = 0; l < NB; ++l) SRa[l] = sk[(2 * NBB + a * NB + l) * d.Tp + j];
        // column term, block row a:  acc[a][b] += sum_l SR[a][l] G[l][b]
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int l = 0; l < NB; ++l) cmac(acc[a * NB + b], SRa[l], G[l * NB + b]);
        // row term, block row a:  sgn * sum_l S[a][l] conj(G[b][l])
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          cplx t = czero();
#pragma unroll
          for (int l = 0; l < NB; ++l) cmacc(t, sS[h][a * NB + l][lane], G[b * NB + l]);
          x[a][2 * b] = rv ? sgn * t.x : 0.0;
          x[a][2 * b + 1] = rv ? sgn * t.y : 0.0;
        }
      }
      reduce_rows<NB>(x);
      int ra = reduced_row<NB>(lane);
      if (ra >= 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) st[(ra * NB + b) * 16 + i] = cmk(x[0][2 * b], x[0][2 * b + 1]);
      }
    }
    __syncthreads();  // both halves of the chunk staged; the other buffer is free again
    flush_rows_fold<NBB>(stg[buf][rg][0], stg[buf][rg][1], rp, d.Tp, rb, r1, lane, h);
    buf ^= 1;
  }
  __syncthreads();  // every wavefront is done with sS
  cplx (*red)[NBB][64] = sS;
  if (rg == 1) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) red[h][e][lane] = acc[e];
  }
  __syncthreads();
  if (rg == 0 && colv) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) colpart[colpart_idx(d, k, ht.g, h * NBB + e, tp)] = cadd(acc[e], red[h][e][lane]);
  }
}

// FP32 form of k_hist_bulk_split: each half's 16 components are 8 column-interleaved pairs,
// one 16-byte load each; FP32 products and row reductions, column sums in FP32 over each
// wavefront's 16 rows of a 32-row chunk, then FP64. The row pair (0, 1) takes the even rows of
// every 32-row chunk and (2, 3) the odd ones, the next row's loads in flight through a row's arithmetic
// (16 x 16, m = 200 / 800 400 -> 387 us, 4.36 -> 4.17 ms; 8 x 8, m = 300 230 -> 205 us; the FP64 kernel has no
// registers for it), so a chunk cut short by m keeps both pairs busy, and
// the whole block stores a chunk's row partials as 512-byte runs (this kernel is bound by the
// vector ALU; the FP64 kernel's stream ran 1.7 % slower with interleaved rows and keeps 16
// consecutive rows per pair).
template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_hist_bulk32_split(
    Dims d, const cplx32* __restrict__ hist, const cplx* __restrict__ sig, cplx* __restrict__ colpart,
    cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  static_assert(NB == 4, "the four block rows share one reduce-scatter");
  static_assert(NBB % 2 == 0, "component pairs must not straddle the halves");
  __shared__ cplx32 sS[2][NBB][64];
  __shared__ cplx stg[2][2][NBB * 32];  // [buffer][half][e * 32 + row - cb]; column-sum combine
                                        // after the row loop
  static_assert(sizeof(stg) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, stg);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<64>(task, m, lgL);
  const int s = ht.s, r0 = ht.r0, r1 = ht.r1;
  int lane = threadIdx.x & 63;
  int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int h = wv & 1, rg = wv >> 1;
  int tp = 64 * s + lane;
  bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  for (int i = threadIdx.x; i < 2 * NBB * 64; i += 256) {
    int x = i / (NBB * 64), e = (i / 64) % NBB, l = i % 64;
    int t = 64 * s + l;
    sS[x][e][l] = to32(t < m ? sk[((1 - x) * NBB + e) * d.Tp + t] : czero());
  }
  __syncthreads();
  cplx acc[NBB];
  cplx32 acc32[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    acc[e] = czero();
    acc32[e] = make_float2(0.f, 0.f);
  }
  const cplx32* hk = hist + strip_lane_base(d, k, s, lane) + 64 * NBB * h;
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, s));
  const float sgn = h ? 1.f : -1.f;
  cplx32 Gq[NBB];        // the wavefront's next unmasked row, if primed
  bool primed = false;
  int buf = 0;
  for (int cb = r0; cb < r1; cb += 32) {  // the same chunks in every wavefront
    const int rb = cb + rg;   // the wave pair's rows of the chunk: rb, rb + 2, ..., rb + 30
    cplx* st = stg[buf][h];
    // One row j from G (rv: the row term's mask)
    auto row = [&](int j, bool rv, const cplx32* G) {
      float x[NB][2 * NB];
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        cplx32 SRa[NB];
#pragma unroll
        for (int l = 0; l < NB; ++l) SRa[l] = to32(sk[(2 * NBB + a * NB + l) * d.Tp + j]);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int l = 0; l < NB; ++l) cmac32(acc32[a * NB + b], SRa[l], G[l * NB + b]);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          cplx32 t = make_float2(0.f, 0.f);
#pragma unroll
          for (int l = 0; l < NB; ++l) cmacc32(t, sS[h][a * NB + l][lane], G[b * NB + l]);
          x[a][2 * b] = rv ? sgn * t.x : 0.f;
          x[a][2 * b + 1] = rv ? sgn * t.y : 0.f;
        }
      }
      reduce_rows32<NB>(x);
      int ra = reduced_row<NB>(lane);
      if (ra >= 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) st[(ra * NB + b) * 32 + (j - cb)] = cmk((double)x[0][2 * b], (double)x[0][2 * b + 1]);
      }
    };
    auto load = [&](int j, cplx32* G) {
      const cplx32* g = hk + 64 * (int64_t)C * j;
#pragma unroll
      for (int p = 0; p < NBB / 2; ++p) load_stream32x2(g + 128 * p, G[2 * p], G[2 * p + 1]);
    };
    if (rb >= 64 * s + 64 && rb + 30 < r1) {
      // groups of 16 rows past the strip's first 64 rows and below the segment's end need no masks; the
      // next row's loads are in flight through a row's arithmetic (across groups too)
      if (!primed) load(rb, Gq);
      for (int i = 0; i < 16; ++i) {
        const int j = rb + 2 * i;
        int jn = i < 15 ? j + 2 : rb + 32;
        if (jn >= r1) jn = j;
        cplx32 Gn[NBB];
        load(jn, Gn);
        row(j, true, Gq);
#pragma unroll
        for (int e = 0; e < NBB; ++e) Gq[e] = Gn[e];
      }
      primed = true;
    } else {
      primed = false;
      for (int i = 0; i < 16; ++i) {
        const int j = rb + 2 * i;
        if (j >= r1) break;
        const bool v = colv && tp <= j;
        cplx32 G[NBB];
        if (v) {
          load(j, G);
        } else {
#pragma unroll
          for (int e = 0; e < NBB; ++e) G[e] = make_float2(0.f, 0.f);
        }
        row(j, tp < j, G);
      }
    }
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      acc[e].x += (double)acc32[e].x;
      acc[e].y += (double)acc32[e].y;
      acc32[e] = make_float2(0.f, 0.f);
    }
    __syncthreads();  // both halves of the chunk staged; the other buffer is free again
    flush_chunk_fold<NBB>(stg[buf][0], stg[buf][1], rp, d.Tp, cb, r1);
    buf ^= 1;
  }
  __syncthreads();  // every wavefront is done with stg
  cplx (*red)[NBB][64] = reinterpret_cast<cplx (*)[NBB][64]>(&stg[0][0][0]);
  if (rg == 1) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) red[h][e][lane] = acc[e];
  }
  __syncthreads();
  if (rg == 0 && colv) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) colpart[colpart_idx(d, k, ht.g, h * NBB + e, tp)] = cadd(acc[e], red[h][e][lane]);
  }
}

// ------------------------------------------------------------------ history sums, FP32-MFMA form
// The same sums as above on the quad layout of the FP32-MFMA form. A block takes strip s of one
// k; its wavefronts split the 64 columns into 4 groups g of 16 (and, at nb = 4, the components
// into their G^< and G^> halves: 8 wavefronts; at nb <= 3 each wavefront takes both halves: 4).
// Per quad of 4 rows a lane L holds the pair (j = j0 + L / 16, t' = 16 g + L % 16):
// * column term, on the matrix cores: for component (half, b) the 16 x 16 tile
//     D[m][t'] += sum_{r < 4} A_l^ri[m][r] G_{l b}^ri(j0 + r, t'),   m = (hi/lo, a, re/im),
//   one v_mfma_f32_16x16x4f32 per (l, re/im) with K = the quad's 4 rows: A holds the real
//   embedding of Sigma^R(t_j)_{a l} (re rows: [Re, -Im]; im rows: [Im, Re]) split into its FP32
//   high part and the FP32 rounding of the remainder (rows m < 2 nb: high, 2 nb <= m < 4 nb: low),
//   so the two compensated products fill the 16-row tile at nb = 4 and are added in FP64 at the
//   end. The tiles accumulate in FP32 over one chunk of quads (8 quads = 32 rows at nb = 4, 16
//   quads = 64 rows otherwise), then into FP64 registers. The A operands of a chunk are split and
//   staged in LDS once per block, one chunk ahead, by all its threads (every wavefront of the block
//   needs the same rows).
// * row term, on the vector ALU in FP32: each lane forms sgn Sigma^{>,<}_{t'} (G_{j t'})^dag of its
//   pair; a DPP reduce-scatter over the 16 lanes of each row (four rows at once) leaves one
//   component per lane; the wavefronts' partials of a chunk are staged in LDS (two buffers) and,
//   after one block barrier per chunk, added in a fixed order in FP64 and stored to the strip's
//   row-partial slot with streaming stores (at nb <= 2 staged over four chunks and stored as
//   4 KB runs).
// Quads past the strip's triangle (its first 16) and below m run without bounds selects. The
// next quad's loads are issued before the current quad is processed, and no load sits behind a
// branch, so the waits for one quad's data are exact.
__device__ __forceinline__ float split_part(double x, bool low) {
  float hi = (float)x;
  return low ? (float)(x - (double)hi) : hi;
}
template <int CTRL, int CNT>
__device__ __forceinline__ void rs16_step(float* x, bool upper) {
  if constexpr (CNT >= 2) {
    constexpr int H = CNT / 2;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      float keep = upper ? x[i + H] : x[i];
      float send = upper ? x[i] : x[i + H];
      x[i] = keep + dpp_f<CTRL>(send);
    }
  } else {
    x[0] += dpp_f<CTRL>(x[0]);
  }
}
// Reduce-scatter of VP values (a power of two) over the 16 lanes of each row: partners differ in
// bit 3 (row mirror), bit 2 (half-row mirror), bit 1 and bit 0 (quad permutations) of the lane.
// Afterwards lane l of a row holds the row sums of values (VP / 16) l .. (VP / 16) l + VP / 16 - 1
// in x[0 ..] if VP >= 16, else of value l / (16 / VP) in x[0].
template <int VP>
__device__ __forceinline__ void reduce_scatter16(float (&x)[VP], int lane) {
  rs16_step<0x140, VP>(x, lane & 8);
  rs16_step<0x141, (VP / 2 > 1 ? VP / 2 : 1)>(x, lane & 4);
  rs16_step<0x4E, (VP / 4 > 1 ? VP / 4 : 1)>(x, lane & 2);
  rs16_step<0xB1, (VP / 8 > 1 ? VP / 8 : 1)>(x, lane & 1);
}

template <int NB>
struct MfmaShape {
  static constexpr int NBB = NB * NB, C = 2 * NBB;
  static constexpr int HS = NB == 4 ? 1 : 2;          // component halves per wavefront
  static constexpr int WAVES = 4 * (2 / HS);
  static constexpr int NCH = HS == 2 ? NBB : NBB / 2;  // 16-byte loads per lane and quad
  static constexpr int VP = 2 * NBB <= 2 ? 2 : (2 * NBB <= 8 ? 8 : 32);           // row-term values, padded
  static constexpr int CQ = NB == 4 ? 8 : 16;         // quads per staged chunk (32 or 64 rows)
  static constexpr int PF = 1;                        // quads whose loads are in flight ahead
  static constexpr int STAGE = 2 * WAVES * CQ * 4 * VP * 4;  // bytes
  static constexpr int AFR = 2 * CQ * 64 * 2 * NB * 4;       // bytes: A operands of two chunks
  static constexpr int FIN = WAVES * HS * NB * 256 * 8;     // bytes
  // row partials leave in runs of ROWS rows per component: at nb <= 2 the FP64 sums of four
  // 64-row chunks are staged (runs of 4 KB; fewer, longer write bursts in the read stream), at
  // nb >= 3 each chunk's rows are stored directly (a 64-row staging costs more than it saves there)
  static constexpr int ROWS = NB <= 2 ? 256 : 4 * CQ;
  static constexpr int RSTG = NB <= 2 ? NBB * ROWS * 16 : 0;   // bytes
  static constexpr int LDS = (STAGE + AFR) > FIN ? (STAGE + AFR) : FIN;
};

// A operands of the quads of one chunk, [quad][lane][l][re/im] (2 nb floats per lane): lane
// L = 16 r + n of quad q gives row n = (hi/lo, a, re/im) of the real embedding of
// Sigma^R(t_j)_{a l}, j = 64 s + 4 q + r, split into the FP32 high part and the FP32 rounding of
// the remainder; zero outside the 4 nb rows of the tile and for j >= m. Each thread takes
// entries e = tid, tid + block, ...: load() issues the FP64 reads, store() splits and writes.
template <int NB, int NE>
struct AfrFill {
  static_assert(NE * MfmaShape<NB>::WAVES * 64 == MfmaShape<NB>::CQ * 64, "every thread fills NE whole entries");
  cplx x[NE][NB];
  double z[NE];
  // every lane loads a valid entry (row clamped below m); entries outside the tile or past m are
  // zeroed only in store(), so no branch or early use sits behind the loads and the waits for
  // the quads' history loads stay exact
  __device__ __forceinline__ void load(const Dims& d, const cplx* sk, int s, int qfirst, int m, int tid, int nthr) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = tid + i * nthr;
      const int L = e & 63, n = L & 15;
      const int j = 64 * s + 4 * (qfirst + (e >> 6)) + (L >> 4);
      z[i] = (n < 4 * NB && j < m) ? 1.0 : 0.0;
      const int aa = (n % (2 * NB)) >> 1;
      const int jl = j < m ? j : m - 1;
#pragma unroll
      for (int l = 0; l < NB; ++l) x[i][l] = sk[(2 * NB * NB + aa * NB + l) * d.Tp + jl];
    }
  }
  __device__ __forceinline__ void store(float* afr, int tid, int nthr) const {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = tid + i * nthr;
      const int n = e & 15;
      const bool low = n >= 2 * NB, im_row = n & 1;
      float* dst = afr + e * 2 * NB;
#pragma unroll
      for (int l = 0; l < NB; ++l) {
        const float pr = split_part(x[i][l].x * z[i], low), pi = split_part(x[i][l].y * z[i], low);
        dst[2 * l] = im_row ? pi : pr;
        dst[2 * l + 1] = im_row ? pr : -pi;
      }
    }
  }
};

template <int NB>
__global__ __launch_bounds__(MfmaShape<NB>::WAVES * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_hist_mfma(
    Dims d, const float2* __restrict__ hist, const cplx* __restrict__ sig, cplx* __restrict__ colpart,
    cplx* __restrict__ rowpart, int m, int lgL, PassExtras x) {
  using Sh = MfmaShape<NB>;
  constexpr int NBB = Sh::NBB, C = Sh::C, HS = Sh::HS, NCH = Sh::NCH, VP = Sh::VP, CQ = Sh::CQ, WAVES = Sh::WAVES;
  static_assert(HS == 2 || NBB % 2 == 0, "halves must not share a 16-byte load");
  __shared__ __align__(16) unsigned char smem[Sh::LDS];
  constexpr int CPF = Sh::ROWS / (4 * CQ);   // chunks per row-partial store
  __shared__ cplx rstg[Sh::RSTG > 0 ? Sh::RSTG / 16 : 1];
  float* stg = reinterpret_cast<float*>(smem);  // [2][WAVES][CQ][4][VP]
  float* afr = reinterpret_cast<float*>(smem + Sh::STAGE);  // [2][CQ][64][2 nb]
  constexpr int NTHR = WAVES * 64, NE = (CQ * 64 + NTHR - 1) / NTHR;
  static_assert(sizeof(smem) >= 8 * extras_lds<NB>(), "the extra blocks' LDS");
  const int nx = x.blocks(d);
  if ((int)blockIdx.x < nx) {
    extras_block<NB>(d, x, blockIdx.x, smem);
    return;
  }
  const int task = (blockIdx.x - nx) / d.nk;
  const int k = blockIdx.x - nx - task * d.nk;
  const HistTask ht = hist_task<64>(task, m, lgL);
  const int s = ht.s, r0 = ht.r0, r1 = ht.r1;
  const int qs = (r0 - 64 * s) >> 2;      // the segment's first quad
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = HS == 1 ? (wv >> 1) : wv;
  const int h0 = HS == 1 ? (wv & 1) : 0;   // first component half of this wavefront
  const int r = lane >> 4, n = lane & 15;
  const int tp = 64 * s + 16 * g + n;
  const bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  // row-term Sigma of this lane's column: half 0 (G^<) takes -Sigma^>, half 1 (G^>) +Sigma^<
  cplx32 Srow[HS * NBB];
#pragma unroll
  for (int hh = 0; hh < HS; ++hh) {
    const int H = h0 + hh;
    const float sg = H ? 1.f : -1.f;
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      cplx v = colv ? sk[((1 - H) * NBB + e) * d.Tp + tp] : czero();
      Srow[hh * NBB + e] = make_float2(sg * (float)v.x, sg * (float)v.y);
    }
  }
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 D[HS][NB];
  double col[HS][NB][4];
#pragma unroll
  for (int hh = 0; hh < HS; ++hh)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      D[hh][b] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) col[hh][b][v] = 0.0;
    }
  // lane's 16-byte loads of quad q: float4 index (q C 128) + (g C/2 + ci) 64 + lane
  const kbe_f4v* hq = reinterpret_cast<const kbe_f4v*>(hist) +
                      ((int64_t)k * C * d.P + 256 * (int64_t)C * quad_base(s, d.N)) / 2 +
                      (int64_t)(g * (C / 2) + h0 * (NBB / 2)) * 64 + lane;
  const int nq = (r1 - 64 * s + 3) >> 2;  // one past its last (segments are whole chunks of 64 rows,
                                          // or end at m)
  constexpr int PF = Sh::PF, RING = PF + 1;
  static_assert(CQ % RING == 0, "a chunk holds whole turns of the load ring");
  // quad x lives in ring[x % RING]; its loads are issued while quad x - PF is processed
  kbe_f4v ring[RING][NCH];
  // loads are never behind a branch (a quad index past the last is clamped to it), so the
  // waits for one quad's data leave the later quads' loads in flight. Quads q < 4 g lie wholly
  // above the diagonal for this wavefront's columns (16 g .. 16 g + 15 of the strip): their loads
  // are pointed at quad 4 g, which the wavefront reads anyway (cache hits instead of HBM traffic
  // for the unused part of the strip's triangle); the masks zero them.
  const int qlo = 4 * g < nq - 1 ? 4 * g : nq - 1;
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int qu = qs + u < qlo ? qlo : (qs + u < nq ? qs + u : nq - 1);
#pragma unroll
    for (int i = 0; i < NCH; ++i) ring[u][i] = __builtin_nontemporal_load(hq + (int64_t)qu * 128 * C + i * 64);
  }
  cplx* rp = const_cast<cplx*>(rowpart_slot(d, rowpart, k, s));
  AfrFill<NB, NE> fill;
  fill.load(d, sk, s, qs, r1, threadIdx.x, NTHR);
  fill.store(afr, threadIdx.x, NTHR);
  __syncthreads();
  int buf = 0;
  for (int q0 = qs, ci = 0; q0 < nq; q0 += CQ, ++ci) {
    float* sb = stg + buf * (WAVES * CQ * 4 * VP);
    const float* ab = afr + buf * (CQ * 64 * 2 * NB);
    const bool more = q0 + CQ < nq;
    if (more) fill.load(d, sk, s, q0 + CQ, r1, threadIdx.x, NTHR);  // the next chunk's A operands
    for (int qt = 0; qt < CQ; qt += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      const int qc = qt + u;
      const int q = q0 + qc;   // quads past the last run masked (all zero), so that every chunk
                               // issues the same loads and the waits at its end stay exact
      {
        const int qn = q + PF < qlo ? qlo : (q + PF < nq ? q + PF : nq - 1);
        const kbe_f4v* nx = hq + (int64_t)qn * 128 * C;
#pragma unroll
        for (int i = 0; i < NCH; ++i) ring[(u + PF) % RING][i] = __builtin_nontemporal_load(nx + i * 64);
      }
      const kbe_f4v* cur = ring[u];
      const int j0 = 64 * s + 4 * q;
      const int j = j0 + r;
      auto quad = [&](auto tag) {
        constexpr bool MASKED = decltype(tag)::value;
        cplx32 G[HS * NBB];
        const bool valid = MASKED ? (colv && tp <= j && j < r1) : true;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
          G[2 * i] = valid ? make_float2(cur[i].x, cur[i].y) : make_float2(0.f, 0.f);
          if (2 * i + 1 < HS * NBB) G[2 * i + 1] = valid ? make_float2(cur[i].z, cur[i].w) : make_float2(0.f, 0.f);
        }
        // A operand of this lane: Sigma^R(t_j)_{a l}, real-embedded and split (staged)
        float Af[NB][2];
        const float* af = ab + (qc * 64 + lane) * 2 * NB;
#pragma unroll
        for (int l = 0; l < NB; ++l) {
          Af[l][0] = af[2 * l];
          Af[l][1] = af[2 * l + 1];
        }
#pragma unroll
        for (int l = 0; l < NB; ++l)
#pragma unroll
          for (int ri = 0; ri < 2; ++ri)
#pragma unroll
            for (int hh = 0; hh < HS; ++hh)
#pragma unroll
              for (int b = 0; b < NB; ++b) {
                const cplx32 gv = G[hh * NBB + l * NB + b];
                D[hh][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(Af[l][ri], ri ? gv.y : gv.x, D[hh][b], 0, 0, 0);
              }
        // row term of this lane's pair
        float x[VP];
#pragma unroll
        for (int i = 0; i < VP; ++i) x[i] = 0.f;
#pragma unroll
        for (int hh = 0; hh < HS; ++hh)
#pragma unroll
          for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
              cplx32 t = make_float2(0.f, 0.f);
#pragma unroll
              for (int l = 0; l < NB; ++l) cmacc32(t, Srow[hh * NBB + a * NB + l], G[hh * NBB + b * NB + l]);
              x[2 * (a * NB + b)] += t.x;
              x[2 * (a * NB + b) + 1] += t.y;
            }
        if constexpr (MASKED) {
          const bool rv = tp < j;   // the diagonal belongs to the end-point terms
#pragma unroll
          for (int i = 0; i < VP; ++i) x[i] = rv ? x[i] : 0.f;
        }
        reduce_scatter16<VP>(x, lane);
        float* row = sb + ((wv * CQ + qc) * 4 + r) * VP;
        if constexpr (VP >= 16) {
#pragma unroll
          for (int i = 0; i < VP / 16; ++i) row[(VP / 16) * n + i] = x[i];
        } else {
          if (n % (16 / VP) == 0) row[n / (16 / VP)] = x[0];
        }
      };
      if (q >= 16 && j0 + 4 <= r1)   // (q >= nq implies j0 >= r1: masked)
        quad(BoolTag<false>{});
      else
        quad(BoolTag<true>{});
    }
    }
    if (more) fill.store(afr + (buf ^ 1) * (CQ * 64 * 2 * NB), threadIdx.x, NTHR);
    // FP32 tiles of this chunk into the FP64 column sums
#pragma unroll
    for (int hh = 0; hh < HS; ++hh)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int v = 0; v < 4; ++v) col[hh][b][v] += (double)D[hh][b][v];
        D[hh][b] = f4{0.f, 0.f, 0.f, 0.f};
      }
    __syncthreads();  // the chunk is staged by every wavefront; the other buffer is free again
    // row partials of the chunk: the wavefronts' parts added in a fixed order
    for (int o = threadIdx.x; o < 4 * CQ * NBB; o += WAVES * 64) {
      const int e = o / (4 * CQ), rho = o - e * (4 * CQ);
      const int jj = 64 * s + 4 * q0 + rho;
      if (jj < r1) {
        double re = 0.0, im = 0.0;
        for (int w = 0; w < WAVES; ++w) {
          const float* src = sb + (w * CQ * 4 + rho) * VP + 2 * e;
          re += (double)src[0];
          im += (double)src[1];
        }
        if constexpr (CPF > 1)
          rstg[e * Sh::ROWS + (ci % CPF) * 4 * CQ + rho] = cmk(re, im);
        else
          store_stream(rp + (int64_t)e * d.Tp + jj, cmk(re, im));
      }
    }
    if constexpr (CPF > 1) {
      if (ci % CPF == CPF - 1 || !more) {
        __syncthreads();
        const int base = 64 * s + 4 * q0 - (ci % CPF) * 4 * CQ;
        const int end = 64 * s + 4 * q0 + 4 * CQ;
        const int nrows = (end < r1 ? end : r1) - base;
        for (int o = threadIdx.x; o < NBB * nrows; o += WAVES * 64) {
          const int e = o / nrows, row = o - e * nrows;
          store_stream(rp + (int64_t)e * d.Tp + base + row, rstg[e * Sh::ROWS + row]);
        }
        __syncthreads();
      }
    }
    buf ^= 1;
  }
  // column sums: high and low parts of each tile added in FP64 through LDS
  __syncthreads();  // every wavefront is done with the staging buffers
  double* fin = reinterpret_cast<double*>(smem) + (int64_t)wv * HS * NB * 256;
#pragma unroll
  for (int hh = 0; hh < HS; ++hh)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) fin[((hh * NB + b) * 16 + 4 * r + v) * 16 + n] = col[hh][b][v];
  __syncthreads();
  const int a = lane >> 4;
  if (a < NB && colv) {
#pragma unroll
    for (int hh = 0; hh < HS; ++hh)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const double* t = fin + (hh * NB + b) * 256;
        const int mre = 2 * a, mim = 2 * a + 1, lo = 2 * NB;
        double re = t[mre * 16 + n] + t[(lo + mre) * 16 + n];
        double im = t[mim * 16 + n] + t[(lo + mim) * 16 + n];
        const int c = (h0 + hh) * NBB + a * NB + b;
        colpart[colpart_idx(d, k, ht.g, c, tp)] = cmk(re, im);
      }
  }
}

// ------------------------------------------------------------------ row assembly and update
// A block carries 64 consecutive t' of one k; its wavefront w = sc NB + a carries row a of
// component sc (2 NB wavefronts, lane = t').
//  EVAL/CORRECT, t' < m: I^{<,>}(t_m, t') = dt [bulk + end-point terms], where the
//   trapezoid corrections of the two integrals of eq. (CI) are
//     + 1/2 SR_mm G_{m t'} - 1/2 SR_m0 G_{0 t'}                                  (first, [0, t_m])
//     + [t' > 0] (-1/2 Sigma_{m t'} GR_{t' t'} + 1/2 Sigma_{m0} GR_{0 t'})       (second, [0, t'])
//   with GR = G^> - G^<, G_{0 t'} = -(G_{t' 0})^dag.
//  PREDICT/CORRECT, t' < m: G(t_m, t') = V G(t_{m-1}, t') + Phi Ibar(t').
//  PREDICT/CORRECT, t' = m: rho_m = V rho_{m-1} V^dag - dt Vh Dbar Vh^dag and the
//   equal-time block G^< = i rho_m, G^> = -i (1 - rho_m).
//  EVAL_NEXT (trapezoid, nb <= 2): EVAL of row m, then PREDICT of row m + 1 with the collision row in
//   registers. The predictor of a t' needs the evaluation of that t' alone, and what a block writes for
//   row m + 1 (working row, history, edge copies) no block reads for row m. One launch less on the
//   critical path of a step: 50.8 -> 49.4 us (16 points, m <= 200), 72.8 -> 69.9 (61 points, nb = 1, m <= 300),
//   249 -> 247 (144 points, m <= 400).
// Bound: HBM, then the latency of the loads. With whole nb x nb blocks in one thread the kernel
// held 118-500 registers, one to four waves per SIMD, and at nb = 4 needed a separate pass that summed
// the strips' row partials and a corrector split into two launches; a matrix row per wavefront needs
// NB complex accumulators, makes Sigma(t_m, t_m), Sigma(t_m, t_0), V and Phi wavefront-uniform (scalar
// loads), and spreads the gather of the row partials over all wavefronts. What several rows need
// (G_{0 t'}, GR_{t' t'}, the gathered row partials; then Ibar and G(t_{m-1}, t')) is loaded once per
// block and passed through LDS. Averages, before -> now: evaluation 9.9 -> 7.1 us (144 points, nb = 2,
// m <= 400), 127 -> 116 us (576 points, nb = 2, m = 1000, 5.1 TB/s), 318 (with the row-partial pass) -> 196 us
// (256 points, nb = 4, m = 800, 5.1 TB/s); corrector with four Gregory nodes 86 -> 30 us (63 points, nb = 3,
// m <= 150).
//
// Gregory corrections: element (a, b) of component sc of the block G(t_j, t') an end correction of
// output t' < m needs: the diagonal from the band copy; stored blocks j > t' from the ring of recent
// rows (row m: the current iterate) or the column copies (j < qp); blocks above the diagonal as
// -G_{t' j}^dag from the column copies (j < qp) or the band (t' - j < qp). Every node the
// corrections visit is in one of these.
template <int NB>
struct EndBlock {
  const cplx* p;     // component 0
  int64_t stride;    // one component further
  bool flip;         // element (a, b) is -conj of the stored (b, a)
  __device__ __forceinline__ EndBlock(const Dims& d, const cplx* __restrict__ row64, const cplx* __restrict__ colq,
                                      const cplx* __restrict__ band, int k, int m, int j, int tp) {
    flip = j < tp;
    stride = (int64_t)d.qp * d.Tp;
    if (j == tp) {
      p = band + band_idx(d, k, 0, tp, 0);
    } else if (j > tp) {
      if (j > m - d.rring) {
        p = row64 + row64_idx(d, j, k, 0, tp);
        stride = d.Tp;
      } else {
        p = colq + colq_idx(d, k, 0, j, tp);
      }
    } else {
      p = j < d.qp ? colq + colq_idx(d, k, 0, tp, j) : band + band_idx(d, k, 0, tp, tp - j);
    }
  }
  __device__ __forceinline__ cplx at(int sc, int a, int b) const {
    cplx v = p[(sc * NB * NB + (flip ? b * NB + a : a * NB + b)) * stride];
    return flip ? cneg(cconj(v)) : v;
  }
};

template <int NB, int MODE, bool GREG>
__global__ __launch_bounds__(128 * NB) void k_row(Dims d, void* __restrict__ hist, cplx* __restrict__ row64,
                                                  const cplx* __restrict__ sig, const cplx* __restrict__ colpart,
                                                  const cplx* __restrict__ rowpart, cplx* __restrict__ col0,
                                                  cplx* __restrict__ diag, const cplx* __restrict__ Iprev,
                                                  cplx* __restrict__ Icur, const cplx* __restrict__ props,
                                                  const cplx* __restrict__ rho_prev, cplx* __restrict__ rho_cur,
                                                  const cplx* __restrict__ Dprev, const cplx* __restrict__ Dcur, int m,
                                                  int lgL, double dt, int commit, double* __restrict__ chg, QuadW Q) {
  constexpr int NBB = NB * NB;
  constexpr bool NEXT = MODE == KBE_ROW_EVAL_NEXT;
  constexpr bool INT = MODE == KBE_ROW_CORRECT || MODE == KBE_ROW_EVAL || NEXT;   // collision row
  constexpr bool UPD = MODE != KBE_ROW_EVAL;                              // update of the row
  __shared__ cplx lds[4 * NBB * 64];
  const int k = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sc = w / NB, a = w - (w / NB) * NB;
  const int tp = blockIdx.x * 64 + lane;
  const bool in = tp < m;
  double dmax = 0.0;
  cplx In[NB];   // the collision row over dt
  if constexpr (INT) {
    cplx* s0 = lds;                    // G(t_0, t') of both components: G_00, or -G(t', t_0)^dag
    cplx* sR = lds + 2 * NBB * 64;     // GR_{t' t'}
    cplx* sP = lds + 3 * NBB * 64;     // row partials of the history sums, summed over the slots
    if (in) {
      if constexpr (!GREG) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          cplx v = tp == 0 ? col0[colq_idx(d, k, sc * NBB + a * NB + b, 0, 0)]
                           : cneg(cconj(col0[colq_idx(d, k, sc * NBB + b * NB + a, tp, 0)]));
          s0[(sc * NBB + a * NB + b) * 64 + lane] = v;
        }
      }
      // the two wavefronts of row a share its entries b
#pragma unroll
      for (int h = 0; h < (NB + 1) / 2; ++h) {
        const int b = 2 * h + sc;
        if (b < NB) {
          const int e = a * NB + b;
          if constexpr (!GREG)
            sR[e * 64 + lane] = csub(diag[band_idx(d, k, NBB + e, tp, 0)], diag[band_idx(d, k, e, tp, 0)]);
          // slots in order, in groups of 4 whose loads are issued together
          const int nslot = (tp >> 6) / d.spb + 1;
          const cplx* rp = rowpart_slot(d, rowpart, k, 0) + (int64_t)e * d.Tp + tp;
          const int64_t step = (int64_t)d.nbb * d.Tp;
          cplx rs = czero();
          int q = 0;
          for (; q + 4 <= nslot; q += 4) {
            cplx v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = rp[(q + u) * step];
#pragma unroll
            for (int u = 0; u < 4; ++u) rs = cadd(rs, v[u]);
          }
          for (; q < nslot; ++q) rs = cadd(rs, rp[q * step]);
          sP[e * 64 + lane] = rs;
        }
      }
    }
    // end-point terms of row a of component sc, accumulated term by term
    cplx E[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) E[b] = czero();
    // E += f S G: S[a][l] of Sigma component cs at t_j, G[l][b] from g(l, b)
    auto sigma_row = [&](int cs, int j, cplx* S) {
#pragma unroll
      for (int l = 0; l < NB; ++l) S[l] = sig[sig_idx(d, k, cs, a * NB + l, j)];
    };
    auto add = [&](cplx* S, double f, auto g) {
#pragma unroll
      for (int l = 0; l < NB; ++l) S[l] = cscal(S[l], f);
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int l = 0; l < NB; ++l) cmac(E[b], S[l], g(l, b));
    };
    auto term = [&](int cs, int j, double f, auto g) {
      cplx S[NB];
      sigma_row(cs, j, S);
      add(S, f, g);
    };
    if constexpr (GREG) {
      // Gregory end corrections (d.qp nodes per end): against the bulk's unit weights,
      //   E = sum_j (w^(m)_j - [j < m]) SR_mj G_jt'  +  sum_{j <= t'} (w^(t')_j - [j < t']) Sigma_mj GA_jt',
      // nonzero on the nodes j < q' and j > N - q' of each interval (q' = min(qp, N + 1)). Per step
      // every wavefront loads its row of one block into LDS for all of them (each block is wanted by NB
      // or 2 NB wavefronts), the next step's rows of G and Sigma meanwhile in flight and the corrections in
      // LDS: 30.4 -> 27.3 us per corrector launch at nb = 3, 63 points, m <= 150, q = 4, against whole blocks
      // loaded by each wavefront.
      auto put = [&](const cplx* v) {
#pragma unroll
        for (int b = 0; b < NB; ++b) s0[(sc * NBB + a * NB + b) * 64 + lane] = v[b];
      };
      cplx v[NB], S0[NB], S1[NB];
      // weight of node j on [0, N], N >= 1, less the bulk's unit weight on j < N (quad_w, corrections in LDS)
      __shared__ double qc[KBE_QMAX + 1][KBE_QMAX];
      for (int i = threadIdx.x; i < (KBE_QMAX + 1) * KBE_QMAX; i += 128 * NB) qc[i / KBE_QMAX][i % KBE_QMAX] = Q.c[i / KBE_QMAX][i % KBE_QMAX];
      auto weight = [&](int j, int N) {
        const int qq = Q.q < N + 1 ? Q.q : N + 1;
        const double w0 = qc[qq][j < qq ? j : 0], w1 = qc[qq][N - j < qq ? N - j : 0];
        return (j < N ? 0.0 : 1.0) + (j < qq ? w0 : 0.0) + (N - j < qq ? w1 : 0.0);
      };
      // first integral: the nodes are the same in every lane; slot sc holds component sc
      {
        const int qm = d.qp < m + 1 ? d.qp : m + 1, hi = qm > m - qm + 1 ? qm : m - qm + 1;
        const int n = qm + m + 1 - hi;
        auto node = [&](int i) { return i < qm ? i : hi + i - qm; };
        auto load = [&](int jn, cplx* S) {
          if (in) {
            const EndBlock<NB> G(d, row64, col0, diag, k, m, jn, tp);
#pragma unroll
            for (int b = 0; b < NB; ++b) v[b] = G.at(sc, a, b);
          }
          sigma_row(2, jn, S);
        };
        load(node(0), S0);
        for (int i = 0; i < n; ++i) {
          put(v);
          __syncthreads();
          if (i + 1 < n) load(node(i + 1), S1);
          if (in)
            add(S0, weight(node(i), m), [&](int l, int b) { return s0[(sc * NBB + l * NB + b) * 64 + lane]; });
#pragma unroll
          for (int l = 0; l < NB; ++l) S0[l] = S1[l];
          __syncthreads();
        }
      }
      // second integral, nodes u (slot 0) and t' - u (slot 1): the wavefronts of component sc load slot sc
      {
        const int qt = d.qp < tp + 1 ? d.qp : tp + 1;
        const int n0 = in && tp > 0 ? qt : 0;                                       // nodes 0 .. qt - 1
        const int n1 = in && tp > 0 ? (qt < tp + 1 - qt ? qt : tp + 1 - qt) : 0;    // the rest of t' - qt + 1 .. t'
        cplx T0[NB], T1[NB];
        auto load = [&](int u, cplx* S, cplx* T) {
          if (u < (sc ? n1 : n0)) {
            const EndBlock<NB> G(d, row64, col0, diag, k, m, sc ? tp - u : u, tp);
#pragma unroll
            for (int b = 0; b < NB; ++b) v[b] = csub(G.at(0, a, b), G.at(1, a, b));   // -(G^> - G^<)
          }
          if (u < n0) sigma_row(sc, u, S);
          if (u < n1) sigma_row(sc, tp - u, T);
        };
        load(0, S0, T0);
        for (int u = 0; u < d.qp; ++u) {
          put(v);
          __syncthreads();
          if (u + 1 < d.qp) load(u + 1, S1, T1);
          if (u < n0) add(S0, weight(u, tp), [&](int l, int b) { return s0[(l * NB + b) * 64 + lane]; });
          if (u < n1) add(T0, weight(tp - u, tp), [&](int l, int b) { return s0[(NBB + l * NB + b) * 64 + lane]; });
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            S0[l] = S1[l];
            T0[l] = T1[l];
          }
          __syncthreads();
        }
      }
    } else {
      __syncthreads();
    }
    if (in) {
      if constexpr (!GREG) {
        // trapezoid: half weights at j = 0 and j = m (first integral), j = 0 and j = t' (second)
        term(2, m, 0.5, [&](int l, int b) { return row64[row64_idx(d, m, k, sc * NBB + l * NB + b, tp)]; });
        term(2, 0, -0.5, [&](int l, int b) { return s0[(sc * NBB + l * NB + b) * 64 + lane]; });
        if (tp > 0) {
          term(sc, tp, -0.5, [&](int l, int b) { return sR[(l * NB + b) * 64 + lane]; });
          term(sc, 0, 0.5, [&](int l, int b) {
            return csub(s0[(NBB + l * NB + b) * 64 + lane], s0[(l * NB + b) * 64 + lane]);
          });
        }
      }
      // column sums over the row segments, in groups whose loads are issued together
      const int nseg = hist_nseg(m - 64 * d.spb * (tp / (64 * d.spb)), lgL);
      const cplx* cp = colpart + colpart_idx(d, k, 0, sc * NBB + a * NB, tp);
      const int64_t cstep = (int64_t)d.C * d.Tp;
      constexpr int CG = NB <= 2 ? 4 : 2;
      cplx cs[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) cs[b] = cp[b * (int64_t)d.Tp];
      int sg = 1;
      for (; sg + CG <= nseg; sg += CG) {
        cplx v[CG][NB];
#pragma unroll
        for (int u = 0; u < CG; ++u)
#pragma unroll
          for (int b = 0; b < NB; ++b) v[u][b] = cp[(sg + u) * cstep + b * (int64_t)d.Tp];
#pragma unroll
        for (int u = 0; u < CG; ++u)
#pragma unroll
          for (int b = 0; b < NB; ++b) cs[b] = cadd(cs[b], v[u][b]);
      }
      for (; sg < nseg; ++sg)
#pragma unroll
        for (int b = 0; b < NB; ++b) cs[b] = cadd(cs[b], cp[sg * cstep + b * (int64_t)d.Tp]);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int e = a * NB + b;
        In[b] = cadd(cadd(cs[b], sP[e * 64 + lane]), E[b]);
        Icur[rowbuf_idx(d, k, sc * NBB + e, tp)] = cscal(In[b], dt);
      }
    }
  }
  if constexpr (UPD) {
    const int mu = NEXT ? m + 1 : m;               // the row that is updated
    const cplx* P = props + (int64_t)k * 3 * NBB;
    cplx* sI = lds + sc * NBB * 64;                // Ibar of this component
    cplx* sG = lds + (2 + sc) * NBB * 64;          // G(t_{m-1}, t')
    if constexpr (INT) __syncthreads();            // the first part's LDS is free
    if (tp < mu) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int e = a * NB + b;
        // (NEXT: the row just computed, its equal-time entry from the history pass)
        cplx ip = NEXT && in ? cscal(In[b], dt) : (NEXT ? Icur : Iprev)[rowbuf_idx(d, k, sc * NBB + e, tp)];
        if constexpr (MODE == KBE_ROW_CORRECT) ip = cscal(cmk(fma(In[b].x, dt, ip.x), fma(In[b].y, dt, ip.y)), 0.5);
        sI[e * 64 + lane] = ip;
        sG[e * 64 + lane] = row64[row64_idx(d, mu - 1, k, sc * NBB + e, tp)];
      }
    }
    __syncthreads();
    if (tp <= mu) {
      cplx g[NB];   // the new row a of component sc
      if (tp < mu) {
        cplx V[NB], Phi[NB];
#pragma unroll
        for (int l = 0; l < NB; ++l) {
          V[l] = P[a * NB + l];
          Phi[l] = P[2 * NBB + a * NB + l];
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          g[b] = czero();
#pragma unroll
          for (int l = 0; l < NB; ++l) cmac(g[b], V[l], sG[(l * NB + b) * 64 + lane]);
#pragma unroll
          for (int l = 0; l < NB; ++l) cmac(g[b], Phi[l], sI[(l * NB + b) * 64 + lane]);
        }
      } else {
        // t' = mu: row a of rho_mu = (V rho) V^dag - dt (Vh Dbar) Vh^dag, the same in both components
        cplx t1[NB], t2[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          t1[b] = t2[b] = czero();
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            const int e = l * NB + b;
            cplx db = Dprev[(int64_t)k * NBB + e];
            if (MODE == KBE_ROW_CORRECT) db = cscal(cadd(db, Dcur[(int64_t)k * NBB + e]), 0.5);
            cmac(t1[b], P[a * NB + l], rho_prev[(int64_t)k * NBB + e]);
            cmac(t2[b], P[NBB + a * NB + l], db);
          }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          cplx r = czero(), x = czero();
#pragma unroll
          for (int l = 0; l < NB; ++l) {
            cmacc(r, t1[l], P[b * NB + l]);
            cmacc(x, t2[l], P[NBB + b * NB + l]);
          }
          cplx rv = cmk(fma(x.x, -dt, r.x), fma(x.y, -dt, r.y));
          if (sc == 0) rho_cur[(int64_t)k * NBB + a * NB + b] = rv;
          g[b] = sc == 0 ? cmuli(rv) : cneg(cmuli(csub(cmk(a == b ? 1.0 : 0.0, 0.0), rv)));
        }
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int c = sc * NBB + a * NB + b;
        if (MODE == KBE_ROW_CORRECT && chg) {
          // change against the iterate this pass started from; one that is not a number counts as
          // infinite (the maxima over lanes, wavefronts and blocks would drop it)
          const cplx dg = csub(g[b], row64[row64_idx(d, m, k, c, tp)]);
          const double c2 = dg.x * dg.x + dg.y * dg.y;
          dmax = fmax(dmax, c2 >= 0.0 ? sqrt(c2) : INFINITY);
        }
      }
      // a corrector wavefront reads only its own row of the old iterate above, but the end-point
      // terms of every row read the whole block: they are behind a block barrier
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int c = sc * NBB + a * NB + b;
        row64[row64_idx(d, mu, k, c, tp)] = g[b];
        if (commit) {
          commit_store(d, hist, k, c, mu, tp, g[b]);
          if (tp < d.qp) col0[colq_idx(d, k, c, mu, tp)] = g[b];
          if (mu - tp < d.qp) diag[band_idx(d, k, c, mu, mu - tp)] = g[b];
        }
      }
    }
    if (MODE == KBE_ROW_CORRECT && chg) {   // one value per block: its largest change
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
      __syncthreads();
      double* red = reinterpret_cast<double*>(lds);
      if (lane == 0) red[w] = dmax;
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int i = 1; i < 2 * NB; ++i) dmax = fmax(dmax, red[i]);
        chg[(int64_t)k * gridDim.x + blockIdx.x] = dmax;
      }
    }
  }
}

// Largest change of the corrector's row: out[0] = max over the row kernel's n blocks; out is in host
// memory, which saves the copy that the host would wait for.
// One block, a fixed reduction order (max is exact, so any order gives the same value); infinite if any
// change is infinite or not a number, which the caller reports.
__global__ __launch_bounds__(1024) void k_change_max(const double* __restrict__ chg, int n, double* __restrict__ out) {
  __shared__ double red[16];
  double mx = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) mx = fmax(mx, chg[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 16; ++i) mx = fmax(mx, red[i]);
    out[0] = mx;
  }
}

// ------------------------------------------------------------------ dipole kick
// The kick of the dipole pulse of eq. (dipole) on the completed slice m: G(t_m, t') <- K G(t_m, t')
// for t' < m and K G K^dag on the equal-time block (both components), rho_m <- K rho_m K^dag,
// K = kc 1 - i ks X (X: ones between bands 0 and 1; nb = 2). Thread per (k, t'); the FP64
// working copy of the row is the source, and every copy of the row is rewritten (packed
// history, working copy, column and diagonal copies). rho goes to rhoX and rhoY (both density
// buffers at t = 0).
template <int NB>
__global__ __launch_bounds__(256) void k_kick_row(Dims d, void* __restrict__ hist, cplx* __restrict__ row64,
                                                  cplx* __restrict__ col0, cplx* __restrict__ diag, cplx* rhoX,
                                                  cplx* rhoY, int m, double kc, double ks) {
  static_assert(NB == 2, "the dipole kick couples the two bands of the paper's model");
  int k = blockIdx.y;
  int tp = blockIdx.x * 256 + threadIdx.x;
  if (tp > m) return;
  // (K G)_ab = kc G_ab - i ks G_{1-a, b};  (T K^dag)_ab = kc T_ab + i ks T_{a, 1-b}
  auto kick = [&](const cplx* G, cplx* out, bool both_sides) {
    cplx T[4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) T[a * 2 + b] = csub(cscal(G[a * 2 + b], kc), cmuli(cscal(G[(1 - a) * 2 + b], ks)));
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        out[a * 2 + b] = both_sides ? cadd(cscal(T[a * 2 + b], kc), cmuli(cscal(T[a * 2 + 1 - b], ks))) : T[a * 2 + b];
  };
#pragma unroll
  for (int sc = 0; sc < 2; ++sc) {
    cplx G[4], R[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) G[e] = row64[row64_idx(d, m, k, sc * 4 + e, tp)];
    kick(G, R, tp == m);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int c = sc * 4 + e;
      row64[row64_idx(d, m, k, c, tp)] = R[e];
      commit_store(d, hist, k, c, m, tp, R[e]);
      if (tp < d.qp) col0[colq_idx(d, k, c, m, tp)] = R[e];
      if (m - tp < d.qp) diag[band_idx(d, k, c, m, m - tp)] = R[e];
    }
  }
  if (tp == m) {
    cplx r[4], R[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = rhoX[(int64_t)k * 4 + e];
    kick(r, R, true);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      rhoX[(int64_t)k * 4 + e] = R[e];
      rhoY[(int64_t)k * 4 + e] = R[e];
    }
  }
}

// ------------------------------------------------------------------ aux copies
// Refresh the FP64 working copies from history rows 0..m: columns 0..qp-1, the diagonal band
// of width qp, and the ring of the last rring rows (m - rring + 1 .. m).
template <int NB>
__global__ void k_aux(Dims d, const void* __restrict__ hist, cplx* __restrict__ row64, cplx* __restrict__ col0,
                      cplx* __restrict__ diag, int m) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  int kc = blockIdx.y;
  if (j > m) return;
  int k = kc / d.C, c = kc - (kc / d.C) * d.C;
  for (int q = 0; q < d.qp && q <= j; ++q) {
    col0[colq_idx(d, k, c, j, q)] = history_load(d, hist, k, c, j, q);
    diag[band_idx(d, k, c, j, q)] = history_load(d, hist, k, c, j, j - q);
  }
  for (int r = m; r >= 0 && r > m - d.rring; --r)
    if (j <= r) row64[row64_idx(d, r, k, c, j)] = history_load(d, hist, k, c, r, j);
}

// ------------------------------------------------------------------ launchers
// Dynamic LDS above 64 KB (the self-energy tile of a long chain: 82 KB at N_k = 1024) is asked
// for explicitly; gfx950 gives a workgroup up to 160 KB.
static hipError_t allow_lds(const void* kern, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Blocks of 64 t' per k of the row kernel: t' < m in the evaluation mode, t' <= m otherwise.
static int row_tiles(int m, int mode) { return mode == KBE_ROW_EVAL ? (m + 63) / 64 : m / 64 + 1; }

// Wavefronts per block of the FP64 nb <= 2 kernel: at nb = 2 eight where that is less time in rounds of
// the chip (its registers allow two wavefronts per SIMD, so it holds 512 blocks of four or 256 of eight,
// which take half as long each): the same rows in flight with half the blocks to start and to combine.
// With one strip pair (m <= 128) the blocks are equal: eight wins up to 256 points and, from 64 rows on
// (below, the small blocks in front of the pass weigh more), for the last half-empty round of 513..768.
// Four -> eight: 230 points, m = 100 58 -> 47 us; 300 points, m = 128 94 -> 100; 513 points, m = 100 118 -> 111,
// m = 32 37 -> 43; 784 points, m = 16 / 100 33 -> 39, 144 -> 155; 961 points, m = 5 26 -> 36 us. With two pairs
// up to 256 points (256 points, m = 200 146 -> 135 us; 300 points 168 -> 177), with more while the pairs give
// less than two rounds of four-wavefront blocks (300 points, m = 300 353 -> 335 us; 144 points, m = 400
// 272 -> 265 us; but 576 points, m = 300 592 -> 608 us). One band (126 registers, four wavefronts per SIMD):
// 61 points, m = 200 12.1 -> 13.2 us.
static int hist_waves(const Dims& d, int m) {
  if (d.nb != 2 || d.fp32) return 4;
  const int pairs = (m + 127) / 128;
  if (pairs == 1) return d.nk <= 256 || (d.nk > 512 && d.nk <= 768 && m >= 64) ? 8 : 4;
  return pairs == 2 ? (d.nk <= 256 ? 8 : 4) : (d.nk * pairs < 1024 ? 8 : 4);
}
// Rows per block of a history pass at row m, as a power of two (30: every strip is one block).
// One block per strip leaves a small N_k with fewer blocks than the chip holds at a time (512: two per
// CU; 256 of eight wavefronts), and a medium one with a last round of a few long blocks; shorter blocks
// cost each a prologue and a column combine (5-10 rows' worth of time) and their column sums are read
// once more by the row kernel. Measured best over N_k = 16..1024, m = 20..500, nb = 1..4: blocks of about
// 1.5 times the rows that an even share of the launch would be (a strip's triangular first 64 rows
// count half; 2.2 times with eight wavefronts), at least 16 (32 in the FP64 nb = 4 kernel and 64 in the
// MFMA form, whose blocks work in chunks of that many). FP64, nb = 2, one four-wavefront block per strip ->
// this rule: 16 points, m = 128 / 200 48 -> 13, 84 -> 19 us; 61 points, m = 200 / 400 93 -> 38, 230 -> 120 us;
// 144 points, m = 128 / 200 / 400 66 -> 48, 102 -> 79, 287 -> 265 us; 1024 points 2.76 ms unsplit against
// 2.83 ms in blocks of 256 rows at m = 500.
// Up to one and a half strips the unsplit blocks are about equal and a split has no long ones to level: where
// the last round of unsplit blocks is more than three quarters full it is taken only if it shortens the
// rounds (two segments -> unsplit: 449 points, m = 128 124 -> 113 us; 401 points, m = 32 31 -> 26 us; 961 points,
// FP32, m = 20 42 -> 35 us; but 300 points, FP32, m = 20 18 -> 20 us; nb = 4, FP32, 400 points, m = 20 62 -> 74 us).
static int hist_lgseg(const Dims& d, int m) {
  if (d.cseg == 1) return 30;
  const int W = 64 * d.spb;
  int64_t rows = 0;
  for (int r = m; r > 0; r -= W) rows += r - (r < 64 ? r / 2 : 32);
  const bool eight = hist_waves(d, m) == 8;
  const int slots = eight ? 256 : 512;
  const double share = (eight ? 2.2 : 1.5) * d.nk * (double)rows / slots;
  int lg = d.mfma ? 6 : (d.nb == 4 && !d.fp32 ? 5 : 4);
  while ((2 << lg) <= share && (1 << lg) < m) ++lg;
  while (hist_nseg(m, lg) > d.cseg) ++lg;
  if ((1 << lg) >= m) return 30;
  if (d.nb <= 2 && 2 * m <= 3 * W) {
    const int held = d.nb == 1 ? 1024 : slots;   // blocks the chip holds
    const int n = hist_nseg(m, lg), rounds = (d.nk + held - 1) / held;
    if (4 * (d.nk - (rounds - 1) * held) > 3 * held && (d.nk * n + held - 1) / held >= n * rounds) return 30;
  }
  return lg;
}
// Blocks per k of a history pass whose strips have W columns.
static int hist_tasks(int W, int m, int lgL) {
  int n = 0;
  for (int r = m; r > 0; r -= W) n += hist_nseg(r, lgL);
  return n;
}

template <int NB>
struct Launch {
  static hipError_t init(const Dims& d, const LaunchArgs& a, hipStream_t st) {
    int nb64 = (d.nk + 63) / 64;
    hipLaunchKernelGGL(k_init_eig<NB>, dim3(nb64), dim3(64), 0, st, d, a.hop, a.Ax, a.Ay, a.eig_w, a.eig_U);
    hipLaunchKernelGGL(k_init_mu, dim3(1), dim3(256), 0, st, d.nk * NB, (const double*)a.eig_w, a.temp,
                       a.target, a.mu);
    hipLaunchKernelGGL(k_init_rho<NB>, dim3(nb64), dim3(64), 0, st, d, (const double*)a.eig_w,
                       (const cplx*)a.eig_U, (const double*)a.mu, a.temp, a.rho_prev, a.rho_cur, a.hist,
                       a.row64, a.col0, a.diag);
    return hipGetLastError();
  }
  static int props_blocks(const Dims& d) { return (d.nk + PropsShape<NB>::KPB - 1) / PropsShape<NB>::KPB; }
  static PropsArgs props_args(const LaunchArgs& a, double wb) {
    return {a.hop, a.rho_prev, a.rho_cur, a.hfbuf, a.props, wb, a.U, a.Ax, a.Ay, a.dt, a.interaction, a.hf};
  }
  static ObsArgs obs_args(const LaunchArgs& a, const ObsStep& o) {
    return {a.hop, o.rho, o.Icur, a.obs, o.t, o.A, o.A * a.polx, o.A * a.poly, a.U, a.spin, o.m, a.interaction, a.hf};
  }
  static hipError_t props(const Dims& d, const LaunchArgs& a, double wb, const ObsStep* o, hipStream_t st) {
    const int nobs = o ? 1 : 0;
    hipLaunchKernelGGL(k_props<NB>, dim3(props_blocks(d) + nobs), dim3(256), 0, st, d, props_args(a, wb),
                       o ? obs_args(a, *o) : ObsArgs{}, nobs);
    return hipGetLastError();
  }
  static hipError_t sigma(const Dims& d, const LaunchArgs& a, int m, hipStream_t st) {
    int total = (m + 1) * NB * NB;
    int per = (total + 7) / 8;
    const size_t shm = (size_t)((pow2_chain(d.nkx, d.nky) ? 2 : 4) * d.nk + d.nkx + d.nky) * sizeof(cplx);
    // large grids: twice the threads (a block's LDS leaves room for one to three blocks per CU)
    const bool large = d.nk >= 512;
    const int fit = (int)(163840 / shm);   // blocks whose LDS a CU holds
    auto rounds = [&](int percu) {
      const int held = 256 * (percu < fit ? percu : fit);
      return (total + held - 1) / held;
    };
    const bool five = !large && rounds(5) < rounds(4);
    if constexpr (NB == 2) {
      if (a.interaction == KBE_DEV_INT_INTERBAND) {
        auto fwd = five ? k_sigma_fwd<0, 0, 2> : k_sigma_fwd<0, 0>;
        auto ib = five ? k_sigma_ib<0, 0, 2> : k_sigma_ib<0, 0>;
        if (d.nkx == 16 && d.nky == 1) {
          fwd = k_sigma_fwd<16, 1>;
          ib = k_sigma_ib<16, 1>;
        }
        hipError_t e = allow_lds((const void*)fwd, shm);
        if (e == hipSuccess) e = allow_lds((const void*)ib, shm);
        if (e != hipSuccess) return e;
        int nthr = large ? 512 : 256;
        if (d.nkx == 16 && d.nky == 1) nthr = sigma_threads<16, 1>();
        hipLaunchKernelGGL(fwd, dim3(per * 8), dim3(nthr), shm, st, d, (const cplx*)a.row64, a.gR, m);
        hipLaunchKernelGGL(ib, dim3(per * 8), dim3(nthr), shm, st, d, (const cplx*)a.gR, a.sig, m, a.UU, a.corr);
        return hipGetLastError();
      }
    }
    // grids of the standard workloads with compile-time transforms, any other grid at run time
    auto kern = five ? k_sigma<NB, 0, 0, 2> : k_sigma<NB, 0, 0>;
    int nthr = large ? 512 : 256;
    if (d.nkx == 24 && d.nky == 24) kern = k_sigma<NB, 24, 24>, nthr = sigma_threads<24, 24>();
    else if (d.nkx == 16 && d.nky == 16) kern = k_sigma<NB, 16, 16>, nthr = sigma_threads<16, 16>();
    else if (d.nkx == 12 && d.nky == 12) kern = k_sigma<NB, 12, 12>, nthr = sigma_threads<12, 12>();
    else if (d.nkx == 16 && d.nky == 1) kern = k_sigma<NB, 16, 1>, nthr = sigma_threads<16, 1>();
    hipError_t e = allow_lds((const void*)kern, shm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(per * 8), dim3(nthr), shm, st, d, (const cplx*)a.row64, a.sig, m, a.UU, a.corr);
    return hipGetLastError();
  }
  // the history sums and the equal-time integral of row m; props: those propagators too
  static hipError_t collide(const Dims& d, const LaunchArgs& a, int m, const LaunchArgs* props, double wb,
                            const ObsStep* o, hipStream_t st) {
    PassExtras x{a.row64, a.sig, a.I_cur, a.D_cur, a.dt, a.quad, m, props ? props_blocks(d) : 0,
                 props_args(props ? *props : a, wb), o ? 1 : 0, o ? obs_args(a, *o) : ObsArgs{}};
    const int nx = x.blocks(d);
    if (m < 1) {
      hipLaunchKernelGGL(k_extras<NB>, dim3(nx), dim3(256), 0, st, d, x);
      return hipGetLastError();
    }
    const int lgL = hist_lgseg(d, m);
    const int ns = hist_tasks(64 * d.spb, m, lgL);
    if (d.mfma) {
      hipLaunchKernelGGL(k_hist_mfma<NB>, dim3(nx + ns * d.nk), dim3(MfmaShape<NB>::WAVES * 64), 0, st, d,
                         (const float2*)a.hist, (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
      return hipGetLastError();
    }
    if constexpr (NB <= 2) {
      if (d.fp32)
        hipLaunchKernelGGL(k_hist_pair32<NB>, dim3(nx + ns * d.nk), dim3(256), 0, st, d, (const cplx32*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
      else
      {
        auto kern = k_hist_pair<NB, 4>;
        const int waves = NB == 2 ? hist_waves(d, m) : 4;
        if constexpr (NB == 2)
          if (waves == 8) kern = k_hist_pair<NB, 8>;
        hipLaunchKernelGGL(kern, dim3(nx + ns * d.nk), dim3(64 * waves), 0, st, d, (const cplx*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
      }
    } else if constexpr (NB == 4) {
      if (d.fp32)
        hipLaunchKernelGGL(k_hist_bulk32_split<NB>, dim3(nx + ns * d.nk), dim3(256), 0, st, d, (const cplx32*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
      else
        hipLaunchKernelGGL(k_hist_bulk_split<NB>, dim3(nx + ns * d.nk), dim3(256), 0, st, d, (const cplx*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
    } else {
      if (d.fp32)
        hipLaunchKernelGGL(k_hist_bulk32<NB>, dim3(nx + ns * d.nk), dim3(256), 0, st, d, (const cplx32*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
      else
        hipLaunchKernelGGL(k_hist_bulk<NB>, dim3(nx + ns * d.nk), dim3(256), 0, st, d, (const cplx*)a.hist,
                           (const cplx*)a.sig, a.colpart, a.rowpart, m, lgL, x);
    }
    return hipGetLastError();
  }
  static hipError_t row(const Dims& d, const LaunchArgs& a, int m, int mode, hipStream_t st) {
    // the trapezoid's end terms are a fixed handful; Gregory corrections loop over their nodes
    auto kern = mode == KBE_ROW_PREDICT ? k_row<NB, KBE_ROW_PREDICT, false>   // (no end terms)
                : mode == KBE_ROW_CORRECT
                    ? (d.qp > 1 ? k_row<NB, KBE_ROW_CORRECT, true> : k_row<NB, KBE_ROW_CORRECT, false>)
                    : (d.qp > 1 ? k_row<NB, KBE_ROW_EVAL, true> : k_row<NB, KBE_ROW_EVAL, false>);
    const int tiles = row_tiles(m, mode);
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(kern, dim3(tiles, d.nk), dim3(128 * NB), 0, st, d, a.hist, a.row64, (const cplx*)a.sig,
                       (const cplx*)a.colpart, (const cplx*)a.rowpart, a.col0, a.diag, (const cplx*)a.I_prev, a.I_cur,
                       (const cplx*)a.props, (const cplx*)a.rho_prev, a.rho_cur, (const cplx*)a.D_prev,
                       (const cplx*)a.D_cur, m, hist_lgseg(d, m), a.dt, a.commit, a.chg, a.quad);
    return hipGetLastError();
  }
  static hipError_t row_next(const Dims& d, const LaunchArgs& a, const LaunchArgs& next, int m, hipStream_t st) {
    if constexpr (NB <= 2)
      hipLaunchKernelGGL((k_row<NB, KBE_ROW_EVAL_NEXT, false>), dim3(row_tiles(m + 1, KBE_ROW_PREDICT), d.nk),
                         dim3(128 * NB), 0, st, d, next.hist, next.row64, (const cplx*)a.sig, (const cplx*)a.colpart,
                         (const cplx*)a.rowpart, next.col0, next.diag, (const cplx*)nullptr, a.I_cur,
                         (const cplx*)next.props, (const cplx*)next.rho_prev, next.rho_cur, (const cplx*)a.D_cur,
                         (const cplx*)nullptr, m, hist_lgseg(d, m), a.dt, next.commit, nullptr, a.quad);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
  static hipError_t obs(const Dims& d, const LaunchArgs& a, const ObsStep& o, hipStream_t st) {
    hipLaunchKernelGGL(k_obs<NB>, dim3(1), dim3(256), 0, st, d, obs_args(a, o));
    return hipGetLastError();
  }
  static hipError_t aux(const Dims& d, const LaunchArgs& a, int m, hipStream_t st) {
    dim3 grid((m + 1 + 255) / 256, d.nk * d.C);
    hipLaunchKernelGGL(k_aux<NB>, grid, dim3(256), 0, st, d, (const void*)a.hist, a.row64, a.col0, a.diag, m);
    return hipGetLastError();
  }
};

hipError_t launch_fill_zero(double* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

#define KBE_DISPATCH(NBV, CALL)                     \
  switch (NBV) {                                    \
    case 1: return Launch<1>::CALL;                 \
    case 2: return Launch<2>::CALL;                 \
    case 3: return Launch<3>::CALL;                 \
    case 4: return Launch<4>::CALL;                 \
    default: return hipErrorInvalidValue;           \
  }

hipError_t launch_init(const Dims& d, const LaunchArgs& a, hipStream_t st) { KBE_DISPATCH(d.nb, init(d, a, st)); }
hipError_t launch_props(const Dims& d, const LaunchArgs& a, double wb, const ObsStep* o, hipStream_t st) {
  KBE_DISPATCH(d.nb, props(d, a, wb, o, st));
}
hipError_t launch_sigma(const Dims& d, const LaunchArgs& a, int m, hipStream_t st) {
  KBE_DISPATCH(d.nb, sigma(d, a, m, st));
}
hipError_t launch_kick(const Dims& d, const LaunchArgs& a, int m, double kc, double ks, cplx* rho_other,
                       hipStream_t st) {
  if (d.nb != 2) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_kick_row<2>, dim3((m + 1 + 255) / 256, d.nk), dim3(256), 0, st, d, a.hist, a.row64, a.col0,
                     a.diag, a.rho_cur, rho_other, m, kc, ks);
  return hipGetLastError();
}
hipError_t launch_sigma_direct(const Dims& d, const LaunchArgs& a, int m, hipStream_t st) {
  size_t shm = (size_t)(6 * d.nk + d.nk / 8) * sizeof(cplx);
  hipError_t e = allow_lds((const void*)k_sigma_direct, shm);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sigma_direct, dim3((m + 1) * 4), dim3(512), shm, st, d, (const cplx*)a.row64, a.sig, m, a.UU,
                     a.corr);
  return hipGetLastError();
}
hipError_t launch_collide(const Dims& d, const LaunchArgs& a, int m, const LaunchArgs* props, double wb,
                          const ObsStep* o, hipStream_t st) {
  KBE_DISPATCH(d.nb, collide(d, a, m, props, wb, o, st));
}
hipError_t launch_row(const Dims& d, const LaunchArgs& a, int m, int mode, hipStream_t st) {
  KBE_DISPATCH(d.nb, row(d, a, m, mode, st));
}
hipError_t launch_row_next(const Dims& d, const LaunchArgs& a, const LaunchArgs& next, int m, hipStream_t st) {
  if (!row_next_fused(d) || m < 1) return hipErrorInvalidValue;
  KBE_DISPATCH(d.nb, row_next(d, a, next, m, st));
}
hipError_t launch_change_max(const Dims& d, const double* chg, int m, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_change_max, dim3(1), dim3(1024), 0, st, chg, d.nk * row_tiles(m, KBE_ROW_CORRECT), out);
  return hipGetLastError();
}
hipError_t launch_obs(const Dims& d, const LaunchArgs& a, const ObsStep& o, hipStream_t st) {
  KBE_DISPATCH(d.nb, obs(d, a, o, st));
}
hipError_t launch_aux(const Dims& d, const LaunchArgs& a, int m, hipStream_t st) {
  KBE_DISPATCH(d.nb, aux(d, a, m, st));
}

}  // namespace kbe
