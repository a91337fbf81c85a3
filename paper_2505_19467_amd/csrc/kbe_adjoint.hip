// Adjoint (reverse-mode) kernels of the Kadanoff-Baym propagation step (gfx950).
//
// The reverse sweep runs the steps of Algorithm "prop" backwards. For a real loss L every
// complex quantity x carries an adjoint xbar = dL/dRe(x) + i dL/dIm(x), with the rules
//   y = A x        -> xbar += A^dag ybar,     Abar += ybar x^dag
//   y = A B^dag    -> Abar += ybar B,         Bbar += ybar^dag A
//   y = conj(x)    -> xbar += conj(ybar)
// and for a real parameter p:  dL/dp += Re sum conj(ybar) dy/dp.
//
//   k_adj_bulk    adjoint of the history sums: reads the stored block, accumulates the
//                 self-energy adjoints (column sums in registers, row sums across lanes); in
//                 its fused form it also updates the adjoint history (read-modify-write, same
//                 strip-major layout) for both collision passes of a reverse step
//   k_adj_row     adjoint of the end-point and equal-time terms of eq. (CI): completes the
//                 self-energy adjoint row and the adjoint of the current row
//   k_adj_sigma   adjoint of eq. (2BSE) through the k <-> R transforms (Wirtinger products)
//   k_adj_update  adjoint of the predictor/corrector update of G(t_m, .) and rho_m
//   k_adj_props1/2 adjoint of V, Vh, Phi: Frechet derivative of the exponential (nb = 1, 2)
//   k_adj_hf      adjoint of the mean field and of the pulse; parameter gradients
//   k_adj_seed    adjoint of the final-time observable
//   k_adj_rho     rho_m = -i G^<(t_m, t_m) read back from the stored history diagonal
#include "kbe_adjoint.hpp"
#include "kbe_device.hpp"
#include "kbe_kernels.hpp"

namespace kbe {

// (A^dag B)_ij = sum_l conj(A_li) B_lj
template <int NB>
__device__ __forceinline__ void mm_acc_adag(cplx* acc, const cplx* A, const cplx* B) {
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int l = 0; l < NB; ++l) {
        cplx a = cconj(A[l * NB + i]);
        cmac(acc[i * NB + j], a, B[l * NB + j]);
      }
}

// ------------------------------------------------------------------ end points and equal time
// Forward terms (times dt) of output t' < m:
//   +1/2 SR_m R_{t'} - 1/2 SR_0 G0(t') + [t'>0](-1/2 S^s_{t'} GR_{t't'} + 1/2 S^s_0 GR0(t')),
//   G0(0) = G_00, G0(t') = -G_{t'0}^dag, GR = G^> - G^<;
// and the equal-time output (both components the same matrix)
//   I_d = dt sum_j a_j [S^>_j Gjm^< - S^<_j Gjm^>],  Gjm = -R_j^dag (j < m), R_m (j = m).
// k_adj_row produces the complete Sigma adjoint row sbar (lesser, greater), the adjoint of the current
// row Rbar (overwritten), and the end-point updates of the adjoint history, one thread per (k, t'),
// 64 t' per block. The sums over t' of the j = 0 and j = m Sigma adjoints (adj_row_sums, one block per
// k) need no result of the history sums and ride in front of their blocks. One block per k for all of
// it took 48.6 us on average on the 12 x 12, 400-step gradient; now 15.3 us.
template <int NB>
__device__ __forceinline__ void adj_row_sums(const Dims& d, const cplx* __restrict__ row64, const cplx* __restrict__ col0,
                                             const cplx* __restrict__ Ibar, cplx* __restrict__ rowtot, int k, int m,
                                             double dt) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr int NR = 4 * NBB;  // SRbar_m, SRbar_0, Sbar^<_0, Sbar^>_0
  __shared__ cplx wred[4][NR];
  cplx r[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) r[i] = czero();
  for (int tp = threadIdx.x; tp < m; tp += blockDim.x) {
    cplx Ib[C], Rr[C], G0[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      Ib[c] = Ibar[rowbuf_idx(d, k, c, tp)];
      Rr[c] = row64[row64_idx(d, m, k, c, tp)];
    }
    if (tp == 0) {
#pragma unroll
      for (int c = 0; c < C; ++c) G0[c] = col0[rowbuf_idx(d, k, c, 0)];
    } else {
#pragma unroll
      for (int sc = 0; sc < 2; ++sc)
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            G0[sc * NBB + a * NB + b] = cneg(cconj(col0[rowbuf_idx(d, k, sc * NBB + b * NB + a, tp)]));
    }
    cplx t[NBB];
#pragma unroll
    for (int sc = 0; sc < 2; ++sc) {
      // SRbar_m += 1/2 dt Ibar^s R^s^dag ;  SRbar_0 -= 1/2 dt Ibar^s G0^s^dag
      mat_zero<NB>(t);
      mm_acc_bdag<NB>(t, Ib + sc * NBB, Rr + sc * NBB);
#pragma unroll
      for (int e = 0; e < NBB; ++e) r[e] = cadd(r[e], cscal(t[e], 0.5 * dt));
      mat_zero<NB>(t);
      mm_acc_bdag<NB>(t, Ib + sc * NBB, G0 + sc * NBB);
#pragma unroll
      for (int e = 0; e < NBB; ++e) r[NBB + e] = csub(r[NBB + e], cscal(t[e], 0.5 * dt));
    }
    if (tp > 0) {
      // Sbar^s_0 += 1/2 dt Ibar^s GR0^dag
      cplx GR0[NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) GR0[e] = csub(G0[NBB + e], G0[e]);
#pragma unroll
      for (int sc = 0; sc < 2; ++sc) {
        mat_zero<NB>(t);
        mm_acc_bdag<NB>(t, Ib + sc * NBB, GR0);
#pragma unroll
        for (int e = 0; e < NBB; ++e) r[(2 + sc) * NBB + e] = cadd(r[(2 + sc) * NBB + e], cscal(t[e], 0.5 * dt));
      }
    }
  }
  {
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      cplx v = cmk(wave_sum(r[i].x), wave_sum(r[i].y));
      if (lane == 0) wred[wv][i] = v;
    }
    __syncthreads();
    if (threadIdx.x < NR) {
      int i = threadIdx.x;
      rowtot[(int64_t)k * NR + i] = cadd(cadd(wred[0][i], wred[1][i]), cadd(wred[2][i], wred[3][i]));
    }
  }
}
template <int NB>
__global__ __launch_bounds__(64) void k_adj_row(Dims d, const cplx* __restrict__ row64, const cplx* __restrict__ sig,
                                                const cplx* __restrict__ col0, const cplx* __restrict__ diag,
                                                const cplx* __restrict__ Ibar, const cplx* __restrict__ Dbar,
                                                const cplx* __restrict__ sbar_col,
                                                const cplx* __restrict__ sbar_rowpart, const cplx* __restrict__ rowtot,
                                                cplx* __restrict__ sbar, cplx* __restrict__ Rbar,
                                                cplx* __restrict__ lam, cplx* __restrict__ lam_diag,
                                                cplx* __restrict__ lam_col0, int m, double dt) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr bool END = NB == 2;
  const int k = blockIdx.y;
  const cplx* tot = rowtot + (int64_t)k * 4 * NBB;
  auto S = [&](int sc, int e, int j) { return sig[sig_idx(d, k, sc, e, j)]; };
  cplx SRm[NBB], SR0[NBB], Sl0[NBB], Sg0[NBB], Id[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    SRm[e] = S(2, e, m);
    SR0[e] = S(2, e, 0);
    Sl0[e] = S(0, e, 0);
    Sg0[e] = S(1, e, 0);
  }
  // adjoint of the equal-time matrix: Ibar^<(m) + Ibar^>(m) + Dbar + Dbar^dag
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      int e = a * NB + b;
      cplx v = cadd(Ibar[rowbuf_idx(d, k, e, m)], Ibar[rowbuf_idx(d, k, NBB + e, m)]);
      v = cadd(v, Dbar[(int64_t)k * NBB + e]);
      v = cadd(v, cconj(Dbar[(int64_t)k * NBB + b * NB + a]));
      Id[e] = v;
    }
  const int tp = blockIdx.x * 64 + threadIdx.x;
  if (tp <= m) {
    cplx sb[C], srb[NBB], rb[C];
#pragma unroll
    for (int c = 0; c < C; ++c) rb[c] = czero();
#pragma unroll
    for (int e = 0; e < NBB; ++e) srb[e] = czero();
    if (tp < m) {
#pragma unroll
      for (int c = 0; c < C; ++c) sb[c] = sbar_col[rowbuf_idx(d, k, c, tp)];
      int ns = (tp >> 6) + 1;
      for (int s = 0; s < ns; ++s) {
        const cplx* rp = sbar_rowpart + ((int64_t)k * d.Smax + s) * NBB * d.Tp;
#pragma unroll
        for (int e = 0; e < NBB; ++e) srb[e] = cadd(srb[e], rp[(int64_t)e * d.Tp + tp]);
      }
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c) sb[c] = czero();
    }
    if (tp < m) {
      cplx Ib[C], G0[C], Gbar0[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        Ib[c] = Ibar[rowbuf_idx(d, k, c, tp)];
        Gbar0[c] = czero();
      }
      if (tp == 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) G0[c] = col0[rowbuf_idx(d, k, c, 0)];
      } else {
#pragma unroll
        for (int sc = 0; sc < 2; ++sc)
#pragma unroll
          for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
              G0[sc * NBB + a * NB + b] = cneg(cconj(col0[rowbuf_idx(d, k, sc * NBB + b * NB + a, tp)]));
      }
#pragma unroll
      for (int sc = 0; sc < 2; ++sc) {
        // Rbar^s_{t'} += 1/2 dt SR_m^dag Ibar^s ;  G0bar^s -= 1/2 dt SR_0^dag Ibar^s
        cplx t[NBB];
        mat_zero<NB>(t);
        mm_acc_adag<NB>(t, SRm, Ib + sc * NBB);
#pragma unroll
        for (int e = 0; e < NBB; ++e) rb[sc * NBB + e] = cadd(rb[sc * NBB + e], cscal(t[e], 0.5 * dt));
        mat_zero<NB>(t);
        mm_acc_adag<NB>(t, SR0, Ib + sc * NBB);
#pragma unroll
        for (int e = 0; e < NBB; ++e) Gbar0[sc * NBB + e] = csub(Gbar0[sc * NBB + e], cscal(t[e], 0.5 * dt));
      }
      if (tp > 0) {
        cplx GRtt[NBB], GRbar[NBB], GR0bar[NBB];
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          GRtt[e] = csub(diag[rowbuf_idx(d, k, NBB + e, tp)], diag[rowbuf_idx(d, k, e, tp)]);
          GRbar[e] = czero();
          GR0bar[e] = czero();
        }
#pragma unroll
        for (int sc = 0; sc < 2; ++sc) {
          cplx St[NBB], S0[NBB], t[NBB];
#pragma unroll
          for (int e = 0; e < NBB; ++e) {
            St[e] = S(sc, e, tp);
            S0[e] = sc ? Sg0[e] : Sl0[e];
          }
          // -1/2 S^s_{t'} GR_{t't'}:  Sbar^s_{t'} -= 1/2 dt Ibar^s GRtt^dag,  GRbar -= 1/2 dt S^s_{t'}^dag Ibar^s
          mat_zero<NB>(t);
          mm_acc_bdag<NB>(t, Ib + sc * NBB, GRtt);
#pragma unroll
          for (int e = 0; e < NBB; ++e) sb[sc * NBB + e] = csub(sb[sc * NBB + e], cscal(t[e], 0.5 * dt));
          mat_zero<NB>(t);
          mm_acc_adag<NB>(t, St, Ib + sc * NBB);
#pragma unroll
          for (int e = 0; e < NBB; ++e) GRbar[e] = csub(GRbar[e], cscal(t[e], 0.5 * dt));
          // +1/2 S^s_0 GR0:  GR0bar += 1/2 dt S^s_0^dag Ibar^s
          mat_zero<NB>(t);
          mm_acc_adag<NB>(t, S0, Ib + sc * NBB);
#pragma unroll
          for (int e = 0; e < NBB; ++e) GR0bar[e] = cadd(GR0bar[e], cscal(t[e], 0.5 * dt));
        }
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          Gbar0[NBB + e] = cadd(Gbar0[NBB + e], GR0bar[e]);
          Gbar0[e] = csub(Gbar0[e], GR0bar[e]);
        }
        // GR_{t't'} = G^>_{t't'} - G^<_{t't'}: adjoint history diagonal block; G0 = -G_{t'0}^dag: its
        // first column. nb = 2 adds them into compact rows that join row t' when the sweep reaches
        // it (in the packed adjoint history each is a cache line of its own: 32.8 -> 15.3 us); nb = 1
        // keeps the order of its sums, as its history passes do
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          cplx* pl = END ? lam_diag + rowbuf_idx(d, k, e, tp) : lam + hist_idx(d, k, e, tp, tp);
          cplx* pg = END ? lam_diag + rowbuf_idx(d, k, NBB + e, tp) : lam + hist_idx(d, k, NBB + e, tp, tp);
          *pl = csub(*pl, GRbar[e]);
          *pg = cadd(*pg, GRbar[e]);
        }
#pragma unroll
        for (int sc = 0; sc < 2; ++sc)
#pragma unroll
          for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
              const int c = sc * NBB + a * NB + b;
              cplx* p0 = END ? lam_col0 + rowbuf_idx(d, k, c, tp) : lam + hist_idx(d, k, c, tp, 0);
              *p0 = csub(*p0, cconj(Gbar0[sc * NBB + b * NB + a]));
            }
      } else {
#pragma unroll
        for (int c = 0; c < C; ++c) {
          cplx* p0 = END ? lam_col0 + rowbuf_idx(d, k, c, 0) : lam + hist_idx(d, k, c, 0, 0);
          *p0 = cadd(*p0, Gbar0[c]);
        }
      }
    }
    // equal-time term, node j = tp
    {
      int j = tp;
      double wgt = (m == 0) ? 0.0 : ((j == 0 || j == m) ? 0.5 : 1.0);
      cplx Rl[NBB], Rg[NBB], Gl[NBB], Gg[NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        Rl[e] = row64[row64_idx(d, m, k, e, j)];
        Rg[e] = row64[row64_idx(d, m, k, NBB + e, j)];
      }
      if (j < m) {
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            Gl[a * NB + b] = cneg(cconj(Rl[b * NB + a]));
            Gg[a * NB + b] = cneg(cconj(Rg[b * NB + a]));
          }
      } else {
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          Gl[e] = Rl[e];
          Gg[e] = Rg[e];
        }
      }
      double f = dt * wgt;
      cplx t[NBB], Glb[NBB], Ggb[NBB];
      // Sbar^>_j += f Id Gl^dag ;  Sbar^<_j -= f Id Gg^dag
      mat_zero<NB>(t);
      mm_acc_bdag<NB>(t, Id, Gl);
#pragma unroll
      for (int e = 0; e < NBB; ++e) sb[NBB + e] = cadd(sb[NBB + e], cscal(t[e], f));
      mat_zero<NB>(t);
      mm_acc_bdag<NB>(t, Id, Gg);
#pragma unroll
      for (int e = 0; e < NBB; ++e) sb[e] = csub(sb[e], cscal(t[e], f));
      // Glbar = f S^>_j^dag Id ;  Ggbar = -f S^<_j^dag Id
      cplx Sj[NBB];
#pragma unroll
      for (int e = 0; e < NBB; ++e) Sj[e] = S(1, e, j);
      mat_zero<NB>(Glb);
      mm_acc_adag<NB>(Glb, Sj, Id);
#pragma unroll
      for (int e = 0; e < NBB; ++e) Sj[e] = S(0, e, j);
      mat_zero<NB>(Ggb);
      mm_acc_adag<NB>(Ggb, Sj, Id);
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        Glb[e] = cscal(Glb[e], f);
        Ggb[e] = cscal(Ggb[e], -f);
      }
      if (j < m) {
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            rb[a * NB + b] = csub(rb[a * NB + b], cconj(Glb[b * NB + a]));
            rb[NBB + a * NB + b] = csub(rb[NBB + a * NB + b], cconj(Ggb[b * NB + a]));
          }
      } else {
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          rb[e] = cadd(rb[e], Glb[e]);
          rb[NBB + e] = cadd(rb[NBB + e], Ggb[e]);
        }
      }
    }
    if (tp == 0) {
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        srb[e] = cadd(srb[e], tot[NBB + e]);
        sb[e] = cadd(sb[e], tot[2 * NBB + e]);
        sb[NBB + e] = cadd(sb[NBB + e], tot[3 * NBB + e]);
      }
    }
    if (tp == m) {
#pragma unroll
      for (int e = 0; e < NBB; ++e) srb[e] = cadd(srb[e], tot[e]);
    }
    // Sigma^R = Sigma^> - Sigma^<
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      sbar[(((int64_t)k * 2 + 0) * NBB + e) * d.Tp + tp] = csub(sb[e], srb[e]);
      sbar[(((int64_t)k * 2 + 1) * NBB + e) * d.Tp + tp] = cadd(sb[NBB + e], srb[e]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) Rbar[rowbuf_idx(d, k, c, tp)] = rb[c];
  }
}

// ------------------------------------------------------------------ adjoint history sums
// Forward (weight 1, times dt), per stored block (j, t'), t' <= j <= m-1:
//   I^s(t') += dt SR_j G^s_{jt'};   t' < j:  I^<(j), I^>(j) += dt [-S^>_{t'} G^<_{jt'}^dag + S^<_{t'} G^>_{jt'}^dag]
// Adjoint with Ibar^s(t') and Irow(j) = Ibar^<(j) + Ibar^>(j):
//   lam^s_{jt'} += dt SR_j^dag Ibar^s(t');   t' < j:  lam^< -= dt Irow(j)^dag S^>_{t'}, lam^> += dt Irow(j)^dag S^<_{t'}
//   SRbar_j     += dt sum_{t'} sum_s Ibar^s(t') G^s_{jt'}^dag           (across lanes, per strip)
//   Sbar^>_{t'} -= dt sum_{j > t'} Irow(j) G^<_{jt'},  Sbar^<_{t'} += dt sum_{j > t'} Irow(j) G^>_{jt'}   (in lane)
// The lam terms are linear in (SR, Ibar, Irow, S): a reverse step's first pass (ADJ_SUMS) only
// reads the history for its Sigma adjoints, and its second pass (ADJ_FUSED) applies the lam
// terms of both passes in one read-modify-write of the adjoint history (the first pass's Sigma
// row and Ibar come in as sig1, Ibar1; their columns sit in LDS): 4 streams per reverse step
// instead of 6. Layout of the work as in the forward history sums: block = (strip s, k); lane l
// owns column 64 s + l (its Sigma, Ibar and Sigma-adjoint column sums in registers); in the
// fused pass each wavefront takes 16 consecutive rows of every 64-row chunk, in the read-only
// pass rows w, w + 4, ..., w + 60 (wavefront w), one row per iteration (the history block and,
// fused, the adjoint-history block of the row: 2 C 1 KB-contiguous loads in flight, then C 1 KB
// stores).
// The SRbar row partial of a row (nb^2 components) goes through one 64-lane reduce-scatter with
// the components as groups; the row partials of four 64-row chunks are staged in LDS and stored
// by the whole block as 4 KB runs per component. Rows past the strip's first 64 (and below m) run
// without bounds selects.
template <int NB, int MODE>
__global__ __launch_bounds__(256) void k_adj_bulk(Dims d, const cplx* __restrict__ hist, cplx* __restrict__ lam,
                                                  const cplx* __restrict__ sig, const cplx* __restrict__ Ibar,
                                                  const cplx* __restrict__ sig1, const cplx* __restrict__ Ibar1,
                                                  cplx* __restrict__ sbar_col, cplx* __restrict__ sbar_rowpart,
                                                  const cplx* __restrict__ row64, const cplx* __restrict__ col0,
                                                  cplx* __restrict__ rowtot, int m, double dt) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  constexpr int CH = (C < 8) ? C : 8;
  __shared__ cplx red[3][CH][64];
  constexpr int ROWS_ST = 256;   // row partials of four 64-row chunks, stored by the block at once
  __shared__ cplx stg[NBB][ROWS_ST];
  if ((int)blockIdx.x < d.nk) {
    adj_row_sums<NB>(d, row64, col0, Ibar, rowtot, blockIdx.x, m, dt);
    return;
  }
  const int s = blockIdx.x / d.nk - 1;
  const int k = blockIdx.x - (s + 1) * d.nk;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // rows wavefront-uniform
  const int tp = 64 * s + lane;
  const bool colv = tp < m;
  const cplx* sk = sig + (int64_t)k * 3 * NBB * d.Tp;
  cplx Sl[NBB], Sg[NBB], Ib[C];
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    Sl[e] = colv ? sk[(0 * NBB + e) * d.Tp + tp] : czero();
    Sg[e] = colv ? sk[(1 * NBB + e) * d.Tp + tp] : czero();
  }
#pragma unroll
  for (int c = 0; c < C; ++c) Ib[c] = colv ? Ibar[rowbuf_idx(d, k, c, tp)] : czero();
  // ADJ_FUSED: the earlier pass's Sigma^<, Sigma^> and Ibar columns of the strip, in LDS
  __shared__ cplx xS[MODE == ADJ_FUSED ? 2 * NBB * 64 : 1];
  __shared__ cplx xI[MODE == ADJ_FUSED ? C * 64 : 1];
  const cplx* sk1 = sig1 + (int64_t)k * 3 * NBB * d.Tp;
  if constexpr (MODE == ADJ_FUSED) {
    for (int q = threadIdx.x; q < 2 * NBB * 64; q += 256) {
      const int l = q & 63, t = 64 * s + l;
      xS[q] = t < m ? sk1[(q >> 6) * d.Tp + t] : czero();
    }
    for (int q = threadIdx.x; q < C * 64; q += 256) {
      const int l = q & 63, t = 64 * s + l;
      xI[q] = t < m ? Ibar1[rowbuf_idx(d, k, q >> 6, t)] : czero();
    }
    __syncthreads();
  }
  cplx acc[C];  // [0, NBB): Sbar^<_{t'}, [NBB, C): Sbar^>_{t'}
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = czero();
  const int64_t base = strip_lane_base(d, k, s, lane);
  const cplx* hk = hist + base;
  cplx* lk = lam + base;
  cplx* rp = sbar_rowpart + ((int64_t)k * d.Smax + s) * NBB * d.Tp;
  for (int cb = 64 * s; cb < m; cb += 64) {
    // the read-only pass: wavefront w takes rows w, w + 4, ..., w + 60 (a chunk cut short by m
    // keeps all four busy); the fused pass: 16 consecutive rows (its read-modify-write stream
    // runs better in 128 KB runs per wavefront)
    constexpr int RS = MODE == ADJ_SUMS ? 4 : 1;
    const int rb = cb + (MODE == ADJ_SUMS ? wv : 16 * wv);
    const int cslot = ((cb - 64 * s) >> 6) % (ROWS_ST / 64);
    cplx* st = &stg[0][64 * cslot];   // st[e * ROWS_ST + (row - cb)]
    for (int i = 0; i < 16; ++i) {
      const int j = rb + RS * i;
      if (j >= m) break;
      auto row = [&](auto tag) {
        constexpr bool MASKED = decltype(tag)::value;
        const bool v = MASKED ? (colv && tp <= j) : true;
        const int64_t off = 64 * (int64_t)C * j;
        cplx G[C], L[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          G[c] = v ? load_stream(hk + off + 64 * c) : czero();
          if constexpr (MODE != ADJ_SUMS) L[c] = v ? load_stream(lk + off + 64 * c) : czero();
        }
        cplx SR[NBB], Irow[NBB];
#pragma unroll
        for (int e = 0; e < NBB; ++e) {
          SR[e] = sk[(2 * NBB + e) * d.Tp + j];
          Irow[e] = cadd(Ibar[rowbuf_idx(d, k, e, j)], Ibar[rowbuf_idx(d, k, NBB + e, j)]);
        }
        const bool rv = MASKED ? tp < j : true;
        if constexpr (MODE == ADJ_FUSED) {
          // adjoint history, accumulated into the loaded block with dt-scaled row factors:
          //   lam^s += (dt SR)^dag Ibar^s;  t' < j:  lam^< += (-dt Irow)^dag S^>,  lam^> += (dt Irow)^dag S^<
          // for this pass (column factors in registers), then for the earlier pass (from LDS,
          // read here in every row: the barrier keeps the compiler from holding them in
          // registers across the loop, which would leave room for one wavefront per SIMD only)
          auto update = [&](const cplx* SRr, const cplx* Irr, auto col_ib, auto col_sg, auto col_sl) {
            cplx A[NBB], X[NBB];
#pragma unroll
            for (int e = 0; e < NBB; ++e) A[e] = cscal(SRr[e], dt);
#pragma unroll
            for (int sc = 0; sc < 2; ++sc) {
#pragma unroll
              for (int e = 0; e < NBB; ++e) X[e] = col_ib(sc * NBB + e);
              mm_acc_adag<NB>(L + sc * NBB, A, X);
            }
            if (rv) {
#pragma unroll
              for (int e = 0; e < NBB; ++e) A[e] = cscal(Irr[e], -dt);
#pragma unroll
              for (int e = 0; e < NBB; ++e) X[e] = col_sg(e);
              mm_acc_adag<NB>(L, A, X);
#pragma unroll
              for (int e = 0; e < NBB; ++e) A[e] = cscal(Irr[e], dt);
#pragma unroll
              for (int e = 0; e < NBB; ++e) X[e] = col_sl(e);
              mm_acc_adag<NB>(L + NBB, A, X);
            }
          };
          update(SR, Irow, [&](int c) { return Ib[c]; }, [&](int e) { return Sg[e]; }, [&](int e) { return Sl[e]; });
          asm volatile("" ::: "memory");
          cplx SR1[NBB], Irow1[NBB];
#pragma unroll
          for (int e = 0; e < NBB; ++e) {
            SR1[e] = sk1[(2 * NBB + e) * d.Tp + j];
            Irow1[e] = cadd(Ibar1[rowbuf_idx(d, k, e, j)], Ibar1[rowbuf_idx(d, k, NBB + e, j)]);
          }
          update(SR1, Irow1, [&](int c) { return xI[c * 64 + lane]; }, [&](int e) { return xS[(NBB + e) * 64 + lane]; },
                 [&](int e) { return xS[e * 64 + lane]; });
          if (v) {
#pragma unroll
            for (int c = 0; c < C; ++c) store_stream(lk + off + 64 * c, L[c]);
          }
        }
        if (rv) {
          // Sigma adjoints of the row term (in lane)
          cplx x[NBB], y[NBB];
          mat_zero<NB>(x);
          mat_zero<NB>(y);
          mm_acc<NB>(x, Irow, G + NBB);  // Irow G^>  -> Sbar^<
          mm_acc<NB>(y, Irow, G);        // Irow G^<  -> -Sbar^>
#pragma unroll
          for (int e = 0; e < NBB; ++e) {
            acc[e] = cadd(acc[e], cscal(x[e], dt));
            acc[NBB + e] = csub(acc[NBB + e], cscal(y[e], dt));
          }
        }
        // SRbar_j partial: sum_s Ibar^s G^s^dag (zero where no block is stored)
        cplx q[NBB];
        mat_zero<NB>(q);
        mm_acc_bdag<NB>(q, Ib, G);
        mm_acc_bdag<NB>(q, Ib + NBB, G + NBB);
        if constexpr (NBB == 4) {
          // the four components are the four groups of one reduce-scatter
          double xg[4][2];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            xg[e][0] = q[e].x * dt;
            xg[e][1] = q[e].y * dt;
          }
          reduce_rows<4>(xg);
          const int e = reduced_row<4>(lane);
          if (e >= 0) st[e * ROWS_ST + (j - cb)] = cmk(xg[0][0], xg[0][1]);
        } else {
          double rt[1][2 * NBB];
#pragma unroll
          for (int e = 0; e < NBB; ++e) {
            rt[0][2 * e] = q[e].x * dt;
            rt[0][2 * e + 1] = q[e].y * dt;
          }
          reduce_rows<1>(rt);
          if (reduced_row<1>(lane) >= 0) {
#pragma unroll
            for (int e = 0; e < NBB; ++e) st[e * ROWS_ST + (j - cb)] = cmk(rt[0][2 * e], rt[0][2 * e + 1]);
          }
        }
      };
      if (j >= 64 * s + 64)
        row(BoolTag<false>{});
      else
        row(BoolTag<true>{});
    }
    if (cslot == ROWS_ST / 64 - 1 || cb + 64 >= m) {
      __syncthreads();
      const int base = cb - 64 * cslot;
      const int nrows = (cb + 64 < m ? cb + 64 : m) - base;
      for (int q = threadIdx.x; q < NBB * nrows; q += 256) {
        const int e = q / nrows, row = q - e * nrows;
        store_stream(rp + (int64_t)e * d.Tp + base + row, stg[e][row]);
      }
      __syncthreads();
    }
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
        if (colv) sbar_col[rowbuf_idx(d, k, c0 + c, tp)] = a;
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ self-energy adjoint
// Forward per (t_j, ab): g = N_k^{-1} F^+ G,  s^< = c g^<^2 conj(g^>),  s^> = c g^>^2 conj(g^<),
// Sigma = F^- s, with c = -U^2 and F^{+-} the index transforms with e^{+-2 pi i j.R/n}.
// Adjoint: sbar(R) = F^+ Sigmabar (no 1/N_k),
//   gbar^< = 2 c conj(g^<) g^> sbar^< + c g^>^2 conj(sbar^>),
//   gbar^> = c g^<^2 conj(sbar^<) + 2 c conj(g^>) g^< sbar^>,
//   Gbar(k) += N_k^{-1} F^- gbar,   dL/dU += sum Re conj(sbar) ds/dU,  ds/dU = 2 s / U.
// NX, NY > 0: the grid is fixed at compile time (unrolled transforms, nb = 2 and the forward kernel's grids:
// 42.0 -> 14.1 us on the 12 x 12 grid, m <= 400); 0: any grid, sizes from d. Averages over m <= 200, before
// either and now: 12 x 12 31.3 -> 11.8 us, 24 x 24 57.3 -> 30.3, 16 points 17.5 -> 6.7; at run time 10 x 10
// 26.9 -> 23.2, 14 x 14 34.0 -> 27.9, 20 x 20 43.7 -> 35.1, 20 points 18.1 -> 14.8.
template <int NB, int NX, int NY>
__global__ __launch_bounds__(256) void k_adj_sigma(Dims d, const cplx* __restrict__ row64,
                                                   const cplx* __restrict__ sbar, cplx* __restrict__ Rbar,
                                                   double* __restrict__ ubar_part, int m, double U, int corr) {
  constexpr int NBB = NB * NB;
  constexpr int PT = 4;  // k points per thread (N_k <= 1024)
  extern __shared__ cplx lds[];
  __shared__ double ured[256], usum[1];
  __shared__ cplx twx[64], twy[64];
  const int nk = NX > 0 ? NX * NY : d.nk;
  const int nx = NX > 0 ? NX : d.nkx, ny = NX > 0 ? NY : d.nky;
  cplx* xl = lds;
  cplx* xg = lds + nk;
  cplx* tl = lds + 2 * nk;
  cplx* tg = lds + 3 * nk;
  auto dft = [&](int sgn, double scale) {
    if constexpr (NX > 0) grid_dft_ct<NX, NY>(xl, xg, tl, tg, twx, twy, sgn, scale);
    else grid_dft(d, xl, xg, tl, tg, twx, twy, sgn, scale);
  };
  int total = (m + 1) * NBB;
  int per = (total + 7) >> 3;
  int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  double up = 0.0;
  if (item < total) {
    int j = item / NBB, ab = item - (item / NBB) * NBB;
    int t = threadIdx.x;
    fill_roots(twx, nx);
    fill_roots(twy, ny);
    for (int k = t; k < nk; k += 256) {
      xl[k] = row64[row64_idx(d, m, k, ab, j)];
      xg[k] = row64[row64_idx(d, m, k, NBB + ab, j)];
    }
    __syncthreads();
    dft(+1, 1.0 / nk);  // g(R)
    cplx ra[PT], rb[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      int o = t + 256 * i;
      ra[i] = o < nk ? xl[o] : czero();
      rb[i] = o < nk ? xg[o] : czero();
    }
    __syncthreads();
    for (int k = t; k < nk; k += 256) {
      xl[k] = sbar[(((int64_t)k * 2 + 0) * NBB + ab) * d.Tp + j];
      xg[k] = sbar[(((int64_t)k * 2 + 1) * NBB + ab) * d.Tp + j];
    }
    __syncthreads();
    dft(+1, 1.0);  // sbar(R)
    double cc = -U * U;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      int o = t + 256 * i;
      if (o >= nk) continue;
      cplx a = ra[i], b = rb[i], sl = xl[o], sg = xg[o];
      cplx ga = czero(), gb = czero();
      if (corr) {
        // gbar^< = 2c conj(a) b sl + c b^2 conj(sg);  gbar^> = c a^2 conj(sl) + 2c conj(b) a sg
        ga = cadd(cscal(cmul(cmul(cconj(a), b), sl), 2.0 * cc), cscal(cmul(cmul(b, b), cconj(sg)), cc));
        gb = cadd(cscal(cmul(cmul(a, a), cconj(sl)), cc), cscal(cmul(cmul(cconj(b), a), sg), 2.0 * cc));
        // ds^</dU = -2U a^2 conj(b), ds^>/dU = -2U b^2 conj(a)
        cplx dsl = cscal(cmul(cmul(a, a), cconj(b)), -2.0 * U);
        cplx dsg = cscal(cmul(cmul(b, b), cconj(a)), -2.0 * U);
        up += sl.x * dsl.x + sl.y * dsl.y + sg.x * dsg.x + sg.y * dsg.y;
      }
      xl[o] = ga;
      xg[o] = gb;
    }
    __syncthreads();
    dft(-1, 1.0 / nk);
    for (int k = t; k < nk; k += 256) {
      int64_t il = rowbuf_idx(d, k, ab, j), ig = rowbuf_idx(d, k, NBB + ab, j);
      Rbar[il] = cadd(Rbar[il], xl[k]);
      Rbar[ig] = cadd(Rbar[ig], xg[k]);
    }
  }
  block_sum_once<1>(&up, ured, usum);
  if (threadIdx.x == 0) ubar_part[blockIdx.x] = usum[0];
}

// ------------------------------------------------------------------ update adjoint
// Forward (t' < m):  G_m(t') = V G_{m-1}(t') + Phi Ibar(t'),  Ibar = f1 I_{m-1} + f2 I_c;
// t' = m:  G_m(m) = (i rho_m, -i (1 - rho_m)),  rho_m = V rho_{m-1} V^dag - dt W Dbar W^dag,
// Dbar = g1 D_{m-1} + g2 D_c. One block per k.
// The block has 256 nb threads (at nb = 2, m <= 400, 23.2 -> 21.7 us on average, 48.3 -> 38.3 at most,
// against 256; at small m it is the latency of the one thread that ends each k, 10 us).
template <int NB>
__global__ __launch_bounds__(256 * NB) void k_adj_update(Dims d, const cplx* __restrict__ lam_rowm,
                                                    const cplx* __restrict__ Gbar_row, cplx* __restrict__ lam,
                                                    const cplx* __restrict__ row64, const cplx* __restrict__ props,
                                                    const cplx* __restrict__ Iprev, const cplx* __restrict__ Ic,
                                                    const cplx* __restrict__ rho_prev, const cplx* __restrict__ Dprev,
                                                    const cplx* __restrict__ Dc, cplx* __restrict__ Ibar_prev,
                                                    cplx* __restrict__ Ibar_c, cplx* __restrict__ rhobar,
                                                    cplx* __restrict__ rhobar_prev, cplx* __restrict__ Dbar_prev,
                                                    cplx* __restrict__ Dbar_c, cplx* __restrict__ pbar, int m,
                                                    double dt, int corrector, const cplx* __restrict__ lam_diag,
                                                    const cplx* __restrict__ lam_col0,
                                                    const double* __restrict__ ubar_part,
                                                    int nubar, double* __restrict__ theta_bar) {
  constexpr int NBB = NB * NB, C = 2 * NBB;
  __shared__ double lds[4 * NBB * 256], sums[4 * NBB];
  if ((int)blockIdx.x == d.nk) {
    // one more block: the self-energy adjoint's dL/dU partials of the collision pass before
    double u = 0.0;
    if (threadIdx.x < 256)
      for (int i = threadIdx.x; i < nubar; i += 256) u += ubar_part[i];
    block_sum_once<1>(&u, lds, sums);
    if (threadIdx.x == 0) theta_bar[2] += sums[0];
    return;
  }
  int k = blockIdx.x;
  const cplx* P = props + (int64_t)k * 3 * NBB;
  cplx V[NBB], W[NBB], Phi[NBB];
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    V[e] = P[e];
    W[e] = P[NBB + e];
    Phi[e] = P[2 * NBB + e];
  }
  double f1 = corrector ? 0.5 : 1.0;
  cplx Vb[NBB], Pb[NBB];  // per-thread partial V-bar, Phi-bar
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    Vb[e] = czero();
    Pb[e] = czero();
  }
  auto gbar = [&](int c, int tp) {
    cplx g = Gbar_row ? Gbar_row[rowbuf_idx(d, k, c, tp)] : czero();
    if (lam_rowm) {
      g = cadd(g, lam_rowm[hist_idx(d, k, c, m, tp)]);
      if constexpr (NB == 2) {   // the end-point terms' part of the adjoint history row
        if (tp == 0) g = cadd(g, lam_col0[rowbuf_idx(d, k, c, m)]);
        if (tp == m) g = cadd(g, lam_diag[rowbuf_idx(d, k, c, m)]);
      }
    }
    return g;
  };
  for (int tp = threadIdx.x; tp < m; tp += blockDim.x) {
    cplx Gb[C], Go[C], Ib[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      Gb[c] = gbar(c, tp);
      Go[c] = row64[row64_idx(d, m - 1, k, c, tp)];
      cplx ip = Iprev[rowbuf_idx(d, k, c, tp)];
      Ib[c] = corrector ? cscal(cadd(ip, Ic[rowbuf_idx(d, k, c, tp)]), 0.5) : ip;
    }
#pragma unroll
    for (int sc = 0; sc < 2; ++sc) {
      cplx t[NBB], u[NBB];
      // lam_{m-1}(t') += V^dag Gbar
      mat_zero<NB>(t);
      mm_acc_adag<NB>(t, V, Gb + sc * NBB);
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        int64_t i = hist_idx(d, k, sc * NBB + e, m - 1, tp);
        lam[i] = cadd(lam[i], t[e]);
      }
      // Ibar_{m-1} += f1 Phi^dag Gbar ;  Ibar_c = 1/2 Phi^dag Gbar
      mat_zero<NB>(u);
      mm_acc_adag<NB>(u, Phi, Gb + sc * NBB);
#pragma unroll
      for (int e = 0; e < NBB; ++e) {
        int64_t i = rowbuf_idx(d, k, sc * NBB + e, tp);
        Ibar_prev[i] = cadd(Ibar_prev[i], cscal(u[e], f1));
        if (corrector) Ibar_c[i] = cscal(u[e], 0.5);
      }
      // Vbar += Gbar Go^dag ;  Phibar += Gbar Ib^dag
      mm_acc_bdag<NB>(Vb, Gb + sc * NBB, Go + sc * NBB);
      mm_acc_bdag<NB>(Pb, Gb + sc * NBB, Ib + sc * NBB);
    }
  }
  if (corrector && threadIdx.x == 0)
#pragma unroll
    for (int c = 0; c < C; ++c) Ibar_c[rowbuf_idx(d, k, c, m)] = czero();  // I_c(t_m, t_m) only enters D_c
  // V-bar, Phi-bar over the block
  {
    double v[4 * NBB];
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      v[2 * e] = Vb[e].x;
      v[2 * e + 1] = Vb[e].y;
      v[2 * (NBB + e)] = Pb[e].x;
      v[2 * (NBB + e) + 1] = Pb[e].y;
    }
    if constexpr (NB == 2) {   // threads 256.. hand theirs to 0..
      const int t = threadIdx.x;
      if (t >= 256)
#pragma unroll
        for (int i = 0; i < 4 * NBB; ++i) lds[i * 256 + t - 256] = v[i];
      __syncthreads();
      if (t < 256)
#pragma unroll
        for (int i = 0; i < 4 * NBB; ++i) v[i] += lds[i * 256 + t];
      __syncthreads();
    }
    block_sum_once<4 * NBB>(v, lds, sums);
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      Vb[e] = cmk(sums[2 * e], sums[2 * e + 1]);
      Pb[e] = cmk(sums[2 * (NBB + e)], sums[2 * (NBB + e) + 1]);
    }
    // equal-time block: G^< = i rho, G^> = -i + i rho  ->  rhobar += -i (Gbar^<_mm + Gbar^>_mm)
    cplx rb[NBB], r0[NBB], Db[NBB], Wb[NBB], t1[NBB], t2[NBB];
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      cplx g = cadd(gbar(e, m), gbar(NBB + e, m));
      rb[e] = cadd(rhobar[(int64_t)k * NBB + e], cmk(g.y, -g.x));
      rhobar[(int64_t)k * NBB + e] = rb[e];
      r0[e] = rho_prev[(int64_t)k * NBB + e];
      cplx dp = Dprev[(int64_t)k * NBB + e];
      Db[e] = corrector ? cscal(cadd(dp, Dc[(int64_t)k * NBB + e]), 0.5) : dp;
      Wb[e] = czero();
    }
    // rho = V r0 V^dag:  r0bar += V^dag rb V ;  Vbar += rb V r0^dag + rb^dag V r0
    mat_zero<NB>(t1);
    mm_acc_adag<NB>(t1, V, rb);
    mat_zero<NB>(t2);
    mm_acc<NB>(t2, t1, V);
#pragma unroll
    for (int e = 0; e < NBB; ++e) rhobar_prev[(int64_t)k * NBB + e] = cadd(rhobar_prev[(int64_t)k * NBB + e], t2[e]);
    mat_zero<NB>(t1);
    mm_acc<NB>(t1, rb, V);
    mm_acc_bdag<NB>(Vb, t1, r0);
    cplx rbd[NBB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) rbd[a * NB + b] = cconj(rb[b * NB + a]);
    mat_zero<NB>(t1);
    mm_acc<NB>(t1, rbd, V);
    mm_acc<NB>(Vb, t1, r0);
    // -dt W Db W^dag:  Wbar += -dt (rb W Db^dag + rb^dag W Db) ;  Dbbar = -dt W^dag rb W
    mat_zero<NB>(t1);
    mm_acc<NB>(t1, rb, W);
    mat_zero<NB>(t2);
    mm_acc_bdag<NB>(t2, t1, Db);
    mat_zero<NB>(t1);
    mm_acc<NB>(t1, rbd, W);
    mm_acc<NB>(t2, t1, Db);
#pragma unroll
    for (int e = 0; e < NBB; ++e) Wb[e] = cscal(t2[e], -dt);
    mat_zero<NB>(t1);
    mm_acc_adag<NB>(t1, W, rb);
    mat_zero<NB>(t2);
    mm_acc<NB>(t2, t1, W);
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      cplx x = cscal(t2[e], -dt);
      if (corrector) {
        Dbar_prev[(int64_t)k * NBB + e] = cadd(Dbar_prev[(int64_t)k * NBB + e], cscal(x, 0.5));
        Dbar_c[(int64_t)k * NBB + e] = cscal(x, 0.5);
      } else {
        Dbar_prev[(int64_t)k * NBB + e] = cadd(Dbar_prev[(int64_t)k * NBB + e], x);
      }
    }
    cplx* pb = pbar + (int64_t)k * 3 * NBB;
#pragma unroll
    for (int e = 0; e < NBB; ++e) {
      pb[e] = Vb[e];
      pb[NBB + e] = Wb[e];
      pb[2 * NBB + e] = Pb[e];
    }
  }
}

// ------------------------------------------------------------------ propagator adjoint
// nb = 2. X = -i hbar dt, V = exp(X), Vh = exp(X/2), Phi = -i dt phi1(X). The adjoint of f(X) with real
// Taylor coefficients is the Frechet derivative Xbar = L_f(X^dag, fbar), so
//   Xbar = L_exp(X^dag, Vbar) + 1/2 L_exp(X^dag/2, Vhbar) + L_phi1(X^dag, i dt Phibar),  hbarbar = i dt Xbar.
// With Y = X^dag / 2^s, ||Y||_F <= 1/4, one Horner chain of phi1(Y) carries the derivatives in the three
// directions (A <- 1 + Y A / n, dA <- (Y dA + D A) / n, degree 13), exp = 1 + Y phi1, then the doublings
// E' = E^2, phi1' = (E + 1) phi1 / 2 and their derivatives. One lane per column of one k, the pair of
// lanes exchanging columns in the doublings only: 19.9 -> 9.0 us (144 points) against one
// wavefront per k on 8 x 8 block matrices through LDS.
__global__ __launch_bounds__(64) void k_adj_props2(Dims d, const cplx* __restrict__ hop, const cplx* __restrict__ hf,
                                                   const cplx* __restrict__ pbar, double Ax, double Ay, double polx,
                                                   double poly, double dt, double* __restrict__ kpart) {
  constexpr int NB = 2, NBB = 4;
  const int t = blockIdx.x * 64 + threadIdx.x, c = t & 1;
  const int k = (t >> 1) < d.nk ? t >> 1 : d.nk - 1;   // (both lanes of a pair; writes are masked)
  cplx Y[NBB], D[3][NBB];   // directions of Phi, V, Vh
  double nrm2 = 0.0;
  {
    cplx h[NBB];
    bloch_h0<NB>(hop, d.nkx, d.nky, k, Ax, Ay, h);
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        Y[a * NB + b] = cscal(cmuli(cconj(cadd(h[b * NB + a], hf[b * NB + a]))), dt);   // X^dag
        nrm2 += cabs2(Y[a * NB + b]);
      }
  }
  int s = 1;
  const double nrm = sqrt(nrm2);
  while (nrm > ldexp(0.25, s) && s < 60) ++s;
  const double sc = ldexp(1.0, -s);
  const cplx* pb = pbar + (int64_t)k * 3 * NBB;
#pragma unroll
  for (int e = 0; e < NBB; ++e) {
    Y[e] = cscal(Y[e], sc);
    D[0][e] = cscal(cmuli(pb[2 * NBB + e]), dt * sc);
    D[1][e] = cscal(pb[e], sc);
    D[2][e] = cscal(pb[NBB + e], 2.0 * sc);
  }
  auto mul = [](const cplx* M, const cplx* v, cplx* out) {   // out += M v
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int l = 0; l < NB; ++l) cmac(out[r], M[r * NB + l], v[l]);
  };
  cplx f[NB], df[3][NB];   // column c of phi1(Y) and of its derivatives
#pragma unroll
  for (int r = 0; r < NB; ++r) {
    f[r] = cmk(r == c ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int q = 0; q < 3; ++q) df[q][r] = czero();
  }
#pragma unroll
  for (int n = 13; n >= 1; --n) {
    const double inv = 1.0 / (n + 1);
    cplx u[NB] = {czero(), czero()};
    mul(Y, f, u);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      cplx v[NB] = {czero(), czero()};
      mul(Y, df[q], v);
      mul(D[q], f, v);
#pragma unroll
      for (int r = 0; r < NB; ++r) df[q][r] = cscal(v[r], inv);
    }
#pragma unroll
    for (int r = 0; r < NB; ++r) f[r] = cadd(cmk(r == c ? 1.0 : 0.0, 0.0), cscal(u[r], inv));
  }
  cplx E[NB], dE[3][NB], x[NB];   // exp = 1 + Y phi1; x: the Vh term
#pragma unroll
  for (int r = 0; r < NB; ++r) E[r] = cmk(r == c ? 1.0 : 0.0, 0.0);
  mul(Y, f, E);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    dE[q][0] = dE[q][1] = czero();
    mul(Y, df[q], dE[q]);
    mul(D[q], f, dE[q]);
  }
  // the whole matrix of which this lane holds column c
  auto whole = [&](const cplx* col, cplx* M) {
#pragma unroll
    for (int r = 0; r < NB; ++r) {
      const cplx o = cmk(__shfl_xor(col[r].x, 1, 64), __shfl_xor(col[r].y, 1, 64));
      M[r * NB] = c == 0 ? col[r] : o;
      M[r * NB + 1] = c == 0 ? o : col[r];
    }
  };
  const int smax = wave_max(s);
  for (int q = 0; q < smax; ++q) {
    cplx EM[NBB], dM[NBB], e2[NB] = {czero(), czero()}, f2[NB], g2[NB];
    whole(E, EM);
    if (q == s - 1)
#pragma unroll
      for (int r = 0; r < NB; ++r) x[r] = cscal(dE[2][r], 0.5);
    mul(EM, E, e2);
#pragma unroll
    for (int r = 0; r < NB; ++r) {
      f2[r] = f[r];
      g2[r] = df[0][r];
    }
    mul(EM, f, f2);        // (E + 1) phi1
    mul(EM, df[0], g2);    // (E + 1) dphi1 + dE phi1
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cplx v[NB] = {czero(), czero()};
      whole(dE[i], dM);
      if (i == 0) mul(dM, f, g2);
      mul(dM, E, v);
      mul(EM, dE[i], v);
      if (q < s)
#pragma unroll
        for (int r = 0; r < NB; ++r) dE[i][r] = v[r];
    }
    if (q < s)
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        E[r] = e2[r];
        f[r] = cscal(f2[r], 0.5);
        df[0][r] = cscal(g2[r], 0.5);
      }
  }
  // hbarbar column c; dL/dhf_aa += Re hbarbar_aa ;  dL/dA += Re sum conj(hbarbar) dh0/dA, dh0/dA = -(pol . v)
  cplx hb[NB], vx[NBB], vy[NBB];
  bloch_vel<NB>(hop, d.nkx, d.nky, k, Ax, Ay, 0, vx);
  bloch_vel<NB>(hop, d.nkx, d.nky, k, Ax, Ay, 1, vy);
  double dA = 0.0;
#pragma unroll
  for (int r = 0; r < NB; ++r) {
    hb[r] = cscal(cmuli(cadd(cadd(dE[1][r], df[0][r]), x[r])), dt);
    const cplx dh = c == 0 ? cneg(cadd(cscal(vx[r * NB], polx), cscal(vy[r * NB], poly)))
                           : cneg(cadd(cscal(vx[r * NB + 1], polx), cscal(vy[r * NB + 1], poly)));
    dA += hb[r].x * dh.x + hb[r].y * dh.y;
  }
  dA += __shfl_xor(dA, 1, 64);
  if ((t >> 1) < d.nk) {
    kpart[(int64_t)k * (NB + 1) + c] = c == 0 ? hb[0].x : hb[1].x;
    if (c == 0) kpart[(int64_t)k * (NB + 1) + NB] = dA;
  }
}
// nb = 1: M = [[-i hbar dt, dt], [0, 0]];  V = exp(M)_tl,  Phi = -i exp(M)_tr,
// Vh = exp(M/2)_tl.
// For E = exp(X) the adjoint is Xbar = L(X^dag, Ebar), the Frechet derivative of exp at X^dag
// in the direction Ebar, read off the top-right block of exp([[X^dag, Ebar], [0, X^dag]]) (4 x 4).
// Ebar = [[Vbar, i Phibar], [0, 0]] for exp(M), [[Vhbar, 0], [0, 0]] for exp(M/2);
// hbarbar = i dt (Mbar)_tl. One wavefront per k.
__global__ __launch_bounds__(256) void k_adj_props1(Dims d, const cplx* __restrict__ hop, const cplx* __restrict__ hf,
                                                    const cplx* __restrict__ pbar, double Ax, double Ay, double polx,
                                                    double poly, double dt, double* __restrict__ kpart) {
  constexpr int N2 = 2, B2 = 2 * N2, BB = B2 * B2;   // sizes of M and of the block matrix
  __shared__ cplx sX[4][BB], sE[4][BB];
  __shared__ cplx hb[4];
  int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int k = blockIdx.x * 4 + wv;
  bool kval = k < d.nk;
  int r = lane / B2, c = lane - (lane / B2) * B2;
  bool act = kval && lane < BB;
  cplx h = czero();
  if (kval) {
    bloch_h0<1>(hop, d.nkx, d.nky, k, Ax, Ay, &h);
    h = cadd(h, hf[0]);
  }
  const cplx* pb = pbar + (int64_t)(kval ? k : 0) * 3;   // Vbar, Vhbar, Phibar
  // M element (i, j)
  auto Mel = [&](int i, int j, double sc) -> cplx {
    if (i == 0) return j == 0 ? cscal(cmuli(h), -dt * sc) : cmk(dt * sc, 0.0);
    return czero();
  };
  cplx mbar = czero();  // (Mbar)_tl, in the lane of row 0, column N2
  for (int pass = 0; pass < 2; ++pass) {
    double sc = pass == 0 ? 1.0 : 0.5;
    // Ebar element (i, j)
    auto Ebar = [&](int i, int j) -> cplx {
      if (i != 0) return czero();
      if (pass == 0) return j == 0 ? pb[0] : cmuli(pb[2]);
      return j == 0 ? pb[1] : czero();
    };
    // block matrix B = [[M^dag, Ebar/nE], [0, M^dag]] with the direction normalised
    double ne = 0.0;
    if (act && r < N2 && c >= N2) ne = cabs2(Ebar(r, c - N2));
    ne = sqrt(wave_sum(ne));
    double inv_ne = ne > 0.0 ? 1.0 / ne : 0.0;
    cplx x = czero();
    if (act) {
      if (r < N2 && c < N2) x = cconj(Mel(c, r, sc));
      else if (r >= N2 && c >= N2) x = cconj(Mel(c - N2, r - N2, sc));
      else if (r < N2 && c >= N2) x = cscal(Ebar(r, c - N2), inv_ne);
    }
    double nrm = sqrt(wave_sum(act ? cabs2(x) : 0.0));
    int s = 0;
    while (nrm > ldexp(0.25, s) && s < 60) ++s;
    x = cscal(x, ldexp(1.0, -s));
    cplx id = cmk((act && r == c) ? 1.0 : 0.0, 0.0);
    if (lane < BB) sX[wv][lane] = x;
    cplx e = id;
    if (lane < BB) sE[wv][lane] = e;
    wave_sync();  // every LDS array here is per wavefront
    for (int n = 18; n >= 1; --n) {
      cplx acc = czero();
      if (lane < BB)
#pragma unroll
        for (int l = 0; l < B2; ++l) cmac(acc, sX[wv][r * B2 + l], sE[wv][l * B2 + c]);
      wave_sync();
      e = cadd(id, cscal(acc, 1.0 / n));
      if (lane < BB) sE[wv][lane] = e;
      wave_sync();
    }
    for (int q = 0; q < s; ++q) {
      cplx acc = czero();
      if (lane < BB)
#pragma unroll
        for (int l = 0; l < B2; ++l) cmac(acc, sE[wv][r * B2 + l], sE[wv][l * B2 + c]);
      wave_sync();
      e = acc;
      if (lane < BB) sE[wv][lane] = e;
      wave_sync();
    }
    // (0, 0) of the top-right block
    if (act && r == 0 && c == N2) mbar = cadd(mbar, cscal(e, ne * sc));
  }
  // hbarbar = i dt Mbar_tl
  if (act && r == 0 && c == N2) hb[wv] = cscal(cmuli(mbar), dt);
  wave_sync();
  if (kval && lane == 0) {
    // dL/dhf += Re hbarbar ;  dL/dA += Re conj(hbarbar) dh0/dA, dh0/dA = -(pol . v)
    cplx vx, vy;
    bloch_vel<1>(hop, d.nkx, d.nky, k, Ax, Ay, 0, &vx);
    bloch_vel<1>(hop, d.nkx, d.nky, k, Ax, Ay, 1, &vy);
    double dA = 0.0;
    cplx dh = cneg(cadd(cscal(vx, polx), cscal(vy, poly)));
    dA += hb[wv].x * dh.x + hb[wv].y * dh.y;
    kpart[2 * (int64_t)k] = hb[wv].x;
    kpart[2 * (int64_t)k + 1] = dA;
  }
}

// ------------------------------------------------------------------ mean field and pulse
// hf_aa = U Re rho_loc,aa, rho_loc = N_k^{-1} sum_k [(1 - wb) rhoA(k) + wb rhoB(k)] (Hubbard);
// A(t_{m-1/2}) enters h0. One block: reduces the per-k partials, then scatters.
template <int NB>
__global__ __launch_bounds__(256) void k_adj_hf(Dims d, const double* __restrict__ kpart,
                                                const cplx* __restrict__ rhoA, const cplx* __restrict__ rhoB,
                                                double wb, int hf, double U, cplx* __restrict__ rbarA,
                                                cplx* __restrict__ rbarB, double dAdamp, double dAdomega,
                                                double* __restrict__ theta_bar) {
  __shared__ double red[(NB + 1 + NB) * 256];
  __shared__ double tot[NB + 1 + NB];
  int t = threadIdx.x;
  double p[NB + 1 + NB];
#pragma unroll
  for (int i = 0; i < 2 * NB + 1; ++i) p[i] = 0.0;
  for (int k = t; k < d.nk; k += 256) {
#pragma unroll
    for (int i = 0; i <= NB; ++i) p[i] += kpart[(int64_t)k * (NB + 1) + i];
#pragma unroll
    for (int a = 0; a < NB; ++a)
      p[NB + 1 + a] += (1.0 - wb) * rhoA[(int64_t)k * NB * NB + a * NB + a].x + wb * rhoB[(int64_t)k * NB * NB + a * NB + a].x;
  }
#pragma unroll
  for (int i = 0; i < 2 * NB + 1; ++i) red[i * 256 + t] = p[i];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s)
#pragma unroll
      for (int i = 0; i < 2 * NB + 1; ++i) red[i * 256 + t] += red[i * 256 + t + s];
    __syncthreads();
  }
  if (t < 2 * NB + 1) tot[t] = red[t * 256];
  __syncthreads();
  double inv = 1.0 / d.nk;
  if (hf) {
    for (int k = t; k < d.nk; k += 256)
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        double g = U * inv * tot[a];
        int64_t i = (int64_t)k * NB * NB + a * NB + a;
        if (1.0 - wb != 0.0) rbarA[i].x += (1.0 - wb) * g;
        if (wb != 0.0) rbarB[i].x += wb * g;
      }
  }
  if (t == 0) {
    double gU = 0.0;
    if (hf)
#pragma unroll
      for (int a = 0; a < NB; ++a) gU += tot[a] * tot[NB + 1 + a] * inv;
    theta_bar[0] += tot[NB] * dAdamp;
    theta_bar[1] += tot[NB] * dAdomega;
    theta_bar[2] += gU;
  }
}

// ------------------------------------------------------------------ observable seed
// O = N_k^{-1} sum_k Re tr[P_k rho_k], P_k the projector on band b of h0(k - A(T)) (or on
// orbital a). rhobar_T = P_k / N_k; for bands also dO/dA(T) by first-order perturbation
// theory, dP_b = sum_{c != b} (u_c u_c^dag dh u_b u_b^dag + h.c.) / (e_b - e_c), dh = -(pol.v) dA.
template <int NB>
__global__ __launch_bounds__(256) void k_adj_seed(Dims d, const cplx* __restrict__ hop, const cplx* __restrict__ rho,
                                                  double Ax, double Ay, double polx, double poly, int obs_id,
                                                  cplx* __restrict__ rhobar, double dAdamp, double dAdomega,
                                                  double* __restrict__ theta_bar) {
  constexpr int NBB = NB * NB;
  __shared__ double red[256];
  double inv = 1.0 / d.nk;
  double dOdA = 0.0;
  for (int k = threadIdx.x; k < d.nk; k += 256) {
    cplx Pm[NBB];
#pragma unroll
    for (int e = 0; e < NBB; ++e) Pm[e] = czero();
    if (obs_id >= KBE_DEV_OBS_NORB && obs_id < KBE_DEV_OBS_NORB + NB) {
      int a = obs_id - KBE_DEV_OBS_NORB;
      Pm[a * NB + a] = cmk(1.0, 0.0);
    } else {
      int b = obs_id - KBE_DEV_OBS_NBAND;
      cplx h[NBB], U[NBB], vx[NBB], vy[NBB], dh[NBB];
      double w[NB];
      bloch_h0<NB>(hop, d.nkx, d.nky, k, Ax, Ay, h);
      jacobi_eigh<NB>(h, w, U);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) Pm[i * NB + j] = cmul(U[i * NB + b], cconj(U[j * NB + b]));
      bloch_vel<NB>(hop, d.nkx, d.nky, k, Ax, Ay, 0, vx);
      bloch_vel<NB>(hop, d.nkx, d.nky, k, Ax, Ay, 1, vy);
#pragma unroll
      for (int e = 0; e < NBB; ++e) dh[e] = cneg(cadd(cscal(vx[e], polx), cscal(vy[e], poly)));
      const cplx* r = rho + (int64_t)k * NBB;
      // Re tr(dP rho) = 2 Re sum_{c != b} <u_b|rho|u_c><u_c|dh|u_b> / (e_b - e_c)
      for (int c = 0; c < NB; ++c) {
        if (c == b) continue;
        cplx rbc = czero(), hcb = czero();
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            rbc = cadd(rbc, cmul(cmul(cconj(U[i * NB + b]), r[i * NB + j]), U[j * NB + c]));
            hcb = cadd(hcb, cmul(cmul(cconj(U[i * NB + c]), dh[i * NB + j]), U[j * NB + b]));
          }
        dOdA += 2.0 * cmul(rbc, hcb).x / (w[b] - w[c]);
      }
    }
#pragma unroll
    for (int e = 0; e < NBB; ++e) rhobar[(int64_t)k * NBB + e] = cscal(Pm[e], inv);
  }
  red[threadIdx.x] = dOdA * inv;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    theta_bar[0] += red[0] * dAdamp;
    theta_bar[1] += red[0] * dAdomega;
  }
}

// The row kernel stores the equal-time block as G^<(t_m, t_m) = i rho_m; multiplying by -i
// swaps the parts and flips one sign, so rho_m comes back bit for bit from the history.
template <int NB>
__global__ void k_adj_rho(Dims d, const void* __restrict__ hist, int m, cplx* __restrict__ rho) {
  constexpr int NBB = NB * NB;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.nk * NBB) return;
  int k = i / NBB, e = i - (i / NBB) * NBB;
  cplx g = static_cast<const cplx*>(hist)[hist_idx(d, k, e, m, m)];  // FP64 history
  rho[i] = cmk(g.y, -g.x);
}

// What a reverse step starts from: the working copies of the committed rows m and m - 1 and rho_{m-1},
// read back from the history (the column and diagonal copies are those of the forward run, refreshed
// once at the seed: no kernel of the sweep writes them), and the cleared accumulators of the step
// after. One thread per (k, component, t').
struct ClearList {
  double* p[4];
  int64_t n[4];
};
template <int NB>
__global__ __launch_bounds__(256) void k_adj_begin(Dims d, const cplx* __restrict__ hist, cplx* __restrict__ row64,
                                                   cplx* __restrict__ rho, int m, ClearList z) {
  constexpr int NBB = NB * NB;
  const int j = blockIdx.x * 256 + threadIdx.x;
  const int k = blockIdx.y / d.C, c = blockIdx.y - k * d.C;
  if (j <= m) row64[row64_idx(d, m, k, c, j)] = hist[hist_idx(d, k, c, m, j)];
  if (j <= m - 1) {
    const cplx g = hist[hist_idx(d, k, c, m - 1, j)];
    row64[row64_idx(d, m - 1, k, c, j)] = g;
    if (j == m - 1 && c < NBB) rho[(int64_t)k * NBB + c] = cmk(g.y, -g.x);   // G^< = i rho
  }
  const int64_t t = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * gridDim.y * 256;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    for (int64_t i = t; i < z.n[q]; i += nt) z.p[q][i] = 0.0;
}

// ------------------------------------------------------------------ launchers
template <int NB>
struct AdjLaunch {
  static hipError_t begin(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, hipStream_t st) {
    const int64_t row = 2 * (int64_t)d.nk * d.C * d.Tp, mat = 2 * (int64_t)d.nk * NB * NB;
    const ClearList z{{(double*)b.Ibar_prev, (double*)b.Dbar_prev, (double*)b.rhobar_prev, (double*)b.rhobar_P},
                      {row, mat, mat, mat}};
    hipLaunchKernelGGL(k_adj_begin<NB>, dim3(m / 256 + 1, d.nk * d.C), dim3(256), 0, st, d, (const cplx*)a.hist,
                       a.row64, b.rho0, m, z);
    return hipGetLastError();
  }
  static hipError_t bulk(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* Ibar, int m, int mode,
                         const cplx* sig1, const cplx* Ibar1, hipStream_t st) {
    if (m < 1) return hipSuccess;
    int ns = (m + 63) / 64;
    if (mode == ADJ_SUMS)
      hipLaunchKernelGGL((k_adj_bulk<NB, ADJ_SUMS>), dim3((ns + 1) * d.nk), dim3(256), 0, st, d, (const cplx*)a.hist,
                         b.lam, (const cplx*)a.sig, Ibar, (const cplx*)a.sig, Ibar, b.sbar_col, b.sbar_rowpart,
                         (const cplx*)a.row64, (const cplx*)a.col0, b.rowtot, m, a.dt);
    else
      hipLaunchKernelGGL((k_adj_bulk<NB, ADJ_FUSED>), dim3((ns + 1) * d.nk), dim3(256), 0, st, d, (const cplx*)a.hist,
                         b.lam, (const cplx*)a.sig, Ibar, sig1, Ibar1, b.sbar_col, b.sbar_rowpart,
                         (const cplx*)a.row64, (const cplx*)a.col0, b.rowtot, m, a.dt);
    return hipGetLastError();
  }
  static hipError_t row(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* Ibar, const cplx* Dbar,
                        int m, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_row<NB>, dim3(m / 64 + 1, d.nk), dim3(64), 0, st, d, (const cplx*)a.row64,
                       (const cplx*)a.sig, (const cplx*)a.col0, (const cplx*)a.diag, Ibar, Dbar,
                       (const cplx*)b.sbar_col, (const cplx*)b.sbar_rowpart, (const cplx*)b.rowtot, b.sbar, b.Rbar,
                       b.lam, b.lam_diag, b.lam_col0, m, a.dt);
    return hipGetLastError();
  }
  static hipError_t sigma(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, int* nblocks,
                          hipStream_t st) {
    int total = (m + 1) * NB * NB;
    int per = (total + 7) / 8;
    *nblocks = per * 8;
    size_t shm = (size_t)(4 * d.nk) * sizeof(cplx);
    auto kern = k_adj_sigma<NB, 0, 0>;
    if constexpr (NB == 2) {
      if (d.nkx == 24 && d.nky == 24) kern = k_adj_sigma<NB, 24, 24>;
      else if (d.nkx == 16 && d.nky == 16) kern = k_adj_sigma<NB, 16, 16>;
      else if (d.nkx == 12 && d.nky == 12) kern = k_adj_sigma<NB, 12, 12>;
      else if (d.nkx == 16 && d.nky == 1) kern = k_adj_sigma<NB, 16, 1>;
    }
    hipLaunchKernelGGL(kern, dim3(per * 8), dim3(256), shm, st, d, (const cplx*)a.row64, (const cplx*)b.sbar, b.Rbar,
                       b.ubar_part, m, a.U, a.corr);
    return hipGetLastError();
  }
  // nubar: dL/dU partials of the collision pass before, added into theta_bar along the way
  static hipError_t update(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, int corrector, int nubar,
                           const cplx* Gbar_hist, const cplx* Gbar_row, const cplx* rho_prev, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_update<NB>, dim3(d.nk + 1), dim3(256 * NB), 0, st, d, Gbar_hist, Gbar_row, b.lam,
                       (const cplx*)a.row64, (const cplx*)(corrector ? b.props_c : b.props_p),
                       (const cplx*)b.Ire_prev, (const cplx*)b.Ire_c, rho_prev, (const cplx*)a.D_prev,
                       (const cplx*)b.Dc, b.Ibar_prev, b.Ibar_c, corrector ? b.rhobar : b.rhobar_P,
                       b.rhobar_prev, b.Dbar_prev, b.Dbar_c, b.pbar, m, a.dt, corrector,
                       (const cplx*)b.lam_diag, (const cplx*)b.lam_col0, (const double*)b.ubar_part, nubar, b.theta_bar);
    return hipGetLastError();
  }
  static hipError_t props(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* hf, hipStream_t st) {
    if constexpr (NB == 2)
      hipLaunchKernelGGL(k_adj_props2, dim3((2 * d.nk + 63) / 64), dim3(64), 0, st, d, (const cplx*)a.hop, hf,
                         (const cplx*)b.pbar, a.Ax, a.Ay, a.polx, a.poly, a.dt, b.kpart);
    else
      hipLaunchKernelGGL(k_adj_props1, dim3((d.nk + 3) / 4), dim3(256), 0, st, d, (const cplx*)a.hop, hf,
                         (const cplx*)b.pbar, a.Ax, a.Ay, a.polx, a.poly, a.dt, b.kpart);
    return hipGetLastError();
  }
  static hipError_t hf(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* rA, const cplx* rB,
                       double wb, cplx* rbA, cplx* rbB, double dAdamp, double dAdomega, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_hf<NB>, dim3(1), dim3(256), 0, st, d, (const double*)b.kpart, rA, rB, wb, a.hf, a.U,
                       rbA, rbB, dAdamp, dAdomega, b.theta_bar);
    return hipGetLastError();
  }
  static hipError_t rho(const Dims& d, const void* hist, int m, cplx* out, hipStream_t st) {
    int n = d.nk * NB * NB;
    hipLaunchKernelGGL(k_adj_rho<NB>, dim3((n + 255) / 256), dim3(256), 0, st, d, hist, m, out);
    return hipGetLastError();
  }
  static hipError_t seed(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* rho_T, int obs_id,
                         double dAdamp, double dAdomega, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_seed<NB>, dim3(1), dim3(256), 0, st, d, (const cplx*)a.hop, rho_T, a.Ax, a.Ay, a.polx,
                       a.poly, obs_id, b.rhobar, dAdamp, dAdomega, b.theta_bar);
    return hipGetLastError();
  }
};

#define KBE_ADJ_DISPATCH(NBV, CALL)       \
  switch (NBV) {                          \
    case 1: return AdjLaunch<1>::CALL;    \
    case 2: return AdjLaunch<2>::CALL;    \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_adj_bulk(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* Ibar, int m, int mode,
                           const cplx* sig1, const cplx* Ibar1, hipStream_t st) {
  if (mode != ADJ_SUMS && (mode != ADJ_FUSED || !sig1 || !Ibar1)) return hipErrorInvalidValue;
  KBE_ADJ_DISPATCH(d.nb, bulk(d, a, b, Ibar, m, mode, sig1, Ibar1, st));
}
hipError_t launch_adj_row(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* Ibar, const cplx* Dbar,
                          int m, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, row(d, a, b, Ibar, Dbar, m, st));
}
hipError_t launch_adj_sigma(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, int* nblocks,
                            hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, sigma(d, a, b, m, nblocks, st));
}
hipError_t launch_adj_update(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, int corrector, int nubar,
                             const cplx* Gbar_hist, const cplx* Gbar_row, const cplx* rho_prev, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, update(d, a, b, m, corrector, nubar, Gbar_hist, Gbar_row, rho_prev, st));
}
hipError_t launch_adj_props(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* hf,
                            hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, props(d, a, b, hf, st));
}
hipError_t launch_adj_hf(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* rho_prev,
                         const cplx* rho_cur, double wb, cplx* rbar_prev, cplx* rbar_cur, double dAdamp,
                         double dAdomega, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, hf(d, a, b, rho_prev, rho_cur, wb, rbar_prev, rbar_cur, dAdamp, dAdomega, st));
}
hipError_t launch_adj_seed(const Dims& d, const LaunchArgs& a, const AdjArgs& b, const cplx* rho_T, int obs_id,
                           double dAdamp, double dAdomega, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, seed(d, a, b, rho_T, obs_id, dAdamp, dAdomega, st));
}

hipError_t launch_adj_begin(const Dims& d, const LaunchArgs& a, const AdjArgs& b, int m, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, begin(d, a, b, m, st));
}

hipError_t launch_adj_rho(const Dims& d, const void* hist, int m, cplx* rho, hipStream_t st) {
  KBE_ADJ_DISPATCH(d.nb, rho(d, hist, m, rho, st));
}

}  // namespace kbe
