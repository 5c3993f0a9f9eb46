// tgks_flux_face.hpp -- the Gauss-point flux (Sec. 2.1, Eqs. 2.2-2.9) from
// moments in the frame of the face: tables of every monomial's moments, the
// micro slopes by closed-form linear solves, the equilibrium part by
// directional derivatives of the Euler flux.  The same flux as gp_flux of
// tgks_device.hpp, which evaluates it in the frame of the tangential velocity
// with 209 fewer instructions per lane; the two agree to rounding.  Used by
// the reverse mode (which differentiates these pieces) and by the 2-D kernels
// with characteristic variables (see gp_flux_face).
#pragma once
#include "tgks_device.hpp"

namespace tgks {

constexpr int NMT = 6;  // tangential tables <u_t^n>, n = 0..5

template <class R>
TGKS_HD void full_table(R U, R h, R* m, int n) {
  m[0] = R(1.0);
  m[1] = U;
  for (int k = 1; k + 1 < n; ++k) m[k + 1] = U * m[k] + ((double)k * h) * m[k - 1];
}

template <int D, class R>
struct MomSet {
  R m1[NM1];
  R mt[D > 1 ? D - 1 : 1][NMT];
  R xi1, xi2;  // <xi^2>, <xi^4>
};

template <int D, class R>
TGKS_HD R mono(const MomSet<D, R>& S, int i, int j, int k) {
  R v = S.m1[i];
  if (D >= 2) v = v * S.mt[0][j];
  if (D >= 3) v = v * S.mt[D >= 3 ? 1 : 0][k];
  return v;
}

// g[alpha] = <psi_alpha u1^i u2^j u3^k xi^(2l)>, l in {0, 1}
template <int D, class R>
TGKS_HD void gpsi(const MomSet<D, R>& S, int i, int j, int k, int l, R* g) {
  const R base = mono(S, i, j, k);
  g[0] = l == 0 ? base : base * S.xi1;
  g[1] = l == 0 ? mono(S, i + 1, j, k) : mono(S, i + 1, j, k) * S.xi1;
  if (D >= 2) g[2] = l == 0 ? mono(S, i, j + 1, k) : mono(S, i, j + 1, k) * S.xi1;
  if (D >= 3) g[D >= 3 ? 3 : 0] = l == 0 ? mono(S, i, j, k + 1) : mono(S, i, j, k + 1) * S.xi1;
  R e = mono(S, i + 2, j, k);
  if (D >= 2) e = e + mono(S, i, j + 2, k);
  if (D >= 3) e = e + mono(S, i, j, k + 2);
  g[D + 1] = l == 0 ? 0.5 * (e + base * S.xi1) : 0.5 * (e * S.xi1 + base * S.xi2);
}

// out[alpha] (+)= s * <psi_alpha a(psi) u1^i u2^j u3^k>
template <int D, bool ACC, class R>
TGKS_HD void mpsia(const MomSet<D, R>& S, const R* a, int i, int j, int k, R s, R* out) {
  constexpr int NC = D + 2;
  R g[NC], t[NC], r[NC];
  gpsi<D>(S, i, j, k, 0, g);
#pragma unroll
  for (int q = 0; q < NC; ++q) r[q] = a[0] * g[q];
  gpsi<D>(S, i + 1, j, k, 0, g);
#pragma unroll
  for (int q = 0; q < NC; ++q) r[q] += a[1] * g[q];
  if (D >= 2) {
    gpsi<D>(S, i, j + 1, k, 0, g);
#pragma unroll
    for (int q = 0; q < NC; ++q) r[q] += a[2] * g[q];
  }
  if (D >= 3) {
    gpsi<D>(S, i, j, k + 1, 0, g);
#pragma unroll
    for (int q = 0; q < NC; ++q) r[q] += a[D >= 3 ? 3 : 0] * g[q];
  }
  gpsi<D>(S, i + 2, j, k, 0, t);
  if (D >= 2) {
    gpsi<D>(S, i, j + 2, k, 0, g);
#pragma unroll
    for (int q = 0; q < NC; ++q) t[q] += g[q];
  }
  if (D >= 3) {
    gpsi<D>(S, i, j, k + 2, 0, g);
#pragma unroll
    for (int q = 0; q < NC; ++q) t[q] += g[q];
  }
  gpsi<D>(S, i, j, k, 1, g);
  const R ae = 0.5 * a[NC - 1];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const R v = r[q] + ae * (t[q] + g[q]);
    if (ACC)
      out[q] += s * v;
    else
      out[q] = s * v;
  }
}

// closed-form solution a of <a psi> = b (per unit density) over the full
// Maxwellian (U, lambda), N = K + D.
template <int D, class R>
TGKS_HD void micro_solve(const Gas<D, R>& g, double N, const R* b, R* a) {
  R ub = R(0.0), u2 = R(0.0);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    ub += g.U[d] * b[d + 1];
    u2 += g.U[d] * g.U[d];
  }
  const R lam = g.lam;
  const R aE = ((4.0 / N) * (lam * lam)) * ((2.0 * b[D + 1] - 2.0 * ub) + (u2 - N * g.h) * b[0]);
  R ua = R(0.0);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    a[d + 1] = (2.0 * lam) * (b[d + 1] - g.U[d] * b[0]) - g.U[d] * aE;
    ua += g.U[d] * a[d + 1];
  }
  a[D + 1] = aE;
  a[0] = (b[0] - ua) - (0.5 * aE) * (u2 + N * g.h);
}

template <int D, class R>
TGKS_HD void tangential_tables(const Gas<D, R>& g, MomSet<D, R>& S) {
#pragma unroll
  for (int d = 1; d < D; ++d) full_table(g.U[d], g.h, S.mt[d - 1], NMT);
}

template <int D, class R>
TGKS_HD void xi_moments(const Gas<D, R>& g, double K, MomSet<D, R>& S) {
  S.xi1 = K * g.h;
  S.xi2 = (K * (K + 2.0)) * (g.h * g.h);
}

// (i, j, k) exponents of u_d
TGKS_HD void unit(int d, int& i, int& j, int& k) {
  i = d == 0;
  j = d == 1;
  k = d == 2;
}

// Directional derivatives of closed-form moments of a Maxwellian g(W).
// The derivative of g along a change dW of its conservative variables is
// g a(psi) with <a psi> = dW / rho, so every full-space moment of g a(psi)
// is the directional derivative of the corresponding moment of g:
//   rho <u_k psi a>      = J_k(W) dW     (Euler flux F_k = rho <u_k psi>)
//   rho <u_1 u_d psi a>  = dG_1d(W) dW   (G_1d = rho <u_1 u_d psi>)
// which replaces micro-slope solves and moment sums over the full space.
template <int D, class R>
struct Prim {
  R dU[D], dp, dh;
};

template <int D, class R>
TGKS_HD void prim_dir(const Gas<D, R>& g, double N, const R* dW, Prim<D, R>& o) {
  R udm = R(0.0), u2 = R(0.0);
#pragma unroll
  for (int e = 0; e < D; ++e) {
    o.dU[e] = (dW[e + 1] - g.U[e] * dW[0]) * g.irho;
    udm += g.U[e] * dW[e + 1];
    u2 += g.U[e] * g.U[e];
  }
  // p = (2/N)(E - rho |U|^2 / 2)
  o.dp = (2.0 / N) * ((dW[D + 1] - udm) + (0.5 * u2) * dW[0]);
  o.dh = (o.dp - g.h * dW[0]) * g.irho;
}

// out = J_k(W) dW, the Euler flux along frame axis k differentiated along dW
template <int D, class R>
TGKS_HD void euler_jvp(const Gas<D, R>& g, R E, int k, const R* dW, const Prim<D, R>& d, R* out) {
  const R p = g.rho * g.h;
  const R mk = g.rho * g.U[k];
  out[0] = dW[k + 1];
#pragma unroll
  for (int e = 0; e < D; ++e) {
    R v = dW[k + 1] * g.U[e] + mk * d.dU[e];
    if (e == k) v += d.dp;
    out[e + 1] = v;
  }
  out[D + 1] = d.dU[k] * (E + p) + g.U[k] * (dW[D + 1] + d.dp);
}

// out = dG_1d(W) dW with G_1d = rho <u_1 u_d psi> (frame axis 0 normal):
//   alpha 0: rho U1 Ud + p [d=0]
//   alpha e: rho U1 Ud Ue + p (U1 [d=e] + Ud [e=0] + Ue [d=0])
//   alpha E: rho U1 Ud (|U|^2 + (N+4) h)/2 + [d=0] p (|U|^2 + (N+2) h)/2
template <int D, class R>
TGKS_HD void g1d_jvp(const Gas<D, R>& g, double N, int d, const R* dW, const Prim<D, R>& q, R* out) {
  const R p = g.rho * g.h;
  const R dp = q.dp;
  R u2 = R(0.0), udu = R(0.0);
#pragma unroll
  for (int e = 0; e < D; ++e) {
    u2 += g.U[e] * g.U[e];
    udu += g.U[e] * q.dU[e];
  }
  const R A = g.U[0] * g.U[d];
  const R dA = q.dU[0] * g.U[d] + g.U[0] * q.dU[d];
  const R dr = dW[0];
  const R rdA = dr * A + g.rho * dA;  // d(rho A)
  out[0] = d == 0 ? rdA + dp : rdA;
  const R rA = g.rho * A;
#pragma unroll
  for (int e = 0; e < D; ++e) {
    R v = rdA * g.U[e] + rA * q.dU[e];
    if (d == e) v += dp * g.U[0] + p * q.dU[0];
    if (e == 0) v += dp * g.U[d] + p * q.dU[d];
    if (d == 0) v += dp * g.U[e] + p * q.dU[e];
    out[e + 1] = v;
  }
  const R Q = u2 + (N + 4.0) * g.h;
  const R dQ = 2.0 * udu + (N + 4.0) * q.dh;
  R vE = rdA * Q + rA * dQ;
  if (d == 0) {
    const R Rr = u2 + (N + 2.0) * g.h;
    const R dRr = 2.0 * udu + (N + 2.0) * q.dh;
    vE += dp * Rr + p * dRr;
  }
  out[D + 1] = 0.5 * vE;
}


// gas state, half-space seeds and the side's share rho_s <psi>_s of W0;
// sgn = +1 for the left side (u1 > 0), -1 for the right side
template <int D, class R>
TGKS_HD void face_side_w0(const R* Ws, const FluxCfg& P, double sgn, Gas<D, R>& gs, R& h0, R& h1, R* w0) {
  constexpr int NC = D + 2;
  make_gas<D>(Ws, P.N, gs);
  half_seed(gs.U[0], gs.lam, sgn, h0, h1);
  MomSet<D, R> S;
  moment_table(gs.U[0], gs.h, h0, h1, S.m1);
  tangential_tables<D>(gs, S);
  xi_moments<D>(gs, P.K, S);
  R g[NC];
  gpsi<D>(S, 0, 0, 0, 0, g);
#pragma unroll
  for (int q = 0; q < NC; ++q) w0[q] = gs.rho * g[q];
}

// the side's shares of the slopes of W0 and of the non-equilibrium moments
template <int D, bool NS, class R>
TGKS_HD void face_side_part(const Gas<D, R>& gs, R h0, R h1, const R* Ws, const R (*dW)[D + 2], const FluxCfg& P,
                       const Gas<D, R>& g0, SidePart<D, R>& o) {
  constexpr int NC = D + 2;
  const double N = P.N;
  MomSet<D, R> Sh;
  moment_table(gs.U[0], gs.h, h0, h1, Sh.m1);
  tangential_tables<D>(gs, Sh);
  xi_moments<D>(gs, P.K, Sh);
  R a[D][NC];
  R Wt[NC];  // rho <(sum_d u_d a_d) psi> = sum_d J_d dW_d; A^s solves <A psi> = -that / rho
#pragma unroll
  for (int d = 0; d < D; ++d) {
    R b[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) b[q] = dW[d][q] * gs.irho;
    micro_solve<D>(gs, N, b, a[d]);
    mpsia<D, false>(Sh, a[d], 0, 0, 0, gs.rho, o.dW0[d]);
    Prim<D, R> pd;
    prim_dir<D>(gs, N, dW[d], pd);
    R jv[NC];
    euler_jvp<D>(gs, Ws[D + 1], d, dW[d], pd, jv);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      if (d == 0)
        Wt[q] = jv[q];
      else
        Wt[q] += jv[q];
    }
  }
  R A[NC];
  {
    R b[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) b[q] = -(Wt[q] * gs.irho);
    micro_solve<D>(gs, N, b, A);
  }
  R g[NC];
  gpsi<D>(Sh, 1, 0, 0, 0, g);
  R v2[NC];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    int i, j, k;
    unit(d, i, j, k);
    if (d == 0)
      mpsia<D, false>(Sh, a[d], 1 + i, j, k, R(1.0), v2);
    else
      mpsia<D, true>(Sh, a[d], 1 + i, j, k, R(1.0), v2);
  }
  R v3[NC];
  mpsia<D, false>(Sh, A, 1, 0, 0, R(1.0), v3);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    o.S1[q] = gs.rho * g[q];
    o.S2[q] = gs.rho * v2[q];
    o.S3[q] = gs.rho * v3[q];
  }
  o.H1 = o.H2 = o.H3 = R(0.0);
  if (NS) {
    R f0[NC], w2[NC], w3[NC];
    gpsi<D>(Sh, 0, 0, 0, 0, f0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      int i, j, k;
      unit(d, i, j, k);
      if (d == 0)
        mpsia<D, false>(Sh, a[d], i, j, k, R(1.0), w2);
      else
        mpsia<D, true>(Sh, a[d], i, j, k, R(1.0), w2);
    }
    mpsia<D, false>(Sh, A, 0, 0, 0, R(1.0), w3);
    o.H1 = gs.rho * heat_combine<D>(g, f0, g0.U);
    o.H2 = gs.rho * heat_combine<D>(v2, w2, g0.U);
    o.H3 = gs.rho * heat_combine<D>(v3, w3, g0.U);
  }
}

// Equilibrium part of Eq. 2.5 and the time integration over dt and dt/2,
// given W0, its gas state g0, the two sides' shares summed left + right
// (dW0, S1..S3, H1..H3) and the side pressures pl, pr (collision time).
template <int D, bool NS, class R>
TGKS_HD void face_flux_combine(const R* W0, const Gas<D, R>& g0, const SidePart<D, R>& T, R pl, R pr,
                          const FluxCfg& P, R dt, R* Fdt, R* Fh) {
  constexpr int NC = D + 2;
  const double N = P.N;
  const R(*dW0)[NC] = T.dW0;
  const R *S1 = T.S1, *S2 = T.S2, *S3 = T.S3;
  const R H1 = T.H1, H2 = T.H2, H3 = T.H3;
  // equilibrium part of Eq. 2.5, rho0-weighted moments in closed form:
  //   T1 = rho0 <u1 psi>_0 = F_1(W0)
  //   W0t = -sum_d J_d(W0) dW0_d = rho0 <Abar psi>_0 (compatibility, Eq. 2.7)
  //   T2 = rho0 sum_d <u1 u_d psi abar_d>_0 = sum_d dG_1d(W0) dW0_d
  //   T3 = rho0 <u1 psi Abar>_0 = J_1(W0) W0t
  R T1[NC], T2[NC], T3[NC], W0t[NC];
  {
    const R p0 = g0.rho * g0.h;
    const R E0 = W0[D + 1];
    T1[0] = W0[1];
#pragma unroll
    for (int e = 0; e < D; ++e) T1[e + 1] = W0[1] * g0.U[e] + (e == 0 ? p0 : R(0.0));
    T1[D + 1] = g0.U[0] * (E0 + p0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      Prim<D, R> pd;
      prim_dir<D>(g0, N, dW0[d], pd);
      R jv[NC], gv[NC];
      euler_jvp<D>(g0, E0, d, dW0[d], pd, jv);
      g1d_jvp<D>(g0, N, d, dW0[d], pd, gv);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        if (d == 0) {
          W0t[q] = -jv[q];
          T2[q] = gv[q];
        } else {
          W0t[q] -= jv[q];
          T2[q] += gv[q];
        }
      }
    }
    Prim<D, R> pt;
    prim_dir<D>(g0, N, W0t, pt);
    euler_jvp<D>(g0, E0, 0, W0t, pt, T3);
  }
  R G2 = R(0.0), G3 = R(0.0);  // heat-flux moments of the equilibrium part (the first vanishes)
  if (NS) {
    // <psi sum_d u_d abar_d>_0 = -<psi Abar>_0 by the compatibility condition
    R w2[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) w2[q] = -W0t[q];
    G2 = heat_combine<D>(T2, w2, g0.U);
    G3 = heat_combine<D>(T3, W0t, g0.U);
  }

  // collision time (Sec. 5 preamble); dt is the full step in both stages.
  // xh = -dt / (2 tau): e^{-dt/tau} = (e^{xh})^2, one expm1 serves both
  // intervals.
  const R S = pl + pr, A = fabs(pl - pr);
  R tau = R(0.0), xh = R(0.0);
  if (P.tau_mode == 1) {
    tau = P.mu * recip(g0.rho * g0.h) + (P.c2 * (A * recip(S))) * dt;
    xh = -(0.5 * dt) * recip(tau);
  } else if (P.tau_mode == 0) {
    // tau = (c1 + c2 A/S) dt = dt T/S with T = c1 S + c2 A; one reciprocal
    const R T = P.c1 * S + P.c2 * A;
    if (T > 0.0) {
      const R inv = recip(S * T);
      tau = dt * ((T * T) * inv);
      xh = -0.5 * ((S * S) * inv);
    }
  }
  R em = R(0.0);
  if (tau != 0.0) em = expm1(xh);

#pragma unroll
  for (int id = 0; id < 2; ++id) {
    const R dl = id == 0 ? dt : 0.5 * dt;
    R e, ome;
    if (tau == 0.0) {
      e = R(0.0);
      ome = R(1.0);
    } else if (id == 1) {
      e = em + 1.0;
      ome = -em;
    } else {
      e = (em + 1.0) * (em + 1.0);
      ome = -em * (em + 2.0);
    }
    const R tt = (tau * tau) * ome;
    const R C1 = dl - tau * ome;
    const R C2 = 2.0 * tt - (tau * dl) * (1.0 + e);
    const R C3 = (0.5 * dl) * dl - tau * dl + tt;
    const R C4 = tau * ome;
    const R C5 = (tau * dl) * e - 2.0 * tt;
    const R C6 = -tt;
    R* F = id == 0 ? Fdt : Fh;
#pragma unroll
    for (int q = 0; q < NC; ++q)
      F[q] = ((C1 * T1[q] + C2 * T2[q]) + C3 * T3[q]) + ((C4 * S1[q] + C5 * S2[q]) + C6 * S3[q]);
    if (NS) {
      const R q = (C2 * G2 + C3 * G3) + ((C4 * H1 + C5 * H2) + C6 * H3);
      F[NC - 1] += P.pr_fix * q;
    }
  }
}

// Time-integrated flux F(dt) and F(dt/2) at one Gauss point.
// Wl, Wr: states; dWl[d], dWr[d]: derivatives along frame axis d.
// Returns false when a state is non-physical.
//
// The 2-D kernels with characteristic variables take their flux from here and
// their Gauss-point values from teno_gauss_powers.  The reason is robustness,
// not speed: long viscous runs with these variables amplify rounding across a
// grid-aligned shock, and how often that ends on a non-physical state depends
// on how the values are rounded.  Viscous shock tube, 500 x 250, Re 200, 40
// runs to t = 0.4 that differ by 1e-13 of the Courant number (half of them with
// the first-order fallback): 40 survive with this pair, 31 with these values
// and the flux of gp_flux, 9 with the values of teno_poly and this flux, 13
// with teno_poly and gp_flux; the run from the unchanged data reaches t = 1
// with this pair and stopped at t = 0.144 with the last.  The two forms agree to
// rounding and teno_poly's is the more exact one (a constant stays one to the
// bit), so the loss is no error of its values; why its rounding suits these
// runs less is not known.  Eight steps take 1.78 ms with this pair and 1.44
// with the last.
template <int D, bool NS, class R>
TGKS_HD bool gp_flux_face(const R* Wl, const R* Wr, const R (*dWl)[D + 2], const R (*dWr)[D + 2], const FluxCfg& P,
                          R dt, R* Fdt, R* Fh) {
  constexpr int NC = D + 2;
  Gas<D, R> gl, gr, g0;
  R hl0, hl1, hr0, hr1, wl[NC], wr[NC], W0[NC];
  // equilibrium state by kinetic weighting (Eq. 2.6): rho_l <psi>_{>0} + rho_r <psi>_{<0}
  face_side_w0<D>(Wl, P, 1.0, gl, hl0, hl1, wl);
  face_side_w0<D>(Wr, P, -1.0, gr, hr0, hr1, wr);
#pragma unroll
  for (int q = 0; q < NC; ++q) W0[q] = wl[q] + wr[q];
  make_gas<D>(W0, P.N, g0);
  // side contributions: dW0 (Eq. 2.6), A^s (Eq. 2.7), and the moments of the
  // non-equilibrium part of Eq. 2.5 over the half space
  SidePart<D, R> L, Rt, T;
  face_side_part<D, NS>(gl, hl0, hl1, Wl, dWl, P, g0, L);
  face_side_part<D, NS>(gr, hr0, hr1, Wr, dWr, P, g0, Rt);
  side_sum<D>(L, Rt, T);
  face_flux_combine<D, NS>(W0, g0, T, gl.rho * gl.h, gr.rho * gr.h, P, dt, Fdt, Fh);
  return gl.ok && gr.ok && g0.ok;
}

// What a stage's update takes from F(dt) and F(dt/2) at a Gauss point of weight
// w, added to accA (stage 1 also accB)
template <int STAGE, int NC, class R>
TGKS_HD void combine_times(const R* Fdt, const R* Fh, double w, R* accA, R* accB) {
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    if (STAGE == 1) {
      accA[q] += w * Fh[q];
      accB[q] += w * ((8.0 / 3.0) * Fh[q] - (1.0 / 3.0) * Fdt[q]);
    } else {
      accA[q] += w * ((4.0 / 3.0) * Fdt[q] - (8.0 / 3.0) * Fh[q]);
    }
  }
}

// teno_gauss from the power series of the selected polynomials about the cell
// centre (one branch per kind of stencil); see gp_flux_face
template <class R>
TGKS_HD void teno_gauss_powers(const R* Q, unsigned flag, R* val, R* der) {
  const R a = Q[0], b = Q[1], c = Q[2], d = Q[3], e = Q[4];
  const double s = 0.28867513459481288225;  // 1/(2 sqrt 3)
  R c0, c1, c2, c3 = R(0.0), c4 = R(0.0);
  if (flag & 1u) {
    c0 = ((2134.0 * c - 116.0 * (d + b)) + 9.0 * (e + a)) * (1.0 / 1920.0);
    c1 = (34.0 * (d - b) - 5.0 * (e - a)) * (1.0 / 48.0);
    c2 = ((12.0 * (d + b) - 22.0 * c) - (e + a)) * (1.0 / 16.0);
    c3 = ((e - a) - 2.0 * (d - b)) * (1.0 / 12.0);
    c4 = ((((a - 4.0 * b) + 6.0 * c) - 4.0 * d) + e) * (1.0 / 24.0);
  } else {
    const bool k0 = flag & 2u, k1 = flag & 4u, k2 = flag & 8u;
    const int cnt = (int)k0 + (int)k1 + (int)k2;
    const double inv = cnt == 1 ? 1.0 : (cnt == 2 ? 0.5 : 1.0 / 3.0);
    R s0 = R(0.0), s1 = R(0.0), s2 = R(0.0);
    if (k0) {
      s0 += (23.0 * c + 2.0 * b - a) * (1.0 / 24.0);
      s1 += (3.0 * c - 4.0 * b + a) * 0.5;
      s2 += (c - 2.0 * b + a) * 0.5;
    }
    if (k1) {
      s0 += (26.0 * c - d - b) * (1.0 / 24.0);
      s1 += (d - b) * 0.5;
      s2 += (d + b - 2.0 * c) * 0.5;
    }
    if (k2) {
      s0 += (23.0 * c + 2.0 * d - e) * (1.0 / 24.0);
      s1 += (4.0 * d - 3.0 * c - e) * 0.5;
      s2 += (c - 2.0 * d + e) * 0.5;
    }
    c0 = s0 * inv;
    c1 = s1 * inv;
    c2 = s2 * inv;
  }
  const double ss = s * s;
  const R even = c0 + ss * (c2 + ss * c4);  // even part of p at +-s
  const R odd = s * (c1 + ss * c3);
  val[0] = even - odd;
  val[1] = even + odd;
  const R deven = c1 + (3.0 * ss) * c3;  // even part of p' at +-s
  const R dodd = s * (2.0 * c2 + (4.0 * ss) * c4);
  der[0] = deven - dodd;
  der[1] = deven + dodd;
}

}  // namespace tgks
