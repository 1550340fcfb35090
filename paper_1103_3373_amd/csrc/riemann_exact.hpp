// Exact Riemann solver for the ideal-gas Euler equations (arXiv:1103.3373,
// Sec. 2 lists it among the solvers: reference solutions and a fallback),
// following the standard construction in Toro, "Riemann Solvers and
// Numerical Methods for Fluid Dynamics", ch. 4:
//  * the star pressure p* is the root of f_L(p) + f_R(p) + (u_R - u_L) = 0,
//    where f_K is the shock (Rankine-Hugoniot) branch for p > p_K and the
//    rarefaction (isentropic) branch otherwise;
//  * Newton iteration from the primitive-variable (PVRS) estimate, bounded
//    below by 1e-8 min(p_L, p_R), until the relative change
//    2 |p_new - p| / (p_new + p) falls below 1e-15 (FP64) or 1e-6 (FP32),
//    at most 200 iterations;
//  * the flux is the physical flux of the self-similar solution sampled on
//    the face (x/t = 0).
// States are in the rotated frame (rho, u_n, u_t1, u_t2, p).  A pair that
// generates vacuum ((2/(gamma-1))(c_L + c_R) <= u_R - u_L) or does not
// converge is counted in *fails and sampled with p* = 0 (vacuum) or the
// last iterate.
#pragma once

#include "hydro_math.hpp"

namespace hy {

template <typename T> HY_DEV T xpow(T a, T b);
template <> HY_DEV double xpow<double>(double a, double b) { return pow(a, b); }
template <> HY_DEV float xpow<float>(float a, float b) { return powf(a, b); }

// f_K(p) and its derivative.  The derivative on the rarefaction branch takes a
// power of its own: from the other, as t / (pr rho_K c_K), it would be 0 / 0
// where the pressure underflows next to vacuum, and its other rounding changes
// which solves stop within the tolerance.  (g1 and g2: the two powers.)
template <typename T>
HY_DEV void exact_pfun(T p, T rk, T pk, T ck, T gm1, T gp1, T g1, T g2, T& f, T& df) {
  if (p > pk) {  // shock
    const T A = T(2) / (gp1 * rk);
    const T B = gm1 / gp1 * pk;
    const T q = sqrt(A / (p + B));
    f = (p - pk) * q;
    df = q * (T(1) - T(0.5) * (p - pk) / (B + p));
  } else {  // rarefaction
    const T pr = p / pk;
    f = T(2) * ck / gm1 * (xpow<T>(pr, g1) - T(1));
    df = T(1) / (rk * ck) * xpow<T>(pr, g2);
  }
}

// The sampled state's flux and 1 if the pair generates vacuum or the iteration
// does not converge.  Not inlined: the Newton iteration dwarfs a call, and the
// fused kernels solve at up to four places.
template <typename T> struct ExactFlux {
  V5<T> F;
  int fail;
};
template <typename T>
__device__ __attribute__((noinline)) ExactFlux<T> exact_solve(V5<T> L, V5<T> R, T gamma, T gm1, T inv_gm1) {
  Phys<T> ph{};
  ph.gamma = gamma;
  ph.gm1 = gm1;
  ph.inv_gm1 = inv_gm1;
  const T gp1 = gamma + T(1), g1 = gm1 / (T(2) * gamma), g2 = -gp1 / (T(2) * gamma);
  const T cL = sqrt(gamma * L[4] / L[0]), cR = sqrt(gamma * R[4] / R[0]);
  const T du = R[1] - L[1];
  ExactFlux<T> r;
  r.fail = 0;
  T p, u;
  const bool vacuum = T(2) / gm1 * (cL + cR) <= du;
  if (vacuum) {
    r.fail = 1;
    p = T(0);
    u = T(0.5) * (L[1] + R[1]);
  } else {
    const T ppv = T(0.5) * (L[4] + R[4]) - T(0.125) * du * (L[0] + R[0]) * (cL + cR);
    p = fmax(ppv, T(1e-8) * fmin(L[4], R[4]));
    const T tol = sizeof(T) == 8 ? T(1e-15) : T(1e-6);
    T fL, dL, fR, dR;
    int it = 0;
    for (; it < 200; ++it) {
      exact_pfun(p, L[0], L[4], cL, gm1, gp1, g1, g2, fL, dL);
      exact_pfun(p, R[0], R[4], cR, gm1, gp1, g1, g2, fR, dR);
      T pn = p - (fL + fR + du) / (dL + dR);
      if (pn < T(0)) pn = T(1e-12) * p;
      const T ch = T(2) * fabs(pn - p) / (pn + p);
      p = pn;
      if (ch < tol) break;
    }
    if (it >= 200) r.fail = 1;
    exact_pfun(p, L[0], L[4], cL, gm1, gp1, g1, g2, fL, dL);
    exact_pfun(p, R[0], R[4], cR, gm1, gp1, g1, g2, fR, dR);
    u = T(0.5) * (L[1] + R[1]) + T(0.5) * (fR - fL);
  }
  // Sample the solution on the face, x/t = 0: on the side K of the contact,
  // with velocities counted away from the wave (mirrored for the right side),
  // so that both sides are the left one.
  const bool left = T(0) <= u;
  const T sg = left ? T(1) : T(-1);
  V5<T> W = left ? L : R;
  const T c = left ? cL : cR, v = sg * W[1], us = sg * u, pk = W[4], pr = p / pk, g6 = gm1 / gp1;
  if (p > pk) {  // shock
    const T S = v - c * sqrt(gp1 / (T(2) * gamma) * p / pk + g1);
    if (!(T(0) <= S)) {
      W[0] = W[0] * (pr + g6) / (g6 * p / pk + T(1));
      W[1] = u;
      W[4] = p;
    }
  } else if (!(T(0) <= v - c)) {  // rarefaction with its head past the face
    const T cs = c * xpow<T>(pr, g1);
    if (T(0) > us - cs) {
      W[0] = vacuum ? T(0) : W[0] * xpow<T>(pr, T(1) / gamma);
      W[1] = u;
      W[4] = p;
    } else {  // inside the fan
      const T b = T(2) / gp1 + gm1 / (gp1 * c) * v;
      W[0] = W[0] * xpow<T>(b, T(2) / gm1);
      W[1] = sg * (T(2) / gp1 * (c + T(0.5) * gm1 * v));
      W[4] = pk * xpow<T>(b, T(2) * gamma / gm1);
    }
  }
  r.F = flux_of(W, ph);
  return r;
}

template <typename T>
HY_DEV V5<T> exact_flux(const V5<T>& L, const V5<T>& R, const Phys<T>& ph, int* fails) {
  const ExactFlux<T> r = exact_solve(L, R, ph.gamma, ph.gm1, ph.inv_gm1);
  *fails += r.fail;
  return r.F;
}

}  // namespace hy
