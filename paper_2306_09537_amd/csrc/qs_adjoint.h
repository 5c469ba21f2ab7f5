// Reverse-mode derivative of one quad's substep (everything before the
// in-env pair pass), float32.  Events take the derivative of the branch the
// forward pass took (recorded in Rec); the resting flag carries none.
#pragma once
#include "qs_device.h"

namespace qs {

// Adjoint of the per-quad state (same fields as Quad, resting flag omitted).
struct Adj {
  float x[3], v[3], R[9], w[3], u[4], e[4];
};

__device__ __forceinline__ void cross3f(const float a[3], const float b[3], float o[3]) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ __forceinline__ float dot3f(const float a[3], const float b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// What the adjoint needs of the parameters beside QuadPar.
struct ParAdj {
  float m, t2w;
  float dlag_dtau;  // d a_lag / d tau = -(1 - a_lag) dt / tau^2
};

// The derivative of a substep in three parts, each the reverse of one part of
// the substep and each with its share of the adjoint: the translation's
// depends on nothing but its own share, the rotation's takes the translation's
// dL/dF, the motor's both others' results.  (One wavefront runs them one after
// the other, or three one substep apart.)

// Translation: x, v.  l.x, l.v: dL/d(after the floor step) on entry,
// dL/d(start of the substep) on exit (the start position receives the end
// position's adjoint unchanged).  lF = dL/dF, F the world-frame thrust;
// returns dL/dm through the acceleration and the friction.
__device__ __forceinline__ float vjp_trans(const Consts& c, const QuadPar& p, uint32_t ev,
                                           const float F[3], const float v0[3], float lx[3],
                                           float lv[3], float lF[3]) {
  const float dt = c.dt;
  // floor hit: z and v were set to constants
  if (ev & SUB_HIT) {
    lx[2] = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) lv[k] = 0.f;
  }
  // walls: decay once, then per-axis mirror and clamp (selects: rare events
  // must not split the scheduling region)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lv[k] = (ev & SUB_BOUNCED) ? lv[k] * c.col_decay : lv[k];
    lv[k] = (ev & SUB_FLIP << k) ? lv[k] * -c.e_wall : lv[k];
    lx[k] = (ev & SUB_CLAMP << k) ? 0.f : lx[k];
  }
  float lm = 0.f, lv0[3];
  // free flight for every lane; a resting lane (rare) redoes this part below
  // x1 = x0 + dt v1, v1 = v0 + dt acc, acc = F/m - c_d v0/m - g e_z
  const float dm = c.drag * p.inv_m;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float lv1 = fmaf(dt, lx[k], lv[k]);
    const float lacc = dt * lv1;
    lv0[k] = fmaf(-dm, lacc, lv1);
    lF[k] = lacc * p.inv_m;
    lm -= (F[k] - c.drag * v0[k]) * lacc * p.inv_m * p.inv_m;
  }
  if (ev & SUB_REST) {
    // resting: v_z zeroed, x_z unchanged
    const Friction f = floor_friction(c, p, F, v0);
    lm = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) lF[k] = lv0[k] = 0.f;
    if (!(ev & SUB_GUARD)) {
      const float lv1[2] = {fmaf(dt, lx[0], lv[0]), fmaf(dt, lx[1], lv[1])};
      const float lfb[2] = {dt * lv1[0] * p.inv_m, dt * lv1[1] * p.inv_m};
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        lv0[k] = lv1[k] * (1.0f - dt * c.drag * p.inv_m);
        lm -= dt * (f.fb[k] - c.drag * v0[k]) * lv1[k] * p.inv_m * p.inv_m;
      }
      float lmu = 0.f;
      if (f.still) {
        if (f.mag > 0.f) {
          const float fx = F[0] / f.nf, fy = F[1] / f.nf;
          const float dd = lfb[0] * fx + lfb[1] * fy;
          lF[0] += lfb[0] - f.mu_n * (lfb[0] - dd * fx) / f.nf;
          lF[1] += lfb[1] - f.mu_n * (lfb[1] - dd * fy) / f.nf;
          lmu = -dd;
        }
      } else {
        const float vx = v0[0] / f.nv, vy = v0[1] / f.nv;
        lF[0] += lfb[0];
        lF[1] += lfb[1];
        lmu = -(lfb[0] * vx + lfb[1] * vy);
        const float lvx = -f.mu_n * lfb[0], lvy = -f.mu_n * lfb[1];
        const float dd = lvx * vx + lvy * vy;
        lv0[0] += (lvx - dd * vx) / f.nv;
        lv0[1] += (lvy - dd * vy) / f.nv;
      }
      // mu_n = mu (m g - F_z)
      lm += c.mu * c.g * lmu;
      lF[2] -= c.mu * lmu;
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) lv[k] = lv0[k];
  return lm;
}

// Rotation: R, w.  Takes lF; lt = dL/d(torques), lJ = dL/d(inertia); returns
// dL/dT, T the thrust along body z.
__device__ __forceinline__ float vjp_rot(const Consts& c, const QuadPar& p, const Rec& r,
                                         uint32_t ev, const float lF[3], float lR[9], float lw[3],
                                         float lt[3], float lJ[3]) {
  const float dt = c.dt;
  // floor hit: omega was set to zero, R levelled from its heading
  if (ev & SUB_HIT) {
#pragma unroll
    for (int k = 0; k < 3; ++k) lw[k] = 0.f;
    const bool held = (ev & SUB_REST) != 0u;
    const Heading h = floor_heading(held ? r.P[0] : r.c0[0], held ? r.P[1] : r.c1[0],
                                    held ? r.P[3] : r.c0[1], held ? r.P[4] : r.c1[1]);
    float g0 = 0.f, g1 = 0.f, g3 = 0.f, g4 = 0.f;
    if (!h.fallback) {
      // column 0 = h = (hx, hy)/nh, column 1 = (-h_y, h_x)
      const float hx = h.hx / h.nh, hy = h.hy / h.nh;
      const float ghx = lR[0] + lR[4], ghy = lR[3] - lR[1];
      const float dd = ghx * hx + ghy * hy;
      g0 = (ghx - dd * hx) / h.nh;
      g3 = (ghy - dd * hy) / h.nh;
    } else if (h.nk > 0.f) {
      // column 1 = k = (kx, ky)/nk, column 0 = (k_y, -k_x)
      const float kx = h.kx / h.nk, ky = h.ky / h.nk;
      const float gkx = lR[1] - lR[3], gky = lR[4] + lR[0];
      const float dd = gkx * kx + gky * ky;
      g1 = (gkx - dd * kx) / h.nk;
      g4 = (gky - dd * ky) / h.nk;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) lR[k] = 0.f;
    lR[0] = g0;
    lR[1] = g1;
    lR[3] = g3;
    lR[4] = g4;
  }
  float lP[9], lw0[3];
  const float J[3] = {p.jx, p.jy, p.jz};
  // free flight for every lane; a resting lane (rare) redoes this part below
  {
    // R = Gram-Schmidt(A): c2 = c0 x c1, c1 = b/|b|, b = A1 - (c0.A1) c0, c0 = A0/|A0|
    float lc0[3] = {lR[0], lR[3], lR[6]}, lc1[3] = {lR[1], lR[4], lR[7]};
    const float lc2[3] = {lR[2], lR[5], lR[8]};
    float tmp[3];
    cross3f(r.c1, lc2, tmp);
#pragma unroll
    for (int k = 0; k < 3; ++k) lc0[k] += tmp[k];
    cross3f(lc2, r.c0, tmp);
#pragma unroll
    for (int k = 0; k < 3; ++k) lc1[k] += tmp[k];
    float dd = dot3f(lc1, r.c1);
    float lb[3];
    const float in1 = r.i1;
#pragma unroll
    for (int k = 0; k < 3; ++k) lb[k] = (lc1[k] - dd * r.c1[k]) * in1;
    const float ldp = -dot3f(lb, r.c0);
    float lA1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lA1[k] = fmaf(ldp, r.c0[k], lb[k]);
      lc0[k] += fmaf(-r.dp, lb[k], ldp * r.A1[k]);
    }
    dd = dot3f(lc0, r.c0);
    float lA0[3];
    const float in0 = r.i0;
#pragma unroll
    for (int k = 0; k < 3; ++k) lA0[k] = (lc0[k] - dd * r.c0[k]) * in0;
    // A0 = P0 + dt (P1 w1z - P2 w1y), A1 = P1 + dt (P2 w1x - P0 w1z) (columns)
    const float P0[3] = {r.P[0], r.P[3], r.P[6]}, P1[3] = {r.P[1], r.P[4], r.P[7]},
                P2[3] = {r.P[2], r.P[5], r.P[8]};
    const float lw1[3] = {fmaf(dt, dot3f(P2, lA1), lw[0]), fmaf(-dt, dot3f(P2, lA0), lw[1]),
                          fmaf(dt, dot3f(P1, lA0) - dot3f(P0, lA1), lw[2])};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lP[3 * k + 0] = fmaf(-dt * r.w1[2], lA1[k], lA0[k]);
      lP[3 * k + 1] = fmaf(dt * r.w1[2], lA0[k], lA1[k]);
      lP[3 * k + 2] = dt * (r.w1[0] * lA1[k] - r.w1[1] * lA0[k]);
    }
    // w1 = w0 + dt wdot, wdot_k = (tau_k - (w0 x J w0)_k) / J_k
    float lc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lw0[k] = lw1[k];
      const float lwd = dt * lw1[k];
      const float iJ = k == 0 ? p.ijx : (k == 1 ? p.ijy : p.ijz);
      lt[k] = lwd * iJ;
      lc[k] = -lwd * iJ;
      lJ[k] = -lwd * r.wdot[k] * iJ;
    }
    const float Jw[3] = {J[0] * r.w0[0], J[1] * r.w0[1], J[2] * r.w0[2]};
    cross3f(Jw, lc, tmp);
    float lJw[3];
    cross3f(lc, r.w0, lJw);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lw0[k] += tmp[k] + J[k] * lJw[k];
      lJ[k] += r.w0[k] * lJw[k];
    }
  }
  if (ev & SUB_REST) {
    // resting: R held, omega zeroed
#pragma unroll
    for (int k = 0; k < 3; ++k) lt[k] = lJ[k] = lw0[k] = 0.f;
#pragma unroll
    for (int k = 0; k < 9; ++k) lP[k] = lR[k];
  }
  // F = T * (third column of R)
  const float lT = lF[0] * r.P[2] + lF[1] * r.P[5] + lF[2] * r.P[8];
  lP[2] = fmaf(r.T, lF[0], lP[2]);
  lP[5] = fmaf(r.T, lF[1], lP[5]);
  lP[8] = fmaf(r.T, lF[2], lP[8]);
#pragma unroll
  for (int k = 0; k < 9; ++k) lR[k] = lP[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) lw[k] = lw0[k];
  return lT;
}

// Motor: u, eps.  Takes dL/dT, dL/d(torques) and the translation's lm;
// gu += dL/d(rotor-speed command uhat); gm, gt2w, gtau +=
// dL/d(mass, thrust-to-weight, motor time constant).
__device__ __forceinline__ void vjp_motor(const Consts& c, const QuadPar& p, const ParAdj& pa,
                                          const float u0[4], const float u1[4], const float z[4],
                                          const float uhat[4], float lT, const float lt[3],
                                          float lm, float lu[4], float le[4], float gu[4],
                                          float& gm, float& gt2w, float& gtau) {
  // thrust and torques from the rotor thrusts (X layout FR, BR, BL, FL)
  const float sx[4] = {-1.f, -1.f, 1.f, 1.f}, sy[4] = {-1.f, 1.f, 1.f, -1.f},
              sz[4] = {1.f, -1.f, 1.f, -1.f};
  float lfmax = 0.f, lalag = 0.f;
  const bool noise = (c.flags & F_NOISE) != 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lf = lT + c.arm_d * (sx[i] * lt[0] + sy[i] * lt[1]) + c.k_tau * sz[i] * lt[2];
    const float lu1 = fmaf(2.0f * p.f_max * u1[i], lf, lu[i]);
    const float le1 = le[i] + lf;
    lfmax = fmaf(u1[i] * u1[i], lf, lfmax);
    // motor noise e1 = a_nd e0 + ns_scale f_max z
    le[i] = noise ? c.a_nd * le1 : le1;
    lfmax = noise ? fmaf(c.ns_scale * z[i], le1, lfmax) : lfmax;
    // motor lag u1 = u0 + a_lag (uhat - u0)
    lu[i] = (1.0f - p.a_lag) * lu1;
    gu[i] = fmaf(p.a_lag, lu1, gu[i]);
    lalag = fmaf(uhat[i] - u0[i], lu1, lalag);
  }
  // f_max = m g t2w / 4, a_lag = 1 - exp(-dt/tau)
  lm += 0.25f * c.g * pa.t2w * lfmax;
  gm += lm;
  gt2w += 0.25f * pa.m * c.g * lfmax;
  gtau = fmaf(lalag, pa.dlag_dtau, gtau);
}

// All three.  l: dL/d(state after the floor step) on entry, dL/d(state at the
// start of the substep) on exit.  gp += dL/d(m, jx, jy, jz, t2w, tau).
__device__ __forceinline__ void quad_vjp(const Consts& c, const QuadPar& p, const ParAdj& pa,
                                         const Rec& r, const float uhat[4], Adj& l,
                                         float gu[4], float gp[6]) {
  const float F[3] = {r.T * r.P[2], r.T * r.P[5], r.T * r.P[8]};
  float lF[3], lt[3], lJ[3];
  const float lm = vjp_trans(c, p, r.ev, F, r.v0, l.x, l.v, lF);
  const float lT = vjp_rot(c, p, r, r.ev, lF, l.R, l.w, lt, lJ);
  vjp_motor(c, p, pa, r.u0, r.u1, r.z, uhat, lT, lt, lm, l.u, l.e, gu, gp[0], gp[4], gp[5]);
#pragma unroll
  for (int k = 0; k < 3; ++k) gp[1 + k] += lJ[k];
}

}  // namespace qs
