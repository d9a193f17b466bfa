// Per-sample arithmetic of the core rollout (rollout_core.hpp) and its output split:
// the same steps as sample_step.hpp's, with every product-sum an explicit fused
// multiply-add, so that the rounding does not depend on the kernel a function is
// inlined into (the layouts of the core must agree bit for bit).
#pragma once
#include "sample_step.hpp"

namespace gpmppi {
namespace core {

// Tightened distance to one obstacle (Eqs. 14, 16): the centre distance rho
// less the radius, less z_p times the position deviation along the centre
// direction n = (dx, dy) / rho, n^T Sigma n = (sa dx^2 + 2 sb dx dy + sc dy^2) / rho^2;
// at rho = 0 the direction is undefined and the largest eigenvalue stands in.
// One reciprocal square root gives both rho and 1 / rho^2.
__device__ __forceinline__ float obstacle_distance(float dx, float dy, float radius, float sa, float sb, float sc,
                                                 float lmax, float z_p) {
    const float rho2 = fmaf(dy, dy, dx * dx);
    const bool pos = rho2 > 0.0f;
    const float rs = __builtin_amdgcn_rsqf(rho2);
    const float rho = pos ? rho2 * rs : 0.0f;
    const float quad = fmaf(sc * dy, dy, fmaf(2.0f * sb * dx, dy, sa * dx * dx));
    const float vn = pos ? quad * (rs * rs) : lmax;
    return fmaf(-z_p, __builtin_amdgcn_sqrtf(fmaxf(vn, 0.0f)), rho - radius);
}

// Squared distance of (X, Y) to the polyline segment s = (ax, ay, ex, ey), inv = 1 / |e|^2.
__device__ __forceinline__ float segment_dist2(v4f s, float inv, float X, float Y) {
    const float rx = X - s.x, ry = Y - s.y;
    const float t = fminf(fmaxf(fmaf(ry, s.w, rx * s.z) * inv, 0.0f), 1.0f);
    const float ex = fmaf(-t, s.z, rx), ey = fmaf(-t, s.w, ry);
    return fmaf(ey, ey, ex * ex);
}

// Largest eigenvalue of the position covariance [[sa, sb], [sb, sc]].
__device__ __forceinline__ float lambda_max(float sa, float sb, float sc) {
    const float hh = 0.5f * (sa - sc);
    return fmaf(0.5f, sa + sc, sqrtf(fmaf(sb, sb, hh * hh)));
}

// Velocities after one explicit Euler step of the dynamic unicycle plus the GP
// residual means m0, m1 (Eqs. 1, 2, 10).
__device__ __forceinline__ void step_velocities(const Dyn &dy, float2 u, float m0, float m1, float &v, float &w) {
    const float v_old = v, w_old = w;
    v = v_old + fmaf(dy.dt, m0, dy.dt_tau_v * (u.x - v_old));
    w = w_old + fmaf(dy.dt, m1, dy.dt_tau_w * (u.y - w_old));
}

// The parts of a step's StageIn that need no loop over the world (dl on a circle
// track, 0 on a polyline; om left +inf).
__device__ __forceinline__ StageIn stage_geometry(const Geometry &geo, const CostWeights &cw, float X, float Y, float v,
                                                  float lmax, float &dgoal_min) {
    StageIn t;
    t.dl = 0.0f;
    if (geo.path_kind == 0) {
        const float dx = X - geo.cx, dyy = Y - geo.cy;
        t.dl = fabsf(sqrtf(fmaf(dyy, dyy, dx * dx)) - geo.R);
    }
    t.rbar = fmaf(-geo.c_p, sqrtf(fmaxf(lmax, 0.0f)), geo.half_width);
    t.om = INFINITY;
    t.dv = cw.v_des - v;
    t.dg = 0.0f;
    if (cw.w_goal != 0.0f || cw.w_term != 0.0f) {   // goal terms (Eq. 12)
        const float gx = X - cw.goal_x, gy = Y - cw.goal_y;
        t.dg = sqrtf(fmaf(gy, gy, gx * gx));
        dgoal_min = fminf(dgoal_min, t.dg);
    }
    return t;
}

// Stage cost (Eqs. 11-12 terms) added to the Kahan-compensated sum (S, Sc) of
// Eq. (5); the lane term is discounted by disc, which then advances.
__device__ __forceinline__ void core_stage_cost(const CostWeights &cw, const Geometry &geo, const StageIn &t, float s2a,
                                               float s2b, float &disc, float &S, float &Sc) {
    float c = fmaf(cw.w_speed, t.dv * t.dv, fmaf(cw.w_dev, t.dl * geo.inv_half_width, cw.w_var * (s2a + s2b)));
    if (t.dl > t.rbar) c = fmaf(cw.w_lane, disc, c);
    if (t.om <= 0.0f) c += cw.w_obs;
    if (cw.w_goal != 0.0f || cw.w_term != 0.0f) c = fmaf(cw.w_goal, t.dg, c);
    const float yk = c - Sc;
    const float tk = S + yk;
    Sc = (tk - S) - yk;
    S = tk;
    disc *= cw.discount;
}

// Per-step trace rows of sample sg (K samples): the state, position covariance,
// means and control of step k ...
__device__ __forceinline__ void write_step(const gpmppi_trace &tr, int K, int sg, int k, float X, float Y, float th,
                                           float v, float w, const Cov &P, float m0, float m1, float2 u) {
    const size_t kk = (size_t)k;
    if (tr.x_d) {
        float *xd = tr.x_d + (kk + 1) * 5 * K;
        xd[0 * K + sg] = X;
        xd[1 * K + sg] = Y;
        xd[2 * K + sg] = th;
        xd[3 * K + sg] = v;
        xd[4 * K + sg] = w;
    }
    if (tr.sxy_d) {
        float *sd = tr.sxy_d + (kk + 1) * 3 * K;
        sd[0 * K + sg] = P.p00;
        sd[1 * K + sg] = P.p01;
        sd[2 * K + sg] = P.p11;
    }
    if (tr.gp_mean_d) {
        tr.gp_mean_d[(kk * 2 + 0) * K + sg] = m0;
        tr.gp_mean_d[(kk * 2 + 1) * K + sg] = m1;
    }
    if (tr.u_d) {
        tr.u_d[(kk * 2 + 0) * K + sg] = u.x;
        tr.u_d[(kk * 2 + 1) * K + sg] = u.y;
    }
}

// ... its variances, and its distances and margins, which come later.
__device__ __forceinline__ void write_variances(const gpmppi_trace &tr, int K, int sg, int k, float s20, float s21) {
    if (!tr.gp_var_d) return;
    tr.gp_var_d[((size_t)k * 2 + 0) * K + sg] = s20;
    tr.gp_var_d[((size_t)k * 2 + 1) * K + sg] = s21;
}
__device__ __forceinline__ void write_margins(const gpmppi_trace &tr, int K, int sg, int k, const StageIn &t) {
    const size_t kk = (size_t)k;
    if (tr.d_lane_d) tr.d_lane_d[kk * K + sg] = t.dl;
    if (tr.lane_margin_d) tr.lane_margin_d[kk * K + sg] = t.rbar - t.dl;
    if (tr.obs_margin_d) tr.obs_margin_d[kk * K + sg] = t.om;
}

}  // namespace core
}  // namespace gpmppi
