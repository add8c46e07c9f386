// mg_eval.h -- terms of an evaluation that both evaluation layouts share:
// pose, joint-limit and smoothness terms, swept-collision traces.
#pragma once

#include "mg_device.h"

namespace mg {
namespace {

// Pose reaching cost (Eq.(14)) of end effector ee whose link pose is T
// (3x4): position term a0 logcosh(a2 |p_g - p|), rotation term
// a1 logcosh(a3 |q_g - s q|) with s the sign of <q_g, q>.  The gradient
// enters as a wrench on the link: force d cost / d p at the tool point and
// the moment conjugate to a world-frame rotation.  pe_row >= 0 (and ee 0)
// records the position and angle errors of that row.
// etf: the tool transform (3x4), gl: the goal (position, quaternion w x y z).
__device__ __forceinline__ void pose_term_at(const EvalArgs& a, const float* etf, const float* gl, int ee,
                                             const float* T, int pe_row, float& cost, float& Fx, float& Fy,
                                             float& Fz, float& Mx, float& My, float& Mz) {
  float E[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) E[i] = T[i];
  compose(E, etf);
  float qw, qx, qy, qz;
  mat_to_quat(E, qw, qx, qy, qz);
  const float px = E[3], py = E[7], pz = E[11];
  const float ex = gl[0] - px, ey = gl[1] - py, ez = gl[2] - pz;
  const float n = sqrtf(ex * ex + ey * ey + ez * ez);
  cost += a.pr.a0 * logcosh_f(a.pr.a2 * n);
  const float fp = -a.pr.a0 * a.pr.a2 * tanh_over(a.pr.a2, n);
  const float gpx = fp * ex, gpy = fp * ey, gpz = fp * ez;     // d cost / d p
  const float dot = gl[3] * qw + gl[4] * qx + gl[5] * qy + gl[6] * qz;
  const float sg = dot >= 0.0f ? 1.0f : -1.0f;
  const float e0 = gl[3] - sg * qw, e1 = gl[4] - sg * qx;
  const float e2 = gl[5] - sg * qy, e3 = gl[6] - sg * qz;
  const float dr = sqrtf(e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3);
  cost += a.pr.a1 * logcosh_f(a.pr.a3 * dr);
  // d cost / d quaternion, then the moment conjugate to a world-frame
  // rotation omega: d quat = 1/2 (0, omega) (x) quat
  const float fq = -sg * a.pr.a1 * a.pr.a3 * tanh_over(a.pr.a3, dr);
  const float gw = fq * e0, gvx = fq * e1, gvy = fq * e2, gvz = fq * e3;
  const float tx = 0.5f * (qw * gvx - gw * qx + (qy * gvz - qz * gvy));
  const float ty = 0.5f * (qw * gvy - gw * qy + (qz * gvx - qx * gvz));
  const float tz = 0.5f * (qw * gvz - gw * qz + (qx * gvy - qy * gvx));
  Fx += gpx; Fy += gpy; Fz += gpz;
  Mx += py * gpz - pz * gpy + tx;
  My += pz * gpx - px * gpz + ty;
  Mz += px * gpy - py * gpx + tz;
  if (a.pe_e && pe_row >= 0 && ee == 0) {
    a.pe_e[(size_t)pe_row * 2 + 0] = n;
    a.pe_e[(size_t)pe_row * 2 + 1] = 2.0f * acosf(fminf(fabsf(dot), 1.0f));
  }
}

// Joint j at waypoint row `row` (waypoint t+1 of its seed): joint-limit cost
// (Eq.(17), weight w_bound, band eta2) and the smoothness terms of Eq.(16)
// whose five-point stencils (centred at t-1..t+3 on the padded trajectory:
// the start before waypoint 1, the last waypoint after T) touch this state.
// jc receives the terms this waypoint owns, js d cost / d q_j.  qj is the
// (candidate) value at row, qval(r, j) the value at another row; lo_, hi_
// are joint j's limits and q0 its start value.
template <typename QV>
__device__ __forceinline__ void joint_terms(const EvalArgs& a, const Problem& pb, int row, int t, int j,
                                            float qj, float lo_, float hi_, float q0, QV&& qval,
                                            float& jc, float& js) {
  const float e2 = a.pr.eta2, wb = a.pr.w_bound;
  const float inv_e2 = a.pr.inv_e2;
  float bc = 0.0f, bs = 0.0f;
  if (qj < lo_) { bc += lo_ - qj + 0.5f * e2; bs -= 1.0f; }
  else if (qj < lo_ + e2) { const float u = lo_ - qj + e2; bc += 0.5f * u * u * inv_e2; bs -= u * inv_e2; }
  if (qj > hi_) { bc += qj - hi_ + 0.5f * e2; bs += 1.0f; }
  else if (qj > hi_ - e2) { const float u = qj - hi_ + e2; bc += 0.5f * u * u * inv_e2; bs += u * inv_e2; }
  jc += wb * bc;
  js += wb * bs;
  if (pb.T <= 1) return;
  // padded states X(s), s = w-4..w+4 around this waypoint w = t+1
  const int w1 = t + 1, Tn = pb.T;
  float X[9];
#pragma unroll
  for (int u = 0; u < 9; ++u) {
    const int sgi = w1 - 4 + u;
    const int wv = sgi < 1 ? 1 : (sgi < Tn ? sgi : Tn);
    const float v = u == 4 ? qj : qval(row - t + wv - 1, j);
    X[u] = sgi <= 0 ? q0 : v;
  }
  const float cv = a.pr.cv, ca = a.pr.ca, cj = a.pr.cj;
  const float kv[5] = {1.0f, -8.0f, 0.0f, 8.0f, -1.0f};
  const float ka[5] = {-1.0f, 16.0f, -30.0f, 16.0f, -1.0f};
  const float kj[5] = {-1.0f, 2.0f, 0.0f, -2.0f, 1.0f};
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const int tau = w1 - 2 + c;          // stencil centre, states X[c..c+4]
    float v = 0.0f, ac = 0.0f, jk = 0.0f;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      v = fmaf(kv[i], X[c + i], v);
      ac = fmaf(ka[i], X[c + i], ac);
      jk = fmaf(kj[i], X[c + i], jk);
    }
    v *= cv; ac *= ca; jk *= cj;
    const bool in = tau >= 0 && tau <= Tn;
    const bool mine = in && (tau == w1 || (tau == 0 && w1 == 1));   // cost owner
    const bool vel = in && (a.pr.vel_all || tau == Tn);
    float gv = 0.0f;
    if (vel) {   // transcendentals only where the velocity term applies
      gv = a.pr.a6 * a.pr.a7 * tanhf(a.pr.a7 * v) * cv;
      if (mine) jc += a.pr.a6 * logcosh_f(a.pr.a7 * v);
    }
    if (mine) jc += a.pr.a8 * ac * ac + a.pr.a9 * jk * jk;
    const float ga = 2.0f * a.pr.a8 * ac * ca, gjk = 2.0f * a.pr.a9 * jk * cj;
    // stencil entry i touches padded state tau - 2 + i; this waypoint's
    // state is entry 4 - c alone, or, for the last waypoint, every entry
    // from 4 - c on (the padding after it repeats it)
    float wv = 0.0f, wa = 0.0f, wj = 0.0f;
#pragma unroll
    for (int i = 4 - c; i < 5; ++i) { wv += kv[i]; wa += ka[i]; wj += kj[i]; }
    const bool last = w1 == Tn;
    const float ev = last ? wv : kv[4 - c], ea = last ? wa : ka[4 - c], ej = last ? wj : kj[4 - c];
    js += in ? gv * ev + ga * ea + gjk * ej : 0.0f;
  }
}

// Continuous collision of one sphere against one cuboid (Alg.11-12 sphere
// tracing): from the centre c toward the neighbouring waypoint's centre,
// step by the clearance (by r + eta inside the band) while short of the
// half-way point, at most sweep_steps samples per side, each costed with the
// Eq.(10) profile.  (px, py, pz) is c in the box frame, sdf its distance.
// ls: the sphere in its link's frame; Tp, Tn: the link's poses at the
// neighbouring waypoints.  The samples' gradients stay in the box frame
// (added to b; the caller rotates the pair's sum back to the world once).
__device__ __forceinline__ void sweep_pair_box(const float4 ls, int steps, const float* Tp, const float* Tn,
                                               bool has_next, float cx, float cy, float cz, const v4f& A0,
                                               const v4f& A1, const v4f& A2, const v4f& Hh, float px, float py,
                                               float pz, float sdf, float r, float w, float eta, float inv_eta,
                                               float& cost, float& bx, float& by, float& bz) {
  const float rh = r + eta;
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const float* Tb = side == 0 ? Tp : Tn;
    if (side == 1 && !has_next) break;
    float ux = Tb[0] * ls.x + Tb[1] * ls.y + Tb[2] * ls.z + Tb[3] - cx;
    float uy = Tb[4] * ls.x + Tb[5] * ls.y + Tb[6] * ls.z + Tb[7] - cy;
    float uz = Tb[8] * ls.x + Tb[9] * ls.y + Tb[10] * ls.z + Tb[11] - cz;
    const float len = sqrtf(ux * ux + uy * uy + uz * uz);
    if (!(len > 0.0f)) continue;
    const float il = 1.0f / len;
    ux *= il; uy *= il; uz *= il;
    const float vx = A0.x * ux + A0.y * uy + A0.z * uz;
    const float vy = A1.x * ux + A1.y * uy + A1.z * uz;
    const float vz = A2.x * ux + A2.y * uy + A2.z * uz;
    const float half = 0.5f * len;
    float j = sdf < rh ? rh : sdf - rh;
    for (int st = 0; st < steps && j < half; ++st) {
      const float qx = fmaf(j, vx, px), qy = fmaf(j, vy, py), qz = fmaf(j, vz, pz);
      float gpx, gpy, gpz;
      const float s2 = box_sdf(qx, qy, qz, fabsf(qx) - Hh.x, fabsf(qy) - Hh.y, fabsf(qz) - Hh.z,
                               gpx, gpy, gpz);
      dc_term_box(s2, gpx, gpy, gpz, r, w, eta, inv_eta, cost, bx, by, bz);
      j += s2 - rh > 0.0f ? s2 - rh : rh;
    }
  }
}

// sweep_pair_box for cost-only evaluations: the trace samples' costs alone.
__device__ __forceinline__ void sweep_pair_cost(const float4 ls, int steps, const float* Tp, const float* Tn,
                                                bool has_next, float cx, float cy, float cz, const v4f& A0,
                                                const v4f& A1, const v4f& A2, const v4f& Hh, float px, float py,
                                                float pz, float sdf, float r, float w, float eta, float inv_eta,
                                                float& cost) {
  const float rh = r + eta;
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const float* Tb = side == 0 ? Tp : Tn;
    if (side == 1 && !has_next) break;
    float ux = Tb[0] * ls.x + Tb[1] * ls.y + Tb[2] * ls.z + Tb[3] - cx;
    float uy = Tb[4] * ls.x + Tb[5] * ls.y + Tb[6] * ls.z + Tb[7] - cy;
    float uz = Tb[8] * ls.x + Tb[9] * ls.y + Tb[10] * ls.z + Tb[11] - cz;
    const float len = sqrtf(ux * ux + uy * uy + uz * uz);
    if (!(len > 0.0f)) continue;
    const float il = 1.0f / len;
    ux *= il; uy *= il; uz *= il;
    const float vx = A0.x * ux + A0.y * uy + A0.z * uz;
    const float vy = A1.x * ux + A1.y * uy + A1.z * uz;
    const float vz = A2.x * ux + A2.y * uy + A2.z * uz;
    const float half = 0.5f * len;
    float j = sdf < rh ? rh : sdf - rh;
    for (int st = 0; st < steps && j < half; ++st) {
      const float qx = fmaf(j, vx, px), qy = fmaf(j, vy, py), qz = fmaf(j, vz, pz);
      const float s2 = box_dist(fabsf(qx) - Hh.x, fabsf(qy) - Hh.y, fabsf(qz) - Hh.z);
      dc_cost(s2, r, w, eta, inv_eta, cost);
      j += s2 - rh > 0.0f ? s2 - rh : rh;
    }
  }
}

}  // namespace
}  // namespace mg
