// Adjoints of the per-item physics with rotation cotangents as vectors
// (device code), for the fused adjoint kernels.
//
// An item reads a body's orientation only through its rotation R (vectors R l
// and inertia tensors R D R^T), and every orientation of a trajectory but the
// first is normalised by the kinematic update, whose adjoint drops the part of
// an orientation cotangent along the quaternion itself. So what matters of it
// is how it acts on a small rotation of the body by the world vector d: one
// vector t with (cotangent) . d(q) = t . d. It replaces the nine cotangents of
// R, the six of the inverse inertia and their conversion to the quaternion's
// four:
//   a = R l with cotangent ab:        t += a x ab
//   y = (R D R^T) v, cotangent yb:    t += y x yb + ((R D R^T) yb) x v
// A quaternion cotangent is formed once, for the state before the first step.
// Kinks follow the branch the forward takes (see bx_adj.h).
#pragma once
#include "bx_access.h"
#include "bx_adj.h"

namespace bx {

// Cotangent of one body's state, its orientation's as the vector t.
struct TBar {
  v3 p, t, v, w;
};
__device__ __forceinline__ TBar tbar_zero() {
  const v3 z = V(0.f, 0.f, 0.f);
  return TBar{z, z, z, z};
}
__device__ __forceinline__ void tbar_add(TBar& a, const TBar& b) {
  a.p += b.p;
  a.t += b.t;
  a.v += b.v;
  a.w += b.w;
}
__device__ __forceinline__ void tbar_put(float4* r, const TBar& a) {
  r[0] = make_float4(a.p.x, a.p.y, a.p.z, a.t.x);
  r[1] = make_float4(a.t.y, a.t.z, a.v.x, a.v.y);
  r[2] = make_float4(a.v.z, a.w.x, a.w.y, a.w.z);
}
__device__ __forceinline__ TBar tbar_get(const float4* r) {
  const float4 a = r[0], b = r[1], c = r[2];
  return TBar{V(a.x, a.y, a.z), V(a.w, b.x, b.y), V(b.z, b.w, c.x), V(c.y, c.z, c.w)};
}

// ------------------------------------------------------------ body
// What the integrators' adjoints need of a body in a substep, from its tape
// record: orientation before the kinematic update, state after it, total
// torque, applied contacts.
struct BodyTan {
  v3 w, e;             // angular velocity (frozen axes masked), h/2 times it
  v3 x, al, u;         // torque minus gyroscopic torque, Iwinv x, R I R^T w
  float k2, inv_n;     // 2 / (1 + e.e), 1 / contacts (0 without)
  m3 R;
  s3 Iwinv;
  q4 q1;               // orientation after the kinematic update
  float inv;           // 1 / norm of the update before normalisation
};
__device__ __forceinline__ BodyTan body_tan(const BodyT& B, q4 q0, const Body& post, v3 ttot, int n, float h) {
  BodyTan k;
  k.w = post.w;
  k.e = (0.5f * h) * k.w;
  const float ee = dot(k.e, k.e);
  k.k2 = 2.f * __builtin_amdgcn_rcpf(1.f + ee);
  k.q1 = post.q;
  // |(1, e) (x) q0| = |(1, e)| |q0|
  k.inv = __builtin_amdgcn_rsqf((1.f + ee) * (q0.w * q0.w + q0.x * q0.x + q0.y * q0.y + q0.z * q0.z));
  k.R = quat_to_mat(post.q);
  k.Iwinv = rot_diag(k.R, B.Iinv);
  const v3 wb = mul_t(k.R, k.w);
  k.u = mul(k.R, V(B.I[0] * wb.x, B.I[1] * wb.y, B.I[2] * wb.z));
  k.x = ttot - cross(k.w, k.u);
  k.al = mul(k.Iwinv, k.x);
  k.inv_n = n > 0 ? __builtin_amdgcn_rcpf((float)n) : 0.f;
  return k;
}
// Cotangents of a substep's force, torque, dv and dw sums from that of the
// state after it (G, its frozen velocity components masked).
__device__ __forceinline__ void body_head(const BodyT& B, const BodyTan& k, float h, const TBar& G, v3& fb, v3& tb,
                                          v3& dvb, v3& dwb) {
  fb = (h * B.inv_m) * G.v;
  tb = mul(k.Iwinv, h * G.w);
  dvb = k.inv_n * G.v;
  dwb = k.inv_n * G.w;
}
// Potential integrator: adds its cotangents of the post-kinematic state to tot.
__device__ __forceinline__ void potential_tan(const BodyT& B, const BodyTan& k, float h, v3 wbar, v3 tb, TBar& tot) {
  const v3 ab = h * wbar;
  tot.t += cross(k.al, ab) + cross(tb, k.x);
  // x = torque - w x u, u = R I R^T w
  const v3 ub = cross(k.w, tb);
  const v3 yb = mul_t(k.R, ub);
  const v3 iu = mul(k.R, V(B.I[0] * yb.x, B.I[1] * yb.y, B.I[2] * yb.z));
  tot.w += cross(tb, k.u) + iu;
  tot.t += cross(k.u, ub) + cross(iu, k.w);
}
// Kinematic integrator: the update rotates the orientation by the unit
// quaternion (1, e) / |(1, e)|.
__device__ __forceinline__ TBar kinematic_tan(const BodyT& B, bool frozen, const BodyTan& k, float h, const TBar& ob) {
  const v3 m = cross(k.e, ob.t);
  TBar r;
  r.p = ob.p;
  r.t = ob.t + k.k2 * (cross(k.e, m) - m);
  r.v = ob.v + h * ob.p;
  r.w = ob.w + (0.5f * h * k.k2) * (ob.t - m);
  if (frozen) {
    r.v = keep(r.v, B.free_p);
    r.w = keep(r.w, B.free_r);
  }
  return r;
}
// The cotangent of a quaternion as the vector of its rotation, and back: the
// quaternion cotangent of the state before the kinematic update.
__device__ __forceinline__ v3 quat_tan(q4 q, q4 qb) {
  const v3 qv = V(q.x, q.y, q.z), bv = V(qb.x, qb.y, qb.z);
  return 0.5f * ((q.w * bv - qb.w * qv) - cross(bv, qv));
}
__device__ __forceinline__ q4 kinematic_tan_quat(const BodyTan& k, float h, v3 t) {
  // of the normalised orientation: 2 (0, t) (x) q1, tangent to it
  const q4 g = qscale(2.f * k.inv, qmul(q4{0.f, t.x, t.y, t.z}, k.q1));
  // and through q0 + (0, e) (x) q0
  return qadd(g, qmul(q4{0.f, -k.e.x, -k.e.y, -k.e.z}, g));
}

// ------------------------------------------------------------ joint
// A joint's forward values its adjoint needs. t[k]: the gradient of Euler
// angle k with respect to a rotation of the parent (the child's is -t[k]); sc:
// the torque about axis k; lim, pd: minus the limit's and the target-angle
// drive's stiffness where they act.
template <int MAXDOF>
struct JointTan {
  v3 rP, rC, F, wP, wC;
  v3 e1P, e1C;
  v3 t[MAXDOF];
  float sc[MAXDOF], st[MAXDOF], gear[MAXDOF];
  float c11;                 // e1P . e1C
  v3 e2C, ax1, n1, e3C;      // further axes, e1P x ax1 (MAXDOF > 1)
  float m01;
};
template <int MAXDOF>
__device__ __forceinline__ void joint_tan_fwd(const JointT& J, const Body& P, const m3& RP, const Body& C, const m3& RC,
                                              const float* a, JointTan<MAXDOF>& k) {
  const JointChild c = joint_child<MAXDOF>(J, C, RC);
  const JointGeo g = joint_geo_step<MAXDOF>(J, RP, c);
  (void)joint_spring<MAXDOF>(J, P, C, g, c.uC, k.F);
  k.rP = g.rP;
  k.rC = g.rC;
  k.wP = P.w;
  k.wC = C.w;
  k.e1P = g.e1P;
  k.e1C = g.e1C;
  k.c11 = dot(g.e1P, g.e1C);
  const float r2 = g.m12 * g.m12 + g.m22 * g.m22;
  const float ir2 = r2 > 0.f ? __builtin_amdgcn_rcpf(r2) : 0.f;
  if (MAXDOF == 1) {
    const v3 f = V(g.m12 * J.FP[2] - g.m22 * J.FP[1], g.m12 * J.FP[5] - g.m22 * J.FP[4], g.m12 * J.FP[8] - g.m22 * J.FP[7]);
    k.t[0] = ir2 * cross(mul(RP, f), g.e3C);
  } else {
    k.t[0] = ir2 * cross(g.m12 * g.e3P - g.m22 * g.e2P, g.e3C);
    const float d1 = 1.f - g.m02 * g.m02;
    k.t[MAXDOF > 1 ? 1 : 0] = (d1 > 0.f ? __builtin_amdgcn_rsqf(d1) : 0.f) * cross(g.e1P, g.e3C);
    const float d3 = g.m00 * g.m00 + g.m01 * g.m01;
    k.t[MAXDOF > 2 ? 2 : 0] = (d3 > 0.f ? __builtin_amdgcn_rcpf(d3) : 0.f) * cross(g.e1P, g.m01 * g.e1C - g.m00 * g.e2C);
    k.e2C = g.e2C;
    k.e3C = g.e3C;
    k.ax1 = g.ax[1];
    k.n1 = cross(g.e1P, g.ax[1]);
    k.m01 = g.m01;
  }
  for (int i = 0; i < MAXDOF; ++i) {
    const bool on = MAXDOF == 1 || i < J.dof;
    const float cl = clampf(g.th[i], J.lo[i], J.hi[i]);
    const bool out = g.th[i] < J.lo[i] || g.th[i] > J.hi[i];
    k.gear[i] = on ? J.gear[i] : 0.f;
    k.sc[i] = on ? J.gear[i] * (a[i] - J.act_pd[i] * g.th[i]) - J.k_lim * (g.th[i] - cl) : 0.f;
    k.st[i] = on ? -(J.act_pd[i] * J.gear[i] + (out ? J.k_lim : 0.f)) : 0.f;
  }
}
// Given the cotangents of the child's (fc, tc) and the parent's (fp, tp):
// the parent's state cotangent bP, the child's rotation's and angular
// velocity's (tC, wC; its position's and velocity's are the parent's negated)
// and the clipped actions' (ab).
template <int MAXDOF>
__device__ __forceinline__ void joint_tan_back(const JointT& J, const JointTan<MAXDOF>& k, v3 fcb, v3 tcb, v3 fpb, v3 tpb,
                                               TBar& bP, v3& tC, v3& wC, float* ab) {
  const v3 taub = tcb - tpb;
  const v3 Fb = (fcb - fpb) + cross(tcb, k.rC) - cross(tpb, k.rP);
  v3 rCb = cross(k.F, tcb), rPb = -cross(k.F, tpb);
  // axes, limits and actuators: torque sc_k about axis k, sc' = st_k theta'
  const float d0 = dot(k.e1P, taub);
  ab[0] = k.gear[0] * d0;
  float thb0 = k.st[0] * d0;
  bP.t = k.sc[0] * cross(k.e1P, taub);
  tC = V(0.f, 0.f, 0.f);
  if (MAXDOF > 1) {
    const float d1 = dot(k.ax1, taub), d2 = dot(k.e3C, taub);
    ab[1] = k.gear[MAXDOF > 1 ? 1 : 0] * d1;
    ab[2] = k.gear[MAXDOF > 2 ? 2 : 0] * d2;
    const float s1 = k.sc[MAXDOF > 1 ? 1 : 0], s2 = k.sc[MAXDOF > 2 ? 2 : 0];
    // axis 1 turns with the parent and, about e1P, with angle 0
    thb0 += s1 * dot(taub, k.n1);
    bP.t += s1 * cross(k.ax1, taub);
    tC = s2 * cross(k.e3C, taub);
    const v3 m = (k.st[MAXDOF > 1 ? 1 : 0] * d1) * k.t[MAXDOF > 1 ? 1 : 0] + (k.st[MAXDOF > 2 ? 2 : 0] * d2) * k.t[MAXDOF > 2 ? 2 : 0];
    bP.t += m;
    tC -= m;
  }
  const v3 t0 = thb0 * k.t[0];
  bP.t += t0;
  tC -= t0;
  // damper
  bP.w = J.c_ang * taub;
  wC = -bP.w;
  // alignment
  if (MAXDOF == 1 || J.dof == 1) {
    // k e1C x e1P
    const v3 ca = (J.k_ang * k.c11) * taub;
    bP.t += ca - (J.k_ang * d0) * k.e1C;
    tC += (J.k_ang * dot(k.e1C, taub)) * k.e1P - ca;
  } else if (J.dof == 2) {
    // -k m01 (e2C x e1P), m01 = e1P . e2C
    const v3 wv = cross(k.e2C, k.e1P);
    const float m01b = -J.k_ang * dot(wv, taub);
    const v3 wb = (-J.k_ang * k.m01) * taub;
    bP.t += cross(k.e1P, cross(wb, k.e2C) + m01b * k.e2C);
    tC += cross(k.e2C, cross(k.e1P, wb) + m01b * k.e1P);
  }
  // anchor spring-damper
  bP.p = J.k_lin * Fb;
  bP.v = J.c_lin * Fb;
  bP.w += cross(k.rP, bP.v);
  rPb += cross(bP.v, k.wP) + bP.p;
  wC -= cross(k.rC, bP.v);
  rCb -= cross(bP.v, k.wC) + bP.p;
  bP.t += cross(k.rP, rPb);
  tC += cross(k.rC, rCb);
}

// ------------------------------------------------------------ ground contact
// A candidate's impulse with what its adjoint needs, from the forward formulas
// (contact_add); on: an impulse applied.
struct ContactTan {
  v3 rr, rl, y, dw, b;           // lever arm, R l, r x J, Iwinv (r x J), Iwinv (r x t)
  v3 bz, az;                     // 2 b x (r x t), 2 a x (r x z) with a = Iwinv (r x z)
  float ax, ay;                  // a
  float Jx, Jy, jn, jt, tx, ty;  // impulse, friction impulse and slip direction
  float ikn, ikt, isp, spk;      // 1/kn, 1/kt, 1/|slip|, |slip| / kt^2
  bool on, cap;                  // cap: the Coulomb cap applies
};
__device__ __forceinline__ void contact_tan_fwd(const ContactT& c, bool has, const TypeT& ty, const BodyT& B, const Body& s,
                                                const m3& R, const s3& I, ContactTan& k) {
  k.rl = mul(R, ld3(c.l));
  const float depth = c.rho - (s.p.z + k.rl.z);
  const v3 r = V(k.rl.x, k.rl.y, k.rl.z - c.rho);
  const v3 u = s.v + cross(s.w, r);
  k.rr = r;
  const v3 a = V(fmaf(I.xx, r.y, -(I.xy * r.x)), fmaf(I.xy, r.y, -(I.yy * r.x)), fmaf(I.xz, r.y, -(I.yz * r.x)));
  const float kn = B.inv_m + fmaf(a.x, r.y, -(a.y * r.x));
  const float num = fmaf(ty.beta_h, depth, -(ty.one_plus_e * u.z));
  k.on = has && depth > 0.f && num > 0.f;
  k.ikn = __builtin_amdgcn_rcpf(kn);
  k.jn = num * k.ikn;
  const float sp2 = fmaf(u.x, u.x, u.y * u.y);
  const bool slip = sp2 > 0.f;  // a zero or NaN slip: t = 0, and with it every friction term
  k.isp = slip ? __builtin_amdgcn_rsqf(sp2) : 0.f;
  k.tx = slip ? u.x * k.isp : 0.f;
  k.ty = slip ? u.y * k.isp : 0.f;
  const float sp = slip ? sp2 * k.isp : 0.f;
  const v3 zt = V(-(r.z * k.ty), r.z * k.tx, fmaf(r.x, k.ty, -(r.y * k.tx)));
  k.b = mul(I, zt);
  k.ikt = __builtin_amdgcn_rcpf(B.inv_m + dot(zt, k.b));
  const float stop = sp * k.ikt, cap = ty.mu * k.jn;
  k.cap = cap <= stop;
  k.jt = k.cap ? cap : stop;
  k.spk = stop * k.ikt;
  k.Jx = -(k.jt * k.tx);
  k.Jy = -(k.jt * k.ty);
  k.y = V(fmaf(r.y, k.jn, -(r.z * k.Jy)), fmaf(r.z, k.Jx, -(r.x * k.jn)), fmaf(r.x, k.Jy, -(r.y * k.Jx)));
  k.dw = k.jn * a - k.jt * k.b;
  k.ax = a.x;
  k.ay = a.y;
  k.az = 2.f * V(a.z * r.x, a.z * r.y, -(a.x * r.x + a.y * r.y));
  k.bz = 2.f * cross(k.b, zt);
  // rounded here, so that a candidate gives the same bits from a register and
  // from the table, whatever the code around it lets the compiler fuse
  for (v3* x : {&k.rr, &k.rl, &k.y, &k.dw, &k.b, &k.bz, &k.az}) pin(*x);
  for (float* x : {&k.ax, &k.ay, &k.Jx, &k.Jy, &k.jn, &k.jt, &k.tx, &k.ty, &k.ikn, &k.ikt, &k.isp, &k.spk}) pin(*x);
}
// The cotangents of a body's dv and dw with their products common to its
// candidates: dv / m and Iwinv dw.
struct ContactBar {
  v3 Jb, dw, yb;
};
__device__ __forceinline__ ContactBar contact_bar(const BodyT& B, const s3& I, v3 dvb, v3 dwb) {
  ContactBar c{B.inv_m * dvb, dwb, mul(I, dwb)};
  pin(c.Jb);
  pin(c.dw);
  pin(c.yb);
  return c;
}
// Adds the body's cotangents to o, given those of its dv and dw.
__device__ __forceinline__ void contact_tan_back(const ContactTan& k, const TypeT& ty, v3 w, const ContactBar& cb, TBar& o) {
  const v3 yb = cb.yb;
  v3 t = cross(k.dw, cb.dw) + cross(yb, k.y);
  const v3 J = V(k.Jx, k.Jy, k.jn);
  v3 rb = cross(J, yb);
  const v3 Jb = cb.Jb + cross(yb, k.rr);
  const float jtb = -(Jb.x * k.tx + Jb.y * k.ty);
  const float capb = k.cap ? jtb : 0.f, stopb = k.cap ? 0.f : jtb;
  const float numb = (Jb.z + ty.mu * capb) * k.ikn, knb = -(numb * k.jn);
  const float ktb = -(stopb * k.spk), spb = stopb * k.ikt;
  t += ktb * k.bz + knb * k.az;
  const v3 ztb = (2.f * ktb) * k.b;
  // r x t with t.z = 0; r x z
  rb.x += k.ty * ztb.z - 2.f * knb * k.ay;
  rb.y += 2.f * knb * k.ax - k.tx * ztb.z;
  rb.z += k.tx * ztb.y - k.ty * ztb.x;
  const float tbx = ztb.y * k.rr.z - ztb.z * k.rr.y - k.jt * Jb.x;
  const float tby = ztb.z * k.rr.x - ztb.x * k.rr.z - k.jt * Jb.y;
  // t = slip / |slip|
  const float td = tbx * k.tx + tby * k.ty;
  const v3 ub = V((tbx - k.tx * td) * k.isp + spb * k.tx, (tby - k.ty * td) * k.isp + spb * k.ty, -(ty.one_plus_e * numb));
  const float depthb = ty.beta_h * numb;
  rb += cross(ub, w);
  rb.z -= depthb;
  TBar c = TBar{V(0.f, 0.f, -depthb), t + cross(k.rl, rb), ub, cross(k.rr, ub)};
  pin(c.p.z);
  pin(c.t);
  pin(c.v);
  pin(c.w);
  o.p.z += c.p.z;
  o.t += c.t;
  o.v += c.v;
  o.w += c.w;
}
// The same for a candidate recomputed on the spot.
__device__ __forceinline__ void contact_tan(const ContactT& c, const TypeT& ty, const BodyT& B, const Body& s, const Frame& f,
                                            const ContactBar& cb, TBar& o) {
  ContactTan k;
  contact_tan_fwd(c, true, ty, B, s, f.R, f.Iwinv, k);
  if (k.on) contact_tan_back(k, ty, s.w, cb, o);
}
// Frame cotangents as a rotation vector: those of Iwinv into R's, and R's
// columns r_j = R l_j with cotangents Rb's columns.
__device__ __forceinline__ v3 frame_tan(const BodyT& B, const Frame& f, const FrameBar& fr) {
  m3 Rb = fr.Rb;
  rot_diag_adj(f.R, B.Iinv, fr.Iwinvb, Rb);
  return cross(col(f.R, 0), col(Rb, 0)) + cross(col(f.R, 1), col(Rb, 1)) + cross(col(f.R, 2), col(Rb, 2));
}

}  // namespace bx
