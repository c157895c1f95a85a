// The substep on two wavefronts per work item (device code): the joint half and
// the contact half of a substep side by side.
#pragma once
#include <type_traits>

#include "bx_access.h"
#include "bx_pair_lanes.h"

namespace bx {

// The form of the ground impulses. Straight in kernels that hold two candidates,
// but not those for one-axis batches with contact lanes: there, and with eight
// candidates, most slots have a few lanes of one body in them. On two wavefronts
// per item (two) the chain counts, and the lanes in contact run straight
// through; on one, two per SIMD share the issue slots, and skipped friction (a
// box at rest) is time. Measured, contact_apply / STRAIGHT / LANES / LANES_SKIP (us):
//   manipulator x 20 steps, boxes tumbling: taped, two wavefronts 4000 environments
//     353 / 334 / 316 / 340, one 14000 478 / 503 / 486 / 484; untaped, two 4000 243 / 236 /
//     231 / 231, one 14000 437 / 436 / 422 / 425
//   boxes at rest: taped 9000 340 / 388 / 366 / 337, 15300 429 / 521 / 502 / 442;
//     untaped 6000 255 / 263 / 263 / 255, 10200 337 / 352 / 354 / 333
// The mixed batch untaped (only one of its types has such a body): 8000 x 100 steps
// contact_apply 1291, STRAIGHT 1276. With body-body contacts (and the penetrating
// first) grasp 14040 x 20 steps 1199, 1172.
constexpr ContactForm contact_form(bool two, bool one_axis, bool pairs, bool cl, int regc) {
  return regc == REG_CONTACTS && (pairs || !cl || !one_axis) ? STRAIGHT : two ? LANES : LANES_SKIP;
}

// A lane's ground-contact candidates: the first REGC from registers (no
// dynamic indexing; a slot no body of the type has is skipped by the whole
// wave), the rest from the table C. Adds the velocity changes to dv, dw and
// the applied candidates to cnt.
// FORM: how the impulses run (the same sums).
// PEN_FIRST (of STRAIGHT kernels): the penetrating candidates first, in
// candidate order (the same sums), so that the second evaluation runs only
// where a lane has two penetrating candidates, not wherever one has its second
// (x 20 steps, without -> with: planar runner 2610 environments 149 -> 144 us,
// biped 11700 519 -> 506, grasp 14040 1190 -> 1169, quadruped 2030 182 -> 178 but
// 16380 370 -> 379).
template <int REGC, ContactForm FORM, bool PEN_FIRST>
__device__ __forceinline__ void ground_contacts(const ContactT* __restrict__ C, const ContactT (&Creg)[REGC], int n_con,
                                                int max_con, const TypeT& ty, const BodyT& B, const Body& s,
                                                const Frame& f, v3& dv, v3& dw, int& cnt) {
  if (PEN_FIRST) {
    const v3 rl0 = mul(f.R, ld3(Creg[0].l)), rl1 = mul(f.R, ld3(Creg[REGC - 1].l));
    const float d0 = Creg[0].rho - (s.p.z + rl0.z), d1 = Creg[REGC - 1].rho - (s.p.z + rl1.z);
    const bool p0 = 0 < max_con && n_con > 0 && d0 > 0.f;
    const bool p1 = 1 < max_con && n_con > 1 && d1 > 0.f;
    if (__ballot(p0 || p1))
      contact_add<FORM>(p0 ? Creg[0].rho : Creg[REGC - 1].rho, ty, B, s, f.Iwinv, sel(p0, rl0, rl1), p0 ? d0 : d1, p0 || p1, dv,
                  dw, cnt);
    if (__ballot(p0 && p1)) contact_add<FORM>(Creg[REGC - 1].rho, ty, B, s, f.Iwinv, rl1, d1, p0 && p1, dv, dw, cnt);
  } else {
#pragma unroll
    for (int k = 0; k < REGC; ++k) {
      if (k < max_con) {
        const v3 rl = mul(f.R, ld3(Creg[k].l));
        const float depth = Creg[k].rho - (s.p.z + rl.z);
        const bool in = n_con > k && depth > 0.f;
        if (FORM == STRAIGHT ? __ballot(in) != 0 : in)
          contact_add<FORM>(Creg[k].rho, ty, B, s, f.Iwinv, rl, depth, in, dv, dw, cnt);
      }
    }
  }
  for (int c = REGC; c < n_con; ++c) cnt += contact_eval(C[c], ty, B, s, f, dv, dw) ? 1 : 0;
}

// A body's contact candidates spread over its lane group: every lane of the
// group adds the group's sums in group order (the same total on each, so the
// copies of the state stay equal), through the exchange rows X.
__device__ __forceinline__ void lane_group_sums(XchRows* X, int lane, int base, int b, const TypeT& ty, const BodyT& B,
                                                v3& dv, v3& dw, int& cnt) {
  X->r[lane][0] = make_float4(dv.x, dv.y, dv.z, (float)cnt);
  X->r[lane][1] = make_float4(dw.x, dw.y, dw.z, 0.f);
  v3 sv = V(0.f, 0.f, 0.f), sw = sv;
  int sc = 0;
  // four rows read together, then added in order (a group has at most 8 lanes)
  for (int i0 = 0; i0 < ty.max_ng; i0 += 4) {
    float4 gv[4], gw[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + j;
      const int src = base + (i < B.ng ? (int)((B.grp_packed >> (4 * (i & 7))) & 15u) : b);
      gv[j] = X->r[src][0];
      gw[j] = X->r[src][1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i0 + j < B.ng) {
        sv += V(gv[j].x, gv[j].y, gv[j].z);
        sw += V(gw[j].x, gw[j].y, gw[j].z);
        sc += (int)gv[j].w;
      }
    }
  }
  dv = sv;
  dw = sw;
  cnt = sc;
}

// ------------------------------------------------------------------ fused path, two wavefronts per group
// The fused step of one work item's environments on a block of two
// wavefronts. Both hold every body's state (one lane per body, as above) and
// advance it alike; each substep's work between the kinematic update and the
// integrators is divided between them:
//   wavefront 0: the parents' states, joints and actuators -> reactions;
//   wavefront 1: the inverse world inertia, the gyroscopic torque, ground and
//                body-body contacts -> velocity changes.
// Their results cross through LDS mail rows, double-buffered by substep
// parity, so that one barrier per substep is enough: a row is rewritten two
// substeps later, after a barrier that its readers reach only once they have
// used what they read. Both then gather the children's reactions and run the
// integrators on the same values.
// What it buys: the substep is one long chain of instructions per wavefront
// (quadruped: 472 VALU, 581 issue slots and 723 quad-cycles with the stalls),
// a SIMD issues at most one of a wavefront's instructions per quad-cycle, and
// gfx950 issues VALU instructions of two resident wavefronts together when
// their operands are VGPRs or literals (measured: add, mul, fma 4.7-5.4 cycles
// each with one wavefront per SIMD and with two; with an SGPR operand, and for
// compares, min/max, selects and transcendentals, 8.5-9.5 with two). A batch
// that leaves SIMDs with one wavefront or none therefore runs the two halves
// side by side. Quadruped 4096 x 1000: 12.84 -> 8.62 ms with the contact impulse
// free of branches.
struct SplitRows {
  XchRows xj;              // wavefront 0's exchange rows (parents' states)
  float4 joint[2][65][3];  // per parity and lane: force on the child, minus the torque on the parent, torque on
                           // the child (9 floats); row 64 stays zero, for lanes without an i-th child
  float4 body[2][64][5];   // per parity and lane: Iwinv (6), gyroscopic torque (3), dv (3), dw (3), 1 / contacts
};
// wavefront 1 needs exchange rows of its own for contact lanes and body-body contacts
static inline size_t split_lds(bool pairs, bool cl) {
  return sizeof(SplitRows) + (pairs || cl ? sizeof(XchRows) : 0) + (pairs ? sizeof(PairLanes) : 0);
}

// The wavefront that writes a substep's tape record (but for the contact
// count): the one with less to do, the contact half beside three-axis joints.
constexpr int tape_role(int maxdof) { return maxdof > 1 ? 1 : 0; }

// One substep of the split step on one of its wavefronts (ROLE 0: joints, 1:
// contacts); advances s. PAR: the mail rows' parity; two consecutive substeps
// use different ones. csrc: the children's mail rows (64: the zero row).
// groups: the batch has contact lanes in this type. torque: the body's total
// torque; cnt (ROLE 1): its applied contacts.
template <int ROLE, int MAXDOF, bool PAIRS, bool CL, int REGC, ContactForm FORM, int PAR>
__device__ __forceinline__ void split_substep(const Tables* __restrict__ tab, int t, const TypeT& ty, const BodyT& B,
                                              const JointT& J, bool has_joint, const ContactT (&Creg)[REGC], int cfirst,
                                              int n_con, int max_con, int lane, int b, int base, bool groups,
                                              int src_parent, const int (&csrc)[GATHER], const float* a, Body& s,
                                              SplitRows* L, XchRows* XC, PairLanes* pl, const PairSlot0& ps0,
                                              v3& torque, int& cnt) {
  constexpr bool JOINT = ROLE == 0;
  kinematic_unmasked(s, ty.h);
  v3 force, gyro, dv = V(0.f, 0.f, 0.f), dw = V(0.f, 0.f, 0.f);
  s3 Iwinv;
  float inv_n = 0.f;
  cnt = 0;
  float4(*mj)[3] = L->joint[PAR];
  float4(*mb)[5] = L->body[PAR];
  if (JOINT) {
    xch_put_pvw(&L->xj, lane, s);
    const m3 R = quat_to_mat(s.q);
    xch_put_rot(&L->xj, lane, s.w.z, R);
    Body P;
    m3 RP;
    xch_get_pvw_rot(&L->xj, src_parent, P, RP);
    P.q = s.q;  // unused: the joint reads the parent's orientation as RP
    const JointChild jc = joint_child<MAXDOF>(J, s, R);
    const JointOut jo = joint_eval<MAXDOF>(J, P, RP, s, jc, a);
    mj[lane][0] = make_float4(jo.fc.x, jo.fc.y, jo.fc.z, jo.tpn.x);
    mj[lane][1] = make_float4(jo.tpn.y, jo.tpn.z, jo.tc.x, jo.tc.y);
    *reinterpret_cast<float*>(&mj[lane][2]) = jo.tc.z;
    force = jo.fc;
    torque = jo.tc;
  } else {
    const m3 R = quat_to_mat(s.q);
    int near0 = 0;
    if (PAIRS && ty.np > 0) {
      xch_put_pvw(XC, lane, s);
      xch_put_rot(XC, lane, s.w.z, R);
      near0 = pair_near0(XC, *pl, ps0);
    }
    const Frame f = derive_inv(B, R);
    ground_contacts<REGC, FORM, FORM == STRAIGHT && (!CL || PAIRS)>(&tab->contact[t][cfirst], Creg, n_con, max_con, ty, B, s, f, dv, dw, cnt);
    gyro = gyro_torque(B, s, f);
    if (groups) lane_group_sums(XC, lane, base, b, ty, B, dv, dw, cnt);
    if (PAIRS && ty.np > 0) pair_phase(tab, t, *pl, XC, lane, b, base, s, f, dv, dw, cnt, near0);
    inv_n = cnt > 0 ? 1.f / (float)cnt : 0.f;
    Iwinv = f.Iwinv;
    mb[lane][0] = make_float4(Iwinv.xx, Iwinv.yy, Iwinv.zz, Iwinv.xy);
    mb[lane][1] = make_float4(Iwinv.xz, Iwinv.yz, gyro.x, gyro.y);
    mb[lane][2] = make_float4(gyro.z, dv.x, dv.y, dv.z);
    mb[lane][3] = make_float4(dw.x, dw.y, dw.z, inv_n);
  }
  block_exchange();
  // the other wavefront's results and the children's reactions (a child's
  // on its parent is the opposite of its force and tpn), all reads in
  // flight together; N: at least the type's largest child count
  auto combine = [&](auto nc) {
    constexpr int N = decltype(nc)::value;
    float4 c0[N + 1];
    float2 c1[N + 1];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      c0[i] = mj[csrc[i]][0];
      c1[i] = *reinterpret_cast<const float2*>(&mj[csrc[i]][1]);
    }
    if (JOINT) {
      const float4 m0 = mb[lane][0], m1 = mb[lane][1], m2 = mb[lane][2], m3_ = mb[lane][3];
      Iwinv = s3{m0.x, m0.y, m0.z, m0.w, m1.x, m1.y};
      gyro = V(m1.z, m1.w, m2.x);
      dv = V(m2.y, m2.z, m2.w);
      dw = V(m3_.x, m3_.y, m3_.z);
      inv_n = m3_.w;
    } else {
      const float4 j0 = mj[lane][0], j1 = mj[lane][1];
      const float j2 = *reinterpret_cast<const float*>(&mj[lane][2]);
      force = V(j0.x, j0.y, j0.z);
      torque = V(j1.z, j1.w, j2);
    }
    force = sel(has_joint, force, V(0.f, 0.f, 0.f));
    torque = sel(has_joint, torque, V(0.f, 0.f, 0.f));
#pragma unroll
    for (int i = 0; i < N; ++i) {
      force -= V(c0[i].x, c0[i].y, c0[i].z);
      torque -= V(c0[i].w, c1[i].x, c1[i].y);
    }
  };
  if (ty.max_children <= 2)
    combine(std::integral_constant<int, 2>{});
  else
    combine(std::integral_constant<int, GATHER>{});
  for (int i = GATHER; i < ty.max_children; ++i) {
    const int src = i < B.nch ? base + (int)((B.ch_packed >> (4 * i)) & 15u) : 64;
    const float4 x0 = mj[src][0];
    const float2 x1 = *reinterpret_cast<const float2*>(&mj[src][1]);
    force -= V(x0.x, x0.y, x0.z);
    torque -= V(x0.w, x1.x, x1.y);
  }
  // without frozen axes in the type (wave-uniform) the integrators skip the masks
  if (ty.frozen) {
    potential_apply(B, ty, s, Iwinv, force, torque, gyro);
    collision_apply(B, s, dv, dw, inv_n);
  } else {
    potential_apply<false>(B, ty, s, Iwinv, force, torque, gyro);
    collision_apply<false>(B, s, dv, dw, inv_n);
  }
}

}  // namespace bx
