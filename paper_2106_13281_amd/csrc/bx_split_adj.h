// The adjoint of a substep on three wavefronts per work item (device code).
//
// Only the state cotangent G runs through the substeps as a chain; everything
// an adjoint recomputes from the tape (post-kinematic states, frames, joint
// geometry, contact impulses) does not depend on it. One lane per body on each
// wavefront; two phases per substep, each ended by a barrier:
//            wavefront 0, body            1, joint                 2, contact
//   phase 1  sums the cotangents of the   recomputes the joint of  recomputes the contacts
//            substep after it, its        this substep             of this substep
//            kinematic adjoint -> G; the
//            force, torque and velocity-
//            change cotangents of this
//            substep
//   phase 2  gyroscopic adjoint; state    joint adjoint -> the     contact adjoints
//            and frame of the next        parent's and the child's
//            substep from its record      cotangents
// Results cross through LDS rows written in one phase and read in the next.
// One wavefront runs all of it as one chain; a small batch leaves most SIMDs
// empty, so the three share the chain between SIMDs: single-step adjoint of
// 700 quadrupeds, forward recompute included, 42.2 -> 24.2 us.
#pragma once
#include "bx_access.h"
#include "bx_adj_tan.h"
#include "bx_pair_lanes.h"
#include "bx_split.h"

namespace bx {

__device__ __forceinline__ Bar load_bar(const Fields& f, int b, int e, int Bm, int E) {
  Body s = load_body(f, b, e, Bm, E);
  Bar r;
  r.p = s.p;
  r.q = s.q;
  r.v = s.v;
  r.w = s.w;
  return r;
}
__device__ __forceinline__ void store_bar(const Fields& f, const Bar& r, int b, int e, int Bm, int E) {
  Body s;
  s.p = r.p;
  s.q = r.q;
  s.v = r.v;
  s.w = r.w;
  store_body(f, 0, s, b, e, Bm, E);
}

struct AdjRows {
  float4 frame[64][7];    // 0 -> 1, 2: post-kinematic p, v, w, R and Iwinv (24 floats)
  float4 head[64][3];     // 0 -> 1, 2: cotangents of the force, torque, dv and dw sums
  float4 joint[65][5];    // 1 -> 0: the parent's cotangent (p, t, v, w), the child's (t, w); row 64 stays zero,
                          // for lanes without an i-th child or a joint
  float4 contact[64][3];  // 2 -> 0: cotangents of p, t, v, w
};

template <int MAXDOF>
__device__ __forceinline__ void pin(JointTan<MAXDOF>& k) {
  pin(k.rP);
  pin(k.rC);
  pin(k.F);
  pin(k.e1P);
  pin(k.e1C);
  pin(k.c11);
  for (int i = 0; i < MAXDOF; ++i) {
    pin(k.t[i]);
    pin(k.sc[i]);
    pin(k.st[i]);
  }
  if (MAXDOF > 1) {
    pin(k.e2C);
    pin(k.e3C);
    pin(k.ax1);
    pin(k.n1);
  }
}
// The reverse substeps of one step on one of the three wavefronts (ROLE 0:
// body, 1: joint, 2: contact), from their tape records in LDS. act, g_act
// [Am][E].
template <int ROLE, int MAXDOF, bool PAIRS, int REGC>
__device__ __forceinline__ void split_adj_run(const Tables* __restrict__ tab, const WaveWork& wk,
                                              const int32_t* __restrict__ env_list,
                                              const int32_t* __restrict__ type_off, int E, int Bm, int Am,
                                              const float* __restrict__ act, const Fields& g_out, const Fields& g_in,
                                              float* __restrict__ g_act, const float* tape, AdjRows* L,
                                              PairLanes* pl) {
  constexpr bool BODY = ROLE == 0, JOINT = ROLE == 1, CONTACT = ROLE == 2;
  const int t = wk.type;
  TypeT ty = tab->type[t];
  const int nb = ty.nb;
  const int lane = threadIdx.x & 63;
  const int per_wave = 64 / nb;
  const bool spare = lane >= per_wave * nb;  // shadows the first slot's lanes
  const int slot = spare ? 0 : lane / nb;
  const int b = spare ? lane - per_wave * nb : lane - slot * nb;
  const int base = slot * nb;
  const bool live = !spare && slot < wk.count;
  const int e = env_list[type_off[t] + wk.k0 + (live ? slot : 0)];
  BodyT B = tab->body[t][b];
  const bool has_joint = B.joint >= 0;
  JointT J = tab->joint[t][has_joint ? B.joint : 0];
  const int src_parent = base + (has_joint ? J.parent : b);
  const int n_con = B.c1 - B.c0;
  ContactT Creg[REGC];
  pin(ty.h);
  pin(B.inv_m);
  pin3(B.free_p);
  pin3(B.free_r);
  if (JOINT) pin_joint<MAXDOF>(J, has_joint);
  if (!JOINT) pin3(B.Iinv);
  if (BODY) pin3(B.I);
  if (CONTACT) {
    pin(ty.beta_h);
    pin(ty.one_plus_e);
    pin(ty.mu);
#pragma unroll
    for (int k = 0; k < REGC; ++k) {
      Creg[k] = tab->contact[t][B.c0 + (n_con > k ? k : 0)];
      pin3(Creg[k].l);
      pin(Creg[k].rho);
    }
    if (PAIRS && ty.np > 0) pair_lanes_load(tab, t, pl, lane, nb);
  }
  const float h = ty.h;
  const int S = ty.substeps;
  int csrc[GATHER];  // the children's rows (the zero row where there is none)
#pragma unroll
  for (int i = 0; i < GATHER; ++i) csrc[i] = i < B.nch ? base + (int)((B.ch_packed >> (4 * i)) & 15u) : 64;
  // this body's joint row; a root has none (its lane's row holds the cotangents
  // of no joint, NaN on a non-finite state)
  const int jrow = has_joint ? lane : 64;
  if (JOINT && lane < 5) L->joint[64][lane] = make_float4(0.f, 0.f, 0.f, 0.f);

  if (BODY) {
    TapeRec rec;
    auto fetch = [&](int sub) { wtape_fetch<false>(tape + (size_t)sub * TAPE_N * 64, lane, rec); };
    // the substep in rec: what this wavefront needs of it, and the frame row
    // of the others; then the record of the substep before it
    auto advance = [&](int sub) {
      Body post;
      v3 ttot;
      int n;
      wtape_unpack(rec, post, ttot, n);
      if (sub > 0) fetch(sub - 1);
      const q4 q0 = post.q;
      kinematic(B, post, h);
      const BodyTan k = body_tan(B, q0, post, ttot, n, h);
      float4* r = L->frame[lane];
      r[0] = make_float4(post.p.x, post.p.y, post.p.z, post.v.x);
      r[1] = make_float4(post.v.y, post.v.z, post.w.x, post.w.y);
      r[2] = make_float4(post.w.z, k.R.m[0], k.R.m[1], k.R.m[2]);
      r[3] = make_float4(k.R.m[3], k.R.m[4], k.R.m[5], k.R.m[6]);
      r[4] = make_float4(k.R.m[7], k.R.m[8], k.Iwinv.xx, k.Iwinv.yy);
      r[5] = make_float4(k.Iwinv.zz, k.Iwinv.xy, k.Iwinv.xz, k.Iwinv.yz);
      return k;
    };
    fetch(S - 1);
    BodyTan k = advance(S - 1);
    TBar G = tbar_zero();
    if (live) {
      const Bar g = load_bar(g_out, b, e, Bm, E);
      G = TBar{g.p, quat_tan(k.q1, g.q), keep(g.v, B.free_p), keep(g.w, B.free_r)};
    }
    q4 gq = q4{0.f, 0.f, 0.f, 0.f};
    block_exchange();
    for (int sub = S - 1; sub >= 0; --sub) {
      v3 fb, tb, dvb, dwb;
      body_head(B, k, h, G, fb, tb, dvb, dwb);
      L->head[lane][0] = make_float4(fb.x, fb.y, fb.z, tb.x);
      L->head[lane][1] = make_float4(tb.y, tb.z, dvb.x, dvb.y);
      L->head[lane][2] = make_float4(dvb.z, dwb.x, dwb.y, dwb.z);
      block_exchange();
      TBar tot = G;
      potential_tan(B, k, h, G.w, tb, tot);
      pin(tot.t);
      pin(tot.w);
      // the next substep's frame while the other wavefronts are busy
      BodyTan kn = k;
      if (sub > 0) kn = advance(sub - 1);
      pin(kn.al);
      block_exchange();
      const TBar c = tbar_get(L->contact[lane]), j = tbar_get(L->joint[jrow]);
      const float4 j3 = L->joint[jrow][3];
      const float2 j4 = *reinterpret_cast<const float2*>(&L->joint[jrow][4]);
      TBar c0 = tbar_get(L->joint[csrc[0]]), c1 = tbar_get(L->joint[csrc[1]]);
      tbar_add(tot, c);
      // this body's joint: the child's p and v cotangents are the parent's
      // negated
      tot.p -= j.p;
      tot.v -= j.v;
      tot.t += V(j3.x, j3.y, j3.z);
      tot.w += V(j3.w, j4.x, j4.y);
      tbar_add(tot, c0);
      tbar_add(tot, c1);
      if (ty.max_children > 2) {
        c0 = tbar_get(L->joint[csrc[2]]);
        c1 = tbar_get(L->joint[csrc[3]]);
        tbar_add(tot, c0);
        tbar_add(tot, c1);
      }
      for (int i = GATHER; i < ty.max_children; ++i)
        tbar_add(tot, tbar_get(L->joint[i < B.nch ? base + (int)((B.ch_packed >> (4 * i)) & 15u) : 64]));
      G = kinematic_tan(B, ty.frozen, k, h, tot);
      if (sub == 0) gq = kinematic_tan_quat(k, h, tot.t);
      k = kn;
    }
    if (live) {
      store_bar(g_in, Bar{G.p, gq, G.v, G.w}, b, e, Bm, E);
      for (int pb = nb + b; pb < Bm; pb += nb) zero_body(g_in, pb, e, Bm, E);
    }
    return;
  }

  float a[3] = {0.f, 0.f, 0.f}, raw[3] = {0.f, 0.f, 0.f}, ga[3] = {0.f, 0.f, 0.f};
  if (JOINT && has_joint)
    for (int x = 0; x < MAXDOF; ++x) {
      raw[x] = act_raw(act, J, x, e, E);
      a[x] = clampf(raw[x], J.act_lo[x], J.act_hi[x]);
    }
  auto frame_get = [&](int src, Body& post, m3& R) {
    const float4* r = L->frame[src];
    const float4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3], r4 = r[4];
    post.p = V(r0.x, r0.y, r0.z);
    post.v = V(r0.w, r1.x, r1.y);
    post.w = V(r1.z, r1.w, r2.x);
    R = m3{{r2.y, r2.z, r2.w, r3.x, r3.y, r3.z, r3.w, r4.x, r4.y}};
    return r4;
  };
  block_exchange();
  for (int sub = S - 1; sub >= 0; --sub) {
    Body post;
    if (JOINT) {
      Body P;
      m3 R, RP;
      (void)frame_get(lane, post, R);
      (void)frame_get(src_parent, P, RP);
      JointTan<MAXDOF> k;
      joint_tan_fwd<MAXDOF>(J, P, RP, post, R, a, k);
      pin(k);
      block_exchange();
      const float4 h0 = L->head[lane][0], p0 = L->head[src_parent][0];
      const float2 h1 = *reinterpret_cast<const float2*>(&L->head[lane][1]);
      const float2 p1 = *reinterpret_cast<const float2*>(&L->head[src_parent][1]);
      TBar bP;
      v3 tC, wC;
      float ab[3];
      joint_tan_back<MAXDOF>(J, k, V(h0.x, h0.y, h0.z), V(h0.w, h1.x, h1.y), V(p0.x, p0.y, p0.z), V(p0.w, p1.x, p1.y),
                             bP, tC, wC, ab);
      for (int x = 0; x < MAXDOF; ++x) ga[x] += ab[x];
      float4* r = L->joint[lane];
      tbar_put(r, bP);
      r[3] = make_float4(tC.x, tC.y, tC.z, wC.x);
      *reinterpret_cast<float2*>(&r[4]) = make_float2(wC.y, wC.z);
    } else {
      Frame f;
      const float4 r4 = frame_get(lane, post, f.R), r5 = L->frame[lane][5];
      f.Iwinv = s3{r4.z, r4.w, r5.x, r5.y, r5.z, r5.w};
      f.Iw = s3_zero();
      ContactTan k[2];
      const bool any0 = 0 < ty.max_contacts, any1 = 1 < ty.max_contacts;
      if (any0) contact_tan_fwd(Creg[0], n_con > 0, ty, B, post, f.R, f.Iwinv, k[0]);
      if (any1) contact_tan_fwd(Creg[REGC > 1 ? 1 : 0], n_con > 1, ty, B, post, f.R, f.Iwinv, k[1]);
      block_exchange();
      const float4 h1 = L->head[lane][1], h2 = L->head[lane][2];
      const v3 dvb = V(h1.z, h1.w, h2.x), dwb = V(h2.y, h2.z, h2.w);
      const ContactBar cb = contact_bar(B, f.Iwinv, dvb, dwb);
      TBar r = tbar_zero();
      if (any0 && k[0].on) contact_tan_back(k[0], ty, post.w, cb, r);
      if (any1 && k[1].on) contact_tan_back(k[1], ty, post.w, cb, r);
#pragma unroll
      for (int i = 2; i < REGC; ++i)
        if (i < ty.max_contacts && n_con > i) contact_tan(Creg[i], ty, B, post, f, cb, r);
      for (int i = REGC; i < n_con; ++i) contact_tan(tab->contact[t][B.c0 + i], ty, B, post, f, cb, r);
      if (PAIRS && ty.np > 0) {
        Bar pb = bar_zero();
        FrameBar fr = framebar_zero();
        float invm_bar = 0.f, mu_bar = 0.f;  // not kept
        pair_phase_adj(tab, t, *pl, b, base, post, f, dvb, dwb, pb, fr, invm_bar, mu_bar);
        tbar_add(r, TBar{pb.p, frame_tan(B, f, fr), pb.v, pb.w});
      }
      tbar_put(L->contact[lane], r);
    }
    block_exchange();
  }
  if (JOINT && live) {
    // action cotangents (zero where the action was clamped)
    if (has_joint)
      for (int x = 0; x < MAXDOF; ++x)
        if (x < J.dof && J.act[x] >= 0)
          g_act[(size_t)J.act[x] * E + e] = (raw[x] >= J.act_lo[x] && raw[x] <= J.act_hi[x]) ? ga[x] : 0.f;
    if (b == 0)
      for (int x = ty.na; x < Am; ++x) g_act[(size_t)x * E + e] = 0.f;
  }
}

// The forward substeps of one step before its adjoint, on wavefronts 1 (the
// joint half of the split step, ROLE 0 there) and 2 (the contact half, ROLE 1),
// their records into LDS.
template <int ROLE, int MAXDOF, bool PAIRS, int REGC>
__device__ __forceinline__ void split_fwd_run(const Tables* __restrict__ tab, const WaveWork& wk,
                                              const int32_t* __restrict__ env_list,
                                              const int32_t* __restrict__ type_off, int E, int Bm, const Fields& in,
                                              const float* __restrict__ act, float* lds_tape, SplitRows* L, XchRows* XC,
                                              PairLanes* pl) {
  constexpr bool JOINT = ROLE == 0, CONTACT = ROLE == 1, RECORD = ROLE == tape_role(MAXDOF);
  const int t = wk.type;
  TypeT ty = tab->type[t];
  const int nb = ty.nb;
  const int lane = threadIdx.x & 63;
  const int per_wave = 64 / nb;
  const bool spare = lane >= per_wave * nb;  // shadows the first slot's lanes
  const int slot = spare ? 0 : lane / nb;
  const int b = spare ? lane - per_wave * nb : lane - slot * nb;
  const int base = slot * nb;
  const int e = env_list[type_off[t] + wk.k0 + (!spare && slot < wk.count ? slot : 0)];
  BodyT B = tab->body[t][b];
  const bool has_joint = B.joint >= 0;
  JointT J = tab->joint[t][has_joint ? B.joint : 0];
  const int src_parent = base + (has_joint ? J.parent : b);
  const int n_con = B.c1 - B.c0;
  ContactT Creg[REGC];
#pragma unroll
  for (int k = 0; k < REGC; ++k) Creg[k] = tab->contact[t][B.c0 + (n_con > k ? k : 0)];
  pin(ty.h);
  if (CONTACT && PAIRS && ty.np > 0) pair_lanes_load(tab, t, pl, lane, nb);
  const PairSlot0 ps0 = (CONTACT && PAIRS && ty.np > 0) ? pair_slot0(*pl, b, base) : PairSlot0{-1, lane, lane};
  int csrc[GATHER];
#pragma unroll
  for (int i = 0; i < GATHER; ++i) csrc[i] = i < B.nch ? base + (int)((B.ch_packed >> (4 * i)) & 15u) : 64;
  if (JOINT && lane < 3) L->joint[0][64][lane] = L->joint[1][64][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
  float a[3] = {0.f, 0.f, 0.f};
  if (JOINT && has_joint)
    for (int x = 0; x < MAXDOF; ++x) a[x] = act_of(act, J, x, e, E);
  Body s = load_body(in, b, e, Bm, E);
  s.v = keep(s.v, B.free_p);
  s.w = keep(s.w, B.free_r);
  auto substep = [&](int sub, auto parity) {
    float* tp = lds_tape + (size_t)sub * TAPE_N * 64;
    const float wz = s.w.z;
    if (RECORD) wtape_state<false>(tp, s, lane);
    v3 torque;
    int cnt;
    split_substep<ROLE, MAXDOF, PAIRS, false, REGC, contact_form(true, false, PAIRS, false, REGC), decltype(parity)::value>(tab, t, ty, B, J, has_joint, Creg, B.c0, n_con,
                                                                             ty.max_contacts, lane, b, base, false,
                                                                             src_parent, csrc, a, s, L, XC, pl, ps0,
                                                                             torque, cnt);
    if (RECORD) wtape_torque<false>(tp, wz, torque, lane);
    if (CONTACT) wtape_count(tp, cnt, lane);
  };
  for (int sub = 0; sub < ty.substeps; sub += 2) {
    substep(sub, std::integral_constant<int, 0>{});
    if (sub + 1 < ty.substeps) substep(sub + 1, std::integral_constant<int, 1>{});
  }
}

}  // namespace bx
