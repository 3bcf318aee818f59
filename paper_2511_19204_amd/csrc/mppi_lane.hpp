// mppi_lane.hpp -- rollouts with one lane per root-to-leaf path of the tree.
//
// The throughput form: a lane walks its whole path (a leg, a torso and an arm),
// so a wavefront holds 64 / G rollouts of a tree with up to G paths (16
// quadrupeds or humanoids, 64 arms) and every issued instruction works on every
// path of every one of them; with one lane per body the sweeps issue each tree
// level for the few lanes of that level.  A wavefront's step is as long as the
// body schedule's (the same arithmetic body after body: 2 960 issue quads for 16
// quadrupeds instead of 2 213 for four, 6 760 for 16 humanoids instead of 5 085
// for two), so this form pays once there are enough rollouts to give most SIMDs
// a wavefront: 16 384 x 200 steps of the quadruped 2.25 -> 1.04 ms.
//
// A body's frame and joint terms stay in registers between the sweeps (one
// wavefront per SIMD has 512 of them), its constants and the knots are read
// from LDS.  The paths meet at the floating base and at bodies that several
// paths share; each path carries its own copy of those.
//
// The per-body arithmetic is the body schedule's helpers, with sums over
// children and costs in the same order: the results are its bits.
#pragma once
#include "mppi_step.hpp"

namespace mppi {

// Adds the inertia and bias that path P hands to the base, as the base's lane
// sees it: every lane of the group for up to four paths (a quad permutation),
// the group's first lane for eight (a row shift).
template <int G, int P>
__device__ __forceinline__ float from_path_lane(float x) {
  if constexpr (G == 1) return x;
  else if constexpr (G == 2) return qperm<P | P << 2 | (2 + P) << 4 | (2 + P) << 6>(x);
  else if constexpr (G == 4) return qperm<P * 0x55>(x);
  else if constexpr (P == 0) return x;
  else return from_row_lane<P>(x);
}
template <int G, int P>
__device__ __forceinline__ void add_path_lane(const float* Ip, const float* pp, float* IA, float* pA) {
  if constexpr (P < G) {
#pragma unroll
    for (int q = 0; q < 21; ++q) IA[q] += from_path_lane<G, P>(Ip[q]);
#pragma unroll
    for (int q = 0; q < 6; ++q) pA[q] += from_path_lane<G, P>(pp[q]);
  }
}

// A body of this lane's path between the sweeps.
struct LaneBody {
  float R[9], p[3], e[3], ax[3], v[6], c[6], beta[6];  // kinematics (see fk_joint)
  float U[6], invD, u;                                 // articulated terms (see backward_joint)
};

// One work item: 64 / G rollouts of one instance, samples first .. first + 64/G - 1
// (those >= N are computed but not stored).  L: the longest path the kernel
// holds; FB: floating base.
template <int G, int L, bool FB>
__device__ __attribute__((always_inline)) void lane_item(const DevInst& I, int first, float* smem,
                                                         const float* x0_in, const float* nominal_in) {
  constexpr bool kBranch = L > 3;  // paths may share bodies
  const float* x0 = x0_in ? x0_in : I.x0;
  switch (I.wave_prio) {
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 3: __builtin_amdgcn_s_setprio(3); break;
    default: break;
  }
  const int lane = threadIdx.x;
  const int grp = lane / G, path = lane % G;
  const DevModel& M = *I.model;
  const int nb = M.nb, nc = M.nc, np = M.n_paths;
  float* tab = smem;
  stage_model_table(M, &I, tab, lane);
  float* rows = tab + body_table_floats(nc);
  for (int i = lane; i < np * L * (kLaneRow / 4); i += 64) {
    const int rec = i / (kLaneRow / 4), w = i % (kLaneRow / 4);
    reinterpret_cast<float4*>(rows)[i] = reinterpret_cast<const float4*>(&M.lane_rows[rec / L][rec % L][0])[w];
  }
  float* exch = rows + np * L * kLaneRow;  // [64 lanes + a record of zeros][kLaneExch]
  if (kBranch && lane < kLaneExch) exch[64 * kLaneExch + lane] = 0.f;
  const int n = first + grp;
  const bool valid = n < I.N;
  float* knots = smem + lane_table_floats(nc, np, L) + grp * path_group_floats(I.E);
  if (I.generate) {
    sample_group<G>(M, I, valid ? n : 0, path, knots, valid, tab, nominal_in);
  } else {
    const float* src = I.samples + (size_t)(valid ? n : 0) * I.E;
    for (int e = path; e < I.E; e += G) knots[e] = src[e];
  }
  wave_sync();

  const StepConst sc = load_step_const(M, &I, 0.f);
  const int nq = FB ? 7 + M.nu : M.nu;
  // a lane past the last path walks the last one again; it owns no body
  const int pp_ = path < np ? path : np - 1;
  const float* my_rows = rows + pp_ * L * kLaneRow;
  int body[L], ct_of[L];  // bodies of this path; their contacts: first row | count << 8
  uint32_t src_of[kBranch ? L : 1];
  float q[L], v[L], acc[L], q0[L];
  uint32_t owner = 0u, cmax = 0u;
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int b = M.path_body[pp_][i], j = b >= 0 ? b - (FB ? 1 : 0) : 0;
    body[i] = b;
    if (b >= 0 && path < np && M.path_owner[pp_][i]) owner |= 1u << i;
    ct_of[i] = (path < np && b >= 0) ? (M.c_begin[b] | (M.c_count[b] << 8)) : 0;
    cmax |= (uint32_t)M.path_cmax[i] << (4 * i);
    if constexpr (kBranch) src_of[i] = M.path_src[pp_][i];
    q[i] = b >= 0 ? x0[(FB ? 7 : 0) + j] : 0.f;
    v[i] = b >= 0 ? x0[nq + (FB ? 6 : 0) + j] : 0.f;
    q0[i] = (b >= 0 && sc.cost_kind == 1) ? I.q0[j] : 0.f;
    acc[i] = 0.f;
  }
  float bq[7], bv[6], acc_base = 0.f;
#pragma unroll
  for (int i = 0; i < 7; ++i) bq[i] = FB ? x0[i] : 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) bv[i] = FB ? x0[nq + i] : 0.f;
  const int n_base_ct = FB ? M.c_count[0] : 0;
  const uint32_t branch = kBranch ? (uint32_t)M.path_branch : 0u;
  const uint32_t base_mask = (uint32_t)M.path_base_mask;
  const int ee_i = sc.cost_kind == 0 ? M.path_ee : -1;
  const int H = I.H, F = sc.F, F_run = H * sc.nsub;
  const float dt = sc.dt, g = sc.g;
  const bool to_end = sc.cost_kind == 0;  // the terminal cost needs the kinematics at x_H
  StepClock clk;
  HermiteSeg hs[L];
#pragma unroll
  for (int i = 0; i < L; ++i) hs[i] = HermiteSeg{0.f, 0.f, 0.f, 0.f};
  int hseg = -1;
  for (int f = 0;; ++f) {
    const bool last = f >= F_run;
    if (last && !to_end) break;
    const bool control = clk.sub == 0;
    if (MPPI_RARE(true, clk.seg != hseg && !last)) {
      hseg = clk.seg;
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (body[i] >= 0) hs[i] = hermite_segment(knots, sc.K, sc.nu, hseg, body[i] - (FB ? 1 : 0), sc.delta);
    }
    float Rb[9], pb[3];
    if constexpr (FB) {
      quat_R(bq + 3, Rb);
      pb[0] = bq[0]; pb[1] = bq[1]; pb[2] = bq[2];
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) Rb[i] = (i % 4 == 0) ? 1.f : 0.f;
      pb[0] = pb[1] = pb[2] = 0.f;
    }
    const float agl[3] = {-g * Rb[6], -g * Rb[7], -g * Rb[8]};

    // ---- PD law and kinematics, root to leaf
    LaneBody B[L];
    float tau[L], gain[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const float* r = my_rows + i * kLaneRow;
      float t[28], C[9];
      load_rotation_constants(r, t);
      const float4 a = get4(r + 28), b = get4(r + 32);  // p_tree, axis_p, kp, kd
      const float tm = r[36];
      const float pt[3] = {a.x, a.y, a.z}, ax[3] = {a.w, b.x, b.y};
      float qref, vref, cq, sq;
      hermite_eval(hs[i], (float)clk.rem * sc.inv_F, sc.inv_delta, &qref, &vref);
      if (sc.spline_mode != 0) vref = 0.f;
      pd_law(b.z, b.w, tm, dt, q[i], v[i], qref, vref, tau[i], gain[i]);
      sincosf(q[i], &sq, &cq);
      joint_rotation_of(t, cq, sq, C);
      LaneBody& o = B[i];
      if (i == 0) {
        if constexpr (FB) {
          fk_base_child(bv, C, pt, ax, v[i], o.R, o.p, o.e, o.ax, o.v, o.c, o.beta);
        } else {
          const float id[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f}, z[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          fk_joint(id, z, z, z, C, pt, ax, v[i], o.R, o.p, o.e, o.ax, o.v, o.c, o.beta);
        }
      } else {
        const LaneBody& par = B[i - 1];
        fk_joint(par.R, par.p, par.v, par.beta, C, pt, ax, v[i], o.R, o.p, o.e, o.ax, o.v, o.c, o.beta);
      }
    }
    float dz = 0.f;
    if (ee_i >= 0) {
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (i == ee_i) dz = ee_height_error(B[i].R, B[i].p, sc.ee_pos, Rb, pb, sc.z_des);
    }
    if (last) {
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (body[i] == sc.ee_body) {
          const float t = sc.w_ee * dz * dz;
          acc[i] += t;
        }
      break;
    }

    // ---- articulated inertias, leaf to root, with each body's running cost
    float Ip[21], pp[6];
#pragma unroll
    for (int i = L - 1; i >= 0; --i) {
      const float* r = my_rows + i * kLaneRow;
      LaneBody& o = B[i];
      float IA[21], pA[6];
      {
        const float4 a = get4(r + 40), b = get4(r + 44), c = get4(r + 48);  // com, Ic, mass, armature
        const float com[3] = {a.x, a.y, a.z}, Ic[6] = {a.w, b.x, b.y, b.z, b.w, c.x};
        body_inertia(o.R, com, Ic, c.y, IA);
      }
      bias_force(IA, o.v, pA);
      float cost = 0.f;
      const int most = (int)((cmax >> (4 * i)) & 15u);
      if (most > 0) {
        const int c0 = ct_of[i] & 255, cn = ct_of[i] >> 8;
#pragma unroll 1
        for (int c = 0; c < most; ++c) {
          if (c < cn) {
            const float* ct = tab + kTabContacts + (c0 + c) * kCt;
            float vw[3], fw[3];
            const float fn = contact_point(ct, o.R, o.p, o.v, o.beta, Rb, pb, agl, dt, sc.law, IA, pA, vw, fw);
            if (control && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], cost);
          }
        }
      }
      if (control) {
        if (sc.cost_kind == 1) {
          const float eq = q[i] - q0[i];
          cost += sc.w_q * eq * eq + sc.w_eff * tau[i] * tau[i];
        } else {
          cost += sc.w_tau * tau[i] * tau[i];
          if (body[i] == sc.ee_body) cost += sc.w_ee * dz * dz;
        }
        acc[i] += cost;
      }
      if (i < L - 1) {
        if (kBranch && ((branch >> i) & 1u)) {
          // some body here has children on several paths: they are added in child order
          put_art(exch + lane * kLaneExch, Ip, pp);
          wave_sync();
          const uint32_t src = src_of[kBranch ? i : 0];
#pragma unroll 1
          for (int c = 0; c < 4; ++c) {
            const uint32_t w = (src >> (8 * c)) & 255u;
            add_art(exch + (w == 255u ? 64 : grp * G + (int)w) * kLaneExch, IA, pA);
          }
          wave_sync();
        } else {
#pragma unroll
          for (int k = 0; k < 21; ++k) IA[k] += Ip[k];
#pragma unroll
          for (int k = 0; k < 6; ++k) pA[k] += pp[k];
        }
      }
      backward_joint(IA, pA, o.ax, o.c, o.e, tau[i], r[50], gain[i], o.U, o.invD, o.u, Ip, pp);
    }

    // ---- root: the base's articulated inertia and its solve, on every lane
    float a[6], ba[6];
    if constexpr (FB) {
      float IA[21], pA[6], base_cost = 0.f;
      {
        const float id[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
        body_inertia(id, M.com[0], M.Ic[0], M.mass[0], IA);
        bias_force(IA, bv, pA);
        const float z[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int c = 0; c < n_base_ct; ++c) {
          const float* ct = tab + kTabContacts + (M.c_begin[0] + c) * kCt;
          float vw[3], fw[3];
          const float fn = contact_point(ct, id, z, bv, z, Rb, pb, agl, dt, sc.law, IA, pA, vw, fw);
          if (control && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], base_cost);
        }
      }
      if (control && sc.cost_kind == 1) {
        base_cost += base_cost_term(sc, bq);
        acc_base += base_cost;
      }
      add_path_lane<G, 0>(Ip, pp, IA, pA);  // (the first path always brings the first child)
      if (base_mask & 2u) add_path_lane<G, 1>(Ip, pp, IA, pA);
      if (base_mask & 4u) add_path_lane<G, 2>(Ip, pp, IA, pA);
      if (base_mask & 8u) add_path_lane<G, 3>(Ip, pp, IA, pA);
      if (base_mask & 16u) add_path_lane<G, 4>(Ip, pp, IA, pA);
      if (base_mask & 32u) add_path_lane<G, 5>(Ip, pp, IA, pA);
      if (base_mask & 64u) add_path_lane<G, 6>(Ip, pp, IA, pA);
      if (base_mask & 128u) add_path_lane<G, 7>(Ip, pp, IA, pA);
      base_solve(IA, pA, a);
      if constexpr (G == 8) {
#pragma unroll
        for (int k = 0; k < 6; ++k) a[k] = from_group_lane0<G>(a[k]);
      }
      ba[0] = a[0]; ba[1] = a[1]; ba[2] = a[2];
      ba[3] = a[3] + agl[0]; ba[4] = a[4] + agl[1]; ba[5] = a[5] + agl[2];
    } else {
      a[0] = a[1] = a[2] = a[3] = a[4] = 0.f;
      a[5] = g;  // a' = -a_g
    }

    // ---- accelerations, root to leaf, and integration
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LaneBody& o = B[i];
      float al[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) al[k] = a[k];
      const float qdd = forward_joint(al, o.e, o.c, o.U, o.u, o.invD, o.ax, a);
      v[i] = fmaf(dt, qdd, v[i]);
      q[i] = fmaf(dt, v[i], q[i]);
    }
    if constexpr (FB) integrate_base_R<true>(bq, bv, ba, dt, Rb);
    clk.advance<true>(sc.K, F, sc.nsub);
  }
  if (FB && sc.cost_kind == 1) {
    const float T = (float)H * I.dt;
    float e = 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float target = (i == 2 && I.targets->terminal_z_abs) ? I.targets->z_terminal : x0[i] + I.targets->v_des[i] * T;
      e += fabsf(bq[i] - target);
    }
    acc_base += I.w_H * e;
  }
  wave_sync();  // the knots are not read any more: the costs by body take their place
#pragma unroll
  for (int i = 0; i < L; ++i)
    if ((owner >> i) & 1u) knots[body[i]] = acc[i];
  if (FB && path == 0) knots[0] = acc_base;
  wave_sync();
  if (path == 0 && valid) {
    float sum = 0.f;
    for (int b = 0; b < nb; ++b) sum += knots[b];
    if (!isfinite(sum)) sum = INFINITY;
    I.costs[n] = sum;
  }
  wave_sync();
}

// The item function of an instance's tree.
template <int L, bool FB>
__device__ __forceinline__ void lane_item_of(const DevInst& I, int first, float* smem, const float* x0_in,
                                             const float* nominal_in) {
  const int quads = I.model->path_lanes / 4;
  if (quads == 1) lane_item<1, L, FB>(I, first, smem, x0_in, nominal_in);
  else if (quads == 2) lane_item<2, L, FB>(I, first, smem, x0_in, nominal_in);
  else if (quads == 4) lane_item<4, L, FB>(I, first, smem, x0_in, nominal_in);
  else lane_item<8, L, FB>(I, first, smem, x0_in, nominal_in);
}
template <bool FB>
__device__ __forceinline__ void lane_item_of(const DevInst& I, int first, float* smem, const float* x0_in,
                                             const float* nominal_in) {
  const int len = I.model->path_len;
  if (len <= 3) lane_item_of<3, FB>(I, first, smem, x0_in, nominal_in);
  else if (len <= 4) lane_item_of<4, FB>(I, first, smem, x0_in, nominal_in);
  else lane_item_of<kMaxPath, FB>(I, first, smem, x0_in, nominal_in);
}

}  // namespace mppi
