// mppi_kernels.hip -- gfx950 kernels of the MPPI hot path: the body, chain and
// team schedules' rollouts and the update.  Launches at the body schedule's default
// lane count run the path kernel (mppi_paths.hip) where it takes the tree.
//
// Rollout kernel: G lanes per rollout (G in {4, 8, 16, 32, 64}), 64/G
// rollouts per wavefront, one lane per rigid body (= one actuated joint).
// Spatial quantities use the axes of the instantaneous base frame B (world
// axes for a fixed base) about each body's own joint origin, so a child's
// articulated inertia reaches its parent by a pure translation; the tree is
// swept level by level through LDS.  The kernel fuses, per rollout: counter-based sampling of
// the knots (Alg. 1 sampling step, eq. vel-clamp), then H control steps of
// Hermite reference (eq. hermite_segment), PD law (eq. pd-controller), soft
// contact, articulated-body forward dynamics, running cost (Sec. IV-A) and a
// linearly implicit Euler step, and finally the terminal cost.
//
// Update kernel: a few workgroups per instance, each a slice of its samples; min / max / argmin of the costs,
// min-max normalised softmax weights (eq. softmax_minmax; eq. omega-weights in
// raw mode), the weighted knot average (eq. update-nominal carried to the
// knots) and best-sample tracking (Sec. III-D).  Every reduction runs in a
// fixed order, so results do not depend on launch shape or co-scheduled work.

#include "mppi_step.hpp"

namespace mppi {

// ---------------------------------------------------------------------------
// Fused rollout of one work item: 64/G rollouts of one instance, samples
// w.y .. w.y + 64/G - 1 (those >= N are computed but not stored).
// ---------------------------------------------------------------------------
// steps control steps are simulated (the horizon for a rollout).  With state_out
// set (state prediction, one sample) the state reached is written there and
// no cost is formed.
// Per-step record of a traced rollout (verification of the simulate step of
// Alg. 1, step by step): record h < H holds the state (q, v) at the start of
// control step h, the accelerations of its first physics substep, its running
// cost and its contact mask (bits); record H the final state, zero
// accelerations, the terminal cost and 0.  Layout [q | v | qdd | cost | mask].
template <int G>
__device__ __forceinline__ void trace_record(const DevInst& I, int n, bool valid, int h, int fb, int nq, int nv,
                                             bool is_joint, int j, int b, int l, const StepIO& io, bool with_acc,
                                             float cost, uint32_t mk) {
  if (!valid) return;
  const int slot = I.trace_map[n];
  if (slot < 0) return;
  const int rec = nq + 2 * nv + 2;
  float* r = I.trace + ((size_t)slot * (I.H + 1) + h) * rec;
  if (is_joint) {
    r[(fb ? 7 : 0) + j] = io.q;
    r[nq + (fb ? 6 : 0) + j] = io.v;
    r[nq + nv + (fb ? 6 : 0) + j] = with_acc ? io.qdd : 0.f;
  }
  if (fb && b == 0) {
    for (int k = 0; k < 7; ++k) r[k] = io.bq[k];
    for (int k = 0; k < 6; ++k) {
      r[nq + k] = io.bv[k];
      r[nq + nv + k] = with_acc ? io.ba[k] : 0.f;
    }
  }
  if (l == 0) {
    r[nq + 2 * nv] = cost;
    r[nq + 2 * nv + 1] = __uint_as_float(mk);
  }
}

// x0_in / nominal_in (nullable) replace the instance's staged state and nominal.
// TR: also write the per-step records of traced rollouts (verification kernel).
// per_item: called once per work item in a loop (the persistent form): the lane
// index is passed through an empty asm statement that claims to change it, so
// what derives from it (group, body, LDS addresses) is formed again for each
// item instead of being held live across the loop, which would take the kernel
// past the two-wavefront register budget.
template <int G, int D = 0, bool TR = false, int LEG = 0>
__device__ __attribute__((always_inline)) void rollout_item(const DevInst& I, int first, int group_stride,
                                                            int table_floats, float* smem, int steps,
                                                            float* state_out, const float* x0_in = nullptr,
                                                            const float* nominal_in = nullptr, bool per_item = false) {
  const float* x0 = x0_in ? x0_in : I.x0;
  // issue priority among the wavefronts sharing a SIMD (the server raises it for
  // the trees with the longest per-step chains)
  switch (I.wave_prio) {
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 3: __builtin_amdgcn_s_setprio(3); break;
    default: break;
  }
  int lane = threadIdx.x;
  if (per_item) asm volatile("" : "+v"(lane));
  const int grp = lane / G, l = lane % G;
  const DevModel& M = *I.model;
  float* tab = smem;
  stage_model_table(M, &I, tab, lane, true);
  const int n = first + grp;
  const bool valid = n < I.N;
  float* gs = smem + table_floats + grp * group_stride;
  float* knots = gs + G * kSlot + 16;
  float* red = knots + ((I.E + 3) & ~3);

  // knots of this sample
  if (I.generate) {
    sample_group<G>(M, I, valid ? n : 0, l, knots, valid, tab, nominal_in);
  } else {
    const float* src = I.samples + (size_t)(valid ? n : 0) * I.E;
    for (int e = l; e < I.E; e += G) knots[e] = src[e];
  }
  wave_sync();

  const StepConst sc = load_step_const(M, &I, 0.f);
  const int fb = LEG == 3 ? 0 : (LEG != 0 ? 1 : sc.fb), nb = M.nb, nq = fb ? 7 + M.nu : M.nu;
  const bool body_lane = l < nb;
  const int b = l;
  const bool is_joint = body_lane && !(fb && b == 0);
  const int j = b - fb;
  StepIO io;
  io.q = io.v = 0.f;
  if (is_joint) {
    io.q = x0[(fb ? 7 : 0) + j];
    io.v = x0[nq + (fb ? 6 : 0) + j];
  }
#pragma unroll
  for (int k = 0; k < 7; ++k) io.bq[k] = fb ? x0[k] : 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) io.bv[k] = fb ? x0[nq + k] : 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) io.ba[k] = 0.f;
  io.qref = io.vref = 0.f;
  io.dt = sc.dt;

  BodyConst bc;
  load_body(M, &I, b, body_lane, tab, bc);
  BodyKin kin_kept;  // legged trees: kept across the steps (see BodyKin)
  if constexpr (LEG != 0) init_kin(kin_kept);
  uint32_t* const masks = I.masks;
  const int H = I.H, F = sc.F, F_run = steps * sc.nsub;
  float acc = 0.f;
  StepClock clk;
  // this joint's knots on the current segment, kept in registers across steps
  // where the register budget allows (depth-specialised kernels), else reloaded
  // every step (the same values)
  HermiteSeg hs{0.f, 0.f, 0.f, 0.f};
  int hseg = -1;
  // rare paths laid out of line (MPPI_RARE) where the registers allow it
  constexpr bool kHints = LEG != 0 || D == 6;
  for (int f = 0; f < F_run; ++f) {
    const bool control = clk.sub == 0;
    if (D == 0 || MPPI_RARE(kHints, clk.seg != hseg)) {
      hseg = clk.seg;
      if (is_joint) hs = hermite_segment(knots, sc.K, sc.nu, hseg, j, sc.delta);
    }
    // (lanes without a joint evaluate zero knots and never use the result)
    hermite_eval(hs, (float)clk.rem * sc.inv_F, sc.inv_delta, &io.qref, &io.vref);
    if (sc.spline_mode != 0) io.vref = 0.f;  // position-only variants: zero velocity targets
    physics_step<G, D, LEG>(sc, bc, tab, gs, b, body_lane, io, kin_kept, control);
    if (control) {
      acc += io.cost;
      if (MPPI_RARE(kHints, masks != nullptr)) {
        const uint32_t mk = group_or<G>(io.mask, red, l);
        if (l == 0 && valid) masks[(size_t)n * H + clk.h] = mk;
        if (TR && I.trace) {
          const float c = group_sum<G>(io.cost, red, l);
          trace_record<G>(I, n, valid, clk.h, fb, nq, nq - fb, is_joint, j, b, l, io, true, c, mk);
        }
      }
    }
    // joints (other lanes hold q = qd = qdd = 0)
    io.v = fmaf(io.dt, io.qdd, io.v);
    io.q = fmaf(io.dt, io.v, io.q);
    if (fb) integrate_base_R<kHints>(io.bq, io.bv, io.ba, io.dt, io.Rb);  // every lane: the same base state
    clk.advance<kHints>(sc.K, F, sc.nsub);
  }
  if (state_out) {
    if (valid) {
      if (is_joint) {
        state_out[(fb ? 7 : 0) + j] = io.q;
        state_out[nq + (fb ? 6 : 0) + j] = io.v;
      }
      if (fb && b == 0) {
#pragma unroll
        for (int k = 0; k < 7; ++k) state_out[k] = io.bq[k];
#pragma unroll
        for (int k = 0; k < 6; ++k) state_out[nq + k] = io.bv[k];
      }
    }
    return;
  }

  // terminal cost
  float term_e = 0.f;
  if (sc.cost_kind == 1) {
    if (fb && b == 0) {
      const float T = (float)H * I.dt;
      float e = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float target = (k == 2 && I.targets->terminal_z_abs) ? I.targets->z_terminal : x0[k] + I.targets->v_des[k] * T;
        e += fabsf(io.bq[k] - target);
      }
      acc += I.w_H * e;
      term_e = e;
    }
  } else {
    // end-effector height at x_H
    physics_step<G, D, LEG>(sc, bc, tab, gs, b, body_lane, io, kin_kept, false, true);
    acc += io.cost;
  }
  if (TR && masks && I.trace) {
    const float ct = group_sum<G>(sc.cost_kind == 1 ? I.w_H * term_e : io.cost, red, l);
    trace_record<G>(I, n, valid, H, fb, nq, nq - fb, is_joint, j, b, l, io, false, ct, 0u);
  }
  float S = group_sum<G>(acc, red, l);
  if (l == 0 && valid) {
    if (!isfinite(S)) S = INFINITY;
    I.costs[n] = S;
  }
  wave_sync();
}

// Block = one wavefront; work[blockIdx] = (instance, first sample) or, when work
// is null, instance 0 and sample blockIdx * 64/G.
// D > 0: every instance of the launch is at most D levels deep.
// x0_in / nominal_in (nullable, one instance only): the state and the nominal
// to use instead of the instance's staged copies.
// LEG: every instance of the launch is a legged tree of that kind (see physics_step).
template <int G, int D, int LEG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void rollout_kernel(
    const DevInst* __restrict__ insts, const int2* __restrict__ work, int group_stride, int table_floats,
    const float* __restrict__ x0_in, const float* __restrict__ nominal_in) {
  extern __shared__ float smem[];
  constexpr int R = 64 / G;
  const int2 w = work ? work[blockIdx.x] : make_int2(0, (int)blockIdx.x * R);
  const DevInst& I = insts[w.x];
  rollout_item<G, D, false, LEG>(I, w.y, group_stride, table_floats, smem, I.H, nullptr, x0_in, nominal_in);
}

// The rollout kernel with per-step records of the traced rollouts (same launch
// shape and arithmetic; verification only).
template <int G, int D, int LEG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void rollout_trace_kernel(
    const DevInst* __restrict__ insts, const int2* __restrict__ work, int group_stride, int table_floats) {
  extern __shared__ float smem[];
  constexpr int R = 64 / G;
  const int2 w = work ? work[blockIdx.x] : make_int2(0, (int)blockIdx.x * R);
  const DevInst& I = insts[w.x];
  rollout_item<G, D, true, LEG>(I, w.y, group_stride, table_floats, smem, I.H, nullptr);
}

// State prediction: sample 0 of the instance (its knots read from samples) run
// for `steps` control steps from x0; the state reached goes to state_out.
template <int G>
__global__ __launch_bounds__(64) void predict_kernel(const DevInst* __restrict__ inst, int steps,
                                                     float* __restrict__ state_out, int group_stride,
                                                     int table_floats) {
  extern __shared__ float smem[];
  rollout_item<G>(*inst, 0, group_stride, table_floats, smem, steps, state_out);
}

// The state predictions of a batch of ticks (instances whose trees take G
// lanes), one workgroup per item; the LDS layout is sized for the largest.
template <int G>
__global__ __launch_bounds__(64) void predict_batch_kernel(const PredItem* __restrict__ items, int group_stride,
                                                           int table_floats) {
  extern __shared__ float smem[];
  const PredItem it = items[blockIdx.x];
  rollout_item<G>(*it.inst, 0, group_stride, table_floats, smem, it.steps, it.state_out);
}

// Persistent form: a grid sized to the resident wavefronts; each wavefront takes
// work items from a device counter until the table is exhausted (every wavefront
// reaches that exit).  Which wavefront runs an item does not change its result.
// The same depth and legged-tree specialisations as rollout_kernel, and the same
// two wavefronts per SIMD: the lane index is made opaque once per item (see
// rollout_item's per_item), so nothing derived from it stays live across items.
template <int G, int D, int LEG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void rollout_persistent_kernel(
    const DevInst* __restrict__ insts, const int2* __restrict__ work, int n_items, unsigned int* __restrict__ counter,
    int group_stride, int table_floats) {
  extern __shared__ float smem[];
  for (;;) {
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
    int item = 0;
    if (lane == 0) item = (int)atomicAdd(counter, 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const int2 w = work[item];
    const DevInst& I = insts[w.x];
    rollout_item<G, D, false, LEG>(I, w.y, group_stride, table_floats, smem, I.H, nullptr, nullptr, nullptr, true);
  }
}

// ---------------------------------------------------------------------------
// Team schedule: every chain of the heavy-path decomposition owns a block of B
// lanes (B = 4 or 8, holding the chain's bodies).  The per-body work runs one
// body per lane of its chain's block (PD law, inertia, bias, contacts, running
// cost, integration); the three sweeps run per chain, one body per level, on the
// block's first three lanes together: lane k holds component k of every
// 3-vector and row k of every 3x3 block with its columns in rotated order
// (entry i is column k + i), and the lanes meet through DPP permutations inside
// their quad.  A cyclic relabelling of the axes is a proper rotation, so a cross
// product keeps its form in every lane: (a x b)_k = a_{k+1} b_{k+2} - a_{k+2} b_{k+1}.
// Sums over the three lanes are taken in the order 0, 1, 2 in every lane, so the
// lanes of a team agree bit for bit on every shared scalar.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float qr1(float x) { return qperm<0xC9>(x); }  // component k + 1 (quad_perm 1,2,0,3)
__device__ __forceinline__ float qr2(float x) { return qperm<0xD2>(x); }  // component k + 2 (quad_perm 2,0,1,3)
__device__ __forceinline__ float qsum3(float x) { return (qperm<0x00>(x) + qperm<0x55>(x)) + qperm<0xAA>(x); }

// frame of one body as seen by coordinate lane k: rotated row k of R, p_k, v_k, beta_k
struct TFrame {
  float R[3], p, va, vl, ba, bl;
};

// Forward kinematics of a revolute body (as fk_joint) from the parent's frame P:
// tc = the body's team constants for this lane; outputs the frame O, e_k, ax_k, c_k.
__device__ __forceinline__ void team_fk(const float* tc, float cq, float sq, float qd, const TFrame& P, TFrame& O,
                                        float& e, float& ax, float& ca, float& cl) {
  float C[3], C1[3], C2[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) C[i] = tc[i] + cq * tc[3 + i] + sq * tc[6 + i];
#pragma unroll
  for (int i = 0; i < 3; ++i) { C1[i] = qr1(C[i]); C2[i] = qr2(C[i]); }
  // R = Rl C: entry j = sum_m Rl[k][k+m] C[k+m][k+j]; lane k+m holds C[k+m][.] rotated by its own index
#pragma unroll
  for (int j = 0; j < 3; ++j) O.R[j] = P.R[0] * C[j] + P.R[1] * C1[(j + 2) % 3] + P.R[2] * C2[(j + 1) % 3];
  e = P.R[0] * tc[9] + P.R[1] * tc[10] + P.R[2] * tc[11];
  ax = P.R[0] * tc[12] + P.R[1] * tc[13] + P.R[2] * tc[14];
  O.p = P.p + e;
  const float e1 = qr1(e), e2 = qr2(e);
  const float w1 = qr1(P.va), w2 = qr2(P.va);
  O.va = P.va + ax * qd;
  O.vl = P.vl + (w1 * e2 - w2 * e1);
  const float aq = ax * qd, aq1 = qr1(aq), aq2 = qr2(aq);
  const float va1 = qr1(O.va), va2 = qr2(O.va), vl1 = qr1(O.vl), vl2 = qr2(O.vl);
  ca = va1 * aq2 - va2 * aq1;
  cl = vl1 * aq2 - vl2 * aq1;
  const float b1 = qr1(P.ba), b2 = qr2(P.ba);
  O.ba = P.ba + ca;
  O.bl = P.bl + (b1 * e2 - b2 * e1) + cl;
}

// Articulated-body step of a revolute joint (as backward_joint).  Rows of lane k:
// A[i] = A[k][k+i], B[i] = B[k][k+i], T[i] = B[k+i][k], C[i] = C[k][k+i] of the
// articulated inertia [[A, B], [B^T, C]] and the bias (pa, pl); the carried
// inertia and bias come out in the same form.
__device__ __forceinline__ void team_backward(const float* A, const float* B, const float* T, const float* C,
                                              float pa, float pl, float ax, float e, float ca, float cl, float tau,
                                              float arm, float gain, float& Ua, float& Ul, float& invD, float& u,
                                              float* Ap, float* Bp, float* Tp, float* Cp, float& ppa, float& ppl) {
  const float ax1 = qr1(ax), ax2 = qr2(ax);
  Ua = A[0] * ax + A[1] * ax1 + A[2] * ax2;
  Ul = T[0] * ax + T[1] * ax1 + T[2] * ax2;
  const float Dv = (arm + gain) + qsum3(ax * Ua);
  invD = rcp(Dv);
  u = tau - qsum3(ax * pa);
  // Ia = IA - U W^T, W = U / D
  const float Wa = Ua * invD, Wl = Ul * invD;
  const float Wa1 = qr1(Wa), Wa2 = qr2(Wa), Wl1 = qr1(Wl), Wl2 = qr2(Wl), Ua1 = qr1(Ua), Ua2 = qr2(Ua);
  const float IA_[3] = {A[0] - Ua * Wa, A[1] - Ua * Wa1, A[2] - Ua * Wa2};
  const float IB[3] = {B[0] - Ua * Wl, B[1] - Ua * Wl1, B[2] - Ua * Wl2};
  const float IT[3] = {T[0] - Ua * Wl, T[1] - Ua1 * Wl, T[2] - Ua2 * Wl};
  const float IC[3] = {C[0] - Ul * Wl, C[1] - Ul * Wl1, C[2] - Ul * Wl2};
  // pa = pA + Ia c + U u / D
  const float ca1 = qr1(ca), ca2 = qr2(ca), cl1 = qr1(cl), cl2 = qr2(cl);
  const float iqa = IA_[0] * ca + IA_[1] * ca1 + IA_[2] * ca2 + IB[0] * cl + IB[1] * cl1 + IB[2] * cl2;
  const float iql = IT[0] * ca + IT[1] * ca1 + IT[2] * ca2 + IC[0] * cl + IC[1] * cl1 + IC[2] * cl2;
  const float uD = u * invD;
  const float pa2 = pa + iqa + Ua * uD, pl2 = pl + iql + Ul * uD;
  // carried to the parent origin: B' = B + E C, A' = A - B'E - (BE)^T, C' = C (E = e^x)
  const float e1 = qr1(e), e2 = qr2(e);
  float IC1[3], IC2[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) { IC1[i] = qr1(IC[i]); IC2[i] = qr2(IC[i]); }
#pragma unroll
  for (int i = 0; i < 3; ++i) Bp[i] = IB[i] + e1 * IC2[(i + 1) % 3] - e2 * IC1[(i + 2) % 3];
  Tp[0] = Bp[0];
  Tp[1] = qr1(Bp[2]);
  Tp[2] = qr2(Bp[1]);
  const float er[3] = {e, e1, e2};
  float y[3], z[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    y[j] = Bp[(j + 1) % 3] * er[(j + 2) % 3] - Bp[(j + 2) % 3] * er[(j + 1) % 3];
    z[j] = IB[(j + 1) % 3] * er[(j + 2) % 3] - IB[(j + 2) % 3] * er[(j + 1) % 3];
  }
  Ap[0] = IA_[0] - y[0] - z[0];
  Ap[1] = IA_[1] - y[1] - qr1(z[2]);
  Ap[2] = IA_[2] - y[2] - qr2(z[1]);
#pragma unroll
  for (int i = 0; i < 3; ++i) Cp[i] = IC[i];
  const float p1 = qr1(pl2), p2 = qr2(pl2);
  ppa = pa2 + (e1 * p2 - e2 * p1);
  ppl = pl2;
}

// Accelerations of a revolute joint (as forward_joint) from the parent's a' (ala, all).
__device__ __forceinline__ float team_forward(float ala, float all, float e, float ax, float ca, float cl, float Ua,
                                              float Ul, float invD, float u, float& aa, float& al) {
  const float a1 = qr1(ala), a2 = qr2(ala), e1 = qr1(e), e2 = qr2(e);
  aa = ala + ca;
  al = all + (a1 * e2 - a2 * e1) + cl;
  const float qdd = (u - qsum3(Ua * aa + Ul * al)) * invD;
  aa = aa + ax * qdd;
  return qdd;
}

// Per-lane roles of the team schedule.
struct TeamRole {
  int c, bl, k;            // chain, lane in the chain's block, coordinate lane (0 for lanes past the third)
  int b, slot;             // body of a body lane and its record slot (0 otherwise: never written)
  int cfirst, cpar, pslot; // depth of the chain's first body, its parent (-1: a root) and the parent's slot
  bool body_lane, team;
};

// Body constants a body lane of the team schedule reads.
struct TeamBody {
  float com[3], Ic[6], mass, kp, kd, taumax, q0;
  int c_begin, c_count;
};
__device__ __forceinline__ void load_team_body(const DevModel& M, const DevInst* I, const TeamRole& r, TeamBody& c) {
  const int bb = r.b;
  const int j = bb - M.fb;
  const bool joint = r.body_lane && j >= 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) c.com[k] = M.com[bb][k];
#pragma unroll
  for (int k = 0; k < 6; ++k) c.Ic[k] = M.Ic[bb][k];
  c.mass = M.mass[bb];
  c.kp = joint ? M.kp[j] : 0.f;
  c.kd = joint ? M.kd[j] : 0.f;
  c.taumax = joint ? M.taumax[j] : 0.f;
  c.q0 = (joint && I && I->cost_kind == 1) ? I->q0[j] : 0.f;
  c.c_begin = M.c_begin[bb];
  c.c_count = r.body_lane ? M.c_count[bb] : 0;
}

// Stage the team constants (by slot) and the table of the slot of chain c's body at
// depth d (or -1) after the model table.
__device__ __forceinline__ void stage_team_table(const DevModel& M, float* tab, int lane) {
  float* tt = tab + body_table_floats(M.nc);
  const int n = M.nb * kTeamRow;
  for (int i = lane; i < n; i += 64) {
    const int b = i / kTeamRow, w = i % kTeamRow;
    tt[M.team_slot[b] * kTeamSlot + (w / 16) * kTeamK + (w % 16)] = M.team_rows[b][w];
  }
  int* tcb = reinterpret_cast<int*>(tt + M.team_slots * kTeamSlot);
  for (int i = lane; i < kMaxChains * kMaxLevels; i += 64) {
    const int bb = M.chain_body[i / kMaxLevels][i % kMaxLevels];
    tcb[i] = bb >= 0 ? M.team_slot[bb] : -1;
  }
  wave_sync();
}

__device__ __forceinline__ void get16(const float* s, float* d) {
  const float4 a = get4(s), b = get4(s + 4), c = get4(s + 8), e = get4(s + 12);
  d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w; d[4] = b.x; d[5] = b.y; d[6] = b.z; d[7] = b.w;
  d[8] = c.x; d[9] = c.y; d[10] = c.z; d[11] = c.w; d[12] = e.x; d[13] = e.y; d[14] = e.z; d[15] = e.w;
}

// What a coordinate lane reads for one level of the backward sweep (loaded a
// level ahead; zeros where the chain has no body at that depth).
struct TeamBwdIn {
  float ir[16], lr[4], tau, gain, arm;
  uint32_t side;
  bool act;
};
__device__ __forceinline__ int team_load_bwd(const TeamRole& r, const int* tcb, const float* tt, const float* ir,
                                             const float* lr, const float* br, int d, int k, TeamBwdIn& o) {
  const int s = r.team ? tcb[r.c * kMaxLevels + d] : -1;
  o.act = s >= 0;
  if (o.act) {
    get16(ir + s * kTeamSlot + k * kTeamK, o.ir);
    const float4 l4 = get4(lr + s * kFrSlot + k * 8);
    o.lr[0] = l4.x; o.lr[1] = l4.y; o.lr[2] = l4.z; o.lr[3] = l4.w;
    const float4 b4 = get4(br + s * 8);
    o.tau = b4.w;
    o.gain = br[s * 8 + 4];
    o.arm = tt[s * kTeamSlot + 15];
    o.side = (uint32_t)__float_as_int(tt[s * kTeamSlot + kTeamK + 15]);
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) o.ir[q] = 0.f;
    o.lr[0] = o.lr[1] = o.lr[2] = o.lr[3] = 0.f;
    o.tau = o.gain = o.arm = 0.f;
    o.side = 0u;
  }
  return s;
}
// the same for the forward sweep
struct TeamFwdIn {
  float lr[8];
  uint32_t side;
  bool act;
};
__device__ __forceinline__ int team_load_fwd(const TeamRole& r, const int* tcb, const float* tt, const float* lr,
                                             int d, int k, TeamFwdIn& o) {
  const int s = r.team ? tcb[r.c * kMaxLevels + d] : -1;
  o.act = s >= 0;
  if (o.act) {
    const float4 l0 = get4(lr + s * kFrSlot + k * 8), l1 = get4(lr + s * kFrSlot + k * 8 + 4);
    o.lr[0] = l0.x; o.lr[1] = l0.y; o.lr[2] = l0.z; o.lr[3] = l0.w;
    o.lr[4] = l1.x; o.lr[5] = l1.y; o.lr[6] = l1.z; o.lr[7] = l1.w;
    o.side = (uint32_t)__float_as_int(tt[s * kTeamSlot + kTeamK + 15]);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) o.lr[q] = 0.f;
    o.side = 0u;
  }
  return s;
}

// One physics step of the team schedule (same stages and formulas as physics_step):
// tt = team constants and tcb = chain-body table in LDS.  Every coordinate-lane
// computation runs with all lanes active (the DPP permutations need them); the
// lanes of a level without a body compute on zeros and store nothing.
template <int D>
__device__ __attribute__((always_inline)) void team_step(const StepConst& sc, const TeamBody& tb, const float* tab,
                                                         const float* tt, const int* tcb,
                          float* __restrict__ gs, const TeamLayout& L, const TeamRole& r, StepIO& io, bool want_cost,
                          bool terminal = false) {
  float* br = gs + L.br;
  float* fr = gs + L.fr;
  float* lr = gs + L.lr;
  float* ir = gs + L.ir;
  float* pr = gs + L.pr;
  float* ar = gs + L.ar;
  float* bs = gs + L.bs;
  float* gr = gs + L.gr;
  const int fb = sc.fb, b = r.b, k = r.k, sl = r.slot;
  const bool is_base = r.body_lane && fb && b == 0;
  const bool is_joint = r.body_lane && !is_base;
  const int maxd = D > 0 ? D : sc.max_depth;

  // ---- PD law, joint trigonometry, frame B
  float tau = 0.f, gain = 0.f;
  if (is_joint) pd_law(tb.kp, tb.kd, tb.taumax, io.dt, io.q, io.v, io.qref, io.vref, tau, gain);
  io.tau = tau;
  float base_term = 0.f;
  if (want_cost && is_base && sc.cost_kind == 1) base_term = base_cost_term(sc, io.bq);
  if (is_joint) {
    float cq, sq;
    sincosf(io.q, &sq, &cq);
    put4(br + sl * 8, cq, sq, io.v, tau);
    br[sl * 8 + 4] = gain;
  }
  if (is_base) {
    float R[9];
    quat_R(io.bq + 3, R);
#pragma unroll
    for (int q = 0; q < 9; ++q) bs[q] = R[q];
    bs[9] = io.bq[0]; bs[10] = io.bq[1]; bs[11] = io.bq[2];
#pragma unroll
    for (int q = 0; q < 6; ++q) bs[12 + q] = io.bv[q];
  }
  if (!fb && r.c == 0 && r.bl == 0) {
#pragma unroll
    for (int q = 0; q < 9; ++q) bs[q] = (q % 4 == 0) ? 1.f : 0.f;
#pragma unroll
    for (int q = 9; q < 18; ++q) bs[q] = 0.f;
  }
  wave_sync();

  // ---- forward kinematics, one body of each chain per level, on the chain's coordinate lanes
  TFrame F;  // this chain's previous body (the base for chain 0 of a floating base)
  F.R[0] = 1.f; F.R[1] = 0.f; F.R[2] = 0.f;
  F.p = 0.f; F.ba = 0.f; F.bl = 0.f;
  F.va = fb ? bs[12 + k] : 0.f;
  F.vl = fb ? bs[15 + k] : 0.f;
#pragma unroll kLevelUnroll<D>
  for (int d = 1; d <= maxd; ++d) {
    const int sd = r.team ? tcb[r.c * kMaxLevels + d] : -1;  // slot of this chain's body at depth d
    const bool act = sd >= 0;
    float tc[16];
    float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (act) {
      get16(tt + sd * kTeamSlot + k * kTeamK, tc);
      s4 = get4(br + sd * 8);
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q) tc[q] = 0.f;
    }
    TFrame P = F;
    if (act && d == r.cfirst) {  // a chain's first body: its parent is elsewhere
      if (r.cpar < 0) {
        P.R[0] = 1.f; P.R[1] = 0.f; P.R[2] = 0.f;
        P.p = P.va = P.vl = P.ba = P.bl = 0.f;
      } else if (fb && r.cpar == 0) {
        P.R[0] = 1.f; P.R[1] = 0.f; P.R[2] = 0.f;
        P.p = 0.f; P.va = bs[12 + k]; P.vl = bs[15 + k]; P.ba = 0.f; P.bl = 0.f;
      } else {
        const float4 f0 = get4(fr + r.pslot * kFrSlot + k * 8), f1 = get4(fr + r.pslot * kFrSlot + k * 8 + 4);
        P.R[0] = f0.x; P.R[1] = f0.y; P.R[2] = f0.z; P.p = f0.w;
        P.va = f1.x; P.vl = f1.y; P.ba = f1.z; P.bl = f1.w;
      }
    }
    TFrame O;
    float e, ax, ca, cl;
    team_fk(tc, s4.x, s4.y, s4.z, P, O, e, ax, ca, cl);
    if (act) {
      put4(fr + sd * kFrSlot + k * 8, O.R[0], O.R[1], O.R[2], O.p);
      put4(fr + sd * kFrSlot + k * 8 + 4, O.va, O.vl, O.ba, O.bl);
      put4(lr + sd * kFrSlot + k * 8, e, ax, ca, cl);
    }
    F = O;
    wave_sync();
  }

  // ---- every body lane: its frame, rigid inertia, bias force, contacts and running cost
  // (every lane reads its slot's record, so the values are chosen, not the memory)
  float R[9], p[3], v[6], beta[6];
#pragma unroll
  for (int kk = 0; kk < 3; ++kk) {
    const float4 f0 = get4(fr + sl * kFrSlot + kk * 8), f1 = get4(fr + sl * kFrSlot + kk * 8 + 4);
    R[kk * 3 + kk] = is_joint ? f0.x : 1.f;
    R[kk * 3 + (kk + 1) % 3] = is_joint ? f0.y : 0.f;
    R[kk * 3 + (kk + 2) % 3] = is_joint ? f0.z : 0.f;
    p[kk] = is_joint ? f0.w : 0.f;
    v[kk] = is_joint ? f1.x : bs[12 + kk];  // the base: its twist (frame B)
    v[3 + kk] = is_joint ? f1.y : bs[15 + kk];
    beta[kk] = is_joint ? f1.z : 0.f;
    beta[3 + kk] = is_joint ? f1.w : 0.f;
  }
  float Rb[9], pb[3];
#pragma unroll
  for (int q = 0; q < 9; ++q) Rb[q] = bs[q];
  pb[0] = bs[9]; pb[1] = bs[10]; pb[2] = bs[11];
  float lane_cost = 0.f;
  if (terminal) {
    if (r.body_lane && sc.cost_kind == 0 && b == sc.ee_body) {
      const float dz = ee_height_error(R, p, sc.ee_pos, Rb, pb, sc.z_des);
      lane_cost = sc.w_ee * dz * dz;
    }
    io.cost = lane_cost;
    io.mask = 0u;
    wave_sync();
    return;
  }
  const float g = sc.g;
  const float agl[3] = {-g * Rb[6], -g * Rb[7], -g * Rb[8]};
  uint32_t mask = 0u;
  if (r.body_lane) {
    float IA[21], pA[6];
    if (is_base) {
      const float eye[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
      body_inertia(eye, tb.com, tb.Ic, tb.mass, IA);
    } else {
      body_inertia(R, tb.com, tb.Ic, tb.mass, IA);
    }
    bias_force(IA, v, pA);
    const int c0 = tb.c_begin, cn = tb.c_count;
    for (int ci = c0; ci < c0 + cn; ++ci) {
      const float* ct = tab + kTabContacts + ci * kCt;
      float vw[3], fw[3];
      const float fn = contact_point(ct, R, p, v, beta, Rb, pb, agl, io.dt, sc.law, IA, pA, vw, fw);
      if (fn > 0.f) mask |= 1u << __float_as_int(ct[4]);
      if (want_cost && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], lane_cost);
    }
    if (want_cost) body_cost(sc, b, is_base, is_joint, base_term, io.q, tb.q0, tau, R, p, Rb, pb, lane_cost);
    // rows for the coordinate lanes
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      float* d = ir + sl * kTeamSlot + kk * kTeamK;
      const int c1 = (kk + 1) % 3, c2 = (kk + 2) % 3;
      put4(d, IA[SI(kk, kk)], IA[SI(kk, c1)], IA[SI(kk, c2)], IA[SI(kk, 3 + kk)]);
      put4(d + 4, IA[SI(kk, 3 + c1)], IA[SI(kk, 3 + c2)], IA[SI(kk, 3 + kk)], IA[SI(c1, 3 + kk)]);
      put4(d + 8, IA[SI(c2, 3 + kk)], IA[SI(3 + kk, 3 + kk)], IA[SI(3 + kk, 3 + c1)], IA[SI(3 + kk, 3 + c2)]);
      put4(d + 12, pA[kk], pA[3 + kk], 0.f, 0.f);
    }
  }
  io.cost = lane_cost;
  io.mask = mask;
  wave_sync();

  // ---- backward sweep, leaves to root, on the coordinate lanes
  float cA[3] = {0.f, 0.f, 0.f}, cB[3] = {0.f, 0.f, 0.f}, cT[3] = {0.f, 0.f, 0.f}, cC[3] = {0.f, 0.f, 0.f};
  float cpa = 0.f, cpl = 0.f;  // carried by this chain's deeper body

#pragma unroll kLevelUnrollRoot<D>
  for (int d = maxd; d >= 0; --d) {
    TeamBwdIn cur;
    const int sd = team_load_bwd(r, tcb, tt, ir, lr, br, d, k, cur);
    const bool act = cur.act;
    float A[3] = {cur.ir[0], cur.ir[1], cur.ir[2]}, B[3] = {cur.ir[3], cur.ir[4], cur.ir[5]};
    float T[3] = {cur.ir[6], cur.ir[7], cur.ir[8]}, C[3] = {cur.ir[9], cur.ir[10], cur.ir[11]};
    float pa = cur.ir[12], pl = cur.ir[13];
    const float e = cur.lr[0], ax = cur.lr[1], ca = cur.lr[2], cl = cur.lr[3];
    const float tau_d = cur.tau, gain_d = cur.gain, arm_d = cur.arm;
    uint32_t side = cur.side;
    const bool deeper = act && d < maxd && tcb[r.c * kMaxLevels + d + 1] >= 0;  // the chain goes on
    if (deeper) {
#pragma unroll
      for (int i = 0; i < 3; ++i) { A[i] += cA[i]; B[i] += cB[i]; T[i] += cT[i]; C[i] += cC[i]; }
      pa += cpa;
      pl += cpl;
    }
    while (side) {
      const int c2 = __builtin_ctz(side);
      side &= side - 1u;
      float q[16];
      get16(pr + c2 * kTeamSlot + k * kTeamK, q);
      A[0] += q[0]; A[1] += q[1]; A[2] += q[2]; B[0] += q[3];
      B[1] += q[4]; B[2] += q[5]; T[0] += q[6]; T[1] += q[7];
      T[2] += q[8]; C[0] += q[9]; C[1] += q[10]; C[2] += q[11];
      pa += q[12]; pl += q[13];
    }
    float Ua, Ul, invD, u, nA[3], nB[3], nT[3], nC[3], npa, npl;
    team_backward(A, B, T, C, pa, pl, ax, e, ca, cl, tau_d, arm_d, gain_d, Ua, Ul, invD, u, nA, nB, nT, nC, npa,
                  npl);
    const bool base_here = act && fb && d == 0;
    if (act && !base_here) {
      put4(lr + sd * kFrSlot + k * 8 + 4, Ua, Ul, invD, u);
      if (d == r.cfirst && r.cpar >= 0) {
        float* q = pr + r.c * kTeamSlot + k * kTeamK;
        put4(q, nA[0], nA[1], nA[2], nB[0]);
        put4(q + 4, nB[1], nB[2], nT[0], nT[1]);
        put4(q + 8, nT[2], nC[0], nC[1], nC[2]);
        put4(q + 12, npa, npl, 0.f, 0.f);
      }
    }
    if (base_here) {  // the floating base: its rows go to the solve
      float* q = gr + k * kTeamK;
      put4(q, A[0], A[1], A[2], B[0]);
      put4(q + 4, B[1], B[2], T[0], T[1]);
      put4(q + 8, T[2], C[0], C[1], C[2]);
      put4(q + 12, pa, pl, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) { cA[i] = nA[i]; cB[i] = nB[i]; cT[i] = nT[i]; cC[i] = nC[i]; }
    cpa = npa;
    cpl = npl;
    wave_sync();
  }

  // ---- root: floating base solves IA0 a0' = -pA0
  if (is_base) {
    float IA[21], pA[6], a0[6];
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      const float* q = gr + kk * kTeamK;
      const int c1 = (kk + 1) % 3, c2 = (kk + 2) % 3;
      IA[SI(kk, kk)] = q[0];
      if (kk <= c1) IA[SI(kk, c1)] = q[1];
      if (kk <= c2) IA[SI(kk, c2)] = q[2];
      IA[SI(kk, 3 + kk)] = q[3]; IA[SI(kk, 3 + c1)] = q[4]; IA[SI(kk, 3 + c2)] = q[5];
      IA[SI(3 + kk, 3 + kk)] = q[9];
      if (kk <= c1) IA[SI(3 + kk, 3 + c1)] = q[10];
      if (kk <= c2) IA[SI(3 + kk, 3 + c2)] = q[11];
      pA[kk] = q[12];
      pA[3 + kk] = q[13];
    }
    base_solve(IA, pA, a0);
#pragma unroll
    for (int q = 0; q < 6; ++q) bs[18 + q] = a0[q];
    io.ba[0] = a0[0]; io.ba[1] = a0[1]; io.ba[2] = a0[2];
    io.ba[3] = a0[3] + agl[0]; io.ba[4] = a0[4] + agl[1]; io.ba[5] = a0[5] + agl[2];
  }
  wave_sync();

  // ---- forward sweep, root to leaves, on the coordinate lanes
  float Fa = fb ? bs[18 + k] : 0.f, Fl = fb ? bs[21 + k] : 0.f;  // chain 0 starts at the base
#pragma unroll kLevelUnroll<D>
  for (int d = 1; d <= maxd; ++d) {
    TeamFwdIn cur;
    const int sd = team_load_fwd(r, tcb, tt, lr, d, k, cur);
    const bool act = cur.act;
    const float* lf = cur.lr;
    const uint32_t side = cur.side;
    float ala = Fa, all = Fl;
    if (act && d == r.cfirst) {
      if (r.cpar < 0) {  // fixed world: a' = -a_g = (0, 0, 0, 0, 0, g)
        ala = 0.f;
        all = k == 2 ? g : 0.f;
      } else if (fb && r.cpar == 0) {
        ala = bs[18 + k];
        all = bs[21 + k];
      } else {
        const float2 a2 = *reinterpret_cast<const float2*>(ar + r.pslot * 8 + k * 2);
        ala = a2.x;
        all = a2.y;
      }
    }
    float aa, al;
    const float qdd = team_forward(ala, all, lf[0], lf[1], lf[2], lf[3], lf[4], lf[5], lf[6], lf[7], aa, al);
    if (act) {
      if (side != 0u) *reinterpret_cast<float2*>(ar + sd * 8 + k * 2) = make_float2(aa, al);
      if (k == 0) br[sd * 8 + 5] = qdd;
    }
    Fa = aa;
    Fl = al;
    wave_sync();
  }
  io.qdd = is_joint ? br[sl * 8 + 5] : 0.f;
}

// Fused rollout of one work item on the team schedule (as rollout_item, per_item
// included).
template <int G, int D = 0>
__device__ __attribute__((always_inline)) void team_item(const DevInst& I, int first, int group_stride,
                                                         int table_floats, float* smem, bool per_item = false) {
  int lane = threadIdx.x;
  if (per_item) asm volatile("" : "+v"(lane));
  const int grp = lane / G, l = lane % G;
  const DevModel& M = *I.model;
  float* tab = smem;
  stage_model_table(M, &I, tab, lane);
  stage_team_table(M, tab, lane);
  const float* tt = tab + body_table_floats(M.nc);
  const int* tcb = reinterpret_cast<const int*>(tt + M.team_slots * kTeamSlot);
  const int n = first + grp;
  const bool valid = n < I.N;
  const TeamLayout L = team_layout(G, M.team_slots, I.E, M.n_chains);
  float* gs = smem + table_floats + grp * group_stride;
  float* knots = gs + L.knots;
  float* red = gs + L.red;

  if (I.generate) {
    sample_group<G>(M, I, valid ? n : 0, l, knots, valid, tab);
  } else {
    const float* src = I.samples + (size_t)(valid ? n : 0) * I.E;
    for (int e = l; e < I.E; e += G) knots[e] = src[e];
  }
  wave_sync();

  const StepConst sc = load_step_const(M, &I, 0.f);
  TeamRole r;
  const int B = M.team_block;
  r.c = l / B;
  r.bl = l % B;
  const bool in_chain = r.c < M.n_chains;
  r.team = in_chain && r.bl < 3;
  r.k = r.bl < 3 ? r.bl : 0;
  r.cfirst = in_chain ? M.chain_first[r.c] : 0;
  r.cpar = in_chain ? M.chain_parent[r.c] : -1;
  r.body_lane = in_chain && r.bl < M.chain_len[r.c];
  r.b = r.body_lane ? M.chain_body[r.c][r.cfirst + r.bl] : 0;
  r.slot = r.body_lane ? M.team_slot[r.b] : 0;
  r.pslot = r.cpar >= 0 ? M.team_slot[r.cpar] : 0;
  const int fb = sc.fb, nq = fb ? 7 + M.nu : M.nu;
  const int b = r.b;
  const bool is_joint = r.body_lane && !(fb && b == 0);
  const bool is_base = r.body_lane && fb && b == 0;
  const int j = b - fb;
  StepIO io;
  io.q = io.v = 0.f;
  if (is_joint) {
    io.q = I.x0[(fb ? 7 : 0) + j];
    io.v = I.x0[nq + (fb ? 6 : 0) + j];
  }
#pragma unroll
  for (int q = 0; q < 7; ++q) io.bq[q] = fb ? I.x0[q] : 0.f;
#pragma unroll
  for (int q = 0; q < 6; ++q) io.bv[q] = fb ? I.x0[nq + q] : 0.f;
#pragma unroll
  for (int q = 0; q < 6; ++q) io.ba[q] = 0.f;
  io.qref = io.vref = 0.f;
  io.dt = sc.dt;

  TeamBody tb;
  load_team_body(M, &I, r, tb);
  uint32_t* const masks = I.masks;
  const int H = I.H, F = sc.F, F_run = H * sc.nsub;
  float acc = 0.f;
  StepClock clk;
  HermiteSeg hs{0.f, 0.f, 0.f, 0.f};
  int hseg = -1;
  for (int f = 0; f < F_run; ++f) {
    const bool control = clk.sub == 0;
    if (clk.seg != hseg) {
      hseg = clk.seg;
      if (is_joint) hs = hermite_segment(knots, sc.K, sc.nu, hseg, j, sc.delta);
    }
    if (is_joint) {
      hermite_eval(hs, (float)clk.rem * sc.inv_F, sc.inv_delta, &io.qref, &io.vref);
      if (sc.spline_mode != 0) io.vref = 0.f;
    }
    team_step<D>(sc, tb, tab, tt, tcb, gs, L, r, io, control);
    if (control) {
      acc += io.cost;
      if (masks) {
        const uint32_t mk = group_or<G>(io.mask, red, l);
        if (l == 0 && valid) masks[(size_t)n * H + clk.h] = mk;
      }
    }
    if (is_joint) {
      io.v = fmaf(io.dt, io.qdd, io.v);
      io.q = fmaf(io.dt, io.v, io.q);
    }
    if (is_base) integrate_base(io.bq, io.bv, io.ba, io.dt);
    clk.advance(sc.K, F, sc.nsub);
  }
  // terminal cost
  if (sc.cost_kind == 1) {
    if (is_base) {
      const float T = (float)H * I.dt;
      float e = 0.f;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float target = (q == 2 && I.targets->terminal_z_abs) ? I.targets->z_terminal : I.x0[q] + I.targets->v_des[q] * T;
        e += fabsf(io.bq[q] - target);
      }
      acc += I.w_H * e;
    }
  } else {
    team_step<D>(sc, tb, tab, tt, tcb, gs, L, r, io, false, true);
    acc += io.cost;
  }
  float S = group_sum<G>(acc, red, l);
  if (l == 0 && valid) {
    if (!isfinite(S)) S = INFINITY;
    I.costs[n] = S;
  }
  wave_sync();
}

// Block = one wavefront; work[blockIdx] = (instance, first sample) or, when work
// is null, instance 0 and sample blockIdx * 64/G.
template <int G, int D>
__global__ __launch_bounds__(64) void team_kernel(const DevInst* __restrict__ insts, const int2* __restrict__ work,
                                                  int group_stride, int table_floats) {
  extern __shared__ float smem[];
  constexpr int R = 64 / G;
  const int2 w = work ? work[blockIdx.x] : make_int2(0, (int)blockIdx.x * R);
  const DevInst& I = insts[w.x];
  team_item<G, D>(I, w.y, group_stride, table_floats, smem);
}

// Persistent form (as rollout_persistent_kernel).
template <int G>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void team_persistent_kernel(
    const DevInst* __restrict__ insts, const int2* __restrict__ work, int n_items, unsigned int* __restrict__ counter,
    int group_stride, int table_floats) {
  extern __shared__ float smem[];
  for (;;) {
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
    int item = 0;
    if (lane == 0) item = (int)atomicAdd(counter, 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const int2 w = work[item];
    const DevInst& I = insts[w.x];
    team_item<G>(I, w.y, group_stride, table_floats, smem, true);
  }
}

// ---------------------------------------------------------------------------
// Chain schedule: one lane per kinematic chain (heavy-path decomposition of
// the tree), 64/GC rollouts per wavefront.  Per step a lane walks its chain
// root to leaf (Hermite reference, PD law, kinematics), leaf to root (inertia,
// bias, contacts, running cost, articulated-body pass, root solve) and root to
// leaf again (accelerations, integration).  Lanes meet only where a chain
// hangs off another chain's body, through attach and publish slots in LDS; a
// level loop with one body per lane keeps every parent ahead of its children.
// Each body goes through the same helpers in the same order as in the body
// schedule (children added in child-list order, costs summed per body in body
// order), so the two schedules give identical results.
//
// LDS: the model table (body rows, chain bodies, contact rows) once per
// wavefront, then one region per rollout group:
//   rec[nb][kRec]  per body: [0,9) R [9,12) p [12,18) v [18,24) beta [24,27) e
//                  [27,30) ax 30 tau 31 gain; after the backward pass [0,6) U
//                  6 1/D 7 u [8,14) c; and, kept across steps, 32 q 33 qd
//                  34 running cost of the body
//   base[16]       world rotation (9) and position (3) of frame B
//   knots[E]       this rollout's knots
//   pub[nch][kPub] articulated inertia and bias a chain's first body hands to
//                  its parent on another chain
//   att[natt][kAtt] frame (R p v beta) and a' of a body other chains hang off
//   red[GC]        reduction scratch
// ---------------------------------------------------------------------------
__device__ __forceinline__ int ibits(float x) { return __float_as_int(x); }

// Root-to-leaf pass: PD law (unless terminal) and kinematics of every body of
// this lane's chain; publishes frames other chains hang off.
__device__ __forceinline__ void chain_fk(const StepConst& sc, const float* rows, const int* cbody, float* rec,
                                         float* bas, const float* knots, float* att, bool act, int c, int cfirst,
                                         int catt, int nlev, int seg, int rem, bool terminal, const float* bq,
                                         const float* bv) {
  const int fb = sc.fb;
  const float dt = sc.dt;
  float fR[9], fp[3], fv[6], fbt[6];  // frame of this chain's previous body
  for (int d = 0; d < nlev; ++d) {
    const int b = act ? cbody[c * kMaxLevels + d] : -1;
    if (b >= 0) {
      const float* rw = rows + b * kRow;
      float* r = rec + b * kRec;
      if (fb && b == 0) {
        float Rw[9];
        quat_R(bq + 3, Rw);
#pragma unroll
        for (int k = 0; k < 9; ++k) bas[k] = Rw[k];
        bas[9] = bq[0]; bas[10] = bq[1]; bas[11] = bq[2];
#pragma unroll
        for (int k = 0; k < 9; ++k) fR[k] = (k % 4 == 0) ? 1.f : 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) fp[k] = 0.f;
#pragma unroll
        for (int k = 0; k < 6; ++k) { fv[k] = bv[k]; fbt[k] = 0.f; }
#pragma unroll
        for (int k = 0; k < 9; ++k) r[k] = fR[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) r[9 + k] = 0.f;
#pragma unroll
        for (int k = 0; k < 6; ++k) { r[12 + k] = fv[k]; r[18 + k] = 0.f; }
#pragma unroll
        for (int k = 24; k < 32; ++k) r[k] = 0.f;
      } else {
        const int j = b - fb;
        const float q = r[32], qd = r[33];
        float tau = 0.f, gain = 0.f;
        if (!terminal) {
          float qref, vref;
          hermite(knots, sc.K, sc.nu, sc.inv_F, sc.delta, sc.inv_delta, seg, rem, j, &qref, &vref);
          if (sc.spline_mode != 0) vref = 0.f;
          pd_law(rw[row::kp], rw[row::kd], rw[row::taumax], dt, q, qd, qref, vref, tau, gain);
        }
        float Rl[9], pl[3], vl[6], bl[6];
        if (d == cfirst) {
          if (catt >= 0) {
            const float* a = att + catt * kAtt;
#pragma unroll
            for (int k = 0; k < 9; ++k) Rl[k] = a[k];
#pragma unroll
            for (int k = 0; k < 3; ++k) pl[k] = a[9 + k];
#pragma unroll
            for (int k = 0; k < 6; ++k) { vl[k] = a[12 + k]; bl[k] = a[18 + k]; }
          } else {
#pragma unroll
            for (int k = 0; k < 9; ++k) Rl[k] = (k % 4 == 0) ? 1.f : 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) pl[k] = 0.f;
#pragma unroll
            for (int k = 0; k < 6; ++k) { vl[k] = 0.f; bl[k] = 0.f; }
          }
        } else {
#pragma unroll
          for (int k = 0; k < 9; ++k) Rl[k] = fR[k];
#pragma unroll
          for (int k = 0; k < 3; ++k) pl[k] = fp[k];
#pragma unroll
          for (int k = 0; k < 6; ++k) { vl[k] = fv[k]; bl[k] = fbt[k]; }
        }
        float cq, sq, C[9];
        sincosf(q, &sq, &cq);
        joint_rotation(rw + row::P, cq, sq, C);
        float e[3], ax[3], cv[6];
        fk_joint(Rl, pl, vl, bl, C, rw + row::p_tree, rw + row::axis_p, qd, fR, fp, e, ax, fv, cv, fbt);
#pragma unroll
        for (int k = 0; k < 9; ++k) r[k] = fR[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) { r[9 + k] = fp[k]; r[24 + k] = e[k]; r[27 + k] = ax[k]; }
#pragma unroll
        for (int k = 0; k < 6; ++k) { r[12 + k] = fv[k]; r[18 + k] = fbt[k]; }
        r[30] = tau;
        r[31] = gain;
      }
      const int aid = ibits(rw[row::att]);
      if (aid >= 0) {
        float* a = att + aid * kAtt;
#pragma unroll
        for (int k = 0; k < 9; ++k) a[k] = fR[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) a[9 + k] = fp[k];
#pragma unroll
        for (int k = 0; k < 6; ++k) { a[12 + k] = fv[k]; a[18 + k] = fbt[k]; }
      }
    }
    wave_sync();
  }
}

// Leaf-to-root pass: inertia, bias, contacts and running cost of each body,
// then the articulated-body step; the floating base solves for its
// acceleration.  Returns this lane's contact activity bits.
__device__ __forceinline__ uint32_t chain_backward(const StepConst& sc, const float* tab, const float* rows,
                                                   const int* cbody, float* rec, const float* bas, float* pub,
                                                   float* att, bool act, int c, int cfirst, int catt, int nlev,
                                                   bool want_cost, float base_term, float* ba, float* ca) {
  const int fb = sc.fb;
  const float dt = sc.dt;
  const float g = sc.g;
  uint32_t mask = 0u;
  float cI[21], cp[6];  // articulated inertia and bias of this chain's deeper body, at this body's origin
  float Rb[9], pb[3];
#pragma unroll
  for (int k = 0; k < 9; ++k) Rb[k] = bas[k];
  pb[0] = bas[9]; pb[1] = bas[10]; pb[2] = bas[11];
  const float agl[3] = {-g * Rb[6], -g * Rb[7], -g * Rb[8]};
  for (int d = nlev - 1; d >= 0; --d) {
    const int b = act ? cbody[c * kMaxLevels + d] : -1;
    if (b >= 0) {
      const float* rw = rows + b * kRow;
      float* r = rec + b * kRec;
      const bool is_base = fb && b == 0;
      float R[9], p[3], v[6], beta[6];
#pragma unroll
      for (int k = 0; k < 9; ++k) R[k] = r[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) p[k] = r[9 + k];
#pragma unroll
      for (int k = 0; k < 6; ++k) { v[k] = r[12 + k]; beta[k] = r[18 + k]; }
      const float tau = r[30], gain = r[31];
      float IA[21], pA[6];
      if (is_base) {
        const float eye[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
        body_inertia(eye, rw + row::com, rw + row::Ic, rw[row::mass], IA);
      } else {
        body_inertia(R, rw + row::com, rw + row::Ic, rw[row::mass], IA);
      }
      bias_force(IA, v, pA);
      float lane_cost = 0.f;
      const int c0 = ibits(rw[row::c_begin]), cn = ibits(rw[row::c_count]);
      for (int ci = c0; ci < c0 + cn; ++ci) {
        const float* ct = tab + kTabContacts + ci * kCt;
        float vw[3], fw[3];
        const float fn = contact_point(ct, R, p, v, beta, Rb, pb, agl, dt, sc.law, IA, pA, vw, fw);
        if (fn > 0.f) mask |= 1u << ibits(ct[4]);
        if (want_cost && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], lane_cost);
      }
      if (want_cost) {
        body_cost(sc, b, is_base, !is_base, base_term, is_base ? 0.f : r[32], rw[row::q0], tau, R, p, Rb, pb,
                  lane_cost);
        r[34] += lane_cost;
      }
      // children in child-list order: the chain's own child from registers, others from their publish slots
      const int nch = ibits(rw[row::n_child]), heavy = ibits(rw[row::heavy]);
      for (int k = 0; k < nch; ++k) {
        const int ch = ibits(rw[row::child + k]);
        if (ch == heavy) {
#pragma unroll
          for (int q = 0; q < 21; ++q) IA[q] += cI[q];
#pragma unroll
          for (int q = 0; q < 6; ++q) pA[q] += cp[q];
        } else {
          const float* s = pub + ibits(rows[ch * kRow + row::chain]) * kPub;
#pragma unroll
          for (int q = 0; q < 21; ++q) IA[q] += s[q];
#pragma unroll
          for (int q = 0; q < 6; ++q) pA[q] += s[21 + q];
        }
      }
      if (!is_base) {
        float e[3], ax[3], cv[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) { e[k] = r[24 + k]; ax[k] = r[27 + k]; }
        vel_product(v, ax, r[33], cv);
        float U[6], invD, u, Ip[21], pp[6];
        backward_joint(IA, pA, ax, cv, e, tau, rw[row::arm], gain, U, invD, u, Ip, pp);
#pragma unroll
        for (int k = 0; k < 6; ++k) { r[k] = U[k]; r[8 + k] = cv[k]; }
        r[6] = invD;
        r[7] = u;
        if (d == cfirst && catt >= 0) {
          float* s = pub + c * kPub;
#pragma unroll
          for (int q = 0; q < 21; ++q) s[q] = Ip[q];
#pragma unroll
          for (int q = 0; q < 6; ++q) s[21 + q] = pp[q];
        } else {
#pragma unroll
          for (int q = 0; q < 21; ++q) cI[q] = Ip[q];
#pragma unroll
          for (int q = 0; q < 6; ++q) cp[q] = pp[q];
        }
      } else {
        float a0[6];
        base_solve(IA, pA, a0);
        ba[0] = a0[0]; ba[1] = a0[1]; ba[2] = a0[2];
        ba[3] = a0[3] + agl[0]; ba[4] = a0[4] + agl[1]; ba[5] = a0[5] + agl[2];
#pragma unroll
        for (int q = 0; q < 6; ++q) ca[q] = a0[q];
        const int aid = ibits(rw[row::att]);
        if (aid >= 0) {
#pragma unroll
          for (int q = 0; q < 6; ++q) att[aid * kAtt + 24 + q] = a0[q];
        }
      }
    }
    wave_sync();
  }
  return mask;
}

// Root-to-leaf pass: joint accelerations and the semi-implicit Euler update of
// the joints (v += dt qdd, q += dt v).
__device__ __forceinline__ void chain_forward(const StepConst& sc, const float* rows, const int* cbody, float* rec,
                                              float* att, bool act, int c, int cfirst, int catt, int nlev, float* ca) {
  const int fb = sc.fb;
  const float dt = sc.dt;
  for (int d = 0; d < nlev; ++d) {
    const int b = act ? cbody[c * kMaxLevels + d] : -1;
    if (b >= 0 && !(fb && b == 0)) {
      const float* rw = rows + b * kRow;
      float* r = rec + b * kRec;
      float al[6];
      if (d == cfirst) {
        if (catt >= 0) {
#pragma unroll
          for (int q = 0; q < 6; ++q) al[q] = att[catt * kAtt + 24 + q];
        } else {
          // fixed world: a' = -a_g = (0, 0, 0, 0, 0, g)
          al[0] = al[1] = al[2] = 0.f; al[3] = 0.f; al[4] = 0.f; al[5] = sc.g;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 6; ++q) al[q] = ca[q];
      }
      float U[6], cv[6], e[3], ax[3];
#pragma unroll
      for (int k = 0; k < 6; ++k) { U[k] = r[k]; cv[k] = r[8 + k]; }
#pragma unroll
      for (int k = 0; k < 3; ++k) { e[k] = r[24 + k]; ax[k] = r[27 + k]; }
      const float qdd = forward_joint(al, e, cv, U, r[7], r[6], ax, ca);
      const int aid = ibits(rw[row::att]);
      if (aid >= 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q) att[aid * kAtt + 24 + q] = ca[q];
      }
      const float qd = fmaf(dt, qdd, r[33]);
      r[33] = qd;
      r[32] = fmaf(dt, qd, r[32]);
    }
    wave_sync();
  }
}

template <int GC>
__device__ __attribute__((always_inline)) void chain_item(const DevInst& I, int first, int group_stride,
                                                          int table_floats, int groups, float* smem) {
  const int lane = threadIdx.x;
  const int grp = lane / GC, l = lane % GC;
  const DevModel& M = *I.model;
  const int nb = M.nb, nc = M.nc, fb = M.fb, nch = M.n_chains;

  // model table of this instance (posture and nominal contact forces patched in)
  float* tab = smem;
  stage_model_table(M, &I, tab, lane);
  float* rows = smem + body_table_floats(nc);
  int* cbody = reinterpret_cast<int*>(rows + nb * kRow);
  {
    const float4* src = reinterpret_cast<const float4*>(&M.rows[0][0]);
    float4* dst = reinterpret_cast<float4*>(rows);
    for (int i = lane; i < nb * kRow / 4; i += 64) dst[i] = src[i];
    const int* cb = &M.chain_body[0][0];
    for (int i = lane; i < kMaxChains * kMaxLevels; i += 64) cbody[i] = cb[i];
  }
  wave_sync();
  if (I.cost_kind == 1)
    for (int b = fb + lane; b < nb; b += 64) rows[b * kRow + row::q0] = I.q0[b - fb];
  wave_sync();
  if (grp >= groups) return;  // the LDS budget holds fewer rollout groups than the wavefront has

  const int n = first + grp;
  const bool valid = n < I.N;
  float* gs = smem + table_floats + grp * group_stride;
  float* rec = gs;
  float* bas = rec + nb * kRec;
  float* knots = bas + 16;
  float* pub = knots + ((I.E + 3) & ~3);
  float* att = pub + nch * kPub;
  float* red = att + M.n_att * kAtt;

  if (I.generate) {
    sample_group<GC>(M, I, valid ? n : 0, l, knots, valid, tab);
  } else {
    const float* src = I.samples + (size_t)(valid ? n : 0) * I.E;
    for (int e = l; e < I.E; e += GC) knots[e] = src[e];
  }

  const bool act = l < nch;
  const int c = act ? l : 0;
  const int cfirst = M.chain_first[c], catt = M.chain_att[c];
  const int nlev = M.n_levels;
  const int nq = fb ? 7 + M.nu : M.nu;
  const bool base_lane = act && fb && c == 0;
  for (int d = 0; d < nlev; ++d) {
    const int b = act ? cbody[c * kMaxLevels + d] : -1;
    if (b >= 0) {
      float* r = rec + b * kRec;
      if (!(fb && b == 0)) {
        const int j = b - fb;
        r[32] = I.x0[(fb ? 7 : 0) + j];
        r[33] = I.x0[nq + (fb ? 6 : 0) + j];
      }
      r[34] = 0.f;
    }
  }
  if (!fb && l == 0) {
#pragma unroll
    for (int k = 0; k < 12; ++k) bas[k] = (k < 9 && k % 4 == 0) ? 1.f : 0.f;
  }
  float bq[7], bv[6], ba[6], ca[6];
#pragma unroll
  for (int k = 0; k < 7; ++k) bq[k] = fb ? I.x0[k] : 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) { bv[k] = fb ? I.x0[nq + k] : 0.f; ba[k] = 0.f; ca[k] = 0.f; }
  wave_sync();

  const StepConst sc = load_step_const(M, &I, 0.f);
  uint32_t* const masks = I.masks;
  const int H = I.H, F = sc.F;
  StepClock clk;
  for (int f = 0; f < F; ++f) {
    const bool control = clk.sub == 0;
    float base_term = 0.f;
    if (control && base_lane && sc.cost_kind == 1) base_term = base_cost_term(sc, bq);
    chain_fk(sc, rows, cbody, rec, bas, knots, att, act, c, cfirst, catt, nlev, clk.seg, clk.rem, false, bq, bv);
    const uint32_t mask = chain_backward(sc, tab, rows, cbody, rec, bas, pub, att, act, c, cfirst, catt, nlev, control,
                                         base_term, ba, ca);
    chain_forward(sc, rows, cbody, rec, att, act, c, cfirst, catt, nlev, ca);
    if (control && masks) {
      const uint32_t mk = group_or<GC>(mask, red, l);
      if (l == 0 && valid) masks[(size_t)n * H + clk.h] = mk;
    }
    if (base_lane) integrate_base(bq, bv, ba, sc.dt);
    clk.advance(sc.K, F, sc.nsub);
  }

  // terminal cost
  if (sc.cost_kind == 1) {
    if (base_lane) {
      const float T = (float)H * I.dt;
      float e = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float target = (k == 2 && I.targets->terminal_z_abs) ? I.targets->z_terminal : I.x0[k] + I.targets->v_des[k] * T;
        e += fabsf(bq[k] - target);
      }
      rec[34] += I.w_H * e;
    }
  } else {
    // end-effector height at x_H
    chain_fk(sc, rows, cbody, rec, bas, knots, att, act, c, cfirst, catt, nlev, 0, 0, true, bq, bv);
    const int ee = sc.ee_body;
    if (act && ee >= 0 && ibits(rows[ee * kRow + row::chain]) == c) {
      float* r = rec + ee * kRec;
      const float dz = ee_height_error(r, r + 9, sc.ee_pos, bas, bas + 9, sc.z_des);
      const float tc = sc.w_ee * dz * dz;
      r[34] += tc;
    }
  }
  wave_sync();
  if (l == 0 && valid) {
    float S = 0.f;
    for (int b = 0; b < nb; ++b) S += rec[b * kRec + 34];
    if (!isfinite(S)) S = INFINITY;
    I.costs[n] = S;
  }
  wave_sync();
}

// Block = one wavefront holding `groups` (<= 64/GC) rollout groups; work[blockIdx]
// = (instance, first sample) or, when work is null, instance 0 and sample
// blockIdx * groups.
template <int GC>
__global__ __launch_bounds__(64) void chain_kernel(const DevInst* __restrict__ insts, const int2* __restrict__ work,
                                                   int group_stride, int table_floats, int groups) {
  extern __shared__ float smem[];
  const int2 w = work ? work[blockIdx.x] : make_int2(0, (int)blockIdx.x * groups);
  chain_item<GC>(insts[w.x], w.y, group_stride, table_floats, groups, smem);
}

template <int GC>
__global__ __launch_bounds__(64) void chain_persistent_kernel(const DevInst* __restrict__ insts,
                                                              const int2* __restrict__ work, int n_items,
                                                              unsigned int* __restrict__ counter, int group_stride,
                                                              int table_floats, int groups) {
  extern __shared__ float smem[];
  for (;;) {
    int item = 0;
    if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const int2 w = work[item];
    chain_item<GC>(insts[w.x], w.y, group_stride, table_floats, groups, smem);
    wave_sync();
  }
}

// A new set of task targets for an instance, ordered on the launch stream.
__global__ void set_targets_kernel(DevTargets* __restrict__ dst, DevTargets v) {
  if (threadIdx.x == 0) *dst = v;
}

__global__ void reset_counters(unsigned int* __restrict__ c, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) c[i] = 0u;
}

// ---------------------------------------------------------------------------
// Weighting, update and best tracking.  Grid (the most workgroups of one of the
// launch's instances, instances): an instance's workgroups each take one slice of
// its samples (U.parts of them, update_shape(N)), where samples are drawn again and
// the launch says so (`tile`) one share of the slice's element blocks; the workgroups
// beyond that return at once.
// out (per call): the final nominal, best knots and info of the last iteration.
// ---------------------------------------------------------------------------

// T (64 or 256, update_shape) is the workgroup's size and the width of the sums'
// order.  An update is bound by latency: the draws of a slice's samples, about 330
// instructions each (at T = 64 one thread per element block drew all 16 of its
// rows, one after another), the statistics' chains and the hand-over to the part
// that finishes last.  So at T = 64 a part is spread over workgroups of `tile`
// element blocks, each of which forms the statistics and weights for itself and
// draws its tile with all lanes; reductions are shuffles; the sums are stored
// through to memory, so that no workgroup needs a fence (a device-scope fence
// writes back the XCD's L2: with one per workgroup a 64-robot round's updates in
// tiles of 32 blocks took 236 us, without 57).  One update before / now: hexapod
// 35 / 14.6 us, humanoid 33 / 17.5, quadruped at 64 samples 20.5 / 12.2, at 4 096
// (T = 256) 27.5 / 22.8, arm 12.5 / 11.9; a 16-robot round's 36 / 23.3, a 64-robot
// round's 80 / 55.  The workgroups at T = 64 stay single wavefronts: one finds room
// wherever a rollout wavefront has ended, while one of four waits until all SIMDs of
// a compute unit are free at once (256 threads sharing the draws were as fast on an
// idle device, but 64 served robots on six streams answered in 3.9 ms p50 / 12 ms
// p99, with single wavefronts in 2.1 / 7.8).

// Sum of x over threads 0 .. T-1 in a fixed order (a tree over threads).
template <int T>
__device__ __forceinline__ float block_sum(float x, float* buf) {
  const int t = threadIdx.x;
  if constexpr (T > 64) {
    buf[t] = x;
    __syncthreads();
#pragma unroll
    for (int off = T / 2; off > 64; off >>= 1) {
      if (t < off) buf[t] += buf[t + off];
      __syncthreads();
    }
    if (t < 64) x = buf[t] + buf[t + 64];
  }
  if (T == 64 || t < 64) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);  // lanes < off hold the tree's sums
    if (t == 0) buf[T] = x;
  }
  __syncthreads();
  return buf[T];
}

// A part's sums are read by the workgroup that finishes last, on any XCD: stored
// through to memory (agent scope), so that publishing them takes a wait for the
// stores and no release, which would write back the XCD's whole L2.  This rests on
// gfx950, not on the language's memory model (which wants that release before the
// counter): an agent-scope store carries sc1, is written through its XCD's L2 to the
// memory that all XCDs share and counts down vmcnt only there; the counters' atomics
// are performed there too, after that wait; and the reader's fence drops its own
// XCD's stale lines (buffer_inv sc1) before it reads.
__device__ __forceinline__ void store_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sums over one index range of a row-major [*, E] array, V consecutive floats
// (V = 4 or 1) per element block.
template <int V>
struct VecT;
template <>
struct VecT<4> {
  using T = float4;
  static __device__ __forceinline__ float4 zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  static __device__ __forceinline__ void fma(float w, const float4& a, float4& acc) {
    acc.x = fmaf(w, a.x, acc.x); acc.y = fmaf(w, a.y, acc.y); acc.z = fmaf(w, a.z, acc.z); acc.w = fmaf(w, a.w, acc.w);
  }
  static __device__ __forceinline__ void add(const float4& a, float4& acc) {
    acc.x += a.x; acc.y += a.y; acc.z += a.z; acc.w += a.w;
  }
};
template <>
struct VecT<1> {
  using T = float;
  static __device__ __forceinline__ float zero() { return 0.f; }
  static __device__ __forceinline__ void fma(float w, float a, float& acc) { acc = fmaf(w, a, acc); }
  static __device__ __forceinline__ void add(float a, float& acc) { acc += a; }
};

// sum_{n < cnt} w[n] rows[n][:] (w null: weight 1); the result goes to
// emit(element block, value).  Each block's rows are split over G groups (rows g,
// g + G, ...), each in index order, whose sums are added in g order; G is what T
// threads give (T / blocks, at least 1).  A thread takes one block of one group.
template <int V, int T, typename Emit>
__device__ __forceinline__ void rows_weighted_sum(const float* __restrict__ rows, int cnt, int E, const float* w,
                                                  float4* s_part, Emit emit) {
  using VT = VecT<V>;
  using F = typename VT::T;
  constexpr int kIn = T == 64 ? 16 : 24;  // loads in flight per thread (rows past cnt are not loaded)
  const int t = threadIdx.x, EV = E / V;
  F* part = reinterpret_cast<F*>(s_part);
  const F* col = reinterpret_cast<const F*>(rows);
  const int G = T / min(T, EV);
  const int EC = T / G;
  for (int e0 = 0; e0 < EV; e0 += EC) {
    const int ec = min(EC, EV - e0);
    const int el = t % ec, g = t / ec, e = e0 + el;
    F acc = VT::zero();
    if (g < G) {
      for (int n = g; n < cnt; n += kIn * G) {
        F a[kIn];
#pragma unroll
        for (int q = 0; q < kIn; ++q) {
          const int r = n + q * G;
          a[q] = r < cnt ? col[(size_t)r * EV + e] : VT::zero();
        }
#pragma unroll
        for (int q = 0; q < kIn; ++q) {
          const int r = n + q * G;
          if (r < cnt) {
            if (w) VT::fma(w[r], a[q], acc);
            else VT::add(a[q], acc);
          }
        }
      }
    }
    __syncthreads();
    if (g < G) part[g * ec + el] = acc;
    __syncthreads();
    if (t < ec) {
      F sum = VT::zero();
      for (int k = 0; k < G; ++k) VT::add(part[k * ec + t], sum);
      emit(e0 + t, sum);
    }
  }
}

// The same sum as rows_weighted_sum<4> over the samples rows n0 .. n0 + cnt - 1,
// with each sample's knots drawn again from the counter-based stream instead of
// read (the rollout kernel then stores none).  Element block b holds positions
// 2b, 2b + 1 and velocities 2b, 2b + 1 (one counter-based block); there are
// E / 4 of them, as many as rows_weighted_sum<4> has, so every element's rows are
// split over as many groups and added in the same order, and the two forms give
// the same bits.  Needs K nu even and the cubic Hermite knots (velocities
// sampled, not derived).  A workgroup of T threads: each draws the rows it adds.
template <int T>
__device__ __forceinline__ void regen_weighted_sum(const DevInst& I, const float* nom, uint32_t tick, int n0, int cnt,
                                                   const float* w, float4* part, float* mine) {
  const DevModel& M = *I.model;
  const int t = threadIdx.x, KU = I.K * I.nu, EV = KU / 2;
  const float* sig = I.sigma + I.iter * I.K;
  const int G = T / min(T, EV);
  for (int e0 = 0; e0 < EV; e0 += T) {
    const int ec = min(T, EV - e0);
    const int el = t % ec, g = t / ec, b = e0 + el;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (g < G) {
      const ElemConst c0 = elem_const(M, I, sig, 2 * b), c1 = elem_const(M, I, sig, 2 * b + 1);
      const float nq0 = nom[2 * b], nq1 = nom[2 * b + 1], nv0 = nom[KU + 2 * b], nv1 = nom[KU + 2 * b + 1];
      // kRow rows are drawn together (independent chains the scheduler can
      // interleave), then added in row order
      constexpr int kRow = 4;
      for (int r0 = g; r0 < cnt; r0 += kRow * G) {
        float4 th[kRow];
#pragma unroll
        for (int q = 0; q < kRow; ++q) {
          const int n = n0 + min(r0 + q * G, cnt - 1);  // rows past the slice are drawn, not added
          const uint4 x = sample_words(I, n, b, tick);
          perturb_element(c0, I.delta, nq0, nv0, n, x.x, x.y, true, th[q].x, th[q].z);
          perturb_element(c1, I.delta, nq1, nv1, n, x.z, x.w, true, th[q].y, th[q].w);
        }
#pragma unroll
        for (int q = 0; q < kRow; ++q) {
          const int r = r0 + q * G;
          if (r < cnt) {
            const float wr = w[r];
            acc.x = fmaf(wr, th[q].x, acc.x); acc.y = fmaf(wr, th[q].y, acc.y);
            acc.z = fmaf(wr, th[q].z, acc.z); acc.w = fmaf(wr, th[q].w, acc.w);
          }
        }
      }
    }
    __syncthreads();
    if (g < G) part[g * ec + el] = acc;
    __syncthreads();
    if (t < ec) {
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int k = 0; k < G; ++k) {
        const float4 a = part[k * ec + t];
        sum.x += a.x; sum.y += a.y; sum.z += a.z; sum.w += a.w;
      }
      const int m = 2 * (e0 + t);
      store_agent(mine + m, sum.x); store_agent(mine + m + 1, sum.y);
      store_agent(mine + KU + m, sum.z); store_agent(mine + KU + m + 1, sum.w);
    }
    __syncthreads();  // before the next blocks' sums
  }
}

// The same at T = 64 (slices of at most kUpdTileRows samples) for block tiles chunk,
// chunk + chunks, ... of `tile` blocks (at most kUpdTile): the wavefront draws a
// tile's samples into LDS, all lanes at work whatever the number of blocks, then
// thread g ec + el adds block el's rows of group g.
struct DrawConst {
  float sq, lo, hi, nq, nv;
};
__device__ __forceinline__ void regen_weighted_sum_tiles(const DevInst& I, const float* nom, uint32_t tick, int n0, int cnt,
                                                         const float* w, float4* draws, DrawConst* consts, float* mine,
                                                         int tile, int chunk, int chunks) {
  const DevModel& M = *I.model;
  const int t = threadIdx.x, KU = I.K * I.nu, EV = KU / 2;
  const float* sig = I.sigma + I.iter * I.K;
  const int G = 64 / min(64, EV);
  for (int e0 = chunk * tile; e0 < EV; e0 += chunks * tile) {
    const int ec = min(tile, EV - e0);  // ec G <= 64, as G = 64 / min(64, EV)
    if (t < 2 * ec) {
      const int m = 2 * e0 + t;
      const ElemConst e = elem_const(M, I, sig, m);
      consts[t] = DrawConst{e.sq, e.lo, e.hi, nom[m], nom[KU + m]};
    }
    __syncthreads();
    for (int p = t; p < cnt * ec; p += 64) {
      const int r = p / ec, b = p % ec, n = n0 + r;
      const DrawConst c0 = consts[2 * b], c1 = consts[2 * b + 1];
      const uint4 x = sample_words(I, n, e0 + b, tick);
      float4 th;
      perturb_element(ElemConst{c0.sq, c0.lo, c0.hi, 0}, I.delta, c0.nq, c0.nv, n, x.x, x.y, true, th.x, th.z);
      perturb_element(ElemConst{c1.sq, c1.lo, c1.hi, 0}, I.delta, c1.nq, c1.nv, n, x.z, x.w, true, th.y, th.w);
      draws[p] = th;
    }
    __syncthreads();
    const int el = t % ec, g = t / ec;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (g < G)
      for (int r = g; r < cnt; r += G) {
        const float wr = w[r];
        const float4 th = draws[r * ec + el];
        acc.x = fmaf(wr, th.x, acc.x); acc.y = fmaf(wr, th.y, acc.y);
        acc.z = fmaf(wr, th.z, acc.z); acc.w = fmaf(wr, th.w, acc.w);
      }
    __syncthreads();
    if (g < G) draws[g * ec + el] = acc;
    __syncthreads();
    if (t < ec) {
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int k = 0; k < G; ++k) {
        const float4 a = draws[k * ec + t];
        sum.x += a.x; sum.y += a.y; sum.z += a.z; sum.w += a.w;
      }
      const int m = 2 * (e0 + t);
      store_agent(mine + m, sum.x); store_agent(mine + m + 1, sum.y);
      store_agent(mine + KU + m, sum.z); store_agent(mine + KU + m + 1, sum.w);
    }
    __syncthreads();  // before the next tile's constants and draws
  }
}

// Knots of sample n (drawn again, as above) into dst [E].
template <int T>
__device__ __forceinline__ void regen_sample(const DevInst& I, const float* nom, uint32_t tick, int n, float* dst) {
  const DevModel& M = *I.model;
  const int KU = I.K * I.nu;
  const float* sig = I.sigma + I.iter * I.K;
  for (int b = threadIdx.x; b < KU / 2; b += T) {
    const uint4 x = sample_words(I, n, b, tick);
    float q0, v0, q1, v1;
    perturb_element(elem_const(M, I, sig, 2 * b), I.delta, nom[2 * b], nom[KU + 2 * b], n, x.x, x.y, true, q0, v0);
    perturb_element(elem_const(M, I, sig, 2 * b + 1), I.delta, nom[2 * b + 1], nom[KU + 2 * b + 1], n, x.z, x.w,
                    true, q1, v1);
    dst[2 * b] = q0; dst[2 * b + 1] = q1;
    dst[KU + 2 * b] = v0; dst[KU + 2 * b + 1] = v1;
  }
}

// The share of one workgroup in an instance's update: its part, and there the
// tiles chunk, chunk + chunks, ... of the knot elements; o: the call's outputs (null
// fields: not wanted).
template <int T>
__device__ __forceinline__ void update_body(const DevUpdate& U, const UpdateOut o, int tile) {
  const int parts = U.parts, chunks = tile && U.regen ? update_chunks(U.E / 4, tile) : 1;
  if ((int)blockIdx.x >= parts * chunks) return;
  const int part = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int t = threadIdx.x, N = U.N, E = U.E;
  // the nominal the iteration's samples perturbed (the call's input on its first
  // iteration when the caller's buffer is read in place)
  const float* nom_in = o.nominal_in ? o.nominal_in : U.nominal_in;
  const uint32_t tick = U.regen ? sample_tick(*U.regen) : 0u;  // read before the last part advances it
  // a tile of draws, or the groups' sums
  __shared__ __align__(16) float4 s_buf[kUpdTileRows * kUpdTile];
  static_assert(kUpdTileRows * kUpdTile >= T, "the groups' sums");
  __shared__ DrawConst s_const[2 * kUpdTile];
  __shared__ float s_w[(65536 + kUpdMaxParts - 1) / kUpdMaxParts];  // this part's normalised weights (N <= 65536)
  __shared__ float s_tree[T + 1], s_min[T / 64], s_max[T / 64];
  __shared__ int s_arg[T / 64], s_fin[T / 64], s_last;

  // this part's slice of the samples
  const int slice = (N + parts - 1) / parts;
  const int n0 = part * slice, cnt = max(0, min(N, n0 + slice) - n0);

  // 1. over all samples (every part the same way, so every part gets the same
  //    values): finite minimum (lowest index), maximum and count
  const float* costs = U.costs;
  float mn = INFINITY, mx = -INFINITY;
  int arg = 0x7fffffff, nf = 0;
  constexpr int kIn = 16;
  for (int m0 = t; m0 < N; m0 += kIn * T) {
    float Sq[kIn];
#pragma unroll
    for (int q = 0; q < kIn; ++q) {
      const int n = m0 + q * T;
      Sq[q] = n < N ? costs[n] : INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kIn; ++q) {
      const int n = m0 + q * T;
      const float S = Sq[q];
      if (n >= n0 && n < n0 + cnt) s_w[n - n0] = S;  // the slice's costs
      if (isfinite(S)) {
        ++nf;
        if (S < mn) { mn = S; arg = n; }
        mx = fmaxf(mx, S);
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float om = __shfl_xor(mn, off, 64), ox = __shfl_xor(mx, off, 64);
    const int oi = __shfl_xor(arg, off, 64), of = __shfl_xor(nf, off, 64);
    if (om < mn || (om == mn && oi < arg)) { mn = om; arg = oi; }
    mx = fmaxf(mx, ox);
    nf += of;
  }
  if (t % 64 == 0) { s_min[t / 64] = mn; s_max[t / 64] = mx; s_arg[t / 64] = arg; s_fin[t / 64] = nf; }
  __syncthreads();
  float smin = s_min[0], smax = s_max[0];
  int nstar = s_arg[0], nfin = s_fin[0];
#pragma unroll
  for (int k = 1; k < T / 64; ++k) {
    if (s_min[k] < smin || (s_min[k] == smin && s_arg[k] < nstar)) { smin = s_min[k]; nstar = s_arg[k]; }
    smax = fmaxf(smax, s_max[k]);
    nfin += s_fin[k];
  }

  // 2. unnormalised weights e_n = exp(-S_hat / lambda) and their sum: thread t < T
  //    adds samples t, t + T, ... in order, then a tree over the T threads
  const float range = smax - smin;
  const float inv_range = (U.weight_mode == 0 && range > 0.f) ? 1.f / range : 0.f;
  const float inv_lam = 1.f / U.lambda;
  auto weight = [&](float S) -> float {
    if (!isfinite(S)) return 0.f;
    const float sh = U.weight_mode == 0 ? (S - smin) * inv_range : (S - smin);
    return expf(-sh * inv_lam);
  };
  float zs = 0.f;
  for (int m0 = t; m0 < N; m0 += kIn * T) {
    float Sq[kIn];
#pragma unroll
    for (int q = 0; q < kIn; ++q) {
      const int n = m0 + q * T;
      Sq[q] = n < N ? costs[n] : INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kIn; ++q) zs += weight(Sq[q]);
  }
  const float Z = block_sum<T>(zs, s_tree);
  const float invZ = nfin > 0 ? 1.f / Z : 0.f;

  // 3. this part's slice: normalised weights, then its weighted knot sum
  for (int i = t; i < cnt; i += T) {
    const float w = weight(s_w[i]) * invZ;
    s_w[i] = w;
    if (U.weights && chunk == 0) U.weights[n0 + i] = w;
  }
  __syncthreads();
  float* mine = U.partial + (size_t)part * E;
  if (U.regen) {
    if (T == 64 && tile)
      regen_weighted_sum_tiles(*U.regen, nom_in, tick, n0, cnt, s_w, s_buf, s_const, mine, tile, chunk, chunks);
    else
      regen_weighted_sum<T>(*U.regen, nom_in, tick, n0, cnt, s_w, s_buf, mine);
  } else if ((E & 3) == 0)
    rows_weighted_sum<4, T>(U.samples + (size_t)n0 * E, cnt, E, s_w, s_buf,
                            [&](int e, float4 v) {
                              store_agent(mine + 4 * e, v.x); store_agent(mine + 4 * e + 1, v.y);
                              store_agent(mine + 4 * e + 2, v.z); store_agent(mine + 4 * e + 3, v.w);
                            });
  else
    rows_weighted_sum<1, T>(U.samples + (size_t)n0 * E, cnt, E, s_w, s_buf, [&](int e, float v) { store_agent(mine + e, v); });

  // 4. the last part to finish adds the slices in part order
  if (parts * chunks > 1) {
    wait_stores();  // every thread's own, then the workgroup's
    __syncthreads();
    if (t == 0) {
      // counted by chunk first (done[1 + chunk], then done[0]): increments of one
      // address follow each other
      bool last = true;
      if (chunks > 1) {
        last = atomicAdd(U.done + 1 + chunk, 1u) == (uint32_t)(parts - 1);
        if (last) U.done[1 + chunk] = 0u;  // ready for the next launch
      }
      if (last) last = atomicAdd(U.done, 1u) == (uint32_t)((chunks > 1 ? chunks : parts) - 1);
      s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    if (t == 0) U.done[0] = 0u;
  }
  __syncthreads();
  float* dst = (U.last_iter && o.knots_out) ? o.knots_out : U.nominal_out;

  // 5. best-sample tracking across the iterations of this call, whose running best
  //    starts from its input nominal.  It reads the nominal before the output is
  //    written, since the two may be the same buffer.
  float* bs = U.best_state;  // [E] knots, then S_best, best_iter, n_nonfinite, all_nonfinite, best_sample
  int* bi = reinterpret_cast<int*>(bs);
  const bool first = U.first_iter;
  float S_best = INFINITY;
  int best_iter = -1, best_sample = -1, nonfinite = 0, all_nonfinite = 0;
  if (!first) {
    S_best = bs[E];
    best_iter = bi[E + 1]; nonfinite = bi[E + 2]; all_nonfinite = bi[E + 3]; best_sample = bi[E + 4];
  }
  const bool improve = nfin > 0 && smin < S_best;
  if (improve) { S_best = smin; best_iter = U.iter; best_sample = nstar; }
  nonfinite += N - nfin;
  all_nonfinite += nfin == 0 ? 1 : 0;
  __syncthreads();  // every thread has read the running best
  if (improve) {
    if (U.regen) regen_sample<T>(*U.regen, nom_in, tick, nstar, bs);
    else
      for (int e = t; e < E; e += T) bs[e] = U.samples[(size_t)nstar * E + e];
  } else if (first) {
    for (int e = t; e < E; e += T) bs[e] = nom_in[e];
  }
  if (t == 0) {
    bs[E] = S_best;
    bi[E + 1] = best_iter; bi[E + 2] = nonfinite; bi[E + 3] = all_nonfinite; bi[E + 4] = best_sample;
  }
  __syncthreads();

  // 6. the nominal: the slices added in part order
  if ((E & 3) == 0)
    rows_weighted_sum<4, T>(U.partial, parts, E, nullptr, s_buf, [&](int e, float4 v) {
      const float c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) dst[4 * e + k] = nfin > 0 ? c[k] : nom_in[4 * e + k];
    });
  else
    rows_weighted_sum<1, T>(U.partial, parts, E, nullptr, s_buf, [&](int e, float v) { dst[e] = nfin > 0 ? v : nom_in[e]; });
  __syncthreads();
  if (U.last_iter) {
    if (o.best_out)
      for (int e = t; e < E; e += T) o.best_out[e] = bs[e];
    if (t == 0 && o.info_out) {
      float* inf = reinterpret_cast<float*>(o.info_out);
      int* ii = reinterpret_cast<int*>(o.info_out);
      inf[0] = S_best;
      ii[1] = best_iter; ii[2] = nonfinite; ii[3] = all_nonfinite; ii[4] = best_sample;
    }
  }
  if (U.last_iter && t == 0 && U.tick) U.tick[0] += 1u;
}

template <int T>
__global__ __launch_bounds__(T) void update_kernel(const DevUpdate* __restrict__ ups, const UpdateOut* __restrict__ outs,
                                                   UpdateOut single, int tile) {
  update_body<T>(ups[blockIdx.y], outs ? outs[blockIdx.y] : single, tile);
}

// One instance whose descriptor arrives as a kernel argument (no device copy of
// it), with no per-call outputs besides the nominal and the weights.
__global__ __launch_bounds__(kUpdThreads) void update_single_kernel(DevUpdate U) {
  update_body<kUpdThreads>(U, UpdateOut{nullptr, nullptr, nullptr, nullptr}, 0);
}
template __global__ void update_kernel<64>(const DevUpdate*, const UpdateOut*, UpdateOut, int);
template __global__ void update_kernel<kUpdThreads>(const DevUpdate*, const UpdateOut*, UpdateOut, int);

// Warm start (Sec. III-E): the knots of a trajectory shifted forward by n_steps
// control steps, i.e. its spline at t_k + n_steps dt clamped to the horizon end
// (the final action repeats).  In fine steps of the horizon (F = H n_sub) the
// knot time is k F / (K - 1), so the segment and remainder come from the
// integer m = k F + n_steps n_sub (K - 1) = seg F + rem.  Position-only spline
// variants then take the slopes of the spline through the shifted positions.
// One workgroup; in and out must not alias.

__device__ __forceinline__ void shift_knots_block(const float* __restrict__ in, float* __restrict__ out, int K,
                                                  int nu, int F, int nsub, int n_steps, float delta, int spline_mode,
                                                  float* dg) {
  for (int i = threadIdx.x; i < K * nu; i += kShiftThreads) {
    const int k = i / nu, jj = i % nu;
    const long long m = (long long)k * F + (long long)n_steps * nsub * (K - 1);
    int seg = (int)(m / F), rem = (int)(m - (long long)seg * F);
    if (seg > K - 2) {
      seg = K - 2;
      rem = F;
    }
    float q, v;
    hermite_eval(hermite_segment(in, K, nu, seg, jj, delta), (float)rem / (float)F, 1.f / delta, &q, &v);
    out[i] = q;
    out[K * nu + i] = v;
  }
  if (spline_mode == 0) return;
  if (threadIdx.x == 0 && spline_mode == 1) natural_cubic_diagonal(K, dg);
  __syncthreads();
  for (int jj = threadIdx.x; jj < nu; jj += kShiftThreads) position_spline_slopes(spline_mode, K, nu, jj, delta, dg, out);
}
__global__ __launch_bounds__(kShiftThreads) void shift_knots_kernel(const float* __restrict__ in,
                                                                    float* __restrict__ out, int K, int nu, int F,
                                                                    int nsub, int n_steps, float delta,
                                                                    int spline_mode) {
  __shared__ float dg[kMaxKnots];
  shift_knots_block(in, out, K, nu, F, nsub, n_steps, delta, spline_mode, dg);
}
// The warm-start shifts of a batch of ticks, one workgroup per item.
__global__ __launch_bounds__(kShiftThreads) void shift_batch_kernel(const ShiftItem* __restrict__ items) {
  __shared__ float dg[kMaxKnots];
  const ShiftItem it = items[blockIdx.x];
  shift_knots_block(it.in, it.out, it.K, it.nu, it.F, it.nsub, it.n_steps, it.delta, it.spline_mode, dg);
}

// Copy per-call inputs (state, warm-start knots) into instance buffers.
struct StageItem {
  const float* src;
  float* dst;
  int32_t count;
};
__global__ void stage_kernel(const StageItem* __restrict__ items) {
  const StageItem it = items[blockIdx.x];
  for (int i = threadIdx.x; i < it.count; i += blockDim.x) it.dst[i] = it.src[i];
}

// Two device copies in one launch (block 0: src0 -> dst0, block 1: src1 -> dst1).
__global__ void copy2_kernel(const float* __restrict__ src0, float* __restrict__ dst0, int n0,
                             const float* __restrict__ src1, float* __restrict__ dst1, int n1) {
  const float* src = blockIdx.x == 0 ? src0 : src1;
  float* dst = blockIdx.x == 0 ? dst0 : dst1;
  const int n = blockIdx.x == 0 ? n0 : n1;
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// Verification kernels (same device functions as the product path)
// ---------------------------------------------------------------------------
__global__ void philox_kernel(const uint32_t* __restrict__ ctr, const uint32_t* __restrict__ key,
                              uint32_t* __restrict__ out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint4 r = philox(make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]),
                         make_uint2(key[2 * i], key[2 * i + 1]));
  out[4 * i] = r.x; out[4 * i + 1] = r.y; out[4 * i + 2] = r.z; out[4 * i + 3] = r.w;
}

template <int G>
__global__ __launch_bounds__(64) void sample_kernel(const DevInst* __restrict__ inst, int group_stride) {
  extern __shared__ float smem[];
  constexpr int R = 64 / G;
  const int lane = threadIdx.x, grp = lane / G, l = lane % G;
  const DevInst& I = *inst;
  float* tab = smem;  // spline diagonal only
  if (I.spline_mode == 1 && lane == 0) natural_cubic_diagonal(I.K, tab + kTabSpline);
  wave_sync();
  const int n = blockIdx.x * R + grp;
  float* knots = smem + kTabContacts + grp * group_stride + G * kSlot + 16;
  sample_group<G>(*I.model, I, n < I.N ? n : 0, l, knots, n < I.N, tab);
}

template <int G>
__global__ __launch_bounds__(64) void dynamics_kernel(const DevModel* __restrict__ model, int n_states,
                                                      const float* __restrict__ q, const float* __restrict__ v,
                                                      const float* __restrict__ qref, const float* __restrict__ vref,
                                                      float dt, float* __restrict__ qdd, int group_stride,
                                                      int table_floats) {
  extern __shared__ float smem[];
  constexpr int R = 64 / G;
  const int lane = threadIdx.x, grp = lane / G, l = lane % G;
  const DevModel& M = *model;
  float* tab = smem;
  stage_model_table(M, nullptr, tab, lane, true);
  const int s_raw = blockIdx.x * R + grp;
  const bool valid = s_raw < n_states;
  const int s = valid ? s_raw : 0;
  const StepConst sc = load_step_const(M, nullptr, dt);
  const int fb = sc.fb, nu = M.nu, nq = fb ? 7 + nu : nu, nv = fb ? 6 + nu : nu;
  float* gs = smem + table_floats + grp * group_stride;
  const bool body_lane = l < M.nb;
  const bool is_joint = body_lane && !(fb && l == 0);
  const int j = l - fb;
  StepIO io;
  io.q = is_joint ? q[(size_t)s * nq + (fb ? 7 : 0) + j] : 0.f;
  io.v = is_joint ? v[(size_t)s * nv + (fb ? 6 : 0) + j] : 0.f;
  io.qref = is_joint ? qref[(size_t)s * nu + j] : 0.f;
  io.vref = is_joint ? vref[(size_t)s * nu + j] : 0.f;
#pragma unroll
  for (int k = 0; k < 7; ++k) io.bq[k] = fb ? q[(size_t)s * nq + k] : 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) { io.bv[k] = fb ? v[(size_t)s * nv + k] : 0.f; io.ba[k] = 0.f; }
  io.dt = dt;
  BodyConst bc;
  load_body(M, nullptr, l, body_lane, tab, bc);
  BodyKin kin;  // (unused: the general kernel takes its kinematics fresh)
  physics_step<G>(sc, bc, tab, gs, l, body_lane, io, kin, false);
  if (!valid) return;
  if (is_joint) qdd[(size_t)s * nv + (fb ? 6 : 0) + j] = io.qdd;
  if (fb && l == 0)
    for (int k = 0; k < 6; ++k) qdd[(size_t)s * nv + k] = io.ba[k];
}

// explicit instantiations
#define MPPI_INST(G)                                                                                   \
  template __global__ void rollout_kernel<G, 0, 0>(const DevInst*, const int2*, int, int, const float*,  \
                                                       const float*);                                     \
  template __global__ void rollout_kernel<G, 3, 0>(const DevInst*, const int2*, int, int, const float*,  \
                                                       const float*);                                     \
  template __global__ void rollout_kernel<G, 6, 0>(const DevInst*, const int2*, int, int, const float*,  \
                                                       const float*);                                     \
  template __global__ void rollout_trace_kernel<G, 0, 0>(const DevInst*, const int2*, int, int);     \
  template __global__ void rollout_trace_kernel<G, 3, 0>(const DevInst*, const int2*, int, int);     \
  template __global__ void rollout_trace_kernel<G, 6, 0>(const DevInst*, const int2*, int, int);     \
  template __global__ void rollout_persistent_kernel<G, 0, 0>(const DevInst*, const int2*, int, unsigned int*, int,  \
                                                             int);                                                \
  template __global__ void rollout_persistent_kernel<G, 3, 0>(const DevInst*, const int2*, int, unsigned int*, int,  \
                                                             int);                                                \
  template __global__ void rollout_persistent_kernel<G, 6, 0>(const DevInst*, const int2*, int, unsigned int*, int,  \
                                                             int);                                                \
  template __global__ void sample_kernel<G>(const DevInst*, int);                                      \
  template __global__ void predict_kernel<G>(const DevInst*, int, float*, int, int);                   \
  template __global__ void predict_batch_kernel<G>(const PredItem*, int, int);                         \
  template __global__ void dynamics_kernel<G>(const DevModel*, int, const float*, const float*,        \
                                              const float*, const float*, float, float*, int, int);  \
  template __global__ void team_kernel<G, 0>(const DevInst*, const int2*, int, int);                   \
  template __global__ void team_kernel<G, 3>(const DevInst*, const int2*, int, int);                   \
  template __global__ void team_kernel<G, 6>(const DevInst*, const int2*, int, int);                   \
  template __global__ void team_persistent_kernel<G>(const DevInst*, const int2*, int, unsigned int*, int, int);
// legged trees up to 3 levels deep (a base and 2..10 chains of up to three bodies)
#define MPPI_LEG_INST(G)                                                                               \
  template __global__ void rollout_kernel<G, 3, 1>(const DevInst*, const int2*, int, int, const float*,   \
                                                      const float*);                                      \
  template __global__ void rollout_trace_kernel<G, 3, 1>(const DevInst*, const int2*, int, int);                \
  template __global__ void rollout_persistent_kernel<G, 3, 1>(const DevInst*, const int2*, int, unsigned int*, int,  \
                                                             int);
MPPI_LEG_INST(8)
MPPI_LEG_INST(16)
MPPI_LEG_INST(32)
#undef MPPI_LEG_INST
// fixed-base serial chains up to 3 bodies
#define MPPI_SERIAL_INST(G)                                                                            \
  template __global__ void rollout_kernel<G, 3, 3>(const DevInst*, const int2*, int, int, const float*,   \
                                                      const float*);                                      \
  template __global__ void rollout_trace_kernel<G, 3, 3>(const DevInst*, const int2*, int, int);                \
  template __global__ void rollout_persistent_kernel<G, 3, 3>(const DevInst*, const int2*, int, unsigned int*, int,  \
                                                             int);
MPPI_SERIAL_INST(4)
MPPI_SERIAL_INST(8)
#undef MPPI_SERIAL_INST
// four chains of three bodies on 16 lanes (the quadruped's shape)
template __global__ void rollout_kernel<16, 3, 2>(const DevInst*, const int2*, int, int, const float*, const float*);
template __global__ void rollout_trace_kernel<16, 3, 2>(const DevInst*, const int2*, int, int);
template __global__ void rollout_persistent_kernel<16, 3, 2>(const DevInst*, const int2*, int, unsigned int*, int, int);
MPPI_INST(4)
MPPI_INST(8)
MPPI_INST(16)
MPPI_INST(32)
MPPI_INST(64)
#undef MPPI_INST
#define MPPI_CHAIN_INST(GC)                                                                          \
  template __global__ void chain_kernel<GC>(const DevInst*, const int2*, int, int, int);             \
  template __global__ void chain_persistent_kernel<GC>(const DevInst*, const int2*, int, unsigned int*, int, int, int);
MPPI_CHAIN_INST(1)
MPPI_CHAIN_INST(2)
MPPI_CHAIN_INST(4)
MPPI_CHAIN_INST(8)
#undef MPPI_CHAIN_INST

}  // namespace mppi
