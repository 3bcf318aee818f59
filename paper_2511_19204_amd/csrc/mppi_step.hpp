// mppi_step.hpp -- device functions the rollout kernels share: the counter-based
// stream and the knot sampler, the Hermite reference, the per-body physics of a
// step (PD law, kinematics, inertias, soft contact, articulated-body steps, base
// solve), the costs and the base integration, and the body schedule's step.
#pragma once
#include "mppi_dev.hpp"

namespace mppi {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Branch-weight hint for a rare path when H holds (a compile-time constant),
// else the condition as is.  With one wavefront per SIMD every taken branch
// costs that wavefront an instruction refetch, so the legged and depth-6
// kernels ask for their rare paths to be laid out of line; the other kernels
// keep the default layout (with the hints their register allocation spills).  A macro: the hint
// has to sit in the branch's own condition.
#define MPPI_RARE(H, c) ((H) ? __builtin_expect(!!(c), 0) : !!(c))

// Philox4x32-10 (Salmon et al., SC'11).
__device__ __forceinline__ uint4 philox(uint4 c, uint2 k) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k.x += 0x9E3779B9u;
      k.y += 0xBB67AE85u;
    }
    // the 64-bit products give high and low words in one multiply each
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    c = make_uint4(hi1 ^ c.y ^ k.x, lo1, hi0 ^ c.w ^ k.y, lo0);
  }
  return c;
}

__device__ __forceinline__ float u01(uint32_t x) { return ((float)(x >> 9) + 0.5f) * 0x1p-23f; }

// 1-ulp hardware reciprocal and reciprocal square root (v_rcp_f32 / v_rsq_f32),
// used where a correctly rounded quotient is not required
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

// packed symmetric 6x6, upper triangle row by row
__host__ __device__ constexpr int SI(int i, int j) {
  return i <= j ? i * 6 - i * (i - 1) / 2 + (j - i) : j * 6 - j * (j - 1) / 2 + (i - j);
}

__device__ __forceinline__ void sym6_mv(const float* A, const float* x, float* y) {
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 6; ++j) s = fmaf(A[SI(i, j)], x[j], s);
    y[i] = s;
  }
}

__device__ __forceinline__ void cross3(const float* a, const float* b, float* c) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}

// rotation matrix of a unit quaternion (w, x, y, z), row-major
__device__ __forceinline__ void quat_R(const float* q, float* R) {
  const float w = q[0], x = q[1], y = q[2], z = q[3];
  R[0] = 1.f - 2.f * (y * y + z * z); R[1] = 2.f * (x * y - w * z); R[2] = 2.f * (x * z + w * y);
  R[3] = 2.f * (x * y + w * z); R[4] = 1.f - 2.f * (x * x + z * z); R[5] = 2.f * (y * z - w * x);
  R[6] = 2.f * (x * z - w * y); R[7] = 2.f * (y * z + w * x); R[8] = 1.f - 2.f * (x * x + y * y);
}

// 16-byte LDS transfers of slot records (addresses are 16-byte aligned)
__device__ __forceinline__ void put4(float* d, float a, float b, float c, float e) {
  *reinterpret_cast<float4*>(d) = make_float4(a, b, c, e);
}
__device__ __forceinline__ float4 get4(const float* s) { return *reinterpret_cast<const float4*>(s); }

// frame record: R (9), p (3), v (6), beta (6)
__device__ __forceinline__ void put_frame(float* d, const float* R, const float* p, const float* v, const float* bt) {
  put4(d, R[0], R[1], R[2], R[3]);
  put4(d + 4, R[4], R[5], R[6], R[7]);
  put4(d + 8, R[8], p[0], p[1], p[2]);
  put4(d + 12, v[0], v[1], v[2], v[3]);
  put4(d + 16, v[4], v[5], bt[0], bt[1]);
  put4(d + 20, bt[2], bt[3], bt[4], bt[5]);
}
__device__ __forceinline__ void get_frame(const float* s, float* R, float* p, float* v, float* bt) {
  const float4 a = get4(s), b = get4(s + 4), c = get4(s + 8), d = get4(s + 12), e = get4(s + 16), f = get4(s + 20);
  R[0] = a.x; R[1] = a.y; R[2] = a.z; R[3] = a.w; R[4] = b.x; R[5] = b.y; R[6] = b.z; R[7] = b.w; R[8] = c.x;
  p[0] = c.y; p[1] = c.z; p[2] = c.w;
  v[0] = d.x; v[1] = d.y; v[2] = d.z; v[3] = d.w; v[4] = e.x; v[5] = e.y;
  bt[0] = e.z; bt[1] = e.w; bt[2] = f.x; bt[3] = f.y; bt[4] = f.z; bt[5] = f.w;
}
// articulated inertia (21, packed) and bias (6) record, one float of padding
__device__ __forceinline__ void put_art(float* d, const float* Ip, const float* pp) {
#pragma unroll
  for (int k = 0; k < 5; ++k) put4(d + 4 * k, Ip[4 * k], Ip[4 * k + 1], Ip[4 * k + 2], Ip[4 * k + 3]);
  put4(d + 20, Ip[20], pp[0], pp[1], pp[2]);
  put4(d + 24, pp[3], pp[4], pp[5], 0.f);
}
__device__ __forceinline__ void add_art(const float* s, float* IA, float* pA) {
  float t[28];
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const float4 x = get4(s + 4 * k);
    t[4 * k] = x.x; t[4 * k + 1] = x.y; t[4 * k + 2] = x.z; t[4 * k + 3] = x.w;
  }
#pragma unroll
  for (int q = 0; q < 21; ++q) IA[q] += t[q];
#pragma unroll
  for (int q = 0; q < 6; ++q) pA[q] += t[21 + q];
}
// spatial acceleration record (6)
__device__ __forceinline__ void put_acc(float* d, const float* a) {
  put4(d, a[0], a[1], a[2], a[3]);
  *reinterpret_cast<float2*>(d + 4) = make_float2(a[4], a[5]);
}
__device__ __forceinline__ void get_acc(const float* s, float* a) {
  const float4 x = get4(s);
  const float2 y = *reinterpret_cast<const float2*>(s + 4);
  a[0] = x.x; a[1] = x.y; a[2] = x.z; a[3] = x.w; a[4] = y.x; a[5] = y.y;
}

// ---------------------------------------------------------------------------
// Per-lane physics of one step.  Lane b (< nb) owns body b and its joint.
//
// Frames: every body's spatial quantities are taken about its own joint origin
// p_b with the axes of the base frame B (world axes for a fixed base).  All
// these frames are inertial at the instant, so the articulated-body recursions
// keep their textbook form, while parent <-> child transforms reduce to pure
// translations by e_b = p_b - p_parent and lever arms stay one link long
// (referring everything to the base origin instead loses about three digits
// in float on a 6-deep leg).
// ---------------------------------------------------------------------------
struct StepIO {
  // inputs
  float q, v;          // joint state (revolute lanes)
  float bq[7], bv[6];  // base state (every lane of a floating-base rollout in the body schedule)
  float qref, vref;    // reference (revolute lanes)
  float dt;
  // outputs
  float qdd;           // joint acceleration
  float ba[6];         // base spatial acceleration, base coordinates (every lane of the rollout)
  float Rb[9];         // rotation of the base quaternion at the start of the step
  float tau;           // clipped PD torque
  float cost;          // running-cost terms of this lane (when want_cost)
  uint32_t mask;       // contact activity bits of this lane's contacts
};

// Per-lane constants of the body (and joint) a lane owns, loaded once per work item.
struct BodyConst {
  const float* P;     // joint rotation C(q) = P0 + cos q P1 + sin q P2, a row of the LDS table
  float p_tree[3], axis_p[3], com[3], Ic[6];
  float mass, kp, kd, taumax, arm, q0;
  int parent, depth, n_child, c_begin, c_count;
  float ct0[5];                 // first contact row: position (body frame), nominal normal force, index bits
  uint32_t child_lo, child_hi;  // children reached through LDS, 8 bits each, child-list order
  uint32_t flags;               // kAdjParent | kAdjChild | kFrameOut | kArtOut
};

// Transfers between a body and its first child in a depth-first numbering go
// through registers: the child (body b + 1) sits in the next lane, so one
// wavefront-wide shift by one lane moves a frame, an acceleration or an
// articulated inertia.  Other parent/child pairs go through the LDS slots.
constexpr uint32_t kAdjParent = 1u;  // joint body whose parent is the previous lane (a joint body)
constexpr uint32_t kAdjChild = 2u;   // first child is the next lane
constexpr uint32_t kFrameOut = 4u;   // joint body with a child that reads its frame and acceleration from LDS
constexpr uint32_t kArtOut = 8u;     // joint body whose parent reads its articulated inertia from LDS

__device__ __forceinline__ void load_body(const DevModel& M, const DevInst* I, int b, bool body_lane, const float* tab,
                                          BodyConst& c) {
  const int bb = body_lane ? b : 0;
  const int j = bb - M.fb;
  const bool joint = body_lane && j >= 0;
  c.P = tab + body_table_floats(M.nc) + bb * kPRow;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c.p_tree[k] = M.p_tree[bb][k];
    c.axis_p[k] = M.axis_p[bb][k];
    c.com[k] = M.com[bb][k];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) c.Ic[k] = M.Ic[bb][k];
  c.mass = M.mass[bb];
  c.kp = joint ? M.kp[j] : 0.f;
  c.kd = joint ? M.kd[j] : 0.f;
  c.taumax = joint ? M.taumax[j] : 0.f;
  c.arm = joint ? M.arm[j] : 0.f;
  c.q0 = (joint && I && I->cost_kind == 1) ? I->q0[j] : 0.f;
  c.parent = M.parent[bb];
  c.depth = body_lane ? M.depth[bb] : -1;
  c.c_begin = M.c_begin[bb];
  c.c_count = body_lane ? M.c_count[bb] : 0;
  {
    const float* ct = tab + kTabContacts + (c.c_count > 0 ? c.c_begin : 0) * kCt;
#pragma unroll
    for (int k = 0; k < 5; ++k) c.ct0[k] = ct[k];
  }
  // children are numbered after their parent in increasing order, so body b + 1,
  // when it is a child of b, is b's first child
  const int par = body_lane ? M.parent[bb] : -1;
  const int nch = body_lane ? M.n_child[bb] : 0;
  const bool adj_child = nch > 0 && M.child[bb][0] == bb + 1;
  c.flags = 0u;
  if (adj_child) c.flags |= kAdjChild;
  if (joint && par >= 0 && par == bb - 1 && !(M.fb && par == 0)) c.flags |= kAdjParent;
  if (joint && par >= 0 && bb != par + 1) c.flags |= kArtOut;
  c.n_child = 0;
  c.child_lo = c.child_hi = 0u;
  for (int k = 0; k < nch; ++k) {
    const int chb = M.child[bb][k];
    if (joint && chb != bb + 1) c.flags |= kFrameOut;
    if (k == 0 && adj_child) continue;
    const uint32_t ch = (uint32_t)chb & 0xffu;
    if (c.n_child < 4) c.child_lo |= ch << (8 * c.n_child);
    else c.child_hi |= ch << (8 * (c.n_child - 4));
    ++c.n_child;
  }
}
__device__ __forceinline__ int child_of(const BodyConst& c, int k) {
  return (int)(((k < 4 ? c.child_lo : c.child_hi) >> (8 * (k & 3))) & 0xffu);
}

// value held by the previous / next lane of the wavefront (DPP wave shift by one
// lane; every lane must be active; lanes past the wavefront's ends read 0)
__device__ __forceinline__ float from_prev_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_next_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x130, 0xf, 0xf, true));
}
// value held by lane l + N of this lane's row of 16 lanes (DPP row shift;
// every lane must be active; lanes past the row's end read 0)
template <int N>
__device__ __forceinline__ float from_row_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x100 + N, 0xf, 0xf, true));
}
// value held by another lane of this lane's quad (DPP quad permutation)
template <int CTRL>
__device__ __forceinline__ float qperm(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// value held by the first lane of this lane's rollout group of G lanes (groups
// are aligned): for G = 16 a DPP broadcast of each row's lane 0
// (row_newbcast:0), for G = 4 a quad permutation (0, 0, 0, 0), else a swizzle
// in bit-mask mode that clears the low lane-index bits within each 32-lane
// half, or the first lane for a whole wavefront; every lane must be active
template <int G>
__device__ __forceinline__ float from_group_lane0(float x) {
  if constexpr (G == 64) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
  } else if constexpr (G == 16) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150, 0xf, 0xf, false));
  } else if constexpr (G == 4) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x00, 0xf, 0xf, false));
  } else {
    constexpr int and_mask = 0x1f & ~(G - 1);
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), and_mask));
  }
}

// motion vector m given about point O, re-expressed about O + e: (w, v + w x e)
__device__ __forceinline__ void shift_motion(const float* m, const float* e, float* out) {
  float we[3];
  cross3(m, e, we);
  out[0] = m[0]; out[1] = m[1]; out[2] = m[2];
  out[3] = m[3] + we[0]; out[4] = m[4] + we[1]; out[5] = m[5] + we[2];
}

// Articulated inertia I (packed) about the child origin carried to the parent
// origin, e = child origin - parent origin: with E = e^x,
// C' = C,  B' = B + E C,  A' = A - B E - (B E)^T - E C E = A - B' E - (B E)^T
// (row r of X E is row r of X crossed with e).
__device__ __forceinline__ void shift_inertia_to_parent(const float* I, const float* e, float* O) {
  float B[9], C[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      B[r * 3 + c] = I[SI(r, c + 3)];
      C[r * 3 + c] = I[SI(r + 3, c + 3)];
    }
  // B' = B + E C: column k of E C is e x C[:, k]
  float Bp[9];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float col[3] = {C[k], C[3 + k], C[6 + k]};
    float o[3];
    cross3(e, col, o);
    Bp[k] = B[k] + o[0]; Bp[3 + k] = B[3 + k] + o[1]; Bp[6 + k] = B[6 + k] + o[2];
  }
  // (x cross e)[c] = x[c+1] e[c+2] - x[c+2] e[c+1]
  auto xe = [&](const float* x, int c) {
    const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    return x[c1] * e[c2] - x[c2] * e[c1];
  };
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = r; c < 3; ++c) O[SI(r, c)] = I[SI(r, c)] - xe(Bp + r * 3, c) - xe(B + c * 3, r);
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) O[SI(r, c + 3)] = Bp[r * 3 + c];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = r; c < 3; ++c) O[SI(r + 3, c + 3)] = I[SI(r + 3, c + 3)];
}

// ---------------------------------------------------------------------------
// Per-body physics shared by both rollout schedules.  Each helper is the
// arithmetic of one body (or joint) in one phase; the schedules differ only in
// which lane runs it and where its operands come from, so they produce the
// same bits.
// ---------------------------------------------------------------------------

// PD law (eq. pd-controller) with the torque clip; on unsaturated joints the
// damping and stiffness act implicitly through the gain dt (Kd + dt Kp).
__device__ __forceinline__ void pd_law(float kp, float kd, float tm, float dt, float q, float v, float qref, float vref,
                                       float& tau, float& gain) {
  const float t = kp * (qref - q) + kd * (vref - v);
  const bool inside = t < tm && t > -tm;
  tau = fminf(fmaxf(t, -tm), tm);
  gain = inside ? dt * (kd + dt * kp) : 0.f;
}

// velocity-product acceleration c = v x_m (S qd) of a revolute joint, S = (ax, 0)
__device__ __forceinline__ void vel_product(const float* v, const float* ax, float qd, float* c) {
  const float aq[3] = {ax[0] * qd, ax[1] * qd, ax[2] * qd};
  cross3(v, aq, c);
  cross3(v + 3, aq, c + 3);
}

// Joint rotation C(q) = P0 + cos q P1 + sin q P2 (row-major 3x3) from the 27
// constants P0 | P1 | P2 (read as 28 floats from a 16-byte aligned address).
__device__ __forceinline__ void load_rotation_constants(const float* P, float* t) {
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const float4 x = *reinterpret_cast<const float4*>(P + 4 * k);
    t[4 * k] = x.x; t[4 * k + 1] = x.y; t[4 * k + 2] = x.z; t[4 * k + 3] = x.w;
  }
}
__device__ __forceinline__ void joint_rotation_of(const float* t, float cq, float sq, float* C) {
#pragma unroll
  for (int k = 0; k < 9; ++k) C[k] = t[k] + cq * t[9 + k] + sq * t[18 + k];
}
__device__ __forceinline__ void joint_rotation(const float* P, float cq, float sq, float* C) {
  float t[28];
  load_rotation_constants(P, t);
  joint_rotation_of(t, cq, sq, C);
}

// Forward kinematics of a revolute body from its parent's frame (Rl, pl), twist
// vl and bias acceleration bl, with joint rotation C: rotation R = Rl C, origin
// p, lever arm e = p - pl, axis ax (base axes), twist v, velocity product c and
// bias acceleration beta, all about the body's own origin.
__device__ __forceinline__ void fk_joint(const float* Rl, const float* pl, const float* vl, const float* bl,
                                         const float* C, const float* p_tree, const float* axis_p, float qd, float* R,
                                         float* p, float* e, float* ax, float* v, float* c, float* beta) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc)
      R[r * 3 + cc] = Rl[r * 3 + 0] * C[0 * 3 + cc] + Rl[r * 3 + 1] * C[1 * 3 + cc] + Rl[r * 3 + 2] * C[2 * 3 + cc];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    e[r] = Rl[r * 3 + 0] * p_tree[0] + Rl[r * 3 + 1] * p_tree[1] + Rl[r * 3 + 2] * p_tree[2];
    p[r] = pl[r] + e[r];
    ax[r] = Rl[r * 3 + 0] * axis_p[0] + Rl[r * 3 + 1] * axis_p[1] + Rl[r * 3 + 2] * axis_p[2];
  }
  // v = shift(v_parent) + S qd with S = (axis, 0) about the joint origin
  shift_motion(vl, e, v);
  v[0] += ax[0] * qd; v[1] += ax[1] * qd; v[2] += ax[2] * qd;
  vel_product(v, ax, qd, c);
  float bs[6];
  shift_motion(bl, e, bs);
#pragma unroll
  for (int k = 0; k < 6; ++k) beta[k] = bs[k] + c[k];
}

// fk_joint for a child of the floating base, whose frame in base axes is the
// identity at the origin with twist bv and no bias acceleration: R = C(q),
// e = p = p_tree, ax = axis_p (the same values fk_joint gives for that parent).
__device__ __forceinline__ void fk_base_child(const float* bv, const float* C, const float* p_tree,
                                              const float* axis_p, float qd, float* R, float* p, float* e, float* ax,
                                              float* v, float* c, float* beta) {
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = C[k];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    e[r] = p_tree[r];
    p[r] = p_tree[r];
    ax[r] = axis_p[r];
  }
  shift_motion(bv, e, v);
  v[0] += ax[0] * qd; v[1] += ax[1] * qd; v[2] += ax[2] * qd;
  vel_product(v, ax, qd, c);
#pragma unroll
  for (int k = 0; k < 6; ++k) beta[k] = c[k];
}

// Spatial inertia (packed) of a rigid body about its origin in base axes, from
// its rotation R, com and inertia Ic about the com (body frame) and mass m.
__device__ __forceinline__ void body_inertia(const float* R, const float* com, const float* Ic, float m, float* IA) {
  float cw[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) cw[r] = R[r * 3 + 0] * com[0] + R[r * 3 + 1] * com[1] + R[r * 3 + 2] * com[2];
  const float Ib[9] = {Ic[0], Ic[3], Ic[4], Ic[3], Ic[1], Ic[5], Ic[4], Ic[5], Ic[2]};
  float RI[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc)
      RI[r * 3 + cc] = R[r * 3 + 0] * Ib[0 * 3 + cc] + R[r * 3 + 1] * Ib[1 * 3 + cc] + R[r * 3 + 2] * Ib[2 * 3 + cc];
  const float c2 = cw[0] * cw[0] + cw[1] * cw[1] + cw[2] * cw[2];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int cc = r; cc < 3; ++cc) {
      const float iw = RI[r * 3 + 0] * R[cc * 3 + 0] + RI[r * 3 + 1] * R[cc * 3 + 1] + RI[r * 3 + 2] * R[cc * 3 + 2];
      IA[SI(r, cc)] = iw + m * ((r == cc ? c2 : 0.f) - cw[r] * cw[cc]);
    }
  IA[SI(0, 3)] = 0.f;        IA[SI(0, 4)] = -m * cw[2]; IA[SI(0, 5)] = m * cw[1];
  IA[SI(1, 3)] = m * cw[2];  IA[SI(1, 4)] = 0.f;        IA[SI(1, 5)] = -m * cw[0];
  IA[SI(2, 3)] = -m * cw[1]; IA[SI(2, 4)] = m * cw[0];  IA[SI(2, 5)] = 0.f;
  IA[SI(3, 3)] = m; IA[SI(3, 4)] = 0.f; IA[SI(3, 5)] = 0.f;
  IA[SI(4, 4)] = m; IA[SI(4, 5)] = 0.f; IA[SI(5, 5)] = m;
}

// bias force v x_f (I v)
__device__ __forceinline__ void bias_force(const float* IA, const float* v, float* pA) {
  float h[6];
  sym6_mv(IA, v, h);
  float t0[3], t1[3], t2[3];
  cross3(v, h, t0);
  cross3(v + 3, h + 3, t1);
  cross3(v, h + 3, t2);
  pA[0] = t0[0] + t1[0]; pA[1] = t0[1] + t1[1]; pA[2] = t0[2] + t1[2];
  pA[3] = t2[0]; pA[4] = t2[1]; pA[5] = t2[2];
}

// One soft contact point at r (body frame) on a body with frame (R, p), twist v
// and bias acceleration beta; frame B is (Rb, pb) in the world, agl is gravity
// in B axes.  Adds the contact force to the bias pA and, while the point
// penetrates, the linearly implicit damping/friction terms to IA and pA.
// Returns the normal force; vw and fw are the point's world velocity and force.
// Position-only spline variants (spline ablation, Sec. V): knot slopes dq/dt
// derived from the position knots and kept in the velocity block, so the curve
// is evaluated in Hermite form.  Natural cubic spline (mode 1): C2 at interior
// knots, zero end second derivatives, i.e. the tridiagonal system
// m_{k-1} + 4 m_k + m_{k+1} = 3 (q_{k+1} - q_{k-1}) / Delta with end rows
// (2, 1) and (1, 2); its eliminated diagonal depends on K only.  Quadratic
// spline (mode 2): m_0 = 0, m_{k+1} = 2 (q_{k+1} - q_k) / Delta - m_k.
__device__ __forceinline__ void natural_cubic_diagonal(int K, float* dg) {
  float d = 2.f;
  dg[0] = d;
  for (int k = 1; k < K; ++k) {
    const float w = 1.f / d;
    d = (k == K - 1 ? 2.f : 4.f) - w;
    dg[k] = d;
  }
}

// Slopes of joint jj for a knot vector in LDS (positions in [0, K nu),
// slopes written to [K nu, 2 K nu)); dg = natural_cubic_diagonal(K) for mode 1.
__device__ __forceinline__ void position_spline_slopes(int mode, int K, int nu, int jj, float delta, const float* dg,
                                                       float* knots) {
  const float* Q = knots;
  float* V = knots + K * nu;
  if (mode == 2) {
    float m = 0.f;
    V[jj] = m;
    for (int k = 0; k + 1 < K; ++k) {
      m = 2.f * (Q[(k + 1) * nu + jj] - Q[k * nu + jj]) / delta - m;
      V[(k + 1) * nu + jj] = m;
    }
    return;
  }
  // forward elimination (right-hand sides into V), then back substitution
  float prev = 0.f;
  for (int k = 0; k < K; ++k) {
    const float qa = Q[(k == 0 ? 0 : k - 1) * nu + jj], qb = Q[(k == K - 1 ? K - 1 : k + 1) * nu + jj];
    float r = 3.f * (qb - qa) / delta;
    if (k > 0) r -= (1.f / dg[k - 1]) * prev;
    V[k * nu + jj] = r;
    prev = r;
  }
  float next = V[(K - 1) * nu + jj] / dg[K - 1];
  V[(K - 1) * nu + jj] = next;
  for (int k = K - 2; k >= 0; --k) {
    next = (V[k * nu + jj] - next) / dg[k];
    V[k * nu + jj] = next;
  }
}

struct ContactLaw {
  float k, d, mu, eps;
};

// Model and instance scalars every step reads, loaded into registers once per
// work item (read through the model pointer inside the step loop, the compiler
// would reload them after every LDS store).
struct StepConst {
  int fb, max_depth, ee_body, cost_kind, K, nu, F, nsub, spline_mode;
  float g, dt, delta, inv_delta, inv_F;
  ContactLaw law;
  float ee_pos[3];
  float w_h, w_or, w_q, w_cv, w_cf, w_eff, w_ee, w_tau, z_des;
  int or_target;
  float q_des[4];
};
__device__ __forceinline__ StepConst load_step_const(const DevModel& M, const DevInst* I, float dt_override) {
  StepConst c;
  c.fb = M.fb; c.max_depth = M.max_depth; c.ee_body = M.ee_body; c.nsub = M.nsub;
  c.g = M.g;
  c.law = ContactLaw{M.k, M.d, M.mu, M.eps};
  c.ee_pos[0] = M.ee_pos[0]; c.ee_pos[1] = M.ee_pos[1]; c.ee_pos[2] = M.ee_pos[2];
  if (I) {
    c.cost_kind = I->cost_kind; c.K = I->K; c.nu = I->nu; c.F = I->H * M.nsub; c.spline_mode = I->spline_mode;
    c.dt = I->dt / (float)M.nsub;
    c.delta = I->delta; c.inv_delta = 1.f / I->delta; c.inv_F = 1.f / (float)c.F;
    c.w_h = I->w_h; c.w_or = I->w_or; c.w_q = I->w_q; c.w_cv = I->w_cv; c.w_cf = I->w_cf; c.w_eff = I->w_eff;
    const DevTargets& tg = *I->targets;
    c.w_ee = I->w_ee; c.w_tau = I->w_tau; c.z_des = tg.z_des;
    c.or_target = tg.or_target;
    c.q_des[0] = tg.q_des[0]; c.q_des[1] = tg.q_des[1]; c.q_des[2] = tg.q_des[2]; c.q_des[3] = tg.q_des[3];
  } else {
    c.cost_kind = -1; c.K = 2; c.nu = M.nu; c.F = 1; c.spline_mode = 0;
    c.dt = dt_override;
    c.delta = 1.f; c.inv_delta = 1.f; c.inv_F = 1.f;
    c.w_h = c.w_or = c.w_q = c.w_cv = c.w_cf = c.w_eff = c.w_ee = c.w_tau = c.z_des = 0.f;
    c.or_target = 0;
    c.q_des[0] = 1.f; c.q_des[1] = c.q_des[2] = c.q_des[3] = 0.f;
  }
  return c;
}

// Stage the model table (contact rows with the instance's nominal
// normal forces) into LDS with all 64 lanes of the wavefront.
__device__ __forceinline__ void stage_model_table(const DevModel& M, const DevInst* I, float* tab, int lane,
                                                  bool joint_rows = false) {
  const float* cs = &M.ctab[0][0];
  for (int i = lane; i < M.nc * kCt; i += 64) tab[kTabContacts + i] = cs[i];
  if (joint_rows) {
    float* rows = tab + body_table_floats(M.nc);
    for (int i = lane; i < M.nb * 27; i += 64) rows[(i / 27) * kPRow + i % 27] = M.P[i / 27][i % 27];
  }
  wave_sync();
  if (I && I->cost_kind == 1)
    for (int ci = lane; ci < M.nc; ci += 64) {
      float* ct = tab + kTabContacts + ci * kCt;
      ct[3] = I->f0z[__float_as_int(ct[4])];
    }
  if (I && I->spline_mode == 1 && lane == 0) natural_cubic_diagonal(I->K, tab + kTabSpline);
  wave_sync();
}
__device__ __forceinline__ float contact_point(const float* r, const float* R, const float* p, const float* v,
                                               const float* beta, const float* Rb, const float* pb, const float* agl,
                                               float dt, const ContactLaw& law, float* IA, float* pA, float* vw,
                                               float* fw) {
  const float r0 = r[0], r1 = r[1], r2 = r[2];
  float x[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) x[q] = R[q * 3 + 0] * r0 + R[q * 3 + 1] * r1 + R[q * 3 + 2] * r2;
  float wx[3];
  cross3(v, x, wx);
  const float vB[3] = {v[3] + wx[0], v[4] + wx[1], v[5] + wx[2]};
  const float xB[3] = {p[0] + x[0], p[1] + x[1], p[2] + x[2]};
  float pw[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    pw[q] = pb[q] + Rb[q * 3 + 0] * xB[0] + Rb[q * 3 + 1] * xB[1] + Rb[q * 3 + 2] * xB[2];
    vw[q] = Rb[q * 3 + 0] * vB[0] + Rb[q * 3 + 1] * vB[1] + Rb[q * 3 + 2] * vB[2];
  }
  float fn = 0.f;
  if (pw[2] < 0.f) fn = fmaxf(0.f, -law.k * pw[2] - law.d * vw[2]);
  const float n2 = vw[0] * vw[0] + vw[1] * vw[1] + law.eps * law.eps;
  const float inv_nrm = rsq(n2);
  const float mfn = law.mu * fn * inv_nrm;
  fw[0] = -mfn * vw[0]; fw[1] = -mfn * vw[1]; fw[2] = fn;
  float fB[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) fB[q] = Rb[0 * 3 + q] * fw[0] + Rb[1 * 3 + q] * fw[1] + Rb[2 * 3 + q] * fw[2];
  float xf[3];
  cross3(x, fB, xf);
  pA[0] -= xf[0]; pA[1] -= xf[1]; pA[2] -= xf[2];
  pA[3] -= fB[0]; pA[4] -= fB[1]; pA[5] -= fB[2];
  if (fn > 0.f) {
    // Velocity Jacobian of the contact law (world), tangential-normal coupling
    // dropped: D_w = a I + (d - a) z z^T - a w w^T with a = mu f_n / n and
    // w = v_t / n.  In B axes z -> zb (third row of Rb) and w -> ub = Rb^T w.
    const float aa = mfn;
    const float al = law.d - aa;
    const float zb[3] = {Rb[6], Rb[7], Rb[8]};
    const float wt[2] = {vw[0] * inv_nrm, vw[1] * inv_nrm};
    const float ub[3] = {Rb[0] * wt[0] + Rb[3] * wt[1], Rb[1] * wt[0] + Rb[4] * wt[1], Rb[2] * wt[0] + Rb[5] * wt[1]};
    // added inertia dt P^T D P with P = [-x^x, 1]: with P^T zb = (x x zb, zb) = y1 and
    // P^T ub = (x x ub, ub) = y2 it is dt (al y1 y1^T - a y2 y2^T + a P^T P), where
    // P^T P has blocks |x|^2 I - x x^T, x^x and I
    float w1[3], w2[3];
    cross3(x, zb, w1);
    cross3(x, ub, w2);
    const float x2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
    const float dta = dt * aa, dtal = dt * al;
    const float y1[6] = {w1[0], w1[1], w1[2], zb[0], zb[1], zb[2]};
    const float y2[6] = {w2[0], w2[1], w2[2], ub[0], ub[1], ub[2]};
    float t1[6], t2[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) { t1[r] = dtal * y1[r]; t2[r] = dta * y2[r]; }
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int cc = r; cc < 6; ++cc) IA[SI(r, cc)] += t1[r] * y1[cc] - t2[r] * y2[cc];
    const float dax[3] = {dta * x[0], dta * x[1], dta * x[2]};
    const float dx2 = dta * x2;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int cc = q; cc < 3; ++cc) IA[SI(q, cc)] += (q == cc ? dx2 : 0.f) - dax[q] * x[cc];
    // dt a x^x in the top-right block, dt a I in the bottom-right block
    IA[SI(0, 4)] -= dax[2]; IA[SI(0, 5)] += dax[1];
    IA[SI(1, 3)] += dax[2]; IA[SI(1, 5)] -= dax[0];
    IA[SI(2, 3)] -= dax[1]; IA[SI(2, 4)] += dax[0];
    IA[SI(3, 3)] += dta; IA[SI(4, 4)] += dta; IA[SI(5, 5)] += dta;
    // bias of the added inertia: dt P^T D P (a_g - beta) = dt (x x Dw', Dw'), w' = P (a_g - beta)
    const float sa[3] = {-beta[0], -beta[1], -beta[2]};
    const float sl[3] = {agl[0] - beta[3], agl[1] - beta[4], agl[2] - beta[5]};
    float sx[3];
    cross3(sa, x, sx);
    const float w3[3] = {sl[0] + sx[0], sl[1] + sx[1], sl[2] + sx[2]};
    const float zw = zb[0] * w3[0] + zb[1] * w3[1] + zb[2] * w3[2];
    const float uw = ub[0] * w3[0] + ub[1] * w3[1] + ub[2] * w3[2];
    float Dw3[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) Dw3[q] = aa * w3[q] + al * zw * zb[q] - aa * uw * ub[q];
    float xd[3];
    cross3(x, Dw3, xd);
    pA[0] += dt * xd[0]; pA[1] += dt * xd[1]; pA[2] += dt * xd[2];
    pA[3] += dt * Dw3[0]; pA[4] += dt * Dw3[1]; pA[5] += dt * Dw3[2];
  }
  return fn;
}

// running-cost terms of one contact point (Sec. IV-A)
__device__ __forceinline__ void contact_cost(const StepConst& sc, float fn, const float* vw, const float* fw, float f0z,
                                             float& lane_cost) {
  if (fn > 0.f) lane_cost += sc.w_cv * (fabsf(vw[0]) + fabsf(vw[1]) + fabsf(vw[2]));
  lane_cost += sc.w_cf * (fabsf(fw[0]) + fabsf(fw[1]) + fabsf(fw[2] - f0z));
}

// end-effector height error: world z of the point ee_pos on a body (R, p) minus z_des
__device__ __forceinline__ float ee_height_error(const float* R, const float* p, const float* ee_pos, const float* Rb,
                                                 const float* pb, float z_des) {
  float xe[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) xe[r] = p[r] + R[r * 3 + 0] * ee_pos[0] + R[r * 3 + 1] * ee_pos[1] + R[r * 3 + 2] * ee_pos[2];
  return pb[2] + Rb[6] * xe[0] + Rb[7] * xe[1] + Rb[8] * xe[2] - z_des;
}

// atan2(y, x) for y, x >= 0: t = min / max in [0, 1], reduced to |u| <= tan(pi/12)
// by atan t = pi/6 + atan((sqrt(3) t - 1) / (t + sqrt(3))) where t > tan(pi/12),
// then the Taylor series of atan u to the u^13 term (truncation below 2e-10);
// atan2 = pi/2 - atan t when y > x.
__device__ __forceinline__ float atan2_pos(float y, float x) {
  const float hi = fmaxf(y, x), lo = fminf(y, x);
  const float t = hi > 0.f ? lo * rcp(hi) : 0.f;
  const float kTan15 = 0.267949192f, kSqrt3 = 1.73205081f;
  const bool big = t > kTan15;
  const float u = big ? (kSqrt3 * t - 1.f) * rcp(t + kSqrt3) : t;
  const float u2 = u * u;
  float sr = 1.f / 13.f;
  sr = fmaf(sr, u2, -1.f / 11.f);
  sr = fmaf(sr, u2, 1.f / 9.f);
  sr = fmaf(sr, u2, -1.f / 7.f);
  sr = fmaf(sr, u2, 1.f / 5.f);
  sr = fmaf(sr, u2, -1.f / 3.f);
  float a = fmaf(sr * u2, u, u);
  if (big) a += 0.523598776f;  // pi/6
  return y > x ? 1.57079633f - a : a;
}

// running-cost terms of the floating base (Sec. IV-A): height error and the
// squared rotation angle between the base and the task's orientation target
// (the identity unless a target is set).
__device__ __forceinline__ float base_cost_term(const StepConst& sc, const float* bq) {
  // orientation residual: rotation angle of R_base^T R_des, i.e. of conj(q_base) q_des
  const float* qt = bq + 3;
  float r0 = qt[0], r1 = qt[1], r2 = qt[2], r3 = qt[3];
  if (sc.or_target) {
    const float d0 = sc.q_des[0], d1 = sc.q_des[1], d2 = sc.q_des[2], d3 = sc.q_des[3];
    r0 = qt[0] * d0 + qt[1] * d1 + qt[2] * d2 + qt[3] * d3;
    r1 = qt[0] * d1 - qt[1] * d0 - qt[2] * d3 + qt[3] * d2;
    r2 = qt[0] * d2 + qt[1] * d3 - qt[2] * d0 - qt[3] * d1;
    r3 = qt[0] * d3 - qt[1] * d2 + qt[2] * d1 - qt[3] * d0;
  }
  const float vn2 = r1 * r1 + r2 * r2 + r3 * r3;
  const float vn = vn2 > 0.f ? vn2 * rsq(vn2) : 0.f;
  const float phi = 2.f * atan2_pos(vn, fabsf(r0));
  return sc.w_h * fabsf(bq[2] - sc.z_des) + sc.w_or * phi * phi;
}

// running-cost terms of a body other than its contacts (Sec. IV-A; effort and
// end-effector terms of the planar-chain task); base_term from base_cost_term
__device__ __forceinline__ void body_cost(const StepConst& sc, int b, bool is_base, bool is_joint, float base_term,
                                          float q, float q0, float tau, const float* R, const float* p,
                                          const float* Rb, const float* pb, float& lane_cost) {
  if (sc.cost_kind == 1) {
    if (is_base) lane_cost += base_term;
    if (is_joint) {
      const float eq = q - q0;
      lane_cost += sc.w_q * eq * eq + sc.w_eff * tau * tau;
    }
  } else {
    if (is_joint) lane_cost += sc.w_tau * tau * tau;
    if (b == sc.ee_body) {
      const float dz = ee_height_error(R, p, sc.ee_pos, Rb, pb, sc.z_des);
      lane_cost += sc.w_ee * dz * dz;
    }
  }
}

// Articulated-body step of a revolute joint (Featherstone's ABA pass 2 in the
// base-axes, own-origin frames): from the body's articulated inertia IA and
// bias pA (children already added) computes U = IA S, 1/D, u and the inertia
// and bias (Ip, pp) carried to the parent's origin.  D includes the armature and
// the implicit PD gain.
__device__ __forceinline__ void backward_joint(const float* IA, const float* pA, const float* ax, const float* c,
                                               const float* e, float tau, float arm, float gain, float* U,
                                               float& invD, float& u, float* Ip, float* pp) {
  // S = (ax, 0): U = IA S, D = S.U + g, u = tau - S.pA
#pragma unroll
  for (int r = 0; r < 6; ++r) U[r] = IA[SI(r, 0)] * ax[0] + IA[SI(r, 1)] * ax[1] + IA[SI(r, 2)] * ax[2];
  const float Dv = (arm + gain) + (ax[0] * U[0] + ax[1] * U[1] + ax[2] * U[2]);
  invD = rcp(Dv);
  u = tau - (ax[0] * pA[0] + ax[1] * pA[1] + ax[2] * pA[2]);
  // Ia = IA - U U^T / D, with W = U / D
  float W[6];
#pragma unroll
  for (int r = 0; r < 6; ++r) W[r] = U[r] * invD;
  float Ia[21];
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int cc = r; cc < 6; ++cc) Ia[SI(r, cc)] = IA[SI(r, cc)] - U[r] * W[cc];
  float Iac[6];
  sym6_mv(Ia, c, Iac);
  const float uD = u * invD;
  float pa[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) pa[q] = pA[q] + Iac[q] + U[q] * uD;
  shift_inertia_to_parent(Ia, e, Ip);
  float ef[3];
  cross3(e, pa + 3, ef);
  pp[0] = pa[0] + ef[0]; pp[1] = pa[1] + ef[1]; pp[2] = pa[2] + ef[2];
  pp[3] = pa[3]; pp[4] = pa[4]; pp[5] = pa[5];
}

// Floating-base root: solves IA0 a0' = -pA0 by Cholesky (a0' = a0 - a_g).
__device__ __forceinline__ void base_solve(const float* IA, const float* pA, float* a0) {
  float L[21], invL[6];
#pragma unroll
  for (int q = 0; q < 21; ++q) L[q] = IA[q];
  // in-place Cholesky of the packed symmetric matrix (lower factor stored as L[SI(i,j)], j <= i)
#pragma unroll
  for (int jj = 0; jj < 6; ++jj) {
    float dsum = L[SI(jj, jj)];
#pragma unroll
    for (int k = 0; k < jj; ++k) dsum -= L[SI(jj, k)] * L[SI(jj, k)];
    const float inv = rsq(dsum);
    invL[jj] = inv;
    L[SI(jj, jj)] = dsum * inv;
#pragma unroll
    for (int i = jj + 1; i < 6; ++i) {
      float sm = L[SI(i, jj)];
#pragma unroll
      for (int k = 0; k < jj; ++k) sm -= L[SI(i, k)] * L[SI(jj, k)];
      L[SI(i, jj)] = sm * inv;
    }
  }
  float y[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    float sm = -pA[i];
#pragma unroll
    for (int k = 0; k < i; ++k) sm -= L[SI(i, k)] * y[k];
    y[i] = sm * invL[i];
  }
#pragma unroll
  for (int i = 5; i >= 0; --i) {
    float sm = y[i];
#pragma unroll
    for (int k = i + 1; k < 6; ++k) sm -= L[SI(k, i)] * a0[k];
    a0[i] = sm * invL[i];
  }
}

// ABA pass 3 for a revolute joint: parent acceleration al (gravity-offset, about
// the parent origin) -> joint acceleration qdd and the body's own a'.
__device__ __forceinline__ float forward_joint(const float* al, const float* e, const float* c, const float* U, float u,
                                               float invD, const float* ax, float* aout) {
  float a[6];
  shift_motion(al, e, a);
#pragma unroll
  for (int q = 0; q < 6; ++q) a[q] += c[q];
  float Ua = 0.f;
#pragma unroll
  for (int q = 0; q < 6; ++q) Ua = fmaf(U[q], a[q], Ua);
  const float qdd = (u - Ua) * invD;
  aout[0] = a[0] + ax[0] * qdd; aout[1] = a[1] + ax[1] * qdd; aout[2] = a[2] + ax[2] * qdd;
  aout[3] = a[3]; aout[4] = a[4]; aout[5] = a[5];
  return qdd;
}

// ---------------------------------------------------------------------------
// Body schedule: one lane per body, the tree swept level by level through LDS.
// terminal = true evaluates only the kinematics and the end-effector height term
// of the terminal cost (end-effector task) at the current state.
// ---------------------------------------------------------------------------
// D > 0: the tree is at most D levels deep, fixed at compile time so the level
// loops unroll (levels below the tree have no body and cost only their shifts).
// Unroll counts of the loops over levels 1..D and D..0 (1: a run-time loop).
// A body's kinematics in a physics step (base axes, about the body origin):
// rotation R, origin p, lever arm e from the parent origin, joint axis ax,
// twist v, velocity product c and bias acceleration beta.  The base's R, p and
// beta are the identity frame and zero (base_frame).  The legged-tree kernels
// keep it across steps (set once by init_kin): a lane whose frame a neighbour
// reads before the lane's own level then hands over its previous step's
// values, which the neighbour does not use (the compiler would otherwise
// materialise the not-yet-computed values); the other kernels, with less
// register room, take it fresh every step.
struct BodyKin {
  float R[9], p[3], e[3], ax[3], v[6], c[6], beta[6];
};
__device__ __forceinline__ void base_frame(BodyKin& k) {
#pragma unroll
  for (int i = 0; i < 9; ++i) k.R[i] = (i % 4 == 0) ? 1.f : 0.f;
#pragma unroll
  for (int i = 0; i < 3; ++i) k.p[i] = 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) k.beta[i] = 0.f;
}
__device__ __forceinline__ void init_kin(BodyKin& k) {
  base_frame(k);
#pragma unroll
  for (int i = 0; i < 3; ++i) k.e[i] = k.ax[i] = 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) k.v[i] = k.c[i] = 0.f;
}

template <int D> constexpr int kLevelUnroll = D > 0 ? D : 1;
template <int D> constexpr int kLevelUnrollRoot = D > 0 ? D + 1 : 1;

// LEG = 1: the tree is a floating base with serial chains hanging off it
// (every joint body's parent is the previous lane, or the base for a chain's
// first body; no body but the base has more than one child), so a frame, an
// acceleration or a carried inertia always comes from the neighbouring lane
// except the base's, which gathers the chains through LDS.  LEG = 2: such a
// tree with four chains of three bodies in groups of 16 lanes (the chains'
// first bodies at lanes 1, 4, 7 and 10), whose base gathers the chains by row
// shifts instead.  LEG = 3: a fixed-base serial chain (body b's parent is body
// b - 1, the first body's the world), so every hand-over is a neighbour's and
// nothing goes through LDS.  The same arithmetic as the general form (children
// added in the same order), with its LDS paths and their branches compiled out.
template <int G, int D = 0, int LEG = 0>
__device__ void physics_step(const StepConst& sc, const BodyConst& bc, const float* tab, float* __restrict__ gs,
                             int b, bool body_lane, StepIO& io, BodyKin& kin_kept, bool want_cost,
                             bool terminal = false) {
  const int maxd = D > 0 ? D : sc.max_depth;
  // the joint-rotation constants are read first so the LDS latency passes
  // under the PD law, the base cost and frame B
  float Pt[28];
  load_rotation_constants(bc.P, Pt);
  float* slots = gs;
  const int fb = LEG == 3 ? 0 : (LEG != 0 ? 1 : sc.fb);  // legged trees have a floating base, serial chains not
  const bool is_base = body_lane && fb && b == 0;
  const bool is_joint = body_lane && !is_base;

  float tau = 0.f, gain = 0.f;
  if (is_joint) pd_law(bc.kp, bc.kd, bc.taumax, io.dt, io.q, io.v, io.qref, io.vref, tau, gain);
  io.tau = tau;
  float base_term = 0.f;
  if (want_cost && is_base && sc.cost_kind == 1) base_term = base_cost_term(sc, io.bq);

  // ---- frame B: world pose of the base.  Every lane carries the base state
  //      (position, quaternion, twist), so every lane forms it in registers.
  float* Rb = io.Rb;
  float pb[3];
  if (fb) {
    quat_R(io.bq + 3, Rb);
    pb[0] = io.bq[0]; pb[1] = io.bq[1]; pb[2] = io.bq[2];
  } else {
#pragma unroll
    for (int k = 0; k < 9; ++k) Rb[k] = (k % 4 == 0) ? 1.f : 0.f;
    pb[0] = pb[1] = pb[2] = 0.f;
  }

  // ---- forward kinematics, level by level (slot: R, p, v, beta about the body origin)
  BodyKin kin_step;  // the other kernels: fresh every step
  BodyKin& kin = LEG != 0 ? kin_kept : kin_step;
  float(&R)[9] = kin.R;
  float(&p)[3] = kin.p;
  float(&e)[3] = kin.e;
  float(&ax)[3] = kin.ax;
  float(&v)[6] = kin.v;
  float(&c)[6] = kin.c;
  float(&beta)[6] = kin.beta;
  const int depth = bc.depth;
  if (is_base) {  // (lever arm, axis and velocity product are never read for the base)
    if constexpr (LEG == 0) base_frame(kin);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = io.bv[k];
  }
  float C[9];
  if (is_joint) {
    float cq, sq;
    sincosf(io.q, &sq, &cq);
    joint_rotation_of(Pt, cq, sq, C);
  }
#pragma unroll kLevelUnroll<D>
  for (int d = 1; d <= maxd; ++d) {
    float sR[9], sp[3], sv[6], sb[6];  // the previous lane's frame (level d - 1)
    if (d > 1) {
#pragma unroll
      for (int k = 0; k < 9; ++k) sR[k] = from_prev_lane(R[k]);
#pragma unroll
      for (int k = 0; k < 3; ++k) sp[k] = from_prev_lane(p[k]);
#pragma unroll
      for (int k = 0; k < 6; ++k) { sv[k] = from_prev_lane(v[k]); sb[k] = from_prev_lane(beta[k]); }
    }
    if (is_joint && depth == d) {
      const int lam = bc.parent;
      if (fb && d == 1) {  // a child of the floating base: frame identity, twist bv
        fk_base_child(io.bv, C, bc.p_tree, bc.axis_p, io.v, R, p, e, ax, v, c, beta);
      } else {
        float Rl[9], pl[3], vl[6], bl[6];
        if (LEG == 3 ? d > 1 : (LEG != 0 || (bc.flags & kAdjParent))) {
#pragma unroll
          for (int k = 0; k < 9; ++k) Rl[k] = sR[k];
#pragma unroll
          for (int k = 0; k < 3; ++k) pl[k] = sp[k];
#pragma unroll
          for (int k = 0; k < 6; ++k) { vl[k] = sv[k]; bl[k] = sb[k]; }
        } else if (LEG != 3 && lam >= 0) {
          get_frame(slots + lam * kSlot, Rl, pl, vl, bl);
        } else {
#pragma unroll
          for (int k = 0; k < 9; ++k) Rl[k] = (k % 4 == 0) ? 1.f : 0.f;
#pragma unroll
          for (int k = 0; k < 3; ++k) pl[k] = 0.f;
#pragma unroll
          for (int k = 0; k < 6; ++k) { vl[k] = 0.f; bl[k] = 0.f; }
        }
        fk_joint(Rl, pl, vl, bl, C, bc.p_tree, bc.axis_p, io.v, R, p, e, ax, v, c, beta);
      }
      if (LEG == 0 && (bc.flags & kFrameOut)) put_frame(slots + b * kSlot, R, p, v, beta);
    }
    wave_sync();
  }

  // ---- rigid-body inertia, bias force, contacts (all body lanes in parallel)
  float IA[21], pA[6];
  float lane_cost = 0.f;
  uint32_t mask = 0u;
  if (terminal) {
    if (body_lane && sc.cost_kind == 0 && b == sc.ee_body) {
      const float dz = ee_height_error(R, p, sc.ee_pos, Rb, pb, sc.z_des);
      lane_cost = sc.w_ee * dz * dz;
    }
    io.cost = lane_cost;
    io.mask = 0u;
    wave_sync();
    return;
  }
  const float g = sc.g;
  // gravity as a spatial acceleration in B axes: (0, Rb^T (0, 0, -g)), the same about any origin
  const float agl[3] = {-g * Rb[6], -g * Rb[7], -g * Rb[8]};
  if (body_lane) {
    // every body's rigid inertia about its origin, the base's too (its frame is
    // the identity: every schedule forms it from the same constants the same way)
    body_inertia(R, bc.com, bc.Ic, bc.mass, IA);
    bias_force(IA, v, pA);

    // contacts carried by this body (point x relative to the body origin); the
    // first one's row is held in registers, further ones are read from the table
    // (LEG = 2: at most one contact per body, so no loop; the depth-6 kernels read
    // the first row from the table too, and spend the registers on the layout
    // hints of rollout_item)
    const int c0 = bc.c_begin, cn = LEG == 2 ? min(bc.c_count, 1) : bc.c_count;
    for (int ci = c0; ci < c0 + cn; ++ci) {
      float ct[5];
      if (ci == c0 && D != 6) {
#pragma unroll
        for (int k = 0; k < 5; ++k) ct[k] = bc.ct0[k];
      } else {
#pragma unroll
        for (int k = 0; k < 5; ++k) ct[k] = tab[kTabContacts + ci * kCt + k];
      }
      float vw[3], fw[3];
      const float fn = contact_point(ct, R, p, v, beta, Rb, pb, agl, io.dt, sc.law, IA, pA, vw, fw);
      if (fn > 0.f) mask |= 1u << __float_as_int(ct[4]);
      if (want_cost && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], lane_cost);
    }
    if (want_cost) body_cost(sc, b, is_base, is_joint, base_term, io.q, bc.q0, tau, R, p, Rb, pb, lane_cost);
  }
  io.cost = lane_cost;
  io.mask = mask;
  wave_sync();

  // ---- backward sweep, leaves to root: each joint lane publishes its
  //      articulated inertia and bias already carried to its parent's origin
  float U[6], invD = 0.f, u = 0.f;
  // kFoldAll (depth-specialised kernels): the inertia and bias carried to the
  // parent are zero until the lane's own level, then its body's (kept for the
  // rest of the sweep), and every lane adds its next lane's after each level.
  // The run-time-depth kernel keeps them per level (unset on lanes of other
  // levels) and adds them on the parents only.
  constexpr bool kFoldAll = D > 0;
  float Ip[21], pp[6];
  if constexpr (kFoldAll) {
#pragma unroll
    for (int q = 0; q < 21; ++q) Ip[q] = 0.f;
#pragma unroll
    for (int q = 0; q < 6; ++q) pp[q] = 0.f;
  }
#pragma unroll kLevelUnrollRoot<D>
  for (int d = maxd; d >= 0; --d) {
    if constexpr (LEG == 2) {
      if (d == 0) {
        // the base adds chains 2, 3 and 4 (lanes 4, 7 and 10 of the group) in
        // child order; every lane adds, only the base's sums are used (the
        // joint lanes' articulated inertias are no longer needed)
#pragma unroll
        for (int q = 0; q < 21; ++q) IA[q] += from_row_lane<4>(Ip[q]);
#pragma unroll
        for (int q = 0; q < 6; ++q) pA[q] += from_row_lane<4>(pp[q]);
#pragma unroll
        for (int q = 0; q < 21; ++q) IA[q] += from_row_lane<7>(Ip[q]);
#pragma unroll
        for (int q = 0; q < 6; ++q) pA[q] += from_row_lane<7>(pp[q]);
#pragma unroll
        for (int q = 0; q < 21; ++q) IA[q] += from_row_lane<10>(Ip[q]);
#pragma unroll
        for (int q = 0; q < 6; ++q) pA[q] += from_row_lane<10>(pp[q]);
      }
    }
    if (body_lane && depth == d) {
      const int nch = bc.n_child;
      if (LEG != 2 && LEG != 3 && (LEG == 0 || d == 0) && nch > 0) {
        // children reached through LDS: the first kFold records are read together
        // (a missing child reads this lane's own slot and is not added), then
        // added in child order; more children follow one by one
        constexpr int kFold = (D > 0 && D != 6) ? 3 : 2;  // (the generic and depth-6 kernels have fewer registers to spare)
        float t[kFold][28];
#pragma unroll
        for (int k = 0; k < kFold; ++k) {
          const float* src = slots + (k < nch ? child_of(bc, k) : b) * kSlot;
#pragma unroll
          for (int q = 0; q < 7; ++q) {
            const float4 x = get4(src + 4 * q);
            t[k][4 * q] = x.x; t[k][4 * q + 1] = x.y; t[k][4 * q + 2] = x.z; t[k][4 * q + 3] = x.w;
          }
        }
#pragma unroll
        for (int k = 0; k < kFold; ++k)
          if (k < nch) {
#pragma unroll
            for (int q = 0; q < 21; ++q) IA[q] += t[k][q];
#pragma unroll
            for (int q = 0; q < 6; ++q) pA[q] += t[k][21 + q];
          }
#pragma unroll 1
        for (int k = kFold; k < nch; ++k) add_art(slots + child_of(bc, k) * kSlot, IA, pA);
      }
      if (is_joint) {
        backward_joint(IA, pA, ax, c, e, tau, bc.arm, gain, U, invD, u, Ip, pp);
        if (LEG != 2 && LEG != 3 && (LEG == 0 || d == 1) && (bc.flags & kArtOut)) put_art(slots + b * kSlot, Ip, pp);
      }
    }
    wave_sync();
    if (d > 0) {
      // a parent at level d - 1 adds its first child's contribution first, then
      // the others'
      if constexpr (kFoldAll) {
        // every lane adds its next lane's carried inertia (one DPP add): in a
        // depth-first numbering the next body is this body's child iff it is
        // one level deeper, so a lane of level d - 1 takes its first child's; a
        // lane not yet swept takes a zero (its next lane is not swept yet
        // either); a lane already swept no longer needs its sums
#pragma unroll
        for (int q = 0; q < 21; ++q) IA[q] += from_next_lane(Ip[q]);
#pragma unroll
        for (int q = 0; q < 6; ++q) pA[q] += from_next_lane(pp[q]);
      } else {
        float sI[21], spp[6];
#pragma unroll
        for (int q = 0; q < 21; ++q) sI[q] = from_next_lane(Ip[q]);
#pragma unroll
        for (int q = 0; q < 6; ++q) spp[q] = from_next_lane(pp[q]);
        if (body_lane && depth == d - 1 && (bc.flags & kAdjChild)) {
#pragma unroll
          for (int q = 0; q < 21; ++q) IA[q] += sI[q];
#pragma unroll
          for (int q = 0; q < 6; ++q) pA[q] += spp[q];
        }
      }
    }
  }

  // ---- root: floating base solves IA0 a0' = -pA0 (Cholesky); fixed roots use -a_g
  float a0[6];  // the base's a' = a0 - a_g, then in every lane of its rollout
  if (is_base) base_solve(IA, pA, a0);
  if (fb) {
#pragma unroll
    for (int k = 0; k < 6; ++k) a0[k] = from_group_lane0<G>(a0[k]);
    io.ba[0] = a0[0]; io.ba[1] = a0[1]; io.ba[2] = a0[2];
    io.ba[3] = a0[3] + agl[0]; io.ba[4] = a0[4] + agl[1]; io.ba[5] = a0[5] + agl[2];
  }

  // ---- forward sweep: accelerations, root to leaves
  float qdd = 0.f;
  float a[6], sa[6];  // this lane's and the previous lane's acceleration
#pragma unroll kLevelUnroll<D>
  for (int d = 1; d <= maxd; ++d) {
    if (is_joint && depth == d) {
      const int lam = bc.parent;
      float al[6];
      if (fb && d == 1) {
#pragma unroll
        for (int k = 0; k < 6; ++k) al[k] = a0[k];
      } else if (LEG == 3 ? d > 1 : (LEG != 0 || (bc.flags & kAdjParent))) {
#pragma unroll
        for (int k = 0; k < 6; ++k) al[k] = sa[k];
      } else if (LEG != 3 && lam >= 0) {
        get_acc(slots + lam * kSlot, al);
      } else {
        // fixed world: a' = -a_g = (0, 0, 0, 0, 0, g); its angular part is zero, so no shift term
        al[0] = al[1] = al[2] = 0.f; al[3] = 0.f; al[4] = 0.f; al[5] = g;
      }
      qdd = forward_joint(al, e, c, U, u, invD, ax, a);
      if (LEG == 0 && (bc.flags & kFrameOut)) put_acc(slots + b * kSlot, a);
    }
    wave_sync();
    if (d < maxd) {
#pragma unroll
      for (int k = 0; k < 6; ++k) sa[k] = from_prev_lane(a[k]);
    }
  }
  io.qdd = qdd;
}

// ---------------------------------------------------------------------------
// Knot sampling for one rollout group: counter-based normals, perturbation,
// position clip and bound-aware velocity clamp.
// ---------------------------------------------------------------------------
// Sample n's position and velocity knot of one element (Alg. 1 sampling step:
// the nominal (nq, nv) perturbed by the iteration's std sq at the element's
// knot, the position clipped to the joint range [lo, hi], the velocity clamped
// by eq. vel-clamp) from the uniform words (xa, xb) of its counter-based block,
// by Box-Muller.  Sample 0 is the nominal itself (clipped and clamped the same
// way).  The rollout's sampler and the update's regeneration both call this, so
// they give the same bits.
struct ElemConst {
  float sq, lo, hi;  // std at the element's knot, joint range
  int m;             // element index k nu + jj
};
__device__ __forceinline__ ElemConst elem_const(const DevModel& M, const DevInst& I, const float* sig, int m) {
  const int k = m / I.nu, jj = m % I.nu;
  return ElemConst{sig[k], M.qmin[jj], M.qmax[jj], m};
}
__device__ __forceinline__ void perturb_element(const ElemConst& ec, float delta, float nq, float nv, int n,
                                                uint32_t xa, uint32_t xb, bool with_velocity, float& tq,
                                                float& tv) {
  float zq = 0.f, zv = 0.f;
  if (n > 0) {
    const float ua = u01(xa), ub = u01(xb);
    const float r = sqrtf(-2.f * logf(ua));
    zq = r * cospif(2.f * ub);
    zv = r * sinpif(2.f * ub);
  }
  tq = fminf(fmaxf(fmaf(ec.sq, zq, nq), ec.lo), ec.hi);
  tv = 0.f;
  if (with_velocity) {
    const float sv = ec.sq / delta;
    const float lim = 2.f * fminf(ec.hi - tq, tq - ec.lo) / delta;
    tv = fminf(fmaxf(fmaf(sv, zv, nv), -lim), lim);
  }
}

// The counter-based block blk of sample n in iteration I.iter at tick `tick`
// (key = seed; counter = (blk, n, iter, tick)); sample 0 draws none.
__device__ __forceinline__ uint4 sample_words(const DevInst& I, int n, int blk, uint32_t tick) {
  if (n == 0) return make_uint4(0u, 0u, 0u, 0u);
  return philox(make_uint4((uint32_t)blk, (uint32_t)n, (uint32_t)I.iter, tick), make_uint2(I.seed_lo, I.seed_hi));
}
__device__ __forceinline__ uint32_t sample_tick(const DevInst& I) {
  return I.use_tick_value ? I.tick_value : *I.tick_ptr;
}

// Knot sampling for one rollout group: block blk gives elements 2 blk and
// 2 blk + 1 (its words x, y and z, w); the lanes of the group take the blocks
// in turn.
template <int G>
__device__ void sample_group(const DevModel& M, const DevInst& I, int n, int l, float* knots, bool valid,
                             const float* tab, const float* nominal = nullptr) {
  const float* nom = nominal ? nominal : I.nominal;
  const int K = I.K, nu = I.nu, KU = K * nu;
  const int nblk = (KU + 1) / 2;
  const float* sig = I.sigma + I.iter * K;
  const uint32_t tick = sample_tick(I);
  const bool store = valid && I.store_samples;
  const bool with_v = I.spline_mode == 0;
  for (int blk = l; blk < nblk; blk += G) {
    const uint4 x = sample_words(I, n, blk, tick);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int m = 2 * blk + half;
      if (m >= KU) break;
      float tq, tv;
      perturb_element(elem_const(M, I, sig, m), I.delta, nom[m], with_v ? nom[KU + m] : 0.f, n,
                      half ? x.z : x.x, half ? x.w : x.y, with_v, tq, tv);
      knots[m] = tq;
      if (store) I.samples[(size_t)n * I.E + m] = tq;
      if (with_v) {
        knots[KU + m] = tv;
        if (store) I.samples[(size_t)n * I.E + KU + m] = tv;
      }
    }
  }
  if (I.spline_mode != 0) {
    // position-only variants: knot slopes of the spline through the sampled positions
    wave_sync();
    for (int jj = l; jj < nu; jj += G) {
      position_spline_slopes(I.spline_mode, K, nu, jj, I.delta, tab + kTabSpline, knots);
      if (store)
        for (int k = 0; k < K; ++k) I.samples[(size_t)n * I.E + KU + k * nu + jj] = knots[KU + k * nu + jj];
    }
  }
}

// Hermite reference of joint jj (eq. hermite_segment and its time derivative).
// The knots of one segment, slopes scaled by the knot spacing delta, are loaded
// once per segment; the curve is then evaluated at local time s in [0, 1].
struct HermiteSeg {
  float q0, q1, m0, m1;
};
__device__ __forceinline__ HermiteSeg hermite_segment(const float* knots, int K, int nu, int seg, int jj, float delta) {
  const int KU = K * nu;
  HermiteSeg h;
  h.q0 = knots[seg * nu + jj];
  h.q1 = knots[(seg + 1) * nu + jj];
  h.m0 = delta * knots[KU + seg * nu + jj];
  h.m1 = delta * knots[KU + (seg + 1) * nu + jj];
  return h;
}
__device__ __forceinline__ void hermite_eval(const HermiteSeg& h, float s, float inv_delta, float* qr, float* vr) {
  const float s2 = s * s, s3 = s2 * s;
  const float h00 = 2.f * s3 - 3.f * s2 + 1.f, h10 = s3 - 2.f * s2 + s, h01 = -2.f * s3 + 3.f * s2, h11 = s3 - s2;
  const float d00 = 6.f * s2 - 6.f * s, d10 = 3.f * s2 - 4.f * s + 1.f, d01 = -6.f * s2 + 6.f * s, d11 = 3.f * s2 - 2.f * s;
  *qr = h00 * h.q0 + h10 * h.m0 + h01 * h.q1 + h11 * h.m1;
  *vr = (d00 * h.q0 + d10 * h.m0 + d01 * h.q1 + d11 * h.m1) * inv_delta;
}
// At fine step f of F inside a rollout: the segment seg = floor(f (K-1) / F) and
// the remainder rem = f (K-1) - seg F are exact integers kept by the caller
// (StepClock); the local time is s = rem (1/F).
__device__ __forceinline__ void hermite(const float* knots, int K, int nu, float inv_F, float delta, float inv_delta,
                                        int seg, int rem, int jj, float* qr, float* vr) {
  hermite_eval(hermite_segment(knots, K, nu, seg, jj, delta), (float)rem * inv_F, inv_delta, qr, vr);
}

// Fine-step bookkeeping without integer division: the Hermite segment and
// remainder of step f (f (K-1) = seg F + rem, 0 <= rem < F; for f < F the
// segment never exceeds K-2), the substep within a control step and the
// control-step index.
struct StepClock {
  int seg = 0, rem = 0, sub = 0, h = 0;
  template <bool H = false>
  __device__ __forceinline__ void advance(int K, int F, int nsub) {
    rem += K - 1;
    while (MPPI_RARE(H, rem >= F)) {
      rem -= F;
      ++seg;
    }
    if (++sub == nsub) {
      sub = 0;
      ++h;
    }
  }
};

template <int G>
__device__ __forceinline__ float group_sum(float x, float* red, int l) {
  red[l] = x;
  wave_sync();
  float s = 0.f;
  if (l == 0)
    for (int k = 0; k < G; ++k) s += red[k];
  wave_sync();
  return s;
}

template <int G>
__device__ __forceinline__ uint32_t group_or(uint32_t x, float* red, int l) {
  uint32_t* r = reinterpret_cast<uint32_t*>(red);
  r[l] = x;
  wave_sync();
  uint32_t s = 0u;
  if (l == 0)
    for (int k = 0; k < G; ++k) s |= r[k];
  wave_sync();
  return s;
}

// semi-implicit Euler on the base: v += dt a, p += dt R(quat) v_lin, quat <- quat (x) exp(dt w)
// (R: the rotation of the quaternion bq[3..6], as quat_R gives it)
template <bool H = false>
__device__ __forceinline__ void integrate_base_R(float* bq, float* bv, const float* ba, float dt, const float* R) {
#pragma unroll
  for (int k = 0; k < 6; ++k) bv[k] = fmaf(dt, ba[k], bv[k]);
#pragma unroll
  for (int r = 0; r < 3; ++r) bq[r] += dt * (R[r * 3 + 0] * bv[3] + R[r * 3 + 1] * bv[4] + R[r * 3 + 2] * bv[5]);
  const float wn2 = bv[0] * bv[0] + bv[1] * bv[1] + bv[2] * bv[2];
  // exp of the half rotation: (cos th, sin th w / |w|), th = |w| dt / 2; below
  // th = 1/4 by the Taylor series of cos th and sin th / th to the th^6 term
  // (truncation below 5e-10, under float rounding), which needs th^2 only
  const float hdt = 0.5f * dt;
  const float t2 = (hdt * hdt) * wn2;
  float e0 = 1.f + t2 * (-0.5f + t2 * (1.f / 24.f + t2 * (-1.f / 720.f)));
  float k = hdt * (1.f + t2 * (-1.f / 6.f + t2 * (1.f / 120.f + t2 * (-1.f / 5040.f))));
  if (MPPI_RARE(H, !(t2 < 0.0625f))) {
    const float wn = sqrtf(wn2);
    float sn, cs;
    sincosf(hdt * wn, &sn, &cs);
    e0 = cs;
    k = sn * rcp(wn);
  }
  const float e1 = k * bv[0], e2 = k * bv[1], e3 = k * bv[2];
  const float a0 = bq[3], a1 = bq[4], a2 = bq[5], a3 = bq[6];
  const float r0 = a0 * e0 - a1 * e1 - a2 * e2 - a3 * e3;
  const float r1 = a0 * e1 + a1 * e0 + a2 * e3 - a3 * e2;
  const float r2 = a0 * e2 - a1 * e3 + a2 * e0 + a3 * e1;
  const float r3 = a0 * e3 + a1 * e2 - a2 * e1 + a3 * e0;
  const float inv = rsq(r0 * r0 + r1 * r1 + r2 * r2 + r3 * r3);
  bq[3] = r0 * inv; bq[4] = r1 * inv; bq[5] = r2 * inv; bq[6] = r3 * inv;
}
__device__ __forceinline__ void integrate_base(float* bq, float* bv, const float* ba, float dt) {
  float R[9];
  quat_R(bq + 3, R);
  integrate_base_R(bq, bv, ba, dt, R);
}

}  // namespace mppi
