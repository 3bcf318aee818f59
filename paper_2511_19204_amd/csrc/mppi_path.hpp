// mppi_path.hpp -- rollouts with one quad of lanes per root-to-leaf path of the tree.
//
// The tree is cut into its root-to-leaf paths (below the floating base, if
// there is one): the quadruped's four legs, the humanoid's legs and torso-arm
// paths, an arm.  Each path belongs to a quad of lanes, which walks it body by
// body; lane k of the quad (k = 0, 1, 2; the fourth lane repeats the third)
// holds component k of every 3-vector and row k of every 3x3 block, and the
// lanes meet through DPP quad permutations.  A body that several paths share
// (the humanoid's torso) is walked by each of them, with the same bits.  The
// floating base, which every path hangs off, is carried by every lane.
//
// What bounds a rollout is the instructions one wavefront issues per physics
// step (its dependency chain is too long to hide behind others at the usual
// sample counts).  One lane per body issues the whole sweep once per tree level
// with the other levels' lanes idle; here the sweeps keep three lanes in four
// busy and need no lane masks and no exchange between levels.  Issue slots
// (quarter-rate cycles) per step and wavefront, body schedule -> here: quadruped
// 2 213 -> 1 820, humanoid 5 085 -> 3 900, arm 1 650 -> 960; a launch at 256
// samples x 200 steps of the quadruped takes 0.78 -> 0.61 ms (4 096 samples: 0.74
// -> 0.64), at 256 x 150 of the humanoid 1.33 -> 1.01 ms, at 32 x 50 of the arm
// 0.140 -> 0.092 ms.  The form needs more than 256 registers, so a SIMD holds
// one wavefront of it.
//
// The results are the body schedule's bit for bit: every scalar is computed by
// the same expression in the same order (the quad permutations only decide
// which lane evaluates it), symmetric blocks hold U_min W_max in both
// triangles, and sums over children and costs keep their order.
#pragma once
#include "mppi_step.hpp"

namespace mppi {

// row of body i of path p for lane k in the LDS table
__device__ __forceinline__ int path_row(int p, int L, int i, int k) { return ((p * L + i) * 3 + k) * kPathRow; }

// components 0, 1, 2 of a vector held one component per lane
struct Rep3 {
  float x0, x1, x2;
};
__device__ __forceinline__ Rep3 rep3(float x) { return Rep3{qperm<0x00>(x), qperm<0x55>(x), qperm<0xAA>(x)}; }
__device__ __forceinline__ float quad0(float x) { return qperm<0x00>(x); }
__device__ __forceinline__ float quad2(float x) { return qperm<0xAA>(x); }
// component k + 1 and k + 2 (the fourth lane as the third)
__device__ __forceinline__ float rot1(float x) { return qperm<0x09>(x); }
__device__ __forceinline__ float rot2(float x) { return qperm<0x52>(x); }
// component min(k, 1) and max(k, 1): column 1 of a symmetric block
__device__ __forceinline__ float lo1(float x) { return qperm<0x54>(x); }
__device__ __forceinline__ float hi1(float x) { return qperm<0xA5>(x); }
// value of component k of (a, b, c)
__device__ __forceinline__ float own3(int k, float a, float b, float c) { return k == 0 ? a : (k == 1 ? b : c); }
template <int K>
__device__ __forceinline__ float quad_of(float x) {
  return qperm<K * 0x55>(x);
}
// component k of a x b, each operand's rotated components given
__device__ __forceinline__ float cross_k(float a1, float a2, float b1, float b2) { return a1 * b2 - a2 * b1; }
__device__ __forceinline__ float cross_k(float a, float b) { return cross_k(rot1(a), rot2(a), rot1(b), rot2(b)); }

// The hot blocks below are written in assembly because the compiler does not
// fold a lane permutation into a fused multiply-add: as DPP operands of
// v_mul_f32 / v_fmac_f32 the permutations cost no instruction, a quarter of the
// kernel's.  The values are those of the plain expressions in the comments.
// A DPP operand must not have been written by the two instructions before it:
// every block first issues instructions without DPP operands on its inputs (or
// an s_nop), since a register copy may stand in front of it, and inside a block a
// value is read through DPP at the earliest three instructions after it was
// written.  The build checks the machine code.
#define Q0 " quad_perm:[0,0,0,0]\n"
#define Q1 " quad_perm:[1,1,1,1]\n"
#define Q2 " quad_perm:[2,2,2,2]\n"
#define ROT1 " quad_perm:[1,2,0,0]\n"
#define ROT2 " quad_perm:[2,0,1,1]\n"
#define LO1 " quad_perm:[0,1,1,1]\n"
#define HI1 " quad_perm:[1,1,2,2]\n"
#define MUL "v_mul_f32_dpp "
#define FMAC "v_fmac_f32_dpp "
#define MOV "v_mov_b32_dpp "

// Rows of lane k of a spatial inertia [[A, B], [B^T, C]]: A[j], B[j], C[j] are
// entries (k, j) of the blocks, T[j] is entry (j, k) of B; bias (pa, pl).
struct PathInertia {
  float A[3], B[3], T[3], C[3], pa, pl;
};
__device__ __forceinline__ void add_inertia(PathInertia& x, const PathInertia& y) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    x.A[j] += y.A[j];
    x.B[j] += y.B[j];
    x.T[j] += y.T[j];
    x.C[j] += y.C[j];
  }
  x.pa += y.pa;
  x.pl += y.pl;
}

// Per-lane pattern of a skew block: entry (k, j) of x^x is sgn[j] times the
// component that skew_part<j> fetches.
template <int J>
__device__ __forceinline__ float skew_part(float x) {
  return qperm<J == 0 ? 0x58 : (J == 1 ? 0x06 : 0xA1)>(x);
}

// Constants of one body on its path, as lane k reads them (kPathRow floats).
struct PathFk {
  float P0[3], P1[3], P2[3], pt[3], ax[3], arm;
};
struct PathMass {
  float com[3], Ic[6], m, pt_k, ax_k;
};
__device__ __forceinline__ PathFk load_path_fk(const float* r) {
  const float4 a = get4(r), b = get4(r + 4), c = get4(r + 8), d = get4(r + 12);
  return PathFk{{a.x, a.y, a.z}, {a.w, b.x, b.y}, {b.z, b.w, c.x}, {c.y, c.z, c.w}, {d.x, d.y, d.z}, d.w};
}
__device__ __forceinline__ PathMass load_path_mass(const float* r) {
  const float4 a = get4(r + 16), b = get4(r + 20), c = get4(r + 24);
  return PathMass{{a.x, a.y, a.z}, {a.w, b.x, b.y, b.z, b.w, c.x}, c.y, c.z, c.w};
}

// Frame of one body: row k of R, component k of the origin p, the lever arm e,
// the axis, the twist v, the velocity product c and the bias acceleration beta.
struct PathFrame {
  float R[3], p, e, ax, va, vl, ca, cl, ba, bl;
};

// fk_joint / fk_base_child, one row per lane; ROOT: the parent is the floating
// base (twist of P) or the fixed world (P's twist zero), whose frame is the identity.
template <bool ROOT>
__device__ __forceinline__ void path_fk(const PathFk& K, float pt_k, float ax_k, const PathFrame& P, float cq, float sq,
                                        float qd, PathFrame& O) {
  float C[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) C[j] = K.P0[j] + cq * K.P1[j] + sq * K.P2[j];
  if constexpr (ROOT) {
#pragma unroll
    for (int j = 0; j < 3; ++j) O.R[j] = C[j];
    O.e = O.p = pt_k;
    O.ax = ax_k;
    const float e1 = rot1(O.e), e2 = rot2(O.e);
    const float we = cross_k(rot1(P.va), rot2(P.va), e1, e2);
    O.va = P.va;
    O.vl = P.vl + we;
    O.va += O.ax * qd;
    const float aq = O.ax * qd, aq1 = rot1(aq), aq2 = rot2(aq);
    O.ca = cross_k(rot1(O.va), rot2(O.va), aq1, aq2);
    O.cl = cross_k(rot1(O.vl), rot2(O.vl), aq1, aq2);
    O.ba = O.ca;
    O.bl = O.cl;
  } else {
    // e = R pt, ax = R axis_p, R' = R C (row C_r broadcast from lane r)
    asm("v_mul_f32 %0, %6, %12\n"
        "v_mul_f32 %1, %6, %15\n"
        "v_fmac_f32 %0, %5, %11\n"
        "v_fmac_f32 %1, %5, %14\n"
        "v_fmac_f32 %0, %7, %13\n"
        "v_fmac_f32 %1, %7, %16\n"
        MUL "%2, %8, %6" Q1 MUL "%3, %9, %6" Q1 MUL "%4, %10, %6" Q1
        FMAC "%2, %8, %5" Q0 FMAC "%3, %9, %5" Q0 FMAC "%4, %10, %5" Q0
        FMAC "%2, %8, %7" Q2 FMAC "%3, %9, %7" Q2 FMAC "%4, %10, %7" Q2
        : "=&v"(O.e), "=&v"(O.ax), "=&v"(O.R[0]), "=&v"(O.R[1]), "=&v"(O.R[2])
        : "v"(P.R[0]), "v"(P.R[1]), "v"(P.R[2]), "v"(C[0]), "v"(C[1]), "v"(C[2]), "v"(K.pt[0]), "v"(K.pt[1]),
          "v"(K.pt[2]), "v"(K.ax[0]), "v"(K.ax[1]), "v"(K.ax[2]));
    O.p = P.p + O.e;
    // va' = va + ax qd, vl' = vl + va x e, c = v' x (ax qd), beta' = shift(beta) + c
    float e1, e2, aq, bs;
    asm("v_mul_f32 %8, %11, %12\n"          // aq
        "v_fma_f32 %0, %11, %12, %13\n"     // va'
        "s_nop 0\n"
        MOV "%6, %10" ROT1 MOV "%7, %10" ROT2
        MUL "%1, -%13, %6" ROT2 FMAC "%1, %13, %7" ROT1
        MUL "%9, -%15, %6" ROT2 FMAC "%9, %15, %7" ROT1
        "v_add_f32 %1, %14, %1\n"           // vl'
        "v_add_f32 %9, %16, %9\n"           // shifted beta, linear
        MOV "%6, %8" ROT1 MOV "%7, %8" ROT2
        MUL "%2, -%0, %6" ROT2 FMAC "%2, %0, %7" ROT1
        MUL "%3, -%1, %6" ROT2 FMAC "%3, %1, %7" ROT1
        "v_add_f32 %4, %15, %2\n"
        "v_add_f32 %5, %9, %3\n"
        : "=&v"(O.va), "=&v"(O.vl), "=&v"(O.ca), "=&v"(O.cl), "=&v"(O.ba), "=&v"(O.bl), "=&v"(e1), "=&v"(e2), "=&v"(aq),
          "=&v"(bs)
        : "v"(O.e), "v"(O.ax), "v"(qd), "v"(P.va), "v"(P.vl), "v"(P.ba), "v"(P.bl));
  }
}

// body_inertia
__device__ __forceinline__ void path_inertia(const float* R, const PathMass& K, int k, const float* sgn, PathInertia& I) {
  const float m = K.m;
  const float Ib[9] = {K.Ic[0], K.Ic[3], K.Ic[4], K.Ic[3], K.Ic[1], K.Ic[5], K.Ic[4], K.Ic[5], K.Ic[2]};
  float RI[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) RI[c] = R[0] * Ib[c] + R[1] * Ib[3 + c] + R[2] * Ib[6 + c];
  // cw = R com; entry (r, c) of R Ib R^T is RI[r] . R[c] for r <= c
  float cw, iw[3], h0, h1, h2;
  asm("v_mul_f32 %0, %8, %14\n"
      "v_fmac_f32 %0, %7, %13\n"
      "v_fmac_f32 %0, %9, %15\n"
      MOV "%4, %7" HI1 MOV "%5, %8" HI1 MOV "%6, %9" HI1
      MUL "%1, %11, %8" Q0 MUL "%3, %8, %11" Q2 MUL "%2, %11, %5" LO1
      FMAC "%1, %10, %7" Q0 FMAC "%3, %7, %10" Q2 FMAC "%2, %10, %4" LO1
      FMAC "%1, %12, %9" Q0 FMAC "%3, %9, %12" Q2 FMAC "%2, %12, %6" LO1
      : "=&v"(cw), "=&v"(iw[0]), "=&v"(iw[1]), "=&v"(iw[2]), "=&v"(h0), "=&v"(h1), "=&v"(h2)
      : "v"(R[0]), "v"(R[1]), "v"(R[2]), "v"(RI[0]), "v"(RI[1]), "v"(RI[2]), "v"(K.com[0]), "v"(K.com[1]),
        "v"(K.com[2]));
  const Rep3 w = rep3(cw);
  const float c2 = w.x0 * w.x0 + w.x1 * w.x1 + w.x2 * w.x2;
  const float wj[3] = {w.x0, w.x1, w.x2};
#pragma unroll
  for (int j = 0; j < 3; ++j) I.A[j] = iw[j] + m * ((k == j ? c2 : 0.f) - cw * wj[j]);
  const float mc = m * cw;
  I.B[0] = sgn[0] * skew_part<0>(mc);
  I.B[1] = sgn[1] * skew_part<1>(mc);
  I.B[2] = sgn[2] * skew_part<2>(mc);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    I.T[j] = -I.B[j];
    I.C[j] = k == j ? m : 0.f;
  }
}

// bias_force of a body's rigid inertia (its C block is m times the identity)
__device__ __forceinline__ void path_bias(float va, float vl, float m, PathInertia& I) {
  // h = I v, then (va x ha + vl x hl, va x hl)
  float ha, hl, a1, a2, l1, l2;
  asm("s_nop 1\n"
      MUL "%2, %8, %11" Q0 MUL "%3, %8, %17" Q0
      FMAC "%2, %8, %12" Q1 FMAC "%3, %8, %18" Q1
      FMAC "%2, %8, %13" Q2 FMAC "%3, %8, %19" Q2
      FMAC "%2, %9, %14" Q0
      "v_fmac_f32 %3, %10, %9\n"
      FMAC "%2, %9, %15" Q1
      FMAC "%2, %9, %16" Q2
      MOV "%4, %8" ROT1 MOV "%5, %8" ROT2 MOV "%6, %9" ROT1 MOV "%7, %9" ROT2
      MUL "%0, -%2, %5" ROT1 FMAC "%0, %2, %4" ROT2
      MUL "%2, -%3, %7" ROT1 FMAC "%2, %3, %6" ROT2
      MUL "%1, -%3, %5" ROT1 FMAC "%1, %3, %4" ROT2
      "v_add_f32 %0, %0, %2\n"
      : "=&v"(I.pa), "=&v"(I.pl), "=&v"(ha), "=&v"(hl), "=&v"(a1), "=&v"(a2), "=&v"(l1), "=&v"(l2)
      : "v"(va), "v"(vl), "v"(m), "v"(I.A[0]), "v"(I.A[1]), "v"(I.A[2]), "v"(I.B[0]), "v"(I.B[1]), "v"(I.B[2]),
        "v"(I.T[0]), "v"(I.T[1]), "v"(I.T[2]));
}

// World pose of the base as the contact points read it: all of Rb, its column k,
// the base height, and component k of gravity in base axes.
struct PathBase {
  float Rb[9], c0, c1, c2, pz, agl;
};

// contact_point, one row per lane (fn, vw and fw come out on every lane)
__device__ __forceinline__ float path_contact(const float* r, const PathFrame& F, const PathBase& B, float dt,
                                              const ContactLaw& law, int k, const float* sgn, PathInertia& I, float* vw,
                                              float* fw) {
  const float* Rb = B.Rb;
  // the point x (about the body's origin), its height pw2 and world velocity vw
  float x, x1, x2_, pw2, vB, xB;
  asm("v_mul_f32 %0, %10, %13\n"
      "v_fmac_f32 %0, %9, %12\n"
      "v_fmac_f32 %0, %11, %14\n"
      "v_mov_b32 %3, %18\n"
      "v_add_f32 %8, %17, %0\n"
      MOV "%1, %0" ROT1 MOV "%2, %0" ROT2
      MUL "%7, -%15, %1" ROT2 FMAC "%7, %15, %2" ROT1
      "v_add_f32 %7, %16, %7\n"
      FMAC "%3, %8, %25" Q0 FMAC "%3, %8, %26" Q1 FMAC "%3, %8, %27" Q2
      MUL "%4, %7, %20" Q1 MUL "%5, %7, %23" Q1 MUL "%6, %7, %26" Q1
      FMAC "%4, %7, %19" Q0 FMAC "%5, %7, %22" Q0 FMAC "%6, %7, %25" Q0
      FMAC "%4, %7, %21" Q2 FMAC "%5, %7, %24" Q2 FMAC "%6, %7, %27" Q2
      : "=&v"(x), "=&v"(x1), "=&v"(x2_), "=&v"(pw2), "=&v"(vw[0]), "=&v"(vw[1]), "=&v"(vw[2]), "=&v"(vB), "=&v"(xB)
      : "v"(F.R[0]), "v"(F.R[1]), "v"(F.R[2]), "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(F.va), "v"(F.vl), "v"(F.p), "v"(B.pz),
        "v"(Rb[0]), "v"(Rb[1]), "v"(Rb[2]), "v"(Rb[3]), "v"(Rb[4]), "v"(Rb[5]), "v"(Rb[6]), "v"(Rb[7]), "v"(Rb[8]));
  float fn = 0.f;
  if (pw2 < 0.f) fn = fmaxf(0.f, -law.k * pw2 - law.d * vw[2]);
  const float n2 = vw[0] * vw[0] + vw[1] * vw[1] + law.eps * law.eps;
  const float inv_nrm = rsq(n2);
  const float mfn = law.mu * fn * inv_nrm;
  fw[0] = -mfn * vw[0]; fw[1] = -mfn * vw[1]; fw[2] = fn;
  if (fn > 0.f) {  // (without force the terms below are all zero)
    const float aa = mfn;
    const float al = law.d - aa;
    const float zb = B.c2;
    const float wt[2] = {vw[0] * inv_nrm, vw[1] * inv_nrm};
    // fB = Rb^T fw, ub = Rb^T wt, w1 = x x zb, w2 = x x ub; the force on the body
    float fB, ub, w1, w2, xf;
    asm("v_mul_f32 %0, %10, %13\n"
        "v_mul_f32 %1, %10, %16\n"
        "v_fmac_f32 %1, %9, %15\n"
        "v_fmac_f32 %0, %9, %12\n"
        "v_fmac_f32 %0, %11, %14\n"
        MUL "%2, -%11, %8" ROT1 FMAC "%2, %11, %7" ROT2
        MUL "%3, -%1, %8" ROT1 FMAC "%3, %1, %7" ROT2
        MUL "%4, -%0, %8" ROT1 FMAC "%4, %0, %7" ROT2
        "v_sub_f32 %6, %6, %0\n"
        "v_sub_f32 %5, %5, %4\n"
        : "=&v"(fB), "=&v"(ub), "=&v"(w1), "=&v"(w2), "=&v"(xf), "+v"(I.pa), "+v"(I.pl)
        : "v"(x1), "v"(x2_), "v"(B.c0), "v"(B.c1), "v"(zb), "v"(fw[0]), "v"(fw[1]), "v"(fw[2]), "v"(wt[0]), "v"(wt[1]));
    const Rep3 xr = rep3(x);
    const float x2 = xr.x0 * xr.x0 + xr.x1 * xr.x1 + xr.x2 * xr.x2;
    const float dta = dt * aa, dtal = dt * al;
    // y1 = (w1, zb), y2 = (w2, ub); t1 = dtal y1, t2 = dta y2
    const float t1a = dtal * w1, t1l = dtal * zb, t2a = dta * w2, t2l = dta * ub;
    const float dax = dta * x;
    const float dx2 = dta * x2;
    float s0 = k == 0 ? dx2 : 0.f, s1 = k == 1 ? dx2 : 0.f, s2 = k == 2 ? dx2 : 0.f;
    const float dk0 = k == 0 ? dta : 0.f, dk1 = k == 1 ? dta : 0.f, dk2 = k == 2 ? dta : 0.f;
    float a, b, h1, h2;
    // A_rc += t1_r y1_c - t2_r y2_c (r <= c), then += (r == c ? dx2 : 0) - dax_r x_c; C alike with dta on the diagonal
    asm("s_nop 1\n"
        MUL "%9, -%14, %18" Q0 MUL "%10, -%18, %14" Q2
        FMAC "%9, %13, %17" Q0 FMAC "%10, %17, %13" Q2
        MOV "%11, %17" HI1 MOV "%12, %18" HI1
        "v_add_f32 %0, %0, %9\n"
        "v_add_f32 %2, %2, %10\n"
        MUL "%9, -%14, %12" LO1 FMAC "%9, %13, %11" LO1
        MOV "%11, %22" HI1
        FMAC "%6, -%21, %22" Q0 FMAC "%8, -%22, %21" Q2 FMAC "%7, -%21, %11" LO1
        "v_add_f32 %1, %1, %9\n"
        "v_add_f32 %0, %0, %6\n"
        "v_add_f32 %2, %2, %8\n"
        "v_add_f32 %1, %1, %7\n"
        MUL "%9, -%16, %20" Q0 MUL "%10, -%20, %16" Q2
        FMAC "%9, %15, %19" Q0 FMAC "%10, %19, %15" Q2
        MOV "%11, %19" HI1 MOV "%12, %20" HI1
        "v_add_f32 %3, %3, %9\n"
        "v_add_f32 %5, %5, %10\n"
        MUL "%9, -%16, %12" LO1 FMAC "%9, %15, %11" LO1
        "v_add_f32 %3, %3, %23\n"
        "v_add_f32 %5, %5, %25\n"
        "v_add_f32 %4, %4, %9\n"
        "v_add_f32 %4, %4, %24\n"
        : "+v"(I.A[0]), "+v"(I.A[1]), "+v"(I.A[2]), "+v"(I.C[0]), "+v"(I.C[1]), "+v"(I.C[2]), "+v"(s0), "+v"(s1),
          "+v"(s2), "=&v"(a), "=&v"(b), "=&v"(h1), "=&v"(h2)
        : "v"(t1a), "v"(t2a), "v"(t1l), "v"(t2l), "v"(w1), "v"(w2), "v"(zb), "v"(ub), "v"(dax), "v"(x), "v"(dk0),
          "v"(dk1), "v"(dk2));
    // B_j += t1a zb_j - t2a ub_j, T_j += t1a_j zb - t2a_j ub, then the skew part of dax
    asm("s_nop 1\n"
        MUL "%6, -%11, %9" Q0 MUL "%7, -%11, %9" Q1
        "v_fmac_f32 %6, %16, %8\n"
        "v_fmac_f32 %7, %17, %8\n"
        "v_add_f32 %0, %0, %6\n"
        "v_add_f32 %1, %1, %7\n"
        MUL "%6, -%11, %9" Q2 MUL "%7, -%9, %11" Q0
        "v_fmac_f32 %6, %18, %8\n"
        FMAC "%7, %8, %10" Q0
        "v_add_f32 %2, %2, %6\n"
        "v_add_f32 %3, %3, %7\n"
        MUL "%6, -%9, %11" Q1 MUL "%7, -%9, %11" Q2
        FMAC "%6, %8, %10" Q1 FMAC "%7, %8, %10" Q2
        "v_add_f32 %4, %4, %6\n"
        "v_add_f32 %5, %5, %7\n"
        MUL "%6, %12, %13 quad_perm:[0,2,1,1]\n"
        MUL "%7, %12, %14 quad_perm:[2,1,0,0]\n"
        "v_add_f32 %0, %0, %6\n"
        "v_sub_f32 %3, %3, %6\n"
        MUL "%6, %12, %15 quad_perm:[1,0,2,2]\n"
        "v_add_f32 %1, %1, %7\n"
        "v_sub_f32 %4, %4, %7\n"
        "v_add_f32 %2, %2, %6\n"
        "v_sub_f32 %5, %5, %6\n"
        : "+v"(I.B[0]), "+v"(I.B[1]), "+v"(I.B[2]), "+v"(I.T[0]), "+v"(I.T[1]), "+v"(I.T[2]), "=&v"(a), "=&v"(b)
        : "v"(t1a), "v"(t2a), "v"(zb), "v"(ub), "v"(dax), "v"(sgn[0]), "v"(sgn[1]), "v"(sgn[2]), "v"(Rb[6]), "v"(Rb[7]),
          "v"(Rb[8]));
    // w3 = (agl - beta) + (-beta_a) x x, zw = zb . w3, uw = ub . w3
    const float sl = B.agl - F.bl;
    float w3, zw, uw, g0, g1, g2;
    asm("s_nop 1\n"
        MUL "%0, %6, %8" ROT2 FMAC "%0, -%6, %9" ROT1
        "v_add_f32 %0, %7, %0\n"
        "s_nop 1\n"
        MOV "%3, %0" Q0 MOV "%4, %0" Q1 MOV "%5, %0" Q2
        "v_mul_f32 %1, %12, %4\n"
        MUL "%2, %10, %4" Q1
        "v_fmac_f32 %1, %11, %3\n"
        FMAC "%2, %10, %3" Q0
        "v_fmac_f32 %1, %13, %5\n"
        FMAC "%2, %10, %5" Q2
        : "=&v"(w3), "=&v"(zw), "=&v"(uw), "=&v"(g0), "=&v"(g1), "=&v"(g2)
        : "v"(F.ba), "v"(sl), "v"(x1), "v"(x2_), "v"(ub), "v"(Rb[6]), "v"(Rb[7]), "v"(Rb[8]));
    const float Dw3 = aa * w3 + al * zw * zb - aa * uw * ub;
    const float xd = cross_k(x1, x2_, rot1(Dw3), rot2(Dw3));
    I.pa += dt * xd;
    I.pl += dt * Dw3;
  }
  return fn;
}

// What the forward sweep needs of a body's articulated step.
struct PathJoint {
  float Ua, Ul, invD, u;
};

// backward_joint: from the articulated inertia I of body F to its joint terms and
// the inertia O carried to the parent's origin.
template <bool FB>
__device__ __forceinline__ void path_backward(const PathInertia& I, const PathFrame& F, int k, float tau, float arm,
                                              float gain, PathJoint& J, PathInertia& O) {
  const Rep3 ax = rep3(F.ax);
  // U = IA S; d = ax . Ua, s = ax . pa
  float d, s;
  asm("v_mul_f32 %0, %5, %11\n"
      "v_mul_f32 %1, %8, %11\n"
      "v_fmac_f32 %0, %4, %10\n"
      "v_fmac_f32 %1, %7, %10\n"
      "v_fmac_f32 %0, %6, %12\n"
      "v_fmac_f32 %1, %9, %12\n"
      MUL "%3, %13, %11" Q1 FMAC "%3, %13, %10" Q0 FMAC "%3, %13, %12" Q2
      MUL "%2, %0, %11" Q1 FMAC "%2, %0, %10" Q0 FMAC "%2, %0, %12" Q2
      : "=&v"(J.Ua), "=&v"(J.Ul), "=&v"(d), "=&v"(s)
      : "v"(I.A[0]), "v"(I.A[1]), "v"(I.A[2]), "v"(I.T[0]), "v"(I.T[1]), "v"(I.T[2]), "v"(ax.x0), "v"(ax.x1), "v"(ax.x2),
        "v"(I.pa));
  const float Dv = (arm + gain) + d;
  J.invD = rcp(Dv);
  // Beside a floating base the difference stays behind the reciprocal, whose wait it
  // fills (quadruped, 256 x 200 steps: 625 us, 631 with the compiler's s_nop there); a
  // fixed base is faster as the compiler orders it (branching arm 825 us, 837).
  // Memory and scalar instructions may cross.
  if constexpr (FB) __builtin_amdgcn_sched_barrier(0x94);
  J.u = tau - s;
  const float Wl = J.Ul * J.invD;
  // uD = u / D and Wa = Ua / D (plain reads, before those through DPP), then
  // Ia = IA - U W^T (entry (r, c) with r <= c takes U_r W_c), then y = Ia c
  PathInertia X = I;
  float ya, yl, t0, t1, uD, Wa;
  asm("v_mul_f32 %16, %23, %24\n"
      "v_mul_f32 %17, %18, %24\n"
      FMAC "%6, -%18, %20" Q0 FMAC "%7, -%18, %20" Q1 FMAC "%8, -%18, %20" Q2   // T_j -= Ua_j Wl
      FMAC "%0, -%18, %17" Q0                                                   // A_0 -= Ua_0 Wa
      FMAC "%3, -%20, %18" Q0 FMAC "%4, -%20, %18" Q1 FMAC "%5, -%20, %18" Q2   // B_j -= Ua Wl_j
      MOV "%14, %17" HI1 MOV "%15, %20" HI1
      FMAC "%2, -%17, %18" Q2                                                   // A_2 -= Ua Wa_2
      FMAC "%1, -%18, %14" LO1
      FMAC "%9, -%19, %20" Q0 FMAC "%11, -%20, %19" Q2 FMAC "%10, -%19, %15" LO1  // C
      MUL "%12, %21, %0" Q0 MUL "%13, %21, %6" Q0
      FMAC "%12, %21, %1" Q1 FMAC "%13, %21, %7" Q1
      FMAC "%12, %21, %2" Q2 FMAC "%13, %21, %8" Q2
      FMAC "%12, %22, %3" Q0 FMAC "%13, %22, %9" Q0
      FMAC "%12, %22, %4" Q1 FMAC "%13, %22, %10" Q1
      FMAC "%12, %22, %5" Q2 FMAC "%13, %22, %11" Q2
      : "+v"(X.A[0]), "+v"(X.A[1]), "+v"(X.A[2]), "+v"(X.B[0]), "+v"(X.B[1]), "+v"(X.B[2]), "+v"(X.T[0]), "+v"(X.T[1]),
        "+v"(X.T[2]), "+v"(X.C[0]), "+v"(X.C[1]), "+v"(X.C[2]), "=&v"(ya), "=&v"(yl), "=&v"(t0), "=&v"(t1), "=&v"(uD),
        "=&v"(Wa)
      : "v"(J.Ua), "v"(J.Ul), "v"(Wl), "v"(F.ca), "v"(F.cl), "v"(J.u), "v"(J.invD));
  // pa = pA + Ia c + U u / D
  const float pa = I.pa + ya + J.Ua * uD;
  const float pl = I.pl + yl + J.Ul * uD;
  // carried to the parent's origin: C' = C, B' = B + E C, A' = A - B'E - (B E)^T
  const float e1 = rot1(F.e), e2 = rot2(F.e);
  float f0, f1, f2, t;
  asm("s_nop 1\n"
      MUL "%0, -%20, %25" ROT1 MUL "%1, -%21, %25" ROT1 MUL "%2, -%22, %25" ROT1   // B'_j = B_j + (e x C_j)
      FMAC "%0, %20, %24" ROT2 FMAC "%1, %21, %24" ROT2 FMAC "%2, %22, %24" ROT2
      MUL "%3, -%23, %21" Q2 MUL "%4, -%23, %22" Q0 MUL "%5, -%23, %20" Q1         // T'_j = T_j + (e x C row)_j
      FMAC "%3, %23, %22" Q1 FMAC "%4, %23, %20" Q2 FMAC "%5, %23, %21" Q0
      "v_add_f32 %0, %14, %0\n"
      "v_add_f32 %1, %15, %1\n"
      "v_add_f32 %2, %16, %2\n"
      "v_add_f32 %3, %17, %3\n"
      "v_add_f32 %4, %18, %4\n"
      "v_add_f32 %5, %19, %5\n"
      MUL "%9, -%27, %25" ROT1 FMAC "%9, %27, %24" ROT2                            // pa' = pa + e x pl
      MUL "%6, -%3, %24" ROT2 MUL "%7, -%4, %24" ROT2 MUL "%8, -%5, %24" ROT2      // y_j = (row j of B') x e
      FMAC "%6, %3, %25" ROT1 FMAC "%7, %4, %25" ROT1 FMAC "%8, %5, %25" ROT1
      "v_add_f32 %9, %26, %9\n"
      "v_sub_f32 %6, %11, %6\n"
      "v_sub_f32 %7, %12, %7\n"
      "v_sub_f32 %8, %13, %8\n"
      MUL "%10, -%23, %16" Q1 FMAC "%10, %23, %15" Q2                              // z_j = (row k of B) x e
      "v_sub_f32 %6, %6, %10\n"
      MUL "%10, -%23, %14" Q2 FMAC "%10, %23, %16" Q0
      "v_sub_f32 %7, %7, %10\n"
      MUL "%10, -%23, %15" Q0 FMAC "%10, %23, %14" Q1
      "v_sub_f32 %8, %8, %10\n"
      : "=&v"(O.B[0]), "=&v"(O.B[1]), "=&v"(O.B[2]), "=&v"(O.T[0]), "=&v"(O.T[1]), "=&v"(O.T[2]), "=&v"(f0), "=&v"(f1),
        "=&v"(f2), "=&v"(O.pa), "=&v"(t)
      : "v"(X.A[0]), "v"(X.A[1]), "v"(X.A[2]), "v"(X.B[0]), "v"(X.B[1]), "v"(X.B[2]), "v"(X.T[0]), "v"(X.T[1]),
        "v"(X.T[2]), "v"(X.C[0]), "v"(X.C[1]), "v"(X.C[2]), "v"(F.e), "v"(e1), "v"(e2), "v"(pa), "v"(pl));
#pragma unroll
  for (int j = 0; j < 3; ++j) O.C[j] = X.C[j];
  // f_j is entry (j, k) of A' for j <= k; the rest comes from the other triangle
  const float g01 = quad_of<1>(f0), g02 = quad2(f0), g12 = quad2(f1);  // (on all lanes, outside the selections)
  O.A[0] = f0;
  O.A[1] = k == 0 ? g01 : f1;
  O.A[2] = own3(k, g02, g12, f2);
  O.pl = pl;
}

// forward_joint: the parent's a' (ala, all) to the body's own; returns the joint acceleration
__device__ __forceinline__ float path_forward(float ala, float all, const PathFrame& F, const PathJoint& J, float& aa,
                                              float& al) {
  // a = shift(a') + c, s = U . a
  float xa, xl, s, t0, t1;
  asm("v_add_f32 %0, %5, %8\n"
      "s_nop 0\n"
      MOV "%3, %7" ROT1 MOV "%4, %7" ROT2
      MUL "%1, -%5, %3" ROT2 FMAC "%1, %5, %4" ROT1
      "v_add_f32 %1, %6, %1\n"
      MOV "%3, %0" Q0 MOV "%4, %0" Q1
      "v_add_f32 %1, %1, %9\n"
      MUL "%2, %10, %3" Q0
      MOV "%3, %0" Q2
      FMAC "%2, %10, %4" Q1
      MOV "%4, %1" Q0
      FMAC "%2, %10, %3" Q2
      MOV "%3, %1" Q1
      FMAC "%2, %11, %4" Q0
      MOV "%4, %1" Q2
      FMAC "%2, %11, %3" Q1
      FMAC "%2, %11, %4" Q2
      : "=&v"(xa), "=&v"(xl), "=&v"(s), "=&v"(t0), "=&v"(t1)
      : "v"(ala), "v"(all), "v"(F.e), "v"(F.ca), "v"(F.cl), "v"(J.Ua), "v"(J.Ul));
  const float qdd = (J.u - s) * J.invD;
  aa = xa + F.ax * qdd;
  al = xl;
  return qdd;
}

// base_solve over the rows of a row of 16 lanes, whose first quad holds the sums:
// lanes 0..2 take rows 0..2 of the 6x6 inertia, lanes 4..6 rows 3..5 (the first
// quad's columns of B and rows of C), and a column of the factor is one value
// per lane; a0 comes out on every lane.
#define BC0 " row_newbcast:0\n"
#define BC1 " row_newbcast:1\n"
#define BC2 " row_newbcast:2\n"
#define BC3 " row_newbcast:4\n"
#define BC4 " row_newbcast:5\n"
#define BC5 " row_newbcast:6\n"
__device__ __forceinline__ float second_quad(float first, float second) {
  // lanes 4..7 take the second value of the first quad, the others keep the first
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first),
                                                               __builtin_bit_cast(int, second), 0x114, 0xf, 0x2, false));
}
__device__ __forceinline__ void path_base_solve(const PathInertia& I, float* a) {
  float m[6], v[6], y[6];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    m[j] = second_quad(I.A[j], I.T[j]);
    m[3 + j] = second_quad(I.B[j], I.C[j]);
  }
  float s = -second_quad(I.pa, I.pl);
  // Factor: v_j = 1 / sqrt(m_j's diagonal) on its own lane, column m_j times it,
  // then subtracted from the later columns (each takes them in order); forward
  // substitution beside it: y_j = s v_j on its own lane, s -= y_j m_j.  Back
  // substitution on every lane: a_i = (y_i - sum over k > i of m_i's row k times a_k) v_i.
  // The independent instructions stand where a value just written has to wait
  // before it is read through DPP.
#define RSQ "v_rsq_f32 "
#define VMUL "v_mul_f32 "
  asm("s_nop 1\n"
      RSQ "%7, %0\ns_nop 1\n" MUL "%0, %7, %0" BC0
      VMUL "%13, %6, %7\ns_nop 0\n"
      FMAC "%1, -%0, %0" BC1
      RSQ "%8, %1\n" FMAC "%2, -%0, %0" BC2 FMAC "%3, -%0, %0" BC3 MUL "%1, %8, %1" BC1
      FMAC "%4, -%0, %0" BC4 FMAC "%5, -%0, %0" BC5
      FMAC "%2, -%1, %1" BC2
      RSQ "%9, %2\n" FMAC "%3, -%1, %1" BC3 FMAC "%4, -%1, %1" BC4 MUL "%2, %9, %2" BC2
      FMAC "%5, -%1, %1" BC5 FMAC "%6, -%13, %0" BC0
      FMAC "%3, -%2, %2" BC3
      RSQ "%10, %3\n" FMAC "%4, -%2, %2" BC4 FMAC "%5, -%2, %2" BC5 MUL "%3, %10, %3" BC3
      VMUL "%14, %6, %8\ns_nop 0\n"
      FMAC "%4, -%3, %3" BC4
      RSQ "%11, %4\n" FMAC "%5, -%3, %3" BC5 FMAC "%6, -%14, %1" BC1 MUL "%4, %11, %4" BC4
      VMUL "%15, %6, %9\ns_nop 0\n"
      FMAC "%5, -%4, %4" BC5
      RSQ "%12, %5\n" FMAC "%6, -%15, %2" BC2
      VMUL "%16, %6, %10\ns_nop 1\n" FMAC "%6, -%16, %3" BC3
      VMUL "%17, %6, %11\ns_nop 1\n" FMAC "%6, -%17, %4" BC4
      VMUL "%18, %6, %12\n"
      MOV "%23, %17" BC4 MOV "%22, %16" BC3 MOV "%21, %15" BC2 MOV "%20, %14" BC1 MOV "%19, %13" BC0
      MOV "%24, %18" BC5
      MUL "%24, %12, %24" BC5
      FMAC "%23, -%4, %24" BC5 MUL "%23, %11, %23" BC4
      FMAC "%22, -%3, %23" BC4 FMAC "%22, -%3, %24" BC5 MUL "%22, %10, %22" BC3
      FMAC "%21, -%2, %22" BC3 FMAC "%21, -%2, %23" BC4 FMAC "%21, -%2, %24" BC5 MUL "%21, %9, %21" BC2
      FMAC "%20, -%1, %21" BC2 FMAC "%20, -%1, %22" BC3 FMAC "%20, -%1, %23" BC4 FMAC "%20, -%1, %24" BC5
      MUL "%20, %8, %20" BC1
      FMAC "%19, -%0, %20" BC1 FMAC "%19, -%0, %21" BC2 FMAC "%19, -%0, %22" BC3 FMAC "%19, -%0, %23" BC4
      FMAC "%19, -%0, %24" BC5 MUL "%19, %7, %19" BC0
      : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(s), "=&v"(v[0]), "=&v"(v[1]),
        "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]),
        "=&v"(y[4]), "=&v"(y[5]), "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]));
#undef RSQ
#undef VMUL
}
#undef BC0
#undef BC1
#undef BC2
#undef BC3
#undef BC4
#undef BC5

// A lane's record of the exchange area (children reached through LDS).
__device__ __forceinline__ void put_exchange(float* d, const PathInertia& x) {
  put4(d, x.A[0], x.A[1], x.A[2], x.pa);
  put4(d + 4, x.B[0], x.B[1], x.B[2], x.pl);
  put4(d + 8, x.T[0], x.T[1], x.T[2], x.C[0]);
  *reinterpret_cast<float2*>(d + 12) = make_float2(x.C[1], x.C[2]);
}
__device__ __forceinline__ PathInertia get_exchange(const float* s) {
  const float4 a = get4(s), b = get4(s + 4), c = get4(s + 8);
  const float2 d = *reinterpret_cast<const float2*>(s + 12);
  return PathInertia{{a.x, a.y, a.z}, {b.x, b.y, b.z}, {c.x, c.y, c.z}, {c.w, d.x, d.y}, a.w, b.w};
}

// value of lane l + N of this lane's row added to this lane's
template <int N>
__device__ __forceinline__ void add_row_lane(PathInertia& x, const PathInertia& y) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    x.A[j] += from_row_lane<N>(y.A[j]);
    x.B[j] += from_row_lane<N>(y.B[j]);
    x.T[j] += from_row_lane<N>(y.T[j]);
    x.C[j] += from_row_lane<N>(y.C[j]);
  }
  x.pa += from_row_lane<N>(y.pa);
  x.pl += from_row_lane<N>(y.pl);
}
// value of lane K of the first quad of this lane's group: the group's sums sit
// there (G = 8 and 16), or in every quad (G = 4 and 32)
template <int G, int K>
__device__ __forceinline__ float from_first_quad(float x) {
  if constexpr (G == 16) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150 + K, 0xf, 0xf, false));
  } else if constexpr (G == 8) {
    // odd quads take the quad before them (row_shr:4 on banks 1 and 3)
    const int xi = __builtin_bit_cast(int, x);
    const int s = __builtin_amdgcn_update_dpp(xi, xi, 0x114, 0xf, 0xa, false);
    return quad_of<K>(__builtin_bit_cast(float, s));
  } else {
    return quad_of<K>(x);
  }
}

// One work item: 64 / G rollouts of one instance, samples first .. first + 64/G - 1
// (those >= N are computed but not stored).  L: the longest path the kernel
// holds; FB: floating base.  Paths that share a body, or more than four of them
// on a base, meet through LDS.  A body's constants stay in registers where the
// 256 the vector instructions address hold them (a fixed-base arm of three
// bodies); beside a floating base's state the inertias are read from LDS at each
// use (in registers they would be fetched back from the accumulation file: 59
// moves, 1.4 % of the quadruped's step), and so are all constants of longer paths.
template <int G, int L, bool FB>
__device__ __attribute__((always_inline)) void path_item(const DevInst& I, int first, float* smem, int steps,
                                                         float* state_out, const float* x0_in,
                                                         const float* nominal_in) {
  constexpr int S = (L + 2) / 3;      // joints a lane looks after (joint 3 s + k of its path)
  constexpr bool kRegs = L <= 3;           // (see above)
  constexpr bool kMassRegs = kRegs && !FB;
  constexpr bool kBranch = L > 3;     // paths may share bodies
  const float* x0 = x0_in ? x0_in : I.x0;
  switch (I.wave_prio) {
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 3: __builtin_amdgcn_s_setprio(3); break;
    default: break;
  }
  const int lane = threadIdx.x;
  const int grp = lane / G, l = lane % G;
  const int path = l >> 2, k4 = l & 3, k = k4 < 3 ? k4 : 2;
  const DevModel& M = *I.model;
  const int nb = M.nb, nc = M.nc, np = M.n_paths;
  float* tab = smem;
  stage_model_table(M, &I, tab, lane);
  float* rows = tab + body_table_floats(nc);
  for (int i = lane; i < np * L * 3 * (kPathRow / 4); i += 64) {
    const int rec = i / (kPathRow / 4), w = i % (kPathRow / 4);
    const int p = rec / (L * 3), ik = rec % (L * 3);
    reinterpret_cast<float4*>(rows)[i] = reinterpret_cast<const float4*>(&M.path_rows[p][ik / 3][ik % 3][0])[w];
  }
  float* exch = rows + np * L * 3 * kPathRow;  // [64 lanes + a record of zeros][kPathExch]
  if (lane < kPathExch) exch[64 * kPathExch + lane] = 0.f;
  const int n = first + grp;
  const bool valid = n < I.N;
  float* knots = smem + path_table_floats(nc, np, L) + grp * path_group_floats(I.E);
  if (I.generate) {
    sample_group<G>(M, I, valid ? n : 0, l, knots, valid, tab, nominal_in);
  } else {
    const float* src = I.samples + (size_t)(valid ? n : 0) * I.E;
    for (int e = l; e < I.E; e += G) knots[e] = src[e];
  }
  wave_sync();

  const StepConst sc = load_step_const(M, &I, 0.f);
  const int nq = FB ? 7 + M.nu : M.nu;
  const float sgn[3] = {own3(k, 0.f, 1.f, -1.f), own3(k, -1.f, 0.f, 1.f), own3(k, 1.f, -1.f, 0.f)};
  // a quad past the last path walks the last one again; it owns no body
  const int pp = path < np ? path : np - 1;
  const float* my_rows = rows + path_row(pp, L, 0, k);
  PathFk KF[kRegs ? L : 1];
  PathMass KM[kMassRegs ? L : 1];
  if constexpr (kRegs) {
#pragma unroll
    for (int i = 0; i < L; ++i) {
      KF[i] = load_path_fk(my_rows + i * 3 * kPathRow);
      if constexpr (kMassRegs) KM[i] = load_path_mass(my_rows + i * 3 * kPathRow);
    }
  }
  int ct_of[L];            // contacts of body i: first row | count << 8
  uint32_t src_of[L];      // children of body i on other paths too: their quads, 8 bits each
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int b = M.path_body[pp][i];
    ct_of[i] = (path < np && b >= 0) ? (M.c_begin[b] | (M.c_count[b] << 8)) : 0;
    if constexpr (kBranch) src_of[i] = M.path_src[pp][i];
  }
  // this lane's joints
  int body[S];
  bool is_joint[S], owner[S];
  float q[S], v[S], kp[S], kd[S], tm[S], q0[S], acc[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int i = 3 * s + k;
    body[s] = i < L ? M.path_body[pp][i < L ? i : 0] : -1;
    is_joint[s] = body[s] >= 0;
    owner[s] = is_joint[s] && path < np && k4 < 3 && M.path_owner[pp][i < L ? i : 0];
    const int j = is_joint[s] ? body[s] - (FB ? 1 : 0) : 0;
    q[s] = is_joint[s] ? x0[(FB ? 7 : 0) + j] : 0.f;
    v[s] = is_joint[s] ? x0[nq + (FB ? 6 : 0) + j] : 0.f;
    kp[s] = is_joint[s] ? M.kp[j] : 0.f;
    kd[s] = is_joint[s] ? M.kd[j] : 0.f;
    tm[s] = is_joint[s] ? M.taumax[j] : 0.f;
    q0[s] = (is_joint[s] && sc.cost_kind == 1) ? I.q0[j] : 0.f;
    acc[s] = 0.f;
  }
  float bq[7], bv[6], acc_base = 0.f;
#pragma unroll
  for (int i = 0; i < 7; ++i) bq[i] = FB ? x0[i] : 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) bv[i] = FB ? x0[nq + i] : 0.f;
  // the base's rigid inertia in its own axes does not change
  PathInertia base0;
  PathMass base_mass;
  PathFrame base_frame_k;
  if constexpr (FB) {
#pragma unroll
    for (int i = 0; i < 3; ++i) base_mass.com[i] = M.com[0][i];
#pragma unroll
    for (int i = 0; i < 6; ++i) base_mass.Ic[i] = M.Ic[0][i];
    base_mass.m = M.mass[0];
#pragma unroll
    for (int j = 0; j < 3; ++j) base_frame_k.R[j] = k == j ? 1.f : 0.f;
    path_inertia(base_frame_k.R, base_mass, k, sgn, base0);
    base_frame_k.p = base_frame_k.ba = base_frame_k.bl = 0.f;
  }
  uint32_t cmax = 0u;  // most contacts of a body at index i, 4 bits each
#pragma unroll
  for (int i = 0; i < L; ++i) cmax |= (uint32_t)M.path_cmax[i] << (4 * i);
  const int n_base_ct = FB ? M.c_count[0] : 0;
  const uint32_t branch = kBranch ? (uint32_t)M.path_branch : 0u;
  const uint32_t base_mask = (uint32_t)M.path_base_mask;
  const int ee_i = sc.cost_kind == 0 ? M.path_ee : -1;
  const int H = I.H, F = sc.F, F_run = steps * sc.nsub;
  const float dt = sc.dt;
  const bool to_end = !state_out && sc.cost_kind == 0;  // the terminal cost needs the kinematics at x_H
  StepClock clk;
  HermiteSeg hs[S];
#pragma unroll
  for (int s = 0; s < S; ++s) hs[s] = HermiteSeg{0.f, 0.f, 0.f, 0.f};
  int hseg = -1;
  for (int f = 0;; ++f) {
    const bool last = f >= F_run;
    if (last && !to_end) break;
    const bool control = clk.sub == 0;
    if (MPPI_RARE(true, clk.seg != hseg && !last)) {
      hseg = clk.seg;
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (is_joint[s]) hs[s] = hermite_segment(knots, sc.K, sc.nu, hseg, body[s] - (FB ? 1 : 0), sc.delta);
    }
    float tau[S], gain[S], cq[S], sq[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      float qref, vref;
      hermite_eval(hs[s], (float)clk.rem * sc.inv_F, sc.inv_delta, &qref, &vref);
      if (sc.spline_mode != 0) vref = 0.f;
      pd_law(kp[s], kd[s], tm[s], dt, q[s], v[s], qref, vref, tau[s], gain[s]);
      sincosf(q[s], &sq[s], &cq[s]);
    }
    PathBase B;
    PathFrame Pb;  // the parent of the paths' first bodies
    if constexpr (FB) {
      quat_R(bq + 3, B.Rb);
      B.c0 = own3(k, B.Rb[0], B.Rb[1], B.Rb[2]);
      B.c1 = own3(k, B.Rb[3], B.Rb[4], B.Rb[5]);
      B.c2 = own3(k, B.Rb[6], B.Rb[7], B.Rb[8]);
      B.pz = bq[2];
      Pb.va = own3(k, bv[0], bv[1], bv[2]);
      Pb.vl = own3(k, bv[3], bv[4], bv[5]);
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) B.Rb[i] = (i % 4 == 0) ? 1.f : 0.f;
      B.c0 = own3(k, 1.f, 0.f, 0.f);
      B.c1 = own3(k, 0.f, 1.f, 0.f);
      B.c2 = own3(k, 0.f, 0.f, 1.f);
      B.pz = 0.f;
      Pb.va = Pb.vl = 0.f;
    }
    B.agl = -sc.g * B.c2;

    // ---- kinematics, root to leaf
    PathFrame Fr[L];
    float arm[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int s = i / 3;
      const float ci = i % 3 == 0 ? quad_of<0>(cq[s]) : (i % 3 == 1 ? quad_of<1>(cq[s]) : quad_of<2>(cq[s]));
      const float si = i % 3 == 0 ? quad_of<0>(sq[s]) : (i % 3 == 1 ? quad_of<1>(sq[s]) : quad_of<2>(sq[s]));
      const float vi = i % 3 == 0 ? quad_of<0>(v[s]) : (i % 3 == 1 ? quad_of<1>(v[s]) : quad_of<2>(v[s]));
      const PathFk K = kRegs ? KF[kRegs ? i : 0] : load_path_fk(my_rows + i * 3 * kPathRow);
      arm[i] = K.arm;
      if (i == 0) {
        const float ptk = own3(k, K.pt[0], K.pt[1], K.pt[2]), axk = own3(k, K.ax[0], K.ax[1], K.ax[2]);
        path_fk<true>(K, ptk, axk, Pb, ci, si, vi, Fr[i]);
      } else {
        path_fk<false>(K, 0.f, 0.f, Fr[i - 1], ci, si, vi, Fr[i]);
      }
    }
    float dz = 0.f;  // end-effector height error
    if (ee_i >= 0) {
#pragma unroll
      for (int i = 0; i < L; ++i)
        if (i == ee_i) {
          const float xe = Fr[i].p + Fr[i].R[0] * sc.ee_pos[0] + Fr[i].R[1] * sc.ee_pos[1] + Fr[i].R[2] * sc.ee_pos[2];
          const Rep3 x = rep3(xe);
          dz = B.pz + B.Rb[6] * x.x0 + B.Rb[7] * x.x1 + B.Rb[8] * x.x2 - sc.z_des;
        }
    }
    if (last) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (body[s] == sc.ee_body) {
          const float t = sc.w_ee * dz * dz;
          acc[s] += t;
        }
      break;
    }

    // ---- articulated inertias, leaf to root
    PathJoint J[L];
    PathInertia Ip;
    float cost[S];
#pragma unroll
    for (int s = 0; s < S; ++s) cost[s] = 0.f;
#pragma unroll
    for (int i = L - 1; i >= 0; --i) {
      const int s = i / 3;
      const PathMass K = kMassRegs ? KM[kMassRegs ? i : 0] : load_path_mass(my_rows + i * 3 * kPathRow);
      PathInertia IA;
      path_inertia(Fr[i].R, K, k, sgn, IA);
      path_bias(Fr[i].va, Fr[i].vl, K.m, IA);
      const int most = (int)((cmax >> (4 * i)) & 15u);
      if (most > 0) {
        float ccost = 0.f;
        const int c0 = ct_of[i] & 255, cn = ct_of[i] >> 8;
#pragma unroll 1
        for (int c = 0; c < most; ++c) {
          if (c < cn) {
            const float* ct = tab + kTabContacts + (c0 + c) * kCt;
            float vw[3], fw[3];
            const float fn = path_contact(ct, Fr[i], B, dt, sc.law, k, sgn, IA, vw, fw);
            if (control && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], ccost);
          }
        }
        if (k == i % 3) cost[s] = ccost;
      }
      if (i < L - 1) {
        if (kBranch && ((branch >> i) & 1u)) {
          // some body here has children on several paths: they are added in child order
          put_exchange(exch + lane * kPathExch, Ip);
          wave_sync();
          const uint32_t src = src_of[i];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const uint32_t w = (src >> (8 * c)) & 255u;
            const int from = w == 255u ? 64 : grp * G + (int)w * 4 + k;
            add_inertia(IA, get_exchange(exch + from * kPathExch));
          }
          wave_sync();
        } else {
          add_inertia(IA, Ip);
        }
      }
      const float ti = i % 3 == 0 ? quad_of<0>(tau[s]) : (i % 3 == 1 ? quad_of<1>(tau[s]) : quad_of<2>(tau[s]));
      const float gi = i % 3 == 0 ? quad_of<0>(gain[s]) : (i % 3 == 1 ? quad_of<1>(gain[s]) : quad_of<2>(gain[s]));
      path_backward<FB>(IA, Fr[i], k, ti, arm[i], gi, J[i], Ip);
    }

    // ---- root: the base's articulated inertia and its solve, on every lane
    float ala, all, ba[6];
    float base_cost = 0.f;
    if constexpr (FB) {
      PathInertia IA = base0;
      base_frame_k.va = Pb.va;
      base_frame_k.vl = Pb.vl;
      path_bias(Pb.va, Pb.vl, base_mass.m, IA);
#pragma unroll 1
      for (int c = 0; c < n_base_ct; ++c) {
        const float* ct = tab + kTabContacts + (M.c_begin[0] + c) * kCt;
        float vw[3], fw[3];
        const float fn = path_contact(ct, base_frame_k, B, dt, sc.law, k, sgn, IA, vw, fw);
        if (control && sc.cost_kind == 1) contact_cost(sc, fn, vw, fw, ct[3], base_cost);
      }
      if constexpr (G == 32) {
        put_exchange(exch + lane * kPathExch, Ip);
        wave_sync();
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if ((base_mask >> c) & 1u) add_inertia(IA, get_exchange(exch + (grp * G + 4 * c + k) * kPathExch));
        wave_sync();
      } else {
        add_inertia(IA, Ip);  // (the first path always brings the first child)
        if (G > 4 && (base_mask & 2u)) add_row_lane<4>(IA, Ip);
        if (G > 8 && (base_mask & 4u)) add_row_lane<8>(IA, Ip);
        if (G > 8 && (base_mask & 8u)) add_row_lane<12>(IA, Ip);
      }
      float a0[6];
      if constexpr (G >= 16) {
        path_base_solve(IA, a0);
      } else {
        float X[21], px[6];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          X[SI(0, c)] = from_first_quad<G, 0>(IA.A[c]);
          if (c >= 1) X[SI(1, c)] = from_first_quad<G, 1>(IA.A[c]);
          if (c >= 2) X[SI(2, c)] = from_first_quad<G, 2>(IA.A[c]);
          X[SI(0, 3 + c)] = from_first_quad<G, 0>(IA.B[c]);
          X[SI(1, 3 + c)] = from_first_quad<G, 1>(IA.B[c]);
          X[SI(2, 3 + c)] = from_first_quad<G, 2>(IA.B[c]);
          X[SI(3, 3 + c)] = from_first_quad<G, 0>(IA.C[c]);
          if (c >= 1) X[SI(4, 3 + c)] = from_first_quad<G, 1>(IA.C[c]);
          if (c >= 2) X[SI(5, 3 + c)] = from_first_quad<G, 2>(IA.C[c]);
        }
        px[0] = from_first_quad<G, 0>(IA.pa); px[1] = from_first_quad<G, 1>(IA.pa); px[2] = from_first_quad<G, 2>(IA.pa);
        px[3] = from_first_quad<G, 0>(IA.pl); px[4] = from_first_quad<G, 1>(IA.pl); px[5] = from_first_quad<G, 2>(IA.pl);
        base_solve(X, px, a0);
      }
      const float g = sc.g;
      const float agl[3] = {-g * B.Rb[6], -g * B.Rb[7], -g * B.Rb[8]};
      ba[0] = a0[0]; ba[1] = a0[1]; ba[2] = a0[2];
      ba[3] = a0[3] + agl[0]; ba[4] = a0[4] + agl[1]; ba[5] = a0[5] + agl[2];
      ala = own3(k, a0[0], a0[1], a0[2]);
      all = own3(k, a0[3], a0[4], a0[5]);
    } else {
      ala = 0.f;
      all = k == 2 ? sc.g : 0.f;  // a' = -a_g
    }

    // ---- accelerations, root to leaf
    float qdd[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
      float aa, al;
      qdd[i] = path_forward(ala, all, Fr[i], J[i], aa, al);
      ala = aa;
      all = al;
    }

    // ---- running cost (Sec. IV-A; each body's terms in the body schedule's order)
    if (control) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        float c = cost[s];
        if (sc.cost_kind == 1) {
          const float eq = q[s] - q0[s];
          c += sc.w_q * eq * eq + sc.w_eff * tau[s] * tau[s];
        } else {
          c += sc.w_tau * tau[s] * tau[s];
          if (body[s] == sc.ee_body) c += sc.w_ee * dz * dz;
        }
        acc[s] += c;
      }
      if (FB && sc.cost_kind == 1) {
        const float bt = base_cost_term(sc, bq);
        base_cost += bt;
        acc_base += base_cost;
      }
    }

    // ---- integration
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float a = own3(k, qdd[3 * s], 3 * s + 1 < L ? qdd[3 * s + 1] : 0.f, 3 * s + 2 < L ? qdd[3 * s + 2] : 0.f);
      v[s] = fmaf(dt, a, v[s]);
      q[s] = fmaf(dt, v[s], q[s]);
    }
    if constexpr (FB) integrate_base_R<true>(bq, bv, ba, dt, B.Rb);
    clk.advance<true>(sc.K, F, sc.nsub);
  }
  if (state_out) {
    if (valid) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (owner[s]) {
          const int j = body[s] - (FB ? 1 : 0);
          state_out[(FB ? 7 : 0) + j] = q[s];
          state_out[nq + (FB ? 6 : 0) + j] = v[s];
        }
      if (FB && l == 0) {
#pragma unroll
        for (int i = 0; i < 7; ++i) state_out[i] = bq[i];
#pragma unroll
        for (int i = 0; i < 6; ++i) state_out[nq + i] = bv[i];
      }
    }
    return;
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
  for (int s = 0; s < S; ++s)
    if (owner[s]) knots[body[s]] = acc[s];
  if (FB && l == 0) knots[0] = acc_base;
  wave_sync();
  if (l == 0 && valid) {
    float sum = 0.f;
    for (int b = 0; b < nb; ++b) sum += knots[b];
    if (!isfinite(sum)) sum = INFINITY;
    I.costs[n] = sum;
  }
  wave_sync();
}

// The item function of an instance's tree (path_fits in mppi_api.hip offers the
// kernels only trees that one of these holds).
template <int L, bool FB>
__device__ __forceinline__ void path_item_of(const DevInst& I, int first, float* smem, int steps, float* state_out,
                                             const float* x0_in, const float* nominal_in) {
  const int lanes = I.model->path_lanes;
  if (lanes == 4) path_item<4, L, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
  else if (lanes == 8) path_item<8, L, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
  else if (lanes == 16) path_item<16, L, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
  else path_item<32, L, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
}
template <bool FB>
__device__ __forceinline__ void path_item_of(const DevInst& I, int first, float* smem, int steps, float* state_out,
                                             const float* x0_in, const float* nominal_in) {
  const int len = I.model->path_len;
  if (len <= 3) path_item_of<3, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
  else if (len <= 4) path_item_of<4, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
  else path_item_of<kMaxPath, FB>(I, first, smem, steps, state_out, x0_in, nominal_in);
}

#undef Q0
#undef Q1
#undef Q2
#undef ROT1
#undef ROT2
#undef LO1
#undef HI1
#undef MUL
#undef FMAC
#undef MOV

}  // namespace mppi
