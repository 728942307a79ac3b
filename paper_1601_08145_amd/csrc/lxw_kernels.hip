// HIP kernels (gfx950) of the positivity-preserving Lax-Wendroff DG step
// (Moe, Rossmanith, Seal, arXiv:1601.08145).
//
// One step is four or five launches on one stream (grid-wide dependencies separate them):
//   k_pre    per element: pending shock-capturing limiter of the previous step (Sec. 1.5 Step 5),
//            moment limiter (Sec. 3.1), cell-average checks, and the global wave speed s
//            (one atomic maximum per workgroup for a single mesh, or a partial one where there are many
//            workgroups; in a batch one atomic maximum per wavefront and mesh);
//   k_dt     a single mesh of many workgroups: reduces the workgroups' partials;
//   k_elem   per element: Galerkin projection of F (Sec. 2.3 Step 1), the time-averaged flux F_T
//            of Eq. (taylor3-flux) at every interior and edge point (Sec. 2.2, 2.3 Step 2), the
//            volume term (Sec. 2.3 Step 3) added to the higher modes, and the edge traces (each
//            side's half of Eq. (LLF), which is linear in the two sides' values);
//   k_flux   per element: on each of its edges the Lax-Friedrichs flux of F_T at the edge points
//            (Eq. (LLF)), the edge-averaged high-order flux f^LxW and the low-order flux f^LxF (Sec. 3.3
//            Step 3); the higher moments' edge terms (Step 6); the flux limiter of Steps 4-5 in float64
//            (Gamma, Lambda_ik, the corner states and the damping-factor solve mu_c), one candidate
//            per (element, edge); and the average's update with the high-order flux everywhere;
//   k_update per element: Lambda_e = min over the two sides; where one is below 1 the average's update
//            of Step 6 with the blended fluxes instead; the positivity check; the first element of each
//            mesh then ends the mesh's step (t += dt);
//   k_final  per mesh, after a state read-out applied the pending shock limiter: marks it done.
// Thread-per-element mapping; reference tables sit in __constant__ memory and are
// read through the scalar cache (every lane of a wave reads the same entry).  State is stored as
// cell averages Qbar[N][V] (float64, one record per element: also gathered by neighbour index) and
// higher modes as structure-of-arrays Qh[V][ML-1][N].
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lxw_internal.hpp"

namespace lxw {

// This file is compiled once per element configuration (LXW_PART, see build.py), side by side: each
// object holds that configuration's kernels in both precisions and its two reference tables.
#ifndef LXW_PART
#error "LXW_PART selects the element configuration: 0 line, 1 quad, 2 triangle, 3 P3 line, 4 P3 triangle, 5 tetrahedron"
#endif
#if LXW_PART == 0
using EL = ElLine;
#elif LXW_PART == 1
using EL = ElQuad;
#elif LXW_PART == 2
using EL = ElTri;
#elif LXW_PART == 3
using EL = ElLine3;
#elif LXW_PART == 4
using EL = ElTri3;
#else
using EL = ElTet;
#endif

static __constant__ RefTab<EL, double> c_tab_d;
static __constant__ RefTab<EL, float> c_tab_f;

template <class E, class R>
struct TabSel;
template <> struct TabSel<EL, double> { static __device__ __forceinline__ const RefTab<EL, double>& get() { return c_tab_d; } };
template <> struct TabSel<EL, float> { static __device__ __forceinline__ const RefTab<EL, float>& get() { return c_tab_f; } };

template <>
hipError_t upload_tables<EL>(const RefTab<EL, double>& d, const RefTab<EL, float>& f) {
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_tab_d), &d, sizeof(d));
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_tab_f), &f, sizeof(f));
  return e;
}

// Error codes (public values, see lxw.h).
enum { E_POSITIVITY = -5, E_NONFINITE = -6, E_CFL = -7 };

__device__ __forceinline__ void report(DevError* err, int code, int elem) {
  if (atomicCAS(&err->code, 0, code) == 0) err->elem = elem;
}

// ---------------------------------------------------------------------------------------------
// Physics.  q = (rho, M_1..M_DIM, E); F_d(q) = (M_d, M u_d + p e_d, u_d (E + p)) (Sec. 1.5) with
// p from Eq. (eos).  Jacobian and Hessian products (Eqs. (fluxderivs-a), (fluxderivs-b)) are
// written as first and second directional variations through the variations of u and p:
//   du_k = (a_Mk - u_k a_rho)/rho,  dp = (gamma-1)(a_E - u.a_M + |u|^2 a_rho / 2),
//   d2u_k = -(du_k[a] b_rho + du_k[b] a_rho)/rho,  d2p = -(gamma-1) rho du[a].du[b].
// ---------------------------------------------------------------------------------------------
template <int DIM, class R>
struct St {
  R rho, r, u[DIM], m[DIM], E, p, Ep, u2;
};

// 1/rho: in the float32 bulk the hardware reciprocal refined by one Newton-Raphson step,
// r + r (1 - x r) with the residual formed exactly by a fused multiply-add (the estimate is within
// 1 ulp; the refined value is within an ulp and almost always the correctly rounded quotient, in 3
// instructions instead of the division's 10; rho is positive and far above the denormal range
// wherever it is used), in float64 the correctly rounded quotient.
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return __fmaf_rn(r, __fmaf_rn(-x, r, 1.0f), r);
}
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

template <int DIM, class R>
__device__ __forceinline__ St<DIM, R> base_state(const R* q, R gm1) {
  St<DIM, R> s;
  s.rho = q[0];
  s.r = recip(q[0]);
  R mu = R(0), u2 = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    s.m[d] = q[1 + d];
    s.u[d] = s.m[d] * s.r;
    mu += s.m[d] * s.u[d];
    u2 += s.u[d] * s.u[d];
  }
  s.u2 = u2;
  s.E = q[DIM + 1];
  s.p = gm1 * (s.E - R(0.5) * mu);
  s.Ep = s.E + s.p;
  return s;
}

template <int DIM, class R>
struct Var {
  R du[DIM];
  R dp;
};

template <int DIM, class R>
__device__ __forceinline__ Var<DIM, R> var1(const St<DIM, R>& s, const R* a, R gm1) {
  Var<DIM, R> v;
  R t = a[DIM + 1] + R(0.5) * s.u2 * a[0];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    v.du[d] = (a[1 + d] - s.u[d] * a[0]) * s.r;
    t -= s.u[d] * a[1 + d];
  }
  v.dp = gm1 * t;
  return v;
}

template <int DIM, class R>
__device__ __forceinline__ void flux(const St<DIM, R>& s, int d, R* F) {
  F[0] = s.m[d];
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = s.m[k] * s.u[d] + (k == d ? s.p : R(0));
  F[DIM + 1] = s.u[d] * s.Ep;
}

// A_d a
template <int DIM, class R>
__device__ __forceinline__ void dflux(const St<DIM, R>& s, int d, const R* a, const Var<DIM, R>& va, R* F) {
  F[0] = a[1 + d];
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = a[1 + k] * s.u[d] + s.m[k] * va.du[d] + (k == d ? va.dp : R(0));
  F[DIM + 1] = va.du[d] * s.Ep + s.u[d] * (a[DIM + 1] + va.dp);
}

// H_d(a, b); d2p = -(gamma-1) rho du[a].du[b] is shared by all d and passed in.
template <int DIM, class R>
__device__ __forceinline__ void d2flux(const St<DIM, R>& s, int d, const R* a, const Var<DIM, R>& va, const R* b,
                                       const Var<DIM, R>& vb, R d2p, R* F) {
  R d2u = -(va.du[d] * b[0] + vb.du[d] * a[0]) * s.r;
  F[0] = R(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = a[1 + k] * vb.du[d] + b[1 + k] * va.du[d] + s.m[k] * d2u + (k == d ? d2p : R(0));
  F[DIM + 1] = d2u * s.Ep + va.du[d] * (b[DIM + 1] + vb.dp) + vb.du[d] * (a[DIM + 1] + va.dp) + s.u[d] * d2p;
}

template <int DIM, class R>
__device__ __forceinline__ R d2p_of(const St<DIM, R>& s, const Var<DIM, R>& va, const Var<DIM, R>& vb, R gm1) {
  R t = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) t += va.du[d] * vb.du[d];
  return -gm1 * s.rho * t;
}

// Degree 2: q_t, q_tt and F_T through the variations of u, p and H = E + p instead of one Jacobian and
// one Hessian product per term and direction.  With F_d = (M_d, M_k u_d + p e_d, u_d H) the product rule
// gives (subscripts t, d: derivatives in time and along x_d; q_t = -D, D = div F^h)
//   w = M_t - u rho_t = rho u_t,   u_d = (M_d - u rho_d)/rho,
//   p_x = (gamma-1)(E_x + |u|^2 rho_x / 2 - u.M_x)  for x = t and every d,
//   p_td = (gamma-1)(E_td + |u|^2 rho_td / 2 - u.M_td - u_d.w),
//   div u_t = (sum_d [M_d,td - u_d rho_td - u_d,t rho_d] - rho_t div u)/rho,
//   rho_tt = -div M_t,   M_k,tt = -(u.grad M_k,t + M_k,t div u + u_t.grad M_k + M_k div u_t) - p_tk,
//   E_tt = -(u.grad H_t + H_t div u + u_t.grad H + H div u_t),
// about 80 operations per point in 2D where the Jacobian and Hessian products took about 130.
// Time derivatives come scaled as F_T = F + c1 F_t + c2 F_tt needs them, q1 = c1 q_t and q2 = c2 q_tt with
// c1 = dt/2, c2 = dt^2/6 (and so w, u_t, p_t, H_t): with gradients of q scaled by c2/c1 = dt/3 and the
// gradient of D by c2 the formulas above hold as they stand, and a product's average is
//   a b + c1 (a b)_t + c2 (a b)_tt = a (b + b1 + b2) + a1 (b + 4/3 b1) + a2 b.
template <int DIM, class R>
struct Pt2 {
  R r, u[DIM], u2h, p, H;    // 1/rho, velocity, |u|^2/2, pressure, E + p
  R w[DIM], ut[DIM], pt, Ht;  // rho u_t, u_t, p_t, H_t
};
// from the state and q1
template <int DIM, class R>
__device__ __forceinline__ Pt2<DIM, R> pt2_of(const R* q, const R* qt, R gm1) {
  constexpr int V = DIM + 2;
  Pt2<DIM, R> s;
  s.r = recip(q[0]);
  R mu = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    s.u[d] = q[1 + d] * s.r;
    mu += q[1 + d] * s.u[d];
  }
  mu *= R(0.5);
  s.u2h = mu * s.r;
  s.p = gm1 * (q[V - 1] - mu);
  s.H = q[V - 1] + s.p;
  R t = qt[V - 1] + s.u2h * qt[0];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    t -= s.u[d] * qt[1 + d];
    s.w[d] = qt[1 + d] - s.u[d] * qt[0];
    s.ut[d] = s.w[d] * s.r;
  }
  s.pt = gm1 * t;
  s.Ht = qt[V - 1] + s.pt;
  return s;
}
// q2 from the scaled gradients of q and of D
template <int DIM, class R>
__device__ __forceinline__ void qtt_of(const Pt2<DIM, R>& s, const R* q, const R* qt, const R gq[DIM][DIM + 2],
                                       const R gD[DIM][DIM + 2], R gm1, R* qtt) {
  constexpr int V = DIM + 2;
  R divu = R(0), sum = R(0), rtt = R(0), ett = R(0), m[DIM], ptd[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) m[k] = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const R* g = gq[d];
    const R* h = gD[d];
    R pd = g[V - 1] + s.u2h * g[0], pt = h[V - 1] + s.u2h * h[0];
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      const R ud = (g[1 + k] - s.u[k] * g[0]) * s.r;
      pd -= s.u[k] * g[1 + k];
      pt -= s.u[k] * h[1 + k];
      pt += ud * s.w[k];  // h is the gradient of -q_t
      if (k == d) divu += ud;
    }
    pd *= gm1;
    ptd[d] = gm1 * pt;  // -p_td
    // sum: rho div u_t + rho_t div u
    sum -= h[1 + d] - s.u[d] * h[0] + s.ut[d] * g[0];
    rtt += h[1 + d];
#pragma unroll
    for (int k = 0; k < DIM; ++k) m[k] += s.u[d] * h[1 + k] - s.ut[d] * g[1 + k];
    ett += s.u[d] * (h[V - 1] + ptd[d]) - s.ut[d] * (g[V - 1] + pd);
  }
  const R divut = (sum - qt[0] * divu) * s.r;
  qtt[0] = rtt;
#pragma unroll
  for (int k = 0; k < DIM; ++k) qtt[1 + k] = m[k] - qt[1 + k] * divu - q[1 + k] * divut + ptd[k];
  qtt[V - 1] = ett - s.Ht * divu - s.H * divut;
}
// c2 p_tt
template <int DIM, class R>
__device__ __forceinline__ R ptt_of(const Pt2<DIM, R>& s, const R* q2, R gm1) {
  constexpr int V = DIM + 2;
  R t = q2[V - 1] + s.u2h * q2[0], ww = R(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    t -= s.u[d] * q2[1 + d];
    ww += s.w[d] * s.ut[d];
  }
  return gm1 * (t - R(2.0 / 3.0) * ww);
}
// F_T (Eq. (taylor3-flux)) in every direction (M_k u_d = M_d u_k: the momentum part is symmetric)
template <int DIM, class R>
__device__ __forceinline__ void ft2(const Pt2<DIM, R>& s, const R* q, const R* q1, const R* q2, R gm1,
                                    R FT[DIM][DIM + 2]) {
  constexpr int V = DIM + 2;
  const R ptt = ptt_of<DIM, R>(s, q2, gm1);
  const R pb = s.p + s.pt + ptt, Htt = q2[V - 1] + ptt;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const R v1 = R(4.0 / 3.0) * s.ut[d];
    const R utt = (q2[1 + d] - s.u[d] * q2[0] - v1 * q1[0]) * s.r;
    const R B = s.u[d] + s.ut[d] + utt, X = s.u[d] + v1, Y = s.u[d];
    FT[d][0] = q[1 + d] + q1[1 + d] + q2[1 + d];
#pragma unroll
    for (int k = d; k < DIM; ++k) {
      R f = q[1 + k] * B + q1[1 + k] * X + q2[1 + k] * Y;
      if (k == d) f += pb;
      FT[d][1 + k] = f;
      FT[k][1 + d] = f;
    }
    FT[d][V - 1] = s.H * B + s.Ht * X + Htt * Y;
  }
}
// along a normal n: n . F_T
template <int DIM, class R>
__device__ __forceinline__ void ftn2(const Pt2<DIM, R>& s, const R* q, const R* q1, const R* q2, const R* n, R gm1,
                                     R* FTn) {
  constexpr int V = DIM + 2;
  const R ptt = ptt_of<DIM, R>(s, q2, gm1);
  const R pb = s.p + s.pt + ptt, Htt = q2[V - 1] + ptt;
  R un = s.u[0] * n[0], utn = s.ut[0] * n[0], mttn = q2[1] * n[0], mn = (q[1] + q1[1] + q2[1]) * n[0];
#pragma unroll
  for (int d = 1; d < DIM; ++d) {
    un += s.u[d] * n[d];
    utn += s.ut[d] * n[d];
    mttn += q2[1 + d] * n[d];
    mn += (q[1 + d] + q1[1 + d] + q2[1 + d]) * n[d];
  }
  const R v1 = R(4.0 / 3.0) * utn;
  const R uttn = (mttn - un * q2[0] - v1 * q1[0]) * s.r;
  const R B = un + utn + uttn, X = un + v1;
  FTn[0] = mn;
#pragma unroll
  for (int k = 0; k < DIM; ++k) FTn[1 + k] = q[1 + k] * B + q1[1 + k] * X + q2[1 + k] * un + pb * n[k];
  FTn[V - 1] = s.H * B + s.Ht * X + Htt * un;
}
// the same from a state and its scaled time derivatives alone (ghost states of Sec. 2.4)
template <int DIM, class R>
__device__ __forceinline__ void ftn_from(const R* q, const R* q1, const R* q2, const R* n, R gm1, R* FTn) {
  ftn2<DIM, R>(pt2_of<DIM, R>(q, q1, gm1), q, q1, q2, n, gm1, FTn);
}

// Degree 3: the third variation F^(3)_d(a, b, c), through the third variations of u and p (the
// first and second are those above):
//   d3u_k[a,b,c] = -(d2u_k[a,b] c_rho + d2u_k[a,c] b_rho + d2u_k[b,c] a_rho)/rho,
//   d3p[a,b,c]   = (gamma-1)(a_rho du[b].du[c] + b_rho du[a].du[c] + c_rho du[a].du[b]);
// M_k u_d picks up a_Mk d2u_d[b,c] (and its two permutations) + M_k d3u_d, and u_d (E + p) the full
// product rule with first, second and third variations a_E + dp, d2p and d3p of E + p.
template <int DIM, class R>
__device__ __forceinline__ void d3flux(const St<DIM, R>& s, int d, const R* a, const Var<DIM, R>& va, const R* b,
                                       const Var<DIM, R>& vb, const R* c, const Var<DIM, R>& vc, R gm1, R* F) {
  constexpr int V = DIM + 2;
  R ab = R(0), ac = R(0), bc = R(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    ab += va.du[k] * vb.du[k];
    ac += va.du[k] * vc.du[k];
    bc += vb.du[k] * vc.du[k];
  }
  const R pab = -gm1 * s.rho * ab, pac = -gm1 * s.rho * ac, pbc = -gm1 * s.rho * bc;
  const R p3 = gm1 * (a[0] * bc + b[0] * ac + c[0] * ab);
  const R uab = -(va.du[d] * b[0] + vb.du[d] * a[0]) * s.r;
  const R uac = -(va.du[d] * c[0] + vc.du[d] * a[0]) * s.r;
  const R ubc = -(vb.du[d] * c[0] + vc.du[d] * b[0]) * s.r;
  const R u3 = -(uab * c[0] + uac * b[0] + ubc * a[0]) * s.r;
  F[0] = R(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = a[1 + k] * ubc + b[1 + k] * uac + c[1 + k] * uab + s.m[k] * u3 + (k == d ? p3 : R(0));
  F[V - 1] = u3 * s.Ep + uab * (c[V - 1] + vc.dp) + uac * (b[V - 1] + vb.dp) + ubc * (a[V - 1] + va.dp) +
             va.du[d] * pbc + vb.du[d] * pac + vc.du[d] * pab + s.u[d] * p3;
}

// F^(3)_d(a, a, a): the terms of d3flux with the three directions equal, gathered (the three
// pairwise products are one, and each permuted sum becomes three times one term).
template <int DIM, class R>
__device__ __forceinline__ void d3flux_sym(const St<DIM, R>& s, int d, const R* a, const Var<DIM, R>& va, R gm1, R* F) {
  constexpr int V = DIM + 2;
  R aa = R(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) aa += va.du[k] * va.du[k];
  const R paa = -gm1 * s.rho * aa;
  const R p3 = R(3) * gm1 * a[0] * aa;
  const R uaa = -R(2) * va.du[d] * a[0] * s.r;
  const R u3 = -R(3) * uaa * a[0] * s.r;
  F[0] = R(0);
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = R(3) * a[1 + k] * uaa + s.m[k] * u3 + (k == d ? p3 : R(0));
  F[V - 1] = u3 * s.Ep + R(3) * (uaa * (a[V - 1] + va.dp) + va.du[d] * paa) + s.u[d] * p3;
}

// Degree 3: F_T one Taylor term further, + dt^3/24 (F^(3)(q_t, q_t, q_t) + 3 H(q_t, q_tt) + A q_ttt).
// A is linear and H bilinear, so the terms are gathered as
//   F + A (c1 q_t + c2 q_tt + c3 q_ttt) + H(q_t, c2 q_t + 3 c3 q_tt) + c3 F^(3)(q_t, q_t, q_t)
// with c1 = dt/2, c2 = dt^2/6, c3 = dt^3/24: one Jacobian and one Hessian product per direction.
template <class R>
__device__ __forceinline__ void ft4_core(const St<1, R>& s, const R* qt, const Var<1, R>& vt, const R* qtt, const R* qttt,
                                         R gm1, R dt, R* FT) {
  constexpr int V = 3;
  const R c1 = R(0.5) * dt, c2 = dt * dt * R(1.0 / 6.0), c3 = dt * dt * dt * R(1.0 / 24.0);
  const R c33 = R(3) * c3;
  R qc[V], qh[V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qc[c] = c1 * qt[c] + c2 * qtt[c] + c3 * qttt[c];
    qh[c] = c2 * qt[c] + c33 * qtt[c];
  }
  const Var<1, R> vc = var1<1, R>(s, qc, gm1), vh = var1<1, R>(s, qh, gm1);
  R F[V], A[V], H[V], T3[V];
  flux<1, R>(s, 0, F);
  dflux<1, R>(s, 0, qc, vc, A);
  d2flux<1, R>(s, 0, qt, vt, qh, vh, d2p_of<1, R>(s, vt, vh, gm1), H);
  d3flux_sym<1, R>(s, 0, qt, vt, gm1, T3);
#pragma unroll
  for (int c = 0; c < V; ++c) FT[c] = F[c] + A[c] + H[c] + c3 * T3[c];
}
template <class R>
__device__ __forceinline__ void ft4_from(const R* q, const R* qt, const R* qtt, const R* qttt, R gm1, R dt, R* FT) {
  const St<1, R> s = base_state<1, R>(q, gm1);
  ft4_core<R>(s, qt, var1<1, R>(s, qt, gm1), qtt, qttt, gm1, dt, FT);
}

// Pressure (double, for the limiters).
template <int DIM>
__device__ __forceinline__ double pressure(const double* q, double gam) {
  double k = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) k += q[1 + d] * q[1 + d];
  return (gam - 1.0) * (q[DIM + 1] - 0.5 * k / q[0]);
}

// Boundary operator of Sec. 2.4: keep the tangential momentum, negate the normal one.
template <int DIM, class T>
__device__ __forceinline__ void reflect(const T* q, const T* nh, T* out) {
  constexpr int V = DIM + 2;
#pragma unroll
  for (int c = 0; c < V; ++c) out[c] = q[c];
  if constexpr (DIM == 1) {
    out[1] = -q[1];
  } else if constexpr (DIM == 2) {
    T mn = q[1] * nh[0] + q[DIM] * nh[DIM - 1];
    out[1] = q[1] - T(2) * mn * nh[0];
    out[DIM] = q[DIM] - T(2) * mn * nh[DIM - 1];
  } else {
    T mn = q[1] * nh[0] + q[2] * nh[1] + q[3] * nh[2];
#pragma unroll
    for (int d = 0; d < 3; ++d) out[1 + d] = q[1 + d] - T(2) * mn * nh[d];
  }
}

template <int DIM, class T>
__device__ __forceinline__ void inflow_state(const double* inflow, T* out) {
  if constexpr (DIM == 1) { out[0] = T(inflow[0]); out[1] = T(inflow[1]); out[2] = T(inflow[3]); }
  else if constexpr (DIM == 2) { out[0] = T(inflow[0]); out[1] = T(inflow[1]); out[DIM] = T(inflow[2]); out[DIM + 1] = T(inflow[3]); }
  else { out[0] = T(inflow[0]); out[1] = T(inflow[1]); out[2] = T(inflow[2]); out[3] = T(0); out[4] = T(inflow[3]); }  // not used: no inflow sides on tetrahedra
}

// Wave speed, time step and end-of-run flag of a step
struct StepDt {
  double s, dt;
  bool idle;  // the end time is reached: the step changes nothing
};
// from the mesh's wave speed (k_pre's maximum): dt from the CFL condition (reading of Sec. 4.1, "CFL 0.08"),
// clipped to T; 0 for a wave speed that is no positive number
__device__ __forceinline__ StepDt step_dt(const Scalars& S, double s, double t) {
  StepDt D;
  D.s = s;
  D.idle = !(t < S.T);
  D.dt = 0.0;
  if (s > 0.0 && isfinite(s)) {
    D.dt = S.cfl / (s * S.geo);
    if (t + D.dt > S.T) D.dt = S.T - t;
  }
  return D;
}
__device__ __forceinline__ StepDt step_dt(const Scalars& S) {
  return step_dt(S, __longlong_as_double((long long)S.s_bits), S.t);
}
// as k_elem left it for the kernels after it
__device__ __forceinline__ StepDt stored_dt(const Scalars& S) { return {S.s, S.dt, S.idle != 0}; }

template <class R>
__device__ __forceinline__ int mesh_id(const int* mesh_of, int i) { return mesh_of ? mesh_of[i] : 0; }

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Elements (and
// edges, numbered in element order) are in space-filling-curve order, so neighbouring work items
// share data; give every XCD one contiguous range of blocks (the grid is padded to a multiple of 8
// blocks) so that shared lines are reused within one L2.
__device__ __forceinline__ int xcd_item() {
  const int nb = (int)gridDim.x;  // multiple of 8
  const int b = (int)blockIdx.x;
  return ((b & 7) * (nb >> 3) + (b >> 3)) * (int)blockDim.x + (int)threadIdx.x;
}

// Per-mesh maximum of a non-negative double: wavefront reduction when the wavefront lies in one
// mesh, else one atomic per lane.
__device__ __forceinline__ void atomic_max_per_mesh(Scalars* sc, int mid, double val, bool valid) {
  int lane = threadIdx.x & 63;
  int m0 = __shfl(mid, 0);
  bool uniform = __all(!valid || mid == m0);
  if (uniform) {
    double x = valid ? val : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
    if (lane == 0 && __any(valid)) atomicMax(&sc[m0].s_bits, (unsigned long long)__double_as_longlong(x));
  } else if (valid) {
    atomicMax(&sc[mid].s_bits, (unsigned long long)__double_as_longlong(val));
  }
}

// ---------------------------------------------------------------------------------------------
// k_pre: pending shock-capturing limiter, moment limiter, checks, wave speed.
//   mode 0: computes the element's total limiter factor theta = theta_shock * theta_moment and
//           stores it (k_elem applies it to the higher modes); wave speed and checks.
//   mode 1: applies only the pending shock-capturing limiter to the stored modes (state read-out).
//   mode 2: stores the pending shock-capturing limiter's factor in theta, changing nothing else
//           (training data for the learned indicator).
// With a learned indicator, elements it clears (ind_flag 0) skip the shock-capturing limiter in
// modes 0 and 1; the positivity limiter is never skipped.
// All limiter arithmetic is float64 on the stored state, its point states those of k_elem (point_dev, limited),
// so the positivity the limiter establishes holds for the states the time-averaged flux is built from.
// ---------------------------------------------------------------------------------------------
// 1/x in float64 for the limiter passes of k_pre (x a positive normal number: a point density
// checked > 0 first, or a cell average >= eps0): the hardware estimate (about 2^-23 relative) and
// two Newton-Raphson steps r <- r + r (1 - x r), each squaring the relative error, to within an ulp
// of the quotient, in 5 instructions instead of the correctly rounded division's 10.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __fma_rn(r, __fma_rn(-x, r, 1.0), r);
  return __fma_rn(r, __fma_rn(-x, r, 1.0), r);
}

template <int DIM>
__device__ __forceinline__ double pressure_r(const double* q, double r, double gam) {
  double k = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) k += q[1 + d] * q[1 + d];
  return (gam - 1.0) * (q[DIM + 1] - 0.5 * k * r);
}

// max and min of float64 values that are no signalling NaNs (results of arithmetic, checked inputs): one
// instruction each.  fmax and fmin come with a second one per operand that would quiet a signalling NaN (11 of
// the 71 instructions per point of k_pre's pass).
__device__ __forceinline__ double max_num(double a, double b) {
  double d;
  asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double min_num(double a, double b) {
  double d;
  asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float max_num(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// sqrt(x) in float64 for x >= 0 (0 gives 1e-140, nothing beside a sound speed; infinity itself):
// the hardware's reciprocal square root and two coupled Newton steps on sqrt(x) and 1/(2 sqrt(x)), to within
// an ulp, in half the instructions of the correctly rounded root with its scaling.  The steps turn infinity
// into a NaN, which the maximum with 1e-200 x, far below the root of every finite x, turns back.
__device__ __forceinline__ double sqrt_nr(double x) {
  const double z = max_num(x, 1e-280);
  const double y = __builtin_amdgcn_rsq(z);
  double g = z * y, h = 0.5 * y;
  double r = __fma_rn(-h, g, 0.5);
  g = __fma_rn(g, r, g);
  h = __fma_rn(h, r, h);
  r = __fma_rn(-g, g, z);
  return max_num(__fma_rn(r, h, g), 1e-200 * z);
}

// Largest |u| + c over states given by u2 = |u|^2 and c2 = gamma p / rho (both float64), for the global
// wave speed s.  Float64 form: in float64.  FP32-mixed form: both square roots by the hardware float32
// square root (a float64 square root, or a correctly rounded float32 one, is a sequence of a dozen
// instructions, and k_pre takes two per limiter point), the largest sum enlarged by a relative 2^-21 in
// float64.  The float32 rounding of u2 and c2 (2^-24 each, halved by the root), the roots (up to
// two ulp, 2^-22) and the sum (2^-24) stay below that margin for u2 and c2 within the float32
// normal range, so the result is never below the float64 value: the condition on s of the
// positivity argument (s at least the largest |u| + c) still holds.
template <class R>
struct Speed {
  R m = R(0);
  __device__ __forceinline__ void add(double u2, double c2) {
    if constexpr (sizeof(R) == sizeof(double)) m = max_num(m, sqrt_nr(u2) + sqrt_nr(c2));
    else m = max_num(m, __builtin_amdgcn_sqrtf(float(u2)) + __builtin_amdgcn_sqrtf(float(c2)));
  }
  __device__ __forceinline__ double get() const {
    if constexpr (sizeof(R) == sizeof(double)) return m;
    else return double(m) * (1.0 + 0x1p-21);
  }
};

// the same of a whole state
template <int DIM, class R>
__device__ __forceinline__ void add_speed(Speed<R>& S, const double* q, double gam) {
  const double r = rcp_nr(q[0]);
  double u2 = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) u2 += (q[1 + d] * r) * (q[1 + d] * r);
  S.add(u2, gam * pressure_r<DIM>(q, r, gam) * r);
}

// Point states in float64, q_bar + theta d with the deviation d = sum_l Q_l phi_l of the unlimited modes.  k_pre's
// limiters and k_elem both evaluate them by these functions, whose every operation is written out, so that the
// states F_T is built from are those the moment limiter made positive, to the last bit.  The factor and the
// average stay outside the sum: where theta brings a density down to eps0, only theta's own few roundings
// (about 4 2^-53 rho_bar) are left in it.  With monomial coefficients scaled by theta and the average among
// them, densities of 1e-12 came out negative beside an average of 100 (P3), of 1000 (P2 and the square).
__device__ __forceinline__ double limited(double qb, double th, double dev) { return __fma_rn(th, dev, qb); }
// mode(l), l = 1 .. ML - 1: the modes
template <int ML, class M>
__device__ __forceinline__ double deviation(M&& mode, const double (&phi)[ML]) {
  double d = mul_rn(mode(1), phi[1]);
#pragma unroll
  for (int l = 2; l < ML; ++l) d = __fma_rn(mode(l), phi[l], d);
  return d;
}
// The square's modes along a line of points: mode(m, j) has degree m along it and j across, leg holds L_1 and L_2 of
// the line's coordinate across; d = U_0 + U_1 L_1 + U_2 L_2 of the coordinate along it.
template <class M>
__device__ __forceinline__ void line_modes(M&& mode, const double* leg, double (&U)[3]) {
  U[0] = __fma_rn(mode(0, 2), leg[1], mul_rn(mode(0, 1), leg[0]));
#pragma unroll
  for (int m = 1; m < 3; ++m) U[m] = __fma_rn(mode(m, 2), leg[1], __fma_rn(mode(m, 1), leg[0], mode(m, 0)));
}
__device__ __forceinline__ double line_deviation(const double (&U)[3], const double* leg) {
  return __fma_rn(leg[1], U[2], __fma_rn(leg[0], U[1], U[0]));
}
// mode numbers of the square: QUAD_AT[i][j] = that of L_i(x) L_j(y)
constexpr int QUAD_AT[3][3] = {{0, 2, 5}, {1, 4, 7}, {3, 6, 8}};

// whether a point's line runs along y (edges 1 and 3)
template <class E>
__device__ __forceinline__ bool along_y(int p) { return p >= E::NI && ((p - E::NI) / E::NQE) % 2 == 1; }
// deviation of variable c from the cell average at point p, from the stored modes (square: y = along_y(p))
template <class E, class R>
__device__ __forceinline__ double point_dev(const RefTab<E, double>& T, const R (&Qh)[E::V][E::ML - 1], int p, bool y, int c) {
  if constexpr (E::kind == ElQuad::kind) {
    double U[3];
    line_modes([&](int m, int j) { return double(Qh[c][(y ? QUAD_AT[j][m] : QUAD_AT[m][j]) - 1]); }, T.leg[p], U);
    return line_deviation(U, T.leg[p] + 2);
  } else {
    return deviation<E::ML>([&](int l) { return double(Qh[c][l - 1]); }, T.phi[p]);
  }
}
// the state q_bar + theta d at point p (one branch for all variables of the square)
template <class E, class R>
__device__ __forceinline__ void point_state(const RefTab<E, double>& T, const double (&qb)[E::V],
                                            const R (&Qh)[E::V][E::ML - 1], double th, int p, double (&q)[E::V]) {
  auto form = [&](auto y) {
#pragma unroll
    for (int c = 0; c < E::V; ++c) q[c] = limited(qb[c], th, point_dev<E, R>(T, Qh, p, y.value, c));
  };
  if constexpr (E::kind == ElQuad::kind)
    if (along_y<E>(p)) return form(std::true_type{});
  form(std::false_type{});
}

// Exact variant of the moment limiter's pressure step (Sec. 3.1; the paper notes the optimal factor
// could be computed at the cost of more arithmetic).  Along the segment q(s) = qb + s D from the
// average to the point state at the density factor, D = q - qb, g(s) = rho (p - eps_p) =
// (gamma-1)(E rho - |M|^2/2) - eps_p rho is the quadratic A s^2 + B s + C (the paper's a_m, b_m, c
// shifted by the target eps_p), with g(0) >= 0 > g(1).  Its root in (0, 1) in the cancellation-free
// form 2C / (-B + sqrt(B^2 - 4AC)) (0 when C <= 0), moved inside by a relative 1e-10 and accepted
// only where p(q(s)) >= eps_p then holds in float64; the result is never below the concavity
// value s_c.
template <int DIM>
__device__ __forceinline__ double exact_segment(const double* qb, const double* q, double epsp, double gam, double s_c) {
  constexpr int V = DIM + 2;
  double D[V];
#pragma unroll
  for (int c = 0; c < V; ++c) D[c] = q[c] - qb[c];
  const double gm1 = gam - 1.0;
  double dMdM = 0.0, dMM = 0.0, MM = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    dMdM += D[1 + d] * D[1 + d];
    dMM += D[1 + d] * qb[1 + d];
    MM += qb[1 + d] * qb[1 + d];
  }
  const double A = gm1 * (D[V - 1] * D[0] - 0.5 * dMdM);
  const double B = gm1 * (D[V - 1] * qb[0] + qb[V - 1] * D[0] - dMM) - epsp * D[0];
  const double C = gm1 * (qb[V - 1] * qb[0] - 0.5 * MM) - epsp * qb[0];
  double sr = 0.0;
  if (C > 0.0) {
    const double den = -B + sqrt(fmax(B * B - 4.0 * A * C, 0.0));
    sr = den > 0.0 ? 2.0 * C / den : 1.0;
  }
  sr = fmin(sr, 1.0) * (1.0 - 1e-10);
  double qs[V];
#pragma unroll
  for (int c = 0; c < V; ++c) qs[c] = qb[c] + sr * D[c];
  if (!(qs[0] > 0.0) || !(pressure<DIM>(qs, gam) >= epsp)) return s_c;
  return fmax(s_c, sr);
}

// The mode is a template argument: each mode's kernel holds only its own path, so the read-out and
// collection paths do not raise the register allocation of the per-step kernel.  Modes: 0 step,
// 1 read-out (pending shock-capturing limiter applied), 2 collection (its factor recorded), 3 step
// with the exact pressure factor of the moment limiter, 4 step with the wave speed from the cell
// averages only, 5 both.
// Element i; returns its wave speed.  mid and pending: its mesh, and whether the shock-capturing limiter of
// the mesh's last step is due.
template <class E, class R, int mode>
__device__ __forceinline__ double pre_elem(const View<R>& v, const int i, const int mid, const bool pending) {
  constexpr int V = E::V, ML = E::ML, DIM = E::DIM, NP = E::NP, K = E::K;
  constexpr bool kStep = mode == 0 || mode >= 3;
  constexpr bool kExact = mode == 3 || mode == 5;  // exact pressure factor of the moment limiter
  constexpr bool kSavg = mode >= 4;                // wave speed from the cell averages only
  const RefTab<E, double>& T = TabSel<E, double>::get();
  const int N = v.N;
  const double gam = v.gamma, eps0 = v.eps0;
  double smax = 0.0;
  {
    double qb[V];
    R Qh[V][ML - 1];
#pragma unroll
    for (int c = 0; c < V; ++c) {
      qb[c] = v.Qbar[(size_t)i * V + c];
#pragma unroll
      for (int l = 0; l < ML - 1; ++l) Qh[c][l] = at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i);
    }
    const double rb = rcp_nr(qb[0]);
    const double pb = pressure_r<DIM>(qb, rb, gam);
    bool finite = true;
#pragma unroll
    for (int c = 0; c < V; ++c) finite = finite && isfinite(qb[c]);
    if (kStep) {
      if (!finite) report(v.err, E_NONFINITE, i);
      else if (!(qb[0] > 0.0) || !(pb > 0.0)) report(v.err, E_POSITIVITY, i);
    }
    const bool ok = finite && qb[0] >= eps0 && pb > 0.0;

    // ---- one pass over the points of the unlimited state: the shock-capturing limiter on the
    // primitive variables (bounds from the edge neighbours' averages relaxed by alpha0 h^1.5;
    // velocity and pressure sampled where the density is positive) when it is due, and the
    // smallest point density and pressure and the largest wave speed, which settle the moment
    // limiter and the wave speed at once when nothing needs limiting
    double th_sc = 1.0;
    // smallest density and pressure over the average and the points of the unlimited state (points with
    // rho > 0; the average itself passes both tests below), largest point wave speed of it
    double rmin = INFINITY, pmin = INFINITY;
    Speed<R> S0;
    bool have_rmin = false;
    const bool detect = mode == 2 || !v.ind_flag || at(v.ind_flag, i) != 0;
    const bool shock_on = v.shock && pending && ok && detect;
    if (shock_on || (kStep && ok)) {
      have_rmin = true;
      // primitive variables of the average (formed again after the point pass, so that they are
      // not live across it)
      auto prim_avg = [&](double* w) {
        w[0] = qb[0];
#pragma unroll
        for (int d = 0; d < DIM; ++d) w[1 + d] = qb[1 + d] * rb;
        w[DIM + 1] = pb;
      };
      // the point pass before the bounds: neither the neighbour states nor the relaxed bounds are
      // live across it (fewer registers)
      double wmax[V], wmin[V];
      prim_avg(wmax);
      prim_avg(wmin);
      // a loop at run time (the table rows are scalar loads): unrolled, the point states of all
      // points were scheduled together and the kernel needed 160 registers (three waves per SIMD
      // instead of four on triangles; 1.5x the time on tetrahedra)
#pragma unroll 1
      for (int p = 0; p < NP; ++p) {
        double q[V];
        point_state<E, R>(T, qb, Qh, 1.0, p, q);
        wmax[0] = max_num(wmax[0], q[0]);
        wmin[0] = min_num(wmin[0], q[0]);
        if (q[0] > 0.0) {
          const double r = rcp_nr(q[0]);
          double u2 = 0.0;
#pragma unroll
          for (int d = 0; d < DIM; ++d) {
            const double u = q[1 + d] * r;
            wmax[1 + d] = max_num(wmax[1 + d], u);
            wmin[1 + d] = min_num(wmin[1 + d], u);
            u2 += u * u;
          }
          const double pp = pressure_r<DIM>(q, r, gam);
          wmax[DIM + 1] = max_num(wmax[DIM + 1], pp);
          wmin[DIM + 1] = min_num(wmin[DIM + 1], pp);
          S0.add(u2, gam * pp * r);
        }
      }
      rmin = wmin[0];
      pmin = wmin[DIM + 1];
      double wb[V], Mx[V], Mn[V];
      prim_avg(wb);
      const double dl = at(v.delta, i);
#pragma unroll
      for (int c = 0; c < V; ++c) { Mx[c] = wb[c] + dl; Mn[c] = wb[c] - dl; }
#pragma unroll
      for (int k = 0; k < K && shock_on; ++k) {
        double qn[V], wn[V];
        const int j = at(v.nbr + (size_t)k * N, i);
        if (j >= 0) {
#pragma unroll
          for (int c = 0; c < V; ++c) qn[c] = v.Qbar[(size_t)j * V + c];
        } else {
          const int bc = at(v.eslot + (size_t)k * N, i) & 3;
          if (bc == SB_REFLECTIVE) {
            double nh[DIM], len2 = 0.0;
#pragma unroll
            for (int d = 0; d < DIM; ++d) { nh[d] = double(at(v.nout + (size_t)(k * DIM + d) * N, i)); len2 += nh[d] * nh[d]; }
            const double il = 1.0 / sqrt(len2);
#pragma unroll
            for (int d = 0; d < DIM; ++d) nh[d] *= il;
            reflect<DIM, double>(qb, nh, qn);
          } else if (bc == SB_INFLOW) {
            inflow_state<DIM, double>(v.inflow, qn);
          } else {
#pragma unroll
            for (int c = 0; c < V; ++c) qn[c] = qb[c];
          }
        }
        const double rn = rcp_nr(qn[0]);
        wn[0] = qn[0];
#pragma unroll
        for (int d = 0; d < DIM; ++d) wn[1 + d] = qn[1 + d] * rn;
        wn[DIM + 1] = pressure_r<DIM>(qn, rn, gam);
#pragma unroll
        for (int c = 0; c < V; ++c) { Mx[c] = max_num(Mx[c], wn[c]); Mn[c] = min_num(Mn[c], wn[c]); }
      }
      if (shock_on) {
#pragma unroll
        for (int c = 0; c < V; ++c) {
          if (wmax[c] > Mx[c]) th_sc = fmin(th_sc, (Mx[c] - wb[c]) / (wmax[c] - wb[c]));
          if (wmin[c] < Mn[c]) th_sc = fmin(th_sc, (wb[c] - Mn[c]) / (wb[c] - wmin[c]));
        }
        th_sc = fmax(0.0, fmin(1.0, th_sc));
      }
    }

    if (mode == 2) {
      at(v.theta, i) = th_sc;  // the factor the limiter would apply; the state is left as it is
    } else if (mode == 1) {
      if (th_sc < 1.0) {
#pragma unroll
        for (int c = 0; c < V; ++c)
#pragma unroll
          for (int l = 0; l < ML - 1; ++l) at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i) = R(th_sc * double(Qh[c][l]));
      }
      if (v.dbg_theta_sc && v.shock && pending) v.dbg_theta_sc[i] = th_sc;
    } else {
      // ---- moment limiter (Sec. 3.1): Step 0 flattens cells below eps0 or with p_bar <= 0;
      // Step 1 density (closed form of the largest theta); Step 2 pressure by concavity, target
      // eps_p = min(eps0, p_bar).
      // When neither the shock limiter nor the density step limits (the common case), the point
      // states of the density, pressure and wave-speed passes are the same; those passes then share
      // one loop.  Every value is computed by the same operations as in the separate passes.
      double th = 1.0;
      Speed<R> S1;
      bool fused = false;
      if (!ok) {
        th = 0.0;
      } else if (have_rmin && th_sc == 1.0 && rmin >= eps0 && pmin >= fmin(eps0, pb)) {
        // nothing limits: the shock pass already evaluated every point's pressure and speed
        fused = true;
        S1 = S0;
      } else {
        double thr = 1.0;
        if (have_rmin && th_sc == 1.0) {
          // the density factor is a decreasing function of the point density: its minimum over
          // the points is its value at the smallest point density
          if (rmin < eps0) thr = fmin(thr, (qb[0] - eps0) / (qb[0] - rmin));
        } else {
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            const double rm = limited(qb[0], th_sc, point_dev<E, R>(T, Qh, p, along_y<E>(p), 0));
            if (rm < eps0) thr = fmin(thr, (qb[0] - eps0) / (qb[0] - rm));
          }
        }
        const double epsp = fmin(eps0, pb);
        const double ts = thr * th_sc;
        th = thr;
        fused = ts == 1.0;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          double q[V];
          point_state<E, R>(T, qb, Qh, ts, p, q);
          const double pt = pressure_r<DIM>(q, rcp_nr(q[0]), gam);
          if (pt < epsp) {
            if (kExact) th = fmin(th, thr * exact_segment<DIM>(qb, q, epsp, gam, (pb - epsp) / (pb - pt)));
            else th = fmin(th, thr * (pb - epsp) / (pb - pt));
          }
          if (fused) add_speed<DIM, R>(S1, q, gam);
        }
      }
      const double tt = th_sc * th;
      at(v.theta, i) = tt;
      if (finite && qb[0] > 0.0 && pb > 0.0) {
        Speed<R> S;
        add_speed<DIM, R>(S, qb, gam);
        if (kSavg) {
          // the cell average's speed only
        } else if (fused && tt == 1.0) {
          S.m = max_num(S.m, S1.m);
        } else if (tt > 0.0) {
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            double q[V];
            point_state<E, R>(T, qb, Qh, tt, p, q);
            add_speed<DIM, R>(S, q, gam);
          }
        }
        smax = S.get();
      }
      if (!isfinite(smax)) {  // |u|^2 or gamma p / rho of a point beyond the range of the arithmetic
        report(v.err, E_NONFINITE, i);
        smax = INFINITY;
      }
      if (v.dbg_theta) v.dbg_theta[i] = th;
      if (v.dbg_theta_sc && v.shock && pending) v.dbg_theta_sc[i] = th_sc;
      if (v.dbg_qlim) {
#pragma unroll
        for (int c = 0; c < V; ++c) {
          v.dbg_qlim[(c * ML) * N + i] = qb[c];
#pragma unroll
          for (int l = 1; l < ML; ++l) v.dbg_qlim[(c * ML + l) * N + i] = tt * double(Qh[c][l - 1]);
        }
      }
    }
  }
  (void)mid;
  return smax;
}

// Element i of k_pre (i may be past the last element: every lane of a wavefront takes part in the
// wave-speed reduction).
template <class E, class R, int mode>
__device__ __forceinline__ void pre_item(const View<R>& v, const int i) {
  constexpr bool kStep = mode == 0 || mode >= 3;
  const bool valid = i < v.N;
  double smax = 0.0;
  int mid = 0;
  if (valid) {
    mid = mesh_id<R>(v.mesh_of, i);
    smax = pre_elem<E, R, mode>(v, i, mid, v.sc[mid].shock_pending != 0);
  }
  if (kStep) {
    if (v.mesh_of) {
      atomic_max_per_mesh(v.sc, mid, smax, valid);
    } else {
      __shared__ double red[4];
      double x = smax;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
      __syncthreads();
      if (threadIdx.x == 0) {
        double m = red[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
        if ((int)gridDim.x <= DIRECT_BLOCKS) atomicMax(&v.sc[0].s_bits, (unsigned long long)__double_as_longlong(m));
        else v.spart[blockIdx.x] = m;
      }
    }
  }
}

template <class E, class R, int mode>
__global__ __launch_bounds__(256) void k_pre(View<R> v) {
  constexpr bool kStep = mode == 0 || mode >= 3;
  // a single mesh at its end time: the step changes nothing (every lane leaves together)
  if (kStep && !v.mesh_of && !(v.sc[0].t < v.sc[0].T)) return;
  pre_item<E, R, mode>(v, xcd_item());
}

// ---------------------------------------------------------------------------------------------
// k_dt: a single mesh of many workgroups: one workgroup of 1024 lanes reduces their maxima.
// ---------------------------------------------------------------------------------------------
static __global__ __launch_bounds__(1024) void k_dt_single(Scalars* sc, const double* spart, int nparts) {
  __shared__ double red[16];
  double x = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) x = fmax(x, spart[b]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x != 0 || !(sc[0].t < sc[0].T)) return;
  double s = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s = fmax(s, red[w]);
  sc[0].s_bits = (unsigned long long)__double_as_longlong(s);
}

// The first element of each mesh keeps the step's values for the kernels after k_elem (which reads other
// fields).
__device__ __forceinline__ void store_dt(Scalars& S, DevError* err, const StepDt& D) {
  S.idle = D.idle;
  if (D.idle) return;
  S.s = D.s;
  S.dt = D.dt;
  if (!(D.s > 0.0) || !isfinite(D.s)) report(err, E_NONFINITE, -1);
}

// ---------------------------------------------------------------------------------------------
// k_elem: projection of F onto the basis, F_T at all points, volume term, edge traces.
// F^h is projected in contravariant form Fc_a = sum_d Jinv[a][d] F_d, so that div F^h =
// sum_a d/dxi_a Fc_a^h and grad D follows from reference second derivatives (affine elements).
// ---------------------------------------------------------------------------------------------
// Stores V values of one record (consecutive, 16-byte aligned when V values fill whole 16-byte
// words) with vector stores.
template <class R, int V>
__device__ __forceinline__ void store_rec(R* p, const R (&x)[V]) {
  if constexpr ((V * sizeof(R)) % 16 == 0) {
    typedef R vec __attribute__((ext_vector_type(V)));
    vec t;
#pragma unroll
    for (int c = 0; c < V; ++c) t[c] = x[c];
    *reinterpret_cast<vec*>(p) = t;
  } else {
#pragma unroll
    for (int c = 0; c < V; ++c) p[c] = x[c];
  }
}

// V values of one record at p (consecutive)
template <class R, int V>
__device__ __forceinline__ void load_rec(const R* p, R (&x)[V]) {
  if constexpr ((V * sizeof(R)) % 16 == 0) {
    typedef R vec __attribute__((ext_vector_type(V)));
    const vec t = *reinterpret_cast<const vec*>(p);
#pragma unroll
    for (int c = 0; c < V; ++c) x[c] = t[c];
  } else {
#pragma unroll
    for (int c = 0; c < V; ++c) x[c] = p[c];
  }
}

// x, formed here as far as the compiler can see: what a rare branch computes from it stays in that
// branch instead of being moved ahead of the loop around it (45 operations per edge, for every element,
// that only boundary edges need).
template <class R>
__device__ __forceinline__ R here(R x) {
  asm volatile("" : "+v"(x));
  return x;
}

// P2 on triangles and tetrahedra (affine elements): everything at a point comes from polynomial
// coefficients formed once per element.
//  * The limited state q_bar + theta sum_l Q_l phi_l in float64 from the modes, as the limiter has it, rounded
//    to the bulk type.  Interior states serve twice (projection and F_T): they wait in LDS between the two
//    where they fit.
//  * grad q in physical coordinates as an affine function of the reference point, G0 + Hx . xi, from the
//    modes' monomial coefficients (the basis in monomials is the table cm).
//  * div F^h and its gradient: Step 1's projection composed with div (and its gradient) at the origin is
//    a fixed table (kd0, kd1), so F^h is never formed; the mass flux M is its own projection, so its
//    divergence comes from grad q.
// The edges come before the volume term: the modes in float64 are dead by the time its accumulators live,
// and are read again for the update.
//
// Bound by instruction issue: 4,020 VALU instructions per wavefront of float32 triangles (5,872 with
// Jacobian and Hessian products and every V_l accumulated at every point): 168 -> 143 us on 999,698 triangles;
// float64 250k 78 -> 62 us; tetrahedra 467 -> 310 us (280k, FP32-mixed) and 163 -> 108 us (25k, float64).
// (States through monomials, whose positivity did not hold, took 3,838 instructions and 140 us; 58, 310, 104.)
template <class E, class R>
struct ElemShape {
  // interior states kept in LDS per lane, where four wavefronts per CU still fit (float64 tetrahedra form
  // them twice)
  static constexpr bool keep = E::kind == ElTri::kind || (E::DIM == 3 && sizeof(R) == 4);
  // bytes per lane: those, or the float32 square's modes and monomials of D
  static constexpr int lds = keep ? E::NI * E::V * (int)sizeof(R)
                                  : (E::kind == ElQuad::kind && sizeof(R) == 4 ? 16 * E::V * (int)sizeof(R) : 0);
  // Waves per SIMD the register allocation targets, the most that spill next to nothing: three for float32
  // triangles (168 registers; 143 us on 999,698 against 146 at two), two for float64 triangles (62 / 67 us on
  // 250k), float32 P3 triangles (152 / 195 us on 250k) and the float32 square (its LDS holds no third; 80 us on
  // 262k with the modes and D in LDS, 128 with them in registers), one elsewhere (float32 tetrahedra: their
  // states fill the LDS with one; 310 us on 280k, 563 at two without them).
  static constexpr int waves = E::DIM != 2 || (sizeof(R) == 8 && E::ML > ElTri::ML) ? 1 : (sizeof(R) == 4 && E::ML == ElTri::ML ? 3 : 2);
};

template <class E, class R>
__device__ __forceinline__ void elem_affine(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = E::V, ML = E::ML, DIM = E::DIM, NI = E::NI, K = E::K, NQE = E::NQE;
  constexpr bool keep = ElemShape<E, R>::keep;
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const RefTab<E, double>& TD = TabSel<E, double>::get();
  const int N = v.N;
  if (i >= N) return;
  // At the end time the step changes nothing: the stored modes are written back as they were.
  // The flag is applied at the store (not by an early return), so its load overlaps the others.
  const bool idle = D.idle;
  const R dt = R(D.dt);
  const R gm1 = R(v.gamma - 1.0);
  extern __shared__ __align__(16) unsigned char dyn[];
  R* sq = reinterpret_cast<R*>(dyn);

  // the stored modes (before the limiter) and the limiter factor theta of this step
  const double th = at(v.theta, i);
  double qb[V], Q[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qbar[(size_t)i * V + c];
    v.Qold[(size_t)i * V + c] = qb[c];  // the step's averages, for the edge fluxes (k_flux, k_update)
#pragma unroll
    for (int l = 1; l < ML; ++l) Q[c][l - 1] = double(at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i));
  }
  // the map's gradient scaled for q's gradients (dt/3) and for D (c1 = dt/2), see Pt2
  R JG[DIM][DIM], JC[DIM][DIM];
#pragma unroll
  for (int x = 0; x < DIM; ++x)
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const R J = at(v.Jinv + (size_t)(x * DIM + d) * N, i);
      JG[x][d] = dt * R(1.0 / 3.0) * J;
      JC[x][d] = R(0.5) * dt * J;
    }

  auto state_at = [&](int p, R* q) {
#pragma unroll
    for (int c = 0; c < V; ++c)
      q[c] = R(limited(qb[c], th, deviation<ML>([&](int l) { return Q[c][l - 1]; }, TD.phi[p])));
  };

  // (dt/3) grad q at the reference point xi: G0[d][c] + sum_b Hx[b][d][c] xi_b
  R G0[DIM][V], Hx[DIM][DIM][V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    double a[ML];  // monomial coefficients of theta sum_l Q_l phi_l (without the constant)
#pragma unroll
    for (int m = 1; m < ML; ++m) {
      double acc = 0.0;
#pragma unroll
      for (int l = m; l < ML; ++l) acc += Q[c][l - 1] * TD.cm[l][m];
      a[m] = th * acc;
    }
    R g[DIM], h[DIM][DIM];  // reference gradient at the origin and (symmetric) Hessian
    if constexpr (DIM == 2) {
      g[0] = R(a[1]); g[1] = R(a[2]);
      h[0][0] = R(2) * R(a[3]); h[0][1] = h[1][0] = R(a[4]); h[1][1] = R(2) * R(a[5]);
    } else {
      g[0] = R(a[1]); g[1] = R(a[2]); g[DIM - 1] = R(a[3]);
      h[0][0] = R(2) * R(a[4]); h[0][1] = h[1][0] = R(a[5]); h[0][DIM - 1] = h[DIM - 1][0] = R(a[6 % ML]);
      h[1][1] = R(2) * R(a[7 % ML]); h[1][DIM - 1] = h[DIM - 1][1] = R(a[8 % ML]); h[DIM - 1][DIM - 1] = R(2) * R(a[9 % ML]);
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      R t = R(0);
#pragma unroll
      for (int x = 0; x < DIM; ++x) t += JG[x][d] * g[x];
      G0[d][c] = t;
#pragma unroll
      for (int b = 0; b < DIM; ++b) {
        R w = R(0);
#pragma unroll
        for (int x = 0; x < DIM; ++x) w += JG[x][d] * h[x][b];
        Hx[b][d][c] = w;
      }
    }
  }

  // Sec. 2.3 Step 1 composed with div: D0 = c1 div F^h and gDr = its reference gradient, at the origin
  R D0[V], gDr[V][DIM];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    D0[c] = R(0);
#pragma unroll
    for (int b = 0; b < DIM; ++b) gDr[c][b] = R(0);
  }
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    D0[0] += R(1.5) * G0[d][1 + d];
#pragma unroll
    for (int b = 0; b < DIM; ++b) gDr[0][b] += R(1.5) * Hx[b][d][1 + d];
  }
#pragma unroll 1
  for (int m = 0; m < NI; ++m) {
    R q[V];
    state_at(m, q);
    if constexpr (keep) {
      R* p = sq + ((size_t)m * blockDim.x + threadIdx.x) * V;
      store_rec<R, V>(p, q);
    }
    const St<DIM, R> s = base_state<DIM, R>(q, gm1);
    R F[DIM][V];
#pragma unroll
    for (int d = 0; d < DIM; ++d) flux<DIM, R>(s, d, F[d]);
#pragma unroll
    for (int x = 0; x < DIM; ++x)
#pragma unroll
      for (int c = 1; c < V; ++c) {
        R fc = R(0);
#pragma unroll
        for (int d = 0; d < DIM; ++d) fc += JC[x][d] * F[d][c];
        D0[c] += T.kd0[m][x] * fc;
#pragma unroll
        for (int b = 0; b < DIM; ++b) gDr[c][b] += T.kd1[m][x][b] * fc;
      }
  }
  R gD[DIM][V];  // c2 times the physical gradient of D, constant
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      R t = R(0);
#pragma unroll
      for (int x = 0; x < DIM; ++x) t += JG[x][d] * gDr[c][x];
      gD[d][c] = t;
    }

  // edge points: the trace n_out . F_T / 2 + hs q (and the ghost side's on boundary edges)
  const double hs0 = 0.5 * D.s;
  auto edge_point = [&](const R* n, R hs, R len2, int slot, int jj, const R* q, const R (&gq)[DIM][V], const R* D) {
    const int e = slot >> 3, side = (slot >> 2) & 1, bc = slot & 3;
    R qt[V], qtt[V], fn[V];
#pragma unroll
    for (int c = 0; c < V; ++c) qt[c] = -D[c];
    const Pt2<DIM, R> s = pt2_of<DIM, R>(q, qt, gm1);
    qtt_of<DIM, R>(s, q, qt, gq, gD, gm1, qtt);
    ftn2<DIM, R>(s, q, qt, qtt, n, gm1, fn);
    R b[V];  // n is half the normal
#pragma unroll
    for (int c = 0; c < V; ++c) b[c] = fn[c] + hs * q[c];
    store_rec<R, V>(v.tr + (((size_t)e * 2 + side) * NQE + jj) * V, b);
    if (bc != SB_INTERIOR) {
      R qg[V], fgn[V], nb[DIM];
#pragma unroll
      for (int d = 0; d < DIM; ++d) nb[d] = here(n[d]);
      if (bc == SB_TRANSPARENT) {
#pragma unroll
        for (int c = 0; c < V; ++c) { qg[c] = q[c]; fgn[c] = fn[c]; }
      } else if (bc == SB_REFLECTIVE) {
        R nh[DIM];
        const R il = R(1) / sqrt(here(len2));
#pragma unroll
        for (int d = 0; d < DIM; ++d) nh[d] = nb[d] * il;
        R qtg[V], qttg[V];
        reflect<DIM, R>(q, nh, qg);
        reflect<DIM, R>(qt, nh, qtg);
        reflect<DIM, R>(qtt, nh, qttg);
        ftn_from<DIM, R>(qg, qtg, qttg, nb, gm1, fgn);
      } else {
        R z[V];
#pragma unroll
        for (int c = 0; c < V; ++c) z[c] = R(0);
        inflow_state<DIM, R>(v.inflow, qg);
        qg[0] = here(qg[0]);
        ftn_from<DIM, R>(qg, z, z, nb, gm1, fgn);
      }
      // the ghost is side 1: its outward normal is -n
      R bg[V];
#pragma unroll
      for (int c = 0; c < V; ++c) bg[c] = hs * qg[c] - fgn[c];
      store_rec<R, V>(v.tr + (((size_t)e * 2 + 1) * NQE + jj) * V, bg);
    }
  };
  // s |n_e| / 2: both elements of an edge hold the same normal up to sign, so they form it alike
  auto load_normal = [&](int k, R* n) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) n[d] = at(v.nout + (size_t)(k * DIM + d) * N, i);
  };
  // (then n is halved, for the trace's factor 1/2, and len2 with it)
  auto half_speed = [&](R* n, R& len2) {
    len2 = R(0);
#pragma unroll
    for (int d = 0; d < DIM; ++d) len2 += n[d] * n[d];
    const R hs = R(hs0 * double(sqrt(len2)));
    len2 *= R(0.25);
#pragma unroll
    for (int d = 0; d < DIM; ++d) n[d] *= R(0.5);
    return hs;
  };
  if constexpr (DIM == 2) {
    // every edge's slot and normal before the first trace is stored (a store holds later loads back)
    int slots[K];
    R nk[K][DIM];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      slots[k] = at(v.eslot + (size_t)k * N, i);
      load_normal(k, nk[k]);
    }
    // along edge k the reference point is (t, 0), (1 - t, t), (0, t), t one of its coordinates: gradients and D are
    // affine in t; edge 1, whose coefficients are sums, last: the others' are the element's own
#pragma unroll
    for (int x = 0; x < K; ++x) {
      const int k = x == 0 ? 0 : 3 - x;
      const int slot = slots[k];
      R* n = nk[k];
      R len2;
      const R hs = half_speed(n, len2);
      R g0[DIM][V], g1[DIM][V], d0[V], d1[V];
#pragma unroll
      for (int c = 0; c < V; ++c) {
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
          g0[d][c] = k == 1 ? G0[d][c] + Hx[0][d][c] : G0[d][c];
          g1[d][c] = k == 0 ? Hx[0][d][c] : (k == 1 ? Hx[1][d][c] - Hx[0][d][c] : Hx[1][d][c]);
        }
        d0[c] = k == 1 ? D0[c] + gDr[c][0] : D0[c];
        d1[c] = k == 0 ? gDr[c][0] : (k == 1 ? gDr[c][1] - gDr[c][0] : gDr[c][1]);
      }
#pragma unroll 1
      for (int jl = 0; jl < NQE; ++jl) {
        const int p = NI + k * NQE + jl;
        const R t = T.xr[p][k == 0 ? 0 : 1];
        R q[V], gq[DIM][V], D[V];
        state_at(p, q);
#pragma unroll
        for (int c = 0; c < V; ++c) {
#pragma unroll
          for (int d = 0; d < DIM; ++d) gq[d][c] = g0[d][c] + g1[d][c] * t;
          D[c] = d0[c] + d1[c] * t;
        }
        // point order of i_e along the edge: reversed on the other side
        edge_point(n, hs, len2, slot, ((slot >> 2) & 1) ? NQE - 1 - jl : jl, q, gq, D);
      }
    }
  } else {
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      const int slot = at(v.eslot + (size_t)k * N, i);
      const int perm = at(v.fperm + (size_t)k * N, i);
      R n[DIM], len2;
      load_normal(k, n);
      const R hs = half_speed(n, len2);
#pragma unroll 1
      for (int jl = 0; jl < NQE; ++jl) {
        const int p = NI + k * NQE + jl;
        R q[V], gq[DIM][V], D[V];
        state_at(p, q);
#pragma unroll
        for (int c = 0; c < V; ++c) {
          D[c] = D0[c];
#pragma unroll
          for (int b = 0; b < DIM; ++b) D[c] += gDr[c][b] * T.xr[p][b];
#pragma unroll
          for (int d = 0; d < DIM; ++d) {
            gq[d][c] = G0[d][c];
#pragma unroll
            for (int b = 0; b < DIM; ++b) gq[d][c] += Hx[b][d][c] * T.xr[p][b];
          }
        }
        edge_point(n, hs, len2, slot, T.pperm[perm][jl], q, gq, D);
      }
    }
  }

  // interior points: volume term V_l = sum_m w_m grad phi_l . F_T, as the moments S = sum_m w_m
  // (1, xi - centroid) F_T (grad phi_l is linear) and their sums once per element: about half the
  // operations of accumulating every V_l at every point.  About the centroid, so that a constant F_T leaves
  // S_0 only, and with the mean gradient in two parts (gmean, gmlo): the balance of S_0 with the edge terms
  // is the same in every step, so what rounding leaves of it adds up.  FP32-mixed against float64 after 100
  // steps of a vortex and a shock: 2.3e-7 (2.3e-7 with every V_l accumulated; 3.0e-7 without gmlo; 1.3e-6
  // with moments about the origin and the basis as monomials, whose coefficients reach 40).
  constexpr int NM = 1 + DIM;
  R S[NM][DIM][V];
#pragma unroll
  for (int y = 0; y < NM; ++y)
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
      for (int c = 0; c < V; ++c) S[y][d][c] = R(0);
#pragma unroll 1
  for (int m = 0; m < NI; ++m) {
    R q[V], qt[V], qtt[V], gq[DIM][V], FT[DIM][V];
    if constexpr (keep) load_rec<R, V>(sq + ((size_t)m * blockDim.x + threadIdx.x) * V, q);
    else state_at(m, q);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      R D = D0[c];
#pragma unroll
      for (int b = 0; b < DIM; ++b) D += gDr[c][b] * T.xr[m][b];
      qt[c] = -D;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        gq[d][c] = G0[d][c];
#pragma unroll
        for (int b = 0; b < DIM; ++b) gq[d][c] += Hx[b][d][c] * T.xr[m][b];
      }
    }
    const Pt2<DIM, R> s = pt2_of<DIM, R>(q, qt, gm1);
    qtt_of<DIM, R>(s, q, qt, gq, gD, gm1, qtt);
    ft2<DIM, R>(s, q, qt, qtt, gm1, FT);
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
      for (int c = 0; c < V; ++c)
        if (c < 1 + d || c == V - 1 || c == 1 + d)  // F_T's momentum part is symmetric: below the diagonal as above
#pragma unroll
          for (int y = 0; y < NM; ++y) S[y][d][c] += T.wm[m][y] * FT[d][c];
  }
#pragma unroll
  for (int d = 0; d < DIM; ++d)
#pragma unroll
    for (int k = 0; k < d; ++k)
#pragma unroll
      for (int y = 0; y < NM; ++y) S[y][k][1 + d] = S[y][d][1 + k];

  // Sec. 2.3 Step 3 / Sec. 3.3 Step 6, volume part: Q^(l) += dt V_l for l >= 2
  // (every load before the first store: a store to the modes would hold the next load back)
  const R thR = R(th);
  R old[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l) old[c][l] = at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i);
  R Ji[DIM][DIM], vol[V][ML - 1];
#pragma unroll
  for (int x = 0; x < DIM; ++x)
#pragma unroll
    for (int d = 0; d < DIM; ++d) Ji[x][d] = at(v.Jinv + (size_t)(x * DIM + d) * N, i);
#pragma unroll
  for (int c = 0; c < V; ++c) {
    // contravariant moments; per pair of directions what a second derivative multiplies; the sums
    R Sc[NM][DIM], P[E::ND2];
#pragma unroll
    for (int y = 0; y < NM; ++y)
#pragma unroll
      for (int x = 0; x < DIM; ++x) {
        R t = R(0);
#pragma unroll
        for (int d = 0; d < DIM; ++d) t += Ji[x][d] * S[y][d][c];
        Sc[y][x] = t;
      }
    int j = 0;
#pragma unroll
    for (int x = 0; x < DIM; ++x)
#pragma unroll
      for (int y = x; y < DIM; ++y) P[j++] = x == y ? Sc[1 + x][x] : Sc[1 + y][x] + Sc[1 + x][y];
#pragma unroll
    for (int l = 1; l < ML; ++l) {
      R t = R(0);
#pragma unroll
      for (int x = 0; x < DIM; ++x) {
        if constexpr (sizeof(R) == 4) t += T.gmlo[x][l] * Sc[0][x];
        t += T.gmean[x][l] * Sc[0][x];
      }
#pragma unroll
      for (int z = 0; z < E::ND2; ++z) t += T.hcen[z][l] * P[z];
      vol[c][l - 1] = t;
    }
  }
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l)
      at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i) = idle ? old[c][l] : thR * old[c][l] + dt * vol[c][l];
  if (v.dbg_vol) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      v.dbg_vol[(c * ML) * N + i] = 0.0;
#pragma unroll
      for (int l = 1; l < ML; ++l) v.dbg_vol[(c * ML + l) * N + i] = double(vol[c][l - 1]);
    }
  }
}

// P2 on the line.
template <class E, class RS>
__device__ __forceinline__ void elem_line2(const View<RS>& v, const int i, const StepDt& D) {
  // The line computes in float64 whatever it stores: the same rate, few registers, and the rounding that is
  // the same in every step where the state is constant does not add up (FP32-mixed against float64 after
  // 60 steps of Riemann problems on 76 cells: 3.2e-7 against 7.4e-7 in float32; a step of 76 cells 7.9 / 7.2 us).
  using R = double;
  constexpr int V = 3, ML = 3, NI = E::NI;
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const int N = v.N;
  if (i >= N) return;
  // At the end time the step changes nothing: the stored modes are written back as they were.
  // The flag is applied at the store (not by an early return), so its load overlaps the others.
  const bool idle = D.idle;
  const R dt = D.dt;
  const R gm1 = v.gamma - 1.0;

  // stored modes (before the limiter) and the limiter factor theta of this step
  R qb[V], Qr[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qbar[(size_t)i * V + c];
    v.Qold[(size_t)i * V + c] = qb[c];  // the step's averages, for the edge fluxes (k_flux, k_update)
#pragma unroll
    for (int l = 1; l < ML; ++l) Qr[c][l - 1] = at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i);
  }
  const R th = at(v.theta, i);
  const R Ji = at(v.Jinv, i);
  // scaled for q's gradient (dt/3) and for F^h (dt/2: D comes out as c1 D, its gradient as c2 grad D), see Pt2
  const R sg3 = dt * (1.0 / 3.0), sc1 = 0.5 * dt;

  // point state of the limited polynomial
  auto state_at = [&](int p, R* q) {
#pragma unroll
    for (int c = 0; c < V; ++c) q[c] = limited(qb[c], th, deviation<ML>([&](int l) { return Qr[c][l - 1]; }, T.phi[p]));
  };

  // grad q and div F^h are linear and their derivatives constant, so they are formed once per element from
  // their values at the reference origin.
  // Sec. 2.3 Step 1: Fc^h = sum_m w_m Fc(q(x_m)) phi_l(x_m)
  R Fh[V][ML];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML; ++l) Fh[c][l] = 0.0;
  for (int m = 0; m < NI; ++m) {
    R q[V], F[V];
    state_at(m, q);
    flux<1, R>(base_state<1, R>(q, gm1), 0, F);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      const R fc = Ji * F[c] * sc1;
#pragma unroll
      for (int l = 0; l < ML; ++l) Fh[c][l] += T.wphi[m][l] * fc;
    }
  }
  // at the origin: D and its derivative, q's gradient and second derivative; the gradient of D along x
  R D0[V], gDr[V], g0[V], Hq[V], gDx[V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    D0[c] = gDr[c] = g0[c] = Hq[c] = 0.0;
#pragma unroll
    for (int l = 0; l < ML; ++l) {
      D0[c] += Fh[c][l] * T.dphi0[0][l];
      gDr[c] += Fh[c][l] * T.d2c[0][l];
    }
#pragma unroll
    for (int l = 1; l < ML; ++l) {
      g0[c] += Qr[c][l - 1] * T.dphi0[0][l];
      Hq[c] += Qr[c][l - 1] * T.d2c[0][l];
    }
    g0[c] *= th;
    Hq[c] *= th;
    gDx[c] = sg3 * (Ji * gDr[c]);
  }

  // Sec. 2.3 Step 2 at point p: q, grad q, D = div F^h, grad D, then q_t, q_tt and what F_T needs.
  auto derivs = [&](int p, R* q, R* qt, R* qtt) {
    R gq[1][V], gD[1][V];
    state_at(p, q);
    const R x = T.xr[p][0];
#pragma unroll
    for (int c = 0; c < V; ++c) {
      qt[c] = -(D0[c] + gDr[c] * x);
      gq[0][c] = sg3 * (Ji * (g0[c] + Hq[c] * x));
      gD[0][c] = gDx[c];
    }
    const Pt2<1, R> s = pt2_of<1, R>(q, qt, gm1);
    qtt_of<1, R>(s, q, qt, gq, gD, gm1, qtt);
    return s;
  };

  // interior points: volume term V_l = sum_m w_m grad phi_l . F_T
  R vol[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l) vol[c][l] = 0.0;
  for (int m = 0; m < NI; ++m) {
    R q[V], qt[V], qtt[V], FT[1][V];
    const Pt2<1, R> s = derivs(m, q, qt, qtt);
    ft2<1, R>(s, q, qt, qtt, gm1, FT);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      const R fc = Ji * FT[0][c];
#pragma unroll
      for (int l = 1; l < ML; ++l) vol[c][l - 1] += T.wdphi[m][0][l] * fc;
    }
  }

  // Sec. 2.3 Step 3 / Sec. 3.3 Step 6, volume part: Q^(l) += dt V_l for l >= 2.  Stored before the
  // edge points (which use the modes held in registers), so the accumulators are free for them.
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 1; l < ML; ++l)
      at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i) = RS(idle ? Qr[c][l - 1] : th * Qr[c][l - 1] + dt * vol[c][l - 1]);
  if (v.dbg_vol) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      v.dbg_vol[(c * ML) * N + i] = 0.0;
#pragma unroll
      for (int l = 1; l < ML; ++l) v.dbg_vol[(c * ML + l) * N + i] = vol[c][l - 1];
    }
  }

  // ends: the trace n_out . F_T / 2 + hs q (and the ghost side's on boundary ends), |n| = 1
  for (int k = 0; k < 2; ++k) {
    const int slot = at(v.eslot + (size_t)k * N, i);
    const int e = slot >> 3, side = (slot >> 2) & 1, bc = slot & 3;
    const R n[1] = {R(at(v.nout + (size_t)k * N, i))};
    const R hs = 0.5 * D.s * fabs(n[0]);
    R q[V], qt[V], qtt[V], fn[V];
    const Pt2<1, R> s = derivs(NI + k, q, qt, qtt);
    ftn2<1, R>(s, q, qt, qtt, n, gm1, fn);
    RS b[V];
#pragma unroll
    for (int c = 0; c < V; ++c) b[c] = RS(0.5 * fn[c] + hs * q[c]);
    store_rec<RS, V>(v.tr + ((size_t)e * 2 + side) * V, b);
    if (bc != SB_INTERIOR) {
      R qg[V], fgn[V];
      if (bc == SB_TRANSPARENT) {
#pragma unroll
        for (int c = 0; c < V; ++c) { qg[c] = q[c]; fgn[c] = fn[c]; }
      } else if (bc == SB_REFLECTIVE) {
        R qtg[V], qttg[V];
        reflect<1, R>(q, n, qg);
        reflect<1, R>(qt, n, qtg);
        reflect<1, R>(qtt, n, qttg);
        ftn_from<1, R>(qg, qtg, qttg, n, gm1, fgn);
      } else {
        const R z[V] = {};
        inflow_state<1, R>(v.inflow, qg);
        ftn_from<1, R>(qg, z, z, n, gm1, fgn);
      }
      // the ghost is side 1: its outward normal is -n
      RS bg[V];
#pragma unroll
      for (int c = 0; c < V; ++c) bg[c] = RS(hs * qg[c] - 0.5 * fgn[c]);
      store_rec<RS, V>(v.tr + ((size_t)e * 2 + 1) * V, bg);
    }
  }
}

// Q2 on the square (its cells are rectangles: the map's gradient is diagonal), by lines of points: the three
// interior rows and the four edges.  A line fixes one coordinate, so the modes and D = div F^h collapse to
// polynomials along it once per line (q and its two derivatives as quadratics, D as its 8 monomials
// collapsed likewise) and a point costs 11 multiply-adds per variable; contracting all 9 modes of q and of
// both F^h at every point took 86.  F^h itself is kept only in the modes that div sees (6 of 9 per direction),
// and the mass flux is its own projection.
//
// Bound by instruction issue.  512x512 squares FP32-mixed 108 -> 79 us, 123,300 in float64 120 -> 62 us.
template <class E, class R>
__device__ __forceinline__ void elem_quad(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = 4, ML = 9, NQE = 3;
  constexpr int MI[9] = {0, 1, 0, 2, 1, 0, 2, 1, 2}, MJ[9] = {0, 0, 1, 0, 1, 2, 1, 2, 2};  // mode l = L_MI(x) L_MJ(y)
  constexpr double r3 = 1.7320508075688772935, r5 = 2.2360679774997896964;  // L_1 = r3 x, L_2 = r5 (3 x^2 - 1) / 2
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const RefTab<E, double>& TD = TabSel<E, double>::get();
  const int N = v.N;
  if (i >= N) return;
  const bool idle = D.idle;  // applied at the store: at the end time the step changes nothing
  const R dt = R(D.dt);
  const R gm1 = R(v.gamma - 1.0);

  // stored modes (before the limiter) and the limiter factor theta of this step
  double qb[V];
  R Qr[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qbar[(size_t)i * V + c];
    v.Qold[(size_t)i * V + c] = qb[c];  // the step's averages, for the edge fluxes (k_flux, k_update)
#pragma unroll
    for (int l = 1; l < ML; ++l) Qr[c][l - 1] = at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i);
  }
  const double th = at(v.theta, i);
  const R thR = R(th);
  const R Ji[2] = {at(v.Jinv, i), at(v.Jinv + (size_t)3 * N, i)};
  // float32: the modes and D's monomials wait in LDS between the lines, which read them once each; read at an
  // offset the compiler cannot follow, or it would keep them in registers
  constexpr bool lds = ElemShape<E, R>::lds > 0;
  extern __shared__ __align__(16) unsigned char dyn[];
  auto put = [&](int at4, const R* x) { *reinterpret_cast<float4*>(dyn + ((size_t)at4 * blockDim.x + threadIdx.x) * 16) = make_float4(x[0], x[1], x[2], x[3]); };
  auto take = [&](int at4, int lane, R* x) {
    const float4 f = *reinterpret_cast<const float4*>(dyn + ((size_t)at4 * blockDim.x + lane) * 16);
    x[0] = f.x; x[1] = f.y; x[2] = f.z; x[3] = f.w;
  };
  auto hidden_lane = [] { int t = (int)threadIdx.x; asm volatile("" : "+v"(t)); return t; };
  auto modes = [&](int lane, int c, R* x) {
    if constexpr (lds) { take(2 * c, lane, x); take(2 * c + 1, lane, x + 4); }
    else {
#pragma unroll
      for (int l = 0; l < ML - 1; ++l) x[l] = Qr[c][l];
    }
  };
  if constexpr (lds)
#pragma unroll
    for (int c = 0; c < V; ++c) { put(2 * c, Qr[c]); put(2 * c + 1, Qr[c] + 4); }
  const R JG[2] = {dt * R(1.0 / 3.0) * Ji[0], dt * R(1.0 / 3.0) * Ji[1]};  // scaled for q's gradients, see Pt2

  // the deviation's modes U on the line through point p (Y: the line runs along y)
  auto state_line = [&](auto Y, int p, int lane, double (&U)[V][3]) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      R Qc[ML - 1];
      modes(lane, c, Qc);
      line_modes([&](int m, int j) { return double(Qc[(Y.value ? QUAD_AT[j][m] : QUAD_AT[m][j]) - 1]); }, TD.leg[p], U[c]);
    }
  };

  // Sec. 2.3 Step 1 composed with div: c1 D in monomials, dm[3 a + b] x^a y^b (x^2 y^2 does not occur)
  R dm[V][8];
  auto monomials = [&](int lane, int c, R* x) {
    if constexpr (lds) { take(2 * V + 2 * c, lane, x); take(2 * V + 2 * c + 1, lane, x + 4); }
    else {
#pragma unroll
      for (int l = 0; l < 8; ++l) x[l] = dm[c][l];
    }
  };
  {
    R Fx[V][2][3], Fy[V][2][3];  // the modes of F^h_x with i = 1, 2 and of F^h_y with j = 1, 2
    const R jc[2] = {R(0.5) * dt * Ji[0], R(0.5) * dt * Ji[1]};
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        Fx[0][m][j] = jc[0] * (thR * Qr[1][QUAD_AT[m + 1][j] - 1]);
        Fy[0][m][j] = jc[1] * (thR * Qr[2][QUAD_AT[j][m + 1] - 1]);
#pragma unroll
        for (int c = 1; c < V; ++c) Fx[c][m][j] = Fy[c][m][j] = R(0);
      }
#pragma unroll 1
    for (int row = 0; row < 3; ++row) {
      double U[V][3];
      state_line(std::false_type{}, 3 * row, lds ? hidden_lane() : 0, U);
#pragma unroll 1
      for (int n = 0; n < 3; ++n) {
        const int m = 3 * row + n;
        R q[V], F[2][V];
#pragma unroll
        for (int c = 0; c < V; ++c) q[c] = R(limited(qb[c], th, line_deviation(U[c], TD.leg[m] + 2)));
        const St<2, R> s = base_state<2, R>(q, gm1);
#pragma unroll
        for (int d = 0; d < 2; ++d) flux<2, R>(s, d, F[d]);
#pragma unroll
        for (int c = 1; c < V; ++c) {
          const R fx = jc[0] * F[0][c], fy = jc[1] * F[1][c];
#pragma unroll
          for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              Fx[c][a][j] += T.wphi[m][QUAD_AT[a + 1][j]] * fx;
              Fy[c][a][j] += T.wphi[m][QUAD_AT[j][a + 1]] * fy;
            }
        }
      }
    }
    // d/dx: L_1' = r3, L_2' = 3 r5 x; the other factor L_j in monomials
#pragma unroll
    for (int c = 0; c < V; ++c) {
#pragma unroll
      for (int a = 0; a < 8; ++a) dm[c][a] = R(0);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const R g = a ? R(3.0 * r5) : R(r3);
        dm[c][3 * a] += g * (Fx[c][a][0] - R(0.5 * r5) * Fx[c][a][2]);
        dm[c][3 * a + 1] += g * (R(r3) * Fx[c][a][1]);
        dm[c][3 * a + 2] += g * (R(1.5 * r5) * Fx[c][a][2]);
        dm[c][a] += g * (Fy[c][a][0] - R(0.5 * r5) * Fy[c][a][2]);
        dm[c][3 + a] += g * (R(r3) * Fy[c][a][1]);
        dm[c][6 + a] += g * (R(1.5 * r5) * Fy[c][a][2]);
      }
      if constexpr (lds) { put(2 * V + 2 * c, dm[c]); put(2 * V + 2 * c + 1, dm[c] + 4); }
    }
  }

  // Sec. 2.3 Step 2 at the three points of a line, p0 .. p0 + 2: body(n, q, qt, qtt, s), n the point's place
  auto line = [&](auto Y, const int p0, auto&& body) {
    constexpr int al = Y.value ? 1 : 0, cr = 1 - al;  // directions along and across
    const R t0 = T.xr[p0][cr];
    double U[V][3];
    const int lane = lds ? hidden_lane() : 0;
    state_line(Y, p0, lane, U);
    R ga[V][2], gc[V][3], e[V][3], ea[V][2], ec[V][3];
    const R c1 = JG[cr] * thR * R(r3), c2 = JG[cr] * thR * R(3.0 * r5) * t0;
#pragma unroll
    for (int c = 0; c < V; ++c) {
      R Qc[ML - 1], dc[8];
      modes(lane, c, Qc);
      monomials(lane, c, dc);
      ga[c][0] = JG[al] * R(r3) * R(th * U[c][1]);
      ga[c][1] = JG[al] * R(3.0 * r5) * R(th * U[c][2]);
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        auto Q = [&](int j) { return Qc[(Y.value ? QUAD_AT[j][m] : QUAD_AT[m][j]) - 1]; };
        auto d = [&](int j) { return dc[Y.value ? 3 * j + m : 3 * m + j]; };
        gc[c][m] = c1 * Q(1) + c2 * Q(2);
        e[c][m] = m == 2 ? d(0) + t0 * d(1) : d(0) + t0 * (d(1) + t0 * d(2));
        ec[c][m] = m == 2 ? JG[cr] * d(1) : JG[cr] * (d(1) + R(2) * t0 * d(2));
      }
      ea[c][0] = JG[al] * e[c][1];
      ea[c][1] = R(2) * JG[al] * e[c][2];
    }
#pragma unroll 1
    for (int n = 0; n < 3; ++n) {
      const int p = p0 + n;
      const R x = T.xr[p][al], l1 = T.leg[p][2], l2 = T.leg[p][3];
      R q[V], qt[V], qtt[V], gq[2][V], gD[2][V];
#pragma unroll
      for (int c = 0; c < V; ++c) {
        q[c] = R(limited(qb[c], th, line_deviation(U[c], TD.leg[p] + 2)));
        qt[c] = -(e[c][0] + x * (e[c][1] + x * e[c][2]));
        gq[al][c] = ga[c][0] + x * ga[c][1];
        gq[cr][c] = gc[c][0] + l1 * gc[c][1] + l2 * gc[c][2];
        gD[al][c] = ea[c][0] + x * ea[c][1];
        gD[cr][c] = ec[c][0] + x * (ec[c][1] + x * ec[c][2]);
      }
      const Pt2<2, R> s = pt2_of<2, R>(q, qt, gm1);
      qtt_of<2, R>(s, q, qt, gq, gD, gm1, qtt);
      body(n, q, qt, qtt, s);
    }
  };

  // interior points: volume term V_l = sum_m w_m grad phi_l . F_T
  {
    R vol[V][ML - 1];
#pragma unroll
    for (int c = 0; c < V; ++c)
#pragma unroll
      for (int l = 0; l < ML - 1; ++l) vol[c][l] = R(0);
#pragma unroll 1
    for (int row = 0; row < 3; ++row)
      line(std::false_type{}, 3 * row, [&](int n, const R* q, const R* qt, const R* qtt, const Pt2<2, R>& s) {
        const int m = 3 * row + n;
        R FT[2][V];
        ft2<2, R>(s, q, qt, qtt, gm1, FT);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int c = 0; c < V; ++c) {
            const R fc = Ji[a] * FT[a][c];
#pragma unroll
            for (int l = 1; l < ML; ++l)
              if ((a == 0 ? MI[l] : MJ[l]) > 0) vol[c][l - 1] += T.wdphi[m][a][l] * fc;
          }
      });
    // Sec. 2.3 Step 3 / Sec. 3.3 Step 6, volume part: Q^(l) += dt V_l for l >= 2.  Stored before the
    // edge points (which use the modes held in registers), so the accumulators are free for them.
    const int lane = lds ? hidden_lane() : 0;
#pragma unroll
    for (int c = 0; c < V; ++c) {
      R Qc[ML - 1];
      modes(lane, c, Qc);
#pragma unroll
      for (int l = 1; l < ML; ++l)
        at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i) = idle ? Qc[l - 1] : thR * Qc[l - 1] + dt * vol[c][l - 1];
    }
    if (v.dbg_vol) {
#pragma unroll
      for (int c = 0; c < V; ++c) {
        v.dbg_vol[(c * ML) * N + i] = 0.0;
#pragma unroll
        for (int l = 1; l < ML; ++l) v.dbg_vol[(c * ML + l) * N + i] = double(vol[c][l - 1]);
      }
    }
  }

  // edge points: the trace n_out . F_T / 2 + hs q (and the ghost side's on boundary edges)
  const double hs0 = 0.5 * D.s;
  // edges 0 (y = -1) and 2 (y = 1, points in descending x), 3 (x = -1, descending y) and 1 (x = 1)
  auto edge_pair = [&](auto Y) {
#pragma unroll 1
    for (int hi = 0; hi < 2; ++hi) {
      const int k = Y.value ? 3 - 2 * hi : 2 * hi;
      const int slot = at(v.eslot + (size_t)k * N, i);
      const int e = slot >> 3, side = (slot >> 2) & 1, bc = slot & 3;
      R n[2], len2 = R(0);
#pragma unroll
      for (int d = 0; d < 2; ++d) { n[d] = at(v.nout + (size_t)(k * 2 + d) * N, i); len2 += n[d] * n[d]; }
      // s |n_e| / 2: both elements of an edge hold the same normal up to sign, so they form it alike
      const R hs = R(hs0 * double(sqrt(len2)));
      line(Y, 9 + 3 * k, [&](int jl, const R* q, const R* qt, const R* qtt, const Pt2<2, R>& s) {
        const int jj = side ? NQE - 1 - jl : jl;  // point order of i_e along the edge
        R fn[V], b[V];
        ftn2<2, R>(s, q, qt, qtt, n, gm1, fn);
#pragma unroll
        for (int c = 0; c < V; ++c) b[c] = R(0.5) * fn[c] + hs * q[c];
        store_rec<R, V>(v.tr + (((size_t)e * 2 + side) * NQE + jj) * V, b);
        if (bc != SB_INTERIOR) {
          R qg[V], fgn[V];
          if (bc == SB_TRANSPARENT) {
#pragma unroll
            for (int c = 0; c < V; ++c) { qg[c] = q[c]; fgn[c] = fn[c]; }
          } else if (bc == SB_REFLECTIVE) {
            const R il = R(1) / sqrt(here(len2));
            const R nh[2] = {n[0] * il, n[1] * il};
            R qtg[V], qttg[V];
            reflect<2, R>(q, nh, qg);
            reflect<2, R>(qt, nh, qtg);
            reflect<2, R>(qtt, nh, qttg);
            ftn_from<2, R>(qg, qtg, qttg, n, gm1, fgn);
          } else {
            R z[V];
#pragma unroll
            for (int c = 0; c < V; ++c) z[c] = R(0);
            inflow_state<2, R>(v.inflow, qg);
            qg[0] = here(qg[0]);
            ftn_from<2, R>(qg, z, z, n, gm1, fgn);
          }
          R bg[V];  // the ghost is side 1: its outward normal is -n
#pragma unroll
          for (int c = 0; c < V; ++c) bg[c] = hs * qg[c] - R(0.5) * fgn[c];
          store_rec<R, V>(v.tr + (((size_t)e * 2 + 1) * NQE + jj) * V, bg);
        }
      });
    }
  };
  edge_pair(std::false_type{});
  edge_pair(std::true_type{});
}

// P3 on triangles.  The Taylor series of Sec. 2.2 one term further: F_T needs q_ttt = -div F_tt, which takes
// the gradient of q_tt, hence the Hessians of q and of D = div F^h (constant: F^h is cubic).  As at degree
// 2 everything goes through the variations of u, p and H = E + p (product rule on F_d = (M_d, M_k u_d +
// p e_d, u_d H)), here with derivatives along the reference coordinates (indices a, e) and the
// contravariant velocity W_a = (dt/3) grad xi_a . u, so that no gradient or Hessian is mapped at a point.
// Scaled time derivatives q1 = c1 q_t, q2 = c2 q_tt, q3 = c3 q_ttt, c1 = dt/2, c2 = dt^2/6, c3 = dt^3/24:
//   u_a = (M_a - u rho_a)/rho,  p_a = (gamma-1)(E_a + |u|^2 rho_a/2 - u.M_a),  and so on (product rule);
//   a transported quantity f (M_k or H) contributes to f2
//     S(f) = -(W.grad f1 + f1 div W + W1.grad f + f div W1),   S_e its derivative along xi_e,
//   M2_k = S(M_k) - grad_k p1,  E2 = S(H),  rho2 = -div M1 (its gradient is constant), and
//   f3 = -(3/4)(W.grad f2 + f2 div W + 4/3 (W1.grad f1 + f1 div W1) + W2.grad f + f div W2);
// a product's time average is a (b + b1 + b2 + b3) + a1 (b + 4/3 b1 + 3/2 b2) + a2 (b + 3/2 b1) + a3 b.
// Second reference derivatives are indexed by their number of eta (0 xx, 1 xy, 2 yy), third ones likewise.
//
// Bound by instruction issue.  250,632 triangles: FP32-mixed 321 -> 151 us, with third variations of the
// flux per direction and every gradient and Hessian mapped at every point before (139 us with the states
// through monomials, whose positivity did not hold); float64 spilled 780 bytes a lane and now nothing.
template <class R>
struct Pt3 {  // what F_T needs of a point besides q and its time derivatives
  R u2[2], p2, H2;  // c2 times the second time derivatives of u, p and H
};
template <class R>
__device__ __forceinline__ Pt3<R> pt3_of(const Pt2<2, R>& s, const R* q1, const R* q2, R gm1) {
  Pt3<R> t;
  R x = q2[3] + s.u2h * q2[0], ww = R(0);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    t.u2[k] = (q2[1 + k] - s.u[k] * q2[0] - R(4.0 / 3.0) * s.ut[k] * q1[0]) * s.r;
    x -= s.u[k] * q2[1 + k];
    ww += s.w[k] * s.ut[k];
  }
  t.p2 = gm1 * (x - R(2.0 / 3.0) * ww);
  t.H2 = q2[3] + t.p2;
  return t;
}
// velocity's third derivative and p3, H3
template <class R>
__device__ __forceinline__ void third(const Pt2<2, R>& s, const Pt3<R>& t, const R* q1, const R* q2, const R* q3, R gm1,
                                      R* u3, R& p3, R& H3) {
  R x = q3[3] + s.u2h * q3[0], w2 = R(0), uu = R(0);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    u3[k] = (q3[1 + k] - s.u[k] * q3[0] - R(1.5) * (s.ut[k] * q2[0] + t.u2[k] * q1[0])) * s.r;
    x -= s.u[k] * q3[1 + k];
    w2 += s.w[k] * t.u2[k];
    uu += s.ut[k] * s.ut[k];
  }
  p3 = gm1 * (x - R(1.5) * w2 - q1[0] * uu);
  H3 = q3[3] + p3;
}
template <class R>
__device__ __forceinline__ void ft3(const Pt2<2, R>& s, const Pt3<R>& t, const R* q, const R* q1, const R* q2, const R* q3,
                                    R gm1, R FT[2][4]) {
  R u3[2], p3, H3;
  third<R>(s, t, q1, q2, q3, gm1, u3, p3, H3);
  const R pb = s.p + s.pt + t.p2 + p3;
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    const R B = s.u[d] + s.ut[d] + t.u2[d] + u3[d], X = s.u[d] + R(4.0 / 3.0) * s.ut[d] + R(1.5) * t.u2[d];
    const R Y = s.u[d] + R(1.5) * s.ut[d], Z = s.u[d];
    FT[d][0] = q[1 + d] + q1[1 + d] + q2[1 + d] + q3[1 + d];
#pragma unroll
    for (int k = d; k < 2; ++k) {
      R f = q[1 + k] * B + q1[1 + k] * X + q2[1 + k] * Y + q3[1 + k] * Z;
      if (k == d) f += pb;
      FT[d][1 + k] = f;
      FT[k][1 + d] = f;
    }
    FT[d][3] = s.H * B + s.Ht * X + t.H2 * Y + H3 * Z;
  }
}
template <class R>
__device__ __forceinline__ void ftn3(const Pt2<2, R>& s, const Pt3<R>& t, const R* q, const R* q1, const R* q2, const R* q3,
                                     const R* n, R gm1, R* FTn) {
  R u3[2], p3, H3;
  third<R>(s, t, q1, q2, q3, gm1, u3, p3, H3);
  const R pb = s.p + s.pt + t.p2 + p3;
  const R un = s.u[0] * n[0] + s.u[1] * n[1], u1n = s.ut[0] * n[0] + s.ut[1] * n[1];
  const R u2n = t.u2[0] * n[0] + t.u2[1] * n[1], u3n = u3[0] * n[0] + u3[1] * n[1];
  const R B = un + u1n + u2n + u3n, X = un + R(4.0 / 3.0) * u1n + R(1.5) * u2n, Y = un + R(1.5) * u1n;
  FTn[0] = R(0);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    FTn[0] += (q[1 + k] + q1[1 + k] + q2[1 + k] + q3[1 + k]) * n[k];
    FTn[1 + k] = q[1 + k] * B + q1[1 + k] * X + q2[1 + k] * Y + q3[1 + k] * un + pb * n[k];
  }
  FTn[3] = s.H * B + s.Ht * X + t.H2 * Y + H3 * un;
}

// q2 and q3 at a point from q, q1 and their reference derivatives (h1, the Hessian of q1, and r2e, the
// gradient of rho2, are the element's constants)
template <class R>
__device__ __forceinline__ void evolve3(const Pt2<2, R>& s, const R* q, const R (&gq)[2][4], const R (&hq)[3][4],
                                        const R* q1, const R (&g1)[2][4], const R (&h1)[3][4], const R (&JG)[2][2],
                                        const R* r2e, R gm1, R* q2, R* q3, Pt3<R>& t) {
  R ua[2][2], u1a[2][2], y[2][2], uab[3][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      ua[a][k] = (gq[a][1 + k] - s.u[k] * gq[a][0]) * s.r;
      y[a][k] = g1[a][1 + k] - s.u[k] * g1[a][0];
      u1a[a][k] = (y[a][k] - ua[a][k] * q1[0] - s.ut[k] * gq[a][0]) * s.r;
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = a; b < 2; ++b)
#pragma unroll
      for (int k = 0; k < 2; ++k)
        uab[a + b][k] = (hq[a + b][1 + k] - s.u[k] * hq[a + b][0] - ua[b][k] * gq[a][0] - ua[a][k] * gq[b][0]) * s.r;
  // p, p1 and with them H, H1: gradients and Hessians
  R Ha[2], H1a[2], p1a[2], Hab[3], H1ab[3], p1ab[3];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    Ha[a] = gq[a][3] + gm1 * (gq[a][3] + s.u2h * gq[a][0] - s.u[0] * gq[a][1] - s.u[1] * gq[a][2]);
    p1a[a] = gm1 * (g1[a][3] + s.u2h * g1[a][0] - s.u[0] * g1[a][1] - s.u[1] * g1[a][2] - ua[a][0] * s.w[0] -
                    ua[a][1] * s.w[1]);
    H1a[a] = g1[a][3] + p1a[a];
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = a; b < 2; ++b) {
      const int j = a + b;
      const R uu = ua[a][0] * ua[b][0] + ua[a][1] * ua[b][1];
      Hab[j] = hq[j][3] + gm1 * (hq[j][3] + s.u2h * hq[j][0] - s.u[0] * hq[j][1] - s.u[1] * hq[j][2] - q[0] * uu);
      p1ab[j] = gm1 * (h1[j][3] + s.u2h * h1[j][0] - s.u[0] * h1[j][1] - s.u[1] * h1[j][2] - ua[b][0] * y[a][0] -
                       ua[b][1] * y[a][1] - ua[a][0] * y[b][0] - ua[a][1] * y[b][1] + uu * q1[0] -
                       uab[j][0] * s.w[0] - uab[j][1] * s.w[1]);
      H1ab[j] = h1[j][3] + p1ab[j];
    }
  // contravariant velocities, their divergences and the divergences' gradients
  R W[2], W1[2], Wa[2][2], W1a[2][2], dW[2], dW1[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    W[c] = JG[c][0] * s.u[0] + JG[c][1] * s.u[1];
    W1[c] = JG[c][0] * s.ut[0] + JG[c][1] * s.ut[1];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      Wa[a][c] = JG[c][0] * ua[a][0] + JG[c][1] * ua[a][1];
      W1a[a][c] = JG[c][0] * u1a[a][0] + JG[c][1] * u1a[a][1];
    }
  }
  const R divW = Wa[0][0] + Wa[1][1], divW1 = W1a[0][0] + W1a[1][1];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    dW[e] = JG[0][0] * uab[e][0] + JG[0][1] * uab[e][1] + JG[1][0] * uab[1 + e][0] + JG[1][1] * uab[1 + e][1];
    R x = -r2e[e];
    x -= W[0] * h1[e][0] + W[1] * h1[1 + e][0] + divW * g1[e][0] + Wa[e][0] * g1[0][0] + Wa[e][1] * g1[1][0] + dW[e] * q1[0];
    x -= divW1 * gq[e][0] + W1a[e][0] * gq[0][0] + W1a[e][1] * gq[1][0] + W1[0] * hq[e][0] + W1[1] * hq[1 + e][0];
    dW1[e] = x * s.r;
  }
  // q2 and its gradient
  R q2a[2][4];
  q2[0] = R(0);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    q2[0] -= JG[a][0] * g1[a][1] + JG[a][1] * g1[a][2];
    q2a[a][0] = r2e[a];
  }
#pragma unroll
  for (int c = 1; c < 4; ++c) {
    const R f = c == 3 ? s.H : q[c], f1 = c == 3 ? s.Ht : q1[c];
    R fa[2], f1a[2], fab[3], f1ab[3];
#pragma unroll
    for (int a = 0; a < 2; ++a) { fa[a] = c == 3 ? Ha[a] : gq[a][c]; f1a[a] = c == 3 ? H1a[a] : g1[a][c]; }
#pragma unroll
    for (int j = 0; j < 3; ++j) { fab[j] = c == 3 ? Hab[j] : hq[j][c]; f1ab[j] = c == 3 ? H1ab[j] : h1[j][c]; }
    R x = W[0] * f1a[0] + W[1] * f1a[1] + f1 * divW + W1[0] * fa[0] + W1[1] * fa[1] + f * divW1;
    if (c < 3) x += JG[0][c - 1] * p1a[0] + JG[1][c - 1] * p1a[1];
    q2[c] = -x;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      R z = Wa[e][0] * f1a[0] + Wa[e][1] * f1a[1] + W[0] * f1ab[e] + W[1] * f1ab[1 + e] + f1a[e] * divW + f1 * dW[e];
      z += W1a[e][0] * fa[0] + W1a[e][1] * fa[1] + W1[0] * fab[e] + W1[1] * fab[1 + e] + fa[e] * divW1 + f * dW1[e];
      if (c < 3) z += JG[0][c - 1] * p1ab[e] + JG[1][c - 1] * p1ab[1 + e];
      q2a[e][c] = -z;
    }
  }
  t = pt3_of<R>(s, q1, q2, gm1);
  // q3
  const R uu = s.ut[0] * s.ut[0] + s.ut[1] * s.ut[1];
  const R z0 = q2[1] - s.u[0] * q2[0], z1 = q2[2] - s.u[1] * q2[0];
  R p2a[2], H2a[2], W2[2];
  R divN = R(0);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    p2a[a] = gm1 * (q2a[a][3] + s.u2h * q2a[a][0] - s.u[0] * q2a[a][1] - s.u[1] * q2a[a][2] - ua[a][0] * z0 - ua[a][1] * z1 -
                    R(2.0 / 3.0) * gq[a][0] * uu - R(4.0 / 3.0) * (s.w[0] * u1a[a][0] + s.w[1] * u1a[a][1]));
    H2a[a] = q2a[a][3] + p2a[a];
    W2[a] = JG[a][0] * t.u2[0] + JG[a][1] * t.u2[1];
    divN += JG[a][0] * q2a[a][1] + JG[a][1] * q2a[a][2];
  }
  const R divW2 = (divN - W[0] * q2a[0][0] - W[1] * q2a[1][0] - divW * q2[0] -
                   R(4.0 / 3.0) * (W1[0] * g1[0][0] + W1[1] * g1[1][0] + divW1 * q1[0]) - W2[0] * gq[0][0] - W2[1] * gq[1][0]) * s.r;
  q3[0] = R(-0.75) * divN;
#pragma unroll
  for (int c = 1; c < 4; ++c) {
    const R f = c == 3 ? s.H : q[c], f1 = c == 3 ? s.Ht : q1[c], f2 = c == 3 ? t.H2 : q2[c];
    R x = W[0] * (c == 3 ? H2a[0] : q2a[0][c]) + W[1] * (c == 3 ? H2a[1] : q2a[1][c]) + f2 * divW;
    x += R(4.0 / 3.0) * (W1[0] * (c == 3 ? H1a[0] : g1[0][c]) + W1[1] * (c == 3 ? H1a[1] : g1[1][c]) + f1 * divW1);
    x += W2[0] * (c == 3 ? Ha[0] : gq[0][c]) + W2[1] * (c == 3 ? Ha[1] : gq[1][c]) + f * divW2;
    if (c < 3) x += JG[0][c - 1] * p2a[0] + JG[1][c - 1] * p2a[1];
    q3[c] = R(-0.75) * x;
  }
}

template <class E, class R>
__device__ __forceinline__ void elem_tri3(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = 4, ML = 10, NI = E::NI, K = E::K, NQE = E::NQE;
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const RefTab<E, double>& TD = TabSel<E, double>::get();
  const int N = v.N;
  if (i >= N) return;
  const bool idle = D.idle;  // applied at the store: at the end time the step changes nothing
  const R dt = R(D.dt);
  const R gm1 = R(v.gamma - 1.0);
  extern __shared__ __align__(16) unsigned char dyn[];
  R* sq = reinterpret_cast<R*>(dyn);

  // the stored modes (before the limiter) and the limiter factor theta of this step; point states
  const double th = at(v.theta, i);
  double qb[V], Q[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qbar[(size_t)i * V + c];
    v.Qold[(size_t)i * V + c] = qb[c];  // the step's averages, for the edge fluxes (k_flux, k_update)
#pragma unroll
    for (int l = 1; l < ML; ++l) Q[c][l - 1] = double(at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i));
  }
  auto state_at = [&](int p, R* q) {
#pragma unroll
    for (int c = 0; c < V; ++c)
      q[c] = R(limited(qb[c], th, deviation<ML>([&](int l) { return Q[c][l - 1]; }, TD.phi[p])));
  };
  R JG[2][2], JC[2][2];  // dt/3 and -dt/2 times the map's gradient
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const R J = at(v.Jinv + (size_t)(x * 2 + d) * N, i);
      JG[x][d] = dt * R(1.0 / 3.0) * J;
      JC[x][d] = R(-0.5) * dt * J;
    }
  // Taylor coefficients at the reference origin (gradient, Hessian, third derivatives) from the monomial ones
  R g0[2][V], h0[3][V], t3[4][V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    double a[ML];
#pragma unroll
    for (int m = 1; m < ML; ++m) {
      double acc = 0.0;
#pragma unroll
      for (int l = m; l < ML; ++l) acc += Q[c][l - 1] * TD.cm[l][m];
      a[m] = th * acc;
    }
    g0[0][c] = R(a[1]); g0[1][c] = R(a[2]);
    h0[0][c] = R(2) * R(a[3]); h0[1][c] = R(a[4]); h0[2][c] = R(2) * R(a[5]);
    t3[0][c] = R(6) * R(a[6]); t3[1][c] = R(2) * R(a[7]); t3[2][c] = R(2) * R(a[8]); t3[3][c] = R(6) * R(a[9]);
  }
  // Sec. 2.3 Step 1 composed with -c1 div and its derivatives at the origin (kd0, kd1, kd2): the Taylor
  // coefficients of q1, a quadratic; M is its own projection, so rho's come from the gradients of M
  R b0[V], b1[2][V], h1[3][V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    b0[c] = R(0);
#pragma unroll
    for (int x = 0; x < 2; ++x) b1[x][c] = R(0);
#pragma unroll
    for (int j = 0; j < 3; ++j) h1[j][c] = R(0);
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const R J = R(-1.5) * JG[x][d];
      b0[0] += J * g0[x][1 + d];
#pragma unroll
      for (int y = 0; y < 2; ++y) b1[y][0] += J * h0[x + y][1 + d];
#pragma unroll
      for (int j = 0; j < 3; ++j) h1[j][0] += J * t3[x + j][1 + d];
    }
#pragma unroll 1
  for (int m = 0; m < NI; ++m) {
    R q[V];
    state_at(m, q);
    store_rec<R, V>(sq + ((size_t)m * blockDim.x + threadIdx.x) * V, q);
    const St<2, R> s = base_state<2, R>(q, gm1);
    R F[2][V];
#pragma unroll
    for (int d = 0; d < 2; ++d) flux<2, R>(s, d, F[d]);
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
      for (int c = 1; c < V; ++c) {
        const R fc = JC[z][0] * F[0][c] + JC[z][1] * F[1][c];
        b0[c] += T.kd0[m][z] * fc;
#pragma unroll
        for (int w = 0; w < 2; ++w) b1[w][c] += T.kd1[m][z][w] * fc;
#pragma unroll
        for (int j = 0; j < 3; ++j) h1[j][c] += T.kd2[m][z][j] * fc;
      }
  }
  R r2e[2];
#pragma unroll
  for (int e = 0; e < 2; ++e)
    r2e[e] = -(JG[0][0] * h1[e][1] + JG[0][1] * h1[e][2] + JG[1][0] * h1[1 + e][1] + JG[1][1] * h1[1 + e][2]);

  // edges (before the volume term: its accumulators and the modes are then not live together)
  {
    const double hs0 = 0.5 * D.s;
    int slots[K];
    R nk[K][2];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      slots[k] = at(v.eslot + (size_t)k * N, i);
#pragma unroll
      for (int d = 0; d < 2; ++d) nk[k][d] = at(v.nout + (size_t)(k * 2 + d) * N, i);
    }
    // along edge k the reference point is (t, 0), (1 - t, t), (0, t); edge 1, whose coefficients are sums,
    // last
#pragma unroll
    for (int x = 0; x < K; ++x) {
      const int k = x == 0 ? 0 : 3 - x;
      const int slot = slots[k];
      const int e = slot >> 3, side = (slot >> 2) & 1, bc = slot & 3;
      R* n = nk[k];
      R len2 = n[0] * n[0] + n[1] * n[1];
      const R hs = R(hs0 * double(sqrt(len2)));  // s |n_e| / 2; then half the normal, for the trace
      len2 *= R(0.25);
      n[0] *= R(0.5);
      n[1] *= R(0.5);
#pragma unroll 1
      for (int jl = 0; jl < NQE; ++jl) {
        const int p = NI + k * NQE + jl;
        const R tt = T.xr[p][k == 0 ? 0 : 1];
        R q[V], q1[V], gq[2][V], g1[2][V], hq[3][V];
        state_at(p, q);
#pragma unroll
        for (int c = 0; c < V; ++c) {
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            const R l0 = k == 1 ? g0[w][c] + h0[w][c] + R(0.5) * t3[w][c] : g0[w][c];
            const R l1 = k == 0 ? h0[w][c] : (k == 2 ? h0[w + 1][c] : h0[w + 1][c] - h0[w][c] - t3[w][c] + t3[w + 1][c]);
            const R l2 = R(0.5) * (k == 0 ? t3[w][c] : (k == 2 ? t3[w + 2][c] : t3[w][c] + t3[w + 2][c])) -
                         (k == 1 ? t3[w + 1][c] : R(0));
            gq[w][c] = l0 + tt * (l1 + tt * l2);
            const R m0 = k == 1 ? b1[w][c] + h1[w][c] : b1[w][c];
            const R m1 = k == 0 ? h1[w][c] : (k == 2 ? h1[w + 1][c] : h1[w + 1][c] - h1[w][c]);
            g1[w][c] = m0 + tt * m1;
          }
#pragma unroll
          for (int j = 0; j < 3; ++j)
            hq[j][c] = (k == 1 ? h0[j][c] + t3[j][c] : h0[j][c]) +
                       tt * (k == 0 ? t3[j][c] : (k == 2 ? t3[j + 1][c] : t3[j + 1][c] - t3[j][c]));
          const R d0 = k == 1 ? b0[c] + b1[0][c] + R(0.5) * h1[0][c] : b0[c];
          const R d1 = k == 0 ? b1[0][c] : (k == 2 ? b1[1][c] : b1[1][c] - b1[0][c] - h1[0][c] + h1[1][c]);
          const R d2 = R(0.5) * (k == 0 ? h1[0][c] : (k == 2 ? h1[2][c] : h1[0][c] + h1[2][c])) - (k == 1 ? h1[1][c] : R(0));
          q1[c] = d0 + tt * (d1 + tt * d2);
        }
        const Pt2<2, R> s = pt2_of<2, R>(q, q1, gm1);
        Pt3<R> t;
        R q2[V], q3[V], fn[V], b[V];
        evolve3<R>(s, q, gq, hq, q1, g1, h1, JG, r2e, gm1, q2, q3, t);
        ftn3<R>(s, t, q, q1, q2, q3, n, gm1, fn);
#pragma unroll
        for (int c = 0; c < V; ++c) b[c] = fn[c] + hs * q[c];
        const int jj = side ? NQE - 1 - jl : jl;  // point order of i_e along the edge
        store_rec<R, V>(v.tr + (((size_t)e * 2 + side) * NQE + jj) * V, b);
        if (bc != SB_INTERIOR) {
          R qg[V], fgn[V], nb[2] = {here(n[0]), here(n[1])};
          if (bc == SB_TRANSPARENT) {
#pragma unroll
            for (int c = 0; c < V; ++c) { qg[c] = q[c]; fgn[c] = fn[c]; }
          } else {
            R q1g[V], q2g[V], q3g[V];
            if (bc == SB_REFLECTIVE) {
              const R il = R(1) / sqrt(here(len2));
              const R nh[2] = {nb[0] * il, nb[1] * il};
              reflect<2, R>(q, nh, qg);
              reflect<2, R>(q1, nh, q1g);
              reflect<2, R>(q2, nh, q2g);
              reflect<2, R>(q3, nh, q3g);
            } else {
              inflow_state<2, R>(v.inflow, qg);
              qg[0] = here(qg[0]);
#pragma unroll
              for (int c = 0; c < V; ++c) q1g[c] = q2g[c] = q3g[c] = R(0);
            }
            const Pt2<2, R> sg = pt2_of<2, R>(qg, q1g, gm1);
            ftn3<R>(sg, pt3_of<R>(sg, q1g, q2g, gm1), qg, q1g, q2g, q3g, nb, gm1, fgn);
          }
          R bg[V];  // the ghost is side 1: its outward normal is -n
#pragma unroll
          for (int c = 0; c < V; ++c) bg[c] = hs * qg[c] - fgn[c];
          store_rec<R, V>(v.tr + (((size_t)e * 2 + 1) * NQE + jj) * V, bg);
        }
      }
    }
  }

  // interior points: moments sum_m w_m (1, x, y, x^2, x y, y^2) F_T of the volume term, (x, y) the reference
  // point less the centroid, the products less their means: a constant F_T leaves the first one only
  constexpr int NM = 6;
  R S[NM][2][V];
#pragma unroll
  for (int y = 0; y < NM; ++y)
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int c = 0; c < V; ++c) S[y][d][c] = R(0);
#pragma unroll 1
  for (int m = 0; m < NI; ++m) {
    const R x = T.xr[m][0], y = T.xr[m][1];
    const R xx = R(0.5) * x * x, xy = x * y, yy = R(0.5) * y * y;
    R q[V], q1[V], gq[2][V], g1[2][V], hq[3][V];
    load_rec<R, V>(sq + ((size_t)m * blockDim.x + threadIdx.x) * V, q);
#pragma unroll
    for (int c = 0; c < V; ++c) {
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        gq[w][c] = g0[w][c] + h0[w][c] * x + h0[w + 1][c] * y + t3[w][c] * xx + t3[w + 1][c] * xy + t3[w + 2][c] * yy;
        g1[w][c] = b1[w][c] + h1[w][c] * x + h1[w + 1][c] * y;
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) hq[j][c] = h0[j][c] + t3[j][c] * x + t3[j + 1][c] * y;
      q1[c] = b0[c] + b1[0][c] * x + b1[1][c] * y + h1[0][c] * xx + h1[1][c] * xy + h1[2][c] * yy;
    }
    const Pt2<2, R> s = pt2_of<2, R>(q, q1, gm1);
    Pt3<R> t;
    R q2[V], q3[V], FT[2][V];
    evolve3<R>(s, q, gq, hq, q1, g1, h1, JG, r2e, gm1, q2, q3, t);
    ft3<R>(s, t, q, q1, q2, q3, gm1, FT);
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int c = 0; c < V; ++c)
        if (d == 1 || c != 2)  // F_T's momentum part is symmetric
#pragma unroll
          for (int z = 0; z < NM; ++z) S[z][d][c] += T.wm[m][z] * FT[d][c];
  }
#pragma unroll
  for (int z = 0; z < NM; ++z) S[z][0][2] = S[z][1][1];

  // Sec. 2.3 Step 3 / Sec. 3.3 Step 6, volume part: Q^(l) += dt V_l for l >= 2
  const R thR = R(th);
  R old[V][ML - 1], Ji[2][2], vol[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l) old[c][l] = at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int d = 0; d < 2; ++d) Ji[x][d] = at(v.Jinv + (size_t)(x * 2 + d) * N, i);
#pragma unroll
  for (int c = 0; c < V; ++c) {
    R C[NM][2];  // contravariant moments; what the second and third derivatives multiply; the sums
#pragma unroll
    for (int z = 0; z < NM; ++z)
#pragma unroll
      for (int x = 0; x < 2; ++x) C[z][x] = Ji[x][0] * S[z][0][c] + Ji[x][1] * S[z][1][c];
    const R P[3] = {C[1][0], C[2][0] + C[1][1], C[2][1]};
    const R U[4] = {R(0.5) * C[3][0], C[4][0] + R(0.5) * C[3][1], R(0.5) * C[5][0] + C[4][1], R(0.5) * C[5][1]};
#pragma unroll
    for (int l = 1; l < ML; ++l) {
      R t = R(0);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        if constexpr (sizeof(R) == 4) t += T.gmlo[x][l] * C[0][x];
        t += T.gmean[x][l] * C[0][x];
      }
#pragma unroll
      for (int z = 0; z < 3; ++z) t += T.hcen[z][l] * P[z];
#pragma unroll
      for (int z = 0; z < 4; ++z) t += T.d3c[z][l] * U[z];
      vol[c][l - 1] = t;
    }
  }
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l)
      at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i) = idle ? old[c][l] : thR * old[c][l] + dt * vol[c][l];
  if (v.dbg_vol) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      v.dbg_vol[(c * ML) * N + i] = 0.0;
#pragma unroll
      for (int l = 1; l < ML; ++l) v.dbg_vol[(c * ML + l) * N + i] = double(vol[c][l - 1]);
    }
  }
}

// P3 on the line.  The Taylor series of Sec. 2.2 one term further, through the variations of the flux: F_T needs
// q_ttt = -F_tt,x, which takes the gradient of q_tt, hence the second derivatives of q and of D = (F^h)_x
// (constant: F^h is cubic).  With subscripts x for derivatives along the line,
//   q_t = -D,  q_tt = H(q_x, D) + A D_x,
//   q_tt,x = F3(q_x, q_x, D) + H(q_xx, D) + 2 H(q_x, D_x) + A D_xx,
//   q_ttt = -(F3(q_x, q_t, q_t) - 2 H(D_x, q_t) + H(q_x, q_tt) + A q_tt,x).
// The point derivatives come from Taylor coefficients at the reference origin, formed once per element.
template <class E, class R>
__device__ __forceinline__ void elem_line3(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = 3, ML = 4, NI = E::NI;
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const RefTab<E, double>& TD = TabSel<E, double>::get();
  const int N = v.N;
  if (i >= N) return;
  const bool idle = D.idle;
  const R dt = R(D.dt);
  const R gm1 = R(v.gamma - 1.0);

  double qb[V];
  R Qr[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qbar[(size_t)i * V + c];
    v.Qold[(size_t)i * V + c] = qb[c];  // the step's averages, for the edge fluxes (k_flux, k_update)
#pragma unroll
    for (int l = 1; l < ML; ++l) Qr[c][l - 1] = at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i);
  }
  const double th = at(v.theta, i);
  const R thR = R(th);
  const R Ji = at(v.Jinv, i);

  // point state of the limited polynomial in float64, then rounded to the bulk precision
  auto state_at = [&](int p, R* q) {
#pragma unroll
    for (int c = 0; c < V; ++c)
      q[c] = R(limited(qb[c], th, deviation<ML>([&](int l) { return double(Qr[c][l - 1]); }, TD.phi[p])));
  };

  // Sec. 2.3 Step 1: Fc^h = sum_m w_m Fc(q(x_m)) phi_l(x_m)
  R Fh[V][ML];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML; ++l) Fh[c][l] = R(0);
  for (int m = 0; m < NI; ++m) {
    R q[V], F[V];
    state_at(m, q);
    flux<1, R>(base_state<1, R>(q, gm1), 0, F);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      const R fc = Ji * F[c];
#pragma unroll
      for (int l = 0; l < ML; ++l) Fh[c][l] += T.wphi[m][l] * fc;
    }
  }

  // Taylor coefficients in the reference coordinate: q's first, second and third derivative (theta folded in),
  // D, its first and second; HD the second derivative of D along x
  R g0[V], h0[V], t3[V], D0[V], D1[V], D2[V], HD[V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    g0[c] = h0[c] = t3[c] = D0[c] = D1[c] = D2[c] = R(0);
#pragma unroll
    for (int l = 0; l < ML; ++l) {
      D0[c] += Fh[c][l] * T.dphi0[0][l];
      D1[c] += Fh[c][l] * T.d2c[0][l];
      D2[c] += Fh[c][l] * T.d3c[0][l];
    }
#pragma unroll
    for (int l = 1; l < ML; ++l) {
      g0[c] += Qr[c][l - 1] * T.dphi0[0][l];
      h0[c] += Qr[c][l - 1] * T.d2c[0][l];
      t3[c] += Qr[c][l - 1] * T.d3c[0][l];
    }
    g0[c] *= thR;
    h0[c] *= thR;
    t3[c] *= thR;
    HD[c] = Ji * Ji * D2[c];
  }

  auto point = [&](int p, R* q, R* qt, R* qtt, R* qttt, R* FT) {
    R gq[V], Hq[V], Dp[V], gD[V];
    state_at(p, q);
    const R x = T.xr[p][0], x2 = R(0.5) * x * x;
#pragma unroll
    for (int c = 0; c < V; ++c) {
      Dp[c] = D0[c] + D2[c] * x2 + D1[c] * x;
      gq[c] = Ji * (g0[c] + h0[c] * x + t3[c] * x2);
      gD[c] = Ji * (D1[c] + D2[c] * x);
      Hq[c] = Ji * Ji * (h0[c] + t3[c] * x);
    }
    const St<1, R> s = base_state<1, R>(q, gm1);
    const Var<1, R> vD = var1<1, R>(s, Dp, gm1), vq = var1<1, R>(s, gq, gm1), vg = var1<1, R>(s, gD, gm1);
    R H[V], A[V];
    d2flux<1, R>(s, 0, gq, vq, Dp, vD, d2p_of<1, R>(s, vq, vD, gm1), H);
    dflux<1, R>(s, 0, gD, vg, A);
#pragma unroll
    for (int c = 0; c < V; ++c) { qt[c] = -Dp[c]; qtt[c] = H[c] + A[c]; }
    Var<1, R> vt;  // the variation of q_t = -D (var1 is linear)
    vt.du[0] = -vD.du[0];
    vt.dp = -vD.dp;
    const Var<1, R> vtt = var1<1, R>(s, qtt, gm1), vH = var1<1, R>(s, Hq, gm1), vHD = var1<1, R>(s, HD, gm1);
    R t1[V], t2[V], t3v[V], t4[V], dq2[V];  // dq2 = q_tt,x
    d3flux<1, R>(s, 0, gq, vq, gq, vq, Dp, vD, gm1, t1);
    d2flux<1, R>(s, 0, Hq, vH, Dp, vD, d2p_of<1, R>(s, vH, vD, gm1), t2);
    d2flux<1, R>(s, 0, gq, vq, gD, vg, d2p_of<1, R>(s, vq, vg, gm1), t3v);
    dflux<1, R>(s, 0, HD, vHD, t4);
#pragma unroll
    for (int c = 0; c < V; ++c) dq2[c] = t1[c] + t2[c] + R(2) * t3v[c] + t4[c];
    const Var<1, R> v2 = var1<1, R>(s, dq2, gm1);
    d3flux<1, R>(s, 0, gq, vq, qt, vt, qt, vt, gm1, t1);
    d2flux<1, R>(s, 0, gD, vg, qt, vt, d2p_of<1, R>(s, vg, vt, gm1), t2);
    d2flux<1, R>(s, 0, gq, vq, qtt, vtt, d2p_of<1, R>(s, vq, vtt, gm1), t3v);
    dflux<1, R>(s, 0, dq2, v2, t4);
#pragma unroll
    for (int c = 0; c < V; ++c) qttt[c] = -(t1[c] - R(2) * t2[c] + t3v[c] + t4[c]);
    ft4_core<R>(s, qt, vt, qtt, qttt, gm1, dt, FT);
  };

  R vol[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 0; l < ML - 1; ++l) vol[c][l] = R(0);
  for (int m = 0; m < NI; ++m) {
    R q[V], qt[V], qtt[V], qttt[V], FT[V];
    point(m, q, qt, qtt, qttt, FT);
#pragma unroll
    for (int c = 0; c < V; ++c) {
      const R fc = Ji * FT[c];
#pragma unroll
      for (int l = 1; l < ML; ++l) vol[c][l - 1] += T.wdphi[m][0][l] * fc;
    }
  }
#pragma unroll
  for (int c = 0; c < V; ++c)
#pragma unroll
    for (int l = 1; l < ML; ++l)
      at(v.Qh + (size_t)(c * (ML - 1) + l - 1) * N, i) = idle ? Qr[c][l - 1] : thR * Qr[c][l - 1] + dt * vol[c][l - 1];
  if (v.dbg_vol) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      v.dbg_vol[(c * ML) * N + i] = 0.0;
#pragma unroll
      for (int l = 1; l < ML; ++l) v.dbg_vol[(c * ML + l) * N + i] = double(vol[c][l - 1]);
    }
  }

  // ends: the trace n_out . F_T / 2 + hs q (and the ghost side's on boundary ends), |n| = 1
  for (int k = 0; k < 2; ++k) {
    const int slot = at(v.eslot + (size_t)k * N, i);
    const int e = slot >> 3, side = (slot >> 2) & 1, bc = slot & 3;
    const R n[1] = {at(v.nout + (size_t)k * N, i)};
    const R hs = R(0.5 * D.s * double(fabs(n[0])));
    R q[V], qt[V], qtt[V], qttt[V], FT[V], b[V];
    point(NI + k, q, qt, qtt, qttt, FT);
#pragma unroll
    for (int c = 0; c < V; ++c) b[c] = R(0.5) * (n[0] * FT[c]) + hs * q[c];
    store_rec<R, V>(v.tr + ((size_t)e * 2 + side) * V, b);
    if (bc != SB_INTERIOR) {
      R qg[V], FTg[V];
      if (bc == SB_TRANSPARENT) {
#pragma unroll
        for (int c = 0; c < V; ++c) { qg[c] = q[c]; FTg[c] = FT[c]; }
      } else if (bc == SB_REFLECTIVE) {
        R qtg[V], qttg[V], q3g[V];
        reflect<1, R>(q, n, qg);
        reflect<1, R>(qt, n, qtg);
        reflect<1, R>(qtt, n, qttg);
        reflect<1, R>(qttt, n, q3g);
        ft4_from<R>(qg, qtg, qttg, q3g, gm1, dt, FTg);
      } else {
        const R z[V] = {};
        inflow_state<1, R>(v.inflow, qg);
        ft4_from<R>(qg, z, z, z, gm1, dt, FTg);
      }
      R bg[V];  // the ghost is side 1: its outward normal is -n
#pragma unroll
      for (int c = 0; c < V; ++c) bg[c] = hs * qg[c] - R(0.5) * (n[0] * FTg[c]);
      store_rec<R, V>(v.tr + ((size_t)e * 2 + 1) * V, bg);
    }
  }
}

template <class E, class R>
__device__ __forceinline__ void elem_step(const View<R>& v, const int i, const StepDt& D) {
  if constexpr (E::DEG == 3 && E::DIM == 2) elem_tri3<E, R>(v, i, D);
  else if constexpr (E::DEG == 3) elem_line3<E, R>(v, i, D);
  else if constexpr (E::kind == ElTri::kind || E::DIM == 3) elem_affine<E, R>(v, i, D);
  else if constexpr (E::kind == ElQuad::kind) elem_quad<E, R>(v, i, D);
  else elem_line2<E, R>(v, i, D);
}

// whether element i is the first of its mesh
template <class R>
__device__ __forceinline__ bool mesh_first(const View<R>& v, int i, int mid) {
  return i == 0 || (v.mesh_of && at(v.mesh_of, i - 1) != mid);
}

template <class E, class R>
__device__ __forceinline__ void elem_item(const View<R>& v, const int i) {
  if (i >= v.N) return;
  const int mid = mesh_id<R>(v.mesh_of, i);
  const StepDt D = step_dt(v.sc[mid]);
  if (mesh_first(v, i, mid)) store_dt(v.sc[mid], v.err, D);
  elem_step<E, R>(v, i, D);
}

template <class E, class R>
__global__ __launch_bounds__(256, (ElemShape<E, R>::waves)) void k_elem(View<R> v) {
  elem_item<E, R>(v, xcd_item());
}

// ---------------------------------------------------------------------------------------------
// Edge fluxes, formed by both elements of an edge from the same data.  F*_T . n_e = (1/2)(n_e.F_T(q+)
// + n_e.F_T(q-)) - (s |n_e| / 2)(q+ - q-) at each edge point (Eq. (LLF) with the scaled normal; it is
// linear in the two sides' values, so each element wrote its half n_out.F_T/2 + (s |n_e|/2) q and F* is
// side 0 minus side 1); f^LxW_e = (1/2) sum_j omega_j F*_j and
// f^LxF_e = (1/2) n_e.(F(q_bar_j) + F(q_bar_i)) - (s |n_e| / 2)(q_bar_j - q_bar_i) in float64.  The two
// elements get the same bits up to the sign (the averages' update is conservative to rounding): F* and
// f^LxW are formed in the first element's orientation and point order, and every operation of f^LxF
// is written out with its own rounding, changes sign with the normal and is symmetric in the two states.
// (Left to the compiler, one side's energy row was fused into the sum and the other's was not.)
// ---------------------------------------------------------------------------------------------
// F* at the points of edge e in the first element's order
template <class E, class R>
__device__ __forceinline__ void edge_points(const View<R>& v, int e, R (&fs)[E::NQE][E::V]) {
  constexpr int V = E::V, NQE = E::NQE;
  const R* t = v.tr + (size_t)e * (2 * NQE * V);
#pragma unroll
  for (int jj = 0; jj < NQE; ++jj) {
    R a[V], b[V];
    load_rec<R, V>(t + jj * V, a);
    load_rec<R, V>(t + (NQE + jj) * V, b);
#pragma unroll
    for (int c = 0; c < V; ++c) fs[jj][c] = a[c] - b[c];
  }
}

// f^LxW_e in float64, summed in the edge's point order
template <class E, class R>
__device__ __forceinline__ void lxw_average(const RefTab<E, R>& T, const R (&fs)[E::NQE][E::V], double (&W)[E::V]) {
#pragma unroll
  for (int c = 0; c < E::V; ++c) W[c] = 0.0;
#pragma unroll
  for (int jj = 0; jj < E::NQE; ++jj) {
    const double w = 0.5 * double(T.om[jj]);
#pragma unroll
    for (int c = 0; c < E::V; ++c) W[c] = __fma_rn(w, double(fs[jj][c]), W[c]);
  }
}

// Velocity and pressure of an average, every operation with its own rounding
template <int DIM>
struct AvgPrim { double u[DIM], p; };
template <int DIM>
__device__ __forceinline__ AvgPrim<DIM> avg_prim(const double* q, double gm1) {
  AvgPrim<DIM> P;
  const double r = 1.0 / q[0];
  double mu = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    P.u[d] = mul_rn(q[1 + d], r);
    mu = __fma_rn(q[1 + d], P.u[d], mu);
  }
  P.p = mul_rn(gm1, __fma_rn(-0.5, mu, q[DIM + 1]));
  return P;
}
// n . F(q)
template <int DIM>
__device__ __forceinline__ void avg_flux(const double* q, const AvgPrim<DIM>& P, const double* n, double* F) {
  double un = mul_rn(P.u[0], n[0]), mn = mul_rn(q[1], n[0]);
#pragma unroll
  for (int d = 1; d < DIM; ++d) { un = __fma_rn(P.u[d], n[d], un); mn = __fma_rn(q[1 + d], n[d], mn); }
  F[0] = mn;
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = __fma_rn(q[1 + k], un, mul_rn(P.p, n[k]));
  F[DIM + 1] = mul_rn(un, add_rn(q[DIM + 1], P.p));
}

// f^LxF through local edge k of element i (edge e on its side `side`), out of the element; q and P are
// the element's average.
template <class E, class R>
__device__ __forceinline__ void lxf_out(const View<R>& v, int i, int k, int e, int side, const double (&q)[E::V],
                                        const AvgPrim<E::DIM>& P, double s, double (&f)[E::V]) {
  constexpr int V = E::V, DIM = E::DIM;
  const double gm1 = v.gamma - 1.0;
  double n[DIM], len2 = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const double x = v.e_n[(size_t)e * DIM + d];
    n[d] = side ? -x : x;
    len2 = __fma_rn(x, x, len2);
  }
  const double len = sqrt(len2);
  const int j = at(v.nbr + (size_t)k * v.N, i);
  double qn[V];
  if (j >= 0) {
#pragma unroll
    for (int c = 0; c < V; ++c) qn[c] = v.Qold[(size_t)j * V + c];
  } else {
    const int bc = at(v.eslot + (size_t)k * v.N, i) & 3;
    if (bc == SB_REFLECTIVE) {
      double nh[DIM];
#pragma unroll
      for (int d = 0; d < DIM; ++d) nh[d] = n[d] / len;
      reflect<DIM, double>(q, nh, qn);
    } else if (bc == SB_INFLOW) {
      inflow_state<DIM, double>(v.inflow, qn);
    } else {
#pragma unroll
      for (int c = 0; c < V; ++c) qn[c] = q[c];
    }
  }
  const AvgPrim<DIM> Pn = avg_prim<DIM>(qn, gm1);
  double Fo[V], Fn[V];
  avg_flux<DIM>(q, P, n, Fo);
  avg_flux<DIM>(qn, Pn, n, Fn);
  const double h = mul_rn(0.5, mul_rn(s, len));
#pragma unroll
  for (int c = 0; c < V; ++c) f[c] = __fma_rn(-h, sub_rn(qn[c], q[c]), mul_rn(0.5, add_rn(Fo[c], Fn[c])));
}

// ---------------------------------------------------------------------------------------------
// Damping factor mu (Sec. 3.3 Step 5b): the largest mu in [0,1] with positive density and
// pressure >= eps_p on qL + mu (qa - qL).  Along the segment (gamma-1)(rho E - |M|^2/2) - eps_p rho
// is a quadratic a mu^2 + b mu + c with c >= 0; its first zero is 2c/(-b + sqrt(b^2 - 4ac)),
// which is then lowered by ulps until the condition holds in float64.
// ---------------------------------------------------------------------------------------------
template <int DIM>
__device__ __forceinline__ bool mu_ok(const double* qL, const double* qa, double mu, double gam, double epsp) {
  constexpr int V = DIM + 2;
  double q[V];
#pragma unroll
  for (int c = 0; c < V; ++c) q[c] = qL[c] + mu * (qa[c] - qL[c]);
  return q[0] > 0.0 && pressure<DIM>(q, gam) >= epsp;
}

// Sufficient for mu_ok at mu = 1 without its division: rho (p - eps_p) exceeds a hundred times the
// rounding of either form (each is a sum of terms no larger than (gamma-1)(|E| rho + |M|^2) and
// eps_p rho, with relative errors of a few 2^-53).
template <int DIM>
__device__ __forceinline__ bool mu_sure(const double* q, double gam, double epsp) {
  double k = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) k += q[1 + d] * q[1 + d];
  const double Er = q[DIM + 1] * q[0], g1 = gam - 1.0;
  return q[0] > 0.0 && g1 * (Er - 0.5 * k) - epsp * q[0] > 1e-13 * (g1 * (fabs(Er) + k) + epsp * q[0]);
}

template <int DIM>
__device__ double mu_solve(const double* qL, const double* qa, double gam, double epsp) {
  constexpr int V = DIM + 2;
  if (mu_ok<DIM>(qL, qa, 1.0, gam, epsp)) return 1.0;
  double dq[V];
#pragma unroll
  for (int c = 0; c < V; ++c) dq[c] = qa[c] - qL[c];
  double mL2 = 0.0, mLd = 0.0, dd2 = 0.0;
#pragma unroll
  for (int k = 1; k <= DIM; ++k) { mL2 += qL[k] * qL[k]; mLd += qL[k] * dq[k]; dd2 += dq[k] * dq[k]; }
  const double g1 = gam - 1.0;
  const double a = g1 * (dq[0] * dq[V - 1] - 0.5 * dd2);
  const double b = g1 * (qL[0] * dq[V - 1] + dq[0] * qL[V - 1] - mLd) - epsp * dq[0];
  const double c = g1 * (qL[0] * qL[V - 1] - 0.5 * mL2) - epsp * qL[0];
  if (!(c > 0.0)) return 0.0;
  // target equal to the LxF corner's own pressure (p(q^LxF) <= eps0): c is zero up to rounding,
  // g(mu) = mu (a mu + b), and with b <= 0 only mu = 0 is feasible (the ulp search would end there)
  if (b <= 0.0 && pressure<DIM>(qL, gam) <= epsp) return 0.0;
  const double den = -b + sqrt(fmax(0.0, b * b - 4.0 * a * c));
  double mu = den > 0.0 ? 2.0 * c / den : 0.0;
  mu = fmin(1.0, fmax(0.0, mu));
  for (int it = 0; it < 64 && mu > 0.0 && !mu_ok<DIM>(qL, qa, mu, gam, epsp); ++it) mu = nextafter(mu, 0.0);
  if (!mu_ok<DIM>(qL, qa, mu, gam, epsp)) mu = 0.0;
  return mu;
}

// ---------------------------------------------------------------------------------------------
// k_flux: everything an element does on its edges, in one kernel: F* at the edge points, f^LxW and
// f^LxF, the higher-moment update of Sec. 3.3 Step 6
//   Q^(l) -= dt/|T| sum_k eps_ik (1/2) sum_j omega_j phi_l(x_kj) F*_kj . n_e,  l >= 2
// (the volume part was added by k_elem), the flux limiter of Steps 4-5 in float64, and the average's
// update with f^LxW on every edge, which k_update replaces where an edge is limited.  Limiter readings:
// every edge flux of the element carries eps_ik (as in the printed Step 4); Cases 1-4 of the sorted
// Delta f are evaluated as "each edge with Delta f_k < 0 gets min(1, Gamma / |sum of the negative
// Delta f|)" (no sort); the corner states keep the Lax-Friedrichs flux on the edges switched off, so that
// corner 000 is the pure LxF update; the pressure target is eps_p = min(eps0, p(q^LxF)).
//
// Bound by HBM: the traces and the modes in and out.  Each edge's fluxes are formed twice (by both
// elements) so that no per-edge flux record is written and gathered again: on 999,698 triangles,
// FP32-mixed, k_edge, k_flim and k_update (380 + 174 + 400 MB) took 67 + 43 + 88 us; k_flux and the new
// k_update (461 + 68 MB) take 120 + 19 us.  Traces of an edge's two sides are one record (96 bytes here): the element
// that reads both touches one or two cache lines.
// ---------------------------------------------------------------------------------------------
// Faces one after another in a loop, their fluxes kept in LDS, or all unrolled, their fluxes in registers:
// unrolled where every face's loads then fit the registers together (1D; float32 P2 triangles: 191
// registers, 120 us on 999,698 against 134 us in the loop), the loop elsewhere (it needs no spill and
// little code: float64 triangles 46 against 50 us on 250k, the float64 square 36 / 41 us on 123k (FP32-mixed
// 42 / 41 on 262k), P3 39 / 39.5 us on 250k, tetrahedra 112 / 138 us on 280k and 37 / 84 us in float64 on 25k).
template <class E, class R>
struct FluxShape {
  static constexpr bool roll = E::DIM > 1 && !(E::kind == ElTri::kind && E::DEG == 2 && sizeof(R) == 4);
  static constexpr int lds = roll ? E::K * 2 * E::V * 8 : 0;  // bytes per lane
};

template <class E, class R>
__device__ __forceinline__ void flux_step(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = E::V, ML = E::ML, DIM = E::DIM, K = E::K, NQE = E::NQE;
  const RefTab<E, R>& T = TabSel<E, R>::get();
  const int N = v.N;
  if (i >= N) return;
  const double dt = D.dt, s = D.s;
  // at the end time the step changes nothing: applied at the stores, and nothing is reported
  const bool idle = D.idle;
  const double gam = v.gamma;
  const double area = at(v.area, i);
  const double r = dt / area;
  double qb[V];
  R Qh[V][ML - 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    qb[c] = v.Qold[(size_t)i * V + c];
#pragma unroll
    for (int l = 0; l < ML - 1; ++l) Qh[c][l] = at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i);
  }
  const AvgPrim<DIM> P = avg_prim<DIM>(qb, gam - 1.0);
  double fW[K][V], fF[K][V];
  int slot[K];
  auto face = [&](const int k, double (&W)[V], double (&F)[V]) -> int {
    const int sl = at(v.eslot + (size_t)k * N, i);
    const int e = sl >> 3, side = (sl >> 2) & 1;
    const double ep = side ? -1.0 : 1.0;
    R fs[NQE][V];
    edge_points<E, R>(v, e, fs);
    lxw_average<E, R>(T, fs, W);
#pragma unroll
    for (int c = 0; c < V; ++c) W[c] *= ep;
    lxf_out<E, R>(v, i, k, e, side, qb, P, s, F);
    // higher moments; the element's point jl is the first element's jl, the reverse of it, or (on a
    // face) that of the vertex permutation, which moves the two three-point orbits 1-3 and 4-6 alike
    const R re = R(r * ep);
    const int perm = (DIM == 3) ? at(v.fperm + (size_t)k * N, i) : 0;
#pragma unroll
    for (int jl = 0; jl < NQE; ++jl) {
      const int pj = (DIM == 3) ? T.pperm[perm][jl] : 0;
#pragma unroll
      for (int c = 0; c < V; ++c) {
        R x;
        if constexpr (DIM == 3) {
          if (jl == 0) x = fs[0][c];
          else {
            const int o = jl < 4 ? 1 : 4;
            x = pj == o ? fs[o][c] : (pj == o + 1 ? fs[o + 1][c] : fs[o + 2][c]);
          }
        } else {
          x = side ? fs[NQE - 1 - jl][c] : fs[jl][c];
        }
        const R f = re * x;
#pragma unroll
        for (int l = 1; l < ML; ++l) Qh[c][l - 1] -= T.ephi[k][jl][l] * f;
      }
    }
    return sl;
  };
  if constexpr (FluxShape<E, R>::roll) {
    // one face at a time: the lane's fluxes wait in LDS (columns of consecutive lanes) until the modes are
    // stored
    extern __shared__ __align__(16) unsigned char dyn[];
    double* sf = reinterpret_cast<double*>(dyn) + threadIdx.x;
    const int bs = (int)blockDim.x;
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      double W[V], F[V];
      face(k, W, F);
#pragma unroll
      for (int c = 0; c < V; ++c) { sf[((2 * k) * V + c) * bs] = W[c]; sf[((2 * k + 1) * V + c) * bs] = F[c]; }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      slot[k] = at(v.eslot + (size_t)k * N, i);
#pragma unroll
      for (int c = 0; c < V; ++c) { fW[k][c] = sf[((2 * k) * V + c) * bs]; fF[k][c] = sf[((2 * k + 1) * V + c) * bs]; }
    }
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) slot[k] = face(k, fW[k], fF[k]);
  }
  if (!idle) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      double q = qb[c];
#pragma unroll
      for (int k = 0; k < K; ++k) q -= r * fW[k][c];
      v.Qbar[(size_t)i * V + c] = q;
#pragma unroll
      for (int l = 0; l < ML - 1; ++l) at(v.Qh + (size_t)(c * (ML - 1) + l) * N, i) = Qh[c][l];
    }
  }
  if (v.fLxW) {  // stage read-out
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int c = 0; c < V; ++c) {
        v.fLxW[(size_t)(slot[k] >> 2) * V + c] = fW[k][c];
        v.fLxF[(size_t)(slot[k] >> 2) * V + c] = fF[k][c];
      }
  }
  // Steps 4-5
  double Gam = area * qb[0] / dt, df[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    Gam -= fF[k][0];
    df[k] = fF[k][0] - fW[k][0];
  }
  double Sneg = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (df[k] < 0.0) Sneg += df[k];
  bool bad = Gam < 0.0;
  double Lam[K];
#pragma unroll
  for (int k = 0; k < K; ++k) Lam[k] = df[k] < 0.0 ? fmax(0.0, fmin(1.0, Gam / fabs(Sneg))) : 1.0;
  double qL[V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) acc += fF[k][c];
    qL[c] = qb[c] - r * acc;
  }
  const double pL = qL[0] > 0.0 ? pressure<DIM>(qL, gam) : -1.0;
  bad = bad || !(pL > 0.0);
  const double epsp = fmin(v.eps0, pL);
  // the flux of an edge that is switched on
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int c = 0; c < V; ++c) fW[k][c] = Lam[k] * fW[k][c] + (1.0 - Lam[k]) * fF[k][c];
  // Corner states: nearly always every one passes the sufficient test mu_sure (then mu = 1 for all of
  // them); otherwise the lane solves every corner, in a loop at run time (15 inlined solves on the
  // tetrahedron are more code than the instruction cache holds, and a wavefront runs through once).
  auto corner = [&](int a, double* qa) {
#pragma unroll
    for (int c = 0; c < V; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < K; ++k) acc += ((a >> k) & 1) ? fW[k][c] : fF[k][c];
      qa[c] = qb[c] - r * acc;
    }
  };
  double mm[K];
#pragma unroll
  for (int k = 0; k < K; ++k) mm[k] = 1.0;
  bool sure = pL > 0.0;
#pragma unroll
  for (int a = 1; a < (1 << K); ++a) {
    double qa[V];
    corner(a, qa);
    sure = sure && mu_sure<DIM>(qa, gam, epsp);
  }
  if (!sure) {
#pragma unroll 1
    for (int a = 1; a < (1 << K); ++a) {
      double qa[V];
      corner(a, qa);
      const double mu = pL > 0.0 ? mu_solve<DIM>(qL, qa, gam, epsp) : 0.0;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if ((a >> k) & 1) mm[k] = fmin(mm[k], mu);
    }
  }
  if (bad && !idle) report(v.err, E_CFL, i);
#pragma unroll
  for (int k = 0; k < K; ++k) v.cedge[(size_t)(slot[k] >> 3) * 2 + ((slot[k] >> 2) & 1)] = Lam[k] * mm[k];
}

template <class E, class R>
__device__ __forceinline__ void flux_item(const View<R>& v, const int i) {
  if (i < v.N) flux_step<E, R>(v, i, stored_dt(v.sc[mesh_id<R>(v.mesh_of, i)]));
}

template <class E, class R>
__global__ __launch_bounds__(256) void k_flux(View<R> v) {
  flux_item<E, R>(v, xcd_item());
}

// ---------------------------------------------------------------------------------------------
// k_update: Sec. 3.3 Step 6 for the averages, theta_k = Lambda_{e_ik} = min(1, both sides' candidates):
//   Q^(1) -= dt/|T| sum_k eps_ik [theta_k f^LxW + (1 - theta_k) f^LxF]            (float64)
// k_flux has formed it for theta = 1 on every edge; an element with a limited edge forms it again
// from the step's averages and the traces (rare: the same functions, so the same fluxes bit for bit).
// Then the positivity check of the new average.
// ---------------------------------------------------------------------------------------------
template <class E, class R>
__device__ __forceinline__ void update_step(const View<R>& v, const int i, const StepDt& D) {
  constexpr int V = E::V, DIM = E::DIM, K = E::K, NQE = E::NQE;
  const int N = v.N;
  if (i >= N) return;
  double q[V];
#pragma unroll
  for (int c = 0; c < V; ++c) q[c] = v.Qbar[(size_t)i * V + c];
  double low = 1.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int e = at(v.eslot + (size_t)k * N, i) >> 3;
    const double th = fmin(1.0, fmin(v.cedge[(size_t)e * 2], v.cedge[(size_t)e * 2 + 1]));
    if (v.dbg_lame) v.dbg_lame[k * N + i] = th;
    low = fmin(low, th);
  }
  if (D.idle) return;  // at the end time the step changes nothing
  if (low < 1.0) {
    const RefTab<E, R>& T = TabSel<E, R>::get();
    const double s = D.s, r = D.dt / at(v.area, i);
    double qb[V];
#pragma unroll
    for (int c = 0; c < V; ++c) q[c] = qb[c] = v.Qold[(size_t)i * V + c];
    const AvgPrim<DIM> P = avg_prim<DIM>(qb, v.gamma - 1.0);
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      const int slot = at(v.eslot + (size_t)k * N, i);
      const int e = slot >> 3, side = (slot >> 2) & 1;
      const double ep = side ? -1.0 : 1.0;
      const double th = fmin(1.0, fmin(v.cedge[(size_t)e * 2], v.cedge[(size_t)e * 2 + 1]));
      R fs[NQE][V];
      edge_points<E, R>(v, e, fs);
      double W[V], F[V];
      lxw_average<E, R>(T, fs, W);
      lxf_out<E, R>(v, i, k, e, side, qb, P, s, F);
#pragma unroll
      for (int c = 0; c < V; ++c) q[c] -= r * (th * (ep * W[c]) + (1.0 - th) * F[c]);
    }
#pragma unroll
    for (int c = 0; c < V; ++c) v.Qbar[(size_t)i * V + c] = q[c];
  }
  bool finite = true;
#pragma unroll
  for (int c = 0; c < V; ++c) finite = finite && isfinite(q[c]);
  if (!finite) report(v.err, E_NONFINITE, i);
  else if (!(q[0] > 0.0) || !(pressure<DIM>(q, v.gamma) > 0.0)) report(v.err, E_POSITIVITY, i);
}

template <class E, class R>
__device__ __forceinline__ void update_item(const View<R>& v, const int i) {
  if (i >= v.N) return;
  const int mid = mesh_id<R>(v.mesh_of, i);
  Scalars& S = v.sc[mid];
  const StepDt D = stored_dt(S);
  update_step<E, R>(v, i, D);
  // The first element of each mesh ends the mesh's step: t += dt, the wave-speed maximum is reset
  // and the shock-capturing limiter becomes due.  No kernel of this step reads the fields written here
  // after this one has begun, and this one does not.
  if (!D.idle && mesh_first(v, i, mid)) {
    S.t += D.dt;
    S.steps += 1;
    S.s_bits = 0ull;
    S.shock_pending = v.shock ? 1 : 0;
  }
}

template <class E, class R>
__global__ __launch_bounds__(256) void k_update(View<R> v) {
  update_item<E, R>(v, xcd_item());
}

// ---------------------------------------------------------------------------------------------
// k_persist: n_steps whole steps of a batch of meshes in one cooperative launch.  Every workgroup
// stays resident and runs each phase of the step (the bodies of k_pre, k_elem, k_flux,
// k_update) over tiles of elements, with a grid-wide barrier where the separate
// launches have a kernel boundary; the arithmetic is that of the separate kernels, so the results
// are the same bit for bit.  The grid is a multiple of 8 workgroups: workgroup b runs on XCD b mod 8,
// and the tiles of each XCD are one contiguous range of the space-filling-curve order.
// ---------------------------------------------------------------------------------------------
template <class E, class R, int pmode>
__global__ __launch_bounds__(256, (ElemShape<E, R>::waves)) void k_persist(View<R> v, int n_steps) {
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const int bs = (int)blockDim.x, nb = (int)gridDim.x;
  const int x = (int)blockIdx.x & 7, r = (int)blockIdx.x >> 3, per = nb >> 3;
  auto tiles = [&](int n_items, auto&& body) {
    const int nt = (n_items + bs - 1) / bs;
    const int t0 = (int)((long long)nt * x / 8), t1 = (int)((long long)nt * (x + 1) / 8);
    for (int t = t0 + r; t < t1; t += per) body(t * bs + (int)threadIdx.x);
  };
  for (int step = 0; step < n_steps; ++step) {
    tiles(v.N, [&](int i) { pre_item<E, R, pmode>(v, i); });
    grid.sync();
    tiles(v.N, [&](int i) { elem_item<E, R>(v, i); });
    grid.sync();
    tiles(v.N, [&](int i) { flux_item<E, R>(v, i); });
    grid.sync();
    tiles(v.N, [&](int i) { update_item<E, R>(v, i); });
    grid.sync();
  }
}

template <class E, class R>
hipError_t launch_persistent(const View<R>& v, int bs, hipStream_t st, int n_steps) {
  if (bs != 128 && bs != 256) return hipErrorInvalidConfiguration;
  if (!v.mesh_of || n_steps < 1) return hipErrorInvalidValue;
  const void* fn = nullptr;
  switch ((v.theta_exact ? 1 : 0) + (v.s_avg ? 2 : 0)) {
    case 0: fn = reinterpret_cast<const void*>(&k_persist<E, R, 0>); break;
    case 1: fn = reinterpret_cast<const void*>(&k_persist<E, R, 3>); break;
    case 2: fn = reinterpret_cast<const void*>(&k_persist<E, R, 4>); break;
    default: fn = reinterpret_cast<const void*>(&k_persist<E, R, 5>); break;
  }
  int dev = 0, per_cu = 0;
  hipDeviceProp_t prop;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
  // the phases take turns with the workgroup's LDS
  const int lds = std::max(ElemShape<E, R>::lds, FluxShape<E, R>::lds) * bs;
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, bs, lds);
  if (e != hipSuccess) return e;
  // every workgroup must be resident for the grid barriers; a multiple of 8 for the XCD mapping
  const int nb = per_cu * prop.multiProcessorCount / 8 * 8;
  if (nb < 8) return hipErrorCooperativeLaunchTooLarge;
  View<R> vv = v;
  void* args[] = {&vv, &n_steps};
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)nb), dim3((unsigned)bs), args, lds, st);
}

// ---------------------------------------------------------------------------------------------
// k_solo: n_steps whole steps of a small mesh in one workgroup, its phases (the bodies of k_pre, k_elem,
// k_flux, k_update) between workgroup barriers.  A step of separate launches takes 4 to 5 us per launch
// whatever the mesh.  Per step, here against separate launches: 200 cells in float64 8.5 / 19.5 us (512:
// 11.9 / 21.4, 1024: 21.8 / 21.3), P3 12.8 / 23.0 (512: 19.6 / 25.1, 1024: 36.1 / 24.9), 242 triangles 28.7 /
// 42.0 us (512: 43.3 / 44.0, FP32-mixed 30.4 / 37.3); hence the limits in SoloMax,
// one for both precisions.
// The wave speed is reduced in LDS and t, dt and s stay in registers; the mesh's scalars are read once and
// written once.
// ---------------------------------------------------------------------------------------------
template <class E, class R, int pmode>
__global__ __launch_bounds__(512) void k_solo(View<R> v, int n_steps) {
  __shared__ double red[8];
  const int tid = (int)threadIdx.x, bs = (int)blockDim.x, N = v.N;
  const Scalars S = v.sc[0];
  double t = S.t;
  bool pending = S.shock_pending != 0;
  StepDt D = {S.s, S.dt, false};
  long long done = 0;
  for (int step = 0; step < n_steps; ++step) {
    if (!(t < S.T)) { D.idle = true; break; }
    double x = 0.0;
    for (int i = tid; i < N; i += bs) x = fmax(x, pre_elem<E, R, pmode>(v, i, 0, pending));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
    if ((tid & 63) == 0) red[tid >> 6] = x;
    __syncthreads();
    x = red[0];
    for (int w = 1; w < (bs >> 6); ++w) x = fmax(x, red[w]);
    D = step_dt(S, x, t);
    if (tid == 0 && (!(x > 0.0) || !isfinite(x))) report(v.err, E_NONFINITE, -1);
    for (int i = tid; i < N; i += bs) elem_step<E, R>(v, i, D);
    __syncthreads();
    for (int i = tid; i < N; i += bs) flux_step<E, R>(v, i, D);
    __syncthreads();
    for (int i = tid; i < N; i += bs) update_step<E, R>(v, i, D);
    __syncthreads();
    t += D.dt;
    pending = v.shock != 0;
    ++done;
  }
  if (tid == 0) {
    Scalars& O = v.sc[0];
    O.s = D.s;
    O.dt = D.dt;
    O.idle = D.idle;
    O.t = t;
    O.steps = S.steps + done;
    O.shock_pending = pending;
  }
}

template <class E, class R>
hipError_t launch_solo(const View<R>& v, hipStream_t st, int n_steps) {
  if constexpr (SoloMax<E>::n == 0) {
    return hipErrorInvalidValue;
  } else {
    if (v.mesh_of || v.N < 1 || v.N > SoloMax<E>::n || n_steps < 1) return hipErrorInvalidValue;
    const int bs = v.N <= 256 ? 256 : 512;
    const int lds = std::max(ElemShape<E, R>::lds, FluxShape<E, R>::lds) * bs;
    switch ((v.theta_exact ? 1 : 0) + (v.s_avg ? 2 : 0)) {
      case 0: hipLaunchKernelGGL((k_solo<E, R, 0>), dim3(1), dim3(bs), lds, st, v, n_steps); break;
      case 1: hipLaunchKernelGGL((k_solo<E, R, 3>), dim3(1), dim3(bs), lds, st, v, n_steps); break;
      case 2: hipLaunchKernelGGL((k_solo<E, R, 4>), dim3(1), dim3(bs), lds, st, v, n_steps); break;
      default: hipLaunchKernelGGL((k_solo<E, R, 5>), dim3(1), dim3(bs), lds, st, v, n_steps); break;
    }
    return hipGetLastError();
  }
}

#if LXW_PART == 0
// Sets the end time of every mesh (a kernel, so that it is ordered on the stream and may be
// captured).
__global__ void k_set_end(Scalars* sc, int n_mesh, double T) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < n_mesh) sc[m].T = T;
}

hipError_t launch_set_end(Scalars* sc, int n_mesh, double T, hipStream_t st) {
  hipLaunchKernelGGL(k_set_end, dim3((unsigned)((n_mesh + 63) / 64)), dim3(64), 0, st, sc, n_mesh, T);
  return hipGetLastError();
}
#endif

// k_final: marks the pending shock-capturing limiter as applied (after a state read-out applied
// it).
static __global__ void k_final(Scalars* sc, int n_mesh) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_mesh) return;
  sc[m].shock_pending = 0;
}

template <class E, class R>
hipError_t launch(KernelId k, const View<R>& v, const LaunchCfg& cfg, hipStream_t st, int n_mesh, int mode) {
  auto grid = [](int n, int b) { return dim3((unsigned)((n + b - 1) / b)); };
  // element and edge kernels: grid padded to a multiple of 8 blocks (XCD-contiguous block order)
  auto egrid = [](int n, int b) { return dim3((unsigned)egrid_blocks(n, b)); };
  const int bs = (k == K_SHOCK) ? cfg.bs[K_PRE] : (tunable(k) ? cfg.bs[k] : 0);
  if (tunable(k == K_SHOCK ? K_PRE : k) && bs != 64 && bs != 128 && bs != 256) return hipErrorInvalidConfiguration;
  switch (k) {
    case K_PRE:
      if (v.N > 0) {
        switch ((v.theta_exact ? 1 : 0) + (v.s_avg ? 2 : 0)) {
          case 0: hipLaunchKernelGGL((k_pre<E, R, 0>), egrid(v.N, bs), dim3(bs), 0, st, v); break;
          case 1: hipLaunchKernelGGL((k_pre<E, R, 3>), egrid(v.N, bs), dim3(bs), 0, st, v); break;
          case 2: hipLaunchKernelGGL((k_pre<E, R, 4>), egrid(v.N, bs), dim3(bs), 0, st, v); break;
          default: hipLaunchKernelGGL((k_pre<E, R, 5>), egrid(v.N, bs), dim3(bs), 0, st, v); break;
        }
      }
      break;
    case K_SHOCK:
      if (mode != 1 && mode != 2) return hipErrorInvalidValue;
      if (v.N > 0) {
        if (mode == 1) hipLaunchKernelGGL((k_pre<E, R, 1>), egrid(v.N, bs), dim3(bs), 0, st, v);
        else hipLaunchKernelGGL((k_pre<E, R, 2>), egrid(v.N, bs), dim3(bs), 0, st, v);
      }
      break;
    case K_IND:
      return hipErrorInvalidValue;  // launched through launch_indicator
    case K_DT:
      if (dt_kernel(v.N, v.mesh_of != nullptr, cfg))
        hipLaunchKernelGGL(k_dt_single, dim3(1), dim3(1024), 0, st, v.sc, v.spart, egrid_blocks(v.N, cfg.bs[K_PRE]));
      break;
    case K_ELEM:
      if (v.N > 0) hipLaunchKernelGGL((k_elem<E, R>), egrid(v.N, bs), dim3(bs), (ElemShape<E, R>::lds * bs), st, v);
      break;
    case K_FLUX:
      if (v.N > 0) hipLaunchKernelGGL((k_flux<E, R>), egrid(v.N, bs), dim3(bs), (FluxShape<E, R>::lds * bs), st, v);
      break;
    case K_UPDATE:
      if (v.N > 0) hipLaunchKernelGGL((k_update<E, R>), egrid(v.N, bs), dim3(bs), 0, st, v);
      break;
    case K_FINAL:
      if (mode != 1) return hipErrorInvalidValue;  // the step itself ends in k_update
      hipLaunchKernelGGL(k_final, grid(n_mesh, 64), dim3(64), 0, st, v.sc, n_mesh);
      break;
  }
  return hipGetLastError();
}

template hipError_t launch<EL, double>(KernelId, const View<double>&, const LaunchCfg&, hipStream_t, int, int);
template hipError_t launch<EL, float>(KernelId, const View<float>&, const LaunchCfg&, hipStream_t, int, int);
template hipError_t launch_solo<EL, double>(const View<double>&, hipStream_t, int);
template hipError_t launch_solo<EL, float>(const View<float>&, hipStream_t, int);
#if LXW_PART == 2
template hipError_t launch_persistent<EL, double>(const View<double>&, int, hipStream_t, int);
template hipError_t launch_persistent<EL, float>(const View<float>&, int, hipStream_t, int);
#endif

}  // namespace lxw
