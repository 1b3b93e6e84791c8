// Mixed-precision SD kernels (gfx950): FP64 state and SSP-RK3 accumulation,
// FP32 interpolation, fluxes and derivatives on perturbations about a
// hydrostatic background at rest (Q0 with zero momentum).
//
// Split of the residual (exact algebra; only rounding differs):
//   R(Q) = R0 + dR,  R0 = R(Q0) computed once in FP64 (stored FP32), and
//   dR = R(Q) - R(Q0) evaluated from P = Q - Q0 without cancellation:
//   * gradients are linear: grad Q = grad Q0 + grad P, each from its own
//     BR1 common values (the wall state enters in perturbation form);
//   * inviscid:  mass m'.S, momentum m'(m'.S)/rho + p'S,
//                energy (gamma E0 + E' + p')(m'.S)/rho,
//                p' = (gamma-1)(E' - |m'|^2/(2 rho));
//   * Rusanov:   1/2 (dF_L + dF_R) - 1/2 |S| [lam (P_R - P_L) + (lam - lam0) dQ0],
//                lam - lam0 formed from the small quantities |u.n| + (c - c0)
//                and the background sound-speed jump;
//   * viscous:   tau(Q) (tau0 = 0), and the diffusive energy flux as
//                kappa/R [p' (gS0.S) + p ((gS - gS0).S)] + kappa_r terms, with
//                (gS - gS0).S written through grad P and the background
//                gradients, and gS0.S (the background entropy gradient along
//                S) computed in FP64 once;
//   * source:    M(P) (linear).
// FP32 rounding therefore scales with the perturbation, and the hydrostatic
// and isentropic cancellations of the background stay in FP64.
//
// k_flux_mixed and k_lift_mixed take one element (several at orders 2 and 3)
// per block of one wave or a few; k_flux_mixed_wide and k_lift_mixed_wide
// spread an element over a block of several waves for meshes that leave most
// of the chip idle.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.hpp"
#include "sd_common.hpp"

namespace chorus {

template <int N>
using OpsF = OpsT<float, N>;

// hardware reciprocal (1 ulp): every FP32 quantity here is
// perturbation-scaled, so this rounding is of the same order as the FP32
// arithmetic itself
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// with a Newton step (half an ulp), for the density: its reciprocal carries the
// energy flux of the whole background.  On the order-4 shell of 1,536 hexes the
// state is 4.7 % nearer to the 64-bit one (8.90e-12 -> 8.49e-12 after ten
// steps); 529 -> 531 us there, nothing measurable on 331,776 hexes.
__device__ __forceinline__ float rcp_near(float x) {
    const float r = rcp(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}

// s + w f.  The line sums are chains of this in the order they are written in:
// left to the compiler, their order followed the layout of the element in LDS,
// and with it the rounding of every result.  A chain rounds its partial sums,
// so the orders are those with small ones on a smooth field: interpolation from
// the middle of the line outwards (squared partial sums of the weights, over
// the flux points of order 4: 6.1 against 7.7 along the line), the derivative
// along the line (222, other orders up to 718).  Mean distance to the FP64 path
// over shells, both integrators, the radial diffusivity and the balanced mode,
// against interpolation along the line: density, momentum and energy -0.8,
// -0.5 and -2.7 % at order 3, -1.9, -1.5 and -3.4 % at order 4, -3.1, -2.6 and
// -4.7 % at order 5, -2.3, -5.0 and -7.2 % at order 6, the same at order 2, in
// the same time.
__device__ __forceinline__ float mac(float w, float f, float s) { return __builtin_fmaf(w, f, s); }

// i-th point of a line, from its middle outwards
template <int N>
__device__ constexpr int from_middle(int i) {
    constexpr int o2[] = {0, 1}, o3[] = {1, 0, 2}, o4[] = {1, 2, 3, 0}, o5[] = {1, 3, 2, 0, 4},
                  o6[] = {3, 1, 4, 2, 5, 0};
    return N == 2 ? o2[i] : N == 3 ? o3[i] : N == 4 ? o4[i] : N == 5 ? o5[i] : o6[i];
}

// ---------------------------------------------------------------------------
// views
// ---------------------------------------------------------------------------
struct GeoF {
    const float *solgeo;   // [E][13][NP]
    const float *fluxgeo;  // [E][3][3][NFL]
    const int32_t *link;   // [E][6]
    const int32_t *info;   // [E][6]
    int64_t E;
    const float *rflux;    // [E][3][NFL] radius at the d-flux points
};

struct MixedBufs {
    const float *bg;    // [E][2][NP]    rho0, E0
    const float *dbg;   // [E][6][2][NF2] neighbour minus own background face trace (rho, E)
    const float *gS0;   // [E][3][NFL]   grad S0 . (|J| grad xi_d) at d-flux points
    const float *R0;    // [5][E][NP]    R(Q0)
    const float *gbg;   // [E][3][NP]    grad rho0 at the solution points (from FP64, once)
};

struct PhysF {
    float gm1, gam, cp, icp, cpR, GM, om, nu, kappaR, kappa_r, RT_top;  // cpR = cp/R, kappaR = kappa/R; RT_top <= 0: off
    float kappa_r1, kappa_r2;                                    // kappa_r(r) = kappa_r + kappa_r1 r + kappa_r2 r^2
};

// (on the host: converted in the kernel it took 50 vector instructions per
// wave, two FP64 divisions among them)
static PhysF physf_of(const PhysParams &P) {
    PhysF f;
    f.gm1 = (float)(P.gamma - 1.0);
    f.gam = (float)P.gamma;
    f.cp = (float)P.cp;
    f.icp = (float)(1.0 / P.cp);
    f.cpR = (float)(P.cp / P.R_gas);
    f.GM = (float)P.GM;
    f.om = (float)P.omega;
    f.nu = (float)P.nu;
    f.kappaR = (float)(P.kappa / P.R_gas);
    f.kappa_r = (float)P.kappa_r;
    f.RT_top = (P.T_top > 0.0) ? (float)(P.R_gas * P.T_top) : -1.0f;
    f.kappa_r1 = (float)P.kappa_r1;
    f.kappa_r2 = (float)P.kappa_r2;
    return f;
}

// radiative-diffusivity variants of the flux pass: none, constant, radial
enum { KR_NONE = 0, KR_CONST = 1, KR_RADIAL = 2 };

// radiative diffusivity at a flux point from the value read with its
// geometry (the radius for KR_RADIAL)
template <int KR>
__device__ __forceinline__ float kr_of(const PhysF &F, float loaded) {
    if constexpr (KR == KR_RADIAL) return F.kappa_r + loaded * (F.kappa_r1 + loaded * F.kappa_r2);
    else return F.kappa_r;
}

// LDS field slots at solution points: perturbation (5), background (2)
enum { F_RP = 0, F_MX = 1, F_MY = 2, F_MZ = 3, F_EP = 4, F_R0 = 5, F_E0 = 6, NFIELD = 7 };
// gradient slots: field f, component c at slot 3 f + c (the perturbation
// fields and rho0; grad E0 enters only along S, through the background
// entropy gradient: see dflux_viscous)
constexpr int NGRAD = 3 * (F_R0 + 1);

// point state at a flux point: background and perturbation values and
// gradients (full gradient = background + perturbation)
struct PtState {
    float r0, E0, rp, m[3], Ep;          // values
    float gr0[3];                        // background density gradient
    float grp[3], gm[3][3], gEp[3];      // perturbation gradients
};

// ---------------------------------------------------------------------------
// pointwise perturbation physics
// ---------------------------------------------------------------------------
__device__ __forceinline__ void dflux_inviscid(const PtState &s, const float S[3], const PhysF &F, float out[5]) {
    const float rho = s.r0 + s.rp, E = s.E0 + s.Ep;
    const float inv = rcp_near(rho);
    const float mS = s.m[0] * S[0] + s.m[1] * S[1] + s.m[2] * S[2];
    const float mm = s.m[0] * s.m[0] + s.m[1] * s.m[1] + s.m[2] * s.m[2];
    const float pp = F.gm1 * (s.Ep - 0.5f * mm * inv);
    const float uS = mS * inv;
    out[0] = mS;
    out[1] = s.m[0] * uS + pp * S[0];
    out[2] = s.m[1] * uS + pp * S[1];
    out[3] = s.m[2] * uS + pp * S[2];
    out[4] = (F.gam * E - F.gm1 * s.Ep + pp) * uS;
}

// (F_v(Q) - F_v(Q0)) . S given gS0S = grad S0 . S.  outer_wall / inner_wall
// select the wall forms (normal traction only; energy as interior at the
// outer wall, none at the inner wall where the prescribed flux is in R0).
// (kr: the radiative diffusivity at the point, used unless KR == KR_NONE)
template <int KR>
__device__ __forceinline__ void dflux_viscous(const PtState &s, const float S[3], float gS0S, const PhysF &F,
                                              float kr, int wall, float out[5]) {
    // with mu = rho nu and du_a/dx_c = (dm_a/dx_c - u_a drho/dx_c) / rho, the
    // stress along S needs the momentum gradient only through its
    // contractions with S: Y_a = sum_c dm_a/dx_c S_c (also in grad p' . S)
    // and Z_a = sum_b dm_b/dx_a S_b
    const float rho = s.r0 + s.rp, inv = rcp_near(rho);
    const float u[3] = {s.m[0] * inv, s.m[1] * inv, s.m[2] * inv};
    float grho[3];
    for (int c = 0; c < 3; ++c) grho[c] = s.gr0[c] + s.grp[c];
    const float gr0S = s.gr0[0] * S[0] + s.gr0[1] * S[1] + s.gr0[2] * S[2];
    const float grpS = s.grp[0] * S[0] + s.grp[1] * S[1] + s.grp[2] * S[2];
    const float grhoS = gr0S + grpS;
    const float uS = (s.m[0] * S[0] + s.m[1] * S[1] + s.m[2] * S[2]) * inv;
    const float ug = u[0] * grho[0] + u[1] * grho[1] + u[2] * grho[2];
    float Y[3];
    for (int a = 0; a < 3; ++a) Y[a] = s.gm[a][0] * S[0] + s.gm[a][1] * S[1] + s.gm[a][2] * S[2];
    // (2/3) rho div u
    const float dv = (2.0f / 3.0f) * (s.gm[0][0] + s.gm[1][1] + s.gm[2][2] - ug);
    float tS[3];
    if (wall == 0) {
        for (int a = 0; a < 3; ++a) {
            const float Za = s.gm[0][a] * S[0] + s.gm[1][a] * S[1] + s.gm[2][a] * S[2];
            tS[a] = F.nu * (Y[a] + Za - u[a] * grhoS - uS * grho[a] - dv * S[a]);
        }
    } else {
        // normal traction: n . tau . n = mu (2 S.grad u.S / |S|^2 - 2/3 div u)
        const float A2 = S[0] * S[0] + S[1] * S[1] + S[2] * S[2];
        const float SY = S[0] * Y[0] + S[1] * Y[1] + S[2] * Y[2];
        const float tnn = F.nu * (2.0f * (SY - uS * grhoS) * rcp(A2) - dv);
        for (int a = 0; a < 3; ++a) tS[a] = tnn * S[a];
    }
    out[0] = 0.0f;
    out[1] = tS[0];
    out[2] = tS[1];
    out[3] = tS[2];
    if (wall == 1) {  // inner wall: stress free, no viscous work, energy flux in R0
        out[4] = 0.0f;
        return;
    }
    // p' and grad p' . S (m0 = 0, u0 = 0)
    const float mm = s.m[0] * s.m[0] + s.m[1] * s.m[1] + s.m[2] * s.m[2], ke = 0.5f * mm * inv;
    const float pp = F.gm1 * (s.Ep - ke);
    const float p0 = F.gm1 * s.E0, p = p0 + pp;
    const float gEpS = s.gEp[0] * S[0] + s.gEp[1] * S[1] + s.gEp[2] * S[2];
    const float gpS = F.gm1 * (gEpS - (u[0] * Y[0] + u[1] * Y[1] + u[2] * Y[2]) + ke * inv * grhoS);
    // (grad S - grad S0).S / c_p with grad p0 . S / p0 = gamma (gS0S / c_p
    // + grad rho0 . S / rho0), the background entropy gradient's definition
    const float igp = rcp(F.gam * p), ir0 = rcp(s.r0);
    const float dgS = igp * (gpS - F.gam * pp * (gS0S * F.icp + gr0S * ir0)) - inv * (grpS - gr0S * s.rp * ir0);
    // rho T grad S . S - rho0 T0 grad S0 . S = (p' gS0S + p c_p dgS) / R
    const float eS = F.kappaR * (pp * gS0S + p * F.cp * dgS);
    // rho c_p grad T . S difference: c_p/R (grad p' . S - [p grad rho' . S / rho + grad rho0 . S (p/rho - p0/rho0)])
    float eT = 0.0f;
    if constexpr (KR != KR_NONE) {
        const float dpr = (pp * s.r0 - p0 * s.rp) * inv * ir0;
        eT = kr * F.cpR * (gpS - (p * grpS * inv + gr0S * dpr));
    }
    const float work = (wall == 0) ? (u[0] * tS[0] + u[1] * tS[1] + u[2] * tS[2]) : 0.0f;
    out[4] = work + eS + eT;
}

// ---------------------------------------------------------------------------
// element phases (generic N; items per thread fixed at compile time)
// ---------------------------------------------------------------------------
// The element of the flux passes: the 7 field values (slots F_*), the
// gradients (slot GR + 3 f + c) and the remainders (the other slots and plo34)
// of a point in one record of 28 floats (REC), read in quads (16 consecutive
// points lie on distinct banks), or a plane per slot.  ND: directions whose
// fluxes are held together.
// k_flux_mixed takes records but at order 4, where memory bounds the pass and
// the quads cost registers.  us per RK3 step, planes -> records (hexes of the
// mesh): N = 3 (98,304) 1,080 -> 1,076; N = 4 (41,472) 802 -> 829; N = 5
// (24,000) 1,070 -> 1,002; N = 6 (12,288) 954 -> 850 (with the radial
// diffusivity 995 -> 974).  k_flux_mixed_wide, whose threads each take one
// field between the flux points, takes planes but at order 2: N = 2 (288) 27.6
// -> 27.3; N = 3 (1,536) 44.3 -> 47.3; N = 4 (648) 40.2 -> 41.4; N = 5 (288)
// 46.3 -> 48.1; N = 6 (162) 43.0 -> 47.4.
template <int N, int ND, bool REC>
struct MixedEl {
    static constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N, GR = 8, SLOTS = 28;
    static_assert(GR + NGRAD + 2 == SLOTS, "slots of a point");
    alignas(16) float r[NP * SLOTS];
    float plo34[2][NP];           // remainders of F_MZ, F_EP
    union {
        float cs[5][6][NF2];       // common values of the perturbation
        float ft[ND][5][NFL];      // transformed fluxes, written after cs is consumed
    } u;
    __device__ __forceinline__ float &at(int slot, int p) { return r[REC ? p * SLOTS + slot : slot * NP + p]; }
    // FP64 perturbation minus its FP32 value (stage update)
    __device__ __forceinline__ float &plo(int v, int p) {
        return v == 0 ? at(NFIELD, p) : v < 3 ? at(GR + NGRAD + v - 1, p) : plo34[v - 3][p];
    }
    // x[i] += w slot 4 j + i of point p
    __device__ __forceinline__ void add_quad(float w, int p, int j, float x[4]) const {
        if constexpr (REC) {
            const float4 t = *reinterpret_cast<const float4 *>(&r[p * SLOTS + 4 * j]);
            x[0] = mac(w, t.x, x[0]);
            x[1] = mac(w, t.y, x[1]);
            x[2] = mac(w, t.z, x[2]);
            x[3] = mac(w, t.w, x[3]);
        } else {
            for (int i = 0; i < 4; ++i) x[i] = mac(w, r[(4 * j + i) * NP + p], x[i]);
        }
    }
    // quads J0..J1-1 at flux point m of the line (base, st)
    template <int J0, int J1>
    __device__ __forceinline__ void line(const OpsF<N> &op, int m, int base, int st, float *x) const {
#pragma unroll
        for (int i = 0; i < 4 * (J1 - J0); ++i) x[i] = 0.0f;
#pragma unroll
        for (int j = J0; j < J1; ++j)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int b = from_middle<N>(i);
                add_quad(op.I[m][b], base + b * st, j, x + 4 * (j - J0));
            }
    }
};

template <int N>
using MixedElem = MixedEl<N, 1, N != 4>;  // of k_flux_mixed

template <int N, int EPB, int NT>
struct Shape {
    static constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N;
    static constexpr int IT_SOL = (EPB * NP + NT - 1) / NT;
    static constexpr int IT_FACE = (EPB * 6 * NF2 + NT - 1) / NT;
    static constexpr int IT_FLUX = (EPB * 3 * NFL + NT - 1) / NT;
    static constexpr int NINTD = (N - 1) * N * N;     // interior flux points per element and direction
    static constexpr int IT_INTD = (EPB * NINTD + NT - 1) / NT;
    static constexpr int MB = 6 * 5 * NF2;             // mailbox floats per element
    static constexpr int DB = 6 * 2 * NF2;
};

// registers holding one thread's share of an element block's global inputs;
// everything is issued before the first use so that a block waits for
// memory once.  Items past the last element (or past the block's item
// count) load element 0's data through a clamped index: no load is
// predicated (a guarded load compiles to a branch that waits for it at
// once) and those items are never stored.
//
// Most addresses are a block-uniform base (scalar registers) plus a 32-bit
// lane offset in bytes plus a constant: one vector register serves all the
// loads of an array, where 64-bit lane addresses took a vector add each.
// The pass issues vector instructions for most of its time at order 4; with
// this, the physics constants converted on the host and the viscous flux's
// kinetic terms in the form of the inviscid ones it has 5 % fewer (2,401 ->
// 2,273): 6.21 -> 6.14 ms per RK3 step on 331,776 hexes.
template <typename T>
__device__ __forceinline__ T ld_at(const T *base, uint32_t bytes, int c = 0) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + bytes + c * (int)sizeof(T));
}
// whether item it = threadIdx.x + k NT lies past the TOTAL items of the block
// (known to be false for the rounds that are full: a guard there is a branch
// under which the compiler moves the loads of its body)
template <int NT, int TOTAL>
__device__ __forceinline__ bool past(int k, int it) {
    return (k + 1) * NT > TOTAL && it >= TOTAL;
}
// element of item it (of n per element) within the block, clamped to the last
// element (elmax)
template <int EPB>
__device__ __forceinline__ uint32_t el_of(int it, int n, int elmax) {
    return EPB == 1 ? 0 : min(it / n, elmax);
}

template <int N, int EPB, int NT>
struct Prologue {
    using Sh = Shape<N, EPB, NT>;
    double P[Sh::IT_SOL][5];
    float bg[Sh::IT_SOL][2];
    float gs[Sh::IT_SOL][9];
    float gb[Sh::IT_SOL][3];  // background density gradient
    // neighbour data at this thread's face items (face item it: el, f, pp):
    // perturbation trace, background jump
    float nq[Sh::IT_FACE][5], db[Sh::IT_FACE][2];
};

template <int N, int EPB, int NT>
__device__ __forceinline__ void prologue_load(const double *Pq, const MixedBufs &B, const GeoF &G,
                                              const float *__restrict__ TQ, int64_t e0, int elmax,
                                              Prologue<N, EPB, NT> &R) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NP = Sh::NP, NF2 = Sh::NF2;
    const int64_t E = G.E;
    // issued in the order of first use, so that each phase waits only for
    // its own inputs: the LDS fields, the neighbour traces (common values)
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const uint32_t el = el_of<EPB>(it, NP, elmax), p = it % NP;
        for (int v = 0; v < 5; ++v) R.P[k][v] = ld_at(Pq + (v * E + e0) * NP, 8 * (el * NP + p));
        for (int t = 0; t < 2; ++t) R.bg[k][t] = ld_at(B.bg + e0 * 2 * NP, 4 * (el * 2 * NP + p), t * NP);
        for (int t = 0; t < 3; ++t) R.gb[k][t] = ld_at(B.gbg + e0 * 3 * NP, 4 * (el * 3 * NP + p), t * NP);
    }
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        const uint32_t el = el_of<EPB>(it, 6 * NF2, elmax), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const uint32_t ef = el * 6 + f;
        for (int v = 0; v < 5; ++v) R.nq[k][v] = ld_at(TQ + e0 * Sh::MB, 4 * (ef * 5 * NF2 + pp), v * NF2);
        for (int t = 0; t < 2; ++t) R.db[k][t] = ld_at(B.dbg + e0 * Sh::DB, 4 * (ef * 2 * NF2 + pp), t * NF2);
    }
}

// the solution-point metrics (first used by the gradients)
template <int N, int EPB, int NT>
__device__ __forceinline__ void prologue_load_metrics(const GeoF &G, int64_t e0, int elmax, Prologue<N, EPB, NT> &R) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NP = Sh::NP;
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const uint32_t el = el_of<EPB>(it, NP, elmax), p = it % NP;
        for (int t = 0; t < 9; ++t) R.gs[k][t] = ld_at(G.solgeo + e0 * 13 * NP, 4 * (el * 13 * NP + p), t * NP);
    }
}

// move the prologue registers into the element LDS
template <int N, int EPB, int NT>
__device__ __forceinline__ void prologue_store(const Prologue<N, EPB, NT> &R, MixedElem<N> *L) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NP = Sh::NP;
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (past<NT, EPB * NP>(k, it)) break;
        const int el = it / NP, p = it % NP;
        for (int v = 0; v < 5; ++v) {
            const float hi = (float)R.P[k][v];
            L[el].at(v, p) = hi;
            L[el].plo(v, p) = (float)(R.P[k][v] - (double)hi);
        }
        L[el].at(F_R0, p) = R.bg[k][0];
        L[el].at(F_E0, p) = R.bg[k][1];
        for (int c = 0; c < 3; ++c) L[el].at(MixedElem<N>::GR + 3 * F_R0 + c, p) = R.gb[k][c];
    }
}

// interpolation of a field stored in LDS at flux point m of the line
// (base, st)
template <int N>
__device__ __forceinline__ float line_val(const OpsF<N> &op, const float *fld, int m, int base, int st) {
    float s = 0.0f;
#pragma unroll
    for (int b = 0; b < N; ++b) s += op.I[m][b] * fld[base + b * st];
    return s;
}

// BR1 common value of the perturbation at a face point with the own values pv
// and background density r0: average with the neighbour trace nq, or the
// wall state in perturbation form (rho' kept, normal momentum removed,
// pressure kept; outer wall with T_top: p = rho R T_top).  The normal
// projection is the same along +-S.  put(v, value) stores variable v.
template <typename PUT>
__device__ __forceinline__ void common_value(const float pv[5], float r0, int32_t nb, int32_t inf, const float nq[5],
                                             const float S[3], const PhysF &F, PUT &&put) {
    if (nb >= 0) {
        for (int v = 0; v < 5; ++v) put(v, 0.5f * (pv[v] + nq[v]));
        return;
    }
    const bool outer = ((inf >> 6) - 1) == CHORUS_BC_OUTER;
    const float A2 = S[0] * S[0] + S[1] * S[1] + S[2] * S[2];
    const float mn = (pv[1] * S[0] + pv[2] * S[1] + pv[3] * S[2]) * rcp(A2);
    float mb[3];
    for (int a = 0; a < 3; ++a) mb[a] = pv[1 + a] - mn * S[a];
    const float irho = rcp(r0 + pv[0]), igm1 = rcp(F.gm1);
    const float mm = pv[1] * pv[1] + pv[2] * pv[2] + pv[3] * pv[3];
    const float mbb = mb[0] * mb[0] + mb[1] * mb[1] + mb[2] * mb[2];
    float Eb;  // E_b - E0_b
    if (outer && F.RT_top > 0.0f) Eb = F.RT_top * pv[0] * igm1 + 0.5f * mbb * irho;
    else Eb = pv[4] + 0.5f * (mbb - mm) * irho;
    put(0, pv[0]);
    for (int a = 0; a < 3; ++a) put(1 + a, mb[a]);
    put(4, Eb);
}

// BR1 common values of the perturbation at the 6 N^2 face points (the
// background's gradients are computed once, in FP64, at set-up); the own
// face values of the 7 fields at the thread's face items are kept in fo when
// given: the face-flux phase reuses them
template <int N, int EPB, int NT>
__device__ __forceinline__ void common_values(const OpsF<N> &op, const GeoF &G, const PhysF &F, int64_t e0,
                                              MixedElem<N> *L, const int32_t (*lk)[6], const int32_t (*inf_)[6],
                                              const Prologue<N, EPB, NT> &R,
                                              float (*fo)[NFIELD], const float (*Sf)[3]) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NF2 = N * N, NFL = (N + 1) * N * N;
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * 6 * NF2) break;
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        MixedElem<N> &l = L[el];
        const int t1 = pp % N, t2 = pp / N;
        const int d = f >> 1, m = (f & 1) ? N : 0, base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d);
        float x[8];
        l.template line<0, 2>(op, m, base, st, x);
        for (int v = 0; v < NFIELD; ++v) fo[k][v] = x[v];
        const int32_t nb = lk[el][f], inf = inf_[el][f];
        common_value(x, x[F_R0], nb, inf, R.nq[k], Sf[k], F, [&](int v, float x) { l.u.cs[v][f][pp] = x; });
    }
}

// gradients of the 5 perturbation fields at the solution points (those of
// the background are loaded)
template <int N, int EPB, int NT>
__device__ __forceinline__ void gradients(const OpsF<N> &op, const GeoF &G, int64_t e0, MixedElem<N> *L,
                                          const float (*gsol)[9]) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NP = N * N * N;
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        MixedElem<N> &l = L[el];
        const float *Gm = gsol[k];
        float dq[3][5];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d), pp = t1 + N * t2;
#pragma unroll
            for (int v = 0; v < 5; ++v)
                dq[d][v] = mac(op.D[a][N], l.u.cs[v][2 * d + 1][pp], op.D[a][0] * l.u.cs[v][2 * d][pp]);
#pragma unroll
            for (int b = 0; b < N; ++b) {
                l.add_quad(op.B[a][b], base + b * st, 0, dq[d]);
                dq[d][4] = mac(op.B[a][b], l.at(F_EP, base + b * st), dq[d][4]);
            }
        }
#pragma unroll
        for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                l.at(MixedElem<N>::GR + 3 * v + c, p) = Gm[c] * dq[0][v] + Gm[3 + c] * dq[1][v] + Gm[6 + c] * dq[2][v];
    }
}

// point state at the flux point m of the line (base, st); with vals given,
// the 7 field values are taken from there and only the gradients are
// interpolated
template <int N, typename EL>
__device__ __forceinline__ void state_at(const OpsF<N> &op, const EL &l, int m, int base, int st, PtState &s,
                                         const float *vals = nullptr) {
    constexpr int NG = EL::SLOTS / 4 - 2;
    float v[8], g[4 * NG];
    if (!vals) l.template line<0, 2>(op, m, base, st, v);
    const float *x = vals ? vals : v;
    s.rp = x[F_RP];
    s.m[0] = x[F_MX];
    s.m[1] = x[F_MY];
    s.m[2] = x[F_MZ];
    s.Ep = x[F_EP];
    s.r0 = x[F_R0];
    s.E0 = x[F_E0];
    l.template line<2, 2 + NG>(op, m, base, st, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        s.grp[c] = g[3 * F_RP + c];
        s.gm[0][c] = g[3 * F_MX + c];
        s.gm[1][c] = g[3 * F_MY + c];
        s.gm[2][c] = g[3 * F_MZ + c];
        s.gEp[c] = g[3 * F_EP + c];
        s.gr0[c] = g[3 * F_R0 + c];
    }
}

// Own-side part of the common transformed flux difference at a face point,
// along the outward area vector So.  Interior face: the Rusanov flux of the
// own state s and the neighbour state (perturbation trace nq, background
// jump db) minus half of the own viscous flux fv (the neighbour's half is
// added by the lift pass from the neighbour's viscous trace).  Wall
// face: the complete wall flux (inviscid (0, p' So, 0); viscous wall form).
template <int KR>
__device__ __forceinline__ void face_flux_own(const PtState &s, const float nq[5], const float db[2], bool interior,
                                              bool outer, const float So[3], float gS0S, float kr,
                                              const float fv_in[5], const PhysF &F, float phi[5]) {
    if (interior) {
        PtState r = s;
        r.rp = nq[0];
        r.m[0] = nq[1];
        r.m[1] = nq[2];
        r.m[2] = nq[3];
        r.Ep = nq[4];
        const float dr0 = db[0], dE0 = db[1];
        r.r0 = s.r0 + dr0;
        r.E0 = s.E0 + dE0;
        float fL[5], fR[5];
        dflux_inviscid(s, So, F, fL);
        dflux_inviscid(r, So, F, fR);
        const float A = sqrtf(So[0] * So[0] + So[1] * So[1] + So[2] * So[2]), iA = rcp(A);
        // |u.n| + (c - c0) on each side; c^2 - c0^2 = gamma (p' rho0 - p0 rho') / (rho rho0)
        auto excess = [&](const PtState &q, float &c0) {
            const float inv = rcp(q.r0 + q.rp), ir0 = rcp(q.r0);
            const float un = fabsf((q.m[0] * So[0] + q.m[1] * So[1] + q.m[2] * So[2]) * iA * inv);
            const float mm = q.m[0] * q.m[0] + q.m[1] * q.m[1] + q.m[2] * q.m[2];
            const float pp_ = F.gm1 * (q.Ep - 0.5f * mm * inv), p0 = F.gm1 * q.E0;
            c0 = sqrtf(F.gam * p0 * ir0);
            const float dc2 = F.gam * (pp_ * q.r0 - p0 * q.rp) * inv * ir0;
            const float c = sqrtf(c0 * c0 + dc2);
            return un + dc2 * rcp(c + c0);
        };
        float c0L, c0R;
        const float eL = excess(s, c0L), eR = excess(r, c0R);
        // background sound-speed jump c0R - c0L from the FP64 background jump
        const float dc0 = F.gam * F.gm1 * (dE0 * s.r0 - s.E0 * dr0) * rcp(s.r0 * r.r0 * (c0L + c0R));
        const float dlam = fmaxf(eL, eR + dc0) - fmaxf(0.0f, dc0);
        const float lam0 = c0L + fmaxf(0.0f, dc0);
        const float hl = 0.5f * (lam0 + dlam) * A, hd = 0.5f * dlam * A;
        const float pR[5] = {r.rp, r.m[0], r.m[1], r.m[2], r.Ep};
        const float pL[5] = {s.rp, s.m[0], s.m[1], s.m[2], s.Ep};
        const float dq0[5] = {dr0, 0.0f, 0.0f, 0.0f, dE0};
        for (int v = 0; v < 5; ++v)
            phi[v] = 0.5f * (fL[v] + fR[v]) - hl * (pR[v] - pL[v]) - hd * dq0[v] - 0.5f * fv_in[v];
    } else {
        const float mm = s.m[0] * s.m[0] + s.m[1] * s.m[1] + s.m[2] * s.m[2];
        const float pp = F.gm1 * (s.Ep - 0.5f * mm * rcp(s.r0 + s.rp));
        float fv[5];
        dflux_viscous<KR>(s, So, gS0S, F, kr, outer ? 2 : 1, fv);
        phi[0] = 0.0f;
        for (int a = 0; a < 3; ++a) phi[1 + a] = pp * So[a] - fv[1 + a];
        phi[4] = -fv[4];
    }
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// P = Q - Q0 (FP64) and the FP32 face traces of P
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_pert_begin(OpsF<N> opa, GeoF G, const double *__restrict__ Q,
                                                   const double *__restrict__ Q0, double *__restrict__ Pq,
                                                   float *__restrict__ TQ) {
    constexpr int NP = N * N * N, NF2 = N * N;
    __shared__ float sp[EPB][5][NP];
    __shared__ OpsF<N> op;
    __shared__ int32_t lk[EPB][6], inf[EPB][6];
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    BlockTables<EPB, NT, float, N> bt;
    bt.load(opa, G.link, G.info, e0, G.E);
    for (int it = threadIdx.x; it < EPB * 5 * NP; it += NT) {
        const int el = it / (5 * NP), r = it % (5 * NP), v = r / NP, p = r % NP;
        const int64_t e = e0 + el;
        float val = 0.0f;
        if (e < G.E) {
            const int64_t gi = ((int64_t)v * G.E + e) * NP + p;
            const double d = Q[gi] - Q0[gi];
            Pq[gi] = d;
            val = (float)d;
        }
        sp[el][v][p] = val;
    }
    bt.store(op, &lk[0][0], &inf[0][0]);
    __syncthreads();
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        const int32_t nb = lk[el][f];
        if (nb < 0) continue;
        const int64_t slot = mailbox_slot<N>(nb, inf[el][f], pp);
        const int d = f >> 1, m = (f & 1) ? N : 0, base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
        for (int v = 0; v < 5; ++v) TQ[slot + v * NF2] = line_val<N>(op, sp[el][v], m, base, st);
    }
}

// stage combination on P (see MixedStageArgs); mode 0 writes R0 + dR
using MixedStage = MixedStageArgs;

// ---------------------------------------------------------------------------
// flux pass + lift pass (the stage split used by the solver)
// ---------------------------------------------------------------------------
// Flux pass: every step that needs the gradients, once per stage.  Common
// values and gradients; at the face points the own viscous flux (pushed to
// the neighbour's viscous mailbox TV) and the own-side common flux (Rusanov
// minus half the own viscous flux, or the wall flux); at the interior flux
// points the transformed flux; the divergence of the flux polynomials with
// the own-side face fluxes at the line ends; the source.  The partial
// residual Rp = R0 - div/|J| - M, which lacks only the neighbours' viscous
// halves at interior interfaces, enters the stage combination here (FP64):
// Pout = c0 A + c1 (P + c2 Rp) (and Tout likewise), or Pout = Rp in
// residual mode; the lift pass adds the missing part in place.
template <int N, int EPB, int NT, int MINW, int KR>
__global__ __launch_bounds__(NT, N == 6 && KR == KR_RADIAL ? 3 : MINW)
void k_flux_mixed(OpsF<N> opa, GeoF G, MixedBufs B, PhysF F, const double *__restrict__ Pq,
                  const float *__restrict__ TQ, float *__restrict__ TV, MixedStage S_) {
    using Sh = Shape<N, EPB, NT>;
    constexpr int NP = Sh::NP, NF2 = Sh::NF2, NFL = Sh::NFL, NINTD = Sh::NINTD;
    __shared__ MixedElem<N> L[EPB];
    __shared__ OpsF<N> op;  // 1D operators (indexed per lane: LDS, not the argument segment)
    __shared__ int32_t lk[EPB][6], inf_[EPB][6];  // neighbour element and info word per face
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    BlockTables<EPB, NT, float, N> bt;
    bt.load(opa, G.link, G.info, e0, G.E);
    // every global input of the element block, issued before the first wait
    // (unpredicated, clamped indices: see Prologue), in the order of first use
    Prologue<N, EPB, NT> R;
    const int elmax = (G.E - 1 - e0 < EPB - 1) ? (int)(G.E - 1 - e0) : EPB - 1;
    prologue_load<N, EPB, NT>(Pq, B, G, TQ, e0, elmax, R);
    const float *fgb = G.fluxgeo + e0 * 9 * NFL, *gsb = B.gS0 + e0 * 3 * NFL, *rfb = G.rflux + e0 * 3 * NFL;
    float Sf[Sh::IT_FACE][3], gSf[Sh::IT_FACE], krf[Sh::IT_FACE];
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        const uint32_t el = el_of<EPB>(it, 6 * NF2, elmax), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const uint32_t d = f >> 1, fl = ((f & 1) ? N : 0) + (N + 1) * pp, o = 4 * ((el * 3 + d) * NFL + fl);
        // along +xi_d here; the face phase turns them outward
        for (int c = 0; c < 3; ++c) Sf[k][c] = ld_at(fgb, 4 * ((el * 3 + d) * 3 * NFL + fl), c * NFL);
        gSf[k] = ld_at(gsb, o);
        krf[k] = (KR == KR_RADIAL) ? ld_at(rfb, o) : 0.0f;
    }
    prologue_load_metrics<N, EPB, NT>(G, e0, elmax, R);
    float Si[3][Sh::IT_INTD][3], gSi[3][Sh::IT_INTD], kri[3][Sh::IT_INTD];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int k = 0; k < Sh::IT_INTD; ++k) {
            const int it = threadIdx.x + k * NT;
            const uint32_t el = el_of<EPB>(it, NINTD, elmax), q = it % NINTD;
            const uint32_t fl = 1 + q % (N - 1) + (N + 1) * (q / (N - 1)), o = 4 * (el * 3 * NFL + fl);
            for (int c = 0; c < 3; ++c) Si[d][k][c] = ld_at(fgb, 4 * (el * 9 * NFL + fl), (d * 3 + c) * NFL);
            gSi[d][k] = ld_at(gsb, o, d * NFL);
            kri[d][k] = (KR == KR_RADIAL) ? ld_at(rfb, o, d * NFL) : 0.0f;
        }
    bt.store(op, &lk[0][0], &inf_[0][0]);
    prologue_store<N, EPB, NT>(R, L);
    __syncthreads();
    float fo[Sh::IT_FACE][NFIELD];
    common_values<N, EPB, NT>(op, G, F, e0, L, lk, inf_, R, fo, Sf);
    __syncthreads();
    gradients<N, EPB, NT>(op, G, e0, L, R.gs);
    __syncthreads();
    // face points: own viscous flux to the neighbour, own-side common flux
    // kept in registers for the divergence
    float ffc[Sh::IT_FACE][5];
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        for (int v = 0; v < 5; ++v) ffc[k][v] = 0.0f;
        if (it >= EPB * 6 * NF2) break;
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        const int32_t nb = lk[el][f], inf = inf_[el][f];
        const int d = f >> 1, m = (f & 1) ? N : 0, t1 = pp % N, t2 = pp / N;
        const float sg = (f & 1) ? 1.0f : -1.0f;
        const float So[3] = {sg * Sf[k][0], sg * Sf[k][1], sg * Sf[k][2]}, gSo = sg * gSf[k];
        float fv[5];
        PtState st;
        state_at<N>(op, L[el], m, sol_of<N>(d, 0, t1, t2), stride_of<N>(d), st, fo[k]);
        const float kr = kr_of<KR>(F, krf[k]);
        if (nb >= 0) {
            dflux_viscous<KR>(st, So, gSo, F, kr, 0, fv);
            // the viscous mass flux is zero: four components per point
            const int64_t slot = mailbox_slot<N, 4>(nb, inf, pp);
            for (int v = 1; v < 5; ++v) st_once(&TV[slot + (v - 1) * NF2], fv[v]);
        }
        face_flux_own<KR>(st, R.nq[k], R.db[k], nb >= 0, ((inf >> 6) - 1) == CHORUS_BC_OUTER, So, gSo, kr, fv,
                          F, ffc[k]);
    }
    // per direction d: transformed flux at the d-flux points, then its
    // derivative added to the divergence at the solution points
    float div[Sh::IT_SOL][5];
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k)
        for (int v = 0; v < 5; ++v) div[k][v] = 0.0f;
    // operands of the source and the stage combination, loaded before the
    // last divergence so that it covers their latency (every one before the
    // first store: the outputs may alias the inputs, and a load issued after
    // a store would wait for it); block-uniform bases, per-lane offsets
    // clamped to the last element
    float r0v[Sh::IT_SOL][5], gq[Sh::IT_SOL][4];
    double pst[Sh::IT_SOL][5], pb[Sh::IT_SOL][5];
    const bool rk = S_.mode != 0;
    const bool useA = rk && S_.c0 != 0.0, useT = rk && S_.Tout != nullptr, useB = useT && S_.d0 != 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int k = 0; k < Sh::IT_INTD; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * NINTD) break;
            const int el = it / NINTD, q = it % NINTD;
            const int m = 1 + q % (N - 1), tt = q / (N - 1), t1 = tt % N, t2 = tt / N;
            if (e0 + el >= G.E) continue;
            MixedElem<N> &l = L[el];
            PtState s;
            state_at<N>(op, l, m, sol_of<N>(d, 0, t1, t2), stride_of<N>(d), s);
            float fi[5], fv[5];
            dflux_inviscid(s, Si[d][k], F, fi);
            dflux_viscous<KR>(s, Si[d][k], gSi[d][k], F, kr_of<KR>(F, kri[d][k]), 0, fv);
            const int fl = m + (N + 1) * tt;
            for (int v = 0; v < 5; ++v) l.u.ft[0][v][fl] = fi[v] - fv[v];
        }
#pragma unroll
        for (int k = 0; k < Sh::IT_FACE; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * 6 * NF2) break;
            const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
            if ((f >> 1) != d || e0 + el >= G.E) continue;
            MixedElem<N> &l = L[el];
            const int m = (f & 1) ? N : 0;
            const float sg = (f & 1) ? 1.0f : -1.0f;
            const int fl = m + (N + 1) * pp;
            for (int v = 0; v < 5; ++v) l.u.ft[0][v][fl] = sg * ffc[k][v];
        }
        __syncthreads();
        if (d == 2) {
            const float *sgb = G.solgeo + e0 * 13 * NP;
#pragma unroll
            for (int k = 0; k < Sh::IT_SOL; ++k) {
                const int it = threadIdx.x + k * NT;
                const uint32_t el = el_of<EPB>(it, NP, elmax), p = it % NP, o = el * NP + p;
                for (int c = 0; c < 4; ++c) gq[k][c] = ld_at(sgb, 4 * (el * 13 * NP + p), (9 + c) * NP);
                for (int v = 0; v < 5; ++v) {
                    const int64_t vb = ((int64_t)v * G.E + e0) * NP;
                    r0v[k][v] = ld_off(B.R0 + vb, o);
                    pst[k][v] = useA ? ld_off(S_.A + vb, o) : 0.0;
                    pb[k][v] = useB ? ld_off(S_.B + vb, o) : 0.0;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < Sh::IT_SOL; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * NP) break;
            const int el = it / NP, p = it % NP;
            if (e0 + el >= G.E) continue;
            const MixedElem<N> &l = L[el];
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int fb = (N + 1) * (t1 + N * t2);
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                float sum = 0.0f;
#pragma unroll
                for (int mm = 0; mm <= N; ++mm) sum = mac(op.D[a][mm], l.u.ft[0][v][fb + mm], sum);
                div[k][v] += sum;
            }
        }
        __syncthreads();
    }
    // source, background residual and stage combination (operands loaded
    // during the last direction's divergence)
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        if (el > elmax) continue;
        MixedElem<N> &l = L[el];
        const float iJ = gq[k][0];
        const float g0 = F.GM * gq[k][1], g1 = F.GM * gq[k][2], g2 = F.GM * gq[k][3];
        const float rp = l.at(F_RP, p), mx = l.at(F_MX, p), my = l.at(F_MY, p), mz = l.at(F_MZ, p);
        float M[5];
        M[0] = 0.0f;
        M[1] = rp * g0 - 2.0f * F.om * my;
        M[2] = rp * g1 + 2.0f * F.om * mx;
        M[3] = rp * g2;
        M[4] = mx * g0 + my * g1 + mz * g2;
        const uint32_t o = (uint32_t)(el * NP + p);
        for (int v = 0; v < 5; ++v) {
            const int64_t vb = ((int64_t)v * G.E + e0) * NP;
            const double Rv = (double)r0v[k][v] + (double)(-div[k][v] * iJ - M[v]);
            if (!rk) {
                st_off(S_.Pout + vb, o, Rv);
                continue;
            }
            // the stage input from its FP32 value and FP32 remainder (48
            // significant bits: 2^-48 relative, far below the FP32 residual)
            const double pin = (double)l.at(v, p) + (double)l.plo(v, p);
            if (useT) st_off(S_.Tout + vb, o, S_.d0 * pb[k][v] + S_.d1 * (pin + S_.d2 * Rv));
            st_off(S_.Pout + vb, o, S_.c0 * pst[k][v] + S_.c1 * (pin + S_.c2 * Rv));
        }
    }
}

// Q = Q0 + P, P rounded before the sum (as if it had been stored) whatever
// the file's floating-point rules
__device__ __forceinline__ double state_of(double q0, double p) {
#pragma clang fp reassociate(off) contract(off)
    return q0 + p;
}

// Lift pass: the neighbours' viscous halves at the interior interface
// points enter the divergence through the end columns of the derivative
// matrix (D[a][0] at the lower, D[a][N] at the upper end of each line); the
// missing residual part -(1/|J|) * that lift is added in place to the
// outputs of the flux pass with their stage weights (Pout: c1 c2, Tout:
// d1 d2; residual mode: 1), and the FP32 face traces of the new P are
// pushed to the neighbours.
// END: the last lift pass of a call, which writes the state Q = Q0 + P
// (S_.Qend) in the place of P and pushes no traces (the next call forms P and
// its traces from Q): a pass over Q0, P and Q and a trace push less per call
// (0.44 ms and 0.1 ms on 331,776 hexes).
// (its tables are copied at once: BlockTables makes no difference here but at
// order 2, 803 -> 820 us per RK3 step on 192,000 hexes)
template <int N, int EPB, int NT, bool END>
__global__ __launch_bounds__(NT) void k_lift_mixed(OpsF<N> opa, GeoF G, const float *__restrict__ TV, MixedStage S_) {
    constexpr int NP = N * N * N, NF2 = N * N;
    constexpr int IT_MB = (EPB * 24 * NF2 + NT - 1) / NT, IT_SOL = (EPB * NP + NT - 1) / NT;
    __shared__ OpsF<N> op;
    ops_to_lds(opa, op);
    __shared__ float nv[EPB][6][4][NF2];  // neighbours' viscous momentum and energy flux, 0 on boundary faces
    __shared__ float sp[EPB][5][NP];      // new perturbation (FP32) for the traces
    __shared__ int32_t lk[EPB][6], inf[EPB][6];
    // blocks walk the elements from the last to the first: the flux pass
    // before ran from the first to the last, so the first blocks here read
    // its latest writes, which are still in the memory-side cache; the next
    // flux pass starts where this pass ends, for the same reason
    const int64_t e0 = (int64_t)(gridDim.x - 1 - blockIdx.x) * EPB;
    const bool useT = S_.mode != 0 && S_.Tout != nullptr;
    // every global input first: face links, the viscous mailbox (boundary
    // slots too: never written, selected away below), outputs of the flux
    // pass and 1/|J|
    int32_t rl = -1, ri = 0;
    {
        const bool okl = (int)threadIdx.x < EPB * 6 && e0 + threadIdx.x / 6 < G.E;
        const int32_t l = G.link[okl ? e0 * 6 + threadIdx.x : 0], i = G.info[okl ? e0 * 6 + threadIdx.x : 0];
        rl = okl ? l : -1;
        ri = okl ? i : 0;
    }
    // (unpredicated loads through clamped indices; items past the end are
    // never stored)
    float mb[IT_MB];
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = threadIdx.x + k * NT;
        const bool ok = it < EPB * 24 * NF2 && e0 + it / (24 * NF2) < G.E;
        mb[k] = ld_once(&TV[ok ? e0 * 24 * NF2 + it : 0]);
    }
    double po[IT_SOL][5], to[IT_SOL][5], q0[IT_SOL][5];
    float iJ[IT_SOL];
#pragma unroll
    for (int k = 0; k < IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const int el = it / NP, p = it % NP;
        const int64_t e = (it < EPB * NP && e0 + el < G.E) ? e0 + el : 0;
        iJ[k] = ld_once(&G.solgeo[(e * 13 + 9) * NP + p]);
        for (int v = 0; v < 5; ++v) {
            const int64_t gi = ((int64_t)v * G.E + e) * NP + p;
            po[k][v] = S_.Pout[gi];
            to[k][v] = useT ? S_.Tout[gi] : 0.0;
            q0[k][v] = END ? S_.Q0[gi] : 0.0;
        }
    }
    if ((int)threadIdx.x < EPB * 6) {
        lk[threadIdx.x / 6][threadIdx.x % 6] = rl;
        inf[threadIdx.x / 6][threadIdx.x % 6] = ri;
    }
    __syncthreads();
    // the mailbox slot of a boundary face is never written: select, do not
    // multiply by zero
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * 24 * NF2) break;
        const int el = it / (24 * NF2), r = it % (24 * NF2), f = r / (4 * NF2);
        (&nv[el][0][0][0])[r] = (lk[el][f] >= 0) ? mb[k] : 0.0f;
    }
    __syncthreads();
    const double wP = (S_.mode == 0) ? 1.0 : S_.c1 * S_.c2, wT = S_.d1 * S_.d2;
#pragma unroll
    for (int k = 0; k < IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        float corr[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int pp = t1 + N * t2;
            const float wl = -0.5f * op.D[a][0], wu = 0.5f * op.D[a][N];
#pragma unroll
            for (int v = 1; v < 5; ++v)
                corr[v] += wl * nv[el][2 * d][v - 1][pp] + wu * nv[el][2 * d + 1][v - 1][pp];
        }
        for (int v = 0; v < 5; ++v) {
            const int64_t gi = ((int64_t)v * G.E + e) * NP + p;
            const double x = -(double)(iJ[k] * corr[v]);
            const double pv = po[k][v] + wP * x;
            if constexpr (END) {
                S_.Qend[gi] = state_of(q0[k][v], pv);
                continue;
            }
            S_.Pout[gi] = pv;
            if (useT) S_.Tout[gi] = to[k][v] + wT * x;
            sp[el][v][p] = (float)pv;
        }
    }
    if (END || S_.mode == 0 || S_.TQout == nullptr) return;
    __syncthreads();
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        const int32_t nb = lk[el][f];
        if (e >= G.E || nb < 0) continue;
        float *out = S_.TQout + mailbox_slot<N>(nb, inf[el][f], pp);
        const int d = f >> 1, m = (f & 1) ? N : 0, base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
        for (int v = 0; v < 5; ++v) st_once(&out[v * NF2], line_val<N>(op, sp[el][v], m, base, st));
    }
}

// ---------------------------------------------------------------------------
// wide passes: one element per block, the work of a phase spread over all
// threads of the block (small meshes)
// ---------------------------------------------------------------------------
// A thread takes one variable of one solution point (gradients, divergence,
// update) or one flux point (faces and interior points of all directions in
// one index range, the three directions' fluxes in LDS together): on a mesh
// that leaves wave slots empty a pass lasts as long as one block, and this
// shortens the block's chain (162 hexes of order 4, SSP-RK3: 43.5 -> 27.5 us
// per step).  The sums run over the same terms in the same order as in the
// element passes.
template <int N, int NT>
struct WideM {
    static constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N, NINT = 3 * (N - 1) * N * N;
    static constexpr int NFACE = 6 * NF2;
    // first interior item: the face points keep waves of their own (but for
    // blocks of one wave)
    static constexpr int FP = NT == 64 ? NFACE : (NFACE + 63) / 64 * 64;
    static constexpr int IT_VP = (5 * NP + NT - 1) / NT;
    static constexpr int IT_FACE = (NFACE + NT - 1) / NT;
    static constexpr int IT_FX = (FP + NINT + NT - 1) / NT;
};

template <int N, int NT, int MINW, int KR>
__global__ __launch_bounds__(NT, MINW) void k_flux_mixed_wide(OpsF<N> opa, GeoF G, MixedBufs B, PhysF F,
                                                              const double *__restrict__ Pq,
                                                              const float *__restrict__ TQ, float *__restrict__ TV,
                                                              MixedStage S_) {
    using W = WideM<N, NT>;
    constexpr int NP = W::NP, NF2 = W::NF2, NFL = W::NFL;
    using EL = MixedEl<N, 3, N == 2>;
    __shared__ EL L;
    __shared__ OpsF<N> op;
    __shared__ int32_t lk[6], inf_[6];
    const int64_t e = blockIdx.x, E = G.E;
    const int t = threadIdx.x;
    BlockTables<1, NT, float, N> bt;
    bt.load(opa, G.link, G.info, e, E);
    // every global input before the first wait (unpredicated, clamped)
    double pv[W::IT_VP];
    float Gm[W::IT_VP][9], bg[W::IT_VP];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        pv[k] = Pq[((int64_t)v * E + e) * NP + p];
        // rows 0, 1: rho0, E0; rows 2..4: grad rho0
        bg[k] = v < 2 ? B.bg[(e * 2 + v) * NP + p] : B.gbg[(e * 3 + v - 2) * NP + p];
    }
    float nq[W::IT_FACE][5], db[W::IT_FACE][2];
#pragma unroll
    for (int k = 0; k < W::IT_FACE; ++k) {
        const int it = t + k * NT < W::NFACE ? t + k * NT : 0;
        const int64_t base = e * 6 + it / NF2;
        for (int v = 0; v < 5; ++v) nq[k][v] = TQ[(base * 5 + v) * NF2 + it % NF2];
        for (int v = 0; v < 2; ++v) db[k][v] = B.dbg[(base * 2 + v) * NF2 + it % NF2];
    }
    // flux point of item x: direction d, position m along line tt
    auto where = [&](int x, int &d, int &m, int &tt) {
        if (x < W::NFACE) {
            const int f = x / NF2;
            d = f >> 1;
            m = (f & 1) ? N : 0;
            tt = x % NF2;
        } else {
            const int i = (x >= W::FP && x < W::FP + W::NINT) ? x - W::FP : 0, q = i % ((N - 1) * NF2);
            d = i / ((N - 1) * NF2);
            m = 1 + q % (N - 1);
            tt = q / (N - 1);
        }
    };
    float S[W::IT_FX][3], gS[W::IT_FX], krl[W::IT_FX];
#pragma unroll
    for (int k = 0; k < W::IT_FX; ++k) {
        int d, m, tt;
        where(t + k * NT, d, m, tt);
        const int fl = m + (N + 1) * tt;
        for (int c = 0; c < 3; ++c) S[k][c] = G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
        gS[k] = B.gS0[(e * 3 + d) * NFL + fl];
        krl[k] = (KR == KR_RADIAL) ? G.rflux[(e * 3 + d) * NFL + fl] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int p = (t + k * NT) % NP;
        for (int c = 0; c < 9; ++c) Gm[k][c] = G.solgeo[(e * 13 + c) * NP + p];
    }
    bt.store(op, lk, inf_);
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        const float hi = (float)pv[k];
        L.at(v, p) = hi;
        L.plo(v, p) = (float)(pv[k] - (double)hi);
        L.at(v < 2 ? F_R0 + v : EL::GR + 3 * F_R0 + v - 2, p) = bg[k];
    }
    __syncthreads();
    // common values; the own face values of the 7 fields are kept
    float fo[W::IT_FACE][8];
#pragma unroll
    for (int k = 0; k < W::IT_FACE; ++k) {
        const int it = t + k * NT;
        if (it >= W::NFACE) break;
        const int f = it / NF2, pp = it % NF2, d = f >> 1, m = (f & 1) ? N : 0;
        const int base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
        L.template line<0, 2>(op, m, base, st, fo[k]);
        common_value(fo[k], fo[k][F_R0], lk[f], inf_[f], nq[k], S[k], F,
                     [&](int v, float x) { L.u.cs[v][f][pp] = x; });
    }
    __syncthreads();
    // gradient of one variable at one solution point
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        float dq[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d), pp = t1 + N * t2;
            float s = mac(op.D[a][N], L.u.cs[v][2 * d + 1][pp], op.D[a][0] * L.u.cs[v][2 * d][pp]);
#pragma unroll
            for (int b = 0; b < N; ++b) s = mac(op.B[a][b], L.at(v, base + b * st), s);
            dq[d] = s;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            L.at(EL::GR + 3 * v + c, p) = Gm[k][c] * dq[0] + Gm[k][3 + c] * dq[1] + Gm[k][6 + c] * dq[2];
    }
    __syncthreads();
    // every flux point of the element
#pragma unroll
    for (int k = 0; k < W::IT_FX; ++k) {
        const int x = t + k * NT;
        int d, m, tt;
        where(x, d, m, tt);
        const int base = sol_of<N>(d, 0, tt % N, tt / N), st = stride_of<N>(d), fl = m + (N + 1) * tt;
        const float kr = kr_of<KR>(F, krl[k]);
        if (k < W::IT_FACE && x < W::NFACE) {
            const int kf = k < W::IT_FACE ? k : 0, f = x / NF2;
            const int32_t nb = lk[f], inf = inf_[f];
            const float sg = (f & 1) ? 1.0f : -1.0f;
            const float So[3] = {sg * S[k][0], sg * S[k][1], sg * S[k][2]}, gSo = sg * gS[k];
            float fv[5], ff[5];
            PtState st_;
            state_at<N>(op, L, m, base, st, st_, fo[kf]);
            if (nb >= 0) {
                dflux_viscous<KR>(st_, So, gSo, F, kr, 0, fv);
                // the viscous mass flux is zero: four components per point
                const int64_t slot = mailbox_slot<N, 4>(nb, inf, tt);
                for (int v = 1; v < 5; ++v) st_once(&TV[slot + (v - 1) * NF2], fv[v]);
            }
            face_flux_own<KR>(st_, nq[kf], db[kf], nb >= 0, ((inf >> 6) - 1) == CHORUS_BC_OUTER, So, gSo, kr, fv, F, ff);
            for (int v = 0; v < 5; ++v) L.u.ft[d][v][fl] = sg * ff[v];
        } else if (x >= W::FP && x < W::FP + W::NINT) {
            PtState s;
            state_at<N>(op, L, m, base, st, s);
            float fi[5], fv[5];
            dflux_inviscid(s, S[k], F, fi);
            dflux_viscous<KR>(s, S[k], gS[k], F, kr, 0, fv);
            for (int v = 0; v < 5; ++v) L.u.ft[d][v][fl] = fi[v] - fv[v];
        }
    }
    // operands of the update, loaded before the divergence (every one before
    // the first store: the outputs may alias the inputs)
    const bool rk = S_.mode != 0;
    const bool useA = rk && S_.c0 != 0.0, useT = rk && S_.Tout != nullptr, useB = useT && S_.d0 != 0.0;
    float r0v[W::IT_VP], gq[W::IT_VP][4];
    double pst[W::IT_VP], pb[W::IT_VP];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        for (int c = 0; c < 4; ++c) gq[k][c] = G.solgeo[(e * 13 + 9 + c) * NP + p];
        r0v[k] = B.R0[gi];
        pst[k] = useA ? S_.A[gi] : 0.0;
        pb[k] = useB ? S_.B[gi] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        float div = 0.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int fb = (N + 1) * (t1 + N * t2);
            float s = 0.0f;
#pragma unroll
            for (int mm = 0; mm <= N; ++mm) s = mac(op.D[a][mm], L.u.ft[d][v][fb + mm], s);
            div += s;
        }
        const float g0 = F.GM * gq[k][1], g1 = F.GM * gq[k][2], g2 = F.GM * gq[k][3];
        const float rp = L.at(F_RP, p), mx = L.at(F_MX, p), my = L.at(F_MY, p), mz = L.at(F_MZ, p);
        const float M = v == 1   ? rp * g0 - 2.0f * F.om * my
                        : v == 2 ? rp * g1 + 2.0f * F.om * mx
                        : v == 3 ? rp * g2
                        : v == 4 ? mx * g0 + my * g1 + mz * g2
                                 : 0.0f;
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        const double Rv = (double)r0v[k] + (double)(-div * gq[k][0] - M);
        if (!rk) {
            S_.Pout[gi] = Rv;
            continue;
        }
        // the stage input from its FP32 value and remainder (as above)
        const double pin = (double)L.at(v, p) + (double)L.plo(v, p);
        if (useT) S_.Tout[gi] = S_.d0 * pb[k] + S_.d1 * (pin + S_.d2 * Rv);
        S_.Pout[gi] = S_.c0 * pst[k] + S_.c1 * (pin + S_.c2 * Rv);
    }
}

template <int N, int NT, bool END>
__global__ __launch_bounds__(NT) void k_lift_mixed_wide(OpsF<N> opa, GeoF G, const float *__restrict__ TV,
                                                        MixedStage S_) {
    using W = WideM<N, NT>;
    constexpr int NP = W::NP, NF2 = W::NF2, MBE = 24 * NF2, IT_MB = (MBE + NT - 1) / NT;
    __shared__ float nv[6][4][NF2];  // neighbours' viscous momentum and energy flux, 0 on boundary faces
    __shared__ float sp[5][NP];      // new perturbation (FP32) for the traces
    __shared__ int32_t lk[6], inf[6];
    __shared__ OpsF<N> op;
    const int64_t e = blockIdx.x, E = G.E;
    const int t = threadIdx.x;
    const bool useT = S_.mode != 0 && S_.Tout != nullptr;
    BlockTables<1, NT, float, N> bt;
    bt.load(opa, G.link, G.info, e, E);
    // every global input first (unpredicated, clamped; the mailbox slots of
    // boundary faces are never written and are selected away below)
    float mb[IT_MB];
    int32_t ml[IT_MB];
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = t + k * NT < MBE ? t + k * NT : 0;
        mb[k] = ld_once(&TV[e * MBE + it]);
        ml[k] = G.link[e * 6 + it / (4 * NF2)];
    }
    double po[W::IT_VP], to[W::IT_VP], q0[W::IT_VP];
    float iJ[W::IT_VP];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        iJ[k] = G.solgeo[(e * 13 + 9) * NP + p];
        po[k] = S_.Pout[gi];
        to[k] = useT ? S_.Tout[gi] : 0.0;
        q0[k] = END ? S_.Q0[gi] : 0.0;
    }
    bt.store(op, lk, inf);
#pragma unroll
    for (int k = 0; k < IT_MB; ++k)
        if (t + k * NT < MBE) (&nv[0][0][0])[t + k * NT] = (ml[k] >= 0) ? mb[k] : 0.0f;
    __syncthreads();
    const double wP = (S_.mode == 0) ? 1.0 : S_.c1 * S_.c2, wT = S_.d1 * S_.d2;
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        float corr = 0.0f;
        if (v > 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                int a, t1, t2;
                split_sol<N>(d, p, a, t1, t2);
                const int pp = t1 + N * t2;
                const float wl = -0.5f * op.D[a][0], wu = 0.5f * op.D[a][N];
                corr += wl * nv[2 * d][v - 1][pp] + wu * nv[2 * d + 1][v - 1][pp];
            }
        }
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        const double x = -(double)(iJ[k] * corr);
        const double pn = po[k] + wP * x;
        if constexpr (END) {
            S_.Qend[gi] = state_of(q0[k], pn);
            continue;
        }
        S_.Pout[gi] = pn;
        if (useT) S_.Tout[gi] = to[k] + wT * x;
        sp[v][p] = (float)pn;
    }
    if (END || S_.mode == 0 || S_.TQout == nullptr) return;
    __syncthreads();
    for (int it = t; it < 30 * NF2; it += NT) {
        const int v = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int32_t nb = lk[f];
        if (nb < 0) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0;
        const float tr = line_val<N>(op, sp[v], m, sol_of<N>(d, 0, pp % N, pp / N), stride_of<N>(d));
        st_once(S_.TQout + mailbox_slot<N>(nb, inf[f], pp) + v * NF2, tr);
    }
}

// background setup (FP64): rho0, E0 (FP32) at solution points; the jump of
// the background face traces across each interface (neighbour minus own,
// from the FP64 traces TQ0 of Q0, rounded to FP32); a flag if Q0 moves
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_bg_setup(Ops<N> opa, Geo G, const double *__restrict__ Q0,
                                                 const double *__restrict__ TQ0, float *__restrict__ bg,
                                                 float *__restrict__ dbg, int *__restrict__ flag) {
    constexpr int NP = N * N * N, NF2 = N * N;
    __shared__ double s0[EPB][2][NP];
    __shared__ Ops<N> op;
    ops_to_lds(opa, op);
    const int64_t e0 = (int64_t)blockIdx.x * EPB, E = G.E;
    for (int it = threadIdx.x; it < EPB * NP; it += NT) {
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= E) continue;
        const double r = Q0[(0 * E + e) * NP + p], en = Q0[(4 * E + e) * NP + p];
        const double mx = Q0[(1 * E + e) * NP + p], my = Q0[(2 * E + e) * NP + p], mz = Q0[(3 * E + e) * NP + p];
        if (mx != 0.0 || my != 0.0 || mz != 0.0) flag[0] = 1;
        s0[el][0][p] = r;
        s0[el][1][p] = en;
        bg[(e * 2 + 0) * NP + p] = (float)r;
        bg[(e * 2 + 1) * NP + p] = (float)en;
    }
    __syncthreads();
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= E) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0, t1 = pp % N, t2 = pp / N;
        const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d);
        const int32_t nb = G.link[e * 6 + f];
        for (int v = 0; v < 2; ++v) {
            double own = 0.0;
            for (int b = 0; b < N; ++b) own += op.I[m][b] * s0[el][v][base + b * st];
            double jump = 0.0;
            if (nb >= 0) {
                const int inf = G.info[e * 6 + f];
                const int pn = map_face_point<N>((inf >> 3) & 7, t1, t2);
                jump = TQ0[(((int64_t)nb * 6 + (inf & 7)) * 5 + (v == 0 ? 0 : 4)) * NF2 + pn] - own;
            }
            dbg[((e * 6 + f) * 2 + v) * NF2 + pp] = (float)jump;
        }
    }
}

__global__ void k_to_float(const double *__restrict__ a, float *__restrict__ b, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int N>
struct CfgM;
// elements per block and threads of the element kernels (trace setup,
// background setup), and the minimum waves per SIMD of the flux pass
template <> struct CfgM<2> { static constexpr int EPB = 8, NT = 64, MINW = 2; };
template <> struct CfgM<3> { static constexpr int EPB = 2, NT = 64, MINW = 3; };
template <> struct CfgM<4> { static constexpr int EPB = 1, NT = 64, MINW = 4; };
template <> struct CfgM<5> { static constexpr int EPB = 1, NT = 128, MINW = 2; };
// (order 6: four waves, 830 against 945 us per step with the three that 130
// registers leave; three with the radial diffusivity, which would spill: 974
// against 1,052)
template <> struct CfgM<6> { static constexpr int EPB = 1, NT = 256, MINW = 4; };
// flux pass (elements per block, threads, minimum waves per SIMD) and lift
// pass (elements per block, threads)
template <int N> struct CfgF { static constexpr int EPB = CfgM<N>::EPB, NT = CfgM<N>::NT, MINW = CfgM<N>::MINW; };
template <int N> struct CfgL { static constexpr int EPB = CfgM<N>::EPB, NT = CfgM<N>::NT; };

// Wide passes: threads per block of the smallest meshes (NT1, minimum waves
// per SIMD W1) and of the next larger ones (NT2, W2), and the largest meshes
// of each and of the lift pass and set-up, in elements per CU.  The limits
// lie where an SSP-RK3 step of a shell crosses (us per step, element
// passes / wide passes with NT1 [/ NT2] threads):
//   order 2: 56.0 / 51.5 at 5,184 hexes, 60.9 / 64.0 at 7,776; lift alone
//            60.9 / 59.9 at 7,776, 72.7 / 80.6 at 12,288
//   order 3: flux alone 39.3 / 26.7 at 288, 59.3 / 52.0 at 2,304, 67.4 / 67.3
//            at 3,600, 83.1 / 85.9 at 5,184; lift alone 53.9 / 53.1 at 1,536, 62.9 / 63.8 at 2,304
//   order 4: 45.8 / 31.6 / 36.4 at 288, 51.0 / 43.0 / 42.1 at 648; flux alone
//            47.7 / - / 43.8 at 864, 56.3 / - / 54.7 at 1,350, 60.3 / - / 58.5
//            at 1,536 (six blocks of three waves per CU, all resident), 62.3 /
//            - / 64.4 at 1,728 (a second round), 63.8 / - / 68.4 at 1,944;
//            lift alone 60.3 / 55.2 at 1,536, 62.3 / 60.2 at 1,728, 63.8 / 65.4
//            at 1,944, 73.0 / 70.2 at 2,304 (the line at the flux pass's)
//   order 5: 52.9 / 33.0 / 42.3 at 162; flux alone 48.1 / - / 44.5 at 288,
//            60.3 / - / 61.5 at 648; lift alone 58.6 / 55.2 at 288, 68.7 / 69.2
//            at 648
//   order 6: 43.4 / 41.3 at 162, 58.9 / 72.1 at 288
template <int N> struct CfgW;
template <> struct CfgW<2> { static constexpr int NT1 = 64, W1 = 1, MAX1 = 20, NT2 = 64, W2 = 1, MAX2 = 0, LIFT = 28; };
template <> struct CfgW<3> { static constexpr int NT1 = 192, W1 = 1, MAX1 = 9, NT2 = 192, W2 = 1, MAX2 = 0, LIFT = 6; };
template <> struct CfgW<4> { static constexpr int NT1 = 320, W1 = 4, MAX1 = 2, NT2 = 192, W2 = 4, MAX2 = 6, LIFT = 6; };
template <> struct CfgW<5> { static constexpr int NT1 = 640, W1 = 3, MAX1 = 1, NT2 = 256, W2 = 4, MAX2 = 2, LIFT = 2; };
template <> struct CfgW<6> { static constexpr int NT1 = 832, W1 = 4, MAX1 = 1, NT2 = 832, W2 = 4, MAX2 = 0, LIFT = 1; };

static GeoF geof_of(const GeoM &g) {
    GeoF o;
    o.solgeo = g.solgeo32;
    o.fluxgeo = g.fluxgeo32;
    o.link = g.link;
    o.info = g.info;
    o.E = g.E;
    o.rflux = g.rflux32;
    return o;
}
static MixedBufs bufs_of(const GeoM &g) {
    MixedBufs b;
    b.bg = g.bg;
    b.dbg = g.dbg;
    b.gS0 = g.gS0;
    b.R0 = g.R0;
    b.gbg = g.gbg;
    return b;
}

template <int N>
static hipError_t pert_begin_t(const Mesh &m, const GeoM &g, const double *Q, double *Pq, float *TQ, hipStream_t s) {
    constexpr int EPB = CfgM<N>::EPB, NT = CfgM<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    if (m.E <= kCUs * CfgW<N>::LIFT) {
        hipLaunchKernelGGL((k_pert_begin<N, 1, CfgW<N>::NT1>), dim3((unsigned)m.E), dim3(CfgW<N>::NT1), 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), Q, g.Q0, Pq, TQ);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_pert_begin<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, make_ops_t<float, N>(m.basis),
                       geof_of(g), Q, g.Q0, Pq, TQ);
    return hipGetLastError();
}
template <int N, int NT, int MINW>
static hipError_t flux_mixed_wide_t(const Mesh &m, const GeoM &g, const PhysParams &P, const double *Pq,
                                    const float *TQ, float *TV, const MixedStage &st, hipStream_t s) {
    const dim3 grid((unsigned)m.E), block(NT);
    if (P.kappa_r1 != 0.0 || P.kappa_r2 != 0.0)
        hipLaunchKernelGGL((k_flux_mixed_wide<N, NT, MINW, KR_RADIAL>), grid, block, 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    else if (P.kappa_r != 0.0)
        hipLaunchKernelGGL((k_flux_mixed_wide<N, NT, MINW, KR_CONST>), grid, block, 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    else
        hipLaunchKernelGGL((k_flux_mixed_wide<N, NT, MINW, KR_NONE>), grid, block, 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    return hipGetLastError();
}
template <int N>
static hipError_t flux_mixed_t(const Mesh &m, const GeoM &g, const PhysParams &P, const double *Pq, const float *TQ,
                               float *TV, const MixedStageArgs &a, hipStream_t s) {
    constexpr int EPB = CfgF<N>::EPB, NT = CfgF<N>::NT, MINW = CfgF<N>::MINW;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    const MixedStage st = a;
    if (m.E <= kCUs * CfgW<N>::MAX1) return flux_mixed_wide_t<N, CfgW<N>::NT1, CfgW<N>::W1>(m, g, P, Pq, TQ, TV, st, s);
    if (m.E <= kCUs * CfgW<N>::MAX2) return flux_mixed_wide_t<N, CfgW<N>::NT2, CfgW<N>::W2>(m, g, P, Pq, TQ, TV, st, s);
    if (P.kappa_r1 != 0.0 || P.kappa_r2 != 0.0)
        hipLaunchKernelGGL((k_flux_mixed<N, EPB, NT, MINW, KR_RADIAL>), dim3(nb), dim3(NT), 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    else if (P.kappa_r != 0.0)
        hipLaunchKernelGGL((k_flux_mixed<N, EPB, NT, MINW, KR_CONST>), dim3(nb), dim3(NT), 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    else
        hipLaunchKernelGGL((k_flux_mixed<N, EPB, NT, MINW, KR_NONE>), dim3(nb), dim3(NT), 0, s,
                           make_ops_t<float, N>(m.basis), geof_of(g), bufs_of(g), physf_of(P), Pq, TQ, TV, st);
    return hipGetLastError();
}
template <int N>
static hipError_t lift_mixed_t(const Mesh &m, const GeoM &g, const float *TV, const MixedStageArgs &a, hipStream_t s) {
    constexpr int EPB = CfgL<N>::EPB, NT = CfgL<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    const MixedStage st = a;
    const bool end = a.Qend != nullptr;
    if (m.E <= kCUs * CfgW<N>::LIFT) {
        constexpr int NW = CfgW<N>::NT1;
        const dim3 grid((unsigned)m.E), block(NW);
        if (end)
            hipLaunchKernelGGL((k_lift_mixed_wide<N, NW, true>), grid, block, 0, s, make_ops_t<float, N>(m.basis),
                               geof_of(g), TV, st);
        else
            hipLaunchKernelGGL((k_lift_mixed_wide<N, NW, false>), grid, block, 0, s, make_ops_t<float, N>(m.basis),
                               geof_of(g), TV, st);
    } else if (end) {
        hipLaunchKernelGGL((k_lift_mixed<N, EPB, NT, true>), dim3(nb), dim3(NT), 0, s, make_ops_t<float, N>(m.basis),
                           geof_of(g), TV, st);
    } else {
        hipLaunchKernelGGL((k_lift_mixed<N, EPB, NT, false>), dim3(nb), dim3(NT), 0, s, make_ops_t<float, N>(m.basis),
                           geof_of(g), TV, st);
    }
    return hipGetLastError();
}
template <int N>
static hipError_t bg_setup_t(const Mesh &m, const Geo &G, const double *Q0, const double *TQ0, float *bg, float *dbg,
                             int *flag, hipStream_t s) {
    constexpr int EPB = CfgM<N>::EPB, NT = CfgM<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((k_bg_setup<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, make_ops_t<double, N>(m.basis), G, Q0,
                       TQ0, bg, dbg, flag);
    return hipGetLastError();
}

#define CHORUS_DISPATCH_M(N_, CALL)          \
    switch (N_) {                            \
        case 2: return CALL(2);              \
        case 3: return CALL(3);              \
        case 4: return CALL(4);              \
        case 5: return CALL(5);              \
        case 6: return CALL(6);              \
        default: return hipErrorInvalidValue; \
    }

hipError_t launch_pert_begin(const Mesh &m, const GeoM &g, const double *Q, double *Pq, float *TQ, hipStream_t s) {
#define C_(n) pert_begin_t<n>(m, g, Q, Pq, TQ, s)
    CHORUS_DISPATCH_M(m.N, C_)
#undef C_
}
hipError_t launch_flux_mixed(const Mesh &m, const GeoM &g, const PhysParams &P, const double *Pq, const float *TQ,
                             float *TV, const MixedStageArgs &a, hipStream_t s) {
#define C_(n) flux_mixed_t<n>(m, g, P, Pq, TQ, TV, a, s)
    CHORUS_DISPATCH_M(m.N, C_)
#undef C_
}
hipError_t launch_lift_mixed(const Mesh &m, const GeoM &g, const float *TV, const MixedStageArgs &a, hipStream_t s) {
#define C_(n) lift_mixed_t<n>(m, g, TV, a, s)
    CHORUS_DISPATCH_M(m.N, C_)
#undef C_
}
hipError_t launch_bg_setup(const Mesh &m, const Geo &G, const double *Q0, const double *TQ0, float *bg, float *dbg,
                           int *flag, hipStream_t s) {
#define C_(n) bg_setup_t<n>(m, G, Q0, TQ0, bg, dbg, flag, s)
    CHORUS_DISPATCH_M(m.N, C_)
#undef C_
}
hipError_t launch_to_float(const double *a, float *b, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_float, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

}  // namespace chorus
