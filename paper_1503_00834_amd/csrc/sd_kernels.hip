// HIP kernels (gfx950) of the FP64 spectral-difference residual and the
// explicit Runge-Kutta update (Section 3 of the paper).
//
// One stage is split in two element passes because BR1 needs two
// neighbour exchanges (Section 3, viscous treatment):
//
//   k_flux64   Q (own element) + neighbours' Q face traces
//              -> common interface solution, gradients, [learned subgrid
//                 flux], own-side common fluxes and own viscous face flux
//                 (pushed to the neighbours), fluxes at the interior flux
//                 points, divergence, source, and the stage combination with
//                 this partial residual
//              (order 4: k_flux64_n4, the line operators as matrix products;
//              meshes that leave most of the chip idle: k_flux64_wide, one
//              element per block of several waves, and likewise
//              k_lift64_wide and k_trace_push_wide)
//   k_lift64   neighbours' viscous face fluxes -> the missing residual part
//              added in place; face traces of the new state pushed to the
//              neighbours for the next stage.
//
// k_trace (traces indexed by their own element) serves the closure features
// and the background set-up of the mixed path; the flux pass's network-only
// variant serves closure inference.
//
// Work mapping: a workgroup of NT threads owns EPB elements; every phase is
// a loop over (element, point) items with all element data staged in LDS.
// No atomics: every output is written by exactly one thread in a fixed
// summation order, so results are bitwise run-to-run deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "launch.hpp"
#include "mlp_bf16.hpp"
#include "sd_common.hpp"

namespace chorus {

// ---------------------------------------------------------------------------
// shared phases
// ---------------------------------------------------------------------------
template <int N, int EPB, int NT, bool SW = false>
__device__ __forceinline__ void load_q(const double *__restrict__ Q, int64_t E, int64_t e0,
                                       double (*sq)[5][N * N * N]) {
    // (every load before the first store; items past the end repeat the last)
    constexpr int NP = N * N * N, TOT = EPB * 5 * NP, IT = (TOT + NT - 1) / NT;
    double q[IT];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int it = min((int)threadIdx.x + k * NT, TOT - 1), v = it % (5 * NP) / NP;
        const int64_t e = e0 + it / (5 * NP);
        q[k] = Q[((int64_t)v * E + (EPB == 1 || e < E ? e : 0)) * NP + it % NP];
    }
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int it = min((int)threadIdx.x + k * NT, TOT - 1), el = it / (5 * NP), v = it % (5 * NP) / NP, p = it % NP;
        sq[el][v][SW ? lds_sol<N>(p) : p] = (EPB == 1 || e0 + el < E) ? q[k] : (v == 0 || v == 4 ? 1.0 : 0.0);
    }
}

// common interface solution Q* at the 6 N^2 face points (BR1 average with
// the neighbour trace, wall state, or average with the far-field state)
template <int N, int EPB, int NT>
__device__ __forceinline__ void common_solution(const Ops<N> &op, const Geo &G, const PhysParams &P,
                                                const double *__restrict__ TQ, int64_t e0,
                                                double (*sq)[5][N * N * N],
                                                double (*sqs)[6][5][N * N]) {
    constexpr int NF2 = N * N, NFL = (N + 1) * N * N;
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0, t1 = pp % N, t2 = pp / N;
        const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d);
        double qo[5], qs[5];
        for (int v = 0; v < 5; ++v) {
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < N; ++b) s += op.I[m][b] * sq[el][v][base + b * st];
            qo[v] = s;
        }
        const int32_t nb = G.link[e * 6 + f];
        const int32_t inf = G.info[e * 6 + f];
        const int bc = (inf >> 6) - 1;
        if (nb >= 0) {
            const int f2 = inf & 7, o = (inf >> 3) & 7;
            const int pn = map_face_point<N>(o, t1, t2);
            const double *tq = TQ + ((int64_t)nb * 6 + f2) * 5 * NF2;
            for (int v = 0; v < 5; ++v) qs[v] = 0.5 * (qo[v] + tq[v * NF2 + pn]);
        } else if (bc == CHORUS_BC_INNER || bc == CHORUS_BC_OUTER) {
            const int fl = m + (N + 1) * (t1 + N * t2);
            const double sg = (f & 1) ? 1.0 : -1.0;
            double S[3];
            for (int c = 0; c < 3; ++c) S[c] = sg * G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
            wall_state(qo, S, bc == CHORUS_BC_OUTER, P, qs);
        } else {
            for (int v = 0; v < 5; ++v) qs[v] = 0.5 * (qo[v] + P.bc_state[v]);
        }
        for (int v = 0; v < 5; ++v) sqs[el][f][v][pp] = qs[v];
    }
}

// gradients of the conserved variables at the solution points:
// dQ/dxi_d = B q_line + D[.,0] Q*_0 + D[.,N] Q*_N, then grad_x = sum_d G_d dQ/dxi_d
template <int N, int EPB, int NT>
__device__ __forceinline__ void gradients(const Ops<N> &op, const Geo &G, int64_t e0,
                                          double (*sq)[5][N * N * N], double (*sqs)[6][5][N * N],
                                          double (*sgr)[15][N * N * N]) {
    constexpr int NP = N * N * N;
    for (int it = threadIdx.x; it < EPB * NP; it += NT) {
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        double dq[3][5];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d), pp = t1 + N * t2;
            for (int v = 0; v < 5; ++v) {
                double s = op.D[a][0] * sqs[el][2 * d][v][pp] + op.D[a][N] * sqs[el][2 * d + 1][v][pp];
#pragma unroll
                for (int b = 0; b < N; ++b) s += op.B[a][b] * sq[el][v][base + b * st];
                dq[d][v] = s;
            }
        }
        const double *gs = G.solgeo + e * 13 * NP + p;
        double Gm[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) Gm[t] = gs[t * NP];
        for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                sgr[el][v * 3 + c][p] = Gm[c] * dq[0][v] + Gm[3 + c] * dq[1][v] + Gm[6 + c] * dq[2][v];
    }
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// face traces of Q: TQ[e][f][v][pp]
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_trace(Ops<N> opa, Geo G, const double *__restrict__ Q,
                                              double *__restrict__ TQ) {
    constexpr int NP = N * N * N, NF2 = N * N;
    __shared__ double sq[EPB][5][NP];
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    __shared__ Ops<N> op;
    OpsWords<NT, double, N> ow;
    ow.load(opa);
    load_q<N, EPB, NT>(Q, G.E, e0, sq);
    ow.store(op);
    __syncthreads();
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0, t1 = pp % N, t2 = pp / N;
        const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d);
        for (int v = 0; v < 5; ++v) {
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < N; ++b) s += op.I[m][b] * sq[el][v][base + b * st];
            TQ[((e * 6 + f) * 5 + v) * NF2 + pp] = s;
        }
    }
}

// Normalised network input of one solution point (state q, gradients g), in
// FP64 before it is rounded, as the B-operand words of the first layer: four
// times eight features (pairs of bfloat16), 20 features and padding.  The
// thread that forms a point's gradients has all of them in registers; when
// each lane of the network fetched its eight features one by one through
// per-lane selects, this took 93 of the fused pass's 694 us on 98,304 hexes.
__device__ __forceinline__ void closure_input(const unsigned char *__restrict__ model, const double q[5],
                                              const double g[15], u32x4_t w[3]) {
    const f32x4_t *mean = reinterpret_cast<const f32x4_t *>(model + kMlpFloatOff + 4 * kMlpXMean);
    const f32x4_t *inv = reinterpret_cast<const f32x4_t *>(model + kMlpFloatOff + 4 * kMlpXInv);
    w[2] = u32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int f4 = 0; f4 < kMlpIn / 4; ++f4) {
        const f32x4_t mu = mean[f4], is = inv[f4];
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 4 * f4 + i;
            x[i] = (float)(((f < 5 ? q[f < 5 ? f : 0] : g[f < 5 ? 0 : f - 5]) - (double)mu[i]) * (double)is[i]);
        }
        w[f4 >> 1][(f4 & 1) * 2] = bf16_pair(x[0], x[1]);
        w[f4 >> 1][(f4 & 1) * 2 + 1] = bf16_pair(x[2], x[3]);
    }
}

// learned subgrid flux at the solution points of the block's elements (one
// wave, all points in 16-point tiles): inputs xf (LDS, four words of eight
// features per point) -> network -> tau[k][E][NP] (global), or into the
// block's LDS copy stau when given, which may share space with xf
template <int N, int EPB, int NT>
__device__ __forceinline__ void closure_tau(const ClosureArgs &C, int64_t E, int64_t e0, const u32x4_t (*xf)[4],
                                            float (*stau)[15][N * N * N] = nullptr) {
    constexpr int NP = N * N * N, NPTS = EPB * NP, NPT = (NPTS + 15) / 16;
    static_assert(NT == 64, "the closure runs one wave per block");
    const int lane = threadIdx.x, g = lane >> 4;
    u32x4_t xb[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        const int pidx = 16 * j + (lane & 15);
        const u32x4_t w = xf[pidx < NPTS ? pidx : 0][g];
        xb[j] = pidx < NPTS ? w : u32x4_t{0, 0, 0, 0};
    }
    __syncthreads();
    // all tiles together: the weights are read once (two tiles at a time take
    // 13 us more per pass on 98,304 hexes)
    f32x4_t out[NPT];
    mlp_eval<NPT>(C.model, xb, out);
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        const int pidx = 16 * j + (lane & 15);
        const int el = pidx / NP, sp = pidx % NP;
        if (pidx >= NPTS || e0 + el >= E) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * g + i;
            if (k >= kMlpOut) continue;
            if (stau) stau[el][k][sp] = out[j][i];
            else C.tau[((int64_t)k * E + e0 + el) * NP + sp] = out[j][i];
        }
    }
}

// raw closure features at the solution points: X[e NP + p][20] = (Q, grad Q)
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_features(Ops<N> opa, Geo G, PhysParams P, const double *__restrict__ Q,
                                                 const double *__restrict__ TQ, float *__restrict__ X) {
    constexpr int NP = N * N * N, NF2 = N * N;
    __shared__ double sq[EPB][5][NP];
    __shared__ double sqs[EPB][6][5][NF2];
    __shared__ double sgr[EPB][15][NP];
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    __shared__ Ops<N> op;
    OpsWords<NT, double, N> ow;
    ow.load(opa);
    load_q<N, EPB, NT>(Q, G.E, e0, sq);
    ow.store(op);
    __syncthreads();
    common_solution<N, EPB, NT>(op, G, P, TQ, e0, sq, sqs);
    __syncthreads();
    gradients<N, EPB, NT>(op, G, e0, sq, sqs, sgr);
    __syncthreads();
    for (int it = threadIdx.x; it < EPB * NP * 20; it += NT) {
        const int el = it / (NP * 20), r = it % (NP * 20), p = r / 20, f = r % 20;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        X[(e * NP + p) * 20 + f] = (float)(f < 5 ? sq[el][f][p] : sgr[el][f - 5][p]);
    }
}



// ---------------------------------------------------------------------------
// flux pass + lift pass (the stage split used by the solver)
// ---------------------------------------------------------------------------
// Per stage: the flux pass takes every step that needs the gradients --
// common interface solution, gradients, [learned subgrid flux], at the face
// points the own viscous flux (pushed to the neighbour's viscous mailbox)
// and the own-side common flux (Rusanov minus half the own viscous flux,
// the wall flux, or the far-field flux), at the interior flux points the
// transformed flux, the divergence with the own-side face fluxes at the line
// ends, the source -- and enters the stage combination with this partial
// residual.  The lift pass adds the neighbours' viscous halves in place and
// pushes the face traces of the new state to the neighbours' mailboxes.
// Mailboxes are indexed by the receiving element, face and point (in the
// receiver's point order), so each element reads its own contiguous block.
template <int N, int EPB, int NT>
struct Sh64 {
    static constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N, NINTD = (N - 1) * N * N;
    // LDS of the flux pass.  A point's state and gradients are one record of SR
    // doubles, read as pairs: a wave's 16-byte LDS read takes 6.3 cycles, an
    // 8-byte one 5.0.  Records of 22 doubles put 16 consecutive points on
    // distinct banks; order 6, with the most line reads, is faster with the
    // two spare doubles (1,125 against 1,230 us per step below), the others
    // with less LDS.  Face and flux points in records of 6 (5 values) at order
    // 6, where they fit beside three blocks per compute unit; at order 5 they
    // cost a block (1,380 against 1,335 us) and at orders 2 and 3 they gain
    // nothing: planes.
    // us per RK3 step, one plane per field -> records (hexes of the mesh):
    // N = 2 (192,000) 1,027 -> 1,010; N = 3 (98,304) 1,433 -> 1,375;
    // N = 5 (24,000) 1,434 -> 1,335; N = 6 (12,288) 1,256 -> 1,125.
    static constexpr bool FREC = N == 6;
    static constexpr int SR = N == 6 ? 22 : 20, NV = FREC ? 6 : 5;
    static constexpr __device__ int face_at(int f, int v, int pp) {
        return FREC ? (f * NF2 + pp) * 6 + v : (f * 5 + v) * NF2 + pp;
    }
    static constexpr __device__ int flux_at(int v, int fl) { return FREC ? fl * 6 + v : v * NFL + fl; }
    static constexpr int IT_SOL = (EPB * NP + NT - 1) / NT;
    static constexpr int IT_FACE = (EPB * 6 * NF2 + NT - 1) / NT;
    static constexpr int IT_INTD = (EPB * NINTD + NT - 1) / NT;
};

// launch shape of the flux/lift passes per order: elements per block,
// threads, minimum waves per SIMD of the flux pass
template <int N>
struct Cfg64;
template <> struct Cfg64<2> { static constexpr int EPB = 8, NT = 64, MINW = 1; };
template <> struct Cfg64<3> { static constexpr int EPB = 2, NT = 64, MINW = 1; };
template <> struct Cfg64<4> { static constexpr int EPB = 1, NT = 64, MINW = 3; };
template <> struct Cfg64<5> { static constexpr int EPB = 1, NT = 128, MINW = 3; };
// (order 6: with a radial diffusivity the pass would otherwise take 170
// registers and lose its third wave: 1,280 against 1,148 us per step)
template <> struct Cfg64<6> { static constexpr int EPB = 1, NT = 256, MINW = 3; };

// face traces of the element block's state (LDS, lds_sol layout) pushed to
// the neighbours
template <int N, int EPB, int NT>
__device__ __forceinline__ void push_traces64(const Ops<N> &op, const Geo &G, int64_t e0, const int32_t (*lk)[6],
                                              const int32_t (*inf)[6], const double (*sq)[5][N * N * N],
                                              double *__restrict__ TQout) {
    constexpr int NF2 = N * N;
    for (int it = threadIdx.x; it < EPB * 6 * NF2; it += NT) {
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int32_t nb = lk[el][f];
        if (e0 + el >= G.E || nb < 0) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0;
        const int base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
        double *out = TQout + mailbox_slot<N>(nb, inf[el][f], pp);
        for (int v = 0; v < 5; ++v) {
            double t = 0.0;
#pragma unroll
            for (int b = 0; b < N; ++b) t += op.I[m][b] * sq[el][v][lds_line<N>(base, b, st)];
            st_once(&out[v * NF2], t);
        }
    }
}

// face traces of Q pushed to the neighbours' mailboxes (start of a call)
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_trace_push(Ops<N> opa, Geo G, const double *__restrict__ Q,
                                                   double *__restrict__ TQ) {
    constexpr int NP = N * N * N;
    __shared__ double sq[EPB][5][NP];
    __shared__ int32_t lk[EPB][6], inf[EPB][6];
    __shared__ Ops<N> op;
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    BlockTables<EPB, NT, double, N> bt;
    bt.load(opa, G.link, G.info, e0, G.E);
    load_q<N, EPB, NT, true>(Q, G.E, e0, sq);
    bt.store(op, &lk[0][0], &inf[0][0]);
    __syncthreads();
    push_traces64<N, EPB, NT>(op, G, e0, lk, inf, sq, TQ);
}

// line interpolation of an LDS field at flux point m of the line (base, st)
template <int N, typename T>
__device__ __forceinline__ double line_interp(const Ops<N> &op, const T *fld, int m, int base, int st) {
    double t = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) t += op.I[m][b] * (double)fld[base + b * st];
    return t;
}
// the same over a field stored in the lds_sol layout
template <int N, typename T>
__device__ __forceinline__ double line_interp_s(const Ops<N> &op, const T *fld, int m, int base, int st) {
    double t = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) t += op.I[m][b] * (double)fld[lds_line<N>(base, b, st)];
    return t;
}

// five values of a record (pairs, 16-byte aligned) or of planes PL apart
template <bool REC, int PL>
__device__ __forceinline__ void load5(const double *r, double x[5]) {
    if constexpr (REC) {
        const double2 a = *reinterpret_cast<const double2 *>(r), b = *reinterpret_cast<const double2 *>(r + 2);
        x[0] = a.x, x[1] = a.y, x[2] = b.x, x[3] = b.y, x[4] = r[4];
    } else {
        for (int v = 0; v < 5; ++v) x[v] = r[v * PL];
    }
}

// An element's state and gradients in LDS, one record per point (5 state
// values, then 15 gradients): the values at flux point m of the line (base,
// st), read as pairs of fields.
template <int N, int SR>
struct Records {
    const double (*r)[SR];
    __device__ __forceinline__ void pair(const Ops<N> &op, int m, int base, int st, int j, double &x, double &y) const {
        x = y = 0.0;
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const double2 t = *reinterpret_cast<const double2 *>(&r[base + b * st][2 * j]);
            x += op.I[m][b] * t.x;
            y += op.I[m][b] * t.y;
        }
    }
    __device__ __forceinline__ void state(const Ops<N> &op, int m, int base, int st, double q[5]) const {
        pair(op, m, base, st, 0, q[0], q[1]);
        pair(op, m, base, st, 1, q[2], q[3]);
        double t = 0.0;
#pragma unroll
        for (int b = 0; b < N; ++b) t += op.I[m][b] * r[base + b * st][4];
        q[4] = t;
    }
    __device__ __forceinline__ void all(const Ops<N> &op, int m, int base, int st, double q[5], double g[5][3]) const {
        double x[20];
#pragma unroll
        for (int j = 0; j < 10; ++j) pair(op, m, base, st, j, x[2 * j], x[2 * j + 1]);
        for (int v = 0; v < 5; ++v) {
            q[v] = x[v];
            for (int c = 0; c < 3; ++c) g[v][c] = x[5 + v * 3 + c];
        }
    }
};

// common interface solution at a face point with the own values fo (BR1
// average with the neighbour trace nq, wall state, or average with the
// far-field state)
__device__ __forceinline__ void common_value64(const double fo[5], int32_t nb, int32_t info, const double nq[5],
                                               const double Sf[3], const PhysParams &P, double qs[5]) {
    const int bc = (info >> 6) - 1;
    if (nb >= 0) {
        for (int v = 0; v < 5; ++v) qs[v] = 0.5 * (fo[v] + nq[v]);
    } else if (bc == CHORUS_BC_INNER || bc == CHORUS_BC_OUTER) {
        wall_state(fo, Sf, bc == CHORUS_BC_OUTER, P, qs);  // (the same along +-S)
    } else {
        for (int v = 0; v < 5; ++v) qs[v] = 0.5 * (fo[v] + P.bc_state[v]);
    }
}

// the same at point pp of face f from the element's state in LDS
template <int N, typename FS>
__device__ __forceinline__ void common_point64(const Ops<N> &op, const FS &fs, int f, int pp,
                                               int32_t nb, int32_t info, const double nq[5], const double Sf[3],
                                               const PhysParams &P, double qs[5]) {
    const int d = f >> 1, m = (f & 1) ? N : 0;
    const int base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
    double fo[5];
    fs.state(op, m, base, st, fo);
    common_value64(fo, nb, info, nq, Sf, P, qs);
}

// own-side common flux ffc along the outward Sf at a face point with the own
// values fo, gradients g and (CL) subgrid flux ts(v) along Sf of variable v;
// the own viscous flux to the neighbour's mailbox TV (pp: the point, kr: the
// radiative diffusivity)
template <int N, bool CL, typename TS>
__device__ __forceinline__ void face_flux64(const double fo[5], const double g[5][3], TS &&ts, int pp,
                                            int32_t nb, int32_t info, const double nq[5], const double Sf[3],
                                            const PhysParams &P, double kr, double *__restrict__ TV, double ffc[5]) {
    constexpr int NF2 = N * N;
    const int bc = (info >> 6) - 1;
    double fv[5];
    if (nb >= 0) {
        flux_viscous(fo, g, Sf, P, kr, fv);
        if constexpr (CL)  // the own-side subgrid flux enters the trace with the sign of -F_v
            for (int v = 0; v < 5; ++v) fv[v] -= ts(v);
        // the viscous mass flux is zero: four components per point
        // unless the subgrid flux (with a mass part) rides along
        constexpr int NV = CL ? 5 : 4;
        double *tv = TV + mailbox_slot<N, NV>(nb, info, pp);
        for (int v = 5 - NV; v < 5; ++v) st_once(&tv[(v - (5 - NV)) * NF2], fv[v]);
        flux_rusanov(fo, nq, Sf, P, ffc);
        for (int v = 0; v < 5; ++v) ffc[v] -= 0.5 * fv[v];
    } else if (bc == CHORUS_BC_INNER || bc == CHORUS_BC_OUTER) {
        flux_wall(fo, g, Sf, bc == CHORUS_BC_OUTER, P, kr, ffc);
    } else {
        flux_viscous(fo, g, Sf, P, kr, fv);
        flux_rusanov(fo, P.bc_state, Sf, P, ffc);
        for (int v = 0; v < 5; ++v) ffc[v] -= 0.5 * fv[v];
    }
}

// the same at point pp of face f from the element's state, gradients and
// (CL) subgrid flux in LDS
template <int N, bool CL, typename FS>
__device__ __forceinline__ void face_point64(const Ops<N> &op, const FS &fs, const float *stau, int f, int pp,
                                             int32_t nb, int32_t info, const double nq[5], const double Sf[3],
                                             const PhysParams &P, double kr, double *__restrict__ TV, double ffc[5]) {
    constexpr int NP = N * N * N;
    const int d = f >> 1, m = (f & 1) ? N : 0;
    const int base = sol_of<N>(d, 0, pp % N, pp / N), st = stride_of<N>(d);
    double fo[5], g[5][3];
    fs.all(op, m, base, st, fo, g);
    auto ts = [&](int v) {
        double x = 0.0;
        for (int c = 0; c < 3; ++c) x += line_interp<N>(op, stau + (v * 3 + c) * NP, m, base, st) * Sf[c];
        return x;
    };
    face_flux64<N, CL>(fo, g, ts, pp, nb, info, nq, Sf, P, kr, TV, ffc);
}

// transformed flux along S at the interior flux point m of line (t1, t2) of
// direction d
template <int N, bool CL, typename FS>
__device__ __forceinline__ void interior_point64(const Ops<N> &op, const FS &fs, const float *stau, int d, int m,
                                                 int tt, const double S[3], const PhysParams &P, double kr,
                                                 double out[5]) {
    constexpr int NP = N * N * N;
    const int base = sol_of<N>(d, 0, tt % N, tt / N), st = stride_of<N>(d);
    double qf[5], g[5][3], fi[5], fv[5];
    fs.all(op, m, base, st, qf, g);
    flux_inviscid(qf, S, P.gamma - 1.0, fi);
    flux_viscous(qf, g, S, P, kr, fv);
    for (int v = 0; v < 5; ++v) {
        double ts = 0.0;
        if constexpr (CL)
            for (int c = 0; c < 3; ++c) ts += line_interp<N>(op, stau + (v * 3 + c) * NP, m, base, st) * S[c];
        out[v] = fi[v] - fv[v] + ts;
    }
}

// source term M of variable v (gravity g = GM x / r^3, Coriolis) at a point
__device__ __forceinline__ double source64(int v, double rho, double mx, double my, double mz, const double g[3],
                                           double omega) {
    if (v == 1) return rho * g[0] - 2.0 * omega * my;
    if (v == 2) return rho * g[1] + 2.0 * omega * mx;
    if (v == 3) return rho * g[2];
    if (v == 4) return mx * g[0] + my * g[1] + mz * g[2];
    return 0.0;
}

// PART 0: the flux pass; PART 1: only the learned subgrid flux (common
// solution, gradients, network -> C.tau: chorus_closure_infer); PART 2: the
// flux pass with the learned subgrid flux evaluated in the pass (network on
// the gradients in LDS, its output kept in LDS)
// RAD: radiative diffusivity varying with radius (radius of each flux point
// read with its geometry), else the constant P.kappa_r (at order 5 with fewer
// waves: 1,518 against 1,595 us per step on 24,000 hexes, where three spill)
template <int N, int EPB, int NT, int PART, bool RAD>
__global__ __launch_bounds__(NT, PART == 2 && RAD ? 3 : N == 5 && RAD ? 2 : Cfg64<N>::MINW)
void k_flux64(Ops<N> opa, Geo G, PhysParams P, const double *__restrict__ Q,
              const double *__restrict__ TQ, double *__restrict__ TV, StageArgs S_, ClosureArgs C) {
    constexpr bool CL = PART != 0;
    using Sh = Sh64<N, EPB, NT>;
    constexpr int NP = Sh::NP, NF2 = Sh::NF2, NFL = Sh::NFL, NINTD = Sh::NINTD;
    constexpr int SR = PART == 1 ? 6 : Sh::SR;
    __shared__ alignas(16) double rec[EPB][NP][SR];  // state, gradients (not in PART 1) at the solution points
    // the common solution is consumed by the gradients before the subgrid
    // flux (PART 2) and the first direction's fluxes are written
    __shared__ union {
        alignas(16) double sqs[EPB][6 * NF2 * Sh::NV];
        struct {
            alignas(16) double sft[EPB][NFL * Sh::NV];
            union {
                u32x4_t xf[CL ? EPB * NP : 1][4];                     // network inputs
                float stau[CL ? EPB : 1][15][CL ? NP : 1];            // subgrid flux (PART 2)
            } C;
        } F;
    } U;
    auto &stau = U.F.C.stau;
    __shared__ int32_t lk[EPB][6], inf[EPB][6];
    __shared__ alignas(16) Ops<N> op;
    const int64_t e0 = (int64_t)blockIdx.x * EPB, E = G.E;
    BlockTables<EPB, NT, double, N> bt;
    bt.load(opa, G.link, G.info, e0, E);
    // every global input of the element block before the first wait;
    // unpredicated loads through clamped indices (items past the end read
    // element 0 and are never stored)
    double qv[Sh::IT_SOL][5], Gm[Sh::IT_SOL][9];
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const int el = it / NP, p = it % NP;
        const int64_t e = (it < EPB * NP && e0 + el < E) ? e0 + el : 0;
        for (int v = 0; v < 5; ++v) qv[k][v] = Q[((int64_t)v * E + e) * NP + p];
        for (int t = 0; t < 9; ++t) Gm[k][t] = G.solgeo[(e * 13 + t) * NP + p];
    }
    // radiative diffusivity at the face and interior flux points
    double nq[Sh::IT_FACE][5], Sf[Sh::IT_FACE][3], krf[Sh::IT_FACE];
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int64_t e = (it < EPB * 6 * NF2 && e0 + el < E) ? e0 + el : 0;
        for (int v = 0; v < 5; ++v) nq[k][v] = TQ[((e * 6 + f) * 5 + v) * NF2 + pp];
        const int d = f >> 1, fl = ((f & 1) ? N : 0) + (N + 1) * pp;
        const double sg = (f & 1) ? 1.0 : -1.0;
        for (int c = 0; c < 3; ++c) Sf[k][c] = sg * G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
        krf[k] = RAD ? G.rflux[(e * 3 + d) * NFL + fl] : P.kappa_r;
    }
    // interior flux-point metrics: one direction at a time, the next one
    // issued while the current one is used (fewer registers in flight)
    double Si[2][Sh::IT_INTD][3], kri[2][Sh::IT_INTD];
    auto load_si = [&](int d, int slot) {
#pragma unroll
        for (int k = 0; k < Sh::IT_INTD; ++k) {
            const int it = threadIdx.x + k * NT;
            const int el = it / NINTD, q = it % NINTD;
            const int fl = 1 + q % (N - 1) + (N + 1) * (q / (N - 1));
            const int64_t e = (it < EPB * NINTD && e0 + el < E) ? e0 + el : 0;
            for (int c = 0; c < 3; ++c) Si[slot][k][c] = G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
            kri[slot][k] = RAD ? G.rflux[(e * 3 + d) * NFL + fl] : P.kappa_r;
        }
    };
    if constexpr (PART != 1) load_si(0, 0);
    bt.store(op, &lk[0][0], &inf[0][0]);
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        for (int v = 0; v < 5; ++v) rec[it / NP][it % NP][v] = qv[k][v];
    }
    __syncthreads();
    // common interface solution (the own face values are formed again in
    // the face-flux phase: fewer registers live across the gradients)
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * 6 * NF2) break;
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        if (e0 + el >= E) continue;
        double qs[5];
        common_point64<N>(op, Records<N, SR>{rec[el]}, f, pp, lk[el][f], inf[el][f], nq[k], Sf[k], P, qs);
        for (int v = 0; v < 5; ++v) U.sqs[el][Sh::face_at(f, v, pp)] = qs[v];
    }
    __syncthreads();
    // gradients at the solution points, network inputs
    u32x4_t xw[CL ? Sh::IT_SOL : 1][3];
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        double dq[3][5], gr[15];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d), pp = t1 + N * t2;
            double ql[5], qr[5];
            load5<Sh::FREC, NF2>(&U.sqs[el][Sh::face_at(2 * d, 0, pp)], ql);
            load5<Sh::FREC, NF2>(&U.sqs[el][Sh::face_at(2 * d + 1, 0, pp)], qr);
            for (int v = 0; v < 5; ++v) dq[d][v] = op.D[a][0] * ql[v] + op.D[a][N] * qr[v];
#pragma unroll
            for (int b = 0; b < N; ++b) {
                double q[5];
                load5<true, 1>(rec[el][base + b * st], q);
                for (int v = 0; v < 5; ++v) dq[d][v] += op.B[a][b] * q[v];
            }
        }
        for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                gr[v * 3 + c] = Gm[k][c] * dq[0][v] + Gm[k][3 + c] * dq[1][v] + Gm[k][6 + c] * dq[2][v];
        if constexpr (PART != 1)
            for (int f = 0; f < 15; ++f) rec[el][p][5 + f] = gr[f];
        if constexpr (CL) {
            double q[5];
            for (int v = 0; v < 5; ++v) q[v] = rec[el][p][v];
            closure_input(C.model, q, gr, xw[k]);
        }
    }
    __syncthreads();
    if constexpr (CL) {
        // (over the common solution, which the gradients have consumed)
#pragma unroll
        for (int k = 0; k < Sh::IT_SOL; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * NP) break;
            for (int w = 0; w < 3; ++w) U.F.C.xf[it][w] = xw[k][w];
            U.F.C.xf[it][3] = u32x4_t{0, 0, 0, 0};
        }
        __syncthreads();
        // subgrid flux at the solution points -> C.tau (PART 1) or LDS
        if constexpr (PART == 1) {
            closure_tau<N, EPB, NT>(C, E, e0, U.F.C.xf);
            return;
        }
        closure_tau<N, EPB, NT>(C, E, e0, U.F.C.xf, stau);
        __syncthreads();
    }
    // face points: own viscous flux to the neighbour, own-side common flux
    // kept in registers for the divergence
    double ffc[Sh::IT_FACE][5];
#pragma unroll
    for (int k = 0; k < Sh::IT_FACE; ++k) {
        const int it = threadIdx.x + k * NT;
        for (int v = 0; v < 5; ++v) ffc[k][v] = 0.0;
        if (it >= EPB * 6 * NF2) break;
        const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        if (e0 + el >= E) continue;
        const double kr = RAD ? kappa_r_at(P, krf[k]) : krf[k];
        face_point64<N, CL>(op, Records<N, SR>{rec[el]}, CL ? &stau[el][0][0] : nullptr, f, pp, lk[el][f],
                            inf[el][f], nq[k], Sf[k], P, kr, TV, ffc[k]);
    }
    // per direction: transformed flux at the d-flux points, its derivative
    // added to the divergence at the solution points
    double div[Sh::IT_SOL][5];
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k)
        for (int v = 0; v < 5; ++v) div[k][v] = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int cur = d & 1;
        if (d < 2) load_si(d + 1, cur ^ 1);
#pragma unroll
        for (int k = 0; k < Sh::IT_INTD; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * NINTD) break;
            const int el = it / NINTD, q = it % NINTD;
            const int m = 1 + q % (N - 1), tt = q / (N - 1);
            if (e0 + el >= E) continue;
            double fi[5];
            interior_point64<N, CL>(op, Records<N, SR>{rec[el]}, CL ? &stau[el][0][0] : nullptr, d, m, tt, Si[cur][k], P,
                                    RAD ? kappa_r_at(P, kri[cur][k]) : kri[cur][k], fi);
            const int fl = m + (N + 1) * tt;
            for (int v = 0; v < 5; ++v) U.F.sft[el][Sh::flux_at(v, fl)] = fi[v];
        }
#pragma unroll
        for (int k = 0; k < Sh::IT_FACE; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * 6 * NF2) break;
            const int el = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
            if ((f >> 1) != d || e0 + el >= E) continue;
            const double sg = (f & 1) ? 1.0 : -1.0;
            const int fl = ((f & 1) ? N : 0) + (N + 1) * pp;
            for (int v = 0; v < 5; ++v) U.F.sft[el][Sh::flux_at(v, fl)] = sg * ffc[k][v];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < Sh::IT_SOL; ++k) {
            const int it = threadIdx.x + k * NT;
            if (it >= EPB * NP) break;
            const int el = it / NP, p = it % NP;
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int fb = (N + 1) * (t1 + N * t2);
            double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int mm = 0; mm <= N; ++mm) {
                double fm[5];
                load5<Sh::FREC, NFL>(&U.F.sft[el][Sh::flux_at(0, fb + mm)], fm);
                for (int v = 0; v < 5; ++v) t[v] += op.D[a][mm] * fm[v];
            }
            for (int v = 0; v < 5; ++v) div[k][v] += t[v];
        }
        __syncthreads();
    }
    // source and the stage combination with the partial residual (operands
    // loaded before the first store: the outputs may alias them)
    const bool rk = S_.mode != 0;
    const bool useA = rk && S_.c0 != 0.0, useT = rk && S_.Tout != nullptr, useB = useT && S_.d0 != 0.0;
    double gq[Sh::IT_SOL][4], av[Sh::IT_SOL][5], bv[Sh::IT_SOL][5];
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const int el = it / NP, p = it % NP;
        const int64_t e = (it < EPB * NP && e0 + el < E) ? e0 + el : 0;
        for (int c = 0; c < 4; ++c) gq[k][c] = G.solgeo[(e * 13 + 9 + c) * NP + p];
        for (int v = 0; v < 5; ++v) {
            const int64_t gi = ((int64_t)v * E + e) * NP + p;
            av[k][v] = useA ? S_.A[gi] : 0.0;
            bv[k][v] = useB ? S_.B[gi] : 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < Sh::IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= E) continue;
        const double iJ = gq[k][0];
        const double g0 = P.GM * gq[k][1], g1 = P.GM * gq[k][2], g2 = P.GM * gq[k][3];
        const double *r = rec[el][p];
        const double rho = r[0], mx = r[1], my = r[2], mz = r[3];
        double M[5];
        M[0] = 0.0;
        M[1] = rho * g0 - 2.0 * P.omega * my;
        M[2] = rho * g1 + 2.0 * P.omega * mx;
        M[3] = rho * g2;
        M[4] = mx * g0 + my * g1 + mz * g2;
        for (int v = 0; v < 5; ++v) {
            const double R = -div[k][v] * iJ - M[v];
            const int64_t gi = ((int64_t)v * E + e) * NP + p;
            if (!rk) {
                S_.Qout[gi] = R;
                continue;
            }
            const double q = r[v];
            if (useT) S_.Tout[gi] = S_.d0 * bv[k][v] + S_.d1 * (q + S_.d2 * R);
            S_.Qout[gi] = S_.c0 * av[k][v] + S_.c1 * (q + S_.c2 * R);
        }
    }
}

// ---------------------------------------------------------------------------
// flux pass of order 4: line operators as 4 x 4 matrix products
// ---------------------------------------------------------------------------
// One wave per element.  At order 4 an operator applied along the 16 lines of
// a direction is one v_mfma_f64_4x4x4 (four independent 4 x 4 x 4 products):
// lane l = l0 + 4 l1 + 16 l2 supplies A[l0][l2] and B[l2][l0] of block l1 and
// receives D[l2][l0].  With the lines (l0, l1) as columns and blocks, the
// field values along a line as K and the operator as A, a field is read from
// LDS once per direction, one value per lane, where the scalar form reads
// the four values of its line in every lane; a lane receives its own point's
// value, so the pointwise flux follows in place and its result is the K
// operand of the divergence as it stands.
//   zeta lines: operand lane (x, y, z) = natural point order, result natural
//   xi lines:   operand lane (z, y, x); used as A with the operator as B the
//               result is natural (gradients, divergence)
//   eta lines:  operand lane (x, z, y), result in the same order: one exchange
//               through LDS to natural order
// The face points of a direction are 2 rows of the product: the xi and eta
// faces fill one wave (lane group l2 = face), the zeta faces half of one.
// FP64 matrix instructions issue at the rate of the vector unit's
// multiply-adds (16 cycles for 4 x 64), so what is saved is LDS traffic and
// its latency and the per-lane operator reads.  Sums run over the same terms
// as the scalar form.
// Measured on 41,472 hexes against the scalar form (one element per wave too,
// 14.6 KB of LDS): 312 -> 222 us per launch, 411 -> 139 LDS and 2,245 -> 1,457
// vector instructions per wave, 12.8 KB of LDS and 160 registers (three waves
// per SIMD).  The pass has to move 27 KB per element: 5.0 TB/s, the rate of a
// large copy, which bounds it now.
__device__ __forceinline__ double mfma44(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

template <bool RAD>
__global__ __launch_bounds__(64, 3) void k_flux64_n4(Ops<4> op, Geo G, PhysParams P, const double *__restrict__ Q,
                                                     const double *__restrict__ TQ, double *__restrict__ TV,
                                                     StageArgs S_) {
    constexpr int N = 4, NP = 64, NF2 = 16, NFL = 80;
    __shared__ double sq[5][NP];
    __shared__ union {
        double g[15][NP];  // gradients
        struct {
            double qs[6][5][NF2];  // common solution by (face, variable, line), consumed by the gradients
            double tr[5][NP];      // eta results on their way to natural order
        } c;
    } U;
    __shared__ double sff[4][5][NF2];  // signed common fluxes: xi upper, eta lower, eta upper, zeta upper faces
    const int64_t e = blockIdx.x, E = G.E;
    const int l = threadIdx.x, l0 = l & 3, l1 = (l >> 2) & 3, l2 = l >> 4, s = l & 15;
    // face points of the two rounds: xi and eta faces (f = l2), zeta faces
    const int ppx = l1 + 4 * l0;  // face point of line slot s on the xi faces (t1 = y = l1, t2 = z = l0)
    const int fa = l2, ppa = l2 < 2 ? ppx : s, fb = 4 + (l2 & 1), ppb = s;
    // every global input of the element before the first wait
    double qv[5], Gm[9], nqa[5], nqb[5], Sa[3], Sb[3], Si[2][3], kra, krb, kri[2];
    for (int v = 0; v < 5; ++v) qv[v] = Q[((int64_t)v * E + e) * NP + l];
    const int32_t lka = G.link[e * 6 + fa], lkb = G.link[e * 6 + fb];
    const int32_t ina = G.info[e * 6 + fa], inb = G.info[e * 6 + fb];
    for (int v = 0; v < 5; ++v) {
        nqa[v] = TQ[((e * 6 + fa) * 5 + v) * NF2 + ppa];
        nqb[v] = TQ[((e * 6 + fb) * 5 + v) * NF2 + ppb];
    }
    const double sga = (fa & 1) ? 1.0 : -1.0, sgb = (fb & 1) ? 1.0 : -1.0;
    const int fla = ((fa & 1) ? N : 0) + (N + 1) * ppa, flb = ((fb & 1) ? N : 0) + (N + 1) * ppb;
    for (int c = 0; c < 3; ++c) {
        Sa[c] = sga * G.fluxgeo[((e * 3 + (fa >> 1)) * 3 + c) * NFL + fla];
        Sb[c] = sgb * G.fluxgeo[((e * 3 + 2) * 3 + c) * NFL + flb];
    }
    kra = RAD ? G.rflux[(e * 3 + (fa >> 1)) * NFL + fla] : 0.0;
    krb = RAD ? G.rflux[(e * 3 + 2) * NFL + flb] : 0.0;
    for (int c = 0; c < 9; ++c) Gm[c] = G.solgeo[(e * 13 + c) * NP + l];
    // flux-point metrics of one direction: lane (m = l2, line slot s)
    auto load_si = [&](int d, int slot) {
        const int fl = l2 + (N + 1) * (d == 0 ? ppx : s);
        for (int c = 0; c < 3; ++c) Si[slot][c] = G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
        kri[slot] = RAD ? G.rflux[(e * 3 + d) * NFL + fl] : 0.0;
    };
    load_si(0, 0);
    // operator entries of this lane
    const double cB = op.B[l0][l2], cF = op.I[(l0 & 1) ? N : 0][l2];
    // LDS slots of the lane's operand of each direction
    const int nx = lds_sol<N>(l2 + 4 * l1 + 16 * l0), ny = lds_sol<N>(l0 + 4 * l2 + 16 * l1), nz = lds_sol<N>(l);
    for (int v = 0; v < 5; ++v) sq[v][nz] = qv[v];
    __syncthreads();
    // common interface solution
    double qx[5], qy[5];
    {
        double fo[5], qs[5];
        for (int v = 0; v < 5; ++v) {
            qx[v] = sq[v][nx];
            qy[v] = sq[v][ny];
            const double a = mfma44(cF, qx[v], 0.0), b = mfma44(cF, qy[v], 0.0);
            fo[v] = l2 < 2 ? a : b;
        }
        common_value64(fo, lka, ina, nqa, Sa, P, qs);
        for (int v = 0; v < 5; ++v) U.c.qs[fa][v][s] = qs[v];
        for (int v = 0; v < 5; ++v) fo[v] = mfma44(cF, qv[v], 0.0);
        if (l < 32) {
            common_value64(fo, lkb, inb, nqb, Sb, P, qs);
            for (int v = 0; v < 5; ++v) U.c.qs[fb][v][s] = qs[v];
        }
    }
    __syncthreads();
    // gradients at the solution points
    {
        const double w0 = op.D[l0][0], w4 = op.D[l0][N], u0 = op.D[l2][0], u4 = op.D[l2][N];
        const int sx = l2 + 4 * l1;  // line slot of the natural point on the xi faces
        double dx[5], dy[5], dz[5];
        for (int v = 0; v < 5; ++v) {
            dy[v] = mfma44(cB, qy[v], u0 * U.c.qs[2][v][s] + u4 * U.c.qs[3][v][s]);
            dx[v] = mfma44(qx[v], cB, w0 * U.c.qs[0][v][sx] + w4 * U.c.qs[1][v][sx]);
            dz[v] = mfma44(cB, qv[v], u0 * U.c.qs[4][v][s] + u4 * U.c.qs[5][v][s]);
        }
        for (int v = 0; v < 5; ++v) U.c.tr[v][ny] = dy[v];
        __syncthreads();
        for (int v = 0; v < 5; ++v) dy[v] = U.c.tr[v][nz];
        __syncthreads();
        for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int c = 0; c < 3; ++c) U.g[v * 3 + c][nz] = Gm[c] * dx[v] + Gm[3 + c] * dy[v] + Gm[6 + c] * dz[v];
    }
    __syncthreads();
    // face points: own viscous flux to the neighbour, own-side common flux;
    // the lower xi and zeta fluxes stay in the lanes that use them
    const auto no_ts = [](int) { return 0.0; };
    double fxl[5], fzl[5];
    {
        double fo[5], g[5][3], ff[5];
        auto both = [&](const double *fld) {
            const double a = mfma44(cF, fld[nx], 0.0), b = mfma44(cF, fld[ny], 0.0);
            return l2 < 2 ? a : b;
        };
        for (int v = 0; v < 5; ++v) {
            fo[v] = both(sq[v]);
            for (int c = 0; c < 3; ++c) g[v][c] = both(U.g[v * 3 + c]);
        }
        face_flux64<N, false>(fo, g, no_ts, ppa, lka, ina, nqa, Sa, P, RAD ? kappa_r_at(P, kra) : P.kappa_r, TV, ff);
        for (int v = 0; v < 5; ++v) {
            fxl[v] = sga * ff[v];
            if (l2 > 0) sff[l2 - 1][v][s] = fxl[v];
        }
    }
    {
        double fo[5], g[5][3], ff[5];
        for (int v = 0; v < 5; ++v) {
            fo[v] = mfma44(cF, sq[v][nz], 0.0);
            for (int c = 0; c < 3; ++c) g[v][c] = mfma44(cF, U.g[v * 3 + c][nz], 0.0);
            fzl[v] = 0.0;
        }
        if (l < 32) {
            face_flux64<N, false>(fo, g, no_ts, ppb, lkb, inb, nqb, Sb, P, RAD ? kappa_r_at(P, krb) : P.kappa_r, TV, ff);
            for (int v = 0; v < 5; ++v) {
                fzl[v] = sgb * ff[v];
                if (l2 == 1) sff[3][v][s] = fzl[v];
            }
        }
    }
    __syncthreads();
    // per direction (xi, zeta, eta): transformed flux at the flux points
    // (lane (m = l2, line slot s), the lower face's in place at m = 0), its
    // derivative added to the divergence
    double div[5];
    const double cI = op.I[l0][l2], cD = op.D[l0][l2], w4 = op.D[l0][N], u4 = op.D[l2][N];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int d = q == 0 ? 0 : q == 1 ? 2 : 1, cur = q & 1, at = d == 0 ? nx : d == 1 ? ny : nz;
        if (q < 2) load_si(q == 0 ? 2 : 1, cur ^ 1);
        double qf[5], g[5][3], fi[5], fv[5], F[5];
        for (int v = 0; v < 5; ++v) {
            qf[v] = mfma44(cI, sq[v][at], 0.0);
            for (int c = 0; c < 3; ++c) g[v][c] = mfma44(cI, U.g[v * 3 + c][at], 0.0);
        }
        flux_inviscid(qf, Si[cur], P.gamma - 1.0, fi);
        flux_viscous(qf, g, Si[cur], P, RAD ? kappa_r_at(P, kri[cur]) : P.kappa_r, fv);
        for (int v = 0; v < 5; ++v) {
            const double lo = d == 0 ? fxl[v] : d == 2 ? fzl[v] : sff[1][v][s];
            F[v] = l2 == 0 ? lo : fi[v] - fv[v];
        }
        if (d == 0) {
            const int sx = l2 + 4 * l1;
            for (int v = 0; v < 5; ++v) div[v] = mfma44(F[v], cD, 0.0) + w4 * sff[0][v][sx];
        } else if (d == 2) {
            for (int v = 0; v < 5; ++v) div[v] += mfma44(cD, F[v], 0.0) + u4 * sff[3][v][s];
        } else {
            double t[5];
            for (int v = 0; v < 5; ++v) t[v] = mfma44(cD, F[v], 0.0) + u4 * sff[2][v][s];
            __syncthreads();  // the gradients are consumed: their space takes the exchange
            for (int v = 0; v < 5; ++v) U.c.tr[v][ny] = t[v];
            __syncthreads();
            for (int v = 0; v < 5; ++v) div[v] += U.c.tr[v][nz];
        }
    }
    // source and the stage combination with the partial residual (operands
    // loaded before the first store: the outputs may alias them)
    const bool rk = S_.mode != 0;
    const bool useA = rk && S_.c0 != 0.0, useT = rk && S_.Tout != nullptr, useB = useT && S_.d0 != 0.0;
    double gq[4], av[5], bv[5];
    for (int c = 0; c < 4; ++c) gq[c] = G.solgeo[(e * 13 + 9 + c) * NP + l];
    for (int v = 0; v < 5; ++v) {
        const int64_t gi = ((int64_t)v * E + e) * NP + l;
        av[v] = useA ? S_.A[gi] : 0.0;
        bv[v] = useB ? S_.B[gi] : 0.0;
    }
    double qn[5];
    for (int v = 0; v < 5; ++v) qn[v] = sq[v][nz];
    const double g[3] = {P.GM * gq[1], P.GM * gq[2], P.GM * gq[3]};
    for (int v = 0; v < 5; ++v) {
        const double R = -div[v] * gq[0] - source64(v, qn[0], qn[1], qn[2], qn[3], g, P.omega);
        const int64_t gi = ((int64_t)v * E + e) * NP + l;
        if (!rk) {
            S_.Qout[gi] = R;
            continue;
        }
        if (useT) S_.Tout[gi] = S_.d0 * bv[v] + S_.d1 * (qn[v] + S_.d2 * R);
        S_.Qout[gi] = S_.c0 * av[v] + S_.c1 * (qn[v] + S_.c2 * R);
    }
}

// Lift pass: the neighbours' viscous halves at interior interface points
// enter the divergence through the end columns of the derivative matrix;
// -(1/|J|) times that lift is added in place to the flux pass's outputs
// with their stage weights (Qout: c1 c2, Tout: d1 d2; residual mode: 1);
// the face traces of the new state are pushed to the neighbours.
// NV: components per mailbox point (4: momentum and energy; 5 with the
// subgrid flux, whose mass part need not vanish)
template <int N, int EPB, int NT, int NV>
__global__ __launch_bounds__(NT) void k_lift64(Ops<N> opa, Geo G, const double *__restrict__ TV, StageArgs S_) {
    constexpr int NP = N * N * N, NF2 = N * N, MBE = 6 * NV * NF2;
    constexpr int IT_MB = (EPB * MBE + NT - 1) / NT, IT_SOL = (EPB * NP + NT - 1) / NT;
    __shared__ double nv[EPB][6][NV][NF2];  // neighbours' viscous flux at own face points, 0 off interfaces
    __shared__ double sq[EPB][5][NP];      // the new state, for the traces
    __shared__ int32_t lk[EPB][6], inf[EPB][6];
    __shared__ Ops<N> op;
    // blocks walk the elements from the last to the first: the flux pass
    // before ran from the first to the last, so the first blocks here read
    // its latest writes, which are still in the memory-side cache; the next
    // flux pass starts where this pass ends, for the same reason
    const int64_t e0 = (int64_t)(gridDim.x - 1 - blockIdx.x) * EPB, E = G.E;
    const bool useT = S_.mode != 0 && S_.Tout != nullptr;
    // every global input first (unpredicated, clamped; the mailbox slots of
    // boundary faces are never written and are selected away below)
    BlockTables<EPB, NT, double, N> bt;
    bt.load(opa, G.link, G.info, e0, E);
    double mb[IT_MB];
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = threadIdx.x + k * NT;
        const bool ok = it < EPB * MBE && e0 + it / MBE < E;
        mb[k] = ld_once(&TV[ok ? e0 * MBE + it : 0]);
    }
    double qo[IT_SOL][5], to[IT_SOL][5], iJ[IT_SOL], r0[IT_SOL][5];
    const bool bal = S_.R0 != nullptr;
#pragma unroll
    for (int k = 0; k < IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        const int el = it / NP, p = it % NP;
        const int64_t e = (it < EPB * NP && e0 + el < E) ? e0 + el : 0;
        iJ[k] = ld_once(&G.solgeo[(e * 13 + 9) * NP + p]);
        for (int v = 0; v < 5; ++v) {
            const int64_t gi = ((int64_t)v * E + e) * NP + p;
            qo[k][v] = S_.Qout[gi];
            to[k][v] = useT ? S_.Tout[gi] : 0.0;
            r0[k][v] = bal ? S_.R0[gi] : 0.0;
        }
    }
    bt.store(op, &lk[0][0], &inf[0][0]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * MBE) break;
        const int el = it / MBE, r = it % MBE, f = r / (NV * NF2);
        (&nv[el][0][0][0])[r] = (lk[el][f] >= 0) ? mb[k] : 0.0;
    }
    __syncthreads();
    const double wP = (S_.mode == 0) ? 1.0 : S_.c1 * S_.c2, wT = S_.d1 * S_.d2;
#pragma unroll
    for (int k = 0; k < IT_SOL; ++k) {
        const int it = threadIdx.x + k * NT;
        if (it >= EPB * NP) break;
        const int el = it / NP, p = it % NP;
        const int64_t e = e0 + el;
        if (e >= E) continue;
        double corr[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            int a, t1, t2;
            split_sol<N>(d, p, a, t1, t2);
            const int pp = t1 + N * t2;
            const double wl = -0.5 * op.D[a][0], wu = 0.5 * op.D[a][N];
#pragma unroll
            for (int v = 0; v < NV; ++v)
                corr[v + 5 - NV] += wl * nv[el][2 * d][v][pp] + wu * nv[el][2 * d + 1][v][pp];
        }
        for (int v = 0; v < 5; ++v) {
            const int64_t gi = ((int64_t)v * E + e) * NP + p;
            const double x = -iJ[k] * corr[v];
            // balanced mode: the background residual leaves R after the
            // lift (at Q = Q0 a residual call then gives exactly zero)
            const double qn = bal ? (qo[k][v] + wP * x) - wP * r0[k][v] : qo[k][v] + wP * x;
            S_.Qout[gi] = qn;
            if (useT) S_.Tout[gi] = bal ? (to[k][v] + wT * x) - wT * r0[k][v] : to[k][v] + wT * x;
            sq[el][v][lds_sol<N>(p)] = qn;
        }
    }
    if (S_.mode == 0 || S_.TQout == nullptr) return;
    __syncthreads();
    push_traces64<N, EPB, NT>(op, G, e0, lk, inf, sq, S_.TQout);
}

// ---------------------------------------------------------------------------
// wide passes: one element per block, the work of a phase spread over all
// threads of the block
// ---------------------------------------------------------------------------
// On a small mesh a pass lasts as long as one block: the passes above walk
// the phases of their elements in turn with one or a few waves, which fills
// the chip when there are blocks for every wave slot but leaves most of it
// idle when there are not.  Here a thread takes one variable of one solution
// point (gradients, divergence, update) or one flux point (all three
// directions and the faces at once; the fluxes of the three directions are
// held in LDS together), so a phase is one round and the chain of a block is
// a third as long: flux and lift pass of the 288-hex order-3 shell 12.7 + 4.8
// -> 7.4 + 4.0 us, ten SSP-RK3 steps 531 -> 326 us; 306 us with the records of
// the element pass for the state and gradients and the early table loads.  The price is in the
// larger meshes: fewer elements in flight per CU and the solution-point
// metrics read by five threads instead of one.  The sums run over the same
// terms in the same order.
template <int N>
struct Wide {
    static constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N, NINT = 3 * (N - 1) * N * N;
    static constexpr int NT = N == 2 ? 64 : N == 3 ? 192 : N == 4 ? 320 : N == 5 ? 640 : 768;
    static constexpr int NFACE = 6 * NF2;
    // first thread of the interior flux points: the face points keep waves
    // of their own (their work differs) where the block has threads for it
    static constexpr int FP = (NFACE + 63) / 64 * 64 + NINT <= NT ? (NFACE + 63) / 64 * 64 : NFACE;
    static constexpr int IT_VP = (5 * NP + NT - 1) / NT;
};

template <int N, bool RAD>
__global__ __launch_bounds__(Wide<N>::NT, 4) void k_flux64_wide(Ops<N> opa, Geo G, PhysParams P,
                                                             const double *__restrict__ Q,
                                                             const double *__restrict__ TQ, double *__restrict__ TV,
                                                             StageArgs S_) {
    using W = Wide<N>;
    static_assert(W::NFACE <= W::NT && W::FP + W::NINT <= W::NT, "one flux point per thread");
    constexpr int NP = W::NP, NF2 = W::NF2, NFL = W::NFL, NT = W::NT;
    constexpr int SR = 22;
    __shared__ alignas(16) double rec[NP][SR];
    __shared__ union {
        double sqs[6][5][NF2];
        double sft[3][5][NFL];  // written after the common solution is consumed
    } U;
    __shared__ int32_t lk[6], inf[6];
    __shared__ alignas(16) Ops<N> op;
    const int64_t e = blockIdx.x, E = G.E;
    const int t = threadIdx.x;
    // this thread's flux point: face point (f, pp) or interior point (d, m, tt)
    const bool isf = t < W::NFACE, isi = t >= W::FP && t < W::FP + W::NINT;
    const int f = isf ? t / NF2 : 0, pp = isf ? t % NF2 : 0;
    const int ii = isi ? t - W::FP : 0, dq = ii / ((N - 1) * NF2), iq = ii % ((N - 1) * NF2);
    const int d = isf ? f >> 1 : dq, m = isf ? ((f & 1) ? N : 0) : 1 + iq % (N - 1), tt = isf ? pp : iq / (N - 1);
    const int fl = m + (N + 1) * tt;
    BlockTables<1, NT, double, N> bt;
    bt.load(opa, G.link, G.info, e, E);
    // every global input before the first wait (unpredicated, clamped)
    double qv[W::IT_VP], Gm[W::IT_VP][9], nq[5], S[3];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        qv[k] = Q[((int64_t)v * E + e) * NP + p];
        for (int c = 0; c < 9; ++c) Gm[k][c] = G.solgeo[(e * 13 + c) * NP + p];
    }
    for (int v = 0; v < 5; ++v) nq[v] = TQ[((e * 6 + f) * 5 + v) * NF2 + pp];
    const double sg = (isf && !(f & 1)) ? -1.0 : 1.0;
    for (int c = 0; c < 3; ++c) S[c] = sg * G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
    const double rl = RAD ? G.rflux[(e * 3 + d) * NFL + fl] : 0.0;
    bt.store(op, lk, inf);
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it < 5 * NP) rec[it % NP][it / NP] = qv[k];
    }
    __syncthreads();
    if (isf) {
        double qs[5];
        common_point64<N>(op, Records<N, SR>{rec}, f, pp, lk[f], inf[f], nq, S, P, qs);
        for (int v = 0; v < 5; ++v) U.sqs[f][v][pp] = qs[v];
    }
    __syncthreads();
    // gradient of one variable at one solution point
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        double dd[3];
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
            int a, t1, t2;
            split_sol<N>(dir, p, a, t1, t2);
            const int base = sol_of<N>(dir, 0, t1, t2), st = stride_of<N>(dir), q = t1 + N * t2;
            double s = op.D[a][0] * U.sqs[2 * dir][v][q] + op.D[a][N] * U.sqs[2 * dir + 1][v][q];
#pragma unroll
            for (int b = 0; b < N; ++b) s += op.B[a][b] * rec[base + b * st][v];
            dd[dir] = s;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            rec[p][5 + v * 3 + c] = Gm[k][c] * dd[0] + Gm[k][3 + c] * dd[1] + Gm[k][6 + c] * dd[2];
    }
    __syncthreads();
    // every flux point of the element at once
    const double kr = RAD ? kappa_r_at(P, rl) : P.kappa_r;
    if (isf) {
        double ffc[5];
        face_point64<N, false>(op, Records<N, SR>{rec}, nullptr, f, pp, lk[f], inf[f], nq, S, P, kr, TV, ffc);
        for (int v = 0; v < 5; ++v) U.sft[d][v][fl] = sg * ffc[v];
    } else if (isi) {
        double fi[5];
        interior_point64<N, false>(op, Records<N, SR>{rec}, nullptr, d, m, tt, S, P, kr, fi);
        for (int v = 0; v < 5; ++v) U.sft[d][v][fl] = fi[v];
    }
    __syncthreads();
    // divergence, source and stage combination of one variable at one
    // solution point (operands loaded before the first store)
    const bool rk = S_.mode != 0;
    const bool useA = rk && S_.c0 != 0.0, useT = rk && S_.Tout != nullptr, useB = useT && S_.d0 != 0.0;
    double gq[W::IT_VP][4], av[W::IT_VP], bv[W::IT_VP];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        for (int c = 0; c < 4; ++c) gq[k][c] = G.solgeo[(e * 13 + 9 + c) * NP + p];
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        av[k] = useA ? S_.A[gi] : 0.0;
        bv[k] = useB ? S_.B[gi] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        double div = 0.0;
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
            int a, t1, t2;
            split_sol<N>(dir, p, a, t1, t2);
            const int fb = (N + 1) * (t1 + N * t2);
            double s = 0.0;
#pragma unroll
            for (int mm = 0; mm <= N; ++mm) s += op.D[a][mm] * U.sft[dir][v][fb + mm];
            div += s;
        }
        const double g[3] = {P.GM * gq[k][1], P.GM * gq[k][2], P.GM * gq[k][3]};
        const double R = -div * gq[k][0] - source64(v, rec[p][0], rec[p][1], rec[p][2], rec[p][3], g, P.omega);
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        if (!rk) {
            S_.Qout[gi] = R;
            continue;
        }
        const double q = rec[p][v];
        if (useT) S_.Tout[gi] = S_.d0 * bv[k] + S_.d1 * (q + S_.d2 * R);
        S_.Qout[gi] = S_.c0 * av[k] + S_.c1 * (q + S_.c2 * R);
    }
}

// face traces of an element's state (LDS) pushed to the neighbours, one
// variable of one face point per thread and round
template <int N>
__device__ __forceinline__ void push_traces64_wide(const Ops<N> &op, const int32_t *lk, const int32_t *inf,
                                                   const double (*sq)[N * N * N], double *__restrict__ TQout) {
    constexpr int NF2 = N * N;
    for (int it = threadIdx.x; it < 30 * NF2; it += Wide<N>::NT) {
        const int v = it / (6 * NF2), r = it % (6 * NF2), f = r / NF2, pp = r % NF2;
        const int32_t nb = lk[f];
        if (nb < 0) continue;
        const int d = f >> 1, m = (f & 1) ? N : 0;
        const double tr = line_interp_s<N>(op, sq[v], m, sol_of<N>(d, 0, pp % N, pp / N), stride_of<N>(d));
        st_once(TQout + mailbox_slot<N>(nb, inf[f], pp) + v * NF2, tr);
    }
}

template <int N>
__global__ __launch_bounds__(Wide<N>::NT) void k_trace_push_wide(Ops<N> opa, Geo G, const double *__restrict__ Q,
                                                                 double *__restrict__ TQ) {
    constexpr int NP = N * N * N;
    __shared__ double sq[5][NP];
    __shared__ int32_t lk[6], inf[6];
    __shared__ Ops<N> op;
    const int64_t e = blockIdx.x;
    BlockTables<1, Wide<N>::NT, double, N> bt;
    bt.load(opa, G.link, G.info, e, G.E);
    for (int it = threadIdx.x; it < 5 * NP; it += Wide<N>::NT)
        sq[it / NP][lds_sol<N>(it % NP)] = Q[((int64_t)(it / NP) * G.E + e) * NP + it % NP];
    bt.store(op, lk, inf);
    __syncthreads();
    push_traces64_wide<N>(op, lk, inf, sq, TQ);
}

template <int N, int NV>
__global__ __launch_bounds__(Wide<N>::NT) void k_lift64_wide(Ops<N> opa, Geo G, const double *__restrict__ TV,
                                                             StageArgs S_) {
    using W = Wide<N>;
    constexpr int NP = W::NP, NF2 = W::NF2, NT = W::NT, MBE = 6 * NV * NF2, IT_MB = (MBE + NT - 1) / NT;
    __shared__ double nv[6][NV][NF2];  // neighbours' viscous flux at own face points, 0 off interfaces
    __shared__ double sq[5][NP];       // the new state, for the traces
    __shared__ int32_t lk[6], inf[6];
    __shared__ Ops<N> op;
    const int64_t e = blockIdx.x, E = G.E;
    const int t = threadIdx.x;
    const bool useT = S_.mode != 0 && S_.Tout != nullptr, bal = S_.R0 != nullptr;
    BlockTables<1, W::NT, double, N> bt;
    bt.load(opa, G.link, G.info, e, E);
    // every global input first (unpredicated, clamped; the mailbox slots of
    // boundary faces are never written and are selected away below)
    double mb[IT_MB];
    int32_t ml[IT_MB];
#pragma unroll
    for (int k = 0; k < IT_MB; ++k) {
        const int it = t + k * NT < MBE ? t + k * NT : 0;
        mb[k] = ld_once(&TV[e * MBE + it]);
        ml[k] = G.link[e * 6 + it / (NV * NF2)];
    }
    double qo[W::IT_VP], to[W::IT_VP], iJ[W::IT_VP], r0[W::IT_VP];
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT < 5 * NP ? t + k * NT : 0, v = it / NP, p = it % NP;
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        iJ[k] = G.solgeo[(e * 13 + 9) * NP + p];
        qo[k] = S_.Qout[gi];
        to[k] = useT ? S_.Tout[gi] : 0.0;
        r0[k] = bal ? S_.R0[gi] : 0.0;
    }
    bt.store(op, lk, inf);
#pragma unroll
    for (int k = 0; k < IT_MB; ++k)
        if (t + k * NT < MBE) (&nv[0][0][0])[t + k * NT] = (ml[k] >= 0) ? mb[k] : 0.0;
    __syncthreads();
    const double wP = (S_.mode == 0) ? 1.0 : S_.c1 * S_.c2, wT = S_.d1 * S_.d2;
#pragma unroll
    for (int k = 0; k < W::IT_VP; ++k) {
        const int it = t + k * NT;
        if (it >= 5 * NP) break;
        const int v = it / NP, p = it % NP;
        double corr = 0.0;
        if (v >= 5 - NV) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                int a, t1, t2;
                split_sol<N>(d, p, a, t1, t2);
                const int pp = t1 + N * t2;
                const double wl = -0.5 * op.D[a][0], wu = 0.5 * op.D[a][N];
                corr += wl * nv[2 * d][v - (5 - NV)][pp] + wu * nv[2 * d + 1][v - (5 - NV)][pp];
            }
        }
        const int64_t gi = ((int64_t)v * E + e) * NP + p;
        const double x = -iJ[k] * corr;
        // (balanced mode as in k_lift64)
        const double qn = bal ? (qo[k] + wP * x) - wP * r0[k] : qo[k] + wP * x;
        S_.Qout[gi] = qn;
        if (useT) S_.Tout[gi] = bal ? (to[k] + wT * x) - wT * r0[k] : to[k] + wT * x;
        sq[v][lds_sol<N>(p)] = qn;
    }
    if (S_.mode == 0 || S_.TQout == nullptr) return;
    __syncthreads();
    push_traces64_wide<N>(op, lk, inf, sq, S_.TQout);
}

// entropy gradient of a state at rest along the flux-point metric:
// out[e][d][fl] = grad S . (|J| grad xi_d) at the d-flux points, with the BR1
// gradients of the FP64 path (S = c_p ln(p^(1/gamma)/rho), p = (gamma-1) E
// for zero momentum); used by the mixed-precision path
template <int N, int EPB, int NT>
__global__ __launch_bounds__(NT) void k_bg_entropy(Ops<N> opa, Geo G, PhysParams P, const double *__restrict__ Q0,
                                                   const double *__restrict__ TQ, float *__restrict__ out,
                                                   float *__restrict__ gout) {
    constexpr int NP = N * N * N, NF2 = N * N, NFL = (N + 1) * N * N;
    __shared__ double sq[EPB][5][NP];
    __shared__ double sqs[EPB][6][5][NF2];
    __shared__ double sgr[EPB][15][NP];
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    __shared__ Ops<N> op;
    ops_to_lds(opa, op);
    load_q<N, EPB, NT>(Q0, G.E, e0, sq);
    __syncthreads();
    common_solution<N, EPB, NT>(op, G, P, TQ, e0, sq, sqs);
    __syncthreads();
    gradients<N, EPB, NT>(op, G, e0, sq, sqs, sgr);
    __syncthreads();
    // gradient of rho0 at the solution points: gout[e][3][NP]
    for (int it = threadIdx.x; it < EPB * 3 * NP; it += NT) {
        const int el = it / (3 * NP), r = it % (3 * NP), k = r / NP, p = r % NP;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        gout[(e * 3 + k) * NP + p] = (float)sgr[el][k][p];
    }
    const double gm1 = P.gamma - 1.0;
    for (int it = threadIdx.x; it < EPB * 3 * NFL; it += NT) {
        const int el = it / (3 * NFL), r = it % (3 * NFL), d = r / NFL, fl = r % NFL;
        const int64_t e = e0 + el;
        if (e >= G.E) continue;
        const int m = fl % (N + 1), t1 = (fl / (N + 1)) % N, t2 = fl / ((N + 1) * N);
        const int base = sol_of<N>(d, 0, t1, t2), st = stride_of<N>(d);
        double rho = 0.0, E = 0.0, gr = 0.0, gE = 0.0;
        for (int b = 0; b < N; ++b) {
            const double w = op.I[m][b];
            rho += w * sq[el][0][base + b * st];
            E += w * sq[el][4][base + b * st];
        }
        for (int c = 0; c < 3; ++c) {
            const double S = G.fluxgeo[((e * 3 + d) * 3 + c) * NFL + fl];
            double a = 0.0, b2 = 0.0;
            for (int b = 0; b < N; ++b) {
                const double w = op.I[m][b];
                a += w * sgr[el][0 * 3 + c][base + b * st];
                b2 += w * sgr[el][4 * 3 + c][base + b * st];
            }
            gr += a * S;
            gE += b2 * S;
        }
        const double p = gm1 * E;
        out[(e * 3 + d) * NFL + fl] = (float)(P.cp * (gm1 * gE / (P.gamma * p) - gr / rho));
    }
}

// fixed-order partial sums of w w w |J| Q_v over element blocks
template <int NT>
__global__ __launch_bounds__(NT) void k_sums_partial(const double *__restrict__ Q,
                                                     const double *__restrict__ solw, int64_t n,
                                                     int64_t chunk, double *__restrict__ part) {
    __shared__ double red[NT];
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = (lo + chunk < n) ? lo + chunk : n;
    for (int v = 0; v < 5; ++v) {
        double s = 0.0;
        for (int64_t i = lo + threadIdx.x; i < hi; i += NT) s += solw[i] * Q[(int64_t)v * n + i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = NT / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) part[(int64_t)v * gridDim.x + blockIdx.x] = red[0];
        __syncthreads();
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_sums_final(const double *__restrict__ part, int nb, int rows,
                                                   double *__restrict__ out) {
    __shared__ double red[NT];
    for (int v = 0; v < rows; ++v) {
        double s = 0.0;
        for (int i = threadIdx.x; i < nb; i += NT) s += part[(int64_t)v * nb + i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = NT / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[v] = red[0];
        __syncthreads();
    }
}

// angular momentum L = sum w|J| x cross m and the diagonal moments of
// inertia I_c = sum w|J| rho (|x|^2 - x_c^2) (Section 6): block partials
// part[q][block], q = Lx, Ly, Lz, Ix, Iy, Iz, over contiguous chunks of
// solution points, fixed tree order
template <int NT>
__global__ __launch_bounds__(NT) void k_am_partial(const double *__restrict__ Q, const double *__restrict__ solw,
                                                   const double *__restrict__ xsol, int64_t E, int NP,
                                                   int64_t chunk, double *__restrict__ part) {
    __shared__ double red[6][NT];
    const int64_t n = E * NP;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = (lo + chunk < n) ? lo + chunk : n;
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t i = lo + threadIdx.x; i < hi; i += NT) {
        const int64_t e = i / NP, p = i % NP;
        const double x = xsol[(e * 3 + 0) * NP + p], y = xsol[(e * 3 + 1) * NP + p], z = xsol[(e * 3 + 2) * NP + p];
        const double w = solw[i], rho = Q[i], mx = Q[n + i], my = Q[2 * n + i], mz = Q[3 * n + i];
        s[0] += w * (y * mz - z * my);
        s[1] += w * (z * mx - x * mz);
        s[2] += w * (x * my - y * mx);
        s[3] += w * rho * (y * y + z * z);
        s[4] += w * rho * (x * x + z * z);
        s[5] += w * rho * (x * x + y * y);
    }
    for (int q = 0; q < 6; ++q) red[q][threadIdx.x] = s[q];
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 6; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 6) part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = red[threadIdx.x][0];
}

// u <- u - dOmega x x at fixed rho and pressure (E changes by the kinetic
// energy change)
__global__ void k_am_apply(double *__restrict__ Q, const double *__restrict__ xsol, int64_t E, int NP, double dx,
                           double dy, double dz) {
    const int64_t n = E * NP;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t e = i / NP, p = i % NP;
    const double x = xsol[(e * 3 + 0) * NP + p], y = xsol[(e * 3 + 1) * NP + p], z = xsol[(e * 3 + 2) * NP + p];
    const double rho = Q[i];
    const double u = Q[n + i] / rho, v = Q[2 * n + i] / rho, w = Q[3 * n + i] / rho;
    const double un = u - (dy * z - dz * y), vn = v - (dz * x - dx * z), wn = w - (dx * y - dy * x);
    const double dke = 0.5 * rho * ((un * un + vn * vn + wn * wn) - (u * u + v * v + w * w));
    Q[n + i] = rho * un;
    Q[2 * n + i] = rho * vn;
    Q[3 * n + i] = rho * wn;
    Q[4 * n + i] += dke;
}

// non-finite / non-positive density or pressure check: flag[0] set to 1
__global__ void k_check(const double *__restrict__ Q, int64_t n, double gm1, int *__restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double r = Q[i], mx = Q[n + i], my = Q[2 * n + i], mz = Q[3 * n + i], E = Q[4 * n + i];
    const double p = gm1 * (E - 0.5 * (mx * mx + my * my + mz * mz) / r);
    const bool ok = (r > 0.0) && (p > 0.0) && (r < 1e300) && (p < 1e300) && (mx == mx) && (my == my) &&
                    (mz == mz);
    if (!ok) flag[0] = 1;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
template <int N>
static Ops<N> make_ops(const Basis1D &b) {
    return make_ops_t<double, N>(b);
}

// elements per block / threads per block for each order
template <int N>
struct Cfg;
template <> struct Cfg<2> { static constexpr int EPB = 8, NT = 64; };
template <> struct Cfg<3> { static constexpr int EPB = 2, NT = 64; };
template <> struct Cfg<4> { static constexpr int EPB = 1, NT = 64; };
template <> struct Cfg<5> { static constexpr int EPB = 1, NT = 128; };
template <> struct Cfg<6> { static constexpr int EPB = 1, NT = 256; };

template <int N>
static hipError_t launch_trace_t(const Mesh &m, const Geo &G, const double *Q, double *TQ, hipStream_t s) {
    constexpr int EPB = Cfg<N>::EPB, NT = Cfg<N>::NT;
    const Ops<N> op = make_ops<N>(m.basis);
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((k_trace<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, op, G, Q, TQ);
    return hipGetLastError();
}

// Largest meshes, in elements per CU, that run the wide passes: where
// an SSP-RK3 step of a shell was no slower with them (us per step, element
// passes / wide passes; the flux pass of order 4 is k_flux64_n4):
//   flux  order 2: 53.8 / 47.1 at 3,600 hexes, 58.3 / 58.9 at 5,184
//         order 3: 43.1 / 30.5 at 288, 68.0 / 63.8 at 2,304, 77.9 / 87.7 at 3,600
//         order 4: 34.4 / 29.5 at 162, 35.5 / 38.4 at 288
//         order 5: 47.5 / 38.0 at 162, 59.7 / 58.9 at 288, 77.5 / 86.6 at 648
//         order 6: 59.4 / 59.4 at 162, 82.2 / 101.6 at 288 (not used)
//   lift and trace push
//         order 2: 74.1 / 70.3 at 7,776, 95.0 / 99.4 at 12,288
//         order 3: 77.8 / 75.5 at 2,304, 89.0 / 103.5 at 3,600
//         order 4: 64.8 / 62.9 at 1,536, 84.3 / 85.5 at 2,304
//         order 5: 83.4 / 80.7 at 648, 126.2 / 126.6 at 1,080
//         order 6: 111.7 / 109.2 at 648, 168.8 / 167.8 at 1,080
template <int N>
constexpr int kWideFlux64 = N == 2 ? 16 : N == 3 ? 9 : N == 6 ? 0 : 1;
template <int N>
static bool wide_lift64(const Mesh &m) {
    constexpr int per_cu = N == 2 ? 32 : N == 3 ? 10 : N == 4 ? 7 : 3;
    return m.E <= kCUs * per_cu;
}

template <int N>
static hipError_t launch_trace_push_t(const Mesh &m, const Geo &G, const double *Q, double *TQ, hipStream_t s) {
    if (wide_lift64<N>(m)) {
        hipLaunchKernelGGL((k_trace_push_wide<N>), dim3((unsigned)m.E), dim3(Wide<N>::NT), 0, s, make_ops<N>(m.basis), G,
                           Q, TQ);
        return hipGetLastError();
    }
    constexpr int EPB = Cfg64<N>::EPB, NT = Cfg64<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((k_trace_push<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, Q, TQ);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_flux64_t(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q,
                                  const double *TQ, double *TV, const StageArgs &sa, const ClosureArgs &C,
                                  hipStream_t s) {
    constexpr int EPB = Cfg64<N>::EPB, NT = Cfg64<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    const bool rad = P.kappa_r1 != 0.0 || P.kappa_r2 != 0.0;
    if (C.model) {
        // the flux pass with the network inside
        if constexpr (N == 3) {
            if (rad)
                hipLaunchKernelGGL((k_flux64<N, EPB, NT, 2, true>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis),
                                   G, P, Q, TQ, TV, sa, C);
            else
                hipLaunchKernelGGL((k_flux64<N, EPB, NT, 2, false>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis),
                                   G, P, Q, TQ, TV, sa, C);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    if constexpr (kWideFlux64<N> > 0) {
        if (m.E <= kCUs * kWideFlux64<N>) {
            if (rad)
                hipLaunchKernelGGL((k_flux64_wide<N, true>), dim3((unsigned)m.E), dim3(Wide<N>::NT), 0, s,
                                   make_ops<N>(m.basis), G, P, Q, TQ, TV, sa);
            else
                hipLaunchKernelGGL((k_flux64_wide<N, false>), dim3((unsigned)m.E), dim3(Wide<N>::NT), 0, s,
                                   make_ops<N>(m.basis), G, P, Q, TQ, TV, sa);
            return hipGetLastError();
        }
    }
    if constexpr (N == 4) {
        if (rad)
            hipLaunchKernelGGL((k_flux64_n4<true>), dim3((unsigned)m.E), dim3(64), 0, s, make_ops<4>(m.basis), G, P, Q,
                               TQ, TV, sa);
        else
            hipLaunchKernelGGL((k_flux64_n4<false>), dim3((unsigned)m.E), dim3(64), 0, s, make_ops<4>(m.basis), G, P,
                               Q, TQ, TV, sa);
    } else if (rad) {
        hipLaunchKernelGGL((k_flux64<N, EPB, NT, 0, true>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, P, Q,
                           TQ, TV, sa, C);
    } else {
        hipLaunchKernelGGL((k_flux64<N, EPB, NT, 0, false>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, P, Q,
                           TQ, TV, sa, C);
    }
    return hipGetLastError();
}

template <int N>
static hipError_t launch_lift64_t(const Mesh &m, const Geo &G, const double *TV, const StageArgs &sa, bool closure,
                                  hipStream_t s) {
    constexpr int EPB = Cfg64<N>::EPB, NT = Cfg64<N>::NT;
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    if (wide_lift64<N>(m)) {
        if (closure)
            hipLaunchKernelGGL((k_lift64_wide<N, 5>), dim3((unsigned)m.E), dim3(Wide<N>::NT), 0, s, make_ops<N>(m.basis),
                               G, TV, sa);
        else
            hipLaunchKernelGGL((k_lift64_wide<N, 4>), dim3((unsigned)m.E), dim3(Wide<N>::NT), 0, s, make_ops<N>(m.basis),
                               G, TV, sa);
        return hipGetLastError();
    }
    if (closure)
        hipLaunchKernelGGL((k_lift64<N, EPB, NT, 5>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, TV, sa);
    else
        hipLaunchKernelGGL((k_lift64<N, EPB, NT, 4>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, TV, sa);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_features_t(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q,
                                    const double *TQ, float *X, hipStream_t s) {
    constexpr int EPB = Cfg<N>::EPB, NT = Cfg<N>::NT;
    const Ops<N> op = make_ops<N>(m.basis);
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((k_features<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, op, G, P, Q, TQ, X);
    return hipGetLastError();
}

#define CHORUS_DISPATCH(N_, CALL)            \
    switch (N_) {                            \
        case 2: return CALL(2);              \
        case 3: return CALL(3);              \
        case 4: return CALL(4);              \
        case 5: return CALL(5);              \
        case 6: return CALL(6);              \
        default: return hipErrorInvalidValue; \
    }

hipError_t launch_trace(const Mesh &m, const Geo &G, const double *Q, double *TQ, hipStream_t s) {
#define C_(n) launch_trace_t<n>(m, G, Q, TQ, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}
template <int N>
static hipError_t launch_closure_tau_t(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q,
                                       const double *TQ, const ClosureArgs &C, hipStream_t s) {
    if constexpr (N == 3) {
        constexpr int EPB = Cfg64<N>::EPB, NT = Cfg64<N>::NT;
        const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
        const StageArgs none{nullptr, nullptr, nullptr, 0.0, 0.0, 0.0, nullptr, nullptr, 0.0, 0.0, 0.0, 0};
        hipLaunchKernelGGL((k_flux64<N, EPB, NT, 1, false>), dim3(nb), dim3(NT), 0, s, make_ops<N>(m.basis), G, P, Q,
                           TQ, nullptr, none, C);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

hipError_t launch_closure_tau(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q, const double *TQ,
                              const ClosureArgs &C, hipStream_t s) {
#define C_(n) launch_closure_tau_t<n>(m, G, P, Q, TQ, C, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}
hipError_t launch_trace_push(const Mesh &m, const Geo &G, const double *Q, double *TQ, hipStream_t s) {
#define C_(n) launch_trace_push_t<n>(m, G, Q, TQ, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}
hipError_t launch_flux64(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q, const double *TQ,
                         double *TV, const StageArgs &sa, const ClosureArgs &C, hipStream_t s) {
#define C_(n) launch_flux64_t<n>(m, G, P, Q, TQ, TV, sa, C, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}
hipError_t launch_lift64(const Mesh &m, const Geo &G, const double *TV, const StageArgs &sa, bool closure,
                         hipStream_t s) {
#define C_(n) launch_lift64_t<n>(m, G, TV, sa, closure, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}
hipError_t launch_features(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q, const double *TQ,
                           float *X, hipStream_t s) {
#define C_(n) launch_features_t<n>(m, G, P, Q, TQ, X, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}

template <int N>
static hipError_t launch_bg_entropy_t(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q0,
                                      const double *TQ, float *out, float *gout, hipStream_t s) {
    constexpr int EPB = Cfg<N>::EPB, NT = Cfg<N>::NT;
    const Ops<N> op = make_ops<N>(m.basis);
    const unsigned nb = (unsigned)((m.E + EPB - 1) / EPB);
    hipLaunchKernelGGL((k_bg_entropy<N, EPB, NT>), dim3(nb), dim3(NT), 0, s, op, G, P, Q0, TQ, out, gout);
    return hipGetLastError();
}

hipError_t launch_bg_entropy(const Mesh &m, const Geo &G, const PhysParams &P, const double *Q0, const double *TQ,
                             float *out, float *gout, hipStream_t s) {
#define C_(n) launch_bg_entropy_t<n>(m, G, P, Q0, TQ, out, gout, s)
    CHORUS_DISPATCH(m.N, C_)
#undef C_
}

hipError_t launch_sums(const double *Q, const double *solw, int64_t n, double *part, int nblocks, double *out,
                       hipStream_t s) {
    const int64_t chunk = (n + nblocks - 1) / nblocks;
    hipLaunchKernelGGL((k_sums_partial<256>), dim3(nblocks), dim3(256), 0, s, Q, solw, n, chunk, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_sums_final<256>), dim3(1), dim3(256), 0, s, part, nblocks, 5, out);
    return hipGetLastError();
}

hipError_t launch_am_sums(const double *Q, const double *solw, const double *xsol, int64_t E, int NP, double *part,
                          int nblocks, double *out, hipStream_t s) {
    const int64_t n = E * NP;
    const int64_t chunk = (n + nblocks - 1) / nblocks;
    hipLaunchKernelGGL((k_am_partial<256>), dim3(nblocks), dim3(256), 0, s, Q, solw, xsol, E, NP, chunk, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_sums_final<256>), dim3(1), dim3(256), 0, s, part, nblocks, 6, out);
    return hipGetLastError();
}

hipError_t launch_am_apply(double *Q, const double *xsol, int64_t E, int NP, const double dO[3], hipStream_t s) {
    const int64_t n = E * NP;
    hipLaunchKernelGGL(k_am_apply, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Q, xsol, E, NP, dO[0], dO[1],
                       dO[2]);
    return hipGetLastError();
}

__global__ void k_clear_flag(int *flag) { flag[0] = 0; }

hipError_t launch_clear_flag(int *flag, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, flag);
    return hipGetLastError();
}

hipError_t launch_check(const double *Q, int64_t n, double gm1, int *flag, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, flag);
    const unsigned nb = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_check, dim3(nb), dim3(256), 0, s, Q, n, gm1, flag);
    return hipGetLastError();
}

}  // namespace chorus
