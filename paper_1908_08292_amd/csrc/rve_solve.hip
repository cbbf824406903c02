// rve_solve.hip -- persistent batched periodic-RVE solver for gfx950.
//
// One workgroup (four wave64; eight in the second compilation, for batches that keep
// every front in global memory) owns one workspace slot and pulls RVE ids from a
// device queue until the batch is exhausted.  Per RVE it runs the
// micro Newton iteration of Sec. 3.3 (residual, tangent, linear solve, update;
// the PBC form in which G^T dLambda = 0), then the post-convergence outputs:
// Pbar = <P> (eq. Average-of-P-and-F) and the tangent transfer of Sec. 3.2 for
// the d^2 unit macro-gradient states, condensed as
//     Abar = <A> - Y^T K_ff^-1 Y = <A> - Z^T D^-1 Z,  Z = L^-1 Y,
// with K_ff = L D L^T the tangent at the converged state (end of Sec. 3.3).
//
// Constitutive law (Sec. 6, neo-Hookean, plane strain in 2D) in first-Piola
// form with Fi = F^-1, g_a = F^-T grad N_a (spatial gradient of N_a),
// c1 = mu - lambda/2 (J^2 - 1), c2 = lambda J^2:
//     P = mu F - c1 F^-T
//     A_iJkL = mu d_ik d_JL + c1 Fi_Jk Fi_Li + c2 Fi_Ji Fi_Lk
//     f_(a,i)       = sum_gp (mu (F grad N_a)_i - c1 g_a,i) w|J|
//     k_(a,i),(b,k) = sum_gp (mu d_ik grad N_a . grad N_b + c1 g_a,k g_b,i + c2 g_a,i g_b,k) w|J|
//     Y_(a,i),(kL)  = sum_gp (mu d_ik dN_a,L + c1 g_a,k Fi_Li + c2 g_a,i Fi_Lk) w|J|
// which equal int B^T S and int B^T C B + S_hat 1 of the paper's eqs. (DG^h,
// G_IK, S_IK) written with P and A = dP/dF.  The two other laws of the paper's
// micro-convergence comparisons (Sec. 6) share one closed form of A with it
// (PointState): St. Venant-Kirchhoff, P = F S with
// S = lambda tr(E) 1 + 2 mu E, A_iJkL = d_ik S_JL + lambda F_iJ F_kL +
// mu (F_iL F_kJ + (F F^T)_ik d_JL); and the fully linear case, P = sigma(eps),
// eps = sym(F - 1), A the constant elasticity tensor.
//
// The linear solve is a multifrontal LDL^T (no pivoting: the tangent can be
// indefinite at the initial guess past a micro-instability of a stiff inclusion)
// driven by the (d, n) plan: element matrices are gathered straight into the
// dense fronts, children's update matrices are extended-added from a stack, the
// forward substitution is fused into the factorization, and the backward
// substitution walks the fronts in reverse.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mesh_common.h"
#include "solver_dev.h"

// Waves per workgroup: four, or eight when compiled with FEHMM_NWAVE=8 into
// namespace fehmm::w8 (batches whose plans all keep their fronts in global memory)
#ifndef FEHMM_NWAVE
#define FEHMM_NWAVE 4
#define FEHMM_VARIANT w4
#endif

namespace fehmm {
namespace FEHMM_VARIANT {

constexpr int NWAVE = FEHMM_NWAVE;
constexpr int NT = 64 * NWAVE;
// plans with panels in LDS run four waves
constexpr bool kLdsPlans = NWAVE == kSolveWaves;
static_assert(NWAVE == 4 || NWAVE == 8, "workgroup size");
static_assert(64 * kSolveWaves / 128 == kStepGroups && kSolveWaves == kStepFronts, "thread groups of a step");

// Optional per-phase clock accounting (slot 0, thread 0), compiled in only
// with -DFEHMM_PHASE_PROF=1; the default build records nothing.
#ifndef FEHMM_PHASE_PROF
#define FEHMM_PHASE_PROF 0
#endif
enum { PH_ELEM, PH_GATHER, PH_ASM, PH_DIAG, PH_TRSM, PH_MFMA, PH_OUT, PH_BACK, PH_LINE, PH_FINAL, PH_TOTAL, PH_N };
#if FEHMM_PHASE_PROF
__device__ unsigned long long g_phase[PH_N];
#define PROF_T0() unsigned long long _pt = clock64()
#define PROF_MARK(ph)                                                        \
    do {                                                                     \
        if (blockIdx.x == 0 && threadIdx.x == 0) {                           \
            unsigned long long _n = clock64();                               \
            g_phase[ph] += _n - _pt;                                         \
            _pt = _n;                                                        \
        }                                                                    \
    } while (0)
#define PROF_RESET() _pt = clock64()
#else
#define PROF_T0()
#define PROF_MARK(ph)
#define PROF_RESET()
#endif

struct Smem {
    double red[NWAVE * 81];
    double dN[8 * 8 * 3];    // [gp][a][k]
    double Fbar[9];
    double outv[96];
    double wJ, atol;
    int flag;
    int rve;
};

__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

// deterministic block reduction of K values per thread; result in sm.outv[0..K)
template <int K>
__device__ inline void block_sum(double (&v)[K], Smem& sm) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double s = wave_sum(v[k]);
        if (lane == 0) sm.red[wave * K + k] = s;
    }
    __syncthreads();
    if (threadIdx.x < K) {
        double s = 0;
        for (int w = 0; w < NWAVE; ++w) s += sm.red[w * K + threadIdx.x];
        sm.outv[threadIdx.x] = s;
    }
    __syncthreads();
}

struct RveCtx {
    const DevPlan* plan;
    int d, n, ne, nn, nen, nd;
    int law;  // RVE_LAW_*: 0 neo-Hookean, 1 St. Venant-Kirchhoff, 2 fully linear
    int elem; // RVE_ELEM_*: 0 Q1 / hex8 with 2^d Gauss points, 1 P1 (d! Kuhn simplices per cell)
    int ke32; // Newton element tangents stored in FP32 (FP32 factors); FP64 at the converged state
    const uint8_t* phase;
    const double* lame;
    double* w;
    double* wt;
    double* R;
    double* rhs;
    double* x;
    double* fe;
    double* ke;
    double* re;
    double* L;
    double* U;
    double* S;
};

// node v holds w = 0: node 0 under periodic coupling, every boundary node
// (some grid index 0) under linear displacements
__device__ inline bool is_pinned(const DevPlan& pl, int v) { return plan_pinned(pl.bc, pl.d, pl.n, v); }

// zero x at the pinned nodes' dofs (node-major [dof][nc]): the triangular
// solves write the free rows only
template <int D>
__device__ inline void zero_pinned(const RveCtx& c, double* x, int nc) {
    const DevPlan& pl = *c.plan;
    if (pl.bc == 0) {
        for (int t = threadIdx.x; t < D * nc; t += NT) x[t] = 0.0;
        return;
    }
    for (int t = threadIdx.x; t < c.nn * D * nc; t += NT)
        if (is_pinned(pl, t / (D * nc))) x[t] = 0.0;
}

// wave-uniform copies of values a non-inlined function receives in vector
// registers: with them the compiler keeps loop bounds and addresses scalar, so
// loops stay uniform and its wait counts across loop edges stay exact
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uni(int64_t v) {
    const uint64_t u = (uint64_t)v;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename P>
__device__ inline P* uni(P* p) {
    return (P*)(uintptr_t)uni((int64_t)(uintptr_t)p);
}

// Address spaces.  The large functions are not inlined into the solver kernel
// and receive generic pointers in vector registers; these views restore what the
// compiler cannot see: workspace pointers are wave-uniform and global (scalar
// bases, 32-bit lane offsets, no flat instructions), the LDS is LDS, and the plan
// is constant while the kernel runs, so wave-uniform reads of it are scalar loads.
#define FEHMM_GLB __attribute__((address_space(1)))
#define FEHMM_LDS __attribute__((address_space(3)))
#define FEHMM_CST __attribute__((address_space(4)))
template <typename T>
__device__ inline FEHMM_GLB T* glb(T* p) {
    return (FEHMM_GLB T*)uni((int64_t)(uintptr_t)p);
}
template <typename S>
__device__ inline S load_const(const FEHMM_GLB S* p) {
    static_assert(sizeof(S) % 4 == 0, "whole words");
    const FEHMM_CST uint32_t* q = (const FEHMM_CST uint32_t*)uni((int64_t)p);
    uint32_t w[sizeof(S) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(S) / 4; ++k) w[k] = q[k];
    S out;
    __builtin_memcpy(&out, w, sizeof(S));
    return out;
}

// Constitutive state at a Gauss point.  For each law the tangent has the form
//     A_iJkL = d_ik S_JL + beta_ik d_JL + a1 M_kJ M_iL + a2 M_iJ M_kL
// neo-Hookean:             S = mu 1, beta = 0,        M = F^-T, a1 = mu - lambda/2 (J^2 - 1), a2 = lambda J^2
// St. Venant-Kirchhoff:    S = S(E), beta = mu F F^T, M = F,    a1 = mu,                      a2 = lambda
// fully linear:            S = mu 1, beta = 0,        M = 1,    a1 = mu,                      a2 = lambda
// so with v_a = M grad N_a, t_a = S grad N_a
//     k_(a,i),(b,k) = d_ik t_a . grad N_b + beta_ik grad N_a . grad N_b + a1 v_a,k v_b,i + a2 v_a,i v_b,k
//     Y_(a,i),(kL)  = d_ik t_a,L + beta_ik dN_a,L + a1 v_a,k M_iL + a2 v_a,i M_kL
//     A : G         = G S + beta G + a1 M G^T M + a2 (M : G) M
// Everything is scaled by the point's weight w|J|.
template <int D>
struct PointState {
    double M[D * D], S[D * D], beta[D * D], P[D * D];
    double a1, a2;
};
// false where J <= 0 (or NaN); beta is set for the St. Venant-Kirchhoff law only
template <int D>
__device__ inline bool point_state(int law, double lam, double mu, double wJ, const double* F, PointState<D>& s) {
    constexpr int D2 = D * D;
    double J, c[D2];  // cofactors: F^-T = c / J
    if constexpr (D == 2) {
        J = F[0] * F[3] - F[1] * F[2];
        c[0] = F[3]; c[1] = -F[2]; c[2] = -F[1]; c[3] = F[0];
    } else {
        c[0] = F[4] * F[8] - F[5] * F[7];
        c[1] = F[5] * F[6] - F[3] * F[8];
        c[2] = F[3] * F[7] - F[4] * F[6];
        c[3] = F[2] * F[7] - F[1] * F[8];
        c[4] = F[0] * F[8] - F[2] * F[6];
        c[5] = F[1] * F[6] - F[0] * F[7];
        c[6] = F[1] * F[5] - F[2] * F[4];
        c[7] = F[2] * F[3] - F[0] * F[5];
        c[8] = F[0] * F[4] - F[1] * F[3];
        J = F[0] * c[0] + F[1] * c[1] + F[2] * c[2];
    }
    if (!(J > 0.0)) return false;
    const double mw = mu * wJ, lw = lam * wJ;
    if (law == 0) {
        const double r = 1.0 / J;
        s.a1 = mw - 0.5 * lw * (J * J - 1.0);
        s.a2 = lw * J * J;
#pragma unroll
        for (int q = 0; q < D2; ++q) {
            s.M[q] = c[q] * r;
            s.P[q] = mw * F[q] - s.a1 * s.M[q];
            s.S[q] = (q % (D + 1)) == 0 ? mw : 0.0;
        }
        return true;
    }
    s.a1 = mw;
    s.a2 = lw;
    if (law == 1) {
        double tr = 0.0;
#pragma unroll
        for (int I = 0; I < D; ++I)
#pragma unroll
            for (int K = 0; K < D; ++K) {
                double g = 0.0, b = 0.0;
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    g += F[k * D + I] * F[k * D + K];
                    b += F[I * D + k] * F[K * D + k];
                }
                g = 0.5 * (g - (I == K ? 1.0 : 0.0));
                if (I == K) tr += g;
                s.S[I * D + K] = 2.0 * mw * g;
                s.beta[I * D + K] = mw * b;
            }
#pragma unroll
        for (int I = 0; I < D; ++I) s.S[I * (D + 1)] += lw * tr;
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int K = 0; K < D; ++K) {
                double v = 0.0;
#pragma unroll
                for (int k = 0; k < D; ++k) v += F[i * D + k] * s.S[k * D + K];
                s.P[i * D + K] = v;
                s.M[i * D + K] = F[i * D + K];
            }
        return true;
    }
    double tr = 0.0;
#pragma unroll
    for (int I = 0; I < D; ++I) tr += F[I * (D + 1)] - 1.0;
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int K = 0; K < D; ++K) {
            const double id = i == K ? 1.0 : 0.0;
            s.P[i * D + K] = mw * (F[i * D + K] + F[K * D + i] - 2.0 * id) + lw * tr * id;
            s.M[i * D + K] = id;
            s.S[i * D + K] = mw * id;
        }
    return true;
}

// t = A : g at a point
template <int D>
__device__ inline void point_apply(int law, const PointState<D>& s, const double* g, double* t) {
    double mg = 0.0, h[D * D];  // M : g; h = g^T M
#pragma unroll
    for (int q = 0; q < D * D; ++q) mg += s.M[q] * g[q];
    mg *= s.a2;
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int J = 0; J < D; ++J) {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) v += g[k * D + i] * s.M[k * D + J];
            h[i * D + J] = v;
        }
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int J = 0; J < D; ++J) {
            double v = mg * s.M[i * D + J], u = 0.0;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                v += g[i * D + k] * s.S[k * D + J];
                u += s.M[i * D + k] * h[k * D + J];
            }
            t[i * D + J] = v + s.a1 * u;
        }
    if (law == 1)
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int J = 0; J < D; ++J)
#pragma unroll
                for (int k = 0; k < D; ++k) t[i * D + J] += s.beta[i * D + k] * g[k * D + J];
}

// What an element pass reads, in scalar registers (the passes are not inlined)
struct ElemCtx {
    int n, ne, law, npt;
    double wJ;
    const FEHMM_GLB uint8_t* phase;
    const FEHMM_GLB double* lame;
    const FEHMM_LDS double* dN;    // [point][node][3]
    const FEHMM_LDS double* Fbar;
    FEHMM_LDS int* flag;
};
template <int D>
__device__ inline ElemCtx elem_ctx(const RveCtx& c, Smem& sm) {
    ElemCtx k;
    k.n = uni(c.n);
    k.ne = uni(c.ne);
    k.law = uni(c.law);
    k.npt = uni(c.elem) == 0 ? (1 << D) : (D == 2 ? 2 : 6);
    k.phase = glb(c.phase);
    k.lame = glb(c.lame);
    k.dN = (const FEHMM_LDS double*)sm.dN;
    k.Fbar = (const FEHMM_LDS double*)sm.Fbar;
    k.flag = (FEHMM_LDS int*)&sm.flag;
    k.wJ = sm.wJ;
    return k;
}

// grid indices of node or element id (id < 2^18: the quotients are exact)
template <int D>
__device__ inline void grid_of(int n, int id, int* c) {
    const float r = 1.0f / (float)n;
#pragma unroll
    for (int k = 0; k + 1 < D; ++k) {
        const int q = (int)(((float)id + 0.5f) * r);
        c[k] = id - q * n;
        id = q;
    }
    c[D - 1] = id;
}
// nodes of element e (numbering of element_nodes, without its divisions)
template <int D>
__device__ inline void nodes_of_element(int n, int e, int* nodes) {
    int c[3];
    grid_of<D>(n, e, c);
    int lo[3], hi[3], s = 1;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        lo[k] = c[k] * s;
        hi[k] = (c[k] + 1 == n ? 0 : c[k] + 1) * s;
        s *= n;
    }
#pragma unroll
    for (int a = 0; a < (1 << D); ++a) {
        int o[3];
        local_offset(D, a, o);
        int id = 0;
#pragma unroll
        for (int k = 0; k < D; ++k) id += o[k] ? hi[k] : lo[k];
        nodes[a] = id;
    }
}
// elements around node v: el[a] is the one in which v is local node a
template <int D>
__device__ inline void elements_of_node(int n, int v, int* el) {
    int c[3];
    grid_of<D>(n, v, c);
    int lo[3], hi[3], s = 1;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        hi[k] = c[k] * s;
        lo[k] = (c[k] == 0 ? n - 1 : c[k] - 1) * s;
        s *= n;
    }
#pragma unroll
    for (int a = 0; a < (1 << D); ++a) {
        int o[3];
        local_offset(D, a, o);
        int id = 0;
#pragma unroll
        for (int k = 0; k < D; ++k) id += o[k] ? lo[k] : hi[k];
        el[a] = id;
    }
}

// Fbar + grad w of an element's nodal values at point gp; Fbar = null: grad w
template <int D>
__device__ inline void grad_at(const ElemCtx& k, const double* wl, int gp, bool with_Fbar, double* F) {
#pragma unroll
    for (int q = 0; q < D * D; ++q) F[q] = with_Fbar ? k.Fbar[q] : 0.0;
#pragma unroll
    for (int b = 0; b < (1 << D); ++b)
#pragma unroll
        for (int J = 0; J < D; ++J) {
            const double dn = k.dN[(gp * 8 + b) * 3 + J];
#pragma unroll
            for (int i = 0; i < D; ++i) F[i * D + J] += wl[b * D + i] * dn;
        }
}
template <int D>
__device__ inline void nodal(const FEHMM_GLB double* x, const int* nodes, double* xl) {
#pragma unroll
    for (int b = 0; b < (1 << D); ++b)
#pragma unroll
        for (int i = 0; i < D; ++i) xl[b * D + i] = x[nodes[b] * D + i];
}

// Element residuals f and symmetric tangents at w, entry planes [entry][element]
// (fe: rows a D + i; ke: sym_entry).  Work items: 2D (element, component i): the
// ten k_(.,i)(.,i) and half of the sixteen k_(.,x)(.,y); 3D (element, node a): the
// blocks of a with a .. a + 3 and, for a < 4, a + 4 (mod 8): each unordered pair of
// nodes once.  Consecutive threads take consecutive elements, so every store is
// contiguous.  Bound by FP64 issue and, in 3D, by registers.  Against one item per
// (element, node[, component]) with full rows of 2^d d entries: a half (2D) to a
// third (3D) of the Gauss-point work and half the stored entries; one pass of a
// workgroup takes 87 instead of 190 kclk at 32 x 32 and 1.3 instead of 7 Mclk at 8^3
// (whose accumulators were in scratch), the batch of 4096 RVEs of 32 x 32 55 instead
// of 64 ms.
template <int D, typename KT>
__device__ __noinline__ void element_tangents(const RveCtx& c, Smem& sm, const double* wgen) {
    constexpr int NEN = 1 << D;
    const ElemCtx k = elem_ctx<D>(c, sm);
    const FEHMM_GLB double* w = glb(wgen);
    FEHMM_GLB double* fe = glb(c.fe);
    FEHMM_GLB KT* ke = (FEHMM_GLB KT*)glb(c.ke);
    const int nitems = k.ne * (D == 2 ? 2 : NEN);
    for (int it = threadIdx.x; it < nitems; it += NT) {
        int sub, e;
        if constexpr (D == 2) {
            sub = it >= k.ne ? 1 : 0;
            e = it - sub * k.ne;
        } else {
            sub = (int)(((float)it + 0.5f) / (float)k.ne);  // (it < 2^18)
            e = it - sub * k.ne;
        }
        int nodes[NEN];
        nodes_of_element<D>(k.n, e, nodes);
        double wl[NEN * D];
        nodal<D>(w, nodes, wl);
        const int ph = k.phase[e];
        const double lam = k.lame[2 * ph], mu = k.lame[2 * ph + 1];
        if constexpr (D == 2) {
            double kii[10], kxy[8], f[4];
#pragma unroll
            for (int q = 0; q < 10; ++q) kii[q] = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) kxy[q] = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = 0.0;
#pragma unroll 1
        for (int gp = 0; gp < k.npt; ++gp) {
                double F[4];
                PointState<2> s;
                grad_at<2>(k, wl, gp, true, F);
                if (!point_state<2>(k.law, lam, mu, k.wJ, F, s)) {
                    *k.flag = 1;
                    continue;
                }
                double dn[4][2], v[4][2];
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    dn[a][0] = k.dN[(gp * 8 + a) * 3];
                    dn[a][1] = k.dN[(gp * 8 + a) * 3 + 1];
                    v[a][0] = s.M[0] * dn[a][0] + s.M[1] * dn[a][1];
                    v[a][1] = s.M[2] * dn[a][0] + s.M[3] * dn[a][1];
                }
                const double p0 = sub ? s.P[2] : s.P[0], p1 = sub ? s.P[3] : s.P[1];
                double bi = 0.0, bxy = 0.0;
                if (k.law == 1) {
                    bi = sub ? s.beta[3] : s.beta[0];
                    bxy = s.beta[1];
                }
                const double a12 = s.a1 + s.a2;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    f[a] += p0 * dn[a][0] + p1 * dn[a][1];
                    const double t0 = s.S[0] * dn[a][0] + s.S[1] * dn[a][1] + bi * dn[a][0];
                    const double t1 = s.S[2] * dn[a][0] + s.S[3] * dn[a][1] + bi * dn[a][1];
                    const double va = (sub ? v[a][1] : v[a][0]) * a12;
#pragma unroll
                    for (int b = 0; b <= a; ++b)
                        kii[a * (a + 1) / 2 + b] += t0 * dn[b][0] + t1 * dn[b][1] + va * (sub ? v[b][1] : v[b][0]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double v0 = sub ? v[2 + h][0] : v[h][0], v1 = sub ? v[2 + h][1] : v[h][1];
                    const double d0 = (sub ? dn[2 + h][0] : dn[h][0]) * bxy, d1 = (sub ? dn[2 + h][1] : dn[h][1]) * bxy;
                    const double x1 = s.a1 * v1, x0 = s.a2 * v0;
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        kxy[4 * h + b] += x1 * v[b][0] + x0 * v[b][1];
                        if (k.law == 1) kxy[4 * h + b] += d0 * dn[b][0] + d1 * dn[b][1];
                    }
                }
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) fe[(a * 2 + sub) * k.ne + e] = f[a];
#pragma unroll
            for (int q = 0; q < 10; ++q) ke[(10 * sub + q) * k.ne + e] = (KT)kii[q];
#pragma unroll
            for (int q = 0; q < 8; ++q) ke[(20 + 8 * sub + q) * k.ne + e] = (KT)kxy[q];
        } else {
            double kd[6], kb[4][9], f[3];
#pragma unroll
            for (int q = 0; q < 6; ++q) kd[q] = 0.0;
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int q = 0; q < 9; ++q) kb[h][q] = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) f[q] = 0.0;
#pragma unroll 1
        for (int gp = 0; gp < k.npt; ++gp) {
                double F[9];
                PointState<3> s;
                grad_at<3>(k, wl, gp, true, F);
                if (!point_state<3>(k.law, lam, mu, k.wJ, F, s)) {
                    *k.flag = 1;
                    continue;
                }
                double da[3], va[3], ta[3];
#pragma unroll
                for (int J = 0; J < 3; ++J) da[J] = k.dN[(gp * 8 + sub) * 3 + J];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    va[i] = s.M[3 * i] * da[0] + s.M[3 * i + 1] * da[1] + s.M[3 * i + 2] * da[2];
                    ta[i] = s.S[3 * i] * da[0] + s.S[3 * i + 1] * da[1] + s.S[3 * i + 2] * da[2];
                    f[i] += s.P[3 * i] * da[0] + s.P[3 * i + 1] * da[1] + s.P[3 * i + 2] * da[2];
                }
                const double a12 = s.a1 + s.a2;
                {
                    const double sd = ta[0] * da[0] + ta[1] * da[1] + ta[2] * da[2];
                    kd[0] += sd + a12 * va[0] * va[0];
                    kd[1] += sd + a12 * va[1] * va[1];
                    kd[2] += sd + a12 * va[2] * va[2];
                    kd[3] += a12 * va[0] * va[1];
                    kd[4] += a12 * va[0] * va[2];
                    kd[5] += a12 * va[1] * va[2];
                    if (k.law == 1) {
                        const double dd = da[0] * da[0] + da[1] * da[1] + da[2] * da[2];
                        kd[0] += s.beta[0] * dd;
                        kd[1] += s.beta[4] * dd;
                        kd[2] += s.beta[8] * dd;
                        kd[3] += s.beta[1] * dd;
                        kd[4] += s.beta[2] * dd;
                        kd[5] += s.beta[5] * dd;
                    }
                }
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int b = (sub + 1 + h) & 7;  // (h = 3 belongs to the items with sub < 4)
                    double db[3], vb[3];
#pragma unroll
                    for (int J = 0; J < 3; ++J) db[J] = k.dN[(gp * 8 + b) * 3 + J];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        vb[i] = s.M[3 * i] * db[0] + s.M[3 * i + 1] * db[1] + s.M[3 * i + 2] * db[2];
                    const double sab = ta[0] * db[0] + ta[1] * db[1] + ta[2] * db[2];
                    const double dab = da[0] * db[0] + da[1] * db[1] + da[2] * db[2];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int l = 0; l < 3; ++l) {
                            double t = (s.a1 * va[l]) * vb[i] + (s.a2 * va[i]) * vb[l];
                            if (i == l) t += sab;
                            if (k.law == 1) t += s.beta[3 * i + l] * dab;
                            kb[h][3 * i + l] += t;
                        }
                }
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) fe[(sub * 3 + i) * k.ne + e] = f[i];
#pragma unroll
            for (int i = 0; i < 3; ++i) ke[sym_entry(3, sub, i, sub, i) * k.ne + e] = (KT)kd[i];
            ke[sym_entry(3, sub, 0, sub, 1) * k.ne + e] = (KT)kd[3];
            ke[sym_entry(3, sub, 0, sub, 2) * k.ne + e] = (KT)kd[4];
            ke[sym_entry(3, sub, 1, sub, 2) * k.ne + e] = (KT)kd[5];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int b = (sub + 1 + h) & 7;
                if (h < 3 || sub < 4)
#pragma unroll
                    for (int q = 0; q < 9; ++q) ke[sym_entry(3, sub, q / 3, b, q % 3) * k.ne + e] = (KT)kb[h][q];
            }
        }
    }
}

// flags sm.flag where some J <= 0 at w
template <int D>
__device__ __noinline__ void element_check(const RveCtx& c, Smem& sm, const double* wgen) {
    const ElemCtx k = elem_ctx<D>(c, sm);
    const FEHMM_GLB double* w = glb(wgen);
    for (int e = threadIdx.x; e < k.ne; e += NT) {
        int nodes[1 << D];
        nodes_of_element<D>(k.n, e, nodes);
        double wl[(1 << D) * D];
        nodal<D>(w, nodes, wl);
#pragma unroll 1
        for (int gp = 0; gp < k.npt; ++gp) {
            double F[D * D], J;
            grad_at<D>(k, wl, gp, true, F);
            if constexpr (D == 2)
                J = F[0] * F[3] - F[1] * F[2];
            else
                J = F[0] * (F[4] * F[8] - F[5] * F[7]) + F[1] * (F[5] * F[6] - F[3] * F[8]) +
                    F[2] * (F[3] * F[7] - F[4] * F[6]);
            if (!(J > 0.0)) *k.flag = 1;
        }
    }
}

// the FP64 tangent at w applied to x, matrix-free, into the force planes (the
// refinement residual of FP32 factors)
template <int D>
__device__ __noinline__ void element_apply(const RveCtx& c, Smem& sm, const double* wgen, const double* xgen) {
    constexpr int NEN = 1 << D;
    const ElemCtx k = elem_ctx<D>(c, sm);
    const FEHMM_GLB double* w = glb(wgen);
    const FEHMM_GLB double* x = glb(xgen);
    FEHMM_GLB double* fe = glb(c.fe);
    for (int e = threadIdx.x; e < k.ne; e += NT) {
        int nodes[NEN];
        nodes_of_element<D>(k.n, e, nodes);
        double wl[NEN * D], xl[NEN * D], f[NEN * D];
        nodal<D>(w, nodes, wl);
        nodal<D>(x, nodes, xl);
        const int ph = k.phase[e];
        const double lam = k.lame[2 * ph], mu = k.lame[2 * ph + 1];
#pragma unroll
        for (int q = 0; q < NEN * D; ++q) f[q] = 0.0;
#pragma unroll 1
        for (int gp = 0; gp < k.npt; ++gp) {
            double F[D * D], g[D * D], t[D * D];
            PointState<D> s;
            grad_at<D>(k, wl, gp, true, F);
            if (!point_state<D>(k.law, lam, mu, k.wJ, F, s)) continue;
            grad_at<D>(k, xl, gp, false, g);
            point_apply<D>(k.law, s, g, t);
#pragma unroll
            for (int a = 0; a < NEN; ++a)
#pragma unroll
                for (int J = 0; J < D; ++J) {
                    const double dn = k.dN[(gp * 8 + a) * 3 + J];
#pragma unroll
                    for (int i = 0; i < D; ++i) f[a * D + i] += t[i * D + J] * dn;
                }
        }
#pragma unroll
        for (int q = 0; q < NEN * D; ++q) fe[q * k.ne + e] = f[q];
    }
}

// rows Y_(a,i),(kL) of every element, planes [((a D + i) D^2 + q)][element];
// work items (element, node)
template <int D>
__device__ __noinline__ void element_coupling(const RveCtx& c, Smem& sm, const double* wgen) {
    constexpr int NEN = 1 << D, D2 = D * D;
    const ElemCtx k = elem_ctx<D>(c, sm);
    const FEHMM_GLB double* w = glb(wgen);
    FEHMM_GLB double* re = glb(c.re);
    const int nitems = k.ne * NEN;
    for (int it = threadIdx.x; it < nitems; it += NT) {
        const int a = (int)(((float)it + 0.5f) / (float)k.ne), e = it - a * k.ne;
        int nodes[NEN];
        nodes_of_element<D>(k.n, e, nodes);
        double wl[NEN * D];
        nodal<D>(w, nodes, wl);
        const int ph = k.phase[e];
        const double lam = k.lame[2 * ph], mu = k.lame[2 * ph + 1];
        double y[D][D2];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int q = 0; q < D2; ++q) y[i][q] = 0.0;
#pragma unroll 1
        for (int gp = 0; gp < k.npt; ++gp) {
            double F[D2];
            PointState<D> s;
            grad_at<D>(k, wl, gp, true, F);
            if (!point_state<D>(k.law, lam, mu, k.wJ, F, s)) continue;
            double da[D], va[D], ta[D];
#pragma unroll
            for (int J = 0; J < D; ++J) da[J] = k.dN[(gp * 8 + a) * 3 + J];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                va[i] = ta[i] = 0.0;
#pragma unroll
                for (int J = 0; J < D; ++J) {
                    va[i] += s.M[i * D + J] * da[J];
                    ta[i] += s.S[i * D + J] * da[J];
                }
            }
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int l = 0; l < D; ++l)
#pragma unroll
                    for (int L = 0; L < D; ++L) {
                        double t = (s.a1 * va[l]) * s.M[i * D + L] + (s.a2 * va[i]) * s.M[l * D + L];
                        if (i == l) t += ta[L];
                        if (k.law == 1) t += s.beta[i * D + l] * da[L];
                        y[i][l * D + L] += t;
                    }
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int q = 0; q < D2; ++q) re[((a * D + i) * D2 + q) * k.ne + e] = y[i][q];
    }
}

// Averages at the converged state, this thread's share: accP = <P> and accA, the
// lower triangle (g (g + 1) / 2 + h) of
//   X = null:  <A>
//   2D, X:     <(E_g - grad X_g) : A : (E_h - grad X_h)>, which is the condensed
//              tangent <A> - Y^T X - X^T Y + X^T K X in the stationary form, with
//              X_g the column g of X ([dof][ldx], zero on the pinned dofs) and E_g
//              the unit macro gradients: neither Y nor K is formed.
// Work items (element, point).
template <int D, bool COND>
__device__ __noinline__ void element_average(const RveCtx& c, Smem& sm, const double* wgen, double* outP, double* outA,
                                             const double* Xgen, int ldx) {
    constexpr int NEN = 1 << D, D2 = D * D, NA = D2 * (D2 + 1) / 2;
    const ElemCtx k = elem_ctx<D>(c, sm);
    const FEHMM_GLB double* w = glb(wgen);
    double accP[D2], accA[NA];
#pragma unroll
    for (int q = 0; q < D2; ++q) accP[q] = 0.0;
#pragma unroll
    for (int q = 0; q < NA; ++q) accA[q] = 0.0;
    const int nitems = k.ne * k.npt;
    for (int it = threadIdx.x; it < nitems; it += NT) {
        const int gp = (int)(((float)it + 0.5f) / (float)k.ne), e = it - gp * k.ne;
        int nodes[NEN];
        nodes_of_element<D>(k.n, e, nodes);
        double wl[NEN * D], F[D2];
        nodal<D>(w, nodes, wl);
        const int ph = k.phase[e];
        const double lam = k.lame[2 * ph], mu = k.lame[2 * ph + 1];
        PointState<D> s;
        grad_at<D>(k, wl, gp, true, F);
        if (!point_state<D>(k.law, lam, mu, k.wJ, F, s)) continue;
#pragma unroll
        for (int q = 0; q < D2; ++q) accP[q] += s.P[q];
        if constexpr (COND) {
            const FEHMM_GLB double* X = glb(Xgen);
            double G[D2][D2];
#pragma unroll
            for (int g = 0; g < D2; ++g)
#pragma unroll
                for (int q = 0; q < D2; ++q) G[g][q] = g == q ? 1.0 : 0.0;
#pragma unroll
            for (int b = 0; b < NEN; ++b)
#pragma unroll
                for (int i = 0; i < D; ++i)
#pragma unroll
                    for (int g = 0; g < D2; ++g) {
                        const double x = X[(nodes[b] * D + i) * ldx + g];
#pragma unroll
                        for (int J = 0; J < D; ++J) G[g][i * D + J] -= x * k.dN[(gp * 8 + b) * 3 + J];
                    }
#pragma unroll
            for (int h = 0; h < D2; ++h) {
                double t[D2];
                point_apply<D>(k.law, s, G[h], t);
#pragma unroll
                for (int g = h; g < D2; ++g)
#pragma unroll
                    for (int q = 0; q < D2; ++q) accA[g * (g + 1) / 2 + h] += G[g][q] * t[q];
            }
        } else {
#pragma unroll
            for (int g = 0; g < D2; ++g)
#pragma unroll
                for (int h = 0; h <= g; ++h) {
                    const int i = g / D, J = g % D, l = h / D, L = h % D;
                    double t = (s.a1 * s.M[l * D + J]) * s.M[i * D + L] + (s.a2 * s.M[i * D + J]) * s.M[l * D + L];
                    if (i == l) t += s.S[J * D + L];
                    if (J == L && k.law == 1) t += s.beta[i * D + l];
                    accA[g * (g + 1) / 2 + h] += t;
                }
        }
    }
#pragma unroll
    for (int q = 0; q < D2; ++q) outP[q] = accP[q];
#pragma unroll
    for (int q = 0; q < NA; ++q) outA[q] = accA[q];
}

// out = sb * b - K x on the free dofs (0 on the pinned ones), from the element
// products k_e x_e that element_apply left in the force planes
template <int D>
__device__ void residual_act(const RveCtx& c, const double* b, double sb, double* out) {
    constexpr int NEN = 1 << D;
    for (int v = threadIdx.x; v < c.nn; v += NT) {
        int el[NEN];
        elements_of_node<D>(c.n, v, el);
        const bool pin = is_pinned(*c.plan, v);
#pragma unroll
        for (int i = 0; i < D; ++i) {
            double s = 0.0;
#pragma unroll
            for (int a = 0; a < NEN; ++a) s += c.fe[(a * D + i) * c.ne + el[a]];
            out[v * D + i] = pin ? 0.0 : sb * b[v * D + i] - s;
        }
    }
}

// node gather of element planes src[((a D + i) nc + col)][element]:
// out[(v D + i) ldo + q0 + col] = sum over the elements around v
template <int D>
__device__ void node_gather(const RveCtx& c, const double* src, int nc, double* out, int ldo, int q0) {
    constexpr int NEN = 1 << D;
    for (int v = threadIdx.x; v < c.nn; v += NT) {
        int el[NEN];
        elements_of_node<D>(c.n, v, el);
        for (int q = 0; q < D * nc; ++q) {
            const int i = q / nc, col = q - i * nc;
            double s = 0.0;
#pragma unroll
            for (int a = 0; a < NEN; ++a) s += src[((a * D + i) * nc + col) * c.ne + el[a]];
            out[(int64_t)(v * D + i) * ldo + q0 + col] = s;
        }
    }
}

// The element tangents a factorization with NRHS right-hand sides reads: the
// Newton factorizations (one rhs, or d^2 + 1 with the condensation's columns)
// read them in the factor type (FP32 for FP32 factors), the condensation
// factorizations at the converged state (d^2 rhs) in FP64.  (The global path
// factors the condensation in FP64 and passes NRHS = 1 with T = double.)
template <int D, int NRHS, typename T>
using KeType = typename std::conditional<NRHS != D * D, T, double>::type;
template <int D, int NRHS, typename T>
__device__ inline const KeType<D, NRHS, T>* ke_of(const RveCtx& c) {
    return reinterpret_cast<const KeType<D, NRHS, T>*>(c.ke);
}

// ---------------------------------------------------------------- packed fronts
// A front's lower triangle is packed column-major: entry (i, j), i >= j, at
// cpk(j, m) + i - j.  The first p columns are the L panel, the only part that LDS
// holds; the trailing columns are exactly the packed update matrix.

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ inline int cpk(int j, int m) { return j * m - ((j * (j - 1)) >> 1); }
// the same for a j that differs between lanes, j, m < 2^12 (24-bit products run at
// the vector unit's full rate, 32-bit ones at a quarter of it; uniform arguments
// belong on the scalar unit, which has no 24-bit product)
__device__ inline int cpkv(int j, int m) { return __mul24(j, m) - (__mul24(j, j - 1) >> 1); }

// 1/x for a pivot on the elimination's dependent chain: the hardware reciprocal
// estimate refined by two Newton-Raphson steps r <- r + r (1 - x r), each of
// which squares the relative error (full double precision for the normal pivots
// that pass the vanishing-pivot test; a pivot that fails it is flagged whatever
// this returns)
__device__ inline double recip_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

__device__ inline double readlane_d(double v, int l) {
    union { double d; int i[2]; } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readlane(u.i[0], l);
    u.i[1] = __builtin_amdgcn_readlane(u.i[1], l);
    return u.d;
}

// the same in the factor type: LDS-front eliminations run in the precision the
// front is stored in (FP32 fronts: one readlane per broadcast, FP32 arithmetic;
// the Newton step is refined against the FP64 residual)
__device__ inline double readlane_t(double v, int l) { return readlane_d(v, l); }
__device__ inline float readlane_t(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double recip_t(double x) { return recip_nr(x); }
__device__ inline float recip_t(float x) {
    float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// ---------------------------------------------------------------- global fronts
// Plans whose fronts exceed LDS (3D from 5^3 up) keep each front in the slot's
// global workspace in the factor type T: the m x p panel column-major (column j
// at Fp + j m, rows i >= j used), its p pivots, and the mu x mu update matrix
// U_s column-major (lower part used) followed by its FP64 rhs rows; the
// forward-substituted rhs stays FP64.  The panel is factored left-looking in
// 64-column blocks: a block first takes the updates of all columns left of it
// as LDS-staged MFMA tiles, then each of its 16-column sub-blocks takes the
// updates of the earlier sub-blocks, wave 0 factors the 16 x 16 diagonal block
// in registers (readlane broadcasts) and forms W = L11^-T D^-1, and the rows
// below become L21 = A21 W on MFMA.  The Schur complement U_s - L21 D L21^T
// goes through the same tiles, straight onto the update stack.

// MFMA 16 x 16 x 4 of the factor type: operand lanes A[l % 16][l / 16] and
// B[l / 16][l % 16]; element v of lane l of the result is at column l % 16 and
// row row(l, v) (FP64: l / 16 + 4 v; FP32: 4 (l / 16) + v; both verified by
// in-bounds probes of the builtins)
typedef float flt4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Mfma16;
template <>
struct Mfma16<double> {
    typedef dbl4 V;
    static __device__ inline V mma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int v) { return (lane >> 4) + 4 * v; }
    static __device__ inline V zero() { return V{0.0, 0.0, 0.0, 0.0}; }
};
template <>
struct Mfma16<float> {
    typedef flt4 V;
    static __device__ inline V mma(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ inline int row(int lane, int v) { return 4 * (lane >> 4) + v; }
    static __device__ inline V zero() { return V{0.f, 0.f, 0.f, 0.f}; }
};

// FP64 rhs rows that follow an mu x mu matrix of T in an update region
template <typename T>
__device__ inline double* urhs(double* base, int mu) {
    return base + ((int64_t)mu * mu * (int64_t)sizeof(T) + 7) / 8;
}

// 16 x 16 diagonal block of a panel by wave 0: LDL^T with readlane broadcasts
// (FP64 arithmetic, stored in T), rhs of the block rows, W = L11^-T D^-1 (16 x
// 16, row-major) into W.  A(r, cc) is the block entry (K + r, K + cc) at
// Ap[cc * ldA + r]; rhs column q of the block rows at yv_base[q * ldy + r].
template <typename T>
__device__ inline void diag_block_wave(T* Ap, int ldA, T* Dd, const T* d0v, int kb, double* yv_base, int ldy,
                                       int nrhs, T* W, int* flag) {
    const int lane = threadIdx.x & 63;
    const bool own = lane < kb;
    double row[16];
    double yv[kMaxNrhs];
#pragma unroll
    for (int cc = 0; cc < 16; ++cc)
        row[cc] = (own && cc < kb && cc <= lane) ? (double)Ap[(int64_t)cc * ldA + lane] : 0.0;
#pragma unroll
    for (int q = 0; q < kMaxNrhs; ++q) yv[q] = (own && q < nrhs) ? yv_base[(int64_t)q * ldy + lane] : 0.0;
    const double d0 = own ? (double)d0v[lane] : 1.0;
    double dpiv = 1.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (j < kb) {
            const double piv = readlane_d(row[j], j);
            const double rp = 1.0 / piv;
            if (lane == j) {
                dpiv = piv;
                if (!(fabs(piv) > 1e-14 * fabs(d0)) || !isfinite(piv)) *flag = 2;
            }
            const double l = (lane > j) ? row[j] * rp : 0.0;
            const double lpv = l * piv;
#pragma unroll
            for (int cc = j + 1; cc < 16; ++cc) {
                if (cc < kb) {
                    const double lc = readlane_d(l, cc);
                    if (cc <= lane) row[cc] -= lpv * lc;
                }
            }
#pragma unroll
            for (int q = 0; q < kMaxNrhs; ++q) {
                if (q < nrhs) {
                    const double yj = readlane_d(yv[q], j);
                    if (lane > j) yv[q] -= l * yj;
                }
            }
            if (lane > j) row[j] = l;
        }
    }
    double inv[16];
#pragma unroll
    for (int cc = 0; cc < 16; ++cc) inv[cc] = (cc == lane) ? 1.0 : 0.0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        if (e < kb) {
            const double le = (lane > e) ? row[e] : 0.0;
#pragma unroll
            for (int cc = 0; cc <= e; ++cc) {
                const double ie = readlane_d(inv[cc], e);
                inv[cc] -= le * ie;
            }
        }
    }
    const double rdp = 1.0 / dpiv;
#pragma unroll
    for (int cc = 0; cc < 16; ++cc)
        if (lane < 16) W[cc * 16 + lane] = (T)((own && cc < kb && cc <= lane) ? inv[cc] * rdp : 0.0);
#pragma unroll
    for (int cc = 0; cc < 16; ++cc)
        if (own && cc < kb && cc <= lane) Ap[(int64_t)cc * ldA + lane] = (T)((cc == lane) ? dpiv : row[cc]);
    if (own) Dd[lane] = (T)dpiv;
#pragma unroll
    for (int q = 0; q < kMaxNrhs; ++q)
        if (own && q < nrhs) yv_base[(int64_t)q * ldy + lane] = yv[q];
}

// Rank-kdim update of the lower triangle of an nrows x ncols block through LDS:
//   Cout(r, c) = Cin(r, c) - sum_{j < kdim} A(r, j) dv(j) A(c, j),   r >= c,
// with A(r, j) at A[j lda + r] and C(r, c) at C[c ldc + r].  The block is
// covered by kTileM x TN tiles (column tiles from the left, row tiles from the
// diagonal down), all processed in one software pipeline: 16-column slabs of A
// (scaled by dv) for the tile rows and columns are staged in LDS
// (double-buffered, one barrier per slab); each step issues the next slab's
// global loads first, runs the MFMAs of the current slab while they are in
// flight, and stages the next slab at its end.  Loads are unconditional at
// clamped addresses; rows and columns past the block only reach outputs that
// are never written, and columns past kdim are zeroed through dv.  Four waves
// compute a 64 x TN/2 quarter of a tile each, eight a 64 x TN/4 eighth.  Every
// thread of the workgroup must call it; it ends with a barrier.
static_assert(kTileLdsElems == 2 * kTileSlab * 2 * kTileStride, "tile update LDS size");
template <typename T, int TN>
struct TileRegs {
    static constexpr int C = kTileSlab / NWAVE;  // slab columns a wave loads
    T a[2 * C], b[(TN / 64) * C], d[C];
    int j0;  // first column of the slab
};
// global-address-space view of a workspace pointer: its loads count only on
// the vector-memory counter, so the LDS waits before the MFMAs do not also wait
// for prefetches in flight (generic pointers give flat loads, which count on both)
template <typename T>
__device__ inline const __attribute__((address_space(1))) T* as_global(const T* p) {
    return (const __attribute__((address_space(1))) T*)p;
}
// walk of the tiles: column tiles c0 = 0, TN, ...; row tiles r0 = c0, c0 + kTileM, ...
template <int TN>
struct TileCursor {
    int r0, c0;
    __device__ inline void next(int nrows) {
        r0 += kTileM;
        if (r0 >= nrows) {
            c0 += TN;
            r0 = c0;
        }
    }
};
template <typename T, int TN>
__device__ __attribute__((noinline)) void tiles_update(const T* A, const T* dv, int64_t lda, int kdim, const T* Cin,
                                                       T* Cout, int64_t ldc, int nrows, int ncols, T* lds) {
    static_assert(TN == 64 || TN == 128, "tile width");
    typedef Mfma16<T> M;
    constexpr int NB = TN / 64;   // B rows per loader thread and column
    constexpr int C = kTileSlab / NWAVE;   // slab columns a wave loads
    constexpr int WC = NWAVE / 2;          // waves across a tile's columns (two across its rows)
    constexpr int WT = TN / 16 / WC;       // MFMA column tiles per wave
    A = uni(A);
    dv = uni(dv);
    lda = uni(lda);
    kdim = uni(kdim);
    Cin = uni(Cin);
    Cout = uni(Cout);
    ldc = uni(ldc);
    nrows = uni(nrows);
    ncols = uni(ncols);  // (lds stays as passed: its LDS address space is inferred from the caller)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = tid & 63, lj = (tid >> 6) * C;
    constexpr int BUF = kTileSlab * 2 * kTileStride;
    const auto* Ag = as_global(A);
    const auto* dg = as_global(dv);
    // slab count rounded up to even: slabs past kdim are zeros
    const int ns = 2 * ((kdim + 2 * kTileSlab - 1) / (2 * kTileSlab));
    // load side of the pipeline: tile and slab of the next load; once every
    // slab is loaded it stays on the last one (loaded again, never computed)
    TileCursor<TN> lc{0, 0};
    int ls = 0;
    auto load = [&](TileRegs<T, TN>& R) {
        const int j0 = kTileSlab * ls;
        R.j0 = j0;
        const int ra0 = min(lc.r0 + lr, nrows - 1), ra1 = min(lc.r0 + lr + 64, nrows - 1);
        int rb[NB];
#pragma unroll
        for (int h = 0; h < NB; ++h) rb[h] = min(lc.c0 + lr + 64 * h, ncols - 1);
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int j = min(j0 + lj + q, kdim - 1);
            const auto* Aj = Ag + (int64_t)j * lda;
            R.a[q] = Aj[ra0];
            R.a[C + q] = Aj[ra1];
#pragma unroll
            for (int h = 0; h < NB; ++h) R.b[C * h + q] = Aj[rb[h]];
            R.d[q] = dg[j];
        }
        // advance with selects only: a branch here would split the loop body
        // and make the compiler drain the loads in flight
        const bool wrap = ls + 1 == ns;
        const bool colwrap = lc.r0 + kTileM >= nrows;
        const int nc0 = colwrap ? lc.c0 + TN : lc.c0;
        const int nr0 = colwrap ? nc0 : lc.r0 + kTileM;
        const bool more = nc0 < ncols;
        lc.r0 = (wrap && more) ? nr0 : lc.r0;
        lc.c0 = (wrap && more) ? nc0 : lc.c0;
        ls = wrap ? (more ? 0 : ns - 1) : ls + 1;
    };
    auto store = [&](const TileRegs<T, TN>& R, int buf) {
        T* As = lds + buf * BUF;
        T* Bs = As + kTileSlab * kTileStride;
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const T dq = R.j0 + lj + q < kdim ? R.d[q] : T(0);  // columns past kdim
            As[(lj + q) * kTileStride + lr] = R.a[q] * dq;
            As[(lj + q) * kTileStride + lr + 64] = R.a[C + q] * dq;
#pragma unroll
            for (int h = 0; h < NB; ++h) Bs[(lj + q) * kTileStride + lr + 64 * h] = R.b[C * h + q];
        }
    };
    typename M::V acc[4][WT];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w2 = 0; w2 < WT; ++w2) acc[u][w2] = M::zero();
    const int wr = 64 * (wave / WC), wc = 16 * WT * (wave % WC);
    auto compute = [&](int buf) {
        const T* As = lds + buf * BUF;
        const T* Bs = As + kTileSlab * kTileStride;
#pragma unroll
        for (int ks = 0; ks < kTileSlab / 4; ++ks) {
            const int kk = 4 * ks + (lane >> 4);
            T av[4], bv[WT];
#pragma unroll
            for (int u = 0; u < 4; ++u) av[u] = As[kk * kTileStride + wr + 16 * u + (lane & 15)];
#pragma unroll
            for (int w2 = 0; w2 < WT; ++w2) bv[w2] = Bs[kk * kTileStride + wc + 16 * w2 + (lane & 15)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int w2 = 0; w2 < WT; ++w2) acc[u][w2] = M::mma(av[u], bv[w2], acc[u][w2]);
        }
    };
    // one pipeline step: the next slab's loads are issued first, the MFMAs of
    // LDS buffer buf run while they are in flight, and the slab is staged into
    // the other buffer at the end (no load stays in flight across steps)
    auto step = [&](int buf, TileRegs<T, TN>& R) {
        load(R);
        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the MFMAs
        compute(buf);
        __builtin_amdgcn_sched_barrier(0);  // and the staging (which waits for it) behind them
        store(R, buf ^ 1);
        __syncthreads();
    };
    TileRegs<T, TN> R0;
    if (ns > 0) {  // kdim = 0: Cout = Cin
        load(R0);
        store(R0, 0);
    }
    __syncthreads();
    for (TileCursor<TN> cc{0, 0}; cc.c0 < ncols; cc.next(nrows)) {
        for (int s = 0; s < ns; s += 2) {
            step(0, R0);
            step(1, R0);
        }
        const int nr = nrows - cc.r0, nc = ncols - cc.c0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int w2 = 0; w2 < WT; ++w2) {
                const int col = wc + 16 * w2 + (lane & 15);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int rr = wr + 16 * u + M::row(lane, v);
                    if (rr < nr && col < nc && cc.r0 + rr >= cc.c0 + col) {
                        const int64_t o = (int64_t)(cc.c0 + col) * ldc + cc.r0 + rr;
                        Cout[o] = Cin[o] - acc[u][w2][v];
                    }
                }
                acc[u][w2] = M::zero();
            }
    }
}

// Multifrontal LDL^T of K_ff with nrhs right-hand sides in c.rhs (node-major
// [dof][nrhs]); forward substitution fused.  Returns via sm.flag = 2 on a
// vanishing pivot.  Fronts in global memory (any size) in the factor type T;
// lds holds the staged slabs of tile_update.
template <int D, typename T>
__device__ __attribute__((noinline)) void factorize_glb(const RveCtx& c, Smem& sm, int nrhs, T* lds) {
    typedef Mfma16<T> M;
    constexpr int NEN = 1 << D;
    const DevPlan& pl = *c.plan;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    T* W = reinterpret_cast<T*>(sm.red);  // 16 x 16
    nrhs = uni(nrhs);
    double* const cL = uni(c.L);
    double* const cU = uni(c.U);
    double* const cS = uni(c.S);
    PROF_T0();
    const int nfront = uni(pl.nfront);
    const FEHMM_GLB int32_t* asm_rc = glb(pl.asm_dst);
    const FEHMM_GLB int32_t* asm_src = glb(pl.asm_src);
    const FEHMM_GLB T* ke = (const FEHMM_GLB T*)glb(c.ke);
    for (int s = 0; s < nfront; ++s) {
        const DevFront fr = pl.fronts[s];
        const int m = uni(fr.m), p = uni(fr.p), mu = m - p;
        const int32_t* rows = uni(pl.rows + fr.rows_off);
        T* Fp = reinterpret_cast<T*>(cL + uni(fr.L_off));
        T* Dg = reinterpret_cast<T*>(cL + uni(fr.D_off));
        double* y = cL + uni(fr.y_off);
        T* Us = reinterpret_cast<T*>(cS);
        double* rus = urhs<T>(cS, mu);
        // 1. zero the parts that are read later (the panel on and below its
        //    diagonal, the lower triangle of U_s), load the pivot rhs
        for (int j = wave; j < p; j += NWAVE)
            for (int i = j + lane; i < m; i += 64) Fp[(int64_t)j * m + i] = T(0);
        for (int k = wave; k < mu; k += NWAVE)
            for (int i = k + lane; i < mu; i += 64) Us[(int64_t)k * mu + i] = T(0);
        for (int t = threadIdx.x; t < mu * nrhs; t += NT) rus[t] = 0.0;
        for (int t = threadIdx.x; t < p * nrhs; t += NT) {
            int j = t % p, col = t / p;
            y[t] = c.rhs[(int64_t)rows[j] * nrhs + col];
        }
        __syncthreads();
        // 2. original entries K(b, a) of the pivot nodes a
        for (int t0 = fr.asm_begin + tid; t0 < fr.asm_end; t0 += 2 * NT) {
            // two strides per pass, every load of both issued together
            int rc[2], src[2][NEN];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = min(t0 + u * NT, fr.asm_end - 1);
                rc[u] = asm_rc[t];
#pragma unroll
                for (int q = 0; q < NEN; ++q) src[u][q] = asm_src[(int64_t)t * NEN + q];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                double v = 0;
#pragma unroll
                for (int q = 0; q < NEN; ++q) {
                    const double kv = (double)ke[max(src[u][q], 0)];
                    v += src[u][q] >= 0 ? kv : 0.0;
                }
                if (t0 + u * NT < fr.asm_end) {
                    const int r = rc[u] >> 16, col = rc[u] & 0xffff;
                    Fp[(int64_t)col * m + r] = (T)v;
                    if (r == col) Dg[col] = (T)v;
                }
            }
        }
        __syncthreads();
        // 3. extend-add of the children's update matrices and rhs updates
        for (int q = fr.child_begin; q < fr.child_end; ++q) {
            const DevFront ch = pl.fronts[pl.children[q]];
            const int mc = ch.m - ch.p;
            const int32_t* rel = pl.relind + ch.relind_off;
            const T* Uc = reinterpret_cast<const T*>(c.U + ch.U_off);
            const double* ruc = urhs<T>(c.U + ch.U_off, mc);
            // lower triangle, 8 columns per pass: a thread first issues the 8
            // loads of its row, then the 8 read-modify-writes, so each pass costs
            // two memory round trips instead of sixteen
            for (int k0 = 0; k0 < mc; k0 += 8) {
                int Ck[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) Ck[u] = rel[min(k0 + u, mc - 1)];
                for (int i = k0 + threadIdx.x; i < mc; i += NT) {
                    const int R = rel[i];
                    T v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = Uc[(int64_t)min(k0 + u, mc - 1) * mc + i];
                    T* dstp[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int C = Ck[u];
                        dstp[u] = C < p ? Fp + (int64_t)C * m + R : Us + (int64_t)(C - p) * mu + (R - p);
                    }
                    T old[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) old[u] = (k0 + u < mc && i >= k0 + u) ? *dstp[u] : T(0);
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (k0 + u < mc && i >= k0 + u) *dstp[u] = old[u] + v[u];
                }
            }
            for (int t = threadIdx.x; t < mc * nrhs; t += NT) {
                const int i = t % mc, col = t / mc;
                const int R = rel[i];
                const double v = ruc[(int64_t)col * mc + i];
                if (R < p) y[(int64_t)col * p + R] += v;
                else rus[(int64_t)col * mu + (R - p)] += v;
            }
            __syncthreads();
        }
        PROF_MARK(PH_ASM);
        // 4. panel LDL^T in 64-column blocks (left-looking), forward rhs.  A
        // block first takes the updates of all columns left of it as LDS tiles,
        // then its four 16-column sub-blocks are factored in turn.
        for (int K64 = 0; K64 < p; K64 += 64) {
            const int kb64 = min(64, p - K64);
            if (K64 > 0) {
                T* Ct = Fp + (int64_t)K64 * m + K64;
                tiles_update<T, 64>(Fp + K64, Dg, m, K64, Ct, Ct, m, m - K64, kb64, lds);
            }
            for (int K = K64; K < K64 + kb64; K += 16) {
                const int kb = min(16, p - K);
                // (a) updates of the earlier columns of the block:
                //     A(i, K + c) -= sum_{K64 <= j < K} L(i, j) D(j) L(K + c, j)
                if (K > K64) {
                    const int nt = (m - K + 15) >> 4;
                    for (int t0 = 2 * wave; t0 < nt; t0 += 2 * NWAVE) {
                        typename M::V acc[2] = {M::zero(), M::zero()};
                        const int cb = K + (lane & 15);
                        // at most 48 earlier columns in the block: unrolled to 12
                        // k-steps so that all operand loads are issued together
                        T av[12][2], bv[12];
#pragma unroll
                        for (int q = 0; q < 12; ++q) {
                            const int j = min(K64 + 4 * q + (lane >> 4), K - 1);
                            const T* colj = Fp + (int64_t)j * m;
                            bv[q] = colj[min(cb, m - 1)];
                            const T dj = Dg[j];
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                av[q][u] = colj[min(K + 16 * (t0 + u) + (lane & 15), m - 1)] * dj;
                        }
#pragma unroll
                        for (int q = 0; q < 12; ++q) {
                            if (K64 + 4 * q < K) {
                                const bool okb = (lane & 15) < kb;
#pragma unroll
                                for (int u = 0; u < 2; ++u) {
                                    const bool oka = K + 16 * (t0 + u) + (lane & 15) < m;
                                    acc[u] = M::mma(oka ? av[q][u] : T(0), okb ? bv[q] : T(0), acc[u]);
                                }
                            }
                        }
                        const int cc = lane & 15;
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int rr = K + 16 * (t0 + u) + M::row(lane, v);
                                if (t0 + u < nt && rr < m && cc < kb && rr >= K + cc)
                                    Fp[(int64_t)(K + cc) * m + rr] -= acc[u][v];
                            }
                    }
                    __syncthreads();
                }
                PROF_MARK(PH_MFMA);
                // (b) diagonal block and its rhs rows by wave 0
                if (wave == 0)
                    diag_block_wave<T>(Fp + (int64_t)K * m + K, m, Dg + K, Dg + K, kb, y + K, p, nrhs, W, &sm.flag);
                __syncthreads();
                PROF_MARK(PH_DIAG);
                // (c) rows below: L21 = A21 W (MFMA)
                const int R0 = K + kb;
                {
                    // four row tiles in flight per wave: every operand is read before
                    // the products (a tile's rows are overwritten by its own results
                    // only)
                    const int nt = (m - R0 + 15) >> 4;
                    FEHMM_GLB T* Fg = glb(Fp);
                    T wv[4];
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) wv[ks] = W[(4 * ks + (lane >> 4)) * 16 + (lane & 15)];
                    for (int t0 = 4 * wave; t0 < nt; t0 += 4 * NWAVE) {
                        T av[4][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int ra = min(R0 + 16 * (t0 + u) + (lane & 15), m - 1);
#pragma unroll
                            for (int ks = 0; ks < 4; ++ks) {
                                const int kk = 4 * ks + (lane >> 4);
                                av[u][ks] = Fg[(int64_t)(K + min(kk, kb - 1)) * m + ra];
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            // (transposed product: consecutive lanes hold consecutive
                            // rows of a column)
                            typename M::V acc = M::zero();
#pragma unroll
                            for (int ks = 0; ks < 4; ++ks)
                                acc = M::mma(wv[ks], 4 * ks + (lane >> 4) < kb ? av[u][ks] : T(0), acc);
                            const int rr = R0 + 16 * (t0 + u) + (lane & 15);
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int cc = M::row(lane, v);
                                if (rr < m && cc < kb) Fg[(int64_t)(K + cc) * m + rr] = acc[v];
                            }
                        }
                    }
                }
                __syncthreads();
                // (d) rhs of the rows below: b_i -= sum_c L(i, K + c) y(K + c),
                //     one row per thread for every column (the row's 16 L entries
                //     read once)
                for (int i = R0 + tid; i < m; i += NT) {
                    double lk[16];
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc) lk[cc] = cc < kb ? (double)Fp[(int64_t)(K + cc) * m + i] : 0.0;
                    for (int q = 0; q < nrhs; ++q) {
                        const double* yq = y + (int64_t)q * p + K;
                        double acc = 0.0;
#pragma unroll
                        for (int cc = 0; cc < 16; ++cc)
                            if (cc < kb) acc += lk[cc] * yq[cc];
                        if (i < p) y[(int64_t)q * p + i] -= acc;
                        else rus[(int64_t)q * mu + (i - p)] -= acc;
                    }
                }
                __syncthreads();
                PROF_MARK(PH_TRSM);
            }
        }
        // 5. Schur complement U = U_s - L21 D L21^T over the tiles of its lower
        //    triangle, written straight onto the update stack with its rhs rows
        if (mu > 0) {
            T* dst = reinterpret_cast<T*>(cU + uni(fr.U_off));
            double* drhs = urhs<T>(cU + uni(fr.U_off), mu);
            tiles_update<T, 128>(Fp + p, Dg, m, p, Us, dst, mu, mu, mu, lds);
            for (int t = tid; t < mu * nrhs; t += NT) drhs[t] = rus[t];
        }
        __syncthreads();
        PROF_MARK(PH_OUT);
    }
}

// forward substitution L y = b with stored global-memory factors, for a new
// rhs b (node-major [dof][NRHS], FP64, overwritten): fronts in elimination
// order; per front the pivot rows are solved in 16-pivot blocks (readlane
// chain in wave 0) and folded into the rows below, whose update goes straight
// into b at the rows' dofs (each is a pivot of a later front); the pivot part
// is stored as the front's forward-substituted rhs for backsolve_glb.
template <int D, int NRHS, typename T>
__device__ __attribute__((noinline)) void forward_glb(const RveCtx& c, Smem& sm, double* b) {
    const DevPlan& pl = *c.plan;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* const cL = uni(c.L);
    b = uni(b);
    const int nfront = uni(pl.nfront);
    for (int s = 0; s < nfront; ++s) {
        const DevFront fr = pl.fronts[s];
        const int m = uni(fr.m), p = uni(fr.p);
        const int32_t* rows = uni(pl.rows + fr.rows_off);
        const T* Fp = reinterpret_cast<const T*>(cL + uni(fr.L_off));
        double* y = cL + uni(fr.y_off);
        for (int t = tid; t < p * NRHS; t += NT) {
            const int j = t % p, q = t / p;
            y[t] = b[(int64_t)rows[j] * NRHS + q];
        }
        __syncthreads();
        for (int K = 0; K < p; K += 16) {
            const int kb = min(16, p - K);
            if (wave == 0) {
                const bool own = lane < kb;
                double Lr[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc)
                    Lr[cc] = (own && cc < kb && cc < lane) ? (double)Fp[(int64_t)(K + cc) * m + K + lane] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double vv = own ? y[(int64_t)q * p + K + lane] : 0.0;
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc) {
                        if (cc < kb) {
                            const double yc = readlane_d(vv, cc);
                            if (lane > cc) vv -= Lr[cc] * yc;
                        }
                    }
                    if (own) y[(int64_t)q * p + K + lane] = vv;
                }
            }
            __syncthreads();
            for (int i = K + kb + tid; i < m; i += NT) {
                double lk[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc) lk[cc] = (cc < kb) ? (double)Fp[(int64_t)(K + cc) * m + i] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double acc = 0.0;
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc)
                        if (cc < kb) acc += lk[cc] * y[(int64_t)q * p + K + cc];
                    if (i < p) y[(int64_t)q * p + i] -= acc;
                    else b[(int64_t)rows[i] * NRHS + q] -= acc;
                }
            }
            __syncthreads();
        }
    }
}

// backward substitution L^T x = D^-1 y with global-memory factors; x
// node-major [dof][NRHS].  Per front: the update rows' contribution v = D^-1 y -
// L21^T x_u on FP64 MFMA (16 pivots x 4 rows x up to 16 rhs columns), one 16-pivot
// tile per wave, or with fewer tiles than waves the rows of a tile split over
// several (partial sums in lds, added in a fixed order); then 16-pivot blocks from
// the last: wave 0 solves the block triangle with readlane broadcasts, all threads
// fold the block into the earlier pivots.  Bound by the one read of L: a thread per
// pivot walking its column, four loads in flight, took 55 Mclk per sweep at 16^3.
template <int D, int NRHS, typename T>
__device__ __attribute__((noinline)) void backsolve_glb(const RveCtx& c, Smem& sm, double* xo, double* ldsgen) {
    typedef Mfma16<double> M;
    const DevPlan& pl = *c.plan;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, lg = lane >> 4;
    zero_pinned<D>(c, xo, NRHS);
    __syncthreads();
    double* const cL = uni(c.L);
    FEHMM_LDS double* const pb = (FEHMM_LDS double*)ldsgen;  // [parts][16 tiles][NRHS] partial sums
    xo = uni(xo);
    const FEHMM_GLB double* const xg = glb((const double*)xo);
    for (int s = uni(pl.nfront) - 1; s >= 0; --s) {
        const DevFront fr = pl.fronts[s];
        const int m = uni(fr.m), p = uni(fr.p), mu = m - p;
        const int32_t* rows = uni(pl.rows + fr.rows_off);
        const FEHMM_GLB int32_t* rg = glb(rows);
        const T* Fp = reinterpret_cast<const T*>(cL + uni(fr.L_off));
        const FEHMM_GLB T* Fg = glb(Fp);
        const T* Dg = reinterpret_cast<const T*>(cL + uni(fr.D_off));
        double* y = cL + uni(fr.y_off);
        const int ntile = (p + 15) >> 4, nks = (mu + 3) >> 2;
        const int parts = mu > 0 ? max(1, NWAVE / ntile) : 1;
        for (int unit = wave; unit < ntile * parts; unit += NWAVE) {
            const int t = unit % ntile, part = unit / ntile;
            const int j = min(16 * t + l15, p - 1);
            const FEHMM_GLB T* col = Fg + (int64_t)j * m + p;
            M::V acc[2] = {M::zero(), M::zero()};
            // (the next eight steps' L and row numbers are requested with this
            // step's solution values)
            T a[8];
            int ri[8];
            auto load = [&](int k0, T (&av)[8], int (&rv)[8]) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = min(4 * (k0 + u * parts) + lg, mu - 1);
                    av[u] = col[i];
                    rv[u] = rg[p + i] * NRHS + (NRHS == 1 ? 0 : min(l15, NRHS - 1));
                }
            };
            if (mu > 0) load(part, a, ri);
            for (int k0 = part; k0 < nks; k0 += 8 * parts) {
                double b[8];
                T an[8];
                int rn[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) b[u] = xg[ri[u]];
                load(k0 + 8 * parts, an, rn);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool ok = 4 * (k0 + u * parts) + lg < mu && l15 < NRHS;
                    acc[u & 1] = M::mma((double)a[u], ok ? b[u] : 0.0, acc[u & 1]);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    a[u] = an[u];
                    ri[u] = rn[u];
                }
            }
            // element e of lane: pivot 16 t + row(lane, e), rhs column l15
            if (l15 < NRHS)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int jj = 16 * t + M::row(lane, e);
                    if (jj < p) {
                        const double sum = acc[0][e] + acc[1][e];
                        if (parts > 1) pb[(part * 16 * ntile + jj) * NRHS + l15] = sum;
                        else y[(int64_t)l15 * p + jj] = y[(int64_t)l15 * p + jj] / (double)Dg[jj] - sum;
                    }
                }
        }
        __syncthreads();
        if (parts > 1) {
            for (int t = tid; t < p * NRHS; t += NT) {
                const int j = t % p, q = t / p;
                double sum = 0.0;
                for (int w = 0; w < parts; ++w) sum += pb[(w * 16 * ntile + j) * NRHS + q];
                y[t] = y[t] / (double)Dg[j] - sum;
            }
            __syncthreads();
        }
        const int nb = (p + 15) >> 4;
        for (int bk = nb - 1; bk >= 0; --bk) {
            const int K = 16 * bk, kb = min(16, p - K);
            if (wave == 0) {
                const bool own = lane < kb;
                double Lr[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc)
                    Lr[cc] = (own && cc < kb && cc > lane) ? (double)Fp[(int64_t)(K + lane) * m + K + cc] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double vv = own ? y[(int64_t)q * p + K + lane] : 0.0;
#pragma unroll
                    for (int cc = 15; cc >= 0; --cc) {
                        if (cc < kb) {
                            const double xc = readlane_d(vv, cc);
                            if (lane < cc) vv -= Lr[cc] * xc;
                        }
                    }
                    if (own) y[(int64_t)q * p + K + lane] = vv;
                }
            }
            __syncthreads();
            for (int j = tid; j < K; j += NT) {
                const T* cj = Fp + (int64_t)j * m + K;
                double lk[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc) lk[cc] = (cc < kb) ? (double)cj[cc] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double acc = y[(int64_t)q * p + j];
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc)
                        if (cc < kb) acc -= lk[cc] * y[(int64_t)q * p + K + cc];
                    y[(int64_t)q * p + j] = acc;
                }
            }
            __syncthreads();
        }
        for (int t = tid; t < p * NRHS; t += NT) {
            const int j = t % p, q = t / p;
            xo[(int64_t)rows[j] * NRHS + q] = y[(int64_t)q * p + j];
        }
        __syncthreads();
    }
}

// Multifrontal LDL^T with the front panels in LDS.  Of a front of m rows and p
// pivots only the m x p panel is held in LDS (packed columns, entry (i, j),
// i >= j, at cpk(j, m) + i - j); the update matrix never is.  Per front:
//   1. the panel takes its original entries (one gather) and the panel part of
//      the children's update matrices (a prefix of each, extend-add);
//   2. 16-column blocks: every row is owned by one thread, which holds its 16
//      block entries in registers beside a copy of the block's own 16 rows,
//      replicated in each 16-lane DPP row.  A pivot's multipliers are broadcast
//      from that copy by row_newbcast moves, so the 16 pivots of a block need
//      neither barriers nor LDS traffic nor readlane;
//   3. the panel columns right of the block are updated on MFMA;
//   4. after the last block the update matrix is formed tile by tile in MFMA
//      accumulators over all p pivots, the children's entries (gathered through
//      the inverse row maps) added, and written once, straight to the stack.
// Storage type T (panels, update matrices) and arithmetic type C of the pivots and the
// right-hand sides (block entries in registers, rhs rows of the blocks and of the
// update matrices): equal, except for FP32 factors of plans whose packed fronts do not
// fit LDS (DevPlan::wide_rhs), which keep C = double: with C = float their condensed
// tangents are 2 to 4 times further from FP64's (43 x 43, stiffness ratio 50, RMS of 64
// RVEs: 8.1e-10 against 2.4e-10), for 1 to 3 % of the time of a solve.
// A panel needs 2 p / m of a packed front's LDS: two four-wave workgroups fit a
// CU up to 32 x 32 in FP64 (81.4 KB each), where whole packed fronts (139 KB)
// allowed one.  Small subtrees run the same code one front per wave first, then
// the workgroup fronts run in the plan's steps of 1, 2 or 4 independent fronts.
// What bounds it: latency (dependent FP64 chains of the pivots, memory round trips
// per front), at a third of the vector unit's issue slots.  Measured against whole
// packed fronts eliminated with a barrier per pivot, on one MI355X: 4096 RVEs of
// 32 x 32 85.7 -> 64 ms (FP32 factors 66.7 -> 56), 14288 of 16 x 16 55.3 -> 48.5 ms.

// what the LDS-plan functions read of the plan and the slot, in scalar registers
struct PanelCtx {
    const FEHMM_GLB DevFront* fronts;
    const FEHMM_GLB DevChild* childrec;
    const FEHMM_GLB int32_t *rows, *asm_dst, *asm_src, *ea_dst, *inv, *wave_hbeg, *wg_steps, *task, *task_beg;
    const FEHMM_GLB BackRec* back;
    int nwave_h, nwg_steps, ntask_lev, ul_base, ul_stride, wave_slice;
    FEHMM_GLB double *L, *U;
};
__device__ inline PanelCtx panel_ctx(const RveCtx& c) {
    const DevPlan pl = load_const(glb(c.plan));
    PanelCtx k;
    k.fronts = glb(pl.fronts);
    k.childrec = glb(pl.childrec);
    k.rows = glb(pl.rows);
    k.asm_dst = glb(pl.asm_dst);
    k.asm_src = glb(pl.asm_src);
    k.ea_dst = glb(pl.ea_dst);
    k.inv = glb(pl.inv);
    k.back = glb(pl.back);
    k.wave_hbeg = glb(pl.wave_hbeg);
    k.wg_steps = glb(pl.wg_steps);
    k.task = glb(pl.task);
    k.task_beg = glb(pl.task_beg);
    k.ntask_lev = uni(pl.ntask_lev);
    k.wave_slice = uni(pl.wave_slice);
    k.ul_base = uni(pl.ul_base);
    k.ul_stride = uni(pl.ul_stride);
    k.nwave_h = uni(pl.nwave_h);
    k.nwg_steps = uni(pl.nwg_steps);
    k.L = glb(c.L);
    k.U = glb(c.U);
    return k;
}

// f(0) .. f(N - 1) with compile-time indices (DPP controls are immediates)
template <int I, int N, typename Fn>
__device__ inline __attribute__((always_inline)) void static_for(Fn&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// lane N of the caller's 16-lane row, in every lane of the row
template <int N, typename T>
__device__ inline T row_bcast(T v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xf, 0xf, true);
}

// barrier of a front's threads: the workgroup's, or (one front per wave) only
// an ordering of the wave's own LDS accesses, which complete in issue order
template <bool WAVE>
__device__ inline void front_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// elements of T before the rhs rows (of type C) of a packed update matrix of mu rows
template <typename T, typename C>
__device__ inline int rhs_at(int mu) {
    const int e = cpk(mu, mu);
    return sizeof(C) == sizeof(T) ? e : (e + 1) & ~1;
}

// masked store into a panel: FP64 under the lane mask; FP32 without a branch, masked
// lanes to F[-1] (eight of them in a row measured 4 % of a solve faster in FP32, 4 %
// slower in FP64, whose same-address stores cost more)
template <typename T>
__device__ inline void put(FEHMM_LDS T* F, bool ok, int at, T v) {
    if constexpr (sizeof(T) == 4) F[ok ? at : -1] = v;
    else if (ok) F[at] = v;
}

// Original entries of a panel from the element matrices (one gather level): U
// strides of the list per pass, every index load first, then every value load
// (clamped addresses, zeros selected), then the stores, so a pass costs two
// memory round trips for all its strides.
template <int NEN, int U, typename KT, typename T>
__device__ inline void gather_original(const PanelCtx& pl, const FEHMM_GLB KT* ke, int a0, int a1, int first, int stride,
                                       FEHMM_LDS T* F) {
    typedef int32_t vint4 __attribute__((ext_vector_type(4)));
    const FEHMM_GLB vint4* src4 = (const FEHMM_GLB vint4*)pl.asm_src;
    for (int t0 = a0 + first; t0 < a1; t0 += U * stride) {
        int dst[U];
        vint4 src[U][NEN / 4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = min(t0 + u * stride, a1 - 1);
            dst[u] = pl.asm_dst[t];
#pragma unroll
            for (int q = 0; q < NEN / 4; ++q) src[u][q] = src4[(int64_t)t * (NEN / 4) + q];
        }
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = 0.0;
#pragma unroll
            for (int q = 0; q < NEN / 4; ++q) {
                const int s[4] = {src[u][q].x, src[u][q].y, src[u][q].z, src[u][q].w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double kv = (double)ke[max(s[k], 0)];
                    v[u] += (s[k] >= 0) ? kv : 0.0;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) put(F, t0 + u * stride < a1, dst[u], (T)v[u]);
    }
}
// one pass of an extend-add in parts, so that its loads can be issued early
template <int U, typename T>
struct ExtendPass {
    int e[U];
    T v[U];
    __device__ inline void index(const FEHMM_GLB int32_t* ea, int nu, int first, int stride) {
#pragma unroll
        for (int u = 0; u < U; ++u) e[u] = nu > 0 ? ea[min(first + u * stride, nu - 1)] : 0;
    }
    template <typename Src>
    __device__ inline void value(const Src* Uc, int nu, int first, int stride) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = Uc[max(min(first + u * stride, nu - 1), 0)];
    }
    __device__ inline void add(int nu, int first, int stride, FEHMM_LDS T* F) {
        T o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = F[e[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) put(F, first + u * stride < nu, e[u], (T)(o[u] + v[u]));
    }
};
template <int U = 8, typename Src, typename T>
__device__ inline void extend_add_packed(const FEHMM_GLB int32_t* ea, const Src* Uc, int nu, int first, int stride,
                                         FEHMM_LDS T* F) {
    for (int t0 = first; t0 < nu; t0 += U * stride) {
        // the targets of a pass are distinct (a child adds to each parent entry
        // once): every target is read before any is written, one LDS round trip
        ExtendPass<U, T> ep;
        ep.index(ea, nu, t0, stride);
        ep.value(Uc, nu, t0, stride);
        ep.add(nu, t0, stride, F);
    }
}

// The 16 pivots of a block on one thread's row (entries row[], rhs b[]) and the
// replicated block rows (blk[], yb[]; lane l of each 16-lane row holds block row
// l).  ib: the row's number in the block (negative above it, >= 16 below).  rows
// below a pivot leave with L and the forward-substituted rhs, a pivot's own row
// with D on its diagonal; entries above a diagonal and columns past kb hold
// garbage that is neither stored nor broadcast.  Pivots past kb (whole groups of
// four are skipped, the others run with a zero reciprocal) change nothing.
template <int NRHS, typename T>
__device__ inline __attribute__((always_inline)) void eliminate16(T (&blk)[16], T (&row)[16], T (&yb)[NRHS],
                                                                  T (&b)[NRHS], int kb, int ib, T& mypiv) {
    static_for<0, 4>([&](auto G) {
        constexpr int g = decltype(G)::value;
        if (4 * g < kb) {
            static_for<4 * g, 4 * g + 4>([&](auto J) {
                constexpr int j = decltype(J)::value;
                const T piv = row_bcast<j>(blk[j]);
                const T rp = j < kb ? recip_t(piv) : T(0);
                mypiv = ib == j ? piv : mypiv;
                const T bj = blk[j], rj = row[j];
                const T lb = bj * rp;
                static_for<j + 1, 16>([&](auto C) {
                    constexpr int cc = decltype(C)::value;
                    const T lc = row_bcast<cc>(lb);
                    blk[cc] -= bj * lc;
                    row[cc] -= rj * lc;
                });
                const T l = ib > j ? rj * rp : T(0);
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    const T yj = row_bcast<j>(yb[q]);
                    b[q] -= l * yj;
                    yb[q] -= lb * yj;
                }
                row[j] = ib > j ? l : rj;
            });
        }
    });
}

// Rank-kb update of the panel columns T0 .. p - 1 (rows >= the column) by the
// block of kb columns at K: tiles of 32 rows x 16 columns, round robin over nw
// waves.  The column operand is the MFMA's row operand, so a lane's result
// element lies in row l % 16: consecutive LDS addresses along a column.
template <typename T>
__device__ inline void panel_update(FEHMM_LDS T* F, int m, int p, int K, int kb, int gw, int nw) {
    typedef Mfma16<T> M;
    const int lane = threadIdx.x & 63, l15 = lane & 15, lg = lane >> 4;
    const int T0 = K + kb;
    const int nR = (m - T0 + 15) >> 4, nC = (p - T0 + 15) >> 4;
    int base[4];
    T dk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int kk = 4 * ks + lg, kc = K + min(kk, kb - 1);
        base[ks] = cpkv(kc, m) - kc;
        dk[ks] = F[base[ks] + kc] * (kk < kb ? T(1) : T(0));
    }
    int t = 0;
    for (int J = 0; J < nC; ++J) {
        const int ca = min(T0 + 16 * J + l15, m - 1);
        for (int I = J; I < nR; I += 2, ++t) {
            if ((t & (nw - 1)) != gw) continue;
            T a[4], b[4][2];
            int rb[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) rb[u] = min(T0 + 16 * (I + u) + l15, m - 1);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                a[ks] = F[base[ks] + ca];
#pragma unroll
                for (int u = 0; u < 2; ++u) b[ks][u] = F[base[ks] + rb[u]];
            }
            int cb[4], cv[4];
            T o[2][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                cv[v] = T0 + 16 * J + M::row(lane, v);
                const int cl = min(cv[v], p - 1);
                cb[v] = cpkv(cl, m) - cl;
#pragma unroll
                for (int u = 0; u < 2; ++u) o[u][v] = F[cb[v] + max(rb[u], cl)];
            }
            typename M::V acc[2] = {M::zero(), M::zero()};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u] = M::mma(a[ks] * dk[ks], b[ks][u], acc[u]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int r = T0 + 16 * (I + u) + l15;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    put(F, cv[v] < p && r < m && r >= cv[v], cb[v] + r, (T)(o[u][v] - acc[u][v]));
            }
        }
    }
}

// Update matrix of a front, U(r, c) = sum over children - sum_k L(r, k) D(k)
// L(c, k), packed lower columns: 32 x 32 tiles (2 x 2 MFMA tiles) round robin over
// nw waves, accumulated in registers over all p pivots (eight per step, the next
// step's operands read ahead).  The entries of the first two children are loaded
// before the products, so that their round trip overlaps them: iv holds their
// inverse row maps in LDS ([child][m]), an entry a child does not have is read from
// the workspace's zero (U[0]).
template <typename T>
struct ChildU {  // a child's update matrix: in LDS (u_lds >= 0) or in the workspace
    int lds, off;
};
template <typename T, typename Out>
__device__ inline void schur_tiles(const PanelCtx& pl, int child_begin, int nch, const FEHMM_LDS T* F,
                                   const FEHMM_LDS T* Ul, const FEHMM_LDS int32_t* iv, ChildU<T> ch0, ChildU<T> ch1,
                                   Out dst, int m, int p, int gw, int nw) {
    typedef Mfma16<T> M;
    const int lane = threadIdx.x & 63, l15 = lane & 15, lg = lane >> 4;
    const int mu = m - p, ns = (mu + 31) >> 5;
    const FEHMM_GLB T* Ug = (const FEHMM_GLB T*)pl.U;
    const int blast = cpk(p - 1, m) - (p - 1);
    int t = 0;
    for (int J = 0; J < ns; ++J)
        for (int I = J; I < ns; ++I, ++t) {
            if ((t & (nw - 1)) != gw) continue;
            // MFMA tiles (row, column) of the four: (0, 0) always, (0, 1) off the
            // diagonal, (1, 0) and (1, 1) where the second row tile exists
            const bool off = I > J, two = 32 * I + 16 < mu;
            int r[2], c[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                r[u] = 32 * I + 16 * u + l15;
#pragma unroll
                for (int v = 0; v < 4; ++v) c[u][v] = 32 * J + 16 * u + M::row(lane, v);
            }
            // inv: child row | column offset cpk(row) - row above it, negative where
            // the child has no such row (then the offsets sum to below zero, and
            // element 0, a zero, is read); entries above the diagonal read some entry
            // of the child and are not stored
            auto child_load = [&](const auto* inv, const ChildU<T>& ch, T (&x)[2][2][4]) {
                constexpr int kNone = -(1 << 28);
                const int base = ch.lds >= 0 ? ch.lds : ch.off;
                int ro[2], co[2][4];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int y = inv[p + min(r[u], mu - 1)];
                    ro[u] = y < 0 ? kNone : base + (y & 0xffff);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int z = inv[p + min(c[u][v], mu - 1)];
                        co[u][v] = z < 0 ? kNone : z >> 16;
                    }
                }
                auto get = [&](int u, int w) {
                    if (ch.lds >= 0) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[u][w][v] = Ul[max(ro[u] + co[w][v], 0)];
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[u][w][v] = Ug[max(ro[u] + co[w][v], 0)];
                    }
                };
                get(0, 0);
                if (off) get(0, 1);
                if (two) {
                    get(1, 0);
                    get(1, 1);
                }
            };
            // the children's entries (the products are summed on their own: added to
            // a running sum of both, FP32 factors lost half a digit)
            T val[2][2][4] = {};  // [row tile][column tile][element]
            if (nch > 0) child_load(iv, ch0, val);
            if (nch > 1) {
                T x[2][2][4] = {};
                child_load(iv + m, ch1, x);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int w = 0; w < 2; ++w)
#pragma unroll
                        for (int v = 0; v < 4; ++v) val[u][w][v] += x[u][w][v];
            }
            for (int q = 2; q < nch; ++q) {
                const DevChild ch = load_const(pl.childrec + child_begin + q);
                T x[2][2][4] = {};
                child_load(pl.inv + ch.inv_off, ChildU<T>{ch.u_lds, (int)(ch.U_off * (8 / (int)sizeof(T)))}, x);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int w = 0; w < 2; ++w)
#pragma unroll
                        for (int v = 0; v < 4; ++v) val[u][w][v] += x[u][w][v];
            }
            typename M::V acc[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 2; ++w) acc[u][w] = M::zero();
            int ra[2], rc[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                ra[u] = min(p + 32 * I + 16 * u + l15, m - 1);
                rc[u] = min(p + 32 * J + 16 * u + l15, m - 1);
            }
            // eight columns per step, k = lg and lg + 4 in it: column k starts at
            // base(k) = cpk(k, m) - k, base(k + 8) - base(k) = 8 m - 8 k - 36; past p
            // the last column's address and a zero pivot
            int bs[2], inc[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = lg + 4 * h;
                bs[h] = cpkv(k, m) - k;
                inc[h] = 8 * m - 8 * k - 36;
            }
            T ob[2][2][2], oa[2][2][2], od[2][2];
            auto load = [&](int k0, int h) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int k = k0 + 4 * s + lg, base = min(bs[s], blast);
                    bs[s] += inc[s];
                    inc[s] -= 64;
                    od[h][s] = F[base + min(k, p - 1)] * (k < p ? T(1) : T(0));
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        oa[h][s][u] = F[base + rc[u]];
                        ob[h][s][u] = F[base + ra[u]];
                    }
                }
            };
            auto mul = [&](int h) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const T a0 = oa[h][s][0] * od[h][s], a1 = oa[h][s][1] * od[h][s];
                    acc[0][0] = M::mma(a0, ob[h][s][0], acc[0][0]);
                    if (off) acc[0][1] = M::mma(a1, ob[h][s][0], acc[0][1]);
                    if (two) {
                        acc[1][0] = M::mma(a0, ob[h][s][1], acc[1][0]);
                        acc[1][1] = M::mma(a1, ob[h][s][1], acc[1][1]);
                    }
                }
            };
            load(0, 0);
            for (int k0 = 0; k0 < p; k0 += 16) {
                load(k0 + 8, 1);
                mul(0);
                if (k0 + 8 < p) {
                    load(k0 + 16, 0);
                    mul(1);
                }
            }
#pragma unroll
            for (int w = 0; w < 2; ++w)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int cb = cpkv(c[w][v], mu) - c[w][v];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (r[u] < mu && r[u] >= c[w][v]) dst[cb + r[u]] = val[u][w][v] - acc[u][w][v];
                }
        }
}

// One front s on threads gt = 0..GT-1 (one per front row, m <= GT) and waves gw =
// 0..nw-1: a wave of its own (WAVE), the workgroup, or one half of it beside a
// second front.  F: the panel, ys: [2][NRHS][16] rhs of the block rows, iv: [2][m]
// inverse row maps of the first two children, Ul: update matrices kept in LDS.
// Fronts sharing a step have equal pivot and child counts, so both halves pass the
// same sequence of barriers.  Every global load that needs no other is issued
// first (rows, children's maps, original entries' sources, the first pass of the
// children's panel entries): a front is about three memory round trips.
template <int D, int NRHS, typename T, typename C, bool WAVE>
__device__ inline void front_lds(const PanelCtx& pl, const FEHMM_GLB KeType<D, NRHS, T>* ke, const FEHMM_GLB double* rhs,
                                 FEHMM_LDS int* flag, int s, FEHMM_LDS T* F, FEHMM_LDS C* ys, FEHMM_LDS int32_t* iv,
                                 FEHMM_LDS T* Ul, int gt, int GT, int gw, int nw) {
    constexpr int NEN = 1 << D;
    constexpr int per = 8 / (int)sizeof(T);
    const int lane = threadIdx.x & 63, l15 = lane & 15;
    PROF_T0();
    const DevFront fr = load_const(pl.fronts + s);
    const int m = fr.m, p = fr.p, mu = m - p, nch = fr.child_end - fr.child_begin;
    const FEHMM_GLB int32_t* rows = pl.rows + fr.rows_off;
    FEHMM_GLB T* Lg = (FEHMM_GLB T*)(pl.L + fr.L_off);
    const int lp = cpk(p, m);
    const int i = gt, ic = min(i, m - 1);
    const FEHMM_GLB T* Ug = (const FEHMM_GLB T*)pl.U;
    DevChild ch[2];
    ChildU<T> cu[2] = {{-1, 0}, {-1, 0}};
    int ivr[2] = {-1, -1};
    const int ri = rows[ic];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (q < nch) {
            ch[q] = load_const(pl.childrec + fr.child_begin + q);
            cu[q] = ChildU<T>{ch[q].u_lds, (int)ch[q].U_off * per};
            ivr[q] = (pl.inv + ch[q].inv_off)[ic];
        }
    // first pass of the children's panel entries
    ExtendPass<8, T> ep[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (q < nch) {
            ep[q].index(pl.ea_dst + ch[q].ea_off, ch[q].npre, gt, GT);
            if (cu[q].lds < 0) ep[q].value(Ug + cu[q].off, ch[q].npre, gt, GT);
        }
    for (int t = gt; t < lp; t += GT) F[t] = T(0);
    // rhs of the thread's row: its own entry and the children's
    C b[NRHS], cr[2][NRHS];
#pragma unroll
    for (int q = 0; q < NRHS; ++q) b[q] = i < p ? (C)rhs[ri * NRHS + q] : C(0);
    // child rhs rows: column k of child row r of a child of mc rows at U
    auto child_rhs = [&](const auto* U, int lds, int off, int mc, int r, int k) -> C {
        const int at = rhs_at<T, C>(mc);
        if (lds >= 0) return ((const FEHMM_LDS C*)(Ul + lds + at))[r + k * mc];
        return ((const FEHMM_GLB C*)(U + off + at))[r + k * mc];
    };
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (q < nch) {
            const int o = ivr[q] >= 0 ? (ivr[q] & 0xffff) : 0;
#pragma unroll
            for (int k = 0; k < NRHS; ++k) cr[q][k] = child_rhs(Ug, cu[q].lds, cu[q].off, ch[q].mc, o, k);
            if (i < m) iv[q * m + i] = ivr[q];
        }
    front_sync<WAVE>();
    gather_original<NEN, WAVE ? 8 : 4>(pl, ke, fr.asm_begin, fr.asm_end, gt, GT, F);
    front_sync<WAVE>();
    // original diagonal of the thread's pivot: the scale of the vanishing-pivot test
    const double d0 = (double)F[i < p ? cpkv(i, m) : 0];
    if (nch > 0) front_sync<WAVE>();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (q < nch) {
            if (cu[q].lds >= 0) {
                ep[q].value((const FEHMM_LDS T*)Ul + cu[q].lds, ch[q].npre, gt, GT);
                ep[q].add(ch[q].npre, gt, GT, F);
                extend_add_packed(pl.ea_dst + ch[q].ea_off, (const FEHMM_LDS T*)Ul + cu[q].lds, ch[q].npre, gt + 8 * GT, GT, F);
            } else {
                ep[q].add(ch[q].npre, gt, GT, F);
                extend_add_packed(pl.ea_dst + ch[q].ea_off, Ug + cu[q].off, ch[q].npre, gt + 8 * GT, GT, F);
            }
#pragma unroll
            for (int k = 0; k < NRHS; ++k) b[k] += ivr[q] >= 0 ? cr[q][k] : C(0);
            front_sync<WAVE>();
        }
    for (int q = 2; q < nch; ++q) {
        const DevChild c2 = load_const(pl.childrec + fr.child_begin + q);
        const int v2 = (pl.inv + c2.inv_off)[ic];
        const int o = v2 >= 0 ? (v2 & 0xffff) : 0;
        if (c2.u_lds >= 0)
            extend_add_packed(pl.ea_dst + c2.ea_off, (const FEHMM_LDS T*)Ul + c2.u_lds, c2.npre, gt, GT, F);
        else
            extend_add_packed(pl.ea_dst + c2.ea_off, Ug + (int)c2.U_off * per, c2.npre, gt, GT, F);
#pragma unroll
        for (int k = 0; k < NRHS; ++k) {
            const C v = child_rhs(Ug, c2.u_lds, (int)c2.U_off * per, c2.mc, o, k);
            b[k] += v2 >= 0 ? v : C(0);
        }
        front_sync<WAVE>();
    }
    if (i < 16)
#pragma unroll
        for (int q = 0; q < NRHS; ++q) ys[q * 16 + i] = b[q];
    front_sync<WAVE>();
    PROF_MARK(PH_ASM);
    C mypiv = C(1);
    for (int K = 0; K < p; K += 16) {
        const int kb = min(16, p - K);
        const int par = (K >> 4) & 1;
        // waves that hold rows from K on
        const bool busy = WAVE || (64 * gw < m && 64 * gw + 63 >= K);
        C blk[16], row[16], yb[NRHS];
        if (busy) {
            const int rb = min(K + l15, m - 1);
#pragma unroll
            for (int cc = 0; cc < 16; ++cc) {
                const int col = min(K + cc, p - 1), base = cpk(col, m) - col;
                blk[cc] = (C)F[base + rb];
                row[cc] = (C)F[base + max(ic, K)];
            }
#pragma unroll
            for (int q = 0; q < NRHS; ++q) yb[q] = ys[(par * NRHS + q) * 16 + l15];
        }
        // (the owners of the block rows overwrite what every wave reads here)
        front_sync<WAVE>();
        if (busy) {
            C piv = C(1);
            eliminate16<NRHS, C>(blk, row, yb, b, kb, i - K, piv);
            if (i >= K && i < K + kb) mypiv = piv;
            const int top = i < m ? i - K : -1;  // the row's last column in the block
#pragma unroll
            for (int cc = 0; cc < 16; ++cc) put(F, cc <= top && cc < kb, cpk(K + cc, m) + i - K - cc, (T)row[cc]);
            if (i >= K + 16 && i < K + 32)
#pragma unroll
                for (int q = 0; q < NRHS; ++q) ys[((par ^ 1) * NRHS + q) * 16 + i - K - 16] = b[q];
        }
        front_sync<WAVE>();
        PROF_MARK(PH_DIAG);
        if (K + kb < p) {
            panel_update<T>(F, m, p, K, kb, gw, nw);
            front_sync<WAVE>();
        }
        PROF_MARK(PH_MFMA);
    }
    if (i < p && (!(fabs((double)mypiv) > 1e-14 * fabs(d0)) || !isfinite((double)mypiv))) *flag = 2;
    // D, y, rhs rows of the update matrix, L panel; then the update matrix
    if (i < p) {
        (pl.L + fr.D_off)[i] = (double)mypiv;
#pragma unroll
        for (int q = 0; q < NRHS; ++q) (pl.L + fr.y_off)[q * p + i] = (double)b[q];
    }
    if constexpr (WAVE) {
        // row-major [m][p]: sixteen columns of four rows at a time (what one pass of
        // backsolve_rows reads); entries above the diagonal are some panel entry
        const int lg = lane >> 4;
        for (int j0 = 0; j0 < p; j0 += 16) {
            const int j = min(j0 + l15, p - 1), cj = cpkv(j, m) - j;
            for (int r0 = j0; r0 < m; r0 += 16) {
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = F[cj + max(min(r0 + 4 * u + lg, m - 1), j)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int r = min(r0 + 4 * u + lg, m - 1);  // (clamped lanes repeat a store)
                    Lg[r * p + j] = v[u];
                }
            }
        }
    } else {
        for (int t0 = gt; t0 < lp; t0 += 8 * GT) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = F[min(t0 + u * GT, lp - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) Lg[min(t0 + u * GT, lp - 1)] = v[u];
        }
    }
    if (mu > 0) {
        auto update_out = [&](auto dst, auto rdst) {
            if (i >= p && i < m)
#pragma unroll
                for (int q = 0; q < NRHS; ++q) rdst[q * mu + i - p] = b[q];
            schur_tiles<T>(pl, fr.child_begin, nch, F, Ul, iv, cu[0], cu[1], dst, m, p, gw, nw);
        };
        const int at = rhs_at<T, C>(mu);
        FEHMM_GLB T* const Uo = (FEHMM_GLB T*)(pl.U + fr.U_off);
        if (WAVE && fr.u_lds >= 0) update_out(Ul + fr.u_lds, (FEHMM_LDS C*)(Ul + fr.u_lds + at));
        else update_out(Uo, (FEHMM_GLB C*)(Uo + at));
    }
    front_sync<WAVE>();
    PROF_MARK(PH_OUT);
}

struct Step {
    int32_t front[kStepFronts];
};

template <int D, int NRHS, typename T, typename C>
__device__ __noinline__ void factorize_lds(const RveCtx& c, Smem& sm, T* Fgen) {
    const PanelCtx pl = panel_ctx(c);
    const auto* ke = glb(ke_of<D, NRHS, T>(c));
    const FEHMM_GLB double* rhs = glb((const double*)c.rhs);
    FEHMM_LDS T* F = (FEHMM_LDS T*)Fgen;
    FEHMM_LDS int* flag = (FEHMM_LDS int*)&sm.flag;
    FEHMM_LDS int32_t* iv = (FEHMM_LDS int32_t*)sm.red;  // inverse row maps of two children of every front in flight
    static_assert(sizeof(Smem::red) >= 2 * NT * sizeof(int32_t), "inverse row maps");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int YS = 2 * NRHS * 16 * (int)(sizeof(C) / sizeof(T)) + 2;  // (F[-1]: where masked stores go)
    // small subtrees, one per wave: a task is a contiguous range of fronts, the
    // update matrices inside it stay in the wave's LDS; tasks of a level are
    // independent
    FEHMM_LDS T* const Fw = F + wave * pl.wave_slice;
    FEHMM_LDS T* const Ul = F + pl.ul_base + wave * pl.ul_stride;
    if (pl.ntask_lev > 0) Ul[0] = T(0);  // read for entries a child does not have
    __syncthreads();
    for (int h = 0; h < pl.ntask_lev; ++h) {
        const int k1 = load_const(pl.task_beg + h + 1);
        for (int k = load_const(pl.task_beg + h) + wave; k < k1; k += NWAVE) {
            const int s1 = load_const(pl.task + 2 * k + 1);
            for (int s = load_const(pl.task + 2 * k); s <= s1; ++s)
                front_lds<D, NRHS, T, C, true>(pl, ke, rhs, flag, s, Fw + YS, (FEHMM_LDS C*)Fw, iv + 128 * wave, Ul,
                                               tid & 63, 64, 0, 1);
        }
        __syncthreads();
    }
    // workgroup fronts: one per step on the whole workgroup, or 2 or 4 side by
    // side on two halves (each half takes one or two of them in turn), a half's
    // storage after the other's
    for (int st = 0; st < pl.nwg_steps; ++st) {
        const Step e = load_const((const FEHMM_GLB Step*)pl.wg_steps + st);
        const int nf = e.front[3] >= 0 ? 4 : (e.front[1] >= 0 ? 2 : 1);
        const int G = min(nf, NT / 128);
        const int GT = NT / G, NW = NWAVE / G, g = wave / NW;
        int need = 0;
        for (int j = 0; j < nf; ++j) {
            const DevFront f = load_const(pl.fronts + e.front[j]);
            need = max(need, cpk(f.p, f.m));
        }
        if constexpr (sizeof(C) != sizeof(T)) need = (need + 1) & ~1;
        FEHMM_LDS T* const base = F + g * (need + YS);
        for (int r = 0; r < nf / G; ++r) {
            const int s = load_const(pl.wg_steps + kStepFronts * st + r * G + g);
            front_lds<D, NRHS, T, C, false>(pl, ke, rhs, flag, s, base + YS, (FEHMM_LDS C*)base, iv + 2 * GT * g,
                                            (FEHMM_LDS T*)nullptr, tid - g * GT, GT, wave - g * NW, NW);
        }
    }
}

// 16-pivot blocks of L11^T v = v from the last, by one wave: each rhs column's chain
// in a 16-lane row with DPP broadcasts, then all lanes fold the block into the
// earlier pivots.  L(i, j) at tri[col(j) + i - j].
template <int NRHS, typename Tri, typename Col>
__device__ inline void back_triangle(const Tri* tri, Col col, FEHMM_LDS double* v, int p) {
    const int lane = threadIdx.x & 63, l15 = lane & 15, lg = lane >> 4;
    for (int K = 16 * ((p - 1) >> 4); K >= 0; K -= 16) {
        const int kb = min(16, p - K);
        // block triangle: L(K + cc, K + l15), cc > l15
        const int jl = min(l15, kb - 1), cl = col(K + jl) - jl;
        double Lr[16];
#pragma unroll
        for (int cc = 1; cc < 16; ++cc)
            Lr[cc] = (double)tri[cl + min(max(cc, jl), kb - 1)] * ((cc < kb && cc > l15) ? 1.0 : 0.0);
        // one rhs column per 16-lane row
#pragma unroll
        for (int q0 = 0; q0 < NRHS; q0 += 4) {
            const int q = min(q0 + lg, NRHS - 1);
            double vv = v[q * p + K + jl];
            static_for<0, 15>([&](auto C) {
                constexpr int cc = 15 - decltype(C)::value;
                if (cc < kb) vv -= Lr[cc] * row_bcast<cc>(vv);
            });
            if (l15 < kb && q0 + lg < NRHS) v[q * p + K + l15] = vv;
        }
        front_sync<true>();
        // the block's rows of the earlier columns
        for (int j0 = 0; j0 < K; j0 += 64) {
            const int j = min(j0 + lane, K - 1), cj = col(j) + K - j;
            double lk[16];
#pragma unroll
            for (int cc = 0; cc < 16; ++cc) lk[cc] = (double)tri[cj + min(cc, kb - 1)] * (cc < kb ? 1.0 : 0.0);
#pragma unroll
            for (int q = 0; q < NRHS; ++q) {
                double acc = v[q * p + j];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc) acc -= lk[cc] * v[q * p + K + min(cc, kb - 1)];
                if (j0 + lane < K) v[q * p + j] = acc;
            }
        }
        front_sync<true>();
    }
}

// Backward substitution of one front s (threads gt, waves gw as in front_lds):
//   v = D^-1 y - L21^T x_u on FP64 MFMA (16 pivots x 4 update rows x up to 16 rhs
//   columns; L21 read from global memory once, the update rows split over the
//   waves, their partial sums added in wave order), then the unit triangle by the
//   first wave (back_triangle) from a copy of L11 in LDS.  Bound by latency: the
//   triangle's copy, the first products' operands, D, y and the row numbers are all
//   requested before the first wait, so a front is two memory round trips.
// vb: FP64 scratch of `cap` doubles: [NRHS][p] pivot values, [NRHS][mu] update rows'
// solution, [nw][NRHS][p] partial sums, then the packed triangle where it fits (else
// it is read from global memory).
template <int D, int NRHS, typename T, bool WAVE>
__device__ inline void backsolve_front(const PanelCtx& pl, int s, FEHMM_LDS double* vb, int cap, FEHMM_GLB double* x,
                                       int gt, int GT, int gw, int nw) {
    typedef Mfma16<double> M;
    const int lane = threadIdx.x & 63, l15 = lane & 15, lg = lane >> 4;
    const DevFront fr = load_const(pl.fronts + s);
    const int m = fr.m, p = fr.p, mu = m - p;
    const FEHMM_GLB int32_t* rows = pl.rows + fr.rows_off;
    const FEHMM_GLB T* Lg = (const FEHMM_GLB T*)(pl.L + fr.L_off);
    const FEHMM_GLB double* Dg = pl.L + fr.D_off;
    const FEHMM_GLB double* yg = pl.L + fr.y_off;
    const int npart = mu > 0 ? nw : 0;
    FEHMM_LDS double* v = vb;                // [NRHS][p]
    FEHMM_LDS double* xs = vb + NRHS * p;    // [NRHS][mu]
    FEHMM_LDS double* part = vb + NRHS * m;  // [npart][NRHS][p]
    const int scratch = NRHS * (m + npart * p), ntri = p * (p + 1) / 2;
    FEHMM_LDS T* tri = (FEHMM_LDS T*)(vb + scratch);
    const bool staged = scratch + (ntri * (int)sizeof(T) + 7) / 8 <= cap;
    // one row and one pivot per thread first (m <= GT but for four-front steps)
    const int r0 = mu > 0 ? rows[p + min(gt, mu - 1)] : 0;
    const int jp = min(gt, p - 1);
    const double d0 = Dg[jp];
    double y0[NRHS];
#pragma unroll
    for (int q = 0; q < NRHS; ++q) y0[q] = yg[q * p + jp];
    // the products' first operands: tile 0, the first eight of this wave's k-steps
    const int nks = (mu + 3) >> 2;
    T a[8];
    auto a_load = [&](int t, int k0) {
        const int j = min(16 * t + l15, p - 1), col = cpkv(j, m) - j + p;
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = Lg[col + min(4 * (k0 + u * nw) + lg, mu - 1)];
    };
    if (mu > 0) a_load(0, gw);
    if (staged) {  // columns of the triangle, wave by wave, eight columns in flight
        for (int jb = gw; jb < p; jb += 8 * nw)
            for (int h = lane; h < p - jb; h += 64) {  // (every eighth column is no longer than its first)
                T c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = min(jb + u * nw, p - 1);
                    c[u] = Lg[cpk(j, m) + min(h, p - 1 - j)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = jb + u * nw;
                    if (j + h < p) tri[cpk(j, p) + h] = c[u];
                }
            }
    }
    if (gt < p)
#pragma unroll
        for (int q = 0; q < NRHS; ++q) v[q * p + gt] = y0[q] / d0;
    for (int j = gt + GT; j < p; j += GT)
#pragma unroll
        for (int q = 0; q < NRHS; ++q) v[q * p + j] = yg[q * p + j] / Dg[j];
    for (int i = gt; i < mu; i += GT) {
        const int xr = (i == gt ? r0 : rows[p + i]) * NRHS;
#pragma unroll
        for (int q = 0; q < NRHS; ++q) xs[q * mu + i] = x[xr + q];
    }
    front_sync<WAVE>();
    if (mu > 0) {
        for (int t = 0; 16 * t < p; ++t) {
            M::V acc[2] = {M::zero(), M::zero()};
            for (int k0 = gw; k0 < nks; k0 += 8 * nw) {
                if (t > 0 || k0 != gw) a_load(t, k0);
                double bx[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = 4 * (k0 + u * nw) + lg;
                    bx[u] = xs[(NRHS == 1 ? 0 : min(l15, NRHS - 1) * mu) + min(i, mu - 1)];
                    bx[u] *= (i < mu && l15 < NRHS) ? 1.0 : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k0 + u * nw < nks) acc[u & 1] = M::mma((double)a[u], bx[u], acc[u & 1]);
            }
            // result element e of lane: pivot 16 t + row(lane, e), rhs column l15
            if (l15 < NRHS)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int jj = 16 * t + M::row(lane, e);
                    if (jj < p) part[(gw * NRHS + l15) * p + jj] = acc[0][e] + acc[1][e];
                }
        }
        front_sync<WAVE>();
        for (int t = gt; t < p * NRHS; t += GT) {
            double sum = part[t];
            for (int w = 1; w < nw; ++w) sum += part[w * NRHS * p + t];
            v[t] -= sum;
        }
        front_sync<WAVE>();
    }
    if (gw == 0) {
        if (staged) back_triangle<NRHS>((const FEHMM_LDS T*)tri, [&](int j) { return cpkv(j, p); }, v, p);
        else back_triangle<NRHS>(Lg, [&](int j) { return cpkv(j, m); }, v, p);
    }
    front_sync<WAVE>();
    for (int j = gt; j < p; j += GT) {
        const int xr = rows[j] * NRHS;
#pragma unroll
        for (int q = 0; q < NRHS; ++q) x[xr + q] = v[q * p + j];
    }
    front_sync<WAVE>();
}

// Backward substitution of four wave fronts k .. k + 3 of the plan's list at once, one
// per 16-lane row of the wave (fronts past `end` repeat the last and store nothing).
// Lane l of a row holds pivot K + l of each 16-pivot block K, from the last block: the
// rows below the block are folded in with their solution values read from LDS
// (xk, [NRHS][64] of each front), the block's own triangle by DPP broadcasts.  L is
// row-major, so a row's 16 entries are one 128-byte load and a chunk of 16 rows is
// requested while the one before it is used.  Bound by those loads' latency.  Against
// one front per wave (MFMA products, packed columns) the wave fronts of a 32 x 32
// solve take 0.13 instead of 0.31 Mclk; with the triangles in LDS above, 4096 of them
// 55.3 -> 52 ms (FP32 factors 46.9 -> 43.3).
template <int NRHS, typename T>
__device__ inline void backsolve_rows(const PanelCtx& pl, int k, int end, FEHMM_LDS double* xk, FEHMM_GLB double* x) {
    constexpr int CH = NRHS == 1 ? 16 : 8;  // rows per chunk (registers)
    const int lane = threadIdx.x & 63, l = lane & 15, r = lane >> 4;
    BackRec f;
    {
        const FEHMM_GLB int32_t* w = (const FEHMM_GLB int32_t*)(pl.back + min(k + r, end - 1));
        f = BackRec{w[0], w[1], w[2], w[3], w[4], w[5]};
    }
    const bool live = k + r < end;
    const int m = f.m, p = f.p;
    const FEHMM_GLB int32_t* rows = pl.rows;
    const FEHMM_GLB T* Lg = (const FEHMM_GLB T*)pl.L;
    const int Lo = f.L_off * (8 / (int)sizeof(T));
    xk += r * (NRHS * 64 + 4);
    auto row_max = [](int w) {  // largest of the four rows' values
        w = max(w, __shfl_xor(w, 16));
        return uni(max(w, __shfl_xor(w, 32)));
    };
    const int pmax = row_max(p);
    // solution of the update rows
    {
        int ri[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ri[u] = rows[f.rows_off + min(p + 16 * u + l, m - 1)] * NRHS;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (p + 16 * u + l < m)
#pragma unroll
                for (int q = 0; q < NRHS; ++q) xk[q * 64 + p + 16 * u + l] = x[ri[u] + q];
    }
    for (int K = 16 * ((pmax - 1) >> 4); K >= 0; K -= 16) {
        const int kb = min(max(p - K, 0), 16), j = min(K + l, p - 1);
        const bool act = l < kb;
        const int ri = rows[f.rows_off + j] * NRHS;
        const double d = (pl.L + f.D_off)[j];
        double v[NRHS];
#pragma unroll
        for (int q = 0; q < NRHS; ++q) v[q] = (pl.L + f.y_off)[q * p + j];
        T Lr[16];
#pragma unroll
        for (int cc = 1; cc < 16; ++cc) Lr[cc] = Lg[Lo + min(K + cc, m - 1) * p + j];
        // rows K + kb .. m - 1 in chunks
        const int i0 = K + kb, trip = row_max(kb > 0 ? m - i0 : 0);
        T a[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) a[u] = Lg[Lo + min(i0 + u, m - 1) * p + j];
        front_sync<true>();
        double acc[NRHS];
#pragma unroll
        for (int q = 0; q < NRHS; ++q) acc[q] = 0.0;
        for (int t = 0; t < trip || t == 0; t += CH) {
            T b[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) b[u] = Lg[Lo + min(i0 + t + CH + u, m - 1) * p + j];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const int i = i0 + t + u;
                const double lv = i < m ? (double)a[u] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) acc[q] += lv * (i < m ? xk[q * 64 + i] : 0.0);
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) a[u] = b[u];
        }
#pragma unroll
        for (int q = 0; q < NRHS; ++q) v[q] = v[q] / d - acc[q];
        static_for<0, 15>([&](auto C) {
            constexpr int cc = 15 - decltype(C)::value;
            if (cc < pmax - K) {  // (uniform)
                const double lc = (cc < kb && cc > l) ? (double)Lr[cc] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) v[q] -= lc * row_bcast<cc>(v[q]);
            }
        });
        if (act) {
#pragma unroll
            for (int q = 0; q < NRHS; ++q) {
                xk[q * 64 + j] = v[q];
                if (live) x[ri + q] = v[q];
            }
        }
        front_sync<true>();
    }
}

// backward substitution L^T x = D^-1 y with NRHS columns; y is each front's
// stored forward-substituted rhs, x (node-major [dof][NRHS], FP64) receives the
// solution.  The workgroup fronts in the plan's steps, in reverse (four-front steps
// one front per wave), then the small subtrees four fronts per wave, parents first.
// S: FP64 scratch, `slice` doubles per wave.
template <int D, int NRHS, typename T>
__device__ __noinline__ void backsolve_lds(const RveCtx& c, double* Sgen, double* xgen, int slice) {
    const PanelCtx pl = panel_ctx(c);
    FEHMM_LDS double* S = (FEHMM_LDS double*)Sgen;
    FEHMM_GLB double* x = glb(xgen);
    slice = uni(slice);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    zero_pinned<D>(c, xgen, NRHS);
    for (int st = pl.nwg_steps - 1; st >= 0; --st) {
        const Step e = load_const((const FEHMM_GLB Step*)pl.wg_steps + st);
        if (e.front[3] >= 0) {
            backsolve_front<D, NRHS, T, true>(pl, load_const(pl.wg_steps + kStepFronts * st + wave), S + wave * slice, slice,
                                              x, tid & 63, 64, 0, 1);
            __syncthreads();
            continue;
        }
        const int G = e.front[1] >= 0 ? 2 : 1;
        const int GT = NT / G, NW = NWAVE / G, g = wave / NW;
        backsolve_front<D, NRHS, T, false>(pl, load_const(pl.wg_steps + kStepFronts * st + g), S + g * NW * slice,
                                           NW * slice, x, tid - g * GT, GT, wave - g * NW, NW);
    }
    // small subtrees: four fronts per wave, parents (greater height) first
    PROF_T0();
    for (int h = pl.nwave_h - 1; h >= 0; --h) {
        const int k1 = load_const(pl.wave_hbeg + h + 1);
        for (int k = load_const(pl.wave_hbeg + h) + 4 * wave; k < k1; k += 4 * NWAVE)
            backsolve_rows<NRHS, T>(pl, k, k1, S + wave * slice, x);
        __syncthreads();
    }
    PROF_MARK(PH_TRSM);
}

// global -> LDS copy, eight strides per pass: all loads first, then all stores
// (the compiler does not move a load past a store that may alias it)
template <typename T>
__device__ inline void copy_in(T* dst, const T* src, int n, int first, int stride) {
    for (int t0 = first; t0 < n; t0 += 8 * stride) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[min(t0 + u * stride, n - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (t0 + u * stride < n) dst[t0 + u * stride] = v[u];
    }
}
// forward substitution L y = b for a new rhs b (node-major [dof][NRHS], FP64,
// overwritten): fronts in elimination order; per front the pivot rows are
// solved in 16-pivot blocks (readlane chain in wave 0) and folded into the rows
// below; the update rows are scattered back into b; the pivot part is stored as
// the front's forward-substituted rhs for backsolve_lds.
template <int D, int NRHS, typename T>
__device__ __noinline__ void forward_lds(const RveCtx& c, Smem& sm, T* F, double* b, int front_elems) {
    const DevPlan& pl = *c.plan;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* vb = reinterpret_cast<double*>(F);  // [NRHS][m] front rows of b
    for (int s = 0; s < pl.nfront; ++s) {
        const DevFront fr = pl.fronts[s];
        const int m = fr.m, p = fr.p;
        const int32_t* rows = pl.rows + fr.rows_off;
        const T* Lp = reinterpret_cast<const T*>(c.L + fr.L_off);
        {
            // stage the panel after the FP64 rows of b when both fit
            const int vneed = (int)((sizeof(double) / sizeof(T)) * m * NRHS);
            const int lp = fr.wave ? m * p : cpk(p, m);
            if (vneed + lp <= front_elems) {
                T* Ls = F + vneed;
                copy_in(Ls, Lp, lp, tid, NT);
                Lp = Ls;
            }
        }
        double* yg = c.L + fr.y_off;
        // L(i, j), i >= j: wave fronts row-major, the others packed columns
        const bool wv = fr.wave != 0;
        auto at = [&](int i, int j) { return wv ? i * p + j : cpk(j, m) + i - j; };
        for (int t = tid; t < m * NRHS; t += NT) {
            const int i = t % m, q = t / m;
            vb[t] = (i < p) ? b[(int64_t)rows[i] * NRHS + q] : 0.0;
        }
        __syncthreads();
        if (p <= 64) {
            // the pivot triangle by wave 0 alone (lane = pivot row, readlane
            // broadcasts of the finished values), then every row below folds in
            // all p pivots in one pass
            if (wave == 0) {
                double vv[NRHS];
#pragma unroll
                for (int q = 0; q < NRHS; ++q) vv[q] = lane < p ? vb[q * m + lane] : 0.0;
                // four pivots per pass, read ahead of the updates (row
                // max(min(lane, m - 1), j + 1) of column j, inside the panel for
                // every lane; masked values)
                for (int j0 = 0; j0 < p - 1; j0 += 4) {
                    double l[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = min(j0 + u, p - 2);
                        const int row = max(min(lane, m - 1), j + 1);
                        l[u] = (double)Lp[at(row, j)] *
                               ((j0 + u < p - 1 && lane > j && lane < p) ? 1.0 : 0.0);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int q = 0; q < NRHS; ++q) vv[q] -= l[u] * readlane_d(vv[q], min(j0 + u, p - 2));
                }
#pragma unroll
                for (int q = 0; q < NRHS; ++q)
                    if (lane < p) vb[q * m + lane] = vv[q];
            }
            __syncthreads();
            for (int i = p + tid; i < m; i += NT) {
                double acc[NRHS];
#pragma unroll
                for (int q = 0; q < NRHS; ++q) acc[q] = vb[q * m + i];
#pragma unroll 4
                for (int j = 0; j < p; ++j) {
                    const double l = (double)Lp[at(i, j)];
#pragma unroll
                    for (int q = 0; q < NRHS; ++q) acc[q] -= l * vb[q * m + j];
                }
#pragma unroll
                for (int q = 0; q < NRHS; ++q) vb[q * m + i] = acc[q];
            }
            __syncthreads();
        }
        for (int K = 0; K < (p <= 64 ? 0 : p); K += 16) {
            const int kb = min(16, p - K);
            if (wave == 0) {
                const bool own = lane < kb;
                double Lr[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc)
                    Lr[cc] = (own && cc < kb && cc < lane) ? (double)Lp[at(K + lane, K + cc)] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double vv = own ? vb[q * m + K + lane] : 0.0;
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc) {
                        if (cc < kb) {
                            const double yc = readlane_d(vv, cc);
                            if (lane > cc) vv -= Lr[cc] * yc;
                        }
                    }
                    if (own) vb[q * m + K + lane] = vv;
                }
            }
            __syncthreads();
            for (int i = K + kb + tid; i < m; i += NT) {
                double lk[16];
#pragma unroll
                for (int cc = 0; cc < 16; ++cc) lk[cc] = (cc < kb) ? (double)Lp[at(i, K + cc)] : 0.0;
#pragma unroll
                for (int q = 0; q < NRHS; ++q) {
                    double acc = vb[q * m + i];
#pragma unroll
                    for (int cc = 0; cc < 16; ++cc)
                        if (cc < kb) acc -= lk[cc] * vb[q * m + K + cc];
                    vb[q * m + i] = acc;
                }
            }
            __syncthreads();
        }
        for (int t = tid; t < p * NRHS; t += NT) {
            const int j = t % p, q = t / p;
            yg[(int64_t)q * p + j] = vb[q * m + j];
        }
        for (int t = tid; t < (m - p) * NRHS; t += NT) {
            const int i = t % (m - p), q = t / (m - p);
            b[(int64_t)rows[p + i] * NRHS + q] += vb[q * m + p + i];  // rows[p+i] holds b; add the update
        }
        __syncthreads();
    }
}

// out = b - K x with the stored FP64 element tangents, free rows only; node-major
// [dof][NRHS], one node per thread
template <int D, int NRHS>
__device__ __noinline__ void residual_ke(const RveCtx& c, const double* bgen, const double* xgen, double* ogen) {
    constexpr int NEN = 1 << D;
    const int n = uni(c.n), ne = uni(c.ne), nn = uni(c.nn);
    const FEHMM_GLB double* b = glb(bgen);
    const FEHMM_GLB double* x = glb(xgen);
    const FEHMM_GLB double* ke = glb(c.ke);
    FEHMM_GLB double* out = glb(ogen);
    for (int v = threadIdx.x; v < nn; v += NT) {
        const bool pin = is_pinned(*c.plan, v);
        int el[NEN];
        elements_of_node<D>(n, v, el);
        double acc[D][NRHS];
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int q = 0; q < NRHS; ++q) acc[i][q] = 0.0;
        // (a rolled loop over the 2^d elements: a is uniform, so the entry planes
        // are scalar)
#pragma unroll 1
        for (int a = 0; a < NEN; ++a) {
            int e = 0;
#pragma unroll
            for (int h = 0; h < NEN; ++h) e = h == a ? el[h] : e;
            int nodes[NEN];
            nodes_of_element<D>(n, e, nodes);
#pragma unroll
            for (int bb = 0; bb < NEN; ++bb)
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    double xr[NRHS];
#pragma unroll
                    for (int q = 0; q < NRHS; ++q) xr[q] = x[(nodes[bb] * D + k) * NRHS + q];
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        const double kv = ke[sym_entry(D, a, i, bb, k) * ne + e];
#pragma unroll
                        for (int q = 0; q < NRHS; ++q) acc[i][q] += kv * xr[q];
                    }
                }
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int q = 0; q < NRHS; ++q)
                out[(v * D + i) * NRHS + q] = pin ? 0.0 : b[(v * D + i) * NRHS + q] - acc[i][q];
    }
}

template <int D>
__device__ double free_norm2(const RveCtx& c, Smem& sm, const double* R) {
    double v[1] = {0.0};
    for (int t = threadIdx.x; t < c.nn * D; t += NT)
        if (!is_pinned(*c.plan, t / D)) v[0] += R[t] * R[t];
    block_sum<1>(v, sm);
    return sm.outv[0];
}

// per-RVE context (plan, phases, Lame table, slot regions) and the uniform-grid
// constants in LDS: grad N at the Gauss points, w|J|, Fbar, the tolerance
template <int D>
__device__ inline void rve_setup(const SolveArgs& a, int rve, double* base, RveCtx& c, Smem& sm) {
    constexpr int NEN = 1 << D, ND = NEN * D, D2 = D * D;
    c.plan = &a.plans[a.rve_plan[rve]];
    c.d = D;
    c.n = c.plan->n;
    c.ne = c.plan->nelem;
    c.nn = c.plan->nnode;
    c.nen = NEN;
    c.nd = ND;
    c.phase = a.phase_pool + a.rve_phase[rve];
    c.lame = a.lame_pool + a.rve_lame[rve];
    const int kind = a.rve_kind ? a.rve_kind[rve] : 0;
    c.law = kind & 0xff;
    c.elem = (kind >> 8) & 0xff;
    c.ke32 = 0;
    c.w = base + a.lay.w;
    c.wt = base + a.lay.wt;
    c.R = base + a.lay.R;
    c.rhs = base + a.lay.rhs;
    c.x = base + a.lay.x;
    c.fe = base + a.lay.fe;
    c.ke = base + a.lay.ke;
    c.re = base + a.lay.re;
    c.L = base + a.lay.L;
    c.U = base + a.lay.U;
    c.S = base + a.lay.S;
    // constants of the uniform grid: grad N at the integration points, w|J|.
    // P1: point p is the Kuhn simplex of axis order perm(p), vertices 0,
    // e_s0, e_s0 + e_s1, ..., 1; a cell corner o is its vertex j when o holds j
    // ones, at s0 .. s(j-1); barycentric gradients -e_s0, e_s(j-1) - e_sj,
    // e_s(d-1) (over h), zero at the corners the simplex misses
    if (c.elem == 1 && threadIdx.x < 8 * NEN) {
        const int p = threadIdx.x / NEN, an = threadIdx.x % NEN;
        // the d! axis orders (p < D!: 2 in 2D, 6 in 3D), lexicographic
        const int perm3[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
        const int perm2[2][3] = {{0, 1, 2}, {1, 0, 2}};
        const int npt = D == 2 ? 2 : 6;
        int oa[3] = {0, 0, 0};
        local_offset(D, an, oa);
        double g[3] = {0.0, 0.0, 0.0};
        if (p < npt) {
            const int* pm = D == 2 ? perm2[p] : perm3[p];
            int ones = 0;
            for (int k = 0; k < D; ++k) ones += oa[k];
            bool vert = true;
            for (int q = 0; q < ones; ++q) vert = vert && oa[pm[q]] == 1;
            if (vert) {
                const double ih = (double)c.n;
                if (ones == 0) g[pm[0]] = -ih;
                else if (ones == D) g[pm[D - 1]] = ih;
                else { g[pm[ones - 1]] = ih; g[pm[ones]] = -ih; }
            }
        }
        for (int k = 0; k < 3; ++k) sm.dN[(p * 8 + an) * 3 + k] = g[k];
    } else if (c.elem == 0 && threadIdx.x < NEN * NEN) {
        const int gp = threadIdx.x / NEN, an = threadIdx.x % NEN;
        const double gq = 0.57735026918962576451, h = 1.0 / c.n;
        int og[3] = {0, 0, 0}, oa[3] = {0, 0, 0};
        local_offset(D, gp, og);
        local_offset(D, an, oa);
        for (int k = 0; k < D; ++k) {
            double v = 1.0;
            for (int q = 0; q < D; ++q) {
                const double sa = oa[q] ? 1.0 : -1.0, xi = og[q] ? gq : -gq;
                v *= (q == k) ? 0.5 * sa : 0.5 * (1.0 + sa * xi);
            }
            sm.dN[(gp * 8 + an) * 3 + k] = v * 2.0 / h;
        }
    }
    if (threadIdx.x < D2) sm.Fbar[threadIdx.x] = a.F[(int64_t)rve * D2 + threadIdx.x];
    if (threadIdx.x == 0) {
        double h = 1.0 / c.n, wj = 1.0;
        for (int k = 0; k < D; ++k) wj *= (c.elem == 1 ? h : 0.5 * h);
        if (c.elem == 1) wj /= (D == 2 ? 2.0 : 6.0);  // simplex volume h^d / d!
        sm.wJ = wj;
        c.U[0] = 0.0;  // the zero that fronts read for entries a child does not have
        sm.flag = 0;
        sm.atol = a.atol >= 0 ? a.atol : a.rve_atol[rve];
    }
    __syncthreads();
}

// factorization, backward and forward substitution of the RVE's plan: panels in LDS
// or fronts in global memory (3D plans in LDS never carry d^2 + 1 columns)
template <int D, int NRHS, typename T>
__device__ inline void factorize(const RveCtx& c, Smem& sm, T* lds) {
    if constexpr (kLdsPlans && (D == 2 || NRHS <= D * D))
        if (c.plan->lds_ok) {
            // (FP32 factors of these plans condense from a factorization in FP64, tan64:
            // no d^2 columns in FP32)
            if constexpr (D == 2 && NRHS != D * D && sizeof(T) == 4)
                if (c.plan->wide_rhs) {
                    factorize_lds<D, NRHS, T, double>(c, sm, lds);
                    return;
                }
            factorize_lds<D, NRHS, T, T>(c, sm, lds);
            return;
        }
    factorize_glb<D, T>(c, sm, NRHS, lds);
}
template <int D, int NRHS, typename T>
__device__ inline void backsolve(const RveCtx& c, Smem& sm, double* x, double* lds, int slice) {
    if constexpr (kLdsPlans && (D == 2 || NRHS <= D * D))
        if (c.plan->lds_ok) {
            backsolve_lds<D, NRHS, T>(c, lds, x, slice);
            return;
        }
    backsolve_glb<D, NRHS, T>(c, sm, x, lds);
}
template <int D, int NRHS, typename T>
__device__ inline void forward(const RveCtx& c, Smem& sm, double* b, T* lds, int elems) {
    if constexpr (kLdsPlans)
        if (c.plan->lds_ok) {
            forward_lds<D, NRHS, T>(c, sm, lds, b, elems);
            return;
        }
    forward_glb<D, NRHS, T>(c, sm, b);
}

template <int D, typename T>
__global__ __launch_bounds__(NT, 2) void rve_solve_kernel(SolveArgs a) {
    __shared__ Smem sm;
    extern __shared__ double dynRaw[];
    T* dynF = reinterpret_cast<T*>(dynRaw);
    constexpr bool IR = sizeof(T) < sizeof(double);  // FP32 factors + FP64 refinement
    constexpr int NEN = 1 << D, ND = NEN * D, D2 = D * D;
    const int64_t slot = blockIdx.x;
    double* base = a.ws + slot * a.lay.stride;
    for (;;) {
        if (threadIdx.x == 0) {
            // queue length: the launch's share of the batch, or a device-side count of
            // a subset list (entries outside [0, B) or of another launch are skipped)
            const unsigned int nq = (unsigned int)(a.count_dev ? min((int64_t)max(*a.count_dev, 0), a.B) : a.nq);
            int r = -1;
            for (;;) {
                if (a.skip && *a.skip) break;
                const unsigned int idx = atomicAdd(a.counter, 1u);
                if (idx >= nq) break;
                const int cand = a.order[idx];
                if (cand >= 0 && (int64_t)cand < a.B && (a.cls < 0 || a.plans[a.rve_plan[cand]].cls == a.cls)) {
                    r = cand;
                    break;
                }
            }
            sm.rve = r;
        }
        __syncthreads();
        const int rve = sm.rve;
        if (rve < 0) return;
        RveCtx c;
        rve_setup<D>(a, rve, base, c, sm);
        c.ke32 = IR ? 1 : 0;
        double* ir1 = base + a.lay.ir1;
        double* ir2 = base + a.lay.ir2;
        const int ndof = c.nn * D;
        // input checks and initial guess
        bool finite_in = true;
#pragma unroll
        for (int q = 0; q < D2; ++q) finite_in = finite_in && isfinite(sm.Fbar[q]);
        double* wst = a.wstate ? a.wstate + a.state_off[rve] : nullptr;
        for (int t = threadIdx.x; t < ndof; t += NT) c.w[t] = (wst && !is_pinned(*c.plan, t / D)) ? wst[t] : 0.0;
        __syncthreads();
        int status = 0, it = 0;
        bool capped = false, restarted = false;
        if (!finite_in) status = 4;
        double r0 = 0.0, rprev = 0.0;
        // tangent from the last Newton factorization (LDS plans in 2D, global-
        // front plans in either dimension): when the
        // quadratic model r_next ~ r^3 / r_prev^2 puts the next residual within
        // the tolerance, the factorization also forward-substitutes the d^2
        // columns Y of the current state (rhs [dof][1 + d^2], R first); if the
        // next state converges, X ~ K^-1 Y is one backward substitution away
        constexpr int NSPEC = D2 + 1;
        const bool spec_on = NSPEC <= kMaxNrhs && a.reuse_tan && (D == 2 || !c.plan->lds_ok);
        bool spec = false;  // the last factorization carries the Y columns
        PROF_T0();
        while (status == 0) {
            PROF_RESET();
            if constexpr (IR) element_tangents<D, float>(c, sm, c.w);
            else element_tangents<D, double>(c, sm, c.w);
            __syncthreads();
            PROF_MARK(PH_ELEM);
            if (sm.flag) {
                if (it == 0 && wst && !restarted) {
                    // a stored fluctuation that folds an element under the new
                    // Fbar is discarded: restart from w = 0 (J = det Fbar > 0)
                    restarted = true;
                    for (int t = threadIdx.x; t < ndof; t += NT) c.w[t] = 0.0;
                    __syncthreads();
                    if (threadIdx.x == 0) sm.flag = 0;
                    __syncthreads();
                    continue;
                }
                status = 2;
                break;
            }
            node_gather<D>(c, c.fe, 1, c.R, 1, 0);
            __syncthreads();
            const double rn = sqrt(free_norm2<D>(c, sm, c.R));
            PROF_MARK(PH_GATHER);
            if (!isfinite(rn)) { status = 4; break; }
            if (it == 0) r0 = rn;
            if (rn <= a.rtol * r0 + sm.atol) break;
            if (it == a.max_iter) {
                if (a.flags & 1) capped = true;  // outputs at the last state, reported as NOCONV
                else status = 1;
                break;
            }
            spec = spec_on && it >= 1 && rn * rn * rn <= (a.rtol * r0 + sm.atol) * rprev * rprev;
            rprev = rn;
            if constexpr (NSPEC <= kMaxNrhs) {
                if (spec) {
                    element_coupling<D>(c, sm, c.w);
                    __syncthreads();
                    node_gather<D>(c, c.re, D2, c.rhs, NSPEC, 1);
                    for (int t = threadIdx.x; t < ndof; t += NT) c.rhs[(int64_t)t * NSPEC] = -c.R[t];
                    __syncthreads();
                    factorize<D, NSPEC, T>(c, sm, dynF);
                }
            }
            if (!spec) {
                for (int t = threadIdx.x; t < ndof; t += NT) c.rhs[t] = -c.R[t];
                __syncthreads();
                factorize<D, 1, T>(c, sm, dynF);
            }
            if (sm.flag) { status = 3; break; }
            PROF_RESET();
            if constexpr (NSPEC <= kMaxNrhs) {
                if (spec) {
                    // every column in one backward sweep, into the rhs buffer
                    // ([dof][1 + d^2]): the Newton step, then X' = K'^-1 Y', which
                    // stays there for the condensation if the next state converges
                    backsolve<D, NSPEC, T>(c, sm, c.rhs, dynRaw, a.bs_slice);
                    for (int t = threadIdx.x; t < ndof; t += NT) c.x[t] = c.rhs[(int64_t)t * NSPEC];
                    __syncthreads();
                }
            }
            if (!spec) {
                backsolve<D, 1, T>(c, sm, c.x, dynRaw, a.bs_slice);
            }
            PROF_MARK(PH_BACK);
            if constexpr (IR) {
                // refinement against the FP64 tangent: dx = K32^-1 (b - K64 x), with
                // K64 x computed matrix-free from the elements in FP64
                for (int ref = 0; ref < a.ir_max; ++ref) {
                    element_apply<D>(c, sm, c.w, c.x);
                    __syncthreads();
                    residual_act<D>(c, c.R, -1.0, ir1);  // b = -R
                    __syncthreads();
                    const double rl2 = sqrt(free_norm2<D>(c, sm, ir1));
                    if (!(rl2 > a.ir_eta * rn)) break;
                    forward<D, 1, T>(c, sm, ir1, dynF, a.lds_elems);
                    backsolve<D, 1, T>(c, sm, ir2, dynRaw, a.bs_slice);
                    for (int t = threadIdx.x; t < ndof; t += NT) c.x[t] += ir2[t];
                    __syncthreads();
                }
            }
            // step with det F backtracking
            double alpha = 1.0;
            bool ok = false;
            for (int bt = 0; bt <= a.backtrack; ++bt) {
                for (int t = threadIdx.x; t < ndof; t += NT) c.wt[t] = c.w[t] + alpha * c.x[t];
                if (threadIdx.x == 0) sm.flag = 0;
                __syncthreads();
                element_check<D>(c, sm, c.wt);
                __syncthreads();
                const int bad = sm.flag;
                __syncthreads();
                if (!bad) { ok = true; break; }
                alpha *= 0.5;
            }
            if (threadIdx.x == 0) sm.flag = 0;
            PROF_MARK(PH_LINE);
            if (!ok) { status = 2; break; }
            for (int t = threadIdx.x; t < ndof; t += NT) c.w[t] = c.wt[t];
            __syncthreads();
            ++it;
        }
        __syncthreads();
        PROF_RESET();
        double* Pout = a.P + (int64_t)rve * D2;
        double* Aout = a.A ? a.A + (int64_t)rve * D2 * D2 : nullptr;
        if (status == 0) {
            // the condensation from X = K'^-1 Y', solved with the last Newton step
            // (still in the rhs buffer, columns 1..d^2): used where the last
            // factorized residual was within 1e-4 of the initial one, so the
            // stationary form's error (second order in that step) stays far
            // below the tangent's tolerance; in 2D element_average<D, true> sums
            // the condensed tangent itself
            const bool stale = Aout && spec && !capped && rprev <= 1e-4 * r0;
            const bool stale2 = stale && D == 2;
            constexpr int NA = D2 * (D2 + 1) / 2;  // lower triangle of a symmetric d^2 x d^2
            double accP[D2], accA[NA];
            if constexpr (D == 2) {
                if (stale2) element_average<D, true>(c, sm, c.w, accP, accA, c.rhs + 1, NSPEC);
                else element_average<D, false>(c, sm, c.w, accP, accA, nullptr, 0);
            } else {
                element_average<D, false>(c, sm, c.w, accP, accA, nullptr, 0);
            }
            if (Aout && !stale2) element_coupling<D>(c, sm, c.w);
            // entry (threadIdx.x / d^2, threadIdx.x % d^2) of such a triangle
            const int sym_g = threadIdx.x / D2, sym_h = threadIdx.x % D2;
            const int sym_at = max(sym_g, sym_h) * (max(sym_g, sym_h) + 1) / 2 + min(sym_g, sym_h);
            __syncthreads();
            block_sum<D2>(accP, sm);
            if (threadIdx.x < D2) Pout[threadIdx.x] = sm.outv[threadIdx.x];
            __syncthreads();
            if (Aout && stale2) {
                block_sum<NA>(accA, sm);
                if (threadIdx.x < D2 * D2) Aout[threadIdx.x] = sm.outv[sym_at];
                __syncthreads();
            } else if (Aout) {
                block_sum<NA>(accA, sm);
                double Aavg = threadIdx.x < D2 * D2 ? sm.outv[sym_at] : 0.0;
                __syncthreads();
                if (c.ke32) {  // the FP64 tangents of w for the condensation
                    element_tangents<D, double>(c, sm, c.w);
                    __syncthreads();
                }
                // otherwise (3D) the stationary form assembled below, refined
                // while ||Y - K X||_F > 1e-4 ||Y||_F (at most twice), or a
                // factorization at w: FP64 (direct Schur form below, no
                // refinement) for global-front plans and for LDS plans whose
                // FP64 front region keeps the occupancy, else in the factor type
                const bool tan64 = !stale && (!IR || !c.plan->lds_ok || a.tan64);
                // Y of w: into the rhs buffer for a factorization at w, else
                // beside X (ir2), X then moved into the element-Y slots
                double* const Y = stale ? ir2 : c.rhs;
                double* const X = c.re;  // [dof][D2] once the element Y rows are gathered
                node_gather<D>(c, c.re, D2, Y, D2, 0);
                __syncthreads();
                if constexpr (NSPEC <= kMaxNrhs) {
                    if (stale) {
                        for (int t = threadIdx.x; t < ndof * D2; t += NT)
                            X[t] = c.rhs[(int64_t)(t / D2) * NSPEC + 1 + t % D2];
                        __syncthreads();
                    }
                }
                if (stale)
                    ;
                else if (!c.plan->lds_ok || (IR && a.tan64))
                    factorize<D, D2, double>(c, sm, dynRaw);
                else
                    factorize<D, D2, T>(c, sm, dynF);
                if (sm.flag) {
                    status = 3;
                } else if (!tan64) {
                    // X ~ K^-1 Y from the factors (FP32, or of the previous state),
                    // refined against the FP64 tangent of w; then the stationary
                    // (second-order) form
                    //   Abar = <A> - Y^T X - X^T r,  r = Y - K X,
                    // whose error is (X - X*)^T K (X - X*) (energy-norm error squared)
                    if (!stale) backsolve<D, D2, T>(c, sm, X, dynRaw, a.bs_slice);
                    // refinement corrections: ir2 unless it holds Y
                    double* const corr = stale ? c.rhs : ir2;
                    const int max_ref = stale ? 2 : a.ir_max_tan;
                    for (int ref = 0;; ++ref) {
                        residual_ke<D, D2>(c, Y, X, ir1);
                        __syncthreads();
                        if (ref == max_ref) break;
                        if (stale) {
                            double nr[2] = {0.0, 0.0};
                            for (int t = threadIdx.x; t < ndof * D2; t += NT) {
                                if (is_pinned(*c.plan, t / D2 / D)) continue;
                                nr[0] += ir1[t] * ir1[t];
                                nr[1] += Y[t] * Y[t];
                            }
                            block_sum<2>(nr, sm);
                            const bool done = !(sm.outv[0] > 1e-8 * sm.outv[1]);
                            __syncthreads();
                            if (done) break;
                        }
                        forward<D, D2, T>(c, sm, ir1, dynF, a.lds_elems);
                        backsolve<D, D2, T>(c, sm, corr, dynRaw, a.bs_slice);
                        for (int t = threadIdx.x; t < ndof * D2; t += NT) X[t] += corr[t];
                        __syncthreads();
                    }
                    double acc[D2 * D2];
#pragma unroll
                    for (int q = 0; q < D2 * D2; ++q) acc[q] = 0;
                    for (int t = threadIdx.x; t < ndof; t += NT) {
                        if (is_pinned(*c.plan, t / D)) continue;
#pragma unroll
                        for (int g = 0; g < D2; ++g)
#pragma unroll
                            for (int h2 = 0; h2 < D2; ++h2)
                                acc[g * D2 + h2] += Y[t * D2 + g] * X[t * D2 + h2] + X[t * D2 + g] * ir1[t * D2 + h2];
                    }
                    block_sum<D2 * D2>(acc, sm);
                    if (threadIdx.x < D2 * D2) Aout[threadIdx.x] = Aavg - sm.outv[threadIdx.x];
                    __syncthreads();
                } else {
                    // Z^T D^-1 Z over every pivot of every front
                    double acc[D2 * D2];
#pragma unroll
                    for (int q = 0; q < D2 * D2; ++q) acc[q] = 0;
                    const DevPlan& pl = *c.plan;
                    for (int s = 0; s < pl.nfront; ++s) {
                        const DevFront fr = pl.fronts[s];
                        const double* Dg = c.L + fr.D_off;
                        const double* y = c.L + fr.y_off;
                        for (int j = threadIdx.x; j < fr.p; j += NT) {
                            const double rd = 1.0 / Dg[j];
                            double z[D2];
#pragma unroll
                            for (int g = 0; g < D2; ++g) z[g] = y[(int64_t)g * fr.p + j];
#pragma unroll
                            for (int g = 0; g < D2; ++g)
#pragma unroll
                                for (int h2 = 0; h2 < D2; ++h2) acc[g * D2 + h2] += z[g] * z[h2] * rd;
                        }
                    }
                    block_sum<D2 * D2>(acc, sm);
                    if (threadIdx.x < D2 * D2) Aout[threadIdx.x] = Aavg - sm.outv[threadIdx.x];
                    __syncthreads();
                }
            }
            if (status == 0 && wst)
                for (int t = threadIdx.x; t < ndof; t += NT) wst[t] = c.w[t];
        }
        if (status != 0) {
            const double qnan = __builtin_nan("");
            if (threadIdx.x < D2) Pout[threadIdx.x] = qnan;
            if (Aout && threadIdx.x < D2 * D2) Aout[threadIdx.x] = qnan;
        }
        PROF_MARK(PH_FINAL);
        if (threadIdx.x == 0) {
            if (a.status) a.status[rve] = (status == 0 && capped) ? 1 : status;
            if (a.iters) a.iters[rve] = it;
            sm.flag = 0;
        }
        __syncthreads();
    }
}

#if FEHMM_NWAVE == 4
// The Newton residual and the element tangents of every RVE at its stored (or
// zero) fluctuation, alone: one element pass and the node gather of R per RVE
// (the assembly phase of a Newton iteration, timed on its own by
// rve_assemble_batch).  status[r] = 2 where some J <= 0, else 0.
template <int D>
__global__ __launch_bounds__(NT, 2) void rve_assembly_kernel(SolveArgs a) {
    __shared__ Smem sm;
    double* base = a.ws + (int64_t)blockIdx.x * a.lay.stride;
    for (;;) {
        if (threadIdx.x == 0) {
            const unsigned int idx = atomicAdd(a.counter, 1u);
            sm.rve = idx < (unsigned int)a.B ? a.order[idx] : -1;
        }
        __syncthreads();
        const int rve = sm.rve;
        if (rve < 0) return;
        RveCtx c;
        rve_setup<D>(a, rve, base, c, sm);
        const int ndof = c.nn * D;
        const double* wst = a.wstate ? a.wstate + a.state_off[rve] : nullptr;
        for (int t = threadIdx.x; t < ndof; t += NT) c.w[t] = (wst && !is_pinned(*c.plan, t / D)) ? wst[t] : 0.0;
        __syncthreads();
        element_tangents<D, double>(c, sm, c.w);
        __syncthreads();
        node_gather<D>(c, c.fe, 1, c.R, 1, 0);
        if (threadIdx.x == 0 && a.status) a.status[rve] = sm.flag ? 2 : 0;
        __syncthreads();
    }
}

int lds_static_bytes() { return (int)sizeof(Smem); }
#endif

__global__ void reset_counter_kernel(unsigned int* counter) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *counter = 0u;
}

// dynamic LDS limits are raised once per process, outside any stream capture
hipError_t prepare_rve_solve() {
    const void* ks[4] = {(const void*)rve_solve_kernel<2, double>, (const void*)rve_solve_kernel<2, float>,
                         (const void*)rve_solve_kernel<3, double>, (const void*)rve_solve_kernel<3, float>};
    for (const void* k : ks) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           kLdsBytesMax - (int)sizeof(Smem));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

#if FEHMM_NWAVE == 4
hipError_t launch_rve_assembly(const SolveArgs& a, int nslots, hipStream_t stream) {
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, stream, a.counter);
    if (a.dim == 2)
        hipLaunchKernelGGL((rve_assembly_kernel<2>), dim3(nslots), dim3(NT), 0, stream, a);
    else
        hipLaunchKernelGGL((rve_assembly_kernel<3>), dim3(nslots), dim3(NT), 0, stream, a);
    return hipGetLastError();
}
#endif

hipError_t launch_rve_solve(const SolveArgs& a, int nslots, size_t dyn_bytes, bool fp32, hipStream_t stream) {
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, stream, a.counter);
    if (a.dim == 2 && fp32)
        hipLaunchKernelGGL((rve_solve_kernel<2, float>), dim3(nslots), dim3(NT), dyn_bytes, stream, a);
    else if (a.dim == 2)
        hipLaunchKernelGGL((rve_solve_kernel<2, double>), dim3(nslots), dim3(NT), dyn_bytes, stream, a);
    else if (fp32)
        hipLaunchKernelGGL((rve_solve_kernel<3, float>), dim3(nslots), dim3(NT), dyn_bytes, stream, a);
    else
        hipLaunchKernelGGL((rve_solve_kernel<3, double>), dim3(nslots), dim3(NT), dyn_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace FEHMM_VARIANT
}  // namespace fehmm

#if FEHMM_PHASE_PROF
#if FEHMM_NWAVE == 4
extern "C" int rve_debug_phase_clocks_w8(unsigned long long* out, int reset);
extern "C" int rve_debug_phase_clocks_w4(unsigned long long* out, int reset);
extern "C" int rve_debug_phase_clocks(unsigned long long* out, int reset) {
    unsigned long long b[fehmm::w4::PH_N];
    if (rve_debug_phase_clocks_w4(out, reset) || rve_debug_phase_clocks_w8(b, reset)) return -3;
    for (int i = 0; i < fehmm::w4::PH_N; ++i) out[i] += b[i];
    return 0;
}
extern "C" int rve_debug_phase_clocks_w4(unsigned long long* out, int reset) {
#else
extern "C" int rve_debug_phase_clocks_w8(unsigned long long* out, int reset) {
#endif
    using namespace fehmm::FEHMM_VARIANT;
    if (hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase), sizeof(unsigned long long) * PH_N) != hipSuccess) return -3;
    if (reset) {
        unsigned long long z[PH_N] = {0};
        if (hipMemcpyToSymbol(HIP_SYMBOL(g_phase), z, sizeof(z)) != hipSuccess) return -3;
    }
    return 0;
}
#endif
