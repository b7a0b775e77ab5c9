// HIP kernels of the reverse sweep through unrolled GBP iterations (PixVOD,
// arXiv 2606.03989) for gfx950: one lane per pixel, FP32 cotangent planes (the
// state's cotangent in the state layout and the intermediate ones: Mb, Ub,
// Eb), FP64 algebra in registers.
//
// Reverse of one canonical iteration X -> X' (linearise + marginals, messages,
// update + relinearise + transport; Sec. 3.4 and Sec. 4.1), given the
// cotangent Xb' of X':
//   forward recompute  the fused passes that recompute X also keep its belief
//                      and depth marginal (37 FP64 planes) and the belief of
//                      the update (35); the information of the new messages
//                      is read from the state X' (the transport keeps it);
//   k_adj_update       reverse of the update at every pixel: cotangents of its
//                      four new messages (Mb, 116 planes) and of its unary
//                      information and point (Ub, 42 planes);
//   k_adj_edges        one wave per direction: the pixel as the sender
//                      of its outgoing message and the receiver of its incoming
//                      one on that edge: cotangents of its marginals, of the
//                      residual's pose and log-depth arguments, and of the
//                      stored message the sender subtracted (gathered from the
//                      neighbours' Mb, no atomics; the four directions of a
//                      pixel are summed through LDS);
//   k_adj_belief       reverse of the marginals and of the unary factors:
//                      completes Xb (cotangent of X) and accumulates the
//                      per-pixel parameter gradients. Every stored message
//                      enters the belief the same way, so its cotangent
//                      there is one 29-value slot-common part Cb per pixel;
//                      it is kept apart from the slot-specific part in Xb
//                      and added by the next reader (k_adj_update), instead
//                      of a read-modify-write of all four slots.
#include "gbp_adjoint.h"
#include "gbp_adjoint.hpp"
#include "gbp_planes.hpp"

namespace pv {

constexpr int MSG_STRIDE = 29;   // per direction: eta 6, Lambda 21, normal eta, normal lambda
constexpr int UB_TAU = 35;       // Ub: L_bar 28, eta_bar 7, tau_bar 6, ell_bar 1
constexpr int UB_ELL = 41;
constexpr int EB_EPS = 29;       // Eb: P_bar 21, p_bar 6, D_bar, dv_bar, eps_bar 6, ell_bar

__device__ inline bool pixel_2d(const Geo& g, int& u, int& v) {
    u = blockIdx.x * blockDim.x + threadIdx.x;
    v = blockIdx.y * blockDim.y + threadIdx.y;
    return u < g.W && v < g.H;
}

// The reverse kernels go through phases: x is finished before what follows, and
// the loads of a phase are not issued before it, so that a kernel's registers
// are its phases' maximum and not their sum.
template <int N>
__device__ inline void phase(double (&x)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(x[k]) : : "memory");
}

// a pointer that is the same in every lane, in scalar registers
template <class T>
__device__ inline T* uniform(T* p) {
    const unsigned long a = (unsigned long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (T*)(((unsigned long)hi << 32) | lo);
}

// n planes from `base` at offset o
template <int N>
__device__ inline void load_planes(const float* base, long stride, unsigned o, float x[N]) {
    GFloat* b = plane_of(base, 0);
    o = here(o);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        x[k] = *at(b, o);
        b = next(stride, b);
    }
}
template <int N>
__device__ inline void load_planes(const double* base, long stride, unsigned o, double x[N]) {
    GDouble* b = plane_of(const_cast<double*>(base));
    o = here(o);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        x[k] = *at(b, o);
        b = next(stride, b);
    }
}
template <int N>
__device__ inline void store_planes(float* base, long stride, unsigned o, const double x[N]) {
    GFloat* b = plane_of(base, 0);
    o = here(o);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        *at(b, o) = (float)x[k];
        b = next(stride, b);
    }
}

// reverse of the update (k_pf_update): belief from the unary and the new
// messages, mean m, relinearisation, transport of the messages. Bound by one
// wave's chain of loads and FP64 steps: every load goes out at the start (the
// information cotangents of the four slots straight into LDS, 84 planes), and
// the transport's sums, which do not need the solve, stand under the belief's
// loads. 320 x 240, beside the recompute: 40.4 us, 51.3 with the loads behind
// the solve and Cholesky factors.
__global__ __launch_bounds__(64, 2) void k_adj_update(Geo g, const float* X, const float* Xn, const double* bel,
                                                      const float* Xb, const float* Cb, float* Mb, float* Ub) {
    __shared__ float buf[84 * 64];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    const unsigned o = off_of(g, u, v);
    const long pl = g.plane;
    const bool has[4] = {u > 0, u + 1 < g.W, v > 0, v + 1 < g.H};
    float xe[4][6], xn[8], ml[4][21], ce[6], cn[2];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        load_planes<21>(Xn + (long)(P_MID + d * MID_STRIDE + 6) * pl, pl, o, ml[d]);
        load_planes<6>(Xb + (long)(P_MID + d * MID_STRIDE) * pl, pl, o, xe[d]);
    }
    float nn[8];
    load_planes<8>(Xn + (long)P_MN * pl, pl, o, nn);
    load_planes<8>(Xb + (long)P_MN * pl, pl, o, xn);
    load_planes<6>(Cb, pl, o, ce);
    load_planes<2>(Cb + 27 * pl, pl, o, cn);
    // the belief of the update (unary + new messages), kept by the recompute
    double L[28], m[7];
    load_planes<28>(bel, pl, o, L);
    load_planes<7>(bel + 28 * pl, pl, o, m);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        GFloat* b = plane_of(Xb, (long)(P_MID + d * MID_STRIDE + 6) * pl);
        const unsigned oh = here(o);
#pragma unroll
        for (int k = 0; k < 21; ++k) {
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(b, oh),
                                             (__attribute__((address_space(3))) void*)(buf + (d * 21 + k) * 64), 4, 0,
                                             0);
            b = next(g, b);
        }
    }
    // transport eta' = eta - Lambda m_p, ne' = ne - nl m6: contribution to
    // m_bar (a missing edge's information is zero in the state)
    double mb[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        double eb[6], y[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) eb[a] = (double)xe[d][a] + (double)ce[a];
        const float zero[6] = {0, 0, 0, 0, 0, 0};
        complete_eta(zero, [&](int k) { return ml[d][k]; }, eb, y);   // y = -Lambda eb
#pragma unroll
        for (int a = 0; a < 6; ++a) mb[a] += y[a];
        mb[6] = fma(-(double)nn[2 * d + 1], (double)xn[2 * d] + (double)cn[0], mb[6]);
    }
    phase(mb);
    float pt[7], xp[7];
    load_point_at(X, g, o, pt);
    load_planes<7>(Xb, pl, o, xp);
    double tau[6], ell, q[4], t[3], id[7], tn[6];
    point_of(pt, tau, ell);
    pose_exp(tau, q, t);
    ldl7_factor(L, id);
    ldl7_substitute(L, id, m);
    pose_retract(q, t, m, tn);
    // relinearisation tau' = Log(Exp(tau) Exp(m_p)):
    //   d tau' = Jl(tau')^-1 Jl(tau) d tau + Jr(tau')^-1 Jr(m_p) d m_p
    double tnb[6], a6[6], taub[6], b6[6], mpb[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) tnb[k] = (double)xp[k];
    const double ellnb = (double)xp[6];
    jac_invT_apply(tn, 1.0, tnb, a6);
    jac_T_apply(tau, 1.0, a6, taub);
    jac_invT_apply(tn, -1.0, tnb, b6);
    jac_T_apply(m, -1.0, b6, mpb);
#pragma unroll
    for (int k = 0; k < 6; ++k) mb[k] += mpb[k];
    mb[6] += ellnb;
    // m = B^-1 beta: betab = B^-1 m_bar, B_bar = -sym(betab m^T)
    phase(mb);
    float cl[21];
    load_planes<21>(Cb + 6 * pl, pl, o, cl);
    load_planes<6>(Cb, pl, o, ce);
    load_planes<2>(Cb + 27 * pl, pl, o, cn);
    load_planes<8>(Xb + (long)P_MN * pl, pl, o, xn);
#pragma unroll
    for (int d = 0; d < 4; ++d) load_planes<6>(Xb + (long)(P_MID + d * MID_STRIDE) * pl, pl, o, xe[d]);
    double betab[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) betab[k] = mb[k];
    ldl7_substitute(L, id, betab);
    wait_lds_loads();
    double Bb[28];
#pragma unroll
    for (int k = 0; k < 28; ++k) Bb[k] = 0.0;
    sym_outer_acc7(Bb, betab, m, -1.0);

    // cotangents of the four new messages: transport + belief
    const float* lds = buf + threadIdx.x;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        GFloat* b = plane_of(Mb, (long)d * MSG_STRIDE * pl);
        const unsigned oh = here(o);
        double eb[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            eb[a] = (double)xe[d][a] + (double)ce[a];
            *at(b, oh) = has[d] ? (float)(eb[a] + betab[a]) : 0.0f;
            b = next(g, b);
        }
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r; c < 6; ++c) {
                const int k = s6(r, c);
                const double tr = (r == c) ? eb[r] * m[r] : fma(eb[r], m[c], eb[c] * m[r]);
                const double x = ((double)lds[(d * 21 + k) * 64] + (double)cl[k]) - tr + Bb[s7(r, c)];
                *at(b, oh) = has[d] ? (float)x : 0.0f;
                b = next(g, b);
            }
        const double neb = (double)xn[2 * d] + (double)cn[0];
        const double nlb = (double)xn[2 * d + 1] + (double)cn[1];
        *at(b, oh) = has[d] ? (float)(neb + betab[6]) : 0.0f;
        b = next(g, b);
        *at(b, oh) = has[d] ? (float)(fma(-neb, m[6], nlb) + Bb[s7(6, 6)]) : 0.0f;
    }
    store_planes<28>(Ub, pl, o, Bb);
    store_planes<7>(Ub + 28 * pl, pl, o, betab);
    store_planes<6>(Ub + (long)UB_TAU * pl, pl, o, taub);
    store_planes<1>(Ub + (long)UB_ELL * pl, pl, o, &ellnb);
}

// reverse of the message step (k_pf_messages): wave d of a workgroup takes
// direction d of 64 pixels j of a row, j as the receiver of the message in its
// slot d (residual cotangent) and as the sender of the message into its
// neighbour in direction d (its marginals and the stored message it
// subtracted). The four waves' contributions to j's marginal and perturbation
// cotangents are summed through LDS in a fixed order. Writes the sender part
// of j's slot-d cotangent to Xbo. (A direction per wave, not per lane: the
// planes of one direction are read 64 pixels at a time, the direction's cases
// are uniform, and the sums take 37 LDS writes instead of 148 lane exchanges:
// 59.6 against 73.9 us at 320 x 240, beside the recompute. The first sums go to
// LDS early: kept in registers, they made the pose marginal spill.)
constexpr int EDGE_SUMS = 37;    // D_bar, dv_bar, eps_bar 6, ell_bar, lamN_bar, P_bar 21, p_bar 6
constexpr int EDGE_FIRST = 10;   // those put into LDS as soon as they are known
constexpr int EDGE_PART = 24;    // summed in two parts: 48 KB of LDS, three workgroups per CU
constexpr int EDGE_LAMN = 9;     // lamN_bar, which goes to gN
static_assert(EDGE_PART % 4 == 0 && EDGE_SUMS <= 2 * EDGE_PART && EDGE_LAMN < EDGE_FIRST && EDGE_FIRST < EDGE_PART,
              "two parts, lamN_bar in the first");
// the plane of Eb (P_bar 21, p_bar 6, D_bar, dv_bar, eps_bar 6, ell_bar) of a sum
__device__ inline int edge_plane(int k) { return k < EDGE_LAMN ? 27 + k : k - EDGE_FIRST; }

__global__ __launch_bounds__(256, 3) void k_adj_edges(Geo g, Strengths s, Inputs in, const float* X,
                                                      const double* marg, const float* Xn, const float* Mb, float* Xbo,
                                                      float* Eb, double* gN) {
    __shared__ double sh[EDGE_PART][4][64];
    const int lane = threadIdx.x;
    const int d = __builtin_amdgcn_readfirstlane(threadIdx.y);
    int u, v;
    segment_pixel(lane, u, v);
    const long pl = g.plane;
    // the direction's planes, own and of the opposite slot
    const int od = opposite(d);
    const float* Ld = uniform(Xn + (long)(P_MID + d * MID_STRIDE + 6) * pl);
    const float* Lo = uniform(Xn + (long)(P_MID + od * MID_STRIDE + 6) * pl);
    const float* Nd = uniform(Xn + (long)(P_MN + 2 * d + 1) * pl);
    const float* No = uniform(Xn + (long)(P_MN + 2 * od + 1) * pl);
    const float* Mbd = uniform(Mb + (long)d * MSG_STRIDE * pl);
    const float* Mbo = uniform(Mb + (long)od * MSG_STRIDE * pl);
    const float* Xd = uniform(X + (long)(P_MID + d * MID_STRIDE) * pl);
    const float* Xnd = uniform(X + (long)(P_MN + 2 * d) * pl);
    float* Xbd = uniform(Xbo + (long)(P_MID + d * MID_STRIDE) * pl);
    float* Xbn = uniform(Xbo + (long)(P_MN + 2 * d) * pl);
    const unsigned oj = off_of(g, u < g.W ? u : g.W - 1, v);
    int nu, nv;
    const bool inside = u < g.W;
    const bool edge = inside && neighbour(g, u, v, d, nu, nv);
    double acc[EDGE_SUMS];   // in the order of the sums
#pragma unroll
    for (int k = 0; k < EDGE_SUMS; ++k) acc[k] = 0.0;
    if (edge) {
        const unsigned oi = oj + (unsigned)(4 * step_of(g, d));
        float pj[7], pi[7], Mj[21], Mi[21], ej[6], ei[6], nej[1], nei[2];
        load_point_at(X, g, oj, pj);
        load_point_at(X, g, oi, pi);
        load_planes<21>(Ld, pl, oj, Mj);
        load_planes<6>(Mbd, pl, oj, ej);
        load_planes<21>(Lo, pl, oi, Mi);
        load_planes<6>(Mbo, pl, oi, ei);
        load_planes<1>(Mbd + 27 * pl, pl, oj, nej);
        load_planes<2>(Mbo + 27 * pl, pl, oi, nei);
        const float ct = d == DIR_L ? ld(in.cxt, oi) : d == DIR_R ? ld(in.cxt, oj) : d == DIR_U ? ld(in.cyt, oi) : ld(in.cyt, oj);
        // residual of the message into j from i, r = Log(Exp(tau_i)^-1 Exp(tau_j));
        // the message into i from j uses -r
        double tau[6], ell, q[4], t[3], ti[6], elli, qi[4], tri[3], r[6];
        point_of(pj, tau, ell);
        point_of(pi, ti, elli);
        pose_exp(tau, q, t);
        pose_exp(ti, qi, tri);
        pose_between(qi, tri, q, t, r);
        // normal-integration factor of the edge
        double nsb = 0.0, nlsb = 0.0;
        if (isfinite(ct) && s.lamN > 0.0) {
            double dm[2];
            load_planes<2>(marg, pl, oj, dm);
            const float lj = ld(Nd, oj), li = ld(No, oi);
            float xn[2];
            load_planes<2>(Xnd, pl, oj, xn);
            const double rn_i = normal_residual_c(ct, od, elli, ell);
            // ne_new = h - lp rn: receiver j and sender j (rn_i depends on ell_j with -1)
            const double neb = (double)nei[0], nlb = (double)nei[1];
            acc[8] = fma(-(double)lj, (double)nej[0], (double)li * neb);
            double lsb, vsb, lnb;
            normal_partial_adjoint(s.lamN, dm[0] - (double)xn[1], dm[1] - (double)xn[0], fma(-neb, rn_i, nlb), neb,
                                   lsb, vsb, lnb);
            acc[0] = lsb;
            acc[1] = vsb;
            acc[EDGE_LAMN] = lnb;
            nsb = -vsb;
            nlsb = -lsb;
        }
        {
            const double ns2[2] = {nsb, nlsb};
            store_planes<2>(Xbn, pl, oj, ns2);
        }
        // eta_new = h - Lp r on both sides: receiver r_bar = -Lp_j eb_j, sender
        // r_bar = -Lp_i eb_i with d(-r) = -d r, so eps_j += Jr(r)^-T (Lp_i eb_i - Lp_j eb_j)
        double hb[6];
        {
            double rb[6], e[6], y[6];
            const float zero[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                e[a] = (double)ej[a];
                hb[a] = (double)ei[a];
            }
            complete_eta(zero, [&](int k) { return Mj[k]; }, e, rb);    // -Lp_j eb_j
            complete_eta(zero, [&](int k) { return Mi[k]; }, hb, y);    // -Lp_i eb_i
#pragma unroll
            for (int a = 0; a < 6; ++a) rb[a] -= y[a];
            double eps[6];
            jac_invT_apply(r, -1.0, rb, eps);
            phase(eps);
#pragma unroll
            for (int a = 0; a < 6; ++a) acc[2 + a] = eps[a];
        }
#pragma unroll
        for (int k = 0; k < EDGE_FIRST; ++k) sh[k][d][lane] = acc[k];
        // sender: the partial of the message into i from j's variable-to-factor
        // message (j's marginal minus j's stored message from this factor)
        double V[21], vv[6], Lpb[21], Vb[21], vb[6];
        {
            double L[28], eta[7];
            load_planes<28>(marg + 2 * pl, pl, oj, L);
            load_planes<7>(marg + 30 * pl, pl, oj, eta);
            pose_marginal(L, eta, L[s7(6, 6)], V, vv);
        }
        {
            float xm[27], lb[21];
            load_planes<27>(Xd, pl, oj, xm);
            load_planes<21>(Mbo + 6 * pl, pl, oi, lb);
#pragma unroll
            for (int k = 0; k < 21; ++k) {
                V[k] -= (double)xm[6 + k];
                Lpb[k] = (double)lb[k];
            }
#pragma unroll
            for (int a = 0; a < 6; ++a) vv[a] -= (double)xm[a];
        }
        // eta_i = h - Lp (-r): Lp_bar += sym(hb r^T)
        sym_outer_acc6(Lpb, hb, r, 1.0);
        identity_partial_adjoint(s.lamR, V, vv, Lpb, hb, Vb, vb);
        GFloat* b = plane_of(Xbd, 0);
        const unsigned oh = here(oj);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            *at(b, oh) = (float)-(k < 6 ? vb[k] : Vb[k - 6]);
            b = next(g, b);
        }
#pragma unroll
        for (int k = 0; k < 21; ++k) acc[EDGE_FIRST + k] = Vb[k];
#pragma unroll
        for (int a = 0; a < 6; ++a) acc[EDGE_FIRST + 21 + a] = vb[a];
    } else if (inside) {
        GFloat* b = plane_of(Xbd, 0);
        const unsigned oh = here(oj);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            *at(b, oh) = 0.0f;
            b = next(g, b);
        }
        const double zero2[2] = {0.0, 0.0};
        store_planes<2>(Xbn, pl, oj, zero2);
#pragma unroll
        for (int k = 0; k < EDGE_FIRST; ++k) sh[k][d][lane] = 0.0;
    }
    // the sums over the four waves, every fourth by each wave, to the planes of
    // Eb and to gN
    const long pj = pix_of(g, inside ? u : g.W - 1, v);
#pragma unroll
    for (int part = 0; part < EDGE_SUMS; part += EDGE_PART) {
        if (part) __syncthreads();
#pragma unroll
        for (int k = part ? part : EDGE_FIRST; k < part + EDGE_PART && k < EDGE_SUMS; ++k) sh[k - part][d][lane] = acc[k];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < EDGE_PART && part + j < EDGE_SUMS; j += 4) {
            const int k = part + j + d;
            if (k >= EDGE_SUMS || !inside) break;
            const double(*q)[64] = sh[j + d];
            const double x = (q[0][lane] + q[1][lane]) + (q[2][lane] + q[3][lane]);
            if (k == EDGE_LAMN) gN[pj] += x;
            else Eb[(long)edge_plane(k) * pl + pj] = (float)x;
        }
    }
}

// reverse of the marginals and of the unary factors; completes Xbo (point
// planes) and writes the slot-common part Cbo. Two phases (marginals, unary),
// each with its own loads, so that two waves share a SIMD: 256 registers and
// six values in scratch (28 bytes per lane), whose reloads wait for the stores of
// Cbo before them; those stores behind the loads gained nothing (24.2 us at 320 x
// 240, beside the recompute; 36.2 with 400 registers).
__global__ __launch_bounds__(64, 2) void k_adj_belief(Geo g, Strengths s, Inputs in, const float* X,
                                                      const double* marg, const float* Ub, const float* Eb, float* Xbo,
                                                      float* Cbo, double* gsig, double* gk) {
    __shared__ float buf[14 * 64];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    const unsigned o = off_of(g, u, v);
    const long pl = g.plane;
    // the cotangents of the point, needed last, wait in LDS: tau_bar 6 and
    // ell_bar of the update, eps_bar 6 and ell_bar of the edges
    {
        GFloat* b = plane_of(Ub, (long)UB_TAU * pl);
        GFloat* c = plane_of(Eb, (long)EB_EPS * pl);
        const unsigned oh = here(o);
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(b, oh),
                                             (__attribute__((address_space(3))) void*)(buf + k * 64), 4, 0, 0);
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(c, oh),
                                             (__attribute__((address_space(3))) void*)(buf + (7 + k) * 64), 4, 0, 0);
            b = next(g, b);
            c = next(g, c);
        }
    }
    double Lb[28], etab[7];
    {
        // the belief of the marginals (unary + stored messages), kept by the recompute
        double L[28], eta[7], Pb[21], pb[6], BbS[28], ebS[7];
        float eb[29];
        load_planes<28>(marg + 2 * pl, pl, o, L);
        load_planes<7>(marg + 30 * pl, pl, o, eta);
        load_planes<29>(Eb, pl, o, eb);
#pragma unroll
        for (int k = 0; k < 21; ++k) Pb[k] = (double)eb[k];
#pragma unroll
        for (int k = 0; k < 6; ++k) pb[k] = (double)eb[21 + k];
#pragma unroll
        for (int k = 0; k < 28; ++k) BbS[k] = 0.0;
#pragma unroll
        for (int k = 0; k < 7; ++k) ebS[k] = 0.0;
        marginals_adjoint(L, eta, Pb, pb, (double)eb[27], (double)eb[28], BbS, ebS);
        // every stored message enters the belief: one slot-common cotangent
        double c[29];
#pragma unroll
        for (int a = 0; a < 6; ++a) c[a] = ebS[a];
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int k = r; k < 6; ++k) c[6 + s6(r, k)] = BbS[s7(r, k)];
        c[27] = ebS[6];
        c[28] = BbS[s7(6, 6)];
        store_planes<29>(Cbo, pl, o, c);
        phase(BbS);
        float ub[35];
        load_planes<35>(Ub, pl, o, ub);
#pragma unroll
        for (int k = 0; k < 28; ++k) Lb[k] = (double)ub[k] + BbS[k];
#pragma unroll
        for (int k = 0; k < 7; ++k) etab[k] = (double)ub[28 + k] + ebS[k];
    }
    phase(Lb);
    phase(etab);
    float pt[7];
    load_point_at(X, g, o, pt);
    double tau[6], ell, q[4], R[9], t[3], epsb[6], taub[6];
    point_of(pt, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
#pragma unroll
    for (int k = 0; k < 6; ++k) epsb[k] = taub[k] = 0.0;
    double ellb = 0.0, sigb = 0.0, kb = 0.0;
    unary_adjoint(g, s, in, u, v, tau, R, t, ell, Lb, etab, epsb, taub, ellb, sigb, kb);
    wait_lds_loads();
    const float* lds = buf + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 6; ++k) epsb[k] += (double)lds[(7 + k) * 64];
    double te[7];
    jac_T_apply(tau, -1.0, epsb, te);
#pragma unroll
    for (int k = 0; k < 6; ++k) te[k] += taub[k] + (double)lds[k * 64];
    te[6] = ellb + ((double)lds[6 * 64] + (double)lds[13 * 64]);
    store_planes<7>(Xbo, pl, o, te);
    *at(plane_of(gsig), here(o)) += sigb;
    *at(plane_of(gk), here(o)) += kb;
}

// cotangents of the per-frame outputs: pose mean (Eq. estimator_avg) and the
// inverse-depth map rho = exp(-ell)
__global__ void k_adj_inject(Geo g, const float* __restrict__ Xend, float* __restrict__ Xb, PoseBar xb,
                             const float* __restrict__ rhob) {
    int u, v;
    if (!pixel_2d(g, u, v)) return;
    const long p = pix_of(g, u, v);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        float* q = Xb + (long)(P_TAU + k) * g.plane + p;
        *q = (float)((double)*q + xb.v[k]);
    }
    if (rhob) {
        const double rho = exp(-(double)Xend[(long)P_ELL * g.plane + p]);
        float* q = Xb + (long)P_ELL * g.plane + p;
        *q = (float)((double)*q - rho * (double)rhob[(long)v * g.W + u]);
    }
}

// per block: sums of two FP64 planes (deterministic two-stage reduction)
constexpr int SUM_THREADS = 256;

__global__ __launch_bounds__(SUM_THREADS) void k_sum2(Geo g, const double* __restrict__ a,
                                                      const double* __restrict__ b, double* __restrict__ partial) {
    __shared__ double sh[2][SUM_THREADS];
    double s0 = 0.0, s1 = 0.0;
    const long N = (long)g.H * g.W;
    for (long i = (long)blockIdx.x * SUM_THREADS + threadIdx.x; i < N; i += (long)gridDim.x * SUM_THREADS) {
        const long p = pix_of(g, (int)(i % g.W), (int)(i / g.W));
        s0 += a[p];
        s1 += b[p];
    }
    sh[0][threadIdx.x] = s0;
    sh[1][threadIdx.x] = s1;
    __syncthreads();
    for (int w = SUM_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + w];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x < 2) partial[(long)blockIdx.x * 2 + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void k_sum2_final(int nblocks, const double* __restrict__ partial, double* __restrict__ result) {
    const int k = threadIdx.x;
    if (k >= 2) return;
    double s = 0.0;
    for (int b = 0; b < nblocks; ++b) s += partial[(long)b * 2 + k];
    result[k] = s;
}

// FP64 plane -> dense FP32 map
__global__ void k_plane_to_dense(Geo g, const double* __restrict__ src, float* __restrict__ dst) {
    int u, v;
    if (!pixel_2d(g, u, v)) return;
    dst[(long)v * g.W + u] = (float)src[pix_of(g, u, v)];
}

// ---------------------------------------------------------------------------
// launchers

static const dim3 kAdjBlock(64, 4);
static dim3 adj_grid(const Geo& g) { return dim3((g.W + 63) / 64, (g.H + 3) / 4); }

hipError_t launch_adj_update(const Geo& g, const float* X, const float* Xn, const double* bel, const float* Xb,
                             const float* Cb, float* Mb, float* Ub, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_update, dim3((g.W + 63) / 64, g.H), dim3(64), 0, st, g, X, Xn, bel, Xb, Cb, Mb, Ub);
    return hipGetLastError();
}

hipError_t launch_adj_edges(const Geo& g, const Strengths& s, const Inputs& in, const float* X, const double* marg,
                            const float* Xn, const float* Mb, float* Xbo, float* Eb, double* gN, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_edges, dim3((g.W + 63) / 64, g.H), dim3(64, 4), 0, st, g, s, in, X, marg, Xn, Mb, Xbo, Eb,
                       gN);
    return hipGetLastError();
}

hipError_t launch_adj_belief(const Geo& g, const Strengths& s, const Inputs& in, const float* X, const double* marg,
                             const float* Ub, const float* Eb, float* Xbo, float* Cbo, double* gsig, double* gk,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_adj_belief, dim3((g.W + 63) / 64, g.H), dim3(64), 0, st, g, s, in, X, marg, Ub, Eb, Xbo, Cbo,
                       gsig, gk);
    return hipGetLastError();
}

hipError_t launch_adj_inject(const Geo& g, const float* Xend, float* Xb, const PoseBar& xb, const float* rhob,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_adj_inject, adj_grid(g), kAdjBlock, 0, st, g, Xend, Xb, xb, rhob);
    return hipGetLastError();
}

int sum2_blocks(const Geo& g) {
    const long N = (long)g.H * g.W;
    long b = (N + SUM_THREADS * 8 - 1) / (SUM_THREADS * 8);
    if (b < 1) b = 1;
    if (b > 1024) b = 1024;
    return (int)b;
}

hipError_t launch_sum2(const Geo& g, const double* a, const double* b, double* partial, double* result,
                       hipStream_t st) {
    const int nb = sum2_blocks(g);
    hipLaunchKernelGGL(k_sum2, dim3(nb), dim3(SUM_THREADS), 0, st, g, a, b, partial);
    hipLaunchKernelGGL(k_sum2_final, dim3(1), dim3(64), 0, st, nb, partial, result);
    return hipGetLastError();
}

hipError_t launch_plane_to_dense(const Geo& g, const double* src, float* dst, hipStream_t st) {
    hipLaunchKernelGGL(k_plane_to_dense, adj_grid(g), kAdjBlock, 0, st, g, src, dst);
    return hipGetLastError();
}

}  // namespace pv
