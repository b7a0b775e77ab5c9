// HIP kernels of the quadtree identity topology (PixVOD, arXiv 2606.03989,
// Fig. 2, Sec. 3.3, Sec. 4.2) for gfx950.
//
// The synchronous iteration of Sec. 4.1 in the same rotated form as the grid's
// fused schedule: a sender turns its belief and its stored message from a
// factor into a partial message (independent of the receiver's linearisation
// point); the receiver completes it with the factor residual at both points,
// updates and relinearises its variable, then sends its next partials. Each
// iteration is one launch over the same buffers: the first workgroups take the
// nodes (one lane per node, all levels, each workgroup inside one level), the
// others the pixels (one lane per pixel, 64 of a row). Both read only what the
// previous iteration wrote.
//
// Where partials live: a variable's partial towards its parent, and a node's
// partials towards its children, stay in the sender's own slots (coalesced
// writes from the wide lower levels; the parent gathers four children from
// two adjacent rows). Normal-integration partials go into the receiver's
// slot: 8 of 42 planes, for which the sender's slot, as on the grid, gains
// nothing (65.9 us per iteration at 640 x 480, 65.5 so). At frame ends the same
// slots hold the canonical messages, each stored at the variable that receives
// it.
#include "gbp_tree.h"
#include "gbp_device.hpp"
#include "gbp_planes.hpp"

#include <cmath>

namespace pv {

namespace {

// receiver-side completion of an identity partial (h, Lambda') with the
// residual r seen by the receiver: eta = h - Lambda' r; the message is added
// to the pose block of the belief and its eta kept at storage precision
template <int LD, class Lam>
__device__ inline void complete_identity(float msg_eta[6], Lam lam, const double r[6], double* L, double* eta) {
    double e[6];
    complete_eta(msg_eta, lam, r, e);
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        eta[a] += e[a];
        msg_eta[a] = (float)e[a];
    }
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int c = i; c < 6; ++c) L[LD == 7 ? s7(i, c) : s6(i, c)] += (double)lam(s6(i, c));
}

template <int LD, class Lam>
__device__ inline void add_identity(const float msg_eta[6], Lam lam, double* L, double* eta) {
#pragma unroll
    for (int a = 0; a < 6; ++a) eta[a] += (double)msg_eta[a];
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = r; c < 6; ++c) L[LD == 7 ? s7(r, c) : s6(r, c)] += (double)lam(s6(r, c));
}

// first-order transport of a stored identity message by the mean step m
template <class Lam>
__device__ inline void transport_identity(float msg_eta[6], Lam lam, const double m[6]) {
    double e[6];
    complete_eta(msg_eta, lam, m, e);
#pragma unroll
    for (int a = 0; a < 6; ++a) msg_eta[a] = (float)e[a];
}

// sender-side partial of an identity factor from the sender's pose marginal
// (P, p) minus the factor's stored message to the sender, to 27 planes from b
template <class Lam>
__device__ inline bool send_identity(double lamR, const double P[21], const double p[6], const float back_eta[6],
                                     Lam back_lam, GFloat* b, long stride, unsigned o) {
    double V[21], v[6], Lp[21], h[6];
#pragma unroll
    for (int k = 0; k < 21; ++k) V[k] = P[k] - (double)back_lam(k);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = p[k] - (double)back_eta[k];
    const bool ok = identity_partial(lamR, V, v, Lp, h);
    o = here(o);
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        put(at(b, o), k < 6 ? (float)h[k] : (float)Lp[k - 6]);
        b = next(stride, b);
    }
    return ok;
}

// (L, eta) = pose prior of a node (Eq. prior) with precision lamP at Exp(tau) = (q, t)
__device__ inline void node_prior(const Strengths& s, double lamP, const double tau[6], const double q[4],
                                  const double t[3], double L[21], double eta[6]) {
    double rp[6];
    prior_residual(s, tau, q, t, rp);
    pose_prior(lamP, rp, eta, [&](int r, int c, double x) { L[s6(r, c)] = x; });
}

// per-workgroup level of a node launch (uniform across the workgroup)
struct Level {
    int l, H, W, off, b0;      // this level
    int Wp, offp;              // parent level
    int Hc, Wc, offc;          // child level
    double lamP, lamR_up, lamR_down;
};

__device__ inline Level level_of_block(const TreeGeo& t, int b) {
    Level v;
    v.l = 1;
#pragma unroll
    for (int k = 2; k <= kTreeMaxLevels; ++k)
        if (k <= t.L && b >= t.bstart[k]) v.l = k;
    // gather the fields with constant indices only (no dynamic indexing of
    // the kernel-argument structure)
    v.H = v.W = v.off = v.b0 = v.Wp = v.offp = v.Hc = v.Wc = v.offc = 0;
    v.lamP = v.lamR_up = v.lamR_down = 0.0;
#pragma unroll
    for (int k = 1; k <= kTreeMaxLevels; ++k)
        if (k == v.l) {
            v.H = t.Hl[k];
            v.W = t.Wl[k];
            v.off = t.off[k];
            v.b0 = t.bstart[k];
            v.Hc = t.Hl[k - 1];
            v.Wc = t.Wl[k - 1];
            v.offc = t.off[k - 1];
            v.lamP = t.lamP[k];
            v.lamR_up = t.lamR[k];
            v.lamR_down = t.lamR[k - 1];
            if (k < kTreeMaxLevels) {
                v.Wp = t.Wl[k + 1];
                v.offp = t.off[k + 1];
            }
        }
    return v;
}

__device__ inline void round6(double tau[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) tau[k] = (double)(float)tau[k];
}

// ---------------------------------------------------------------------------
// pixels

// a pixel's stored messages: of the edge to its parent (27 values) and of its
// four normal-integration factors
struct PixelMessages {
    float eta[6], lam[21];
    float mn[4][2];
};

// sender side of a pixel: partial towards the parent (own slot) and the
// normal-integration partials (neighbours' slots) from the belief (L, eta)
__device__ inline bool pixel_emit(const Geo& g, const Strengths& s, unsigned o, const bool has[4], const bool act[4],
                                  const double L[28], const double eta[7], const PixelMessages& ms, float* Y) {
    double P[21], p[6], D, dv, l66 = L[s7(6, 6)];
    bool ok = depth_marginal(L, eta, D, dv);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!has[d]) continue;
        GFloat* b = plane_of(Y, (long)(TP_MN + 2 * opposite(d)) * g.plane + step_of(g, d));
        const unsigned oh = here(o);
        double lp, hn;
        normal_partial(s.lamN, D - (double)ms.mn[d][1], dv - (double)ms.mn[d][0], lp, hn);
        put(at(b, oh), act[d] ? (float)hn : 0.0f);
        put(at(next(g, b), oh), act[d] ? (float)lp : 0.0f);
    }
    asm volatile("" : "+v"(l66), "+v"(D), "+v"(dv));
    pose_marginal(L, eta, l66, P, p);
    ok = send_identity(s.lamR, P, p, ms.eta, [&](int k) { return ms.lam[k]; }, plane_of(Y, (long)TP_UP * g.plane),
                       g.plane, o) && ok;
    return ok;
}

__device__ inline void pixel_store_point(float* Y, const Geo& g, unsigned o, const double tau[6], double ell) {
    GFloat* b = plane_of(Y, 0);
    o = here(o);
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        put(at(b, o), k < 6 ? (float)tau[k] : (float)ell);
        b = next(g, b);
    }
}

template <bool PROLOGUE, bool FINAL>
__device__ __attribute__((always_inline)) inline void pixel_pass(const Geo& g, const TreeGeo& t, const Strengths& s,
                                                                 const Inputs& in, const float* X, const float* NX,
                                                                 float* Y, float* var_ll, float* valid, int* health,
                                                                 int u, int v) {
    const unsigned o = off_of(g, u, v);
    bool has[4], act[4];
    unsigned on[4];
    float c[4], pt[7], ellj[4];
    load_point_at(X, g, o, pt);
    const PixelInputs pin = load_inputs_at(s, in, o);
    edges_of(g, in, u, v, has, on, c);
    active_edges(s, c, act);
    PixelMessages ms;
    // normal messages or partials; the parent edge's message (prologue) or the
    // parent's partial for this child slot
    const float* ub = PROLOGUE ? X + (long)TP_UP * g.plane : NX;
    const long us = PROLOGUE ? g.plane : t.nplane;
    const long pn = (long)t.off[1] + (long)(v >> 1) * t.Wl[1] + (u >> 1);
    const long ul = PROLOGUE ? 0 : pn + (long)(TN_CH + 27 * (((v & 1) << 1) | (u & 1))) * t.nplane;
    float tpf[6];
    if constexpr (!PROLOGUE) {
#pragma unroll
        for (int d = 0; d < 4; ++d) ellj[d] = ld(X + (long)P_ELL * g.plane, on[d]);
#pragma unroll
        for (int k = 0; k < 6; ++k) tpf[k] = NX[(long)(TN_TAU + k) * t.nplane + pn];
    }
    {
        GFloat* b = plane_of(X, (long)TP_MN * g.plane);
        const unsigned oh = here(o);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            ms.mn[d][0] = *at(b, oh);
            b = next(g, b);
            ms.mn[d][1] = *at(b, oh);
            b = next(g, b);
        }
        const GFloat* q = PROLOGUE ? at((GFloat*)const_cast<float*>(ub), oh) : (GFloat*)const_cast<float*>(ub) + ul;
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            const float x = q[(long)k * us];
            if (k < 6) ms.eta[k] = x;
            else ms.lam[k - 6] = x;
        }
    }
    const auto lam = [&](int k) { return ms.lam[k]; };
    double tau[6], ell, q4[4], R[9], tt[3], L[28], eta[7];
    point_of(pt, tau, ell);
    pose_exp(tau, q4, tt);
    pose_rotation(q4, R);
    const bool val = unary_factors<true>(g, s, in, u, v, tau, q4, R, tt, ell, pin, L, eta);
    bool ok = true;
    if constexpr (!PROLOGUE) {
        // the parent's partial, completed at both points
        {
            double tp[6], qp[4], trp[3], r[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) tp[k] = (double)tpf[k];
            pose_exp(tp, qp, trp);
            pose_between(qp, trp, q4, tt, r);
            complete_identity<7>(ms.eta, lam, r, L, eta);
        }
        // normal-integration partials in this pixel's slots
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            if (act[d] && has[d]) {
                const double rn = normal_residual_c(c[d], d, ell, (double)ellj[d]);
                const double ne = fma(-(double)ms.mn[d][1], rn, (double)ms.mn[d][0]);
                eta[6] += ne;
                L[s7(6, 6)] += (double)ms.mn[d][1];
                ms.mn[d][0] = (float)ne;
            } else {
                ms.mn[d][0] = ms.mn[d][1] = 0.0f;
            }
        }
        // update: mean, relinearisation (Eq. var), transport of the stored messages
        double m[7], var;
        ok = ldl7_solve(L, eta, m, var);
        pose_retract(q4, tt, m, tau);
        ell += m[6];
        transport_identity(ms.eta, lam, m);
#pragma unroll
        for (int d = 0; d < 4; ++d) ms.mn[d][0] = (float)fma(-(double)ms.mn[d][1], m[6], (double)ms.mn[d][0]);
        round6(tau);
        ell = (double)(float)ell;
        if constexpr (FINAL) {
            pixel_store_point(Y, g, o, tau, ell);
            GFloat* b = plane_of(Y, (long)TP_UP * g.plane);
            const unsigned oh = here(o);
#pragma unroll
            for (int k = 0; k < 35; ++k) {   // TP_MN follows TP_UP
                put(at(b, oh), k < 6 ? ms.eta[k] : k < 27 ? ms.lam[k - 6] : ms.mn[(k - 27) >> 1][(k - 27) & 1]);
                b = next(g, b);
            }
            *at((GFloat*)var_ll, oh) = (float)var;
            *at((GFloat*)valid, oh) = val ? 1.0f : 0.0f;
            if (!ok) atomicOr(health, 1);
            return;
        }
        pose_exp(tau, q4, tt);
        pose_rotation(q4, R);
        unary_factors<true>(g, s, in, u, v, tau, q4, R, tt, ell, pin, L, eta);
    }
    add_identity<7>(ms.eta, lam, L, eta);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        eta[6] += (double)ms.mn[d][0];
        L[s7(6, 6)] += (double)ms.mn[d][1];
    }
    pixel_store_point(Y, g, o, tau, ell);
    ok = pixel_emit(g, s, o, has, act, L, eta, ms, Y) && ok;
    if (!ok) atomicOr(health, 1);
}

// ---------------------------------------------------------------------------
// nodes

// The messages of a node's five edges (0: parent, 1 .. 4: children). As in the
// grid's pass, the information matrices of three of them stay in LDS, where
// they are loaded without passing through registers, so that the node fits 256
// registers and two waves share a SIMD.
constexpr int NODE_LDS = 3 * 21 * 64;   // floats per wave: edges 1 .. 3

struct NodeMessages {
    float eta[5][6];
    float lam0[21], lam4[21];
    const float* lds;

    __device__ inline float lam(int e, int k) const {
        return e == 0 ? lam0[k] : e == 4 ? lam4[k] : lds[((e - 1) * 21 + k) * 64];
    }
};

template <bool PROLOGUE, bool FINAL>
__device__ __attribute__((always_inline)) inline void node_pass(const Geo& g, const TreeGeo& t, const Strengths& s,
                                                                const float* X, const float* NX, float* NY,
                                                                int* health, float* buf) {
    const Level lv = level_of_block(t, (int)blockIdx.x);
    const int lane = (int)threadIdx.x;
    const int i = ((int)blockIdx.x - lv.b0) * kTreeThreads + lane;
    if (i >= lv.H * lv.W) return;
    const int x = i % lv.W, y = i / lv.W;
    const unsigned n = (unsigned)(lv.off + i);
    const unsigned o = n * 4u;
    // --- every load issued before any use: the node's pose, the parent's pose
    // and its partial for this child slot, the children's poses and partials
    // towards this node (the prologue: the node's own stored messages). A
    // missing parent or child reads the node itself or the first child; its
    // values are not used.
    const bool has_par = lv.l < t.L;
    bool has[5];
    has[0] = has_par;
    unsigned oc[4];   // byte offsets of the children in their planes
    const bool pix = lv.l == 1;
    const float* cb = pix ? X : NX;
    const long cs = pix ? g.plane : t.nplane;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int cx = 2 * x + (q & 1), cy = 2 * y + (q >> 1);
        has[1 + q] = cx < lv.Wc && cy < lv.Hc;
        const int cxc = has[1 + q] ? cx : 2 * x, cyc = has[1 + q] ? cy : 2 * y;
        oc[q] = pix ? off_of(g, cxc, cyc) : (unsigned)(lv.offc + cyc * lv.Wc + cxc) * 4u;
    }
    const unsigned op = has_par ? (unsigned)(lv.offp + (y >> 1) * lv.Wp + (x >> 1)) : n;
    float tnf[6], tpf[6], tcf[4][6];
    NodeMessages ms;
    ms.lds = buf + lane;
    {
        GFloat* b = plane_of(NX, (long)TN_TAU * t.nplane);
        const unsigned oh = here(o), oph = here(op * 4u);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            tnf[k] = *at(b, oh);
            if constexpr (!PROLOGUE) tpf[k] = *at(b, oph);
            b = next(t.nplane, b);
        }
    }
    if constexpr (!PROLOGUE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            GFloat* b = plane_of(cb, 0);   // the pose planes are the first of both
            const unsigned oh = here(oc[q]);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                tcf[q][k] = *at(b, oh);
                b = next(cs, b);
            }
        }
    }
    {
        // edge 0: own slot (prologue) or the parent's slot of this child
        const int qn = ((y & 1) << 1) | (x & 1);
        const GFloat* q = (GFloat*)const_cast<float*>(NX) +
                          (PROLOGUE ? (long)TN_UP * t.nplane + n : (long)(TN_CH + 27 * qn) * t.nplane + op);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            const float v = q[(long)k * t.nplane];
            if (k < 6) ms.eta[0][k] = v;
            else ms.lam0[k - 6] = v;
        }
    }
    static_assert(TN_UP == 6 && TP_UP == 7, "planes of the upward partials");
#pragma unroll
    for (int e = 1; e < 5; ++e) {
        GFloat* b = PROLOGUE ? plane_of(NX, (long)(TN_CH + 27 * (e - 1)) * t.nplane)
                             : plane_of(cb, (pix ? (long)TP_UP : (long)TN_UP) * cs);
        const long st = PROLOGUE ? t.nplane : cs;
        const unsigned oh = here(PROLOGUE ? o : oc[e - 1]);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            if (k < 6) ms.eta[e][k] = *at(b, oh);
            else if (e == 4) ms.lam4[k - 6] = *at(b, oh);
            else
                __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(b, oh),
                                                 (__attribute__((address_space(3))) void*)(buf + ((e - 1) * 21 + k - 6) * 64),
                                                 4, 0, 0);
            b = next(st, b);
        }
    }
    double tau[6], q4[4], tt[3], L[21], eta[6];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) tau[k] = (double)tnf[k];
    pose_exp(tau, q4, tt);
    node_prior(s, lv.lamP, tau, q4, tt, L, eta);
    wait_lds_loads();
    if constexpr (!PROLOGUE) {
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            if (!has[e]) {
#pragma unroll
                for (int k = 0; k < 6; ++k) ms.eta[e][k] = 0.0f;
                continue;
            }
            double tj[6], qj[4], trj[3], r[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) tj[k] = (double)(e == 0 ? tpf[k] : tcf[e == 0 ? 0 : e - 1][k]);
            pose_exp(tj, qj, trj);
            pose_between(qj, trj, q4, tt, r);
            complete_identity<6>(ms.eta[e], [&](int k) { return ms.lam(e, k); }, r, L, eta);
        }
        reread_lds();
        // update: mean, relinearisation, transport
        double m[6];
        ok = ldl6_solve(L, eta, m);
        pose_retract(q4, tt, m, tau);
#pragma unroll
        for (int e = 0; e < 5; ++e)
            if (has[e]) transport_identity(ms.eta[e], [&](int k) { return ms.lam(e, k); }, m);
        round6(tau);
        reread_lds();
    }
    {
        GFloat* b = plane_of(NY, (long)TN_TAU * t.nplane);
        const unsigned oh = here(o);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            put(at(b, oh), (float)tau[k]);
            b = next(t.nplane, b);
        }
    }
    if constexpr (FINAL) {
        GFloat* b = plane_of(NY, (long)TN_UP * t.nplane);
        const unsigned oh = here(o);
#pragma unroll
        for (int e = 0; e < 5; ++e)   // TN_CH follows TN_UP
#pragma unroll
            for (int k = 0; k < 27; ++k) {
                put(at(b, oh), k < 6 ? ms.eta[e][k] : has[e] ? ms.lam(e, k - 6) : 0.0f);
                b = next(t.nplane, b);
            }
    } else {
        if constexpr (!PROLOGUE) {
            pose_exp(tau, q4, tt);
            node_prior(s, lv.lamP, tau, q4, tt, L, eta);
        }
#pragma unroll
        for (int e = 0; e < 5; ++e)
            if (PROLOGUE || has[e]) add_identity<6>(ms.eta[e], [&](int k) { return ms.lam(e, k); }, L, eta);
        // partials towards the parent and the children, in the node's own slots
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            if (!has[e]) continue;
            reread_lds();
            ok = send_identity(e == 0 ? lv.lamR_up : lv.lamR_down, L, eta, ms.eta[e],
                               [&](int k) { return ms.lam(e, k); }, plane_of(NY, (long)(TN_UP + 27 * e) * t.nplane),
                               t.nplane, o) && ok;
        }
    }
    if (!ok) atomicOr(health, 1);
}

// One iteration (or the prologue) of the whole tree: workgroups 0 .. nblocks - 1
// take the nodes, the others the pixels, 64 of a row, tiles_x per row. The two
// parts are independent within an iteration; in one launch the nodes' longer
// waves start first and the pixels fill the SIMDs beside them.
// 640 x 480: 64 us per iteration; 102 us as two launches (47 us of pixels, 55 us
// of nodes at one wave per SIMD). The copy of its 238 MB at this card's
// 4.74 TB/s takes 50 us.
template <bool PROLOGUE, bool FINAL>
__global__ __launch_bounds__(kTreeThreads, 2) void k_tr_pass(Geo g, TreeGeo t, Strengths s, Inputs in, const float* X,
                                                             const float* NX, float* Y, float* NY, float* var_ll,
                                                             float* valid, int* health, int tiles_x) {
    __shared__ float buf[NODE_LDS];
    if ((int)blockIdx.x < t.nblocks) {
        node_pass<PROLOGUE, FINAL>(g, t, s, X, NX, NY, health, buf);
        return;
    }
    const int b = (int)blockIdx.x - t.nblocks;
    const int u = (b % tiles_x) * 64 + (int)threadIdx.x, v = b / tiles_x;
    if (u < g.W) pixel_pass<PROLOGUE, FINAL>(g, t, s, in, X, NX, Y, var_ll, valid, health, u, v);
}

__global__ void k_tr_clear(float* __restrict__ p, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

__global__ void k_tr_pack_pixels(Geo g, float* __restrict__ X, float* __restrict__ dense, int to_dense) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long p = pix_of(g, u, v), d = (long)v * g.W + u, N = (long)g.H * g.W;
    for (int k = 0; k < TP_PLANES; ++k) {
        if (to_dense) dense[(long)k * N + d] = X[(long)k * g.plane + p];
        else X[(long)k * g.plane + p] = dense[(long)k * N + d];
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// host side

bool make_tree_geo(int H, int W, double sigma_P, double sigma_R, TreeGeo* t) {
    *t = TreeGeo{};
    t->Hl[0] = H;
    t->Wl[0] = W;
    int L = 0;
    while (t->Hl[L] > 1 || t->Wl[L] > 1) {
        if (L == kTreeMaxLevels) return false;
        t->Hl[L + 1] = (t->Hl[L] + 1) / 2;
        t->Wl[L + 1] = (t->Wl[L] + 1) / 2;
        ++L;
    }
    if (L == 0) return false;
    t->L = L;
    t->off[0] = 0;
    t->off[1] = 0;
    t->bstart[1] = 0;
    for (int l = 1; l <= L; ++l) {
        const int n = t->Hl[l] * t->Wl[l];
        t->off[l + 1] = t->off[l] + n;
        t->bstart[l + 1] = t->bstart[l] + (n + kTreeThreads - 1) / kTreeThreads;
    }
    t->NT = t->off[L + 1];
    t->nblocks = t->bstart[L + 1];
    t->nplane = ((long)t->NT + 63) / 64 * 64;
    for (int l = 0; l <= L; ++l) {
        const double sp = std::ldexp(sigma_P, -l), sr = std::ldexp(sigma_R, -l);
        t->lamP[l] = 1.0 / (sp * sp);
        t->lamR[l] = 1.0 / (sr * sr);
    }
    return true;
}

hipError_t launch_tree_prologue(const Geo& g, const TreeGeo& t, const Strengths& s, const Inputs& in,
                                const float* X, const float* NX, float* Y, float* NY, int* health, hipStream_t st) {
    const int tx = (g.W + 63) / 64;
    hipLaunchKernelGGL((k_tr_pass<true, false>), dim3(t.nblocks + tx * g.H), dim3(kTreeThreads), 0, st, g, t, s, in, X,
                       NX, Y, NY, nullptr, nullptr, health, tx);
    return hipGetLastError();
}

hipError_t launch_tree_iterate(const Geo& g, const TreeGeo& t, const Strengths& s, const Inputs& in,
                               const float* X, const float* NX, float* Y, float* NY, bool final_pass,
                               float* var_ll, float* valid, int* health, hipStream_t st) {
    const int tx = (g.W + 63) / 64;
    if (final_pass)
        hipLaunchKernelGGL((k_tr_pass<false, true>), dim3(t.nblocks + tx * g.H), dim3(kTreeThreads), 0, st, g, t, s,
                           in, X, NX, Y, NY, var_ll, valid, health, tx);
    else
        hipLaunchKernelGGL((k_tr_pass<false, false>), dim3(t.nblocks + tx * g.H), dim3(kTreeThreads), 0, st, g, t, s,
                           in, X, NX, Y, NY, var_ll, valid, health, tx);
    return hipGetLastError();
}

hipError_t launch_tree_clear_nodes(const TreeGeo& t, float* NX, hipStream_t st) {
    const long n = (long)TN_PLANES * t.nplane;
    hipLaunchKernelGGL(k_tr_clear, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, NX, n);
    return hipGetLastError();
}

hipError_t launch_tree_pack_pixels(const Geo& g, float* X, float* dense, int to_dense, hipStream_t st) {
    const dim3 b(64, 1), gr((g.W + 63) / 64, g.H);
    hipLaunchKernelGGL(k_tr_pack_pixels, gr, b, 0, st, g, X, dense, to_dense);
    return hipGetLastError();
}

}  // namespace pv
