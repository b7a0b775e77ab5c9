// HIP kernels of the per-pixel GBP iteration (PixVOD, arXiv 2606.03989) for
// gfx950. One lane per pixel; FP32 structure-of-arrays state planes with a
// padded row pitch, FP64 per-pixel algebra in registers.
//
// Two schedules of the same synchronous iteration (Sec. 4.1):
//   per-factor: linearise + marginals -> messages -> belief update, one kernel
//               each, intermediates through device memory;
//   fused:      each pixel completes the partial messages its neighbours sent
//               (partials do not depend on the receiver's linearisation point),
//               updates and relinearises its variable, then linearises again
//               and sends the next partials. One pass over the state per
//               iteration; a prologue pass per frame starts the rotation and
//               the last pass writes the canonical messages back.
#include "gbp_kernels.h"
#include "gbp_device.hpp"
#include "gbp_planes.hpp"

#include <hip/hip_cooperative_groups.h>

namespace cg = cooperative_groups;

namespace pv {

// The four stored messages of a pixel in a fused pass. A pass needs each
// message's information matrix three times (sum of the belief, transport,
// what its sender subtracts), with a 7x7 solve between the first and the
// second, and 4 x 29 values beside the FP64 algebra would leave one wave per
// SIMD. The matrices of three directions are therefore kept in LDS, where they
// are loaded straight from memory without passing through registers (63 planes
// of 64 lanes, 16 KB per wave: eight waves fit a CU's 160 KB), the fourth and
// everything else in registers: at most 256 registers, so that two waves share
// a SIMD and fill each other's waits. Passes that also store the messages of
// each iteration (with a tape, damped) spilled at that, and a spilled value's
// load waits for every store before it; they keep 78 planes in LDS, which is
// enough for none (160 KB would give eight waves 80; 320 x 240: with tape, beside
// the reverse kernels, 54.5 us against 66.5; damped 34.5 against 41.4), but costs
// the other passes 2% (256 x 256: 20.25 us against 19.75). Every lane reads only
// what it loaded itself, so no barrier is needed.
constexpr int LDS_PLANES = 63, LDS_PLANES_STORING = 78;

template <int PLANES>
struct Messages {
    static constexpr int kPlanes = PLANES, kRest = 4 * 21 - PLANES, kFloats = PLANES * 64;   // LDS floats per wave
    float eta[4][6];     // identity messages
    float rest[kRest];   // information: what LDS does not hold, the end of direction 3's
    float mn[4][2];      // normal messages: eta, lambda
    float* lds;          // information, direction by direction: this lane's column of the wave's LDS planes

    __device__ inline float lam(int d, int k) const {
        const int i = d * 21 + k;
        return i < PLANES ? lds[i * 64] : rest[i - PLANES];
    }
    __device__ inline void set_lam(int d, int k, float x) {
        const int i = d * 21 + k;
        if (i < PLANES) lds[i * 64] = x;
        else rest[i - PLANES] = x;
    }
};

// issues the loads of a pixel's messages but the information that LDS
// does not hold.
// at_: where each slot is read, the pixel itself for stored messages and the
// neighbour that sends it for partials in flight (a missing neighbour's is the
// pixel's own: finite and not used). buf: the wave's LDS planes, lane: the lane
// of the wave. The information may be read after wait_lds_loads() only.
template <int PLANES>
__device__ inline void load_messages(const float* X, const Geo& g, const unsigned at_[4], float* buf, int lane,
                                     Messages<PLANES>& m) {
    GFloat* b = plane_of(X, (long)P_MID * g.plane);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned o = here(at_[d]);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            m.eta[d][k] = *at(b, o);
            b = next(g, b);
        }
#pragma unroll
        for (int k = 0; k < 21 && d * 21 + k < PLANES; ++k) {
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(b, o),
                                             (__attribute__((address_space(3))) void*)(buf + (d * 21 + k) * 64), 4, 0,
                                             0);
            b = next(g, b);
        }
    }
    b = plane_of(X, (long)P_MN * g.plane);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned o = here(at_[d]);
        m.mn[d][0] = *at(b, o);
        b = next(g, b);
        m.mn[d][1] = *at(b, o);
        b = next(g, b);
    }
    m.lds = buf + lane;
}

// issues the loads of the rest: late, so that they are not held in registers
// beside the linearisation
template <int PLANES>
__device__ inline void load_rest(const float* X, const Geo& g, unsigned o, Messages<PLANES>& m) {
    GFloat* b = plane_of(X, (long)(P_MID + 4 * MID_STRIDE - m.kRest) * g.plane);
    o = here(o);
#pragma unroll
    for (int k = 0; k < m.kRest; ++k) {
        m.rest[k] = *at(b, o);
        b = next(g, b);
    }
}

// B += a stored message (embedded: identity -> pose block, normal -> depth entry)
template <class M>
__device__ inline void add_message(double L[28], double eta[7], const M& m, int d) {
#pragma unroll
    for (int a = 0; a < 6; ++a) eta[a] += (double)m.eta[d][a];
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = r; c < 6; ++c) L[s7(r, c)] += (double)m.lam(d, s6(r, c));
    eta[6] += (double)m.mn[d][0];
    L[s7(6, 6)] += (double)m.mn[d][1];
}

// first-order transport of a stored message by the mean step (Sec. 4.1)
template <class Lam>
__device__ inline void transport(float eta[6], float mn[2], Lam lam, const double m[7]) {
    double e[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) e[a] = (double)eta[a];
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = r; c < 6; ++c) {
            const double l = (double)lam(s6(r, c));
            e[r] = fma(-l, m[c], e[r]);
            if (r != c) e[c] = fma(-l, m[r], e[c]);
        }
#pragma unroll
    for (int a = 0; a < 6; ++a) eta[a] = (float)e[a];
    mn[0] = (float)fma(-(double)mn[1], m[6], (double)mn[0]);
}
template <class M>
__device__ inline void transport_message(M& ms, int d, const double m[7]) {
    transport(ms.eta[d], ms.mn[d], [&](int k) { return ms.lam(d, k); }, m);
}

// per-lane tape of the reverse sweep's recompute. The new messages'
// information is not on it: it is the next canonical state's, unchanged by the
// transport.
struct Tape {
    double* bel;         // belief of the update (35 FP64 planes)
    float* canonical;    // canonical state after the update (not the last iteration of a segment)
    double* marg;        // depth marginal and belief of the next emission (37 FP64 planes)
};

// the depth marginal D, dv and the belief of an emission: L 28, eta 7 (the
// pose marginal is one division and 27 multiply-adds of the belief and is
// formed again by its reader). The tape is written non-temporally: it is read
// back only by the reverse sweep.
__device__ inline void tape_marginals(double* marg, const Geo& g, unsigned o, double D, double dv, const double L[28],
                                      const double eta[7]) {
    GDouble* b = plane_of(marg);
    o = here(o);
#pragma unroll
    for (int k = 0; k < 37; ++k) {
        const double x = k == 0 ? D : k == 1 ? dv : k < 30 ? L[k - 2] : eta[k - 30];
        __builtin_nontemporal_store(x, at(b, o));
        b = next(g, b);
    }
}

template <bool NT = false>
__device__ inline void store_point(float* Y, const Geo& g, unsigned o, const double tau[6], double ell) {
    GFloat* b = plane_of(Y, 0);
    o = here(o);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        put<NT>(at(b, o), (float)tau[k]);
        b = next(g, b);
    }
    put<NT>(at(b, o), (float)ell);
}

template <bool NT = false, class M>
__device__ inline void store_messages(float* Y, const Geo& g, unsigned o, const M& m) {
    GFloat* b = plane_of(Y, (long)P_MID * g.plane);
    o = here(o);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            put<NT>(at(b, o), k < 6 ? m.eta[d][k] : m.lam(d, k - 6));
            b = next(g, b);
        }
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        put<NT>(at(b, o), m.mn[d][0]);
        b = next(g, b);
        put<NT>(at(b, o), m.mn[d][1]);
        b = next(g, b);
    }
}

// rounds a double point to the stored FP32 precision
__device__ inline void round_point(double tau[6], double& ell) {
#pragma unroll
    for (int k = 0; k < 6; ++k) tau[k] = (double)(float)tau[k];
    ell = (double)(float)ell;
}

// ---------------------------------------------------------------------------
// frame and keyframe preparation

// central differences inside, one-sided at the border
__device__ __attribute__((always_inline)) inline void frame_prep_pixel(const Geo& g, const float* __restrict__ src, long src_pitch,
                                        float* __restrict__ It, float* __restrict__ Gx, float* __restrict__ Gy,
                                        int u, int v) {
    const float* row = src + (long)v * src_pitch;
    const float c = row[u];
    float gx, gy;
    if (u == 0) gx = row[1] - row[0];
    else if (u == g.W - 1) gx = row[u] - row[u - 1];
    else gx = 0.5f * (row[u + 1] - row[u - 1]);
    if (v == 0) gy = src[src_pitch + u] - row[u];
    else if (v == g.H - 1) gy = row[u] - src[(long)(v - 1) * src_pitch + u];
    else gy = 0.5f * (src[(long)(v + 1) * src_pitch + u] - src[(long)(v - 1) * src_pitch + u]);
    const long p = pix_of(g, u, v);
    It[p] = c;
    Gx[p] = gx;
    Gy[p] = gy;
}

__global__ void k_frame_prep(Geo g, const float* __restrict__ src, long src_pitch, float* __restrict__ It,
                             float* __restrict__ Gx, float* __restrict__ Gy, int* __restrict__ clear) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (clear && u == 0 && v == 0) *clear = 0;
    if (u >= g.W || v >= g.H) return;
    frame_prep_pixel(g, src, src_pitch, It, Gx, Gy, u, v);
}

// keyframe image, normal-integration targets and the state reset:
// pose linearisation points to identity, messages to zero, log-depth kept
__device__ __attribute__((always_inline)) inline void keyframe_prep_pixel(
    const Geo& g, const float* __restrict__ img, const float* __restrict__ normals, float* __restrict__ Is,
    float* __restrict__ cxt, float* __restrict__ cyt, float* __restrict__ X, float* __restrict__ X2, int u, int v) {
    const long dense = (long)v * g.W + u;
    const long p = pix_of(g, u, v);
    Is[p] = img[dense];
    const double q0 = ((double)u - g.cx) / g.fx, q1 = ((double)v - g.cy) / g.fy;
    const double n0 = normals[3 * dense], n1 = normals[3 * dense + 1], n2 = normals[3 * dense + 2];
    const double nq = n0 * q0 + n1 * q1 + n2;
    const double qn = sqrt(q0 * q0 + q1 * q1 + 1.0);
    const bool ok = isfinite(nq) && fabs(nq) >= 1e-3 * qn;
    cxt[p] = ok ? (float)(n0 / (g.fx * nq)) : __int_as_float(0x7fc00000);
    cyt[p] = ok ? (float)(n1 / (g.fy * nq)) : __int_as_float(0x7fc00000);
    const float ell = X[P_ELL * g.plane + p];
    for (int k = 0; k < N_PLANES; ++k) {
        X[(long)k * g.plane + p] = 0.0f;
        X2[(long)k * g.plane + p] = 0.0f;
    }
    X[P_ELL * g.plane + p] = ell;
    X2[P_ELL * g.plane + p] = ell;
}

__global__ void k_keyframe_prep(Geo g, const float* __restrict__ img, const float* __restrict__ normals,
                                float* __restrict__ Is, float* __restrict__ cxt, float* __restrict__ cyt,
                                float* __restrict__ X, float* __restrict__ X2) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    keyframe_prep_pixel(g, img, normals, Is, cxt, cyt, X, X2, u, v);
}

__global__ void k_init_state(Geo g, float* __restrict__ X, float ell0) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long p = pix_of(g, u, v);
    for (int k = 0; k < N_PLANES; ++k) X[(long)k * g.plane + p] = 0.0f;
    X[P_ELL * g.plane + p] = ell0;
}

// ---------------------------------------------------------------------------
// per-factor schedule

// L + B + V: unary factors, belief, pose and depth marginals (FP64 scratch,
// 29 planes: P packed 21, p 6, D, dv)
__global__ __launch_bounds__(256) void k_pf_linearise(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                      double* __restrict__ marg, float* __restrict__ valid,
                                                      int* __restrict__ health) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long p = pix_of(g, u, v);
    double tau[6], ell, q[4], R[9], t[3], L[28], eta[7];
    load_point(X, g, p, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    const bool val = unary_factors(g, s, in, u, v, tau, q, R, t, ell, load_pixel_inputs(g, s, in, u, v), L, eta);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const float* m = X + (long)(P_MID + d * MID_STRIDE) * g.plane + p;
#pragma unroll
        for (int a = 0; a < 6; ++a) eta[a] += (double)m[a * g.plane];
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r; c < 6; ++c) L[s7(r, c)] += (double)m[(6 + s6(r, c)) * g.plane];
        eta[6] += (double)X[(long)(P_MN + 2 * d) * g.plane + p];
        L[s7(6, 6)] += (double)X[(long)(P_MN + 2 * d + 1) * g.plane + p];
    }
    double P[21], pv_[6], D, dv;
    pose_marginal(L, eta, L[s7(6, 6)], P, pv_);
    const bool ok = depth_marginal(L, eta, D, dv);
#pragma unroll
    for (int k = 0; k < 21; ++k) marg[(long)k * g.plane + p] = P[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) marg[(long)(21 + k) * g.plane + p] = pv_[k];
    marg[(long)27 * g.plane + p] = D;
    marg[(long)28 * g.plane + p] = dv;
    valid[p] = val ? 1.0f : 0.0f;
    if (!ok) atomicOr(health, 1);
}

// F: every pixel computes its four incoming messages from its neighbours'
// marginals and the messages those neighbours hold from the shared factor.
// Output (FP64 scratch, 29 planes per direction): identity eta(6), identity
// Lambda(21, already at storage precision), normal eta, normal lambda.
__global__ __launch_bounds__(256, 2) void k_pf_messages(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                     const double* __restrict__ marg, double* __restrict__ M,
                                                     int* __restrict__ health) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long pi = pix_of(g, u, v);
    double tau[6], ell, q[4], t[3];
    load_point(X, g, pi, tau, ell);
    pose_exp(tau, q, t);
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        double out[29];
#pragma unroll
        for (int k = 0; k < 29; ++k) out[k] = 0.0;
        int nu, nv;
        if (neighbour(g, u, v, d, nu, nv)) {
            const long pj = pix_of(g, nu, nv);
            const int slot = opposite(d);
            double V[21], vv[6], Lp[21], h[6];
#pragma unroll
            for (int k = 0; k < 21; ++k)
                V[k] = marg[(long)k * g.plane + pj] - (double)X[(long)(P_MID + slot * MID_STRIDE + 6 + k) * g.plane + pj];
#pragma unroll
            for (int k = 0; k < 6; ++k)
                vv[k] = marg[(long)(21 + k) * g.plane + pj] - (double)X[(long)(P_MID + slot * MID_STRIDE + k) * g.plane + pj];
            ok = identity_partial(s.lamR, V, vv, Lp, h) && ok;
            // the partial is rounded to storage precision as in the fused schedule
            float part[27];
#pragma unroll
            for (int k = 0; k < 6; ++k) part[k] = (float)h[k];
#pragma unroll
            for (int k = 0; k < 21; ++k) part[6 + k] = (float)Lp[k];
            double tj[6], ellj, qj[4], trj[3], r[6];
            load_point(X, g, pj, tj, ellj);
            pose_exp(tj, qj, trj);
            pose_between(qj, trj, q, t, r);
            complete_eta(part, [&](int k) { return part[6 + k]; }, r, out);
#pragma unroll
            for (int k = 0; k < 21; ++k) out[6 + k] = (double)part[6 + k];
            double rn;
            if (s.lamN > 0.0 && normal_residual(g, in, pi, pj, d, ell, ellj, rn)) {
                const double ls = marg[(long)27 * g.plane + pj] - (double)X[(long)(P_MN + 2 * slot + 1) * g.plane + pj];
                const double vs = marg[(long)28 * g.plane + pj] - (double)X[(long)(P_MN + 2 * slot) * g.plane + pj];
                double lp, hn;
                normal_partial(s.lamN, ls, vs, lp, hn);
                const float fl = (float)lp, fh = (float)hn;
                out[27] = fma(-(double)fl, rn, (double)fh);
                out[28] = (double)fl;
            }
        }
#pragma unroll
        for (int k = 0; k < 29; ++k) M[(long)(d * 29 + k) * g.plane + pi] = out[k];
    }
    if (!ok) atomicOr(health, 1);
}

// U: new belief from the recomputed unary and the new messages, relinearise,
// transport, write the state in place
__global__ __launch_bounds__(64, 2) void k_pf_update(Geo g, Strengths s, Inputs in, float* __restrict__ X,
                                                     const double* __restrict__ M, float* __restrict__ var_ll,
                                                     float* __restrict__ valid, int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    const long p = pix_of(g, u, v);
    double tau[6], ell, q[4], R[9], t[3], L[28], eta[7], m[7], var;
    load_point(X, g, p, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    const bool val = unary_factors(g, s, in, u, v, tau, q, R, t, ell, load_pixel_inputs(g, s, in, u, v), L, eta);
    // the new messages: added to the belief in FP64, kept at storage precision
    // (the information matrices are at storage precision already)
    Messages<LDS_PLANES> ms;
    ms.lds = buf + threadIdx.x;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const double* md = M + (long)(d * 29) * g.plane + p;
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            const double e = md[a * g.plane];
            eta[a] += e;
            ms.eta[d][a] = (float)e;
        }
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r; c < 6; ++c) {
                const double l = md[(6 + s6(r, c)) * g.plane];
                L[s7(r, c)] += l;
                ms.set_lam(d, s6(r, c), (float)l);
            }
        const double ne = md[27 * g.plane], nl = md[28 * g.plane];
        eta[6] += ne;
        L[s7(6, 6)] += nl;
        ms.mn[d][0] = (float)ne;
        ms.mn[d][1] = (float)nl;
    }
    reread_lds();
    const bool ok = ldl7_solve(L, eta, m, var);
    pose_retract(q, t, m, tau);
    ell += m[6];
    round_point(tau, ell);
#pragma unroll
    for (int d = 0; d < 4; ++d) transport_message(ms, d, m);
    store_point(X, g, off_of(g, u, v), tau, ell);
    store_messages(X, g, off_of(g, u, v), ms);
    var_ll[p] = (float)var;
    valid[p] = val ? 1.0f : 0.0f;
    if (!ok) atomicOr(health, 1);
}

// ---------------------------------------------------------------------------
// fused schedule

// sender side: partial messages of a pixel towards each neighbour, from its
// belief (L, eta) and its stored messages. They are written at the sender's
// pixel, in the planes of the receiver's slot, and the receiver reads them at
// its neighbour: a wave then stores whole cache lines. (Stored at the receiver,
// a horizontal neighbour's line is written in two pieces by two waves, which
// costs more than reading it twice: the pass's loads and stores alone, 1920 x
// 1080, take 575 us with the stores shifted and 430 with the loads shifted.)
// mn, eta, lam: the pixel's stored messages of direction d; act: whether its
// normal-integration factor is active
template <bool NT>
__device__ inline void emit_normal(const Geo& g, const Strengths& s, unsigned o, int d, double D, double dv,
                                   const float mn[2], bool act, float* Y) {
    GFloat* b = plane_of(Y, (long)(P_MN + 2 * opposite(d)) * g.plane);
    const unsigned oh = here(o);
    double lp, hn;
    normal_partial(s.lamN, D - (double)mn[1], dv - (double)mn[0], lp, hn);
    put<NT>(at(b, oh), act ? (float)hn : 0.0f);
    put<NT>(at(next(g, b), oh), act ? (float)lp : 0.0f);
}
template <bool NT, class Lam>
__device__ inline bool emit_identity(const Geo& g, const Strengths& s, unsigned o, int d, const double P[21],
                                     const double p[6], const float eta[6], Lam lam, float* Y) {
    double V[21], vv[6], Lp[21], h[6];
#pragma unroll
    for (int k = 0; k < 21; ++k) V[k] = P[k] - (double)lam(k);
#pragma unroll
    for (int k = 0; k < 6; ++k) vv[k] = p[k] - (double)eta[k];
    const bool ok = identity_partial(s.lamR, V, vv, Lp, h);
    GFloat* b = plane_of(Y, (long)(P_MID + opposite(d) * MID_STRIDE) * g.plane);
    const unsigned oh = here(o);
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        put<NT>(at(b, oh), k < 6 ? (float)h[k] : (float)Lp[k - 6]);
        b = next(g, b);
    }
    return ok;
}

template <bool NT, bool TAPE, class M>
__device__ inline bool emit_partials(const Geo& g, const Strengths& s, unsigned o, const bool has[4], const bool act[4],
                                     const double L[28], const double eta[7], const M& ms,
                                     float* __restrict__ Y, double* __restrict__ marg) {
    double P[21], pm[6], D, dv, l66 = L[s7(6, 6)];
    bool ok = depth_marginal(L, eta, D, dv);
    // the depth marginal and what is sent of it are finished before the pose
    // marginal takes the belief's registers
#pragma unroll
    for (int d = 0; d < 4; ++d)
        if (has[d]) emit_normal<NT>(g, s, o, d, D, dv, ms.mn[d], act[d], Y);
    asm volatile("" : "+v"(l66), "+v"(D), "+v"(dv));
    if constexpr (TAPE) tape_marginals(marg, g, o, D, dv, L, eta);
    pose_marginal(L, eta, l66, P, pm);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!has[d]) continue;
        reread_lds();
        ok = emit_identity<NT>(g, s, o, d, P, pm, ms.eta[d], [&](int k) { return ms.lam(d, k); }, Y) && ok;
    }
    return ok;
}

// prologue of one pixel: belief of the canonical state and the first partials
template <bool TAPE>
__device__ __attribute__((always_inline)) inline void prologue_pixel(const Geo& g, const Strengths& s, const Inputs& in,
                                                                     const float* __restrict__ X,
                                                                     float* __restrict__ Y, int* __restrict__ health,
                                                                     int u, int v, float* buf, int lane,
                                                                     double* __restrict__ marg) {
    const unsigned o = off_of(g, u, v);
    Messages<LDS_PLANES> ms;
    bool has[4];
    unsigned on[4];
    float c[4], pt[7];
    load_point_at(X, g, o, pt);
    const PixelInputs pin = load_inputs_at(s, in, o);
    edges_of(g, in, u, v, has, on, c);
    const unsigned own[4] = {o, o, o, o};
    load_messages(X, g, own, buf, lane, ms);
    double tau[6], ell, q[4], R[9], t[3], L[28], eta[7];
    point_of(pt, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    unary_factors(g, s, in, u, v, tau, q, R, t, ell, pin, L, eta);
    wait_lds_loads();
    load_rest(X, g, o, ms);
#pragma unroll
    for (int d = 0; d < 4; ++d) add_message(L, eta, ms, d);
    bool act[4];
    active_edges(s, c, act);
    const bool ok = emit_partials<false, TAPE>(g, s, o, has, act, L, eta, ms, Y, marg);
    store_point<false>(Y, g, o, tau, ell);
    if (!ok) atomicOr(health, 1);
}

// one iteration of one pixel: complete the partials in flight, update and
// relinearise, then (not FINAL) linearise again and emit the next partials or
// (FINAL) write the canonical state and the per-pixel outputs. Every load
// whose address does not depend on computed values is issued before its first
// use; the bilinear samples at the two warps stand under the prior's
// arithmetic. The point is stored after the second samples' arrival: a wait
// for loads also waits for the stores issued before them. TAPE: also writes the
// reverse sweep's tape. The state is stored non-temporally: no line of it is
// used again before the pass ends, and what is left in the L2 has to be written
// back then (256 x 256: 19.7 us against 21.2; 1920 x 1080: 459 against 475; 64
// mixed sequences: 1,747 against 1,785). Beside the reverse kernels, which read
// the state soon, it is not (320 x 240: the pass with tape 66.5 us, 71 with);
// neither is a damped state, which the next pass updates (34.5 us, 35.5 with).
// DAMPED: a new message is mixed with the one that the receiver holds, whose
// stored form is kept beside the partials (damp.state, updated in place: a pixel
// reads and writes its own).
struct Damp {
    float* state;
    float beta;
};

constexpr int iterate_planes(bool tape, bool damped) { return tape || damped ? LDS_PLANES_STORING : LDS_PLANES; }

template <bool FINAL, bool TAPE, bool DAMPED = false>
__device__ __attribute__((always_inline)) inline void iterate_pixel(const Geo& g, const Strengths& s, const Inputs& in,
                                                                    const float* __restrict__ X,
                                                                    float* __restrict__ Y, float* __restrict__ var_ll,
                                                                    float* __restrict__ valid,
                                                                    int* __restrict__ health, int u, int v, float* buf,
                                                                    int lane, const Tape& tape,
                                                                    const Damp& damp = Damp{}) {
    constexpr bool NT = !TAPE && !DAMPED;
    const unsigned o = off_of(g, u, v);
    Messages<iterate_planes(TAPE, DAMPED)> ms;
    bool has[4];
    unsigned on[4];
    float c[4], pt[7], npt[4][7];
    load_point_at(X, g, o, pt);
    const PixelInputs pin = load_inputs_at(s, in, o);
    edges_of(g, in, u, v, has, on, c);
#pragma unroll
    for (int d = 0; d < 4; ++d) load_point_at(X, g, on[d], npt[d]);
    load_messages(X, g, on, buf, lane, ms);

    // --- linearise at the current point
    double tau[6], ell, q[4], R[9], t[3], L[28], eta[7];
    point_of(pt, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    const bool val = unary_factors(g, s, in, u, v, tau, q, R, t, ell, pin, L, eta);

    // --- complete the partials in flight with the residuals at both points
    wait_lds_loads();
    load_rest(X, g, on[3], ms);
    if constexpr (FINAL || TAPE || DAMPED)
#pragma unroll
        for (int k = 0; k < ms.kRest; ++k) ms.rest[k] = has[3] ? ms.rest[k] : 0.0f;
    bool act[4];
    active_edges(s, c, act);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!has[d]) {
#pragma unroll
            for (int k = 0; k < 6; ++k) ms.eta[d][k] = 0.0f;
            ms.mn[d][0] = ms.mn[d][1] = 0.0f;
            if constexpr (FINAL || TAPE || DAMPED)   // what is stored of it
#pragma unroll
                for (int k = 0; k < 21 && d * 21 + k < ms.kPlanes; ++k) ms.set_lam(d, k, 0.0f);
            continue;
        }
        double tj[6], ellj, qj[4], trj[3], r[6], e[6];
        point_of(npt[d], tj, ellj);
        pose_exp(tj, qj, trj);
        pose_between(qj, trj, q, t, r);
        complete_eta(ms.eta[d], [&](int k) { return ms.lam(d, k); }, r, e);
        double ne = 0.0, rn;
        float nl = 0.0f;
        if (act[d]) {
            rn = normal_residual_c(c[d], d, ell, ellj);
            nl = ms.mn[d][1];
            ne = fma(-(double)nl, rn, (double)ms.mn[d][0]);
        }
        if constexpr (DAMPED) {
            // the blended information is rounded to storage precision like
            // every stored one
            const double b1 = (double)damp.beta, a1 = 1.0 - b1;
            GFloat* b = plane_of(damp.state, (long)(P_MID + d * MID_STRIDE) * g.plane);
            const unsigned oh = here(o);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                e[k] = fma(a1, e[k], b1 * (double)*at(b, oh));
                b = next(g, b);
            }
#pragma unroll
            for (int k = 0; k < 21; ++k) {
                const float l = (float)fma(a1, (double)ms.lam(d, k), b1 * (double)*at(b, oh));
                b = next(g, b);
                ms.set_lam(d, k, l);
            }
            b = plane_of(damp.state, (long)(P_MN + 2 * d) * g.plane);
            ne = fma(a1, ne, b1 * (double)*at(b, oh));
            nl = (float)fma(a1, (double)nl, b1 * (double)*at(next(g, b), oh));
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            eta[a] += e[a];
            ms.eta[d][a] = (float)e[a];
        }
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int k = i; k < 6; ++k) L[s7(i, k)] += (double)ms.lam(d, s6(i, k));
        eta[6] += ne;
        L[s7(6, 6)] += (double)nl;
        ms.mn[d][0] = (float)ne;
        ms.mn[d][1] = nl;
    }
    if constexpr (TAPE) {
        GDouble* b = plane_of(tape.bel);
#pragma unroll
        for (int k = 0; k < 35; ++k) {
            __builtin_nontemporal_store(k < 28 ? L[k] : eta[k - 28], at(b, o));
            b = next(g, b);
        }
    }

    // --- update, relinearise (Eq. var), transport the stored messages
    reread_lds();
    double m[7], var;
    bool ok = ldl7_solve(L, eta, m, var);
    pose_retract(q, t, m, tau);
    ell += m[6];
    round_point(tau, ell);
#pragma unroll
    for (int d = 0; d < 4; ++d)
        if (has[d]) transport_message(ms, d, m);
    reread_lds();
    if constexpr (FINAL) {
        float* out = DAMPED ? damp.state : Y;
        store_point<NT>(out, g, o, tau, ell);
        store_messages<NT>(out, g, o, ms);
        *at((GFloat*)var_ll, o) = (float)var;
        *at((GFloat*)valid, o) = val ? 1.0f : 0.0f;
    } else {
        // --- linearise at the new point and send the next partials
        pose_exp(tau, q, t);
        pose_rotation(q, R);
        unary_factors(g, s, in, u, v, tau, q, R, t, ell, pin, L, eta);
        store_point<NT>(Y, g, o, tau, ell);
        if constexpr (TAPE) {
            store_point(tape.canonical, g, o, tau, ell);
            store_messages(tape.canonical, g, o, ms);
        }
        if constexpr (DAMPED) store_messages<NT>(damp.state, g, o, ms);
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (has[d]) add_message(L, eta, ms, d);
        ok = emit_partials<NT, TAPE>(g, s, o, has, act, L, eta, ms, Y, tape.marg) && ok;
    }
    if (!ok) atomicOr(health, 1);
}

// Fused passes of one image: one wave per workgroup, 64 pixels of a row, so
// that a SIMD takes the next row segment as soon as one of its two waves ends.
// Bound by memory where the image fills the chip (640 x 480: 74 to 82 us per
// pass, 310 MB of algorithmic bytes, whose copy at this card's 4.74 TB/s takes 65
// us; 1920 x 1080: 455 us, copy 441; 127 us at 640 x 480 before, as one wave per
// SIMD of a persistent workgroup with 504 registers) and by one wave's chain of
// instructions and loads where it does not (256 x 256: 19.7 us, 27 before; 4,303
// vector instructions per wave, 6,234 before; the smallest images take
// k_fu_split).
__global__ __launch_bounds__(64, 2) void k_fu_prologue(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                       float* __restrict__ Y, int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    prologue_pixel<false>(g, s, in, X, Y, health, u, v, buf, threadIdx.x, nullptr);
}

template <bool FINAL>
__global__ __launch_bounds__(64, 2) void k_fu_iterate(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                      float* __restrict__ Y, float* __restrict__ var_ll,
                                                      float* __restrict__ valid, int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    iterate_pixel<FINAL, false>(g, s, in, X, Y, var_ll, valid, health, u, v, buf, threadIdx.x, Tape{});
}

// the same passes for the reverse sweep's recompute: the prologue also writes
// the belief of its state and its depth marginal, the final pass the belief of
// the update (exactly the values of k_pf_linearise, k_pf_messages, k_pf_update)
__global__ __launch_bounds__(64, 2) void k_fu_prologue_tape(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                            float* __restrict__ Y, double* __restrict__ marg,
                                                            int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    prologue_pixel<true>(g, s, in, X, Y, health, u, v, buf, threadIdx.x, marg);
}

// the rotated form of the recompute: the update of iteration k from its
// partial state X (belief into tape.bel, canonical state k + 1 into
// tape.canonical) and the prologue of iteration k + 1 (partials into Y, depth
// marginal and belief into tape.marg) in one pass; the same arithmetic as the
// final form followed by k_fu_prologue_tape on the canonical state. Bound by its
// stores, 1,560 bytes per pixel: 320 x 240, beside the reverse kernels, 54.5 us
// (2,128 bytes, with the messages' information and the pose marginal on the tape
// as well, took 8 us more).
template <bool FINAL>
__global__ __launch_bounds__(64, 2) void k_fu_tape(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                   float* __restrict__ Y, Tape tape, float* __restrict__ var_ll,
                                                   float* __restrict__ valid, int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES_STORING>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    iterate_pixel<FINAL, true>(g, s, in, X, Y, var_ll, valid, health, u, v, buf, threadIdx.x, tape);
}

// The pass of an image that leaves the chip idle: four waves per 64 pixels, a
// direction each. A wave completes, transports and sends on its own direction's
// message; what they all need, the linearisations, the solve and the marginals,
// each computes for itself from the same values in the same order, so that the
// pass agrees with iterate_pixel bit for bit. Bound by one wave's chain, which
// the split shortens: 32 x 24, 10.2 us per pass and 16.8 in one wave; with tape,
// 48 x 48, 13.1 and 23.3.

template <bool FINAL, bool TAPE>
__global__ __launch_bounds__(256, 2) void k_fu_split(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                     float* __restrict__ Y, Tape tape, float* __restrict__ var_ll,
                                                     float* __restrict__ valid, int* __restrict__ health) {
    constexpr bool NT = !TAPE;
    __shared__ float lam_[4 * 21 * 64];   // the four directions' information
    __shared__ double done_[4][7][64];    // the completed messages: eta 6, normal eta
    __shared__ float msg_[4][8][64];      // the transported messages: eta 6, normal eta; normal lambda
    const int lane = threadIdx.x;
    const int d = __builtin_amdgcn_readfirstlane(threadIdx.y);
    int u, v;
    segment_pixel(lane, u, v);
    // lanes past the row's end repeat its last pixel and store nothing
    const bool inside = u < g.W;
    if (!inside) u = g.W - 1;
    const unsigned o = off_of(g, u, v);
    bool has[4];
    unsigned on[4];
    float c[4], pt[7], npt[7], eta_d[6], mn[2];
    load_point_at(X, g, o, pt);
    const PixelInputs pin = load_inputs_at(s, in, o);
    edges_of(g, in, u, v, has, on, c);
    const unsigned od = d == 0 ? on[0] : d == 1 ? on[1] : d == 2 ? on[2] : on[3];
    const bool has_d = d == 0 ? has[0] : d == 1 ? has[1] : d == 2 ? has[2] : has[3];
    const float c_d = d == 0 ? c[0] : d == 1 ? c[1] : d == 2 ? c[2] : c[3];
    load_point_at(X, g, od, npt);
    {
        GFloat* b = plane_of(X, (long)(P_MID + d * MID_STRIDE) * g.plane);
        const unsigned oh = here(od);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            if (k < 6) eta_d[k] = *at(b, oh);
            else
                __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)at(b, oh),
                                                 (__attribute__((address_space(3))) void*)(lam_ + (d * 21 + k - 6) * 64),
                                                 4, 0, 0);
            b = next(g, b);
        }
        b = plane_of(X, (long)(P_MN + 2 * d) * g.plane);
        mn[0] = *at(b, oh);
        mn[1] = *at(next(g, b), oh);
    }
    const auto lam = [&](int dd, int k) { return lam_[(dd * 21 + k) * 64 + lane]; };
    const auto own = [&](int k) { return lam_[(d * 21 + k) * 64 + lane]; };

    // --- linearise at the current point, complete the direction's partial
    double tau[6], ell, q[4], R[9], t[3], L[28], eta[7];
    point_of(pt, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    const bool val = unary_factors(g, s, in, u, v, tau, q, R, t, ell, pin, L, eta);
    const bool act = isfinite(c_d) && s.lamN > 0.0;
    wait_lds_loads();
    if (has_d) {
        double tj[6], ellj, qj[4], trj[3], r[6], e[6];
        point_of(npt, tj, ellj);
        pose_exp(tj, qj, trj);
        pose_between(qj, trj, q, t, r);
        complete_eta(eta_d, own, r, e);
        double ne = 0.0;
        float nl = 0.0f;
        if (act) {
            nl = mn[1];
            ne = fma(-(double)nl, normal_residual_c(c_d, d, ell, ellj), (double)mn[0]);
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            done_[d][a][lane] = e[a];
            eta_d[a] = (float)e[a];
        }
        done_[d][6][lane] = ne;
        mn[0] = (float)ne;
        mn[1] = nl;
    } else {
#pragma unroll
        for (int a = 0; a < 6; ++a) eta_d[a] = 0.0f;
        mn[0] = mn[1] = 0.0f;
    }
    msg_[d][7][lane] = mn[1];
    __syncthreads();
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        if (!has[dd]) continue;
#pragma unroll
        for (int a = 0; a < 6; ++a) eta[a] += done_[dd][a][lane];
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int k = i; k < 6; ++k) L[s7(i, k)] += (double)lam(dd, s6(i, k));
        eta[6] += done_[dd][6][lane];
        L[s7(6, 6)] += (double)msg_[dd][7][lane];
    }
    if constexpr (TAPE) {
        if (d == 0 && inside) {
            GDouble* b = plane_of(tape.bel);
            const unsigned oh = here(o);
#pragma unroll
            for (int k = 0; k < 35; ++k) {
                __builtin_nontemporal_store(k < 28 ? L[k] : eta[k - 28], at(b, oh));
                b = next(g, b);
            }
        }
    }

    // --- update, relinearise (Eq. var), transport the direction's message
    double m[7], var;
    bool ok = ldl7_solve(L, eta, m, var);
    pose_retract(q, t, m, tau);
    ell += m[6];
    round_point(tau, ell);
    if (has_d) transport(eta_d, mn, own, m);
    // the stored form of the direction's message, to `S`
    const auto store_own = [&](float* S) {
        GFloat* b = plane_of(S, (long)(P_MID + d * MID_STRIDE) * g.plane);
        const unsigned oh = here(o);
#pragma unroll
        for (int k = 0; k < 27; ++k) {
            put<NT>(at(b, oh), k < 6 ? eta_d[k] : has_d ? own(k - 6) : 0.0f);
            b = next(g, b);
        }
        b = plane_of(S, (long)(P_MN + 2 * d) * g.plane);
        put<NT>(at(b, oh), mn[0]);
        put<NT>(at(next(g, b), oh), mn[1]);
    };
    if constexpr (FINAL) {
        if (inside) {
            store_own(Y);
            if (d == 0) {
                store_point<NT>(Y, g, o, tau, ell);
                *at((GFloat*)var_ll, o) = (float)var;
                *at((GFloat*)valid, o) = val ? 1.0f : 0.0f;
            }
        }
    } else {
#pragma unroll
        for (int a = 0; a < 6; ++a) msg_[d][a][lane] = eta_d[a];
        msg_[d][6][lane] = mn[0];
        // --- linearise at the new point and send the direction's next partial
        pose_exp(tau, q, t);
        pose_rotation(q, R);
        unary_factors(g, s, in, u, v, tau, q, R, t, ell, pin, L, eta);
        if (inside && d == 0) store_point<NT>(Y, g, o, tau, ell);
        if constexpr (TAPE) {
            if (inside) {
                store_own(tape.canonical);
                if (d == 1) store_point<NT>(tape.canonical, g, o, tau, ell);
            }
        }
        __syncthreads();
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            if (!has[dd]) continue;
#pragma unroll
            for (int a = 0; a < 6; ++a) eta[a] += (double)msg_[dd][a][lane];
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int k = i; k < 6; ++k) L[s7(i, k)] += (double)lam(dd, s6(i, k));
            eta[6] += (double)msg_[dd][6][lane];
            L[s7(6, 6)] += (double)msg_[dd][7][lane];
        }
        double P[21], pm[6], D, dv;
        ok = depth_marginal(L, eta, D, dv) && ok;
        if constexpr (TAPE)
            if (d == 2 && inside) tape_marginals(tape.marg, g, o, D, dv, L, eta);
        pose_marginal(L, eta, L[s7(6, 6)], P, pm);
        if (has_d && inside) {
            emit_normal<NT>(g, s, o, d, D, dv, mn, act, Y);
            ok = emit_identity<NT>(g, s, o, d, P, pm, eta_d, own, Y) && ok;
        }
    }
    if (!ok) atomicOr(health, 1);
}

// ---------------------------------------------------------------------------
// damped iterations
//
// The fused pass with the receiver's stored messages beside the partials: what
// a sender contributes to a damped message still travels as a partial. Bound by
// memory and, below two waves per SIMD, by one wave's chain: 320 x 240, 34.5 us
// per iteration; 41 us as a pass that gathered the senders' FP64 marginals, 87 us
// as three launches per iteration.
template <bool FINAL>
__global__ __launch_bounds__(64, 2) void k_damped_iterate(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                          float* __restrict__ Y, float* state, float beta,
                                                          float* __restrict__ var_ll, float* __restrict__ valid,
                                                          int* __restrict__ health) {
    __shared__ float buf[Messages<LDS_PLANES_STORING>::kFloats];
    int u, v;
    segment_pixel(threadIdx.x, u, v);
    if (u >= g.W) return;
    iterate_pixel<FINAL, false, true>(g, s, in, X, Y, var_ll, valid, health, u, v, buf, threadIdx.x,
                                      Tape{}, Damp{state, beta});
}

// ---------------------------------------------------------------------------
// per-frame statistics (pose mean, valid count, health), deterministic two-stage reduction

constexpr int RED_THREADS = 256;

// the eight sums of a workgroup of RED_THREADS work-items: wavefront
// butterflies (every lane adds the same two operands, in either order), then
// the wavefronts' sums in order
__device__ inline void red8_block(double acc[8], double* __restrict__ out) {
    __shared__ double sh[RED_THREADS / 64][8];
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += __shfl_xor(acc[k], m, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 8; ++k) sh[threadIdx.x >> 6][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 8) {
        double t = 0.0;
        for (int w = 0; w < RED_THREADS / 64; ++w) t += sh[w][threadIdx.x];
        out[threadIdx.x] = t;
    }
}

// The sums are taken over a fixed decomposition of the image, independent of
// any launch shape: 64 x 4 pixel tiles in row-major tile order, one record per
// tile, then the records of an image in one strided order. A single context and
// a batch therefore reduce a sequence's planes in the same order and agree bit
// for bit.
constexpr int ST_X = 64, ST_Y = RED_THREADS / ST_X;

__host__ __device__ inline int stat_tiles_x(int W) { return (W + ST_X - 1) / ST_X; }
__host__ __device__ inline int stat_tiles(int H, int W) { return stat_tiles_x(W) * ((H + ST_Y - 1) / ST_Y); }

// one 64 x 4 tile: sum of the six pose planes, valid count (when use_valid),
// non-finite count, written as out[0..7]; one workgroup of RED_THREADS
__device__ inline void tile_stats(const Geo& g, const float* __restrict__ X, const float* __restrict__ valid,
                                  int use_valid, int tile, double* __restrict__ out) {
    const int ntx = stat_tiles_x(g.W);
    const int u = (tile % ntx) * ST_X + (int)(threadIdx.x % ST_X);
    const int v = (tile / ntx) * ST_Y + (int)(threadIdx.x / ST_X);
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (u < g.W && v < g.H) {
        const long p = pix_of(g, u, v);
        bool fin = true;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const float x = X[(long)k * g.plane + p];
            acc[k] = (double)x;
            fin = fin && isfinite(x);
        }
        fin = fin && isfinite(X[(long)P_ELL * g.plane + p]);
        acc[6] = use_valid ? (double)valid[p] : 0.0;
        acc[7] = fin ? 0.0 : 1.0;
    }
    red8_block(acc, out);
}

// the n tile records of one image, strided over the workgroup, then reduced
__device__ inline void image_stats(const double* __restrict__ partial, int n, double* __restrict__ out) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < n; b += RED_THREADS)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += partial[(long)b * 8 + k];
    red8_block(acc, out);
}

__global__ __launch_bounds__(RED_THREADS) void k_frame_stats(Geo g, const float* __restrict__ X,
                                                            const float* __restrict__ valid, int use_valid,
                                                            double* __restrict__ partial) {
    tile_stats(g, X, valid, use_valid, blockIdx.x, partial + (long)blockIdx.x * 8);
}

// one workgroup: the sum of the nb tile records, in one fixed order;
// result[8] receives the health flag (when given) so that one copy returns both
__global__ __launch_bounds__(RED_THREADS) void k_frame_final(int nblocks, const double* __restrict__ partial,
                                                            double* __restrict__ result,
                                                            const int* __restrict__ health) {
    image_stats(partial, nblocks, result);
    if (health && threadIdx.x == 0) result[8] = (double)*health;
}

// a pixel's output maps: inverse depth and its delta-method variance
__device__ inline void output_pixel(const Geo& g, const float* X, const float* var_ll, int have_var, long p, long o,
                                    float* inv_depth, float* inv_var) {
    const double rho = exp(-(double)X[(long)P_ELL * g.plane + p]);
    if (inv_depth) inv_depth[o] = (float)rho;
    if (inv_var) inv_var[o] = have_var ? (float)(rho * rho * (double)var_ll[p]) : __int_as_float(0x7fc00000);
}

// the output maps (dense H x W)
__global__ void k_outputs(Geo g, const float* __restrict__ X, const float* __restrict__ var_ll, int have_var,
                          float* __restrict__ inv_depth, float* __restrict__ inv_var) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    output_pixel(g, X, var_ll, have_var, pix_of(g, u, v), (long)v * g.W + u, inv_depth, inv_var);
}

// valid-warp flags of the current state without iterating (n_iters == 0)
__global__ __launch_bounds__(256) void k_valid_only(Geo g, Strengths s, Inputs in, const float* __restrict__ X,
                                                    float* __restrict__ valid) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long p = pix_of(g, u, v);
    double tau[6], ell, q[4], R[9], t[3];
    load_point(X, g, p, tau, ell);
    pose_exp(tau, q, t);
    pose_rotation(q, R);
    valid[p] = photometric_begin(g, in, u, v, R, t, ell).valid ? 1.0f : 0.0f;
}

// state exchange: pitched planes <-> dense planes
__global__ void k_pack_state(Geo g, const float* __restrict__ X, float* __restrict__ dense, int to_dense) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long p = pix_of(g, u, v);
    const long N = (long)g.H * g.W, o = (long)v * g.W + u;
    for (int k = 0; k < N_PLANES; ++k) {
        if (to_dense) dense[(long)k * N + o] = X[(long)k * g.plane + p];
        else ((float*)X)[(long)k * g.plane + p] = dense[(long)k * N + o];
    }
}

__global__ void k_copy_plane(Geo g, const float* __restrict__ dense, float* __restrict__ plane) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    plane[pix_of(g, u, v)] = dense[(long)v * g.W + u];
}

// ---------------------------------------------------------------------------
// batched schedule: many sequences of mixed resolution in one launch per pass.
// Each workgroup takes one (sequence, tile) item of the work list; the
// per-pixel arithmetic is the single-sequence code, so results do not depend
// on batching or on the tile shape.

__device__ inline bool batch_pixel(const SeqDesc* __restrict__ seqs, const int2* __restrict__ work,
                                   const SeqDesc*& d, int& u, int& v, int& item) {
    const int2 w = work[blockIdx.x];
    item = w.x;
    d = &seqs[w.y];
    const int tile = w.x - d->tile_base;
    u = (tile % d->tiles_x) * (int)blockDim.x + (int)threadIdx.x;
    v = (tile / d->tiles_x) * (int)blockDim.y + (int)threadIdx.y;
    return u < d->g.W && v < d->g.H;
}

__global__ void k_batch_frame_prep(const SeqDesc* __restrict__ seqs, const int2* __restrict__ work) {
    const SeqDesc* d;
    int u, v, item;
    if (!batch_pixel(seqs, work, d, u, v, item)) return;
    frame_prep_pixel(d->g, d->frame, d->g.W, d->It, d->Gx, d->Gy, u, v);
}

// the wave's LDS planes of a workgroup of any tile shape (batch_lds bytes of
// dynamic LDS) and the lane in its wave
__device__ inline float* batch_buf(int& lane) {
    extern __shared__ float batch_lds_[];
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    lane = tid & 63;
    return batch_lds_ + __builtin_amdgcn_readfirstlane(tid >> 6) * Messages<LDS_PLANES>::kFloats;
}

static size_t batch_lds(int tile_x, int tile_y) {
    return (size_t)((tile_x * tile_y + 63) / 64) * Messages<LDS_PLANES>::kFloats * sizeof(float);
}

__global__ __launch_bounds__(256, 2) void k_batch_prologue(const SeqDesc* __restrict__ seqs, const int2* __restrict__ work,
                                                        int parity, Strengths s, int* __restrict__ health) {
    const SeqDesc* d;
    int u, v, item, lane;
    float* buf = batch_buf(lane);
    if (!batch_pixel(seqs, work, d, u, v, item)) return;
    const float* X = parity ? d->X1 : d->X0;
    float* Y = parity ? d->X0 : d->X1;
    prologue_pixel<false>(d->g, s, d->in, X, Y, health, u, v, buf, lane, nullptr);
}

template <bool FINAL>
__global__ __launch_bounds__(256, 2) void k_batch_iterate(const SeqDesc* __restrict__ seqs, const int2* __restrict__ work,
                                                       int parity, Strengths s, int* __restrict__ health) {
    const SeqDesc* d;
    int u, v, item, lane;
    float* buf = batch_buf(lane);
    if (!batch_pixel(seqs, work, d, u, v, item)) return;
    const float* X = parity ? d->X1 : d->X0;
    float* Y = parity ? d->X0 : d->X1;
    iterate_pixel<FINAL, false>(d->g, s, d->in, X, Y, d->var_ll, d->valid, health, u, v, buf, lane, Tape{});
}

// per sequence (blockIdx.y) and 64 x 4 tile of its image (blockIdx.x): the
// tile's sums, at the sequence's record base; the same tiles and order as a
// single context's statistics
__global__ __launch_bounds__(RED_THREADS) void k_batch_stats(const SeqDesc* __restrict__ seqs, int parity,
                                                            double* __restrict__ partial) {
    const SeqDesc* d = &seqs[blockIdx.y];
    if ((int)blockIdx.x >= stat_tiles(d->g.H, d->g.W)) return;
    const float* X = parity ? d->X1 : d->X0;
    tile_stats(d->g, X, d->valid, 1, blockIdx.x, partial + (long)(d->stat_base + (int)blockIdx.x) * 8);
}

// one workgroup per sequence: its tile records in the single-context order
__global__ __launch_bounds__(RED_THREADS) void k_batch_final(const SeqDesc* __restrict__ seqs,
                                                            const double* __restrict__ partial,
                                                            double* __restrict__ result) {
    const SeqDesc* d = &seqs[blockIdx.x];
    image_stats(partial + (long)d->stat_base * 8, stat_tiles(d->g.H, d->g.W), result + (long)blockIdx.x * 8);
}

// the output maps of the sequences that ask for them, sequence blockIdx.y: in
// dense order, so that maps in pinned host memory leave the chip in whole lines
__global__ __launch_bounds__(256) void k_batch_outputs(const SeqDesc* __restrict__ seqs, int parity) {
    const SeqDesc* d = &seqs[blockIdx.y];
    if (!d->inv_depth && !d->inv_var) return;
    const float* X = parity ? d->X1 : d->X0;
    const int W = d->g.W, N = d->g.H * W;
    for (int i = blockIdx.x * 256 + (int)threadIdx.x; i < N; i += gridDim.x * 256)
        output_pixel(d->g, X, d->var_ll, 1, pix_of(d->g, i % W, i / W), i, d->inv_depth, d->inv_var);
}

static void launch_batch_stats(const BatchLaunch& b, int parity, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_stats, dim3(b.max_stat_tiles, b.n_seq), dim3(RED_THREADS), 0, st, b.seqs, parity,
                       b.partial);
    hipLaunchKernelGGL(k_batch_final, dim3(b.n_seq), dim3(RED_THREADS), 0, st, b.seqs, b.partial, b.result);
}

__global__ void k_clear_int(int* __restrict__ p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) p[0] = 0;
}

// keyframe test of the frame just tracked for every sequence (Sec. 3.5: frame
// count and overlap), on the device: flags and the frame counter
__global__ void k_batch_keyframe_test(const SeqDesc* __restrict__ seqs, int n_seq, const double* __restrict__ result,
                                      const int* __restrict__ health, int* __restrict__ fsk,
                                      unsigned* __restrict__ flags, int max_frames, float min_valid, int reanchor) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_seq) return;
    const double inv_n = 1.0 / ((double)seqs[i].g.H * seqs[i].g.W);
    const float vf = (float)(result[8 * i + 6] * inv_n);
    const int count = fsk[i] + 1;
    unsigned f = 0;
    if (count >= max_frames || vf < min_valid) f |= 1u;          // keyframe due
    if (vf < min_valid) f |= 4u;                                  // low overlap
    if (result[8 * i + 7] > 0.0 || *health != 0) f |= 2u;         // diverged
    flags[i] = f;
    fsk[i] = (reanchor && (f & 1u)) ? 0 : count;
}

// re-anchoring on the frame just tracked, predicated on the device flag of
// the tile's sequence: the frame becomes the keyframe image, its normals the
// normal-integration targets; pose linearisation points and messages reset,
// log-depths kept (the graph of a frame step has no branches)
__global__ __launch_bounds__(256) void k_batch_keyframe_apply(const SeqDesc* __restrict__ seqs,
                                                              const int2* __restrict__ work, int parity,
                                                              const unsigned* __restrict__ flags) {
    const SeqDesc* d;
    int u, v, item;
    const bool in_img = batch_pixel(seqs, work, d, u, v, item);
    const int seq = work[blockIdx.x].y;
    if (!in_img || !(flags[seq] & 1u)) return;
    float* X = parity ? d->X1 : d->X0;
    float* X2 = parity ? d->X0 : d->X1;
    keyframe_prep_pixel(d->g, d->frame, d->normals, d->Is, d->cxt, d->cyt, X, X2, u, v);
}

__global__ void k_set_ints(int* __restrict__ p, int n, int value) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

// the iteration block of a frame step in one launch: the n_passes non-final
// passes that follow the prologue, with a grid-wide barrier between passes
// (the prologue and the final pass, which writes the canonical messages, are
// launches of their own). The grid is co-resident (cooperative launch) and a
// multiple of 8 workgroups, so workgroup b, which runs items b, b + G,
// b + 2G, ..., stays with the work list's range of its XCD. Every workgroup
// reaches every barrier: pixels outside an image skip the arithmetic, not the
// barrier.
__global__ __launch_bounds__(256, 2) void k_batch_persistent(const SeqDesc* __restrict__ seqs,
                                                          const int2* __restrict__ work, int n_work, int parity,
                                                          int n_passes, Strengths s, int* __restrict__ health) {
    cg::grid_group grid = cg::this_grid();
    int lane;
    float* buf = batch_buf(lane);
    for (int pass = 0; pass < n_passes; ++pass) {
        const int par = parity ^ (pass & 1);
        for (int w = blockIdx.x; w < n_work; w += gridDim.x) {
            const int2 wi = work[w];
            const SeqDesc* d = &seqs[wi.y];
            const int tile = wi.x - d->tile_base;
            const int u = (tile % d->tiles_x) * (int)blockDim.x + (int)threadIdx.x;
            const int v = (tile / d->tiles_x) * (int)blockDim.y + (int)threadIdx.y;
            if (u < d->g.W && v < d->g.H) {
                const float* X = par ? d->X1 : d->X0;
                float* Y = par ? d->X0 : d->X1;
                wait_lds_reads();   // of the wave's previous item
                iterate_pixel<false, false>(d->g, s, d->in, X, Y, d->var_ll, d->valid, health, u, v, buf, lane,
                                                  Tape{});
            }
        }
        if (pass + 1 < n_passes) grid.sync();
    }
}

hipError_t launch_batch_frame_step(const BatchLaunch& b, int n_iters, hipStream_t st) {
    const dim3 blk(b.tile_x, b.tile_y), grid(b.n_work);
    const size_t lds = batch_lds(b.tile_x, b.tile_y);
    hipLaunchKernelGGL(k_clear_int, dim3(1), dim3(64), 0, st, b.health);
    hipLaunchKernelGGL(k_batch_frame_prep, grid, blk, 0, st, b.seqs, b.work);
    int parity = b.parity;
    if (n_iters > 0) {
        hipLaunchKernelGGL(k_batch_prologue, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
        parity ^= 1;
        for (int it = 0; it < n_iters; ++it) {
            if (it == n_iters - 1)
                hipLaunchKernelGGL(k_batch_iterate<true>, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
            else
                hipLaunchKernelGGL(k_batch_iterate<false>, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
            parity ^= 1;
        }
    }
    launch_batch_stats(b, parity, st);
    return launch_batch_keyframe(b, parity, st);
}

hipError_t launch_batch_outputs(const BatchLaunch& b, int parity, hipStream_t st) {
    // eight workgroups per CU over all sequences, 64 for each if they are many
    // (device maps of a 1920 x 1080 sequence alone: 26 us of the step, 118 with
    // 64; of 64 sequences of 320 x 240: 22 and 30); a statistics tile is 256
    // pixels of the largest image
    const int share = 2048 / b.n_seq > 64 ? 2048 / b.n_seq : 64;
    const int blocks = b.max_stat_tiles < share ? b.max_stat_tiles : share;
    hipLaunchKernelGGL(k_batch_outputs, dim3(blocks, b.n_seq), dim3(256), 0, st, b.seqs, parity);
    return hipGetLastError();
}

hipError_t launch_set_ints(int* p, int n, int value, hipStream_t st) {
    hipLaunchKernelGGL(k_set_ints, dim3((n + 255) / 256), dim3(256), 0, st, p, n, value);
    return hipGetLastError();
}

hipError_t launch_batch_keyframe(const BatchLaunch& b, int parity, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_keyframe_test, dim3((b.n_seq + 63) / 64), dim3(64), 0, st, b.seqs, b.n_seq, b.result,
                       b.health, b.fsk, b.flags, b.kf_max_frames, b.kf_min_valid, b.reanchor);
    if (b.reanchor)
        hipLaunchKernelGGL(k_batch_keyframe_apply, dim3(b.n_work), dim3(b.tile_x, b.tile_y), 0, st, b.seqs, b.work,
                           parity, b.flags);
    return hipGetLastError();
}

int batch_persistent_grid(const BatchLaunch& b) {
    int per_cu = 0, dev = 0, n_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(k_batch_persistent),
                                                     b.tile_x * b.tile_y, batch_lds(b.tile_x, b.tile_y)) != hipSuccess)
        return 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    int g = per_cu * n_cu;
    if (g > b.n_work) g = b.n_work;
    if (g >= 8) g -= g % 8;
    return g;
}

hipError_t launch_batch_frame_step_persistent(const BatchLaunch& b, int n_iters, int grid_blocks, hipStream_t st) {
    const dim3 blk(b.tile_x, b.tile_y), grid(b.n_work);
    const size_t lds = batch_lds(b.tile_x, b.tile_y);
    hipLaunchKernelGGL(k_clear_int, dim3(1), dim3(64), 0, st, b.health);
    hipLaunchKernelGGL(k_batch_frame_prep, grid, blk, 0, st, b.seqs, b.work);
    hipLaunchKernelGGL(k_batch_prologue, grid, blk, lds, st, b.seqs, b.work, b.parity, b.s, b.health);
    const SeqDesc* seqs = b.seqs;
    const int2* work = b.work;
    int n_work = b.n_work, parity = b.parity ^ 1, n_passes = n_iters - 1;
    Strengths s = b.s;
    int* health = b.health;
    if (n_passes > 0) {
        void* args[] = {&seqs, &work, &n_work, &parity, &n_passes, &s, &health};
        hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_batch_persistent), dim3(grid_blocks),
                                                  blk, args, (unsigned)lds, st);
        if (e != hipSuccess) return e;
    }
    const int fin = b.parity ^ 1 ^ (n_passes & 1);
    hipLaunchKernelGGL(k_batch_iterate<true>, grid, blk, lds, st, b.seqs, b.work, fin, b.s, b.health);
    const int par = fin ^ 1;
    launch_batch_stats(b, par, st);
    return launch_batch_keyframe(b, par, st);
}

hipError_t launch_batch_passes(const BatchLaunch& b, int n_iters, bool prologue, bool final_last, hipStream_t st) {
    const dim3 blk(b.tile_x, b.tile_y), grid(b.n_work);
    const size_t lds = batch_lds(b.tile_x, b.tile_y);
    int parity = b.parity;
    if (prologue) {
        hipLaunchKernelGGL(k_batch_prologue, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
        parity ^= 1;
    }
    for (int it = 0; it < n_iters; ++it) {
        if (final_last && it == n_iters - 1)
            hipLaunchKernelGGL(k_batch_iterate<true>, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
        else
            hipLaunchKernelGGL(k_batch_iterate<false>, grid, blk, lds, st, b.seqs, b.work, parity, b.s, b.health);
        parity ^= 1;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers

static dim3 grid2d(const Geo& g, dim3 b) { return dim3((g.W + b.x - 1) / b.x, (g.H + b.y - 1) / b.y); }
static const dim3 kBlock(64, 1);
static const dim3 kSplitBlock(64, 4);
// One workgroup of four waves per CU, a wave per SIMD: up to there the split
// pass is faster (256 CUs, frames of 20 iterations, 24 row segments: 248 against
// 388 us; 256: 321 against 384), from there on its repeated parts share SIMDs
// (288: 391 against 394; 384: 427 against 418; 576: 609 against 473).
static bool use_split(const Geo& g) {
    static const int n_cu = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return n;
    }();
    return (long)((g.W + 63) / 64) * g.H <= n_cu;
}

hipError_t launch_frame_prep(const Geo& g, const float* src, long src_pitch, float* It, float* Gx, float* Gy,
                             hipStream_t st, int* clear) {
    hipLaunchKernelGGL(k_frame_prep, grid2d(g, kBlock), kBlock, 0, st, g, src, src_pitch, It, Gx, Gy, clear);
    return hipGetLastError();
}

hipError_t launch_keyframe_prep(const Geo& g, const float* img, const float* normals, float* Is, float* cxt,
                                float* cyt, float* X, float* X2, hipStream_t st) {
    hipLaunchKernelGGL(k_keyframe_prep, grid2d(g, kBlock), kBlock, 0, st, g, img, normals, Is, cxt, cyt, X, X2);
    return hipGetLastError();
}

hipError_t launch_init_state(const Geo& g, float* X, float ell0, hipStream_t st) {
    hipLaunchKernelGGL(k_init_state, grid2d(g, kBlock), kBlock, 0, st, g, X, ell0);
    return hipGetLastError();
}

hipError_t launch_damped(const Geo& g, const Strengths& s, const Inputs& in, float* X, float* const part[2],
                         int n_iters, float beta, float* var_ll, float* valid, int* health, hipStream_t st) {
    if (n_iters < 1) return hipSuccess;
    hipLaunchKernelGGL(k_fu_prologue, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, part[0], health);
    for (int it = 0; it < n_iters; ++it) {
        const float* src = part[it & 1];
        float* dst = part[(it & 1) ^ 1];
        if (it + 1 < n_iters)
            hipLaunchKernelGGL(k_damped_iterate<false>, grid2d(g, kBlock), kBlock, 0, st, g, s, in, src, dst, X, beta,
                               var_ll, valid, health);
        else
            hipLaunchKernelGGL(k_damped_iterate<true>, grid2d(g, kBlock), kBlock, 0, st, g, s, in, src, dst, X, beta,
                               var_ll, valid, health);
    }
    return hipGetLastError();
}

hipError_t launch_pf_iteration(const Geo& g, const Strengths& s, const Inputs& in, float* X, double* marg,
                               double* M, float* var_ll, float* valid, int* health, hipStream_t st) {
    hipLaunchKernelGGL(k_pf_linearise, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, marg, valid, health);
    hipLaunchKernelGGL(k_pf_messages, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, marg, M, health);
    hipLaunchKernelGGL(k_pf_update, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, M, var_ll, valid, health);
    return hipGetLastError();
}

hipError_t launch_fu_prologue(const Geo& g, const Strengths& s, const Inputs& in, const float* X, float* Y,
                              int* health, hipStream_t st) {
    hipLaunchKernelGGL(k_fu_prologue, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, Y, health);
    return hipGetLastError();
}

hipError_t launch_fu_iterate(const Geo& g, const Strengths& s, const Inputs& in, const float* X, float* Y,
                             bool final_pass, float* var_ll, float* valid, int* health, hipStream_t st) {
    if (use_split(g)) {
        if (final_pass)
            hipLaunchKernelGGL((k_fu_split<true, false>), grid2d(g, kBlock), kSplitBlock, 0, st, g, s, in, X, Y, Tape{},
                               var_ll, valid, health);
        else
            hipLaunchKernelGGL((k_fu_split<false, false>), grid2d(g, kBlock), kSplitBlock, 0, st, g, s, in, X, Y,
                               Tape{}, var_ll, valid, health);
    } else if (final_pass)
        hipLaunchKernelGGL(k_fu_iterate<true>, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, Y, var_ll, valid, health);
    else
        hipLaunchKernelGGL(k_fu_iterate<false>, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, Y, var_ll, valid,
                           health);
    return hipGetLastError();
}

hipError_t launch_fu_segment_tape(const Geo& g, const Strengths& s, const Inputs& in, const float* X0, float* seg,
                                  long seg_stride, int len, float* tA, float* tB, double* marg, long marg_stride,
                                  double* bel, long bel_stride, float* var_ll, float* valid, int* health,
                                  hipStream_t st) {
    if (len < 1) return hipSuccess;
    const dim3 grid = grid2d(g, kBlock);
    const bool split = use_split(g);
    hipLaunchKernelGGL(k_fu_prologue_tape, grid, kBlock, 0, st, g, s, in, X0, tA, marg, health);
    float* t[2] = {tA, tB};
    for (int k = 0; k < len; ++k) {
        const Tape tape{bel + bel_stride * k, seg + seg_stride * k, marg + marg_stride * (k + 1)};
        const float* src = t[k & 1];
        float* dst = t[(k + 1) & 1];
        if (split && k + 1 < len)
            hipLaunchKernelGGL((k_fu_split<false, true>), grid, kSplitBlock, 0, st, g, s, in, src, dst, tape, var_ll,
                               valid, health);
        else if (split)
            hipLaunchKernelGGL((k_fu_split<true, true>), grid, kSplitBlock, 0, st, g, s, in, src, dst, tape, var_ll,
                               valid, health);
        else if (k + 1 < len)
            hipLaunchKernelGGL(k_fu_tape<false>, grid, kBlock, 0, st, g, s, in, src, dst, tape, var_ll, valid, health);
        else
            hipLaunchKernelGGL(k_fu_tape<true>, grid, kBlock, 0, st, g, s, in, src, dst, tape, var_ll, valid, health);
    }
    return hipGetLastError();
}

hipError_t launch_valid_only(const Geo& g, const Strengths& s, const Inputs& in, const float* X, float* valid,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_valid_only, grid2d(g, kBlock), kBlock, 0, st, g, s, in, X, valid);
    return hipGetLastError();
}

int stats_blocks(const Geo& g) { return stat_tiles(g.H, g.W); }

hipError_t launch_frame_stats(const Geo& g, const float* X, const float* valid, int use_valid, double* partial,
                              double* result, hipStream_t st, const int* health) {
    const int nb = stats_blocks(g);
    hipLaunchKernelGGL(k_frame_stats, dim3(nb), dim3(RED_THREADS), 0, st, g, X, valid, use_valid, partial);
    hipLaunchKernelGGL(k_frame_final, dim3(1), dim3(RED_THREADS), 0, st, nb, partial, result, health);
    return hipGetLastError();
}

hipError_t launch_outputs(const Geo& g, const float* X, const float* var_ll, int have_var, float* inv_depth,
                          float* inv_var, hipStream_t st) {
    hipLaunchKernelGGL(k_outputs, grid2d(g, kBlock), kBlock, 0, st, g, X, var_ll, have_var, inv_depth, inv_var);
    return hipGetLastError();
}

hipError_t launch_pack_state(const Geo& g, const float* X, float* dense, int to_dense, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_state, grid2d(g, kBlock), kBlock, 0, st, g, X, dense, to_dense);
    return hipGetLastError();
}

hipError_t launch_copy_plane(const Geo& g, const float* dense, float* plane, hipStream_t st) {
    hipLaunchKernelGGL(k_copy_plane, grid2d(g, kBlock), kBlock, 0, st, g, dense, plane);
    return hipGetLastError();
}

}  // namespace pv
