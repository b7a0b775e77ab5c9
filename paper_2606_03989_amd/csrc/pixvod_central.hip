// Centralised direct tracking on the GPU (PixVOD, arXiv 2606.03989, Sec. 3.1,
// Eq. photo; the centralised baseline of Sec. 4.4): one global pose and a
// log-depth per keyframe pixel, solved by IRLS Gauss-Newton with every pixel
// accessible at once.
//
// The energy is Eq. (photo) with the per-pixel model's factors at exact
// consensus (every pixel's pose equal to the global one): photometric factors
// with the Huber covariance weighting frozen at the current residuals, each
// pixel's log-depth prior, the normal-integration factors, and one prior
// factor on the pose. Each IRLS iteration:
//   1. linearises every pixel's photometric factor with the per-pixel model's
//      code at the shared pose (the pose block and gradient summed over pixels
//      by a deterministic two-stage reduction, the pose-depth coupling and
//      depth diagonal kept per pixel), its log-depth prior and the
//      normal-integration terms; the pose prior is added once;
//   2. solves the (6 + N) normal equations
//        [A  B ] [d_xi ]   [g_xi ]
//        [B' D ] [d_ell] = [g_ell],  D = diag + lamN * graph Laplacian,
//      by preconditioned conjugate gradients with a block-Jacobi
//      preconditioner (A^-1 for the pose, 1/D_ii for the depths), FP64
//      vectors, to a relative residual tolerance;
//   3. applies xi <- Log(Exp(xi) Exp(d_xi)), ell <- ell + d_ell.
// The conjugate gradients take the single-reduction form of Chronopoulos and
// Gear (1989): with u = P^-1 r and w = M u carried along, the two inner
// products of an iteration (r.u, w.u) come out of one reduction, so each CG
// iteration is one launch over the pixels. The launch updates p, s = M p, x
// and r, forms the new u and, from the neighbours' new u (recomputed by each
// pixel from the neighbours' stored r, w, s, so that no pixel waits for
// another), the new w, and writes per-workgroup partial sums. Its scalar step
// (alpha and beta from the previous launch's partial sums, the pose block's
// part of every vector, the stop test) is evaluated by every workgroup in
// one fixed order, so all take the same values. The scalars pass between
// launches in two alternating records, the per-pixel vectors read by
// neighbours (r, w, s) in two alternating plane sets, the partial sums in two
// alternating buffers, so no launch reads what it writes. The host launches
// the iterations in chunks and stops after the chunk that follows the first
// one whose end state reports convergence (launches after convergence return
// at once).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/pixvod.h"
#include "gbp_device.hpp"
#include "gbp_kernels.h"
#include "runtime_internal.h"

using namespace pv;

namespace {

constexpr int kThreads = 256;      // 64 x 4 pixel blocks
constexpr int kLinPartials = 29;   // A (21), g_xi (6), r.r, valid count
constexpr int kCgPartials = 9;     // r.u, w.u, r.r, sum b_i u_i (6)
constexpr int kCgThreads = 256;    // work-items per workgroup of the CG launches
constexpr int kCgMaxBlocks = 768;  // most workgroups of those launches (a multiple of 8): three per CU
// CG iterations launched between convergence checks. The launches that follow
// the last needed one, up to two chunks, take 10 us each for nothing; a check
// costs about 2 us (640 x 480, 385 iterations in three solves: chunks of 16
// 7.10 ms, 8 6.72, 4 6.64, 2 6.84).
constexpr int kCgChunk = 4;

// solver state in device memory
struct CgState {
    double xi[6];
    double A[21];        // pose block, packed upper
    double Ainv[21];     // its inverse (the pose part of the preconditioner)
    double g[6];         // pose right-hand side
    double x[6];         // the pose step of the last solve
    double rr0, rr;      // |r|^2 at the start and the end of the last solve
    double nvalid;
    int done, iters;     // this solve
    int total;           // CG iterations since the frame started
};

// the CG state between launches: pose parts of the vectors and the scalars
// of the last step
struct CgIter {
    double x[6], r[6], u[6], p[6], s[6];
    double gamma, alpha, rr;
    int done, iters;
};

struct Planes {            // per-pixel FP64 planes (pitched); idiag = 1 / D_ii
    double *ell, *idiag, *b, *gl, *x, *p;
    double *r[2], *w[2], *s[2];   // read by neighbours: two alternating sets
};

// ---------------------------------------------------------------------------
// reductions: wavefront butterflies of lane exchanges, then the wavefronts'
// sums in order. Every step adds the same two operands in every lane (in
// either order), so all lanes hold the same sum, and a reduction evaluated
// in several workgroups over the same data gives the same value in each.

template <int NV>
__device__ inline void wave_sum(double v[NV]) {
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], m, 64);
}

// workgroup (NT work-items) sum of NV doubles per work-item into
// partial[block * NV + k]
template <int NV, int NT>
__device__ inline void block_reduce(double v[NV], double* __restrict__ partial) {
    __shared__ double sh[NT / 64][NV];
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    const int lane = tid & 63, w = tid >> 6;
    const long blk = (long)blockIdx.x + (long)blockIdx.y * gridDim.x;
    wave_sum<NV>(v);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) sh[w][k] = v[k];
    __syncthreads();
    if (tid < NV) {
        double t = 0.0;
        for (int j = 0; j < NT / 64; ++j) t += sh[j][tid];
        partial[blk * NV + tid] = t;
    }
}

// sum of nb partial records of NV doubles, in one fixed order, given to
// every work-item of the workgroup (NT work-items, 1-D); once per kernel
template <int NV, int NT>
__device__ inline void final_sum(const double* __restrict__ partial, int nb, double out[NV]) {
    __shared__ double sh[NT / 64][NV];
    __shared__ double tot[NV];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double t[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) t[k] = 0.0;
    for (int b = threadIdx.x; b < nb; b += NT)
#pragma unroll
        for (int k = 0; k < NV; ++k) t[k] += partial[(long)b * NV + k];
    wave_sum<NV>(t);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) sh[w][k] = t[k];
    __syncthreads();
    if (threadIdx.x < NV) {
        double u = 0.0;
        for (int j = 0; j < NT / 64; ++j) u += sh[j][threadIdx.x];
        tot[threadIdx.x] = u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = tot[k];
}

// inverse of the packed 6x6 pose block (through its Cholesky factor)
__device__ inline void pose_inverse(const double A[21], double Ai[21]) {
    double L[21], idg[6];
    for (int k = 0; k < 21; ++k) L[k] = A[k];
    chol6(L, idg);
    chol6_inverse(L, idg, Ai);
}

__device__ inline double dot6(const double a[6], const double b[6]) {
    double s = 0.0;
    for (int k = 0; k < 6; ++k) s += a[k] * b[k];
    return s;
}

__device__ inline void sym6_mul(const double A[21], const double x[6], double y[6]) {
    for (int r = 0; r < 6; ++r) {
        double s = 0.0;
        for (int c = 0; c < 6; ++c) s += A[s6(r, c)] * x[c];
        y[r] = s;
    }
}

// pose prior (Eq. prior) at xi with precision lamP added to (A, g):
// r = Log(Exp(xi_hat)^-1 Exp(xi)), J = I + ad(r)/2 + ad(r)^2/12
__device__ inline void add_pose_prior(const Strengths& s, const double xi[6], double A[21], double g[6]) {
    double R[9], t[3], rp[6];
    se3_exp(xi, R, t);
    if (s.prior_is_identity) {
        for (int k = 0; k < 6; ++k) rp[k] = xi[k];
    } else {
        double Rr[9], tr[3];
        se3_compose(s.prior_R, s.prior_t, R, t, Rr, tr);
        se3_log(Rr, tr, rp);
    }
    double ad[36], J[36];
    for (int k = 0; k < 36; ++k) ad[k] = 0.0;
    const double* w = rp;
    const double* p = rp + 3;
    const double Wm[9] = {0.0, -w[2], w[1], w[2], 0.0, -w[0], -w[1], w[0], 0.0};
    const double Pm[9] = {0.0, -p[2], p[1], p[2], 0.0, -p[0], -p[1], p[0], 0.0};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            ad[r * 6 + c] = Wm[r * 3 + c];
            ad[(r + 3) * 6 + c] = Pm[r * 3 + c];
            ad[(r + 3) * 6 + c + 3] = Wm[r * 3 + c];
        }
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c) {
            double a2 = 0.0;
            for (int k = 0; k < 6; ++k) a2 += ad[r * 6 + k] * ad[k * 6 + c];
            J[r * 6 + c] = (r == c ? 1.0 : 0.0) + 0.5 * ad[r * 6 + c] + a2 * (1.0 / 12.0);
        }
    for (int a = 0; a < 6; ++a) {
        double e = 0.0;
        for (int k = 0; k < 6; ++k) e += J[k * 6 + a] * rp[k];
        g[a] -= s.lamP * e;
        for (int b = a; b < 6; ++b) {
            double m = 0.0;
            for (int k = 0; k < 6; ++k) m += J[k * 6 + a] * J[k * 6 + b];
            A[s6(a, b)] += s.lamP * m;
        }
    }
}

// ---------------------------------------------------------------------------
// kernels

__global__ void k_c_keyframe(Geo g, const float* __restrict__ img, const float* __restrict__ normals,
                             float* __restrict__ Is, float* __restrict__ cxt, float* __restrict__ cyt) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long dense = (long)v * g.W + u;
    const long p = pix_of(g, u, v);
    Is[p] = img[dense];
    // normal-integration targets of Eq. (gbpni), inactive at grazing normals
    const double q0 = ((double)u - g.cx) / g.fx, q1 = ((double)v - g.cy) / g.fy;
    const double n0 = normals[3 * dense], n1 = normals[3 * dense + 1], n2 = normals[3 * dense + 2];
    const double nq = n0 * q0 + n1 * q1 + n2;
    const double qn = sqrt(q0 * q0 + q1 * q1 + 1.0);
    const bool ok = isfinite(nq) && fabs(nq) >= 1e-3 * qn;
    cxt[p] = ok ? (float)(n0 / (g.fx * nq)) : __int_as_float(0x7fc00000);
    cyt[p] = ok ? (float)(n1 / (g.fy * nq)) : __int_as_float(0x7fc00000);
}

// per pixel, bit d: the normal edge to neighbour d exists and is active (a
// keyframe property)
__global__ void k_c_edges(Geo g, Inputs in, unsigned char* __restrict__ act) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long pi = pix_of(g, u, v);
    int a = 0;
    for (int d = 0; d < 4; ++d) {
        int nu, nv;
        if (neighbour(g, u, v, d, nu, nv) && normal_active(g, in, pi, pix_of(g, nu, nv), d)) a |= 1 << d;
    }
    act[pi] = (unsigned char)a;
}

// linearisation at the shared pose and CG start (x = 0, r = g)
__global__ __launch_bounds__(kThreads) void k_c_linearise(Geo g, Strengths s, Inputs in,
                                                          const CgState* __restrict__ cs, Planes P,
                                                          double* __restrict__ partial) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    double red[kLinPartials];
    for (int k = 0; k < kLinPartials; ++k) red[k] = 0.0;
    if (u < g.W && v < g.H) {
        const long pi = pix_of(g, u, v);
        double tau[6], q[4], R[9], t[3], L[28], eta[7];
        for (int k = 0; k < 6; ++k) tau[k] = cs->xi[k];
        pose_exp(tau, q, t);
        pose_rotation(q, R);
        const double ell = P.ell[pi];
        // the photometric factor alone; the log-depth prior is added here, the
        // pose prior once per solve
        for (int k = 0; k < 28; ++k) L[k] = 0.0;
        for (int k = 0; k < 7; ++k) eta[k] = 0.0;
        const Photo f = photometric(g, s, in, u, v, R, t, ell, load_pixel_inputs(g, s, in, u, v));
        add_photometric(f, L, eta);
        const bool val = f.valid;
        double diag = L[s7(6, 6)] + s.lamP, gl = eta[6] - s.lamP * (ell - s.prior_ell);
        if (s.lamN > 0.0) {
            for (int d = 0; d < 4; ++d) {
                int nu, nv;
                if (!neighbour(g, u, v, d, nu, nv)) continue;
                const long pj = pix_of(g, nu, nv);
                double rn;
                if (normal_residual(g, in, pi, pj, d, ell, P.ell[pj], rn)) {
                    diag += s.lamN;
                    gl -= s.lamN * rn;
                }
            }
        }
        P.idiag[pi] = rcp_nr(diag);
        for (int k = 0; k < 6; ++k) P.b[(long)k * g.plane + pi] = L[s7(k, 6)];
        P.gl[pi] = gl;
        P.x[pi] = 0.0;
        P.r[0][pi] = gl;
        for (int r = 0, k = 0; r < 6; ++r)
            for (int c = r; c < 6; ++c) red[k++] = L[s7(r, c)];
        for (int k = 0; k < 6; ++k) red[21 + k] = eta[k];
        red[27] = gl * gl;
        red[28] = val ? 1.0 : 0.0;
    }
    block_reduce<kLinPartials, kThreads>(red, partial);
}

// the pose block, its inverse, the pose part of the CG start (x = 0, r = g,
// u = A^-1 g) and |r_0|^2
__global__ __launch_bounds__(kThreads) void k_c_lin_final(Strengths s, int nb, const double* __restrict__ partial,
                                                          CgState* __restrict__ cs, CgIter* __restrict__ rec0) {
    double tot[kLinPartials];
    final_sum<kLinPartials, kThreads>(partial, nb, tot);
    if (threadIdx.x != 0) return;
    double xi[6];
    for (int k = 0; k < 6; ++k) xi[k] = cs->xi[k];
    add_pose_prior(s, xi, tot, tot + 21);
    for (int k = 0; k < 21; ++k) cs->A[k] = tot[k];
    for (int k = 0; k < 6; ++k) cs->g[k] = tot[21 + k];
    pose_inverse(cs->A, cs->Ainv);
    CgIter st;
    for (int k = 0; k < 6; ++k) {
        st.x[k] = 0.0;
        st.r[k] = cs->g[k];
        st.p[k] = 0.0;
        st.s[k] = 0.0;
    }
    sym6_mul(cs->Ainv, st.r, st.u);
    cs->rr0 = tot[27] + dot6(st.r, st.r);
    cs->rr = cs->rr0;
    cs->nvalid = tot[28];
    cs->iters = 0;
    cs->done = (cs->rr0 > 0.0) ? 0 : 1;
    st.gamma = 0.0;
    st.alpha = 0.0;
    st.rr = cs->rr0;
    st.done = cs->done;
    st.iters = 0;
    *rec0 = st;
}

// The CG launches: kCgThreads work-items per workgroup, each with two pixels
// of a column, v even and v + 1, per round (item base + work-item, along row
// pairs): either is the other's vertical neighbour, so that a pair needs two
// recomputed neighbours and not four. Workgroup b takes range
// (b mod 8) * (nbx / 8) + b / 8 (nbx, the grid, a multiple of 8): workgroups are
// dealt to the eight XCDs in turn, so each XCD gets adjacent ranges and finds
// most of their vertical neighbours in its own L2. Rounds stride over the image
// when the grid is smaller than it.
//
// Since D u = r, w = M u needs no diagonal: w = r - lamN sum u_j + b.u_pose,
// and 1 / D_ii is kept instead of it. A pixel's horizontal neighbours are the
// adjacent lanes (the items of a range are consecutive), whose new u comes by a
// lane exchange; the lanes at the ends of a wave and the pairs above and below
// are recomputed from their stored r, w, s.

__device__ inline int cg_range(int b, int nbx) { return (b & 7) * (nbx >> 3) + (b >> 3); }

struct CgOther {           // what a neighbour's new u is computed from
    double r, w, s, idiag;
};

struct CgPair {            // what an iteration needs of an item's two pixels
    int act[2];
    long pi[2];
    bool in[2];            // whether there is such a pixel
    double x[2], p[2], r[2], w[2], s[2], idiag[2], b[2][6];
    CgOther up, down;      // the pixels above and below the pair
    CgOther side[2];       // first and last lane of a wave: the left or right neighbours
};

__device__ inline CgOther cg_other(const Planes& P, int cur, bool first, long pj) {
    return {P.r[cur][pj], P.w[cur][pj], first ? 0.0 : P.s[cur][pj], P.idiag[pj]};
}

__device__ inline int cg_items(const Geo& g) { return g.W * ((g.H + 1) / 2); }

// loads item i of n; one past the end repeats the last, a missing pixel or
// neighbour reads one that is there, and its value is not used
__device__ inline void cg_load(const Geo& g, const Planes& P, const unsigned char* __restrict__ act, int cur,
                               bool first, int i, int n, CgPair& a) {
    const int ic = i < n ? i : n - 1;
    const int u = ic % g.W, v = ic / g.W * 2;
    a.pi[0] = pix_of(g, u, v);
    a.in[0] = i < n;
    a.in[1] = i < n && v + 1 < g.H;
    a.pi[1] = v + 1 < g.H ? a.pi[0] + g.pitch : a.pi[0];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const long pi = a.pi[j];
        a.act[j] = act[pi];
        a.r[j] = P.r[cur][pi];
        a.w[j] = P.w[cur][pi];
        a.s[j] = first ? 0.0 : P.s[cur][pi];
        a.idiag[j] = P.idiag[pi];
    }
    a.up = cg_other(P, cur, first, v > 0 ? a.pi[0] - g.pitch : a.pi[0]);
    a.down = cg_other(P, cur, first, v + 2 < g.H ? a.pi[0] + 2 * g.pitch : a.pi[1]);
    const int lane = threadIdx.x & 63;
    if (lane == 0 || lane == 63) {
        const int step = lane == 0 ? (u > 0 ? -1 : 0) : (u + 1 < g.W ? 1 : 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) a.side[j] = cg_other(P, cur, first, a.pi[j] + step);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const long pi = a.pi[j];
        a.x[j] = P.x[pi];
        a.p[j] = first ? 0.0 : P.p[pi];
#pragma unroll
        for (int k = 0; k < 6; ++k) a.b[j][k] = P.b[(long)k * g.plane + pi];
    }
}

// one pixel's new residual from its stored r, w, s (explicit FMAs, so that a
// pixel and its neighbours evaluate the same expression bit for bit)
__device__ inline double cg_new_r(double r, double w, double s_prev, double alpha, double beta, double& s_new) {
    s_new = fma(beta, s_prev, w);
    return fma(-alpha, s_new, r);
}

// the sums of kCgPartials values over the workgroup into column `block` of
// part (kCgPartials rows of kCgMaxBlocks). The first eight are reduced
// together: in three steps a lane keeps half of its values and takes the other
// lane's part of that half, so that 16 lane exchanges do the work of 54.
__device__ inline void cg_block_reduce(double v[kCgPartials], double* __restrict__ part, int block) {
    static_assert(kCgPartials == 9, "eight sums and one");
    __shared__ double sh[kCgThreads / 64][kCgPartials];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double h[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) h[k] = v[k];
#pragma unroll
    for (int n = 4, m = 32; n > 0; n >>= 1, m >>= 1) {
        const bool up = lane & m;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const double give = up ? h[k] : h[n + k], keep = up ? h[n + k] : h[k];
            h[k] = keep + __shfl_xor(give, m, 64);
        }
    }
    double t8 = v[8];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) t8 += __shfl_xor(t8, m, 64);
#pragma unroll
    for (int m = 4; m > 0; m >>= 1) h[0] += __shfl_xor(h[0], m, 64);
    // lanes 8 j hold sum j (bit-reversed: the first step's bit is the top one)
    if ((lane & 7) == 0) sh[w][lane >> 3] = h[0];
    if (lane == 0) sh[w][8] = t8;
    __syncthreads();
    if (threadIdx.x < kCgPartials) {
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < kCgThreads / 64; ++j) t += sh[j][threadIdx.x];
        part[(long)threadIdx.x * kCgMaxBlocks + block] = t;
    }
}

// the totals over nb workgroups' records in one fixed order, wave w takes the
// sums w and w + 4, the first wave the last one as well; tot is in LDS and
// complete after the next barrier
__device__ inline void cg_totals(const double* __restrict__ part, int nb, double* tot) {
    static_assert(kCgThreads / 64 == 4 && kCgPartials == 9, "two sums per wave and one more");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* row = part + (long)w * kCgMaxBlocks;
    double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kCgMaxBlocks / 64; ++j) {
        const int b = lane + 64 * j;
        if (b < nb) {
            t[0] += row[b];
            t[1] += row[4 * kCgMaxBlocks + b];
            if (w == 0) t[2] += row[8 * kCgMaxBlocks + b];
        }
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) t[k] += __shfl_xor(t[k], m, 64);
    if (lane == 0) {
        tot[w] = t[0];
        tot[4 + w] = t[1];
        if (w == 0) tot[8] = t[2];
    }
}

// the new vectors, w = M u and the partial sums of one pixel; un: the
// neighbours' new u, up the pose's
__device__ inline void cg_apply_pixel(const double b[6], const double un[4], int act, double lamN,
                                      const double upose[6], double r, double u, double& w, double red[kCgPartials]) {
    double q = r;
#pragma unroll
    for (int d = 0; d < 4; ++d) q = fma(-lamN, (act & (1 << d)) ? un[d] : 0.0, q);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        q = fma(b[k], upose[k], q);
        red[3 + k] = fma(b[k], u, red[3 + k]);
    }
    w = q;
    red[0] = fma(r, u, red[0]);
    red[1] = fma(q, u, red[1]);
    red[2] = fma(r, r, red[2]);
}

// the four neighbours' u of a pair's pixels, from the pair's own and the
// recomputed ones above, below and (edge lanes) beside it
__device__ inline void cg_neighbours(const double u[2], double up, double down, const double side[2],
                                     double un[2][4]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const double l = __shfl_up(u[j], 1, 64), r = __shfl_down(u[j], 1, 64);
        un[j][DIR_L] = lane == 0 ? side[j] : l;
        un[j][DIR_R] = lane == 63 ? side[j] : r;
    }
    un[0][DIR_U] = up;
    un[0][DIR_D] = u[1];
    un[1][DIR_U] = u[0];
    un[1][DIR_D] = down;
}

// CG start: u_0 = P^-1 r_0 and w_0 = M u_0 (planes of set 0), partial sums
__global__ __launch_bounds__(kCgThreads) void k_c_cg_init(Geo g, Strengths s, Planes P,
                                                          const unsigned char* __restrict__ act,
                                                          const CgIter* __restrict__ rec0,
                                                          double* __restrict__ part_out) {
    __shared__ double sh_u[6];
    __shared__ int sh_done;
    if (threadIdx.x == 0) {
        for (int k = 0; k < 6; ++k) sh_u[k] = rec0->u[k];
        sh_done = rec0->done;
    }
    __syncthreads();
    if (sh_done) return;
    double up[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) up[k] = sh_u[k];
    double red[kCgPartials];
#pragma unroll
    for (int k = 0; k < kCgPartials; ++k) red[k] = 0.0;
    const int n = cg_items(g);
    for (int rb = cg_range(blockIdx.x, gridDim.x); rb * kCgThreads < n; rb += gridDim.x) {
        CgPair c;
        cg_load(g, P, act, 0, true, rb * kCgThreads + threadIdx.x, n, c);
        double u[2], un[2][4], side[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            u[j] = c.r[j] * c.idiag[j];
            side[j] = c.side[j].r * c.side[j].idiag;
        }
        cg_neighbours(u, c.up.r * c.up.idiag, c.down.r * c.down.idiag, side, un);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (!c.in[j]) continue;
            double w;
            cg_apply_pixel(c.b[j], un[j], s.lamN > 0.0 ? c.act[j] : 0, s.lamN, up, c.r[j], u[j], w, red);
            P.w[0][c.pi[j]] = w;
        }
    }
    cg_block_reduce(red, part_out, blockIdx.x);
}

// CG iteration k (planes of set cur in, set 1 - cur out): the scalar step
//   gamma = r.u, delta = w.u (w's pose part: A u + sum b_i u_i), stop test,
//   beta = gamma / gamma_prev, alpha = gamma / (delta - beta gamma / alpha_prev)
//   (k = 0: beta = 0, alpha = gamma / delta),
// then p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s, u = P^-1 r,
// w = M u and the partial sums for the next step. The scalar step runs on the
// first wave of each workgroup, a lane per pose component, and reaches the
// others via LDS. Every load of the launch (the previous partial sums, the pose
// block and its inverse, the scalar record, the first round's pixels and
// neighbours) is issued before the first wait. The launch is bound by its chain
// of latencies (the waves wait on memory for 71% of their life) and by the 42 MB
// that it moves at 640 x 480: 14.7 us per launch there, 7.5 us at 32 x 24. Three
// solves of 385 iterations, 640 x 480: 6.52 ms; 6.67 with a pixel at a time and
// so four recomputed neighbours per two pixels.
__global__ __launch_bounds__(kCgThreads, 3) void k_c_cg_iter(Geo g, Strengths s, const CgState* __restrict__ cs,
                                                             Planes P, const unsigned char* __restrict__ act,
                                                             const CgIter* __restrict__ rin,
                                                             CgIter* __restrict__ rout,
                                                             const double* __restrict__ part_in,
                                                             double* __restrict__ part_out, int cur, double tol2,
                                                             int first, int* __restrict__ done_flag) {
    __shared__ double sh_tot[kCgPartials];
    __shared__ double sh_ab[2];
    __shared__ double sh_A[42];     // the pose block and its inverse
    __shared__ CgIter sh_st;
    static_assert(sizeof(CgIter) % 8 == 0 && sizeof(CgIter) / 8 <= 64, "the record fits one wave");
    static_assert(offsetof(CgState, Ainv) == offsetof(CgState, A) + 21 * sizeof(double), "A and its inverse");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (wv == 1 && lane < 42) sh_A[lane] = cs->A[lane];
    if (wv == 2 && lane < (int)(sizeof(CgIter) / 8))
        reinterpret_cast<double*>(&sh_st)[lane] = reinterpret_cast<const double*>(rin)[lane];
    cg_totals(part_in, gridDim.x, sh_tot);
    const int n = cg_items(g);
    int rb = cg_range(blockIdx.x, gridDim.x);
    CgPair c;
    cg_load(g, P, act, cur, first != 0, rb * kCgThreads + tid, n, c);
    const double rr0 = cs->rr0;
    __syncthreads();
    if (wv == 0) {
        // lane k < 6: component k of the pose's part (the other lanes repeat
        // component 5 and add nothing)
        CgIter& st = sh_st;
        const int k = lane < 6 ? lane : 5;
        const bool own = lane < 6;
        const double u = st.u[k], r = st.r[k];
        double w = sh_tot[3 + k];
#pragma unroll
        for (int c = 0; c < 6; ++c) w = fma(sh_A[s6(k, c)], st.u[c], w);
        double gamma = own ? r * u : 0.0, delta = own ? w * u : 0.0, rr = own ? r * r : 0.0;
#pragma unroll
        for (int m = 4; m > 0; m >>= 1) {
            gamma += __shfl_xor(gamma, m, 64);
            delta += __shfl_xor(delta, m, 64);
            rr += __shfl_xor(rr, m, 64);
        }
        gamma = __shfl(gamma, 0, 64) + sh_tot[0];
        delta = __shfl(delta, 0, 64) + sh_tot[1];
        rr = __shfl(rr, 0, 64) + sh_tot[2];
        const int was = st.done, iters = st.iters;
        const int done = (was || (!first && rr <= tol2 * rr0)) ? 1 : 0;
        if (!done) {
            const double beta = first ? 0.0 : gamma * rcp_nr(st.gamma);
            const double alpha = first ? gamma * rcp_nr(delta) : gamma * rcp_nr(delta - beta * gamma * rcp_nr(st.alpha));
            const double pk = fma(beta, st.p[k], u), sk = fma(beta, st.s[k], w);
            const double rk = fma(-alpha, sk, r), xk = fma(alpha, pk, st.x[k]);
            double un = 0.0;
#pragma unroll
            for (int c = 0; c < 6; ++c) un = fma(sh_A[21 + s6(k, c)], __shfl(rk, c, 64), un);
            __builtin_amdgcn_wave_barrier();   // every lane has read the record
            if (own) {
                st.p[k] = pk;
                st.s[k] = sk;
                st.x[k] = xk;
                st.r[k] = rk;
                st.u[k] = un;
            }
            if (lane == 0) {
                sh_ab[0] = alpha;
                sh_ab[1] = beta;
                st.gamma = gamma;
                st.alpha = alpha;
            }
        }
        if (lane == 0 && !was) {
            st.rr = rr;
            if (!first) st.iters = iters + 1;
            st.done = done;
        }
    }
    __syncthreads();
    const int done = sh_st.done;
    if (blockIdx.x == 0 && wv == 1) {
        if (lane < (int)(sizeof(CgIter) / 8))
            reinterpret_cast<double*>(rout)[lane] = reinterpret_cast<const double*>(&sh_st)[lane];
        if (lane == 0 && done_flag) *done_flag = done;
    }
    if (done) return;
    const double alpha = sh_ab[0], beta = sh_ab[1], lamN = s.lamN;
    const int nxt = 1 - cur;
    double up[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) up[k] = sh_st.u[k];
    double red[kCgPartials];
#pragma unroll
    for (int k = 0; k < kCgPartials; ++k) red[k] = 0.0;
    const auto other = [&](const CgOther& o) {
        double sn;
        return cg_new_r(o.r, o.w, o.s, alpha, beta, sn) * o.idiag;
    };
    while (true) {
        double u[2], r[2], sv[2], un[2][4], side[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            r[j] = cg_new_r(c.r[j], c.w[j], c.s[j], alpha, beta, sv[j]);
            u[j] = r[j] * c.idiag[j];
            side[j] = other(c.side[j]);
        }
        cg_neighbours(u, other(c.up), other(c.down), side, un);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (!c.in[j]) continue;
            const long pi = c.pi[j];
            const double pn = fma(beta, c.p[j], c.r[j] * c.idiag[j]);
            double w;
            cg_apply_pixel(c.b[j], un[j], lamN > 0.0 ? c.act[j] : 0, lamN, up, r[j], u[j], w, red);
            P.x[pi] = fma(alpha, pn, c.x[j]);
            P.p[pi] = pn;
            P.s[nxt][pi] = sv[j];
            P.r[nxt][pi] = r[j];
            P.w[nxt][pi] = w;
        }
        rb += gridDim.x;
        if (rb * kCgThreads >= n) break;
        cg_load(g, P, act, cur, first != 0, rb * kCgThreads + tid, n, c);
    }
    cg_block_reduce(red, part_out, blockIdx.x);
}

// after the last launched iteration: the stop test of the last update (if the
// solve had not stopped) and the solve's results into the solver state
__global__ __launch_bounds__(kCgThreads) void k_c_cg_end(CgState* __restrict__ cs, const CgIter* __restrict__ rin,
                                                         const double* __restrict__ part_in, int nbx, double tol2) {
    __shared__ double sh_tot[kCgPartials];
    cg_totals(part_in, nbx, sh_tot);
    __syncthreads();
    if (threadIdx.x != 0) return;
    CgIter st = *rin;
    if (!st.done) {
        st.rr = sh_tot[2] + dot6(st.r, st.r);
        st.iters += 1;
        if (st.rr <= tol2 * cs->rr0) st.done = 1;
    }
    for (int k = 0; k < 6; ++k) cs->x[k] = st.x[k];
    cs->rr = st.rr;
    cs->done = st.done;
    cs->iters = st.iters;
    cs->total += st.iters;
}

__global__ void k_c_apply(Geo g, Planes P) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long pi = pix_of(g, u, v);
    P.ell[pi] += P.x[pi];
}

// xi <- Log(Exp(xi) Exp(d_xi))
__global__ void k_c_apply_pose(CgState* __restrict__ cs) {
    if (threadIdx.x != 0) return;
    double R0[9], t0[3], Rd[9], td[3], R1[9], t1[3], d[6], xi[6];
    for (int k = 0; k < 6; ++k) {
        xi[k] = cs->xi[k];
        d[k] = cs->x[k];
    }
    se3_exp(xi, R0, t0);
    se3_exp(d, Rd, td);
    se3_compose(R0, t0, Rd, td, R1, t1);
    se3_log(R1, t1, xi);
    for (int k = 0; k < 6; ++k) cs->xi[k] = xi[k];
}

__global__ void k_c_dense_depth(Geo g, double* __restrict__ ell, double* __restrict__ dense, int to_dense,
                                float* __restrict__ inv_depth) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= g.W || v >= g.H) return;
    const long pi = pix_of(g, u, v), d = (long)v * g.W + u;
    if (dense) {
        if (to_dense) dense[d] = ell[pi];
        else ell[pi] = dense[d];
    }
    if (inv_depth) inv_depth[d] = (float)exp(-ell[pi]);
}

__global__ void k_c_reset_total(CgState* __restrict__ cs) {
    if (threadIdx.x == 0) cs->total = 0;
}

__global__ void k_c_fill(double* __restrict__ p, long n, double v) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
// the ABI

struct pixvod_central {
    int H = 0, W = 0, pitch = 0;
    long plane = 0;
    pixvod_intrinsics K{};
    pixvod_params P{};
    int max_cg = 0;
    double tol = 0.0;
    hipStream_t own_stream = nullptr, stream = nullptr;
    float *Is = nullptr, *cxt = nullptr, *cyt = nullptr, *It = nullptr, *Gx = nullptr, *Gy = nullptr;
    float *stage = nullptr, *out_stage = nullptr;
    double* planes = nullptr;       // ell, diag, b (6), gl, x, p, r (2), w (2), s (2)
    double* partial = nullptr;
    double* dense = nullptr;
    CgState* cs = nullptr;
    CgState* h_cs = nullptr;        // pinned host copy
    int nb = 0;
    bool have_kf = false;
    double last_ms = 0.0;
    hipEvent_t ev[2] = {nullptr, nullptr};
    CgIter* rec = nullptr;          // the CG launches' two scalar records
    double* part_cg = nullptr;      // their per-workgroup partial sums (two alternating buffers)
    unsigned char* act = nullptr;   // active normal edges per pixel (bit per direction)
    int* h_done = nullptr;          // pinned, coherent: the stop flag after each of the last two chunks
    int* d_done = nullptr;          // its device address
    hipEvent_t evc[2] = {nullptr, nullptr};
    std::string err;
};

namespace {

int cfail(pixvod_central* c, int code, const std::string& m) {
    if (c) c->err = m;
    record_error(m);
    return code;
}

#define C_TRY(c, expr)                                                                        \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return cfail((c), PIXVOD_EHIP, std::string(#expr ": ") + hipGetErrorString(e_));  \
    } while (0)

Geo cgeo(const pixvod_central* c) {
    Geo g;
    g.H = c->H;
    g.W = c->W;
    g.pitch = c->pitch;
    g.plane = c->plane;
    g.fx = c->K.fx;
    g.fy = c->K.fy;
    g.cx = c->K.cx;
    g.cy = c->K.cy;
    g.ifx = 1.0 / g.fx;
    g.ify = 1.0 / g.fy;
    return g;
}

Planes cplanes(const pixvod_central* c) {
    const long pl = c->plane;
    double* b = c->planes;
    Planes P;
    P.ell = b;
    P.idiag = b + pl;
    P.b = b + 2 * pl;
    P.gl = b + 8 * pl;
    P.x = b + 9 * pl;
    P.p = b + 10 * pl;
    for (int k = 0; k < 2; ++k) {
        P.r[k] = b + (11 + k) * pl;
        P.w[k] = b + (13 + k) * pl;
        P.s[k] = b + (15 + k) * pl;
    }
    return P;
}
constexpr int kPlanes = 17;

Inputs cinputs(const pixvod_central* c) {
    Inputs in;
    std::memset(&in, 0, sizeof(in));
    in.Is = c->Is;
    in.cxt = c->cxt;
    in.cyt = c->cyt;
    in.It = c->It;
    in.Gx = c->Gx;
    in.Gy = c->Gy;
    return in;
}

dim3 cgrid(const Geo& g) { return dim3((g.W + 63) / 64, (g.H + 3) / 4); }

void crelease(pixvod_central* c) {
    void* bufs[] = {c->Is,     c->cxt,   c->cyt,   c->It,      c->Gx,         c->Gy,    c->stage, c->out_stage,
                    c->planes, c->partial, c->dense, c->cs, c->rec, c->part_cg, c->act};
    for (void* b : bufs)
        if (b) (void)hipFree(b);
    if (c->h_cs) (void)hipHostFree(c->h_cs);
    if (c->h_done) (void)hipHostFree(c->h_done);
    for (hipEvent_t e : c->ev)
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : c->evc)
        if (e) (void)hipEventDestroy(e);
    if (c->own_stream) (void)hipStreamDestroy(c->own_stream);
}

template <class T>
int calloc_dev(pixvod_central* c, T** p, size_t n) {
    if (hipMalloc((void**)p, n * sizeof(T)) != hipSuccess) {
        *p = nullptr;
        return cfail(c, PIXVOD_ENOMEM, "device allocation failed");
    }
    return PIXVOD_OK;
}

}  // namespace

extern "C" {

int pixvod_central_create(int H, int W, const pixvod_intrinsics* K, const pixvod_params* params, int max_cg,
                          double cg_tol, pixvod_central** out) {
    if (!out) return cfail(nullptr, PIXVOD_EINVAL, "out is NULL");
    *out = nullptr;
    if (H < 2 || W < 2 || (long)H * W > (1L << 26)) return cfail(nullptr, PIXVOD_EINVAL, "need 2 <= H, W and H*W <= 2^26");
    if (!K || !(K->fx > 0) || !(K->fy > 0) || !std::isfinite(K->cx) || !std::isfinite(K->cy))
        return cfail(nullptr, PIXVOD_EINVAL, "intrinsics must be finite with fx, fy > 0");
    if (max_cg < 1 || !(cg_tol > 0.0) || !(cg_tol < 1.0)) return cfail(nullptr, PIXVOD_EINVAL, "need max_cg >= 1, 0 < cg_tol < 1");
    pixvod_params P;
    if (params) P = *params;
    else pixvod_default_params(&P);
    if (!params_valid(&P)) return cfail(nullptr, PIXVOD_EINVAL, "invalid parameters");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) return cfail(nullptr, PIXVOD_ENODEV, "no HIP device");
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess ||
        std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return cfail(nullptr, PIXVOD_ENODEV, "need a gfx950 device");
    pixvod_central* c = new pixvod_central();
    c->H = H;
    c->W = W;
    c->pitch = (W + 63) / 64 * 64;
    c->plane = (long)H * c->pitch;
    c->K = *K;
    c->P = P;
    c->max_cg = max_cg;
    c->tol = cg_tol;
    const Geo g = cgeo(c);
    const dim3 gr = cgrid(g);
    c->nb = (int)(gr.x * gr.y);
    const size_t pl = (size_t)c->plane, N = (size_t)H * W;
    int rc = PIXVOD_OK;
    float** fb[] = {&c->Is, &c->cxt, &c->cyt, &c->It, &c->Gx, &c->Gy};
    for (float** f : fb)
        if (!rc) rc = calloc_dev(c, f, pl);
    if (!rc) rc = calloc_dev(c, &c->stage, 4 * N);
    if (!rc) rc = calloc_dev(c, &c->out_stage, N);
    if (!rc) rc = calloc_dev(c, &c->planes, pl * kPlanes);
    if (!rc) rc = calloc_dev(c, &c->partial, (size_t)c->nb * kLinPartials);
    if (!rc) rc = calloc_dev(c, &c->dense, N);
    if (!rc) rc = calloc_dev(c, &c->cs, 1);
    if (!rc) rc = calloc_dev(c, &c->rec, 2);
    if (!rc) rc = calloc_dev(c, &c->part_cg, (size_t)2 * kCgMaxBlocks * kCgPartials);
    if (!rc && hipHostMalloc((void**)&c->h_cs, sizeof(CgState)) != hipSuccess) rc = cfail(c, PIXVOD_ENOMEM, "pinned allocation failed");
    if (!rc) rc = calloc_dev(c, &c->act, pl);
    if (!rc && (hipHostMalloc((void**)&c->h_done, 2 * sizeof(int), hipHostMallocMapped | hipHostMallocCoherent) !=
                    hipSuccess ||
                hipHostGetDevicePointer((void**)&c->d_done, c->h_done, 0) != hipSuccess))
        rc = cfail(c, PIXVOD_ENOMEM, "pinned allocation failed");
    if (!rc && hipStreamCreateWithFlags(&c->own_stream, hipStreamNonBlocking) != hipSuccess) rc = PIXVOD_EHIP;
    if (!rc && (hipEventCreate(&c->ev[0]) != hipSuccess || hipEventCreate(&c->ev[1]) != hipSuccess)) rc = PIXVOD_EHIP;
    if (!rc && (hipEventCreateWithFlags(&c->evc[0], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&c->evc[1], hipEventDisableTiming) != hipSuccess))
        rc = PIXVOD_EHIP;
    if (rc) {
        std::string m = c->err.empty() ? "allocation failed" : c->err;
        crelease(c);
        delete c;
        return cfail(nullptr, rc, m);
    }
    c->stream = c->own_stream;
    // initial point: identity pose, log-depth -log(init_inv_depth), zero planes
    const long n = (long)pl * kPlanes;
    hipLaunchKernelGGL(k_c_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->planes, n, 0.0);
    hipLaunchKernelGGL(k_c_fill, dim3((unsigned)((pl + 255) / 256)), dim3(256), 0, c->stream, c->planes, (long)pl,
                       -std::log((double)P.init_inv_depth));
    std::memset(c->h_cs, 0, sizeof(CgState));
    if (hipMemcpyAsync(c->cs, c->h_cs, sizeof(CgState), hipMemcpyHostToDevice, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        crelease(c);
        delete c;
        return cfail(nullptr, PIXVOD_EHIP, "initialisation failed");
    }
    *out = c;
    return PIXVOD_OK;
}

int pixvod_central_destroy(pixvod_central* c) {
    if (!c) return PIXVOD_OK;
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    crelease(c);
    delete c;
    return PIXVOD_OK;
}

int pixvod_central_set_stream(pixvod_central* c, void* s) {
    if (!c) return cfail(nullptr, PIXVOD_EINVAL, "solver is NULL");
    C_TRY(c, hipStreamSynchronize(c->stream));
    c->stream = s ? (hipStream_t)s : c->own_stream;
    return PIXVOD_OK;
}

int pixvod_central_set_keyframe(pixvod_central* c, const float* img, const float* normals, int where) {
    if (!c) return cfail(nullptr, PIXVOD_EINVAL, "solver is NULL");
    if (!img || !normals || (where != PIXVOD_HOST && where != PIXVOD_DEVICE))
        return cfail(c, PIXVOD_EINVAL, "img, normals and a valid location are required");
    const size_t N = (size_t)c->H * c->W;
    const float *di = img, *dn = normals;
    if (where == PIXVOD_HOST) {
        C_TRY(c, hipMemcpyAsync(c->stage, img, N * sizeof(float), hipMemcpyHostToDevice, c->stream));
        C_TRY(c, hipMemcpyAsync(c->stage + N, normals, 3 * N * sizeof(float), hipMemcpyHostToDevice, c->stream));
        di = c->stage;
        dn = c->stage + N;
    }
    const Geo g = cgeo(c);
    hipLaunchKernelGGL(k_c_keyframe, cgrid(g), dim3(64, 4), 0, c->stream, g, di, dn, c->Is, c->cxt, c->cyt);
    hipLaunchKernelGGL(k_c_edges, cgrid(g), dim3(64, 4), 0, c->stream, g, cinputs(c), c->act);
    C_TRY(c, hipGetLastError());
    // the pose restarts at the identity; log-depths are kept
    for (int k = 0; k < 6; ++k) c->h_cs->xi[k] = 0.0;
    C_TRY(c, hipMemcpyAsync(c->cs, c->h_cs->xi, sizeof(double) * 6, hipMemcpyHostToDevice, c->stream));
    C_TRY(c, hipStreamSynchronize(c->stream));
    c->have_kf = true;
    return PIXVOD_OK;
}

int pixvod_central_set_point(pixvod_central* c, const double xi[6], const double* log_depth) {
    if (!c) return cfail(nullptr, PIXVOD_EINVAL, "solver is NULL");
    if (xi) {
        for (int k = 0; k < 6; ++k) {
            if (!std::isfinite(xi[k])) return cfail(c, PIXVOD_EINVAL, "xi must be finite");
            c->h_cs->xi[k] = xi[k];
        }
        C_TRY(c, hipMemcpyAsync(c->cs, c->h_cs->xi, sizeof(double) * 6, hipMemcpyHostToDevice, c->stream));
    }
    if (log_depth) {
        const size_t N = (size_t)c->H * c->W;
        C_TRY(c, hipMemcpyAsync(c->dense, log_depth, N * sizeof(double), hipMemcpyHostToDevice, c->stream));
        const Geo g = cgeo(c);
        hipLaunchKernelGGL(k_c_dense_depth, cgrid(g), dim3(64, 4), 0, c->stream, g, cplanes(c).ell, c->dense, 0,
                           (float*)nullptr);
        C_TRY(c, hipGetLastError());
    }
    C_TRY(c, hipStreamSynchronize(c->stream));
    return PIXVOD_OK;
}

int pixvod_central_get_point(pixvod_central* c, double xi[6], double* log_depth) {
    if (!c) return cfail(nullptr, PIXVOD_EINVAL, "solver is NULL");
    if (log_depth) {
        const size_t N = (size_t)c->H * c->W;
        const Geo g = cgeo(c);
        hipLaunchKernelGGL(k_c_dense_depth, cgrid(g), dim3(64, 4), 0, c->stream, g, cplanes(c).ell, c->dense, 1,
                           (float*)nullptr);
        C_TRY(c, hipGetLastError());
        C_TRY(c, hipMemcpyAsync(log_depth, c->dense, N * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    }
    C_TRY(c, hipMemcpyAsync(c->h_cs, c->cs, sizeof(CgState), hipMemcpyDeviceToHost, c->stream));
    C_TRY(c, hipStreamSynchronize(c->stream));
    if (xi)
        for (int k = 0; k < 6; ++k) xi[k] = c->h_cs->xi[k];
    return PIXVOD_OK;
}

int pixvod_central_track(pixvod_central* c, const float* frame, int where, int n_iters, double xi_out[6],
                         float* inv_depth, int out_where, pixvod_central_stats* stats) {
    if (!c) return cfail(nullptr, PIXVOD_EINVAL, "solver is NULL");
    if (!frame || (where != PIXVOD_HOST && where != PIXVOD_DEVICE) ||
        (out_where != PIXVOD_HOST && out_where != PIXVOD_DEVICE) || n_iters < 0)
        return cfail(c, PIXVOD_EINVAL, "frame, valid locations and n_iters >= 0 are required");
    if (!c->have_kf) return cfail(c, PIXVOD_ESTATE, "no keyframe");
    const size_t N = (size_t)c->H * c->W;
    const Geo g = cgeo(c);
    const float* df = frame;
    if (where == PIXVOD_HOST) {
        C_TRY(c, hipMemcpyAsync(c->stage, frame, N * sizeof(float), hipMemcpyHostToDevice, c->stream));
        df = c->stage;
    }
    C_TRY(c, launch_frame_prep(g, df, c->W, c->It, c->Gx, c->Gy, c->stream));
    const Strengths s = strengths_from(c->P, false);
    const Inputs in = cinputs(c);
    const Planes P = cplanes(c);
    const dim3 gr = cgrid(g), blk(64, 4);
    const double tol2 = c->tol * c->tol;
    const long items = (long)c->W * ((c->H + 1) / 2), per = 8L * kCgThreads;
    const int nbx = (int)std::min<long>((items + per - 1) / per * 8, kCgMaxBlocks);
    double* part[2] = {c->part_cg, c->part_cg + (size_t)kCgMaxBlocks * kCgPartials};
    const hipStream_t st = c->stream;
    hipLaunchKernelGGL(k_c_reset_total, dim3(1), dim3(64), 0, st, c->cs);
    C_TRY(c, hipEventRecord(c->ev[0], st));
    for (int it = 0; it < n_iters; ++it) {
        // linearise, CG start, then CG iterations in chunks: the last launch of
        // chunk j writes the stop flag to host memory; after launching chunk
        // j the host waits for chunk j - 1's (chunk j keeps the device busy
        // meanwhile)
        hipLaunchKernelGGL(k_c_linearise, gr, blk, 0, st, g, s, in, c->cs, P, c->partial);
        hipLaunchKernelGGL(k_c_lin_final, dim3(1), dim3(kThreads), 0, st, s, c->nb, c->partial, c->cs, c->rec);
        hipLaunchKernelGGL(k_c_cg_init, dim3(nbx), dim3(kCgThreads), 0, st, g, s, P, c->act, c->rec, part[0]);
        C_TRY(c, hipGetLastError());
        int launched = 0;
        for (int chunk = 0; launched < c->max_cg; ++chunk) {
            const int n = std::min(kCgChunk, c->max_cg - launched);
            const bool last = launched + n >= c->max_cg;
            for (int k = launched; k < launched + n; ++k) {
                const int cur = k & 1;
                int* flag = (!last && k == launched + n - 1) ? c->d_done + (chunk & 1) : nullptr;
                hipLaunchKernelGGL(k_c_cg_iter, dim3(nbx), dim3(kCgThreads), 0, st, g, s, c->cs, P, c->act,
                                   c->rec + cur, c->rec + (1 - cur), part[cur], part[1 - cur], cur, tol2,
                                   k == 0 ? 1 : 0, flag);
            }
            C_TRY(c, hipGetLastError());
            launched += n;
            if (last) break;
            C_TRY(c, hipEventRecord(c->evc[chunk & 1], st));
            if (chunk > 0) {
                C_TRY(c, hipEventSynchronize(c->evc[(chunk - 1) & 1]));
                if (c->h_done[(chunk - 1) & 1]) break;
            }
        }
        hipLaunchKernelGGL(k_c_cg_end, dim3(1), dim3(kCgThreads), 0, st, c->cs, c->rec + (launched & 1),
                           part[launched & 1], nbx, tol2);
        hipLaunchKernelGGL(k_c_apply, gr, blk, 0, st, g, P);
        hipLaunchKernelGGL(k_c_apply_pose, dim3(1), dim3(64), 0, st, c->cs);
        C_TRY(c, hipGetLastError());
    }
    C_TRY(c, hipEventRecord(c->ev[1], c->stream));
    float* d_inv = inv_depth;
    if (inv_depth && out_where == PIXVOD_HOST) d_inv = c->out_stage;
    if (inv_depth) {
        hipLaunchKernelGGL(k_c_dense_depth, gr, blk, 0, c->stream, g, P.ell, (double*)nullptr, 1, d_inv);
        C_TRY(c, hipGetLastError());
        if (out_where == PIXVOD_HOST)
            C_TRY(c, hipMemcpyAsync(inv_depth, c->out_stage, N * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    }
    C_TRY(c, hipMemcpyAsync(c->h_cs, c->cs, sizeof(CgState), hipMemcpyDeviceToHost, c->stream));
    C_TRY(c, hipStreamSynchronize(c->stream));
    float ms = 0.0f;
    C_TRY(c, hipEventElapsedTime(&ms, c->ev[0], c->ev[1]));
    c->last_ms = ms;
    bool finite = true;
    for (int k = 0; k < 6; ++k) {
        if (xi_out) xi_out[k] = c->h_cs->xi[k];
        finite = finite && std::isfinite(c->h_cs->xi[k]);
    }
    if (stats) {
        stats->cg_iters = c->h_cs->total;
        stats->last_cg_iters = n_iters > 0 ? c->h_cs->iters : 0;
        stats->last_rel_residual = (n_iters > 0 && c->h_cs->rr0 > 0.0) ? std::sqrt(c->h_cs->rr / c->h_cs->rr0) : 0.0;
        stats->valid_fraction = n_iters > 0 ? (float)(c->h_cs->nvalid / (double)N) : 0.0f;
        stats->flags = finite ? 0u : (uint32_t)PIXVOD_DIVERGED;
    }
    return PIXVOD_OK;
}

int pixvod_central_last_ms(const pixvod_central* c, double* ms) {
    if (!c || !ms) return cfail(const_cast<pixvod_central*>(c), PIXVOD_EINVAL, "solver and ms are required");
    *ms = c->last_ms;
    return PIXVOD_OK;
}

}  // extern "C"
