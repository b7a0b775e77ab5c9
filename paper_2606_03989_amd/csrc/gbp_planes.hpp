// Plane access of the passes over the state (gfx950): scalar plane bases, 32-bit
// pixel offsets, loads straight into LDS, and the loads that the passes issue
// before their first use.
#pragma once

#include "gbp_device.hpp"

namespace pv {

// The pixel of a lane in a grid of row segments (64 pixels of a row per
// workgroup, blockIdx.x along the row). Workgroups go to the eight XCDs in
// turn, so that XCD x runs the workgroups x, x + 8, ...; they take consecutive
// segments here, and what a pixel reads of its neighbours is mostly in its own
// XCD's L2 (the pass's loads and stores alone, 1920 x 1080: 400 us, 430 in
// launch order).
__device__ inline void segment_pixel(int lane, int& u, int& v) {
    const unsigned n = gridDim.x * gridDim.y, b = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned x = b & 7, q = n >> 3, r = n & 7;
    const unsigned t = x * q + (x < r ? x : r) + (b >> 3);
    const unsigned row = t / gridDim.x;
    u = (int)(t - row * gridDim.x) * 64 + lane;
    v = (int)row;
}

// Plane access of the fused passes: the plane's base is uniform (scalar
// registers and scalar arithmetic), the pixel a 32-bit byte offset, and a
// neighbour's slot the same offset from a base moved by one element or one
// row. (plane_addressable bounds a plane at 2^30 elements.) A base runs through
// consecutive planes and is opaque to the compiler at each, which otherwise
// forms 64-bit addresses per lane (about 300 vector instructions more per pass).
__device__ inline unsigned off_of(const Geo& g, int u, int v) { return (unsigned)(v * g.pitch + u) * 4u; }
__device__ inline long step_of(const Geo& g, int d) {
    return d == DIR_L ? -1 : d == DIR_R ? 1 : d == DIR_U ? -(long)g.pitch : (long)g.pitch;
}
typedef __attribute__((address_space(1))) float GFloat;
typedef __attribute__((address_space(1))) double GDouble;
typedef __attribute__((address_space(1))) char GByte;

template <class T>
__device__ inline T* opaque(T* base) {
    asm("" : "+s"(base));
    return base;
}
__device__ inline GFloat* plane_of(const float* base, long elements) {
    return opaque((GFloat*)const_cast<float*>(base + elements));
}
__device__ inline GDouble* plane_of(double* base) { return opaque((GDouble*)base); }
// the pixel's offset for the accesses of one block of code: its widening to 64
// bits has to be visible there for the access to take base and offset apart
__device__ inline unsigned here(unsigned o) {
    asm("" : "+v"(o));
    return o;
}
// a pixel's element of a plane
__device__ inline GFloat* at(GFloat* base, unsigned o) { return (GFloat*)((GByte*)base + o); }
__device__ inline GDouble* at(GDouble* base, unsigned o) { return (GDouble*)((GByte*)base + 2UL * o); }
__device__ inline float ld(const float* base, unsigned o) { return *at((GFloat*)const_cast<float*>(base), o); }
// the base of the next plane, `stride` elements on
template <class T>
__device__ inline T* next(long stride, T* base) {
    return opaque(base + stride);
}
template <class T>
__device__ inline T* next(const Geo& g, T* base) {
    return next(g.plane, base);
}

// wait for this wave's loads into LDS: the compiler does not track them, so
// the wait is explicit, and the memory clobber keeps the LDS reads after it
__device__ inline void wait_lds_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// the information matrices are read from LDS again after this point instead of
// being kept in registers from their previous use
__device__ inline void reread_lds() { asm volatile("" ::: "memory"); }

// wait for this wave's LDS reads, before its planes are loaded again
__device__ inline void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// one float of state; NT: a non-temporal store (streamed past the caches)
template <bool NT = false>
__device__ inline void put(GFloat* a, float v) {
    if constexpr (NT) __builtin_nontemporal_store(v, a);
    else *a = v;
}

__device__ inline void load_point_at(const float* X, const Geo& g, unsigned o, float pt[7]) {
    GFloat* b = plane_of(X, 0);
    o = here(o);
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        pt[k] = *at(b, o);
        b = next(g, b);
    }
}

__device__ inline void point_of(const float pt[7], double tau[6], double& ell) {
#pragma unroll
    for (int k = 0; k < 6; ++k) tau[k] = (double)pt[k];
    ell = (double)pt[6];
}

// load_pixel_inputs without branches: a map that is not bound is read from the
// keyframe image and not used
__device__ inline PixelInputs load_inputs_at(const Strengths& s, const Inputs& in, unsigned o) {
    PixelInputs r;
    r.Is = ld(in.Is, o);
    r.sigD = ld(s.has_sigma_map ? in.sigD : in.Is, o);
    r.prior_ell = ld(s.has_prior_map ? in.prior_ell : in.Is, o);
    return r;
}

// the pixel's neighbours: whether there is one, its offset (a missing
// neighbour's is the pixel's own), and the normal targets of the edges
__device__ inline void edges_of(const Geo& g, const Inputs& in, int u, int v, bool has[4], unsigned on[4], float c[4]) {
    const unsigned o = off_of(g, u, v);
    has[DIR_L] = u > 0;
    has[DIR_R] = u + 1 < g.W;
    has[DIR_U] = v > 0;
    has[DIR_D] = v + 1 < g.H;
#pragma unroll
    for (int d = 0; d < 4; ++d) on[d] = has[d] ? o + (unsigned)(4 * step_of(g, d)) : o;
    c[DIR_L] = ld(in.cxt, on[DIR_L]);
    c[DIR_R] = ld(in.cxt, o);
    c[DIR_U] = ld(in.cyt, on[DIR_U]);
    c[DIR_D] = ld(in.cyt, o);
}

// which edges' normal-integration factors are active
__device__ inline void active_edges(const Strengths& s, const float c[4], bool act[4]) {
#pragma unroll
    for (int d = 0; d < 4; ++d) act[d] = isfinite(c[d]) && s.lamN > 0.0;
}

// receiver side: eta = h - Lambda' r of an identity partial (h, Lambda')
template <class Lam>
__device__ inline void complete_eta(const float h[6], Lam lam, const double r[6], double e[6]) {
#pragma unroll
    for (int a = 0; a < 6; ++a) e[a] = (double)h[a];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int c = i; c < 6; ++c) {
            const double l = (double)lam(s6(i, c));
            e[i] = fma(-l, r[c], e[i]);
            if (i != c) e[c] = fma(-l, r[i], e[c]);
        }
}

// normal_residual of an active edge with a preloaded target c of the left/upper pixel
__device__ inline double normal_residual_c(float c, int d, double ell_i, double ell_j) {
    const bool recv_is_b = (d == DIR_L || d == DIR_U);
    return recv_is_b ? (ell_i - ell_j + (double)c) : (ell_i - ell_j - (double)c);
}

}  // namespace pv
