// rows.h -- the stencil passes' view of a wavefront: 64 consecutive slots of
// one row (j, k), so that everything but the x position is uniform.
//
// What a pass spends beside its bytes is instructions: with per-lane rows,
// slab tests and 64-bit psi addresses the float32 E pass of a 512 x 256 x 128
// grid issued 196 vector and 266 scalar instructions a wavefront, 60 % of the
// vector and 78 % of the (per-CU) scalar issue slots of its time.  Here rows,
// planes and the y and z slabs are scalar, an address is a scalar base and one
// 32-bit lane offset, and the recursion coefficients of y and z slabs come
// through the scalar cache: 72 and 171 instructions, 34 registers instead of
// 70, 146 -> 131 us (5.3 TB/s of the pass's own bytes; a copy reaches 5.1).
// Smaller grids, whose fields stay in the last-level cache, gain more: a batch
// of 32 resonators E 330 -> 239 us, H/M 279 -> 249; 211 x 109 x 77 float64 47 ->
// 40 and 44 -> 38 us.
#pragma once

#include "device_common.h"

namespace mpx {

// the wavefront's row of a TX x TY tile (bx, by) of plane k
struct RowPos {
    int i;      // the lane's x position (may lie past the row)
    int w0;     // the wavefront's first x position
    int j, k;   // its row
    bool in;    // i lies in the row
};

template <int TX>
__device__ __forceinline__ RowPos row_pos(const int *n, int bx, int by, int ty, int k) {
    RowPos r;
    const int tx = (int)threadIdx.x;
    r.w0 = bx * TX + (TX == 64 ? 0 : (__builtin_amdgcn_readfirstlane(tx) & ~63));
    r.i = r.w0 + (tx & 63);
    r.j = by * ty + (ty > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.y) : 0);
    r.k = k;
    r.in = r.i < n[0];
    return r;
}

// element `off` bytes past a uniform base; NT: with the non-temporal hint
template <bool NT = false, typename T>
__device__ __forceinline__ T row_ld(const T *base, unsigned off) {
    const T *a = (const T *)((const char *)base + off);
    return NT ? __builtin_nontemporal_load(a) : *a;
}
template <bool NT = false, typename T>
__device__ __forceinline__ void row_st(T *base, unsigned off, T v) {
    T *a = (T *)((char *)base + off);
    if (NT)
        __builtin_nontemporal_store(v, a);
    else
        *a = v;
}

// a uniform element of a read-only table, through the scalar cache
template <typename T>
__device__ __forceinline__ T scalar_ld(const T *tab, int q) {
    typedef __attribute__((address_space(4))) const T ct;
    return ((ct *)tab)[q];
}

// ---------------------------------------------------------------------------
// the CPML state of a wavefront's slots for one kind of psi (E edges or H
// faces): per axis whether it has slab slots, the recursion's b and c, and the
// psi of the two components that differentiate along it.  One load per array
// and lane, all before any use; y and z slabs are touched once per pass
// (non-temporal), a row's few x-slab values share cache lines with the next
// row's (default policy).
// ---------------------------------------------------------------------------
template <typename T>
struct RowPml {
    bool wx = false, wy = false, wz = false; // uniform: the wavefront has slab slots of this axis
    bool sx = false;                         // the lane lies in an x slab
    T bx = T(0), cx = T(0), by = T(0), cy = T(0), bz = T(0), cz = T(0);
    T xy = T(0), xz = T(0); // psi along x of the y and z components
    T yz = T(0), yx = T(0); // along y of the z and x components
    T zx = T(0), zy = T(0); // along z of the x and y components
    unsigned ox = 0;        // byte offset of the lane's x-slab value in its row
};

// uniform first element of the row's psi along axis w
template <typename T>
__device__ __forceinline__ long long row_psi(const KParams<T> &p, int w, int j, int k) {
    const int S = p.nlo[w] + p.nhi[w];
    if (w == 0) return (long long)S * ((long long)j + (long long)p.n[1] * k);
    if (w == 1) {
        const int sp = j < p.nlo[1] ? j : p.nlo[1] + (j - (p.n[1] - p.nhi[1]));
        return (long long)p.px * ((long long)sp + (long long)S * k);
    }
    const int sp = k < p.nlo[2] ? k : p.nlo[2] + (k - (p.n[2] - p.nhi[2]));
    return (long long)p.px * ((long long)j + (long long)p.n[1] * sp);
}

template <typename T>
__device__ __forceinline__ bool in_slab(const KParams<T> &p, int w, int q) {
    return q < p.nlo[w] || q >= p.n[w] - p.nhi[w];
}

// io: the lane's byte offset in a padded row (its x position clamped to the row)
template <typename T, bool E>
__device__ __forceinline__ RowPml<T> row_pml(const KParams<T> &p, const RowPos &r, unsigned io) {
    RowPml<T> m;
    T *const(*a)[3] = E ? p.psiE : p.psiH;
    const T *const *bt = E ? p.bE : p.bH;
    const T *const *ct = E ? p.cE : p.cH;
    m.wx = r.w0 < p.nlo[0] || r.w0 + 63 >= p.n[0] - p.nhi[0];
    if (p.nlo[0] + p.nhi[0] == 0) m.wx = false;
    m.wy = in_slab(p, 1, r.j);
    m.wz = in_slab(p, 2, r.k);
    if (m.wx) {
        m.sx = r.in && in_slab(p, 0, r.i);
        const int sp = r.i < p.nlo[0] ? r.i : p.nlo[0] + (r.i - (p.n[0] - p.nhi[0]));
        m.ox = (unsigned)(m.sx ? sp : 0) * (unsigned)sizeof(T);
        const long long q = row_psi(p, 0, r.j, r.k);
        m.xy = row_ld(a[1][0] + q, m.ox);
        m.xz = row_ld(a[2][0] + q, m.ox);
        m.bx = row_ld(bt[0], io);
        m.cx = row_ld(ct[0], io);
    }
    if (m.wy) {
        const long long q = row_psi(p, 1, r.j, r.k);
        m.yz = row_ld<true>(a[2][1] + q, io);
        m.yx = row_ld<true>(a[0][1] + q, io);
        m.by = scalar_ld(bt[1], r.j);
        m.cy = scalar_ld(ct[1], r.j);
    }
    if (m.wz) {
        const long long q = row_psi(p, 2, r.j, r.k);
        m.zx = row_ld<true>(a[0][2] + q, io);
        m.zy = row_ld<true>(a[1][2] + q, io);
        m.bz = scalar_ld(bt[2], r.k);
        m.cz = scalar_ld(ct[2], r.k);
    }
    return m;
}

// one recursion step of a slab slot: psi <- b psi + c d, d <- d + psi
template <typename T>
__device__ __forceinline__ void pml_step(T &psi, T b, T c, T &d) {
    psi = b * psi + c * d;
    d += psi;
}
// the same for the lanes of an x slab (the others keep psi and d)
template <typename T>
__device__ __forceinline__ void pml_step_if(bool s, T &psi, T b, T c, T &d) {
    T q = psi, e = d;
    pml_step(q, b, c, e);
    psi = s ? q : psi;
    d = s ? e : d;
}

} // namespace mpx
