// rows.h -- the stencil passes' view of a wavefront: 64 (or, with V slots a
// lane, 64 V) consecutive slots of one row (j, k), so that everything but the x
// position is uniform.
//
// What a pass spends beside its bytes is instructions: with per-lane rows,
// slab tests and 64-bit psi addresses the float32 E pass of a 512 x 256 x 128
// grid issued 196 vector and 266 scalar instructions a wavefront, 60 % of the
// vector and 78 % of the (per-CU) scalar issue slots of its time.  Here rows,
// planes and the y and z slabs are scalar, an address is a scalar base and one
// 32-bit lane offset, and the recursion coefficients of y and z slabs come
// through the scalar cache: 80 and 138 instructions, 35 registers instead of
// 70; 146 -> 131 us (5.3 TB/s of the pass's own bytes; a copy reaches 5.1), and
// 121 with the tiles and coefficients of passes.hip.  Smaller grids, whose
// fields stay in the last-level cache, gain more: a batch of 32 resonators E
// 330 -> 215 us, H/M 279 -> 226; 211 x 109 x 77 float64 47 -> 34 and 44 -> 35 us.
#pragma once

#include "device_common.h"

namespace mpx {

// the wavefront's row of a TX x TY tile (bx, by) of plane k
struct RowPos {
    int i;      // the lane's (first) x position (may lie past the row)
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

// the wavefront's row when a lane holds V consecutive slots: blocks of 64 x 4
// threads, WX wavefronts side by side in x and 4 / WX rows
template <int V, int WX>
__device__ __forceinline__ RowPos row_pos_v(const int *n, int bx, int by, int k) {
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    RowPos r;
    r.w0 = (bx * WX + w % WX) * 64 * V;
    r.i = r.w0 + (int)threadIdx.x * V;
    r.j = by * (4 / WX) + w / WX;
    r.k = k;
    r.in = r.i < n[0];
    return r;
}

// V consecutive elements (aligned to their size) `off` bytes past a base
template <int V, bool NT = false, typename T>
__device__ __forceinline__ void row_ldv(const T *base, unsigned off, T (&o)[V]) {
    if constexpr (V == 1) {
        o[0] = row_ld<NT>(base, off);
    } else {
        typedef T vec __attribute__((ext_vector_type(V)));
        const vec *a = (const vec *)((const char *)base + off);
        const vec x = NT ? __builtin_nontemporal_load(a) : *a;
#pragma unroll
        for (int v = 0; v < V; v++) o[v] = x[v];
    }
}
// those of them with st[v]: one store where all of a lane's are
template <int V, bool NT = false, typename T>
__device__ __forceinline__ void row_stv(T *base, unsigned off, const T (&o)[V], const bool (&st)[V]) {
    if constexpr (V == 1) {
        if (st[0]) row_st<NT>(base, off, o[0]);
    } else {
        typedef T vec __attribute__((ext_vector_type(V)));
        bool all = true;
        vec x;
#pragma unroll
        for (int v = 0; v < V; v++) {
            all = all && st[v];
            x[v] = o[v];
        }
        if (all) {
            vec *a = (vec *)((char *)base + off);
            if (NT)
                __builtin_nontemporal_store(x, a);
            else
                *a = x;
        } else {
#pragma unroll
            for (int v = 0; v < V; v++)
                if (st[v]) row_st<NT>(base, off + (unsigned)(v * (int)sizeof(T)), o[v]);
        }
    }
}

// a kernel's first argument once more, from its argument segment: what is read
// through it is read from here on.  Arguments named plainly are all fetched at
// the kernel's start, and those of its last part, past the scalar registers,
// then go to vector lanes and come back one instruction each.
template <typename P>
__device__ __forceinline__ const P &args_again() {
    typedef __attribute__((address_space(4))) const char cbyte;
    cbyte *q = (cbyte *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return *(const P *)q;
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
template <typename T, int V = 1>
struct RowPml {
    bool wx = false, wy = false, wz = false; // uniform: the wavefront has slab slots of this axis
    bool sx[V] = {};                         // the slot lies in an x slab
    T bx[V] = {}, cx[V] = {}, by = T(0), cy = T(0), bz = T(0), cz = T(0);
    T xy[V] = {}, xz[V] = {}; // psi along x of the y and z components
    T yz[V] = {}, yx[V] = {}; // along y of the z and x components
    T zx[V] = {}, zy[V] = {}; // along z of the x and y components
    unsigned ox[V] = {};      // byte offset of the slot's x-slab value in its row
};

// uniform first element of the row's psi along axis w (row counts fit 32 bits)
template <typename T>
__device__ __forceinline__ long long row_psi(const KParams<T> &p, int w, int j, int k) {
    const int S = p.nlo[w] + p.nhi[w];
    unsigned row;
    if (w == 0) {
        row = (unsigned)j + (unsigned)p.n[1] * (unsigned)k;
    } else if (w == 1) {
        const int sp = j < p.nlo[1] ? j : p.nlo[1] + (j - (p.n[1] - p.nhi[1]));
        row = (unsigned)sp + (unsigned)S * (unsigned)k;
    } else {
        const int sp = k < p.nlo[2] ? k : p.nlo[2] + (k - (p.n[2] - p.nhi[2]));
        row = (unsigned)j + (unsigned)p.n[1] * (unsigned)sp;
    }
    return (long long)((unsigned long long)(unsigned)(w == 0 ? S : p.px) * row);
}

template <typename T>
__device__ __forceinline__ bool in_slab(const KParams<T> &p, int w, int q) {
    return q < p.nlo[w] || q >= p.n[w] - p.nhi[w];
}

// io: the lane's byte offset in a padded row (its x position clamped to the row)
template <typename T, bool E, int V = 1>
__device__ __forceinline__ RowPml<T, V> row_pml(const KParams<T> &p, const RowPos &r, unsigned io) {
    RowPml<T, V> m;
    T *const(*a)[3] = E ? p.psiE : p.psiH;
    const T *const *bt = E ? p.bE : p.bH;
    const T *const *ct = E ? p.cE : p.cH;
    m.wx = r.w0 < p.nlo[0] || r.w0 + 64 * V - 1 >= p.n[0] - p.nhi[0];
    if (p.nlo[0] + p.nhi[0] == 0) m.wx = false;
    m.wy = in_slab(p, 1, r.j);
    m.wz = in_slab(p, 2, r.k);
    if (m.wx) {
        const long long q = row_psi(p, 0, r.j, r.k);
#pragma unroll
        for (int v = 0; v < V; v++) {
            const int i = r.i + v;
            m.sx[v] = i < p.n[0] && in_slab(p, 0, i);
            const int sp = i < p.nlo[0] ? i : p.nlo[0] + (i - (p.n[0] - p.nhi[0]));
            m.ox[v] = (unsigned)(m.sx[v] ? sp : 0) * (unsigned)sizeof(T);
            m.xy[v] = row_ld(a[1][0] + q, m.ox[v]);
            m.xz[v] = row_ld(a[2][0] + q, m.ox[v]);
            // (of the lane's slots past the row: its first one's, unused)
            const unsigned ib = i < p.n[0] ? io + (unsigned)(v * (int)sizeof(T)) : io;
            m.bx[v] = row_ld(bt[0], ib);
            m.cx[v] = row_ld(ct[0], ib);
        }
    }
    if (m.wy) {
        const long long q = row_psi(p, 1, r.j, r.k);
        row_ldv<V, true>(a[2][1] + q, io, m.yz);
        row_ldv<V, true>(a[0][1] + q, io, m.yx);
        m.by = scalar_ld(bt[1], r.j);
        m.cy = scalar_ld(ct[1], r.j);
    }
    if (m.wz) {
        const long long q = row_psi(p, 2, r.j, r.k);
        row_ldv<V, true>(a[0][2] + q, io, m.zx);
        row_ldv<V, true>(a[1][2] + q, io, m.zy);
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
