// passes.hip -- the separate-pass schedule: an E pass, then an H/M pass, each
// in place with one or two slots a thread (blocks of 256 threads on one plane).
// Also the bracket half steps of every schedule (an H/M pass with one half
// step) and the E pass of a call's last step.
//
// Scheme (arXiv:2510.22221, Methods, "Numerical Model"): the E update that
// follows eq. iterate_H, and eq. iterate_H with M = 0 for non-magnetic faces
// (the magnetic ones are the film kernels' work).
//
// Memory access: a wavefront is 64 or 128 slots of one row (rows.h), so every array
// is read at its own base and a 32-bit lane offset (arrays of 4 GiB and more:
// at the plane's base); rows, slabs and their coefficients are scalar.  With a
// 64-bit plane base per array, and 64-bit tile and psi indices, the float32 E
// pass of a 512 x 256 x 128 grid issued 196 scalar instructions a wavefront,
// now 138: 128 x 64 x 64 8.4 -> 7.2 us (H/M 8.8 -> 7.2), a batch of 32
// resonators 225 -> 215 (239 -> 226).  One path serves interior and boundary.
// Per-tile source / film flags come from a host table (one per tile shape);
// edge coefficients come from the packed row of the slot's class (its six
// values in one or two 16-byte loads; no per-block staging).
#include "film.h"
#include "rows.h"
#include "stencil.h"

namespace mpx {

constexpr int PTX = kPassTX, PTY = kPassTY;

// ---------------------------------------------------------------------------
// E pass: E_c <- ca E_c + cb ((curl H)_c - J_c) on the three edges of slot
// (i, j, k); reads H at the slot and at its -x, -y, -z neighbours.  One path
// for every tile: a -1 neighbour wraps on a periodic axis and is, at a wall,
// any in-range value (only edges held at zero would read it); lanes past the
// domain (partial tiles) compute nothing that is stored.  Each edge takes its
// coefficients from the table entry of its slot's class and component (a
// material, or a compound class of a slot whose eight cells differ); on a
// grid with more distinct triples than the class byte holds (XC) the slot's
// 16-bit class also reaches the extended table's rows.  A slot on the mixed
// list (class byte 255, or 16-bit class 0xffff) is skipped and updated
// afterwards by the mixed-slot kernel from the same old values.
// ---------------------------------------------------------------------------
// the current of the sources on the edge of component C at (i, j, k)
template <typename T>
__device__ __forceinline__ double src_current(const KParams<T> &p, int C, int i, int j, int k, long long step) {
    double J = 0.0;
    for (int s = 0; s < p.nsrc; s++) {
        const SrcDev &S = p.srcs[s]; // device copy: no dynamic index into the kernel argument
        if (S.comp != C) continue;
        if (i < S.box[0] || i >= S.box[0] + S.box[3] || j < S.box[1] || j >= S.box[1] + S.box[4] || k < S.box[2] ||
            k >= S.box[2] + S.box[5])
            continue;
        if (step < S.n) J += S.table[step];
    }
    return J;
}

// TAPE: E^n and the curl input x^n = (d1 + psi1') - (d2 + psi2') - J^n of the
// slots of an eps box go to the adjoint's tape as well (the pass holds both
// anyway; a launch of its own took 4.6 us a step on a 128 x 64 x 64 grid).
// CLS: the slot class read, 0 the class byte, 1 the 16-bit class (a grid
// with extended triples), 2 whichever the instance has (batch members of one
// launch differ; the test is uniform over a member's lanes).  f: the tile's
// flag byte, first used after every field load has been issued (so that the
// loads do not wait for it).
template <typename T, int CLS, int V, bool BIG, bool TAPE = false>
__device__ __forceinline__ void epass_row(const KParams<T> &p, const RowPos &r, int f, const BoxTape &bt = BoxTape()) {
    if (r.j >= p.n[1]) return; // a partial tile's row (uniform)
    const unsigned es = (unsigned)sizeof(T);
    // the lane's first slot, clamped to the row's last whole or partial group
    const int ic = min(r.i, (p.n[0] - 1) & -V), j = r.j, k = r.k;
    // an array below 4 GiB: bases are the kernel's arguments, the plane is in
    // the lanes' 32-bit offsets; else (BIG) bases are the plane's
    const unsigned plane = (unsigned)p.px * (unsigned)p.n[1], rowb = (unsigned)p.px * es;
    const unsigned io = (unsigned)ic * es, po = BIG ? 0u : (unsigned)k * plane * es, vo = io + (po + (unsigned)j * rowb);
    const long long zo = BIG ? (long long)((unsigned long long)plane * (unsigned)k) : 0;
    // the -1 neighbours: wrapped on a periodic axis, any in-range value at a wall
    const unsigned vxm = ic > 0 ? vo - es : (p.per[0] ? vo + (unsigned)(p.n[0] - 1) * es : vo);
    const unsigned jm = (unsigned)(j > 0 ? j - 1 : (p.per[1] ? p.n[1] - 1 : j)), vym = io + (po + jm * rowb);
    const unsigned kb = (unsigned)(k > 0 ? k - 1 : (p.per[2] ? p.n[2] - 1 : k));
    const unsigned vzm = BIG ? vo : io + (kb * plane * es + (unsigned)j * rowb);
    const long long zb = BIG ? (long long)((unsigned long long)plane * kb) : 0;
    // the class first: its coefficient row is the one load that waits for another
    bool c16 = CLS == 1;
    if constexpr (CLS == 2) c16 = p.cls16 != nullptr;
    int c0[V];
    {
        const unsigned vc = (unsigned)ic + ((BIG ? 0u : (unsigned)k * plane) + (unsigned)j * (unsigned)p.px);
        if (c16) {
            uint16_t c[V];
            row_ldv<V, CLS != 2>(p.cls16 + zo, 2u * vc, c);
#pragma unroll
            for (int v = 0; v < V; v++) c0[v] = c[v];
        } else {
            uint8_t c[V];
            row_ldv<V, CLS != 2>(p.cls + zo, vc, c);
#pragma unroll
            for (int v = 0; v < V; v++) c0[v] = c[v];
        }
    }
    const T *Hx = p.H[0] + zo, *Hy = p.H[1] + zo, *Hz = p.H[2] + zo;
    // the -z plane's H is read here for the last time (the tiles of its own
    // plane and of the next row read it before): non-temporal
    T hx0[V], hx_km[V], hx_ym[V], hy0[V], hy_km[V], hy_xm[V], hz0[V], hz_xm[V], hz_ym[V];
    row_ldv<V>(Hx, vo, hx0);
    row_ldv<V, true>(p.H[0] + zb, vzm, hx_km);
    row_ldv<V>(Hx, vym, hx_ym);
    row_ldv<V>(Hy, vo, hy0);
    row_ldv<V, true>(p.H[1] + zb, vzm, hy_km);
    hy_xm[0] = row_ld(Hy, vxm);
    row_ldv<V>(Hz, vo, hz0);
    hz_xm[0] = row_ld(Hz, vxm);
    row_ldv<V>(Hz, vym, hz_ym);
    // E, the class and the new E are touched once per pass: non-temporal, so
    // that they leave L2 first and the H rows and planes the neighbouring
    // tiles read again, and the coefficient rows, stay
    T *Ex = p.E[0] + zo, *Ey = p.E[1] + zo, *Ez = p.E[2] + zo;
    T e0[V], e1[V], e2[V];
    row_ldv<V, true>(Ex, vo, e0);
    row_ldv<V, true>(Ey, vo, e1);
    row_ldv<V, true>(Ez, vo, e2);
    RowPml<T, V> m = row_pml<T, true, V>(p, r, io);
    // the slots' six coefficients in one or two wide loads (a slot on the
    // mixed list, class byte 255 or 16-bit class 0xffff, reads row 0 and uses
    // none)
    const int kSkip = c16 ? 0xffff : kMixed;
#pragma unroll
    for (int v = 1; v < V; v++)
        if (ic + v >= p.n[0]) c0[v] = kSkip; // past the row: no class there
    CoefRow<T> L[V];
    // one class for the whole wavefront (most are inside one material): its
    // row comes through the scalar cache, not as a gather of 24 (48) bytes a
    // lane.  E pass, 512 x 256 x 128 float32 128 -> 122 us, 211 x 109 x 77
    // float64 40.9 -> 37.4; a layout with a class for every block of cells, so
    // many that it needs 16 bits, only pays for the test (866 -> 871)
    const int cu = __builtin_amdgcn_readfirstlane(c0[0]);
    bool same = true;
#pragma unroll
    for (int v = 0; v < V; v++) same = same && (c0[v] == cu || (v > 0 && ic + v >= p.n[0]));
    if (CLS != 1 && __builtin_amdgcn_ballot_w64(!same) == 0) {
        const T *q = p.coefv + kCoefRow<T> * (long long)(cu == kSkip ? 0 : cu);
        CoefRow<T> S;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            S.ca[c] = scalar_ld(q, 2 * c);
            S.cb[c] = scalar_ld(q, 2 * c + 1);
        }
#pragma unroll
        for (int v = 0; v < V; v++) L[v] = S;
    } else {
#pragma unroll
        for (int v = 0; v < V; v++) L[v] = coef_row<T>(p.coefv, c0[v] == kSkip ? 0 : c0[v]);
    }
#pragma unroll
    for (int v = 1; v < V; v++) {
        hy_xm[v] = hy0[v - 1];
        hz_xm[v] = hz0[v - 1];
    }
    const T dx = p.dT[0], dy = p.dT[1], dz = p.dT[2], ix = p.invd[0], iy = p.invd[1], iz = p.invd[2];
    // an edge on a lower wall (an axis other than its own) or on a conductor
    // (cb = 0) stays zero and keeps its psi
    const bool oy = j > 0 || p.per[1], oz = k > 0 || p.per[2];
    bool s0[V], s1[V], s2[V], ok[V]; // the edge's psi moves; the slot is stored
    T n0[V], n1[V], n2[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        // E_x: along y then z; E_y: z, x; E_z: x, y
        T ay = dif(hz0[v], hz_ym[v], dy, iy), az = dif(hy0[v], hy_km[v], dz, iz);
        T bz = dif(hx0[v], hx_km[v], dz, iz), bx = dif(hz0[v], hz_xm[v], dx, ix);
        T cx = dif(hy0[v], hy_xm[v], dx, ix), cy = dif(hx0[v], hx_ym[v], dy, iy);
        const bool ox = r.i + v > 0 || p.per[0];
        const bool u0 = oy && oz && L[v].cb[0] != T(0), u1 = ox && oz && L[v].cb[1] != T(0),
                   u2 = ox && oy && L[v].cb[2] != T(0);
        if (m.wx) {
            pml_step_if(m.sx[v], m.xy[v], m.bx[v], m.cx[v], bx);
            pml_step_if(m.sx[v], m.xz[v], m.bx[v], m.cx[v], cx);
        }
        if (m.wy) {
            pml_step(m.yx[v], m.by, m.cy, ay);
            pml_step(m.yz[v], m.by, m.cy, cy);
        }
        if (m.wz) {
            pml_step(m.zx[v], m.bz, m.cz, az);
            pml_step(m.zy[v], m.bz, m.cz, bz);
        }
        T x0 = ay - az, x1 = bz - bx, x2 = cx - cy;
        double xt[3] = {(double)x0, (double)x1, (double)x2}; // TAPE
        (void)xt;
        if (f & 2) {
            const long long step = p.step[0];
            // (x - 0) is x bitwise, so subtracting only here matches the plain form
            const double J0 = src_current(p, 0, r.i + v, j, k, step), J1 = src_current(p, 1, r.i + v, j, k, step),
                         J2 = src_current(p, 2, r.i + v, j, k, step);
            if constexpr (TAPE) {
                xt[0] = (double)x0 - J0;
                xt[1] = (double)x1 - J1;
                xt[2] = (double)x2 - J2;
            }
            x0 = x0 - T(J0);
            x1 = x1 - T(J1);
            x2 = x2 - T(J2);
        }
        ok[v] = r.i + v < p.n[0] && c0[v] != kSkip;
        if constexpr (TAPE) {
            const int rb[3] = {bt.size[0] + 1, bt.size[1] + 1, bt.size[2] + 1};
            int lj = j - bt.b0[1], lk = k - bt.b0[2], li = r.i + v - bt.b0[0];
            if (lj < 0 && p.per[1]) lj += p.n[1];
            if (lk < 0 && p.per[2]) lk += p.n[2];
            if (lj >= 0 && lj < rb[1] && lk >= 0 && lk < rb[2]) { // uniform
                if (li < 0 && p.per[0]) li += p.n[0];
                if (r.i + v < p.n[0] && li >= 0 && li < rb[0]) {
                    const long long tb = (long long)rb[0] * rb[1] * rb[2];
                    double *d = bt.dst + li + (long long)rb[0] * ((long long)lj + (long long)rb[1] * lk);
                    d[0] = (double)e0[v];
                    d[tb] = (double)e1[v];
                    d[2 * tb] = (double)e2[v];
                    d[3 * tb] = xt[0];
                    d[4 * tb] = xt[1];
                    d[5 * tb] = xt[2];
                }
            }
        }
        n0[v] = u0 ? L[v].ca[0] * e0[v] + L[v].cb[0] * x0 : T(0);
        n1[v] = u1 ? L[v].ca[1] * e1[v] + L[v].cb[1] * x1 : T(0);
        n2[v] = u2 ? L[v].ca[2] * e2[v] + L[v].cb[2] * x2 : T(0);
        s0[v] = ok[v] && u0;
        s1[v] = ok[v] && u1;
        s2[v] = ok[v] && u2;
    }
    row_stv<V, true>(Ex, vo, n0, ok);
    row_stv<V, true>(Ey, vo, n1, ok);
    row_stv<V, true>(Ez, vo, n2, ok);
    if (m.wx) {
        const long long q = row_psi(p, 0, j, k);
#pragma unroll
        for (int v = 0; v < V; v++)
            if (m.sx[v]) {
                if (s1[v]) row_st(p.psiE[1][0] + q, m.ox[v], m.xy[v]);
                if (s2[v]) row_st(p.psiE[2][0] + q, m.ox[v], m.xz[v]);
            }
    }
    if (m.wy) {
        const long long q = row_psi(p, 1, j, k);
        row_stv<V, true>(p.psiE[0][1] + q, io, m.yx, s0);
        row_stv<V, true>(p.psiE[2][1] + q, io, m.yz, s2);
    }
    if (m.wz) {
        const long long q = row_psi(p, 2, j, k);
        row_stv<V, true>(p.psiE[0][2] + q, io, m.zx, s0);
        row_stv<V, true>(p.psiE[1][2] + q, io, m.zy, s1);
    }
}

// the flags of a wavefront's row: those of its tiles (one of 256 x 1 slots on
// a wide grid, else V of 64 x 4), read through the scalar cache (the aligned
// word that holds each; the tables are whole words): a vector load here would
// put the field loads behind its wait, since the vector memory counter
// completes in order.  A row past the grid (of a partial block) reads the last
// row's tile.
template <typename T, int V>
__device__ __forceinline__ int row_flags(const KParams<T> &p, const RowPos &r, bool wide) {
    typedef __attribute__((address_space(4))) const uint32_t cword;
    const unsigned tx = wide ? kWideTX : PTX, ty = wide ? kWideTY : PTY;
    const unsigned nxt = ((unsigned)p.n[0] + tx - 1) / tx, nyt = ((unsigned)p.n[1] + ty - 1) / ty;
    const cword *tab = (cword *)(wide ? p.pflags_w : p.pflags);
    const unsigned bx = (unsigned)r.w0 / tx, t0 = bx + nxt * ((unsigned)min(r.j, p.n[1] - 1) / ty + nyt * (unsigned)r.k);
    int f = 0;
#pragma unroll
    for (unsigned v = 0; v < (unsigned)V; v++) {
        const unsigned ti = v == 0 || bx + v < nxt ? t0 + v : t0;
        f |= (int)(tab[ti >> 2] >> (8 * (ti & 3)));
        if (wide) break;
    }
    return f & 0xff;
}

// a block of 64 x 4 threads: 64 V WX x 4 / WX slots (bx, by) of plane k
template <typename T, int CLS, int V, int WX, bool WIDE, bool BIG, bool TAPE = false>
__device__ __forceinline__ void epass_block(const KParams<T> &p, int bx, int by, int k,
                                            const BoxTape &bt = BoxTape()) {
    const RowPos r = row_pos_v<V, WX>(p.n, bx, by, k);
    if (r.w0 >= p.n[0]) return; // uniform: a wavefront past the row
    epass_row<T, CLS, V, BIG, TAPE>(p, r, row_flags<T, V>(p, r, WIDE), bt);
}

// the mixed slots, one thread each: the general path (folded loads; edge
// coefficients from the slot's entry of the extended table, or else from the
// four cell ids), in place after the E pass
template <typename T, bool MIXED>
__device__ __forceinline__ void emixed_apply(const KParams<T> &p, const CoefMem<T> &L, int4 s, int cls) {
    const int i = s.x, j = s.y, k = s.z;
    const T hx0 = ldz(p, p.H[0], i, j, k), hx_km = ldz(p, p.H[0], i, j, k - 1), hx_ym = ldz(p, p.H[0], i, j - 1, k);
    const T hy0 = ldz(p, p.H[1], i, j, k), hy_km = ldz(p, p.H[1], i, j, k - 1), hy_xm = ldz(p, p.H[1], i - 1, j, k);
    const T hz0 = ldz(p, p.H[2], i, j, k), hz_xm = ldz(p, p.H[2], i - 1, j, k), hz_ym = ldz(p, p.H[2], i, j - 1, k);
    const long long q = p.slot(i, j, k);
    const bool tpml = true, tsrc = p.nsrc > 0;
    const long long step = tsrc ? p.step[0] : 0;
    const T dx = p.dT[0], dy = p.dT[1], dz = p.dT[2], ix = p.invd[0], iy = p.invd[1], iz = p.invd[2];
    const T e0 = p.E[0][q], e1 = p.E[1][q], e2 = p.E[2][q];
    const T n0 = e_upd<T, 0, true, true, CoefMem<T>, MIXED>(p, L, i, j, k, cls, e0, dif(hz0, hz_ym, dy, iy),
                                                          dif(hy0, hy_km, dz, iz), tpml, tsrc, step, true);
    const T n1 = e_upd<T, 1, true, true, CoefMem<T>, MIXED>(p, L, i, j, k, cls, e1, dif(hx0, hx_km, dz, iz),
                                                          dif(hz0, hz_xm, dx, ix), tpml, tsrc, step, true);
    const T n2 = e_upd<T, 2, true, true, CoefMem<T>, MIXED>(p, L, i, j, k, cls, e2, dif(hy0, hy_xm, dx, ix),
                                                          dif(hx0, hx_ym, dy, iy), tpml, tsrc, step, true);
    p.E[0][q] = n0;
    p.E[1][q] = n1;
    p.E[2][q] = n2;
}

template <typename T>
__device__ __forceinline__ void emixed_slot(const KParams<T> &p, int m) {
    const int4 s = p.mixed[m];
    if (s.w >= 0)
        emixed_apply<T, false>(p, CoefMem<T>{p.coefx}, s, s.w);
    else
        emixed_apply<T, true>(p, CoefMem<T>{p.coef}, s, kMixed);
}

// the magnetic faces of a wavefront's slots: not stored (st).  Which films' face
// boxes meet the row's slots is scalar work, four films a round trip through the
// scalar cache, which waits for no field load; boxes do not overlap, and the
// films that meet it, one or none mostly, are then taken one by one.  Face by
// face over the list, a tile near a film waited some 2 us a film with two slots
// a lane and 1.3 with one.  H/M launch, us: 200 x 160 x 40 with 48 films float64
// 124 -> 39, float32 80 -> 35; 160 x 144 x 128 with one 45.5 -> 44.8, 34.5 -> 27.4.
// (A lane a film and a ballot: 35.5 and 24 with 48, but 47.8 and 27.4 with one,
// the box loads waiting behind the fields'.)
template <typename T, int V>
__device__ __forceinline__ void film_faces(const KParams<T> &p, const RowPos &r, bool (&st0)[V], bool (&st1)[V],
                                           bool (&st2)[V]) {
    constexpr int G = 4;
    for (int g0 = 0; g0 < p.nfilm; g0 += G) {
        int b[G][6]; // b0, bn
#pragma unroll
        for (int g = 0; g < G; g++) {
            const cword_t *src = (const cword_t *)(p.films + min(g0 + g, p.nfilm - 1));
#pragma unroll
            for (int w = 0; w < 6; w++) b[g][w] = (int)src[w];
        }
        unsigned meet = 0;
#pragma unroll
        for (int g = 0; g < G; g++) {
            const int y = r.j - b[g][1], z = r.k - b[g][2];
            const bool in = g0 + g < p.nfilm && y >= 0 && y < b[g][4] && z >= 0 && z < b[g][5] &&
                            b[g][0] < r.w0 + 64 * V && b[g][0] + b[g][3] > r.w0;
            meet |= in ? 1u << g : 0u;
        }
        for (; meet; meet &= meet - 1) {
            const FilmDev F = film_desc(p.films, g0 + __builtin_ctz(meet));
            // (a film's faces of one family fit 32 bits)
            const double *ms = F.prm + (unsigned)F.bn[0] * (unsigned)(r.j - F.b0[1] + F.bn[1] * (r.k - F.b0[2]));
#pragma unroll
            for (int v = 0; v < V; v++) {
                const int x = r.i + v - F.b0[0];
                const bool in = x >= 0 && x < F.bn[0];
                const double *q = ms + (in ? x : 0);
                const double m0 = q[0], m1 = q[3 * F.ns], m2 = q[6 * F.ns];
                st0[v] = st0[v] && !(in && m0 > 0.0);
                st1[v] = st1[v] && !(in && m1 > 0.0);
                st2[v] = st2[v] && !(in && m2 > 0.0);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// H/M pass: NHALF half steps of the non-magnetic faces of slot (i, j, k);
// reads E at the slot and at its +x, +y, +z neighbours.  A +1 neighbour wraps
// on a periodic axis and reads zero at a wall (the E there is tangential to
// it); lanes past the domain store nothing.
// ---------------------------------------------------------------------------
// LATE: the neighbours in the plane are loaded last
template <typename T, int NHALF, int V, bool BIG, bool LATE>
__device__ __forceinline__ void hpass_row(const KParams<T> &p, const RowPos &r, int f) {
    if (r.j >= p.n[1]) return; // a partial tile's row (uniform)
    const unsigned es = (unsigned)sizeof(T);
    const int ic = min(r.i, (p.n[0] - 1) & -V), j = r.j, k = r.k;
    // an array below 4 GiB: bases are the kernel's arguments, the plane is in
    // the lanes' 32-bit offsets; else (BIG) bases are the plane's
    const unsigned plane = (unsigned)p.px * (unsigned)p.n[1], rowb = (unsigned)p.px * es;
    const unsigned io = (unsigned)ic * es, po = BIG ? 0u : (unsigned)k * plane * es, vo = io + (po + (unsigned)j * rowb);
    const long long zo = BIG ? (long long)((unsigned long long)plane * (unsigned)k) : 0;
    // the +1 neighbours: wrapped on a periodic axis; past a wall the own
    // value is read and dropped
    const bool wly = !p.per[1] && j + 1 >= p.n[1], wlz = !p.per[2] && k + 1 >= p.n[2];
    const unsigned vxp = ic + V < p.n[0] ? vo + V * es : (p.per[0] ? vo - io : vo);
    const unsigned jp = (unsigned)(j + 1 < p.n[1] ? j + 1 : (p.per[1] ? 0 : j)), vyp = io + (po + jp * rowb);
    const unsigned ka = (unsigned)(k + 1 < p.n[2] ? k + 1 : (p.per[2] ? 0 : k));
    const unsigned vzp = BIG ? vo : io + (ka * plane * es + (unsigned)j * rowb);
    const long long za = BIG ? (long long)((unsigned long long)plane * ka) : 0;
    const T *Ex = p.E[0] + zo, *Ey = p.E[1] + zo, *Ez = p.E[2] + zo;
    T ex0[V], ex_yp[V], ex_kp[V], ey0[V], ey_xp[V], ey_kp[V], ez0[V], ez_xp[V], ez_yp[V];
    T ey_nx, ez_nx; // the slot after the lane's last
    row_ldv<V>(Ex, vo, ex0);
    if constexpr (!LATE) row_ldv<V>(Ex, vyp, ex_yp);
    row_ldv<V>(p.E[0] + za, vzp, ex_kp);
    row_ldv<V>(Ey, vo, ey0);
    if constexpr (!LATE) ey_nx = row_ld(Ey, vxp);
    row_ldv<V>(p.E[1] + za, vzp, ey_kp);
    row_ldv<V>(Ez, vo, ez0);
    if constexpr (!LATE) {
        ez_nx = row_ld(Ez, vxp);
        row_ldv<V>(Ez, vyp, ez_yp);
    }
    // H and the new H are touched once per pass: non-temporal (the E halo
    // stays in L2)
    T *Hx = p.H[0] + zo, *Hy = p.H[1] + zo, *Hz = p.H[2] + zo;
    T h0[V], h1[V], h2[V];
    row_ldv<V, true>(Hx, vo, h0);
    row_ldv<V, true>(Hy, vo, h1);
    row_ldv<V, true>(Hz, vo, h2);
    RowPml<T, V> m = row_pml<T, false, V>(p, r, io);
    if constexpr (LATE) {
        // the neighbours in the plane last: by then their own wavefronts have
        // asked for the same lines (512 x 256 x 128 float32: 126 us, with them
        // first 138; but float64 with two slots a lane 252, among the others
        // 244, and a batch of 32 small grids 232 : 226)
        __builtin_amdgcn_sched_barrier(0);
        ey_nx = row_ld(Ey, vxp);
        ez_nx = row_ld(Ez, vxp);
        row_ldv<V>(Ex, vyp, ex_yp);
        row_ldv<V>(Ez, vyp, ez_yp);
    }
    // the tile's flags, first used after every field load has been issued
    bool st0[V], st1[V], st2[V]; // stored: not past the row, not magnetic
#pragma unroll
    for (int v = 0; v < V; v++) st0[v] = st1[v] = st2[v] = r.i + v < p.n[0];
    if (f & 4) film_faces<T, V>(p, r, st0, st1, st2);
#pragma unroll
    for (int v = 0; v < V; v++) {
        // inside the lane's group the next slot's, unless the row ends there
        // (a wall reads zero)
        const bool end = ic + v + 1 >= p.n[0];
        const T a = v + 1 < V ? ey0[v + 1 < V ? v + 1 : v] : ey_nx, b = v + 1 < V ? ez0[v + 1 < V ? v + 1 : v] : ez_nx;
        ey_xp[v] = end ? (p.per[0] ? ey_nx : T(0)) : a;
        ez_xp[v] = end ? (p.per[0] ? ez_nx : T(0)) : b;
    }
    if (wly)
#pragma unroll
        for (int v = 0; v < V; v++) ex_yp[v] = ez_yp[v] = T(0);
    if (wlz)
#pragma unroll
        for (int v = 0; v < V; v++) ex_kp[v] = ey_kp[v] = T(0);
    const T dx = p.dT[0], dy = p.dT[1], dz = p.dT[2], ix = p.invd[0], iy = p.invd[1], iz = p.invd[2];
    const bool pml = m.wx || m.wy || m.wz;
#pragma unroll
    for (int v = 0; v < V; v++) {
        const T ay = dif(ez_yp[v], ez0[v], dy, iy), az = dif(ey_kp[v], ey0[v], dz, iz);
        const T bz = dif(ex_kp[v], ex0[v], dz, iz), bx = dif(ez_xp[v], ez0[v], dx, ix);
        const T cx = dif(ey_xp[v], ey0[v], dx, ix), cy = dif(ex_yp[v], ex0[v], dy, iy);
        if (pml) {
#pragma unroll
            for (int hs = 0; hs < NHALF; hs++) {
                T a1 = ay, a2 = az, b1 = bz, b2 = bx, c1 = cx, c2 = cy;
                if (m.wx) {
                    pml_step_if(m.sx[v], m.xy[v], m.bx[v], m.cx[v], b2);
                    pml_step_if(m.sx[v], m.xz[v], m.bx[v], m.cx[v], c1);
                }
                if (m.wy) {
                    pml_step(m.yx[v], m.by, m.cy, a1);
                    pml_step(m.yz[v], m.by, m.cy, c2);
                }
                if (m.wz) {
                    pml_step(m.zx[v], m.bz, m.cz, a2);
                    pml_step(m.zy[v], m.bz, m.cz, b1);
                }
                h0[v] = h0[v] - p.hc * (a1 - a2);
                h1[v] = h1[v] - p.hc * (b1 - b2);
                h2[v] = h2[v] - p.hc * (c1 - c2);
            }
        } else {
            const T g0 = p.hc * (ay - az), g1 = p.hc * (bz - bx), g2 = p.hc * (cx - cy);
#pragma unroll
            for (int hs = 0; hs < NHALF; hs++) {
                h0[v] = h0[v] - g0;
                h1[v] = h1[v] - g1;
                h2[v] = h2[v] - g2;
            }
        }
    }
    row_stv<V, true>(Hx, vo, h0, st0);
    row_stv<V, true>(Hy, vo, h1, st1);
    row_stv<V, true>(Hz, vo, h2, st2);
    if (m.wx) {
        const long long q = row_psi(p, 0, j, k);
#pragma unroll
        for (int v = 0; v < V; v++)
            if (m.sx[v]) {
                if (st1[v]) row_st(p.psiH[1][0] + q, m.ox[v], m.xy[v]);
                if (st2[v]) row_st(p.psiH[2][0] + q, m.ox[v], m.xz[v]);
            }
    }
    if (m.wy) {
        const long long q = row_psi(p, 1, j, k);
        row_stv<V, true>(p.psiH[0][1] + q, io, m.yx, st0);
        row_stv<V, true>(p.psiH[2][1] + q, io, m.yz, st2);
    }
    if (m.wz) {
        const long long q = row_psi(p, 2, j, k);
        row_stv<V, true>(p.psiH[0][2] + q, io, m.zx, st0);
        row_stv<V, true>(p.psiH[1][2] + q, io, m.zy, st1);
    }
}

template <typename T, int NHALF, int V, int WX, bool WIDE, bool BIG, bool LATE = V == 1>
__device__ __forceinline__ void hpass_block(const KParams<T> &p, int bx, int by, int k) {
    const RowPos r = row_pos_v<V, WX>(p.n, bx, by, k);
    if (r.w0 >= p.n[0]) return; // uniform: a wavefront past the row
    hpass_row<T, NHALF, V, BIG, LATE>(p, r, row_flags<T, V>(p, r, WIDE));
}

// grid (x tiles, y tiles, planes) in natural order: the blocks resident at
// one time cover a few consecutive planes, so neighbour rows and planes are
// cache hits, and no block decodes its tile with divisions.  The tile is the
// grid's (with_shape).  XC: the variant for grids with extended-table slots
// (16-bit classes).
template <typename T, int V, int WX, bool WIDE, bool BIG, bool XC>
__global__ void __launch_bounds__(256) k_epass(KParams<T> p) {
    epass_block<T, XC ? 1 : 0, V, WX, WIDE, BIG>(p, blockIdx.x, blockIdx.y, blockIdx.z);
}

template <typename T, int V, int WX, bool WIDE, bool BIG, bool XC>
__global__ void __launch_bounds__(256) k_epass_tape(KParams<T> p, BoxTape bt) {
    epass_block<T, XC ? 1 : 0, V, WX, WIDE, BIG, true>(p, blockIdx.x, blockIdx.y, blockIdx.z, bt);
}

template <typename T, int NHALF, int V, int WX, bool WIDE, bool BIG>
__global__ void __launch_bounds__(256) k_hbulk(KParams<T> p, int inc_step) {
    if (inc_step && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0 && threadIdx.y == 0)
        p.step[0] = p.step[0] + 1;
    hpass_block<T, NHALF, V, WX, WIDE, BIG>(p, blockIdx.x, blockIdx.y, blockIdx.z);
}

// the H/M pass and the film's part of it in one launch: the first zf planes
// of the grid are the film blocks (256 threads, one block of magnetic faces
// each), dispatched first so that their latency-bound work overlaps the bulk
// planes.  NHALF 2: the merged pair, with the film's second half step; NHALF
// 1: a bracket half step, with the commit of the film's half step.  The two
// touch disjoint data: the film blocks read the prepass (or the scratch) the
// first half step wrote and write M and H of magnetic faces, which the bulk
// blocks load but never store or use.
// The probes of an integer time when every one of them reads only E, a film's
// mean-M partials or its energy partials (which this launch does not write)
// ride in the block right after the film blocks: its first wavefront reads the step counter,
// samples each probe due and then advances the counter (no other block of
// the launch reads it).
// Every tile shape uses it: on a grid of 10^4..10^6 cells a launch of its own
// costs the film blocks or the probes 4-7 us (their chain of dependent loads)
// against no measurable time beside the bulk blocks.
// tid: the thread's index in its block of 256
template <typename T>
__device__ __forceinline__ void probe_block(const KParams<T> &p, int nprobe, int inc_step, int tid) {
    const long long step = p.step[0];
    for (int pb = 0; pb < nprobe; pb++) {
        const ProbeDev &P = p.probes[pb];
        long long sample;
        if (!probe_due(P, step, sample)) continue; // uniform over the block
        double v[3] = {0.0, 0.0, 0.0};
        if (P.kind == 3) {
            double sum[2];
            block_order_sum_pairs(P.part, P.npart, sum);
            v[0] = 0.5 * p.dV * (sum[0] + p.mu0 * sum[1]);
        } else if (tid < 64) // one wavefront does it all
            folded_probe_values(p, P, v);
        if (tid < 64) probe_store(p, P, sample, v);
    }
    // the counter advances after every thread has read it
    __syncthreads();
    if (inc_step && tid == 0) p.step[0] = step + 1;
}

template <typename T, int NHALF>
__device__ __forceinline__ void film_part(const KParams<T> &p, int blk, int tid) {
    if constexpr (NHALF == 2)
        film_body(p, 2, 0, blk, tid);
    else
        film_commit_body(p, blk, tid);
}

template <typename T, int NHALF, int V, int WX, bool WIDE, bool BIG>
__global__ void __launch_bounds__(256) k_hbulk_film(KParams<T> p, int inc_step, int zf, int nfb, int nprobe) {
    if ((int)blockIdx.z < zf) {
        const int fb = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
        const int tid = (int)threadIdx.x + 64 * (int)threadIdx.y;
        if (fb < nfb)
            film_part<T, NHALF>(p, fb, tid);
        else if (fb == nfb && nprobe > 0)
            probe_block(p, nprobe, inc_step, tid);
        return;
    }
    const int k = (int)blockIdx.z - zf;
    if (inc_step && nprobe == 0 && blockIdx.x == 0 && blockIdx.y == 0 && k == 0 && threadIdx.x == 0 &&
        threadIdx.y == 0)
        p.step[0] = p.step[0] + 1;
    hpass_block<T, NHALF, V, WX, WIDE, BIG>(p, blockIdx.x, blockIdx.y, k);
}

template <typename T>
__global__ void __launch_bounds__(256) k_emixed(KParams<T> p) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m < p.nmixed) emixed_slot<T>(p, m);
}

// batched: work[w] = (instance, x tile, y tile, plane)
template <typename T, bool XC, bool BIG>
__global__ void __launch_bounds__(PTX *PTY)
    k_epass_batch(const KParams<T> *__restrict__ plist, const int4 *__restrict__ work, int nwork) {
    const int w = blockIdx.x;
    if (w >= nwork) return;
    const int4 wk = work[w];
    epass_block<T, XC ? 2 : 0, 1, 1, false, BIG>(plist[wk.x], wk.y, wk.z, wk.w);
}

// work[w] = (instance, first list entry of a 256-entry block)
template <typename T>
__global__ void __launch_bounds__(256)
    k_emixed_batch(const KParams<T> *__restrict__ plist, const int2 *__restrict__ work, int nwork) {
    const int w = blockIdx.x;
    if (w >= nwork) return;
    const int2 wk = work[w];
    const KParams<T> &p = plist[wk.x];
    const int m = wk.y + threadIdx.x;
    if (m < p.nmixed) emixed_slot<T>(p, m);
}

// work[w] = (instance, x tile, y tile, plane), or (instance, -1 - film block,
// 0, 0), or (instance, kBatchProbes, 0, 0): the film blocks and the probe
// block of an instance ride in the launch as in k_hbulk_film.  The step
// counter of an instance moves with its probe block, or else its first tile.
template <typename T, int NHALF, bool BIG>
__global__ void __launch_bounds__(PTX *PTY)
    k_hbulk_batch(const KParams<T> *__restrict__ plist, const int4 *__restrict__ work, int nwork, int inc_step) {
    const int w = blockIdx.x;
    if (w >= nwork) return;
    const int4 wk = work[w];
    const KParams<T> &p = plist[wk.x];
    if (wk.y < 0) {
        const int tid = (int)threadIdx.x + 64 * (int)threadIdx.y;
        if (wk.y == kBatchProbes)
            probe_block(p, p.nfold, inc_step, tid);
        else
            film_part<T, NHALF>(p, -1 - wk.y, tid);
        return;
    }
    if (inc_step && p.nfold == 0 && wk.y == 0 && wk.z == 0 && wk.w == 0 && threadIdx.x == 0 && threadIdx.y == 0)
        p.step[0] = p.step[0] + 1;
    hpass_block<T, NHALF, 1, 1, false, BIG, false>(p, wk.y, wk.z, wk.w);
}

template <int V, int WX>
static dim3 pass_grid(const int *n) {
    const int tx = 64 * V * WX, ty = 4 / WX;
    return dim3((n[0] + tx - 1) / tx, (n[1] + ty - 1) / ty, n[2]);
}

template <typename T, int V, int WX, bool WIDE, bool BIG>
static void launch_e(const KParams<T> &p, hipStream_t s, const BoxTape *tape) {
    const dim3 g = pass_grid<V, WX>(p.n), b(64, 4);
    if (tape && p.cls16)
        k_epass_tape<T, V, WX, WIDE, BIG, true><<<g, b, 0, s>>>(p, *tape);
    else if (tape)
        k_epass_tape<T, V, WX, WIDE, BIG, false><<<g, b, 0, s>>>(p, *tape);
    else if (p.cls16)
        k_epass<T, V, WX, WIDE, BIG, true><<<g, b, 0, s>>>(p);
    else
        k_epass<T, V, WX, WIDE, BIG, false><<<g, b, 0, s>>>(p);
}

template <typename T, int NHALF, int V, int WX, bool WIDE, bool BIG>
static void launch_hm(const KParams<T> &p, int nblk, int inc, int nprobe, hipStream_t s) {
    const dim3 g = pass_grid<V, WX>(p.n), b(64, 4);
    if (nblk == 0 && nprobe == 0) {
        k_hbulk<T, NHALF, V, WX, WIDE, BIG><<<g, b, 0, s>>>(p, inc);
        return;
    }
    const int per_plane = (int)(g.x * g.y), nfront = nblk + (nprobe > 0 ? 1 : 0);
    const int zf = (nfront + per_plane - 1) / per_plane;
    if (g.z + zf > kMaxGridZ) {
        // a long narrow grid whose film fills most of its cross section: the
        // film and probe blocks in a launch of their own, along x (its one
        // "plane" holds no tile), then the tiles; the two touch disjoint data
        k_hbulk_film<T, NHALF, V, WX, WIDE, BIG><<<dim3(nfront), b, 0, s>>>(p, inc, 1, nblk, nprobe);
        k_hbulk<T, NHALF, V, WX, WIDE, BIG><<<g, b, 0, s>>>(p, nprobe > 0 ? 0 : inc);
        return;
    }
    k_hbulk_film<T, NHALF, V, WX, WIDE, BIG><<<dim3(g.x, g.y, g.z + zf), b, 0, s>>>(p, inc, zf, nblk, nprobe);
}

// calls f with the shape of a grid's passes: V slots a lane, WX wavefronts
// side by side in a block's 4 / WX rows, the wide or the 64 x 4 flag table.
//
// float64, V = 2: 16-byte loads and stores, half the instructions a slot; 4
// wavefronts a SIMD instead of 7 still hold more bytes in flight.  E + H/M, us,
// one slot a lane : two: 128 x 64 x 64 30 : 25, 211 x 109 x 77 78 : 70,
// 512 x 256 x 128 516 : 480, 1536 x 384 x 64 1126 : 1056.  A row's last
// wavefront is then emptier: with 160 or 192 slots (62 and 75 % of the lanes
// instead of 83 and 100 %) 96 : 99 and 38 : 39, so V = 2 asks that 64-slot
// wavefronts would have at least 90 % as many lanes.
// float, V = 1: two slots a lane (8-byte loads) lose everywhere (33.4 : 38 us
// on 256 x 128 x 48), four gain nothing (248 : 259 us on 512 x 256 x 128).
//
// WX: a block of several rows fetches fewer -y (+y) rows that another XCD's
// block fetches too, a longer row fewer planes' worth of partly used lines:
// 512 x 256 x 128 float 128 x 2 slots 249, 256 x 1 263; float64 256 x 2 480,
// 128 x 4 504; from 1024 slots in float 256 x 1 (1024 x 384 x 96 555 : 562,
// 1536 x 384 x 96 801 : 832; 768 x 256 x 96 279 : 272).  Narrow rows whose last
// block would have an idle wavefront take one wavefront a row: blocks go
// round-robin to the XCDs, and with an even number of blocks a row some XCDs
// would get only the emptier ones (160 x 144 x 128 float64, 64 x 4 : 128 x 2
// slots: 96 : 115 us; 160 x 100 x 60 float 26 : 29; but 256 x 128 x 48 float
// 34.6 : 33.5, 96 x 64 x 48 13.6 : 13.2).
template <int V, int WX, bool WIDE, bool BIG = false>
struct PassShape {
    static constexpr int v = V, wx = WX;
    static constexpr bool wide = WIDE, big = BIG;
};
template <typename T, typename F>
static void with_shape(const KParams<T> &p, F f) {
    const int w64 = (p.n[0] + 63) / 64, w128 = (p.n[0] + 127) / 128; // wavefronts a row
    const bool big = big_array(p.px, p.n, sizeof(T));
    // (schedule 6 takes the large arrays' form at every size)
    if (p.wide < 0 || (big && !p.wide)) return f(PassShape<1, 1, false, true>());
    if constexpr (sizeof(T) == 8) {
        if (10 * w64 < 18 * w128) return f(PassShape<1, 1, false>());
        if (big && p.wide) return f(PassShape<2, 2, true, true>());
        if (p.wide) return f(PassShape<2, 2, true>());
        return f(PassShape<2, 1, false>());
    } else {
        if (big && p.wide) return f(PassShape<1, 4, true, true>());
        if (p.wide && p.n[0] >= 1024) return f(PassShape<1, 4, true>());
        if (p.wide) return f(PassShape<1, 2, true>());
        if (w64 % 2 == 0) return f(PassShape<1, 2, false>());
        return f(PassShape<1, 1, false>());
    }
}

// the E pass and then its mixed slots
template <typename T>
hipError_t launch_epass(const KParams<T> &p, hipStream_t s, const BoxTape *tape) {
    with_shape(p, [&](auto h) {
        typedef decltype(h) S;
        launch_e<T, S::v, S::wx, S::wide, S::big>(p, s, tape);
    });
    if (p.nmixed > 0) k_emixed<T><<<dim3((p.nmixed + 255) / 256), dim3(256), 0, s>>>(p);
    return hipGetLastError();
}

// the H/M pass with the film's part (nblk blocks: the second half step of a
// merged pair, nhalf = 2, or the commit of a bracket half step, nhalf = 1)
// and nprobe probes
template <typename T>
hipError_t launch_hbulk_film(const KParams<T> &p, int nhalf, int nblk, int inc, hipStream_t s, int nprobe) {
    with_shape(p, [&](auto h) {
        typedef decltype(h) S;
        if (nhalf == 1)
            launch_hm<T, 1, S::v, S::wx, S::wide, S::big>(p, nblk, inc, nprobe, s);
        else
            launch_hm<T, 2, S::v, S::wx, S::wide, S::big>(p, nblk, inc, nprobe, s);
    });
    return hipGetLastError();
}

template <typename T>
hipError_t launch_epass_batch(const KParams<T> *plist, const int4 *work, int nwork, const int2 *mwork, int nmwork,
                              bool xcls, bool big, hipStream_t s) {
    if (nwork == 0) return hipSuccess;
    if (big)
        k_epass_batch<T, true, true><<<dim3(nwork), dim3(PTX, PTY), 0, s>>>(plist, work, nwork);
    else if (xcls)
        k_epass_batch<T, true, false><<<dim3(nwork), dim3(PTX, PTY), 0, s>>>(plist, work, nwork);
    else
        k_epass_batch<T, false, false><<<dim3(nwork), dim3(PTX, PTY), 0, s>>>(plist, work, nwork);
    if (nmwork > 0) k_emixed_batch<T><<<dim3(nmwork), dim3(256), 0, s>>>(plist, mwork, nmwork);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_hbulk_batch(const KParams<T> *plist, const int4 *work, int nwork, int inc, bool big,
                              hipStream_t s) {
    if (nwork == 0) return hipSuccess;
    const dim3 g(nwork), b(PTX, PTY);
    if (big)
        k_hbulk_batch<T, 2, true><<<g, b, 0, s>>>(plist, work, nwork, inc);
    else
        k_hbulk_batch<T, 2, false><<<g, b, 0, s>>>(plist, work, nwork, inc);
    return hipGetLastError();
}

#define MPX_PASSES(T)                                                                                      \
    template hipError_t launch_epass<T>(const KParams<T> &, hipStream_t, const BoxTape *);                \
    template hipError_t launch_hbulk_film<T>(const KParams<T> &, int, int, int, hipStream_t, int);             \
    template hipError_t launch_epass_batch<T>(const KParams<T> *, const int4 *, int, const int2 *, int,   \
                                              bool, bool, hipStream_t);                                   \
    template hipError_t launch_hbulk_batch<T>(const KParams<T> *, const int4 *, int, int, bool, hipStream_t);
MPX_PASSES(float)
MPX_PASSES(double)

} // namespace mpx
