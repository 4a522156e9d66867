// film.h -- the magnetic-face LLG half step of one block of film sites and
// the float64 helpers it uses; included by the kernel files that launch it
// (the film kernels, and the merged H/M pass that runs the second half step
// of a pair beside the bulk faces).
//
// Scheme: arXiv:2510.22221, Methods, "Numerical Model": B^ = H + M,
// B^* = B^ - dt/(2 mu0) curl E (eq. iterate_H); the trapezoidal LLG (eqs.
// llg_tra4-llg_tra6) at its fixed point, normalised to Ms; H = B^*_c - M_c.
#pragma once

#include "device_common.h"

namespace mpx {

template <typename T>
__device__ __forceinline__ long long film_local(const FilmDev &F, const int *idx, bool &inside) {
    int r[3];
    for (int a = 0; a < 3; a++) {
        r[a] = idx[a] - F.b0[a];
        if (r[a] < 0 || r[a] >= F.bn[a]) {
            inside = false;
            return 0;
        }
    }
    inside = true;
    return (long long)r[0] + (long long)F.bn[0] * ((long long)r[1] + (long long)F.bn[1] * r[2]);
}

// (curl E)_c parts at the H_c site idx, in float64
template <typename T>
__device__ __forceinline__ void curl_e64(const KParams<T> &p, int c, const int *idx, double &d1, double &d2) {
    const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    int u1[3] = {idx[0], idx[1], idx[2]}, u2[3] = {idx[0], idx[1], idx[2]};
    u1[c1] += 1;
    u2[c2] += 1;
    const double e2a = (double)ldz(p, p.E[c2], idx[0], idx[1], idx[2]);
    const double e2b = (double)ldz(p, p.E[c2], u1[0], u1[1], u1[2]);
    const double e1a = (double)ldz(p, p.E[c1], idx[0], idx[1], idx[2]);
    const double e1b = (double)ldz(p, p.E[c1], u2[0], u2[1], u2[2]);
    d1 = (e2b - e2a) / p.d[c1];
    d2 = (e1b - e1a) / p.d[c2];
}

__device__ __forceinline__ void cross3(const double *a, const double *b, double *r) {
    r[0] = a[1] * b[2] - a[2] * b[1];
    r[1] = a[2] * b[0] - a[0] * b[2];
    r[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dot3(const double *a, const double *b) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// the site solve of one magnetic face: P, Q are B^* and B^ at the face
// (own family) and the means of the four nearest faces of each other family,
// M the magnetisation of the half step's start; the bias is added to P and Q
// here.  Trapezoidal LLG over the half step at its fixed point:
// b = M - k (M x H_eff(M)) with H_eff = Q - M, a = -(k P + (alpha/Ms) M),
// X = (b + (a.b) a - a x b) / (1 + |a|^2), M' = Ms X / |X|
__device__ __forceinline__ void llg_site(double kf, const double *H0, double ms, double al, double ga, double *P,
                                         double *Q, const double *M, double *Mn) {
    for (int w = 0; w < 3; w++) {
        P[w] += H0[w];
        Q[w] += H0[w];
    }
    const double kk = kf * ga;
    // b = M^n - k (M^n x H_eff^n), with H_eff^n = Q - M^n
    double MxQ[3], b[3], a[3];
    cross3(M, Q, MxQ);
    for (int w = 0; w < 3; w++) b[w] = M[w] - kk * MxQ[w];
    // a at the fixed point: H_eff^{n+1} = P - M^{n+1}
    for (int w = 0; w < 3; w++) a[w] = -(kk * P[w] + (al / ms) * M[w]);
    // X = (b + (a.b) a - a x b) / (1 + |a|^2), then M' = Ms X/|X|
    double axb[3], X[3];
    cross3(a, b, axb);
    const double ab = dot3(a, b), aa = dot3(a, a);
    for (int w = 0; w < 3; w++) X[w] = (b[w] + ab * a[w] - axb[w]) / (1.0 + aa);
    const double nx = sqrt(dot3(X, X));
    for (int w = 0; w < 3; w++) Mn[w] = ms * X[w] / nx;
}

// B^ (Q) and B^* (P) of family-c face r (position in film F's face box): the
// face's own in component c, the mean of the four nearest faces of family c'
// in each other (indices {-1, 0} along c and {0, 1} along c'), from the
// prepass arrays over the grown face box.  Every load is issued, a neighbour
// outside the grown box at its element 0 with the value dropped (only
// non-magnetic faces have any): a magnetic face waits for one round trip.
__device__ __forceinline__ void film_gather(const int *n, const int *per, const FilmDev &F, int c, const int *r,
                                            const double *Bn, const double *Bs, double *P, double *Q, int &le) {
    // position in the grown box of the site and of its -1 and +1 neighbours
    int o[3], lo[3], hi[3];
    const int st[3] = {1, F.en[0], F.en[0] * F.en[1]};
    bool okl[3], okh[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const int i = F.b0[a] + r[a];
        o[a] = (i - F.e0[a]) * st[a];
        const int m = fold(i - 1, n[a], per[a]) - F.e0[a], q = fold(i + 1, n[a], per[a]) - F.e0[a];
        okl[a] = m >= 0 && m < F.en[a];
        okh[a] = q >= 0 && q < F.en[a];
        lo[a] = m * st[a];
        hi[a] = q * st[a];
    }
    le = o[0] + o[1] + o[2];
    P[c] = Bs[c * F.nse + le];
    Q[c] = Bn[c * F.nse + le];
#pragma unroll
    for (int w = 1; w < 3; w++) {
        const int cp = c + w < 3 ? c + w : c + w - 3, ct = 3 - c - cp;
        double vn[2][2], vs[2][2];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++) {
                const bool ok = (u || okl[c]) && (!v || okh[cp]);
                const int q = (u ? o[c] : lo[c]) + (v ? hi[cp] : o[cp]) + o[ct];
                const double xn = Bn[cp * F.nse + (ok ? q : 0)], xs = Bs[cp * F.nse + (ok ? q : 0)];
                vn[u][v] = ok ? xn : 0.0;
                vs[u][v] = ok ? xs : 0.0;
            }
        Q[cp] = ((vn[0][0] + vn[1][0]) + (vn[0][1] + vn[1][1])) * 0.25;
        P[cp] = ((vs[0][0] + vs[1][0]) + (vs[0][1] + vs[1][1])) * 0.25;
    }
}

// film_gather() from the state the prepass reads, in the prepass's
// operations: what a face takes from its own and eight neighbours' prepass is
// 20 values of E, nine of H and of the films' tables.  With cu, the curl term
// of the face's phase-2 values.
template <typename T, int C>
__device__ __forceinline__ void film_gather_state(const KParams<T> &p, const FilmDev &F, const int *r, unsigned l,
                                                  double *P, double *Q, double &cu, int &le) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    // offsets of the -1, 0 and +1 neighbours along each axis, in the grid and
    // in the face box (0 for one outside: its value is dropped)
    const long long st[3] = {1, p.px, (long long)p.px * p.n[1]};
    const int sl[3] = {1, F.bn[0], F.bn[0] * F.bn[1]}, se[3] = {1, F.en[0], F.en[0] * F.en[1]};
    long long o[3], dg[3][3];
    int dl[3][3];
    bool dom[3], ok[3][3], in[3][3];
    le = 0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const int i = F.b0[a] + r[a];
        o[a] = i * st[a];
        le += (i - F.e0[a]) * se[a];
#pragma unroll
        for (int u = 0; u < 3; u++) {
            const int q = fold(i + u - 1, p.n[a], p.per[a]);
            const bool d = q >= 0;
            const int m = q - F.e0[a], b = q - F.b0[a];
            ok[a][u] = d && m >= 0 && m < F.en[a];
            in[a][u] = d && b >= 0 && b < F.bn[a];
            dg[a][u] = d ? (q - i) * st[a] : 0;
            dl[a][u] = in[a][u] ? (b - r[a]) * sl[a] : 0;
            if (u == 2) dom[a] = d;
        }
    }
    const long long g0 = o[0] + o[1] + o[2];
    T eC[2][2][2], e1[3][2], e2[3][2]; // E_C [C][C1][C2], E_C1 [C][C2], E_C2 [C][C1]
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int v = 0; v < 2; v++)
#pragma unroll
            for (int w = 0; w < 2; w++)
                eC[u][v][w] = p.E[C][g0 + dg[C][u] + (v ? dg[C1][2] : 0) + (w ? dg[C2][2] : 0)];
#pragma unroll
    for (int u = 0; u < 3; u++)
#pragma unroll
        for (int v = 0; v < 2; v++) {
            e1[u][v] = p.E[C1][g0 + dg[C][u] + (v ? dg[C2][2] : 0)];
            e2[u][v] = p.E[C2][g0 + dg[C][u] + (v ? dg[C1][2] : 0)];
        }
    T h[2][2][2], hC = p.H[C][g0]; // H of C1 and C2 [C][own axis]
    double ms[2][2][2], m[2][2][2];
    const double msC = F.prm[(C * 3) * F.ns + l], mC = F.M[(C * 3 + C) * F.ns + l];
    bool use[2][2][2], mag[2][2][2];
#pragma unroll
    for (int w = 0; w < 2; w++) {
        const int cp = w ? C2 : C1;
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++) {
                use[w][u][v] = ok[C][u] && ok[cp][v + 1];
                mag[w][u][v] = in[C][u] && in[cp][v + 1];
                const long long n = (long long)l + (mag[w][u][v] ? dl[C][u] + dl[cp][v + 1] : 0);
                h[w][u][v] = p.H[cp][g0 + dg[C][u] + dg[cp][v + 1]];
                ms[w][u][v] = F.prm[(cp * 3) * F.ns + n];
                m[w][u][v] = F.M[(cp * 3 + cp) * F.ns + n];
            }
    }
    // zero past a wall
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int v = 0; v < 2; v++)
#pragma unroll
            for (int w = 0; w < 2; w++)
                if ((v && !dom[C1]) || (w && !dom[C2])) eC[u][v][w] = T(0);
#pragma unroll
    for (int u = 0; u < 3; u++)
#pragma unroll
        for (int v = 0; v < 2; v++) {
            if ((u == 2 && !dom[C]) || (v && !dom[C2])) e1[u][v] = T(0);
            if ((u == 2 && !dom[C]) || (v && !dom[C1])) e2[u][v] = T(0);
        }
    {
        const double d1 = over_spacing(p, (double)e2[1][1] - (double)e2[1][0], C1);
        const double d2 = over_spacing(p, (double)e1[1][1] - (double)e1[1][0], C2);
        cu = p.hcd * (d1 - d2);
        const double b = msC > 0.0 ? (double)hC + mC : (double)hC + 0.0;
        Q[C] = b;
        P[C] = b - cu;
    }
#pragma unroll
    for (int w = 0; w < 2; w++) {
        const int cp = w ? C2 : C1;
        double vn[2][2], vs[2][2];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++) {
                double d1, d2;
                if (w == 0) {
                    d1 = over_spacing(p, (double)eC[u][v][1] - (double)eC[u][v][0], C2);
                    d2 = over_spacing(p, (double)e2[u + 1][v] - (double)e2[u][v], C);
                } else {
                    d1 = over_spacing(p, (double)e1[u + 1][v] - (double)e1[u][v], C);
                    d2 = over_spacing(p, (double)eC[u][1][v] - (double)eC[u][0][v], C1);
                }
                const double h0 = (double)h[w][u][v];
                const double b = mag[w][u][v] && ms[w][u][v] > 0.0 ? h0 + m[w][u][v] : h0 + 0.0;
                const double bs = b - p.hcd * (d1 - d2);
                vn[u][v] = use[w][u][v] ? b : 0.0;
                vs[u][v] = use[w][u][v] ? bs : 0.0;
            }
        Q[cp] = ((vn[0][0] + vn[1][0]) + (vn[0][1] + vn[1][1])) * 0.25;
        P[cp] = ((vs[0][0] + vs[1][0]) + (vs[0][1] + vs[1][1])) * 0.25;
    }
}

// keeps a value from being computed only behind the branch that uses it (the
// compiler moves loads there, one round trip later)
__device__ __forceinline__ void hold(double &v) { asm volatile("" : "+v"(v)); }

// one half step of a block of 256 magnetic faces.  Latency-bound (a film of
// 10^3..10^5 faces is a few waves per CU): the chain is table entry and
// descriptor, one round trip for all of a face's loads, the float64 solve, the
// stores.  32-bit indices, the loads ahead of the magnetic test and the block
// sum in one barrier took the 64 x 12 x 4 film of a 128 x 64 x 64 grid from
// 7.0 to 4.2 us, a 400 x 60 x 4 film from 11.3 to 9.0 us; eight 200 x 40 x 4
// films stay at 30.5 us (bandwidth: 24 float64 loads a face, from cache)
// tid: the thread's index in its block of 256 (film blocks also run in
// launches whose blocks are 64 x 4)
// STATE: a first half step without its prepass (film_gather_state)
template <typename T, int C, bool STATE>
__device__ __forceinline__ double film_face(const KParams<T> &p, const FilmDev &F, int phase, unsigned l) {
    int r[3];
    box_split(l, F.bn, r);
    const double ms = F.prm[(C * 3 + 0) * F.ns + l];
    const double al = F.prm[(C * 3 + 1) * F.ns + l];
    const double ga = F.prm[(C * 3 + 2) * F.ns + l];
    const double *Msrc = (phase == 1) ? F.M : F.M1;
    double P[3], Q[3], M[3];
#pragma unroll
    for (int w = 0; w < 3; w++) M[w] = Msrc[(C * 3 + w) * F.ns + l];
    int le;
    double cu = 0.0;
    if (STATE)
        film_gather_state<T, C>(p, F, r, l, P, Q, cu, le);
    else {
        film_gather(p.n, p.per, F, C, r, phase == 1 ? F.Bn : F.Bn2, phase == 1 ? F.Bs : F.Bs2, P, Q, le);
        // the curl term the prepass left for the face's phase-2 values
        if (phase == 1 && F.Bn2) cu = F.Bs2[C * F.nse + le];
    }
#pragma unroll
    for (int w = 0; w < 3; w++) {
        hold(M[w]);
        hold(P[w]);
        hold(Q[w]);
    }
    hold(cu);
    if (!(ms > 0.0)) return 0.0;
    const double bs = P[C];
    double Mn[3];
    llg_site(p.kf, p.H0, ms, al, ga, P, Q, M, Mn);
    const double hnew = bs - Mn[C];
    if (phase == 1) {
#pragma unroll
        for (int w = 0; w < 3; w++) F.M1[(C * 3 + w) * F.ns + l] = Mn[w];
        F.H1[C * F.ns + l] = hnew;
        if (F.Bn2) {
            // the phase-2 prepass of this face: B^ = H1 + M1_c, B^* =
            // B^ - dt/(2 mu0) curl E with the same E
            const double b2 = hnew + Mn[C];
            F.Bn2[C * F.nse + le] = b2;
            F.Bs2[C * F.nse + le] = b2 - cu;
        }
    } else {
#pragma unroll
        for (int w = 0; w < 3; w++) F.M[(C * 3 + w) * F.ns + l] = Mn[w];
        p.Hw[C][p.slot(F.b0[0] + r[0], F.b0[1] + r[1], F.b0[2] + r[2])] = (T)hnew;
    }
    return Mn[C];
}

template <typename T, bool STATE = false>
__device__ __forceinline__ void film_body(const KParams<T> &p, int phase, int inc_step, int blk, int tid) {
    __shared__ double red[256];
    if (inc_step && blk == 0 && tid == 0) p.step[0] = p.step[0] + 1;
    const int4 bt = block_entry(p.blocktab, blk); // film, family, first local index
    const FilmDev F = block_desc(p.films, p.nfilm, bt.x);
    const unsigned l = (unsigned)bt.z + (unsigned)tid;
    double own = 0.0;
    if (l < (unsigned)F.ns)
        own = bt.y == 0   ? film_face<T, 0, STATE>(p, F, phase, l)
              : bt.y == 1 ? film_face<T, 1, STATE>(p, F, phase, l)
                          : film_face<T, 2, STATE>(p, F, phase, l);
    // block partial of the own component (mean-M probes, which read it
    // between the two half steps: the second half step's would go unread): a
    // halving tree, its first two levels over LDS, the rest in one wavefront
    if (phase != 1) return;
    red[tid] = own;
    __syncthreads();
    if (tid >= 64) return;
    double s = (red[tid] + red[tid + 128]) + (red[tid + 64] + red[tid + 192]);
    for (int st = 32; st > 0; st >>= 1) {
        const double o = __shfl_down(s, st, 64);
        if (tid < st) s = s + o;
    }
    if (tid == 0) p.partial[blk] = s;
}

// copy the scratch of a single (bracket) half step into the state: the block
// of magnetic faces blk
template <typename T>
__device__ __forceinline__ void film_commit_body(const KParams<T> &p, int blk, int tid) {
    const int4 bt = block_entry(p.blocktab, blk);
    const int c = bt.y;
    const FilmDev F = block_desc(p.films, p.nfilm, bt.x);
    const unsigned l = (unsigned)bt.z + (unsigned)tid;
    if (l >= (unsigned)F.ns) return;
    int r[3];
    box_split(l, F.bn, r);
    const double ms = F.prm[(c * 3) * F.ns + l];
    double m[3], h = F.H1[c * F.ns + l];
    for (int w = 0; w < 3; w++) {
        m[w] = F.M1[(c * 3 + w) * F.ns + l];
        hold(m[w]);
    }
    hold(h);
    if (!(ms > 0.0)) return;
    for (int w = 0; w < 3; w++) F.M[(c * 3 + w) * F.ns + l] = m[w];
    p.Hw[c][p.slot(F.b0[0] + r[0], F.b0[1] + r[1], F.b0[2] + r[2])] = (T)h;
}

// A region of slots [b0, b0 + r) (a cell box grown by one slot on the high
// side of each axis: the edges and faces of its cells).  Thread t owns the
// slot of region index t after folding; a slot that the fold maps onto an
// index the region already holds (a box spanning a periodic axis) belongs to
// that index.  Returns false for no slot or a slot owned elsewhere.
__device__ __forceinline__ bool region_slot(const int *n, const int *per, const int *b0, const int *r, unsigned t,
                                            int *q) {
    int loc[3];
    box_split(t, r, loc);
    for (int a = 0; a < 3; a++) {
        int v = b0[a] + loc[a];
        if (v >= n[a]) {
            if (!per[a]) return false;
            v -= n[a];
            if (v >= b0[a]) return false;
        }
        q[a] = v;
    }
    return true;
}

// the film's E and H at an integer time over its cell box grown by one slot:
// [6][region] (Ex, Ey, Ez, Hx, Hy, Hz).  merged = 1: between the two film half
// steps of a merged pair (magnetic faces' H in the film's staging, bulk faces'
// H one bulk half step ahead of the stored H); 0: a state at an integer time.
// No other film's faces lie in the region (films are at least two cells
// apart); every load goes out at once, what a face does not use is dropped.
template <typename T>
__device__ __forceinline__ void tape_loss_body(const KParams<T> &p, int film, int merged, double *dst, unsigned blk) {
    const FilmDev F = film_desc(p.films, film);
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long tb = (long long)r[0] * r[1] * r[2];
    const unsigned t = blk * 256u + threadIdx.x;
    if (t >= tb) return;
    int q[3];
    if (!region_slot(p.n, p.per, b0, r, t, q)) {
        for (int w = 0; w < 6; w++) dst[w * tb + t] = 0.0;
        return;
    }
    const long long sl = p.slot(q[0], q[1], q[2]);
    // the +1 neighbours along each axis (zero past a wall)
    long long su[3];
    bool ok[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        int u[3] = {q[0], q[1], q[2]};
        u[a] = fold(q[a] + 1, p.n[a], p.per[a]);
        ok[a] = u[a] >= 0;
        su[a] = ok[a] ? p.slot(u[0], u[1], u[2]) : sl;
    }
    T e[3], h[3], eu[3][3];
    double h1[3] = {0.0, 0.0, 0.0}, ms[3] = {0.0, 0.0, 0.0};
    bool inside = false;
    long long l = 0;
    if (merged && p.nfilm) l = film_local<T>(F, q, inside);
#pragma unroll
    for (int C = 0; C < 3; C++) {
        e[C] = p.E[C][sl];
        h[C] = p.H[C][sl];
        if (merged) {
            // E_C at +1 along the other two axes
            eu[C][(C + 1) % 3] = p.E[C][su[(C + 1) % 3]];
            eu[C][(C + 2) % 3] = p.E[C][su[(C + 2) % 3]];
            if (p.nfilm) {
                h1[C] = F.H1[C * F.ns + l];
                ms[C] = F.prm[(C * 3) * F.ns + l];
            }
        }
    }
#pragma unroll
    for (int C = 0; C < 3; C++) {
        dst[C * tb + t] = (double)e[C];
        double hv = (double)h[C];
        if (merged) {
            const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
            const T d1 = dif(ok[C1] ? eu[C2][C1] : T(0), e[C2], p.dT[C1], p.invd[C1]);
            const T d2 = dif(ok[C2] ? eu[C1][C2] : T(0), e[C1], p.dT[C2], p.invd[C2]);
            hv = (double)(h[C] - p.hc * (d1 - d2));
            if (inside && ms[C] > 0.0) hv = h1[C];
        }
        dst[(3 + C) * tb + t] = hv;
    }
}

} // namespace mpx
