// adjoint.hip -- reverse-mode (discrete adjoint) kernels of the coupled step.
//
// The forward step (arXiv:2510.22221, Methods, "Numerical Model") is
//   HALF1(E^n): H/M half step (eq. iterate_H; LLG eqs. llg_tra4-llg_tra6 at
//               magnetic faces, solved in closed form and normalised),
//   ESTEP(H):   the E update after eq. iterate_H, with CPML and the source,
//   HALF2(E^{n+1}),
// and the adjoint runs the transposes of these maps in reverse order.  Given
// the adjoint state lambda of the state after a map and the map's input
// state (recomputed from checkpoints), a kernel here returns lambda of the
// input state and accumulates the parameter gradients:
//   * non-magnetic faces and E edges are linear: transposed curls and
//     transposed CPML recursions;
//   * a magnetic face's update M' = Ms X/|X|, X = (b + (a.b)a - a x b) /
//     (1 + |a|^2), a = -(k P + (alpha/Ms) M), b = M - k M x Q, with P, Q the
//     site's B^* and B^ (own component, and the mean of four neighbouring
//     faces of each other family) plus H0, is differentiated by hand; H0, Ms
//     of each face and the edge coefficients ca, cb collect gradients.
// One thread per slot or per film face; every sum a thread forms is a gather
// (no atomics), so results do not depend on scheduling.
#include "film.h"
#include "rows.h"

namespace mpx {

// local index of face idx (folded) in the film's face box, -1 outside
__device__ __forceinline__ long long film_local_idx(const FilmDev &F, const int *idx) {
    const int r0 = idx[0] - F.b0[0], r1 = idx[1] - F.b0[1], r2 = idx[2] - F.b0[2];
    if (r0 < 0 || r0 >= F.bn[0] || r1 < 0 || r1 >= F.bn[1] || r2 < 0 || r2 >= F.bn[2]) return -1;
    return (long long)r0 + (long long)F.bn[0] * ((long long)r1 + (long long)F.bn[1] * r2);
}

// the magnetic face of family c at idx: (film, local index) or (-1, -1)
template <typename T>
__device__ __forceinline__ int mag_site(const KParams<T> &p, int c, const int *idx, long long &l) {
    for (int f = 0; f < p.nfilm; f++) {
        const FilmDev &F = p.films[f];
        const long long q = film_local_idx(F, idx);
        if (q >= 0) {
            if (F.prm[(c * 3) * F.ns + q] > 0.0) {
                l = q;
                return f;
            }
            return -1;
        }
    }
    l = -1;
    return -1;
}

// ---------------------------------------------------------------------------
// magnetic faces: lambda of (M', H'_c) -> lambda of M (direct), P, Q; the
// prepass (B^n, B^* of the input state) must have run
// ---------------------------------------------------------------------------
// (latency-bound like the forward film kernel: all loads of a face go out
// before the magnetic test; 8.9 to 5.5 us on a 64 x 12 x 4 film, 16.4 to 14.2
// on 256 x 48 x 4)
template <typename T, int c>
__device__ __forceinline__ void adj_film_face(const AdjParams<T> &A, const FilmDev &F, const AdjFilmDev &G,
                                              unsigned l) {
    const KParams<T> &p = A.p;
    int r[3];
    box_split(l, F.bn, r);
    double ms = F.prm[(c * 3 + 0) * F.ns + l];
    const double al = F.prm[(c * 3 + 1) * F.ns + l];
    const double ga = F.prm[(c * 3 + 2) * F.ns + l];
    // the forward quantities (as the film kernel computes them), lambda M' and
    // lambda H' of the face, the accumulators
    double P[3], Q[3], M[3], lMt[3], gh[3];
    int le;
    film_gather(p.n, p.per, F, c, r, F.Bn, F.Bs, P, Q, le);
    const long long sl = p.slot(F.b0[0] + r[0], F.b0[1] + r[1], F.b0[2] + r[2]);
    double lh = (double)A.lH[c][sl], g0 = G.gMs[c * F.ns + l];
#pragma unroll
    for (int w = 0; w < 3; w++) {
        M[w] = F.M[(c * 3 + w) * F.ns + l];
        lMt[w] = G.lM[(c * 3 + w) * F.ns + l];
        gh[w] = G.gH0[(c * 3 + w) * F.ns + l];
    }
#pragma unroll
    for (int w = 0; w < 3; w++) {
        hold(P[w]);
        hold(Q[w]);
        hold(M[w]);
        hold(lMt[w]);
        hold(gh[w]);
    }
    hold(lh);
    hold(g0);
    if (!(ms > 0.0)) return;
    for (int w = 0; w < 3; w++) {
        P[w] += p.H0[w];
        Q[w] += p.H0[w];
    }
    const double kk = p.kf * ga;
    double MxQ[3], b[3], a[3];
    cross3(M, Q, MxQ);
    for (int w = 0; w < 3; w++) b[w] = M[w] - kk * MxQ[w];
    for (int w = 0; w < 3; w++) a[w] = -(kk * P[w] + (al / ms) * M[w]);
    double axb[3], X[3];
    cross3(a, b, axb);
    const double ab = dot3(a, b), aa = dot3(a, a);
    const double D = 1.0 + aa;
    for (int w = 0; w < 3; w++) X[w] = (b[w] + ab * a[w] - axb[w]) / D;
    const double nx = sqrt(dot3(X, X));
    double u[3];
    for (int w = 0; w < 3; w++) u[w] = X[w] / nx;

    // lambda of M' (the face's H' = B^*_c - M'_c contributes -lambda H'_c)
    lMt[c] -= lh;
    // M' = Ms u, u = X/|X|
    const double ul = dot3(u, lMt);
    double gms = ul;
    double lX[3];
    for (int w = 0; w < 3; w++) lX[w] = ms * (lMt[w] - u[w] * ul) / nx;
    // X = N / D, N = b + (a.b) a - a x b, D = 1 + a.a
    double lN[3];
    for (int w = 0; w < 3; w++) lN[w] = lX[w] / D;
    const double lD = -dot3(lX, X) / D;
    const double alN = dot3(a, lN);
    double lNxb[3], lNxa[3];
    cross3(lN, b, lNxb);
    cross3(lN, a, lNxa);
    double la[3], lb[3];
    for (int w = 0; w < 3; w++) {
        la[w] = 2.0 * a[w] * lD + b[w] * alN + ab * lN[w] + lNxb[w];
        lb[w] = lN[w] + a[w] * alN - lNxa[w];
    }
    // a = -(k P + (alpha/Ms) M);  b = M - k M x Q
    double lP[3], lQ[3], lMd[3], Qxlb[3], lbxM[3];
    cross3(Q, lb, Qxlb);
    cross3(lb, M, lbxM);
    for (int w = 0; w < 3; w++) {
        lP[w] = -kk * la[w];
        lQ[w] = -kk * lbxM[w];
        lMd[w] = -(al / ms) * la[w] + lb[w] - kk * Qxlb[w];
    }
    gms += (al / (ms * ms)) * dot3(M, la);
    for (int w = 0; w < 3; w++) {
        G.lp[(c * 3 + w) * F.ns + l] = lP[w];
        G.lq[(c * 3 + w) * F.ns + l] = lQ[w];
        G.lMout[(c * 3 + w) * F.ns + l] = lMd[w];
        G.gH0[(c * 3 + w) * F.ns + l] = gh[w] + (lP[w] + lQ[w]);
    }
    G.gMs[c * F.ns + l] = g0 + gms;
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_film(AdjParams<T> A) {
    const KParams<T> &p = A.p;
    const int4 bt = block_entry(p.blocktab, blockIdx.x);
    const FilmDev F = block_desc(p.films, p.nfilm, bt.x);
    const AdjFilmDev G = block_desc(A.af, p.nfilm, bt.x);
    const unsigned l = (unsigned)bt.z + threadIdx.x;
    if (l >= (unsigned)F.ns) return;
    if (bt.y == 0)
        adj_film_face<T, 0>(A, F, G, l);
    else if (bt.y == 1)
        adj_film_face<T, 1>(A, F, G, l);
    else
        adj_film_face<T, 2>(A, F, G, l);
}

// can the face at idx be magnetic or be read by a magnetic face's solve (a
// face within one slot of a film's face box on every non-periodic axis)?
template <typename T>
__device__ __forceinline__ bool near_film(const KParams<T> &p, const int *idx) {
    for (int f = 0; f < p.nfilm; f++) {
        const FilmDev &F = p.films[f];
        bool in = true;
        for (int a = 0; a < 3; a++)
            if (!p.per[a] && (idx[a] < F.b0[a] - 1 || idx[a] > F.b0[a] + F.bn[a])) in = false;
        if (in) return true;
    }
    return false;
}

// ---------------------------------------------------------------------------
// every face: lambda of H' (and psi') -> lambda of H (and psi), the face's
// curl-part adjoints aD, and for magnetic faces lambda of M from B^
// ---------------------------------------------------------------------------
// lin1/lin2: lambda psiH of the derivative axes C+1, C+2 before the map;
// lout1/lout2: where the values after it go (the same arrays in place)
template <typename T, int C>
__device__ __forceinline__ void adj_face_core(const AdjParams<T> &A, const int *idx, const T *lin1, const T *lin2,
                                              T *lout1, T *lout2, T &ad0, T &ad1) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    const KParams<T> &p = A.p;
    const int i = idx[0], j = idx[1], k = idx[2];
    const long long q = p.slot(i, j, k);
    const T lHp = A.lH[C][q];
    const int a1 = idx[C1], a2 = idx[C2];
    const bool s1 = p.psiH[C][C1] && (a1 < p.nlo[C1] || a1 >= p.n[C1] - p.nhi[C1]);
    const bool s2 = p.psiH[C][C2] && (a2 < p.nlo[C2] || a2 >= p.n[C2] - p.nhi[C2]);
    const bool film_reach = p.nfilm && near_film(p, idx);
    if (!film_reach && !s1 && !s2) {
        // bulk face out of every film's reach: H' = H - hc (d1 - d2)
        ad0 = -(p.hc * lHp);
        ad1 = p.hc * lHp;
        return; // lambda H unchanged
    }
    long long lm;
    const int fm = film_reach ? mag_site(p, C, idx, lm) : -1;
    // CPML face (never next to a film)
    if (fm < 0 && (s1 || s2)) {
        const T g1 = -p.hc * lHp, g2 = p.hc * lHp; // d H' / d (d1 + psi1'), d (d2 + psi2')
        ad0 = g1;
        ad1 = g2;
        if (s1) {
            const long long qq = p.psi_index(C1, idx);
            const T aps = lin1[qq] + g1;
            lout1[qq] = p.bH[C1][a1] * aps;
            ad0 = g1 + p.cH[C1][a1] * aps;
        }
        if (s2) {
            const long long qq = p.psi_index(C2, idx);
            const T aps = lin2[qq] + g2;
            lout2[qq] = p.bH[C2][a2] * aps;
            ad1 = g2 + p.cH[C2][a2] * aps;
        }
        return; // lambda H unchanged (dH'/dH = 1)
    }
    // lambda of B^* and B^ of this face: from the face's own update and from
    // the solves of magnetic faces that read it (P, Q of the film kernel)
    double lbs_f = 0.0, lbn = 0.0;
    if (fm >= 0) {
        const FilmDev &F = p.films[fm];
        const AdjFilmDev &G = A.af[fm];
        lbs_f += G.lp[(C * 3 + C) * F.ns + lm];
        lbn += G.lq[(C * 3 + C) * F.ns + lm];
    }
    // transverse reads: the magnetic faces s of each other family cs with this
    // face in their four-face mean: s = t + a e_cs - b e_C, a, b in {0, 1}
    if (film_reach) {
#pragma unroll
        for (int cs = 0; cs < 3; cs++) {
            if (cs == C) continue;
            for (int aa = 0; aa < 2; aa++)
                for (int bb = 0; bb < 2; bb++) {
                    int s[3] = {i, j, k};
                    s[cs] += aa;
                    s[C] -= bb;
                    bool ok = true;
                    for (int ax = 0; ax < 3; ax++) {
                        s[ax] = fold(s[ax], p.n[ax], p.per[ax]);
                        if (s[ax] < 0) ok = false;
                    }
                    if (!ok) continue;
                    long long ls;
                    const int fs = mag_site(p, cs, s, ls);
                    if (fs < 0) continue;
                    const FilmDev &F = p.films[fs];
                    const AdjFilmDev &G = A.af[fs];
                    lbs_f += 0.25 * G.lp[(cs * 3 + C) * F.ns + ls];
                    lbn += 0.25 * G.lq[(cs * 3 + C) * F.ns + ls];
                }
        }
    }
    if (fm >= 0) {
        // magnetic face: H' = B^*_C - M'_C, B^* = B^ - hc (d1 - d2) in float64,
        // B^ = H + M_C
        const double lbs = (double)lHp + lbs_f;
        const double lbt = lbn + lbs;
        A.lH[C][q] = (T)lbt;
        const FilmDev &F = p.films[fm];
        const AdjFilmDev &G = A.af[fm];
        G.lMout[(C * 3 + C) * F.ns + lm] += lbt;
        ad0 = (T)(-p.hcd * lbs);
        ad1 = (T)(p.hcd * lbs);
    } else {
        // bulk face: H' = H - hc (d1 - d2) in the field precision; its B^ and
        // B^* as read by the solves are H and H - hc (d1 - d2) in float64
        A.lH[C][q] = (T)((double)lHp + lbn + lbs_f);
        ad0 = (T)(-(double)p.hc * (double)lHp - p.hcd * lbs_f);
        ad1 = (T)((double)p.hc * (double)lHp + p.hcd * lbs_f);
    }
}

template <typename T, int C>
__device__ __forceinline__ void adj_face(const AdjParams<T> &A, int i, int j, int k) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    const int idx[3] = {i, j, k};
    T a0, a1;
    adj_face_core<T, C>(A, idx, A.lpsiH[C][C1], A.lpsiH[C][C2], A.lpsiH[C][C1], A.lpsiH[C][C2], a0, a1);
    const long long q = A.p.slot(i, j, k);
    A.aD[C][0][q] = a0;
    A.aD[C][1][q] = a1;
}


template <typename T>
__global__ void __launch_bounds__(256) k_adj_face(AdjParams<T> A) {
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= A.p.n[0] || j >= A.p.n[1]) return;
    adj_face<T, 0>(A, i, j, k);
    adj_face<T, 1>(A, i, j, k);
    adj_face<T, 2>(A, i, j, k);
}

// magnetic faces: lambda of M before the map (the face kernel has added the
// B^ part); copies lMout -> lM
__global__ void __launch_bounds__(256) k_adj_film_commit(const int4 *blocktab, const FilmDev *films,
                                                         const AdjFilmDev *af) {
    const int4 bt = blocktab[blockIdx.x];
    const FilmDev &F = films[bt.x];
    const AdjFilmDev &G = af[bt.x];
    const int c = bt.y;
    const long long l = (long long)bt.z + threadIdx.x;
    if (l >= F.ns || !(F.prm[(c * 3) * F.ns + l] > 0.0)) return;
    for (int w = 0; w < 3; w++) G.lM[(c * 3 + w) * F.ns + l] = G.lMout[(c * 3 + w) * F.ns + l];
}

// face adjoints of a slot (folded; zero outside)
template <typename T>
__device__ __forceinline__ T ldD(const KParams<T> &p, const T *a, int i, int j, int k) {
    return ldz(p, a, i, j, k);
}

// lambda E += (transposed curl of E) applied to the faces' aD
template <typename T, int C>
__device__ __forceinline__ void adj_curlE(const AdjParams<T> &A, int i, int j, int k) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    const KParams<T> &p = A.p;
    // family C+1 (= C1): E_C enters its d1 along C2 ; family C+2 (= C2): its d2 along C1
    int u1[3] = {i, j, k}, u2[3] = {i, j, k};
    u1[C2] -= 1;
    u2[C1] -= 1;
    const T a1 = ldD(p, A.aD[C1][0], u1[0], u1[1], u1[2]) - ldD(p, A.aD[C1][0], i, j, k);
    const T a2 = ldD(p, A.aD[C2][1], u2[0], u2[1], u2[2]) - ldD(p, A.aD[C2][1], i, j, k);
    const long long q = p.slot(i, j, k);
    A.lE[C][q] = A.lE[C][q] + (dif(a1, T(0), p.dT[C2], p.invd[C2]) + dif(a2, T(0), p.dT[C1], p.invd[C1]));
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_curlE(AdjParams<T> A) {
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= A.p.n[0] || j >= A.p.n[1]) return;
    adj_curlE<T, 0>(A, i, j, k);
    adj_curlE<T, 1>(A, i, j, k);
    adj_curlE<T, 2>(A, i, j, k);
}

// ---------------------------------------------------------------------------
// E step: lambda E' (and psi') -> lambda E (and psi), the edge's curl-part
// adjoints eD, and dL/dca, dL/dcb
// ---------------------------------------------------------------------------
template <typename T, int C>
__device__ __forceinline__ void adj_edge(const AdjParams<T> &A, int i, int j, int k, long long step) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    const KParams<T> &p = A.p;
    const long long q = p.slot(i, j, k);
    int idx[3] = {i, j, k};
    // coefficients (zero for a PEC or wall edge: E' = 0 does not depend on anything)
    bool valid = true;
    for (int a = 0; a < 3; a++)
        if (!p.per[a] && a != C && idx[a] == 0) valid = false;
    double ca = 0.0, cb = 0.0;
    if (valid) {
        int m[4];
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int cc[3] = {i, j, k};
                cc[C1] -= 1 - u;
                cc[C2] -= 1 - v;
                for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                m[2 * u + v] = p.id[p.slot(cc[0], cc[1], cc[2])];
            }
        const MatDev &M0 = p.mat[m[0]], &M1 = p.mat[m[1]], &M2 = p.mat[m[2]], &M3 = p.mat[m[3]];
        if (M0.is_pec || M1.is_pec || M2.is_pec || M3.is_pec) {
            valid = false;
        } else {
            double se = 0.0, ss = 0.0;
            se += M0.eps_r;
            ss += M0.sigma;
            se += M1.eps_r;
            ss += M1.sigma;
            se += M2.eps_r;
            ss += M2.sigma;
            se += M3.eps_r;
            ss += M3.sigma;
            const double eps = p.eps0 * (se / 4), sig = ss / 4;
            const double den = sig / 2.0 + eps / p.dt;
            ca = -(sig / 2.0 - eps / p.dt) / den;
            cb = 1.0 / den;
        }
    }
    if (!valid) {
        A.lE[C][q] = T(0);
        A.eD[C][0][q] = T(0);
        A.eD[C][1][q] = T(0);
        return;
    }
    // forward quantities: raw curl parts of H, psi', the source
    int d1i[3] = {i, j, k}, d2i[3] = {i, j, k};
    d1i[C1] -= 1;
    d2i[C2] -= 1;
    T d1 = dif(ldz(p, p.H[C2], i, j, k), ldz(p, p.H[C2], d1i[0], d1i[1], d1i[2]), p.dT[C1], p.invd[C1]);
    T d2 = dif(ldz(p, p.H[C1], i, j, k), ldz(p, p.H[C1], d2i[0], d2i[1], d2i[2]), p.dT[C2], p.invd[C2]);
    const int a1 = idx[C1], a2 = idx[C2];
    const bool s1 = p.psiE[C][C1] && (a1 < p.nlo[C1] || a1 >= p.n[C1] - p.nhi[C1]);
    const bool s2 = p.psiE[C][C2] && (a2 < p.nlo[C2] || a2 >= p.n[C2] - p.nhi[C2]);
    long long q1 = 0, q2 = 0;
    T b1 = T(0), c1 = T(0), b2 = T(0), c2 = T(0);
    if (s1) {
        q1 = p.psi_index(C1, idx);
        b1 = p.bE[C1][a1];
        c1 = p.cE[C1][a1];
        d1 += b1 * p.psiE[C][C1][q1] + c1 * d1;
    }
    if (s2) {
        q2 = p.psi_index(C2, idx);
        b2 = p.bE[C2][a2];
        c2 = p.cE[C2][a2];
        d2 += b2 * p.psiE[C][C2][q2] + c2 * d2;
    }
    double J = 0.0;
    for (int s = 0; s < p.nsrc; s++) {
        const SrcDev &S = p.srcs[s];
        if (S.comp != C) continue;
        if (idx[0] < S.box[0] || idx[0] >= S.box[0] + S.box[3] || idx[1] < S.box[1] || idx[1] >= S.box[1] + S.box[4] ||
            idx[2] < S.box[2] || idx[2] >= S.box[2] + S.box[5])
            continue;
        if (step < S.n) J += S.table[step];
    }
    const double x = (double)(d1 - d2) - J;
    const T lEp = A.lE[C][q];
    A.gca[C][q] += (double)lEp * (double)p.E[C][q];
    A.gcb[C][q] += (double)lEp * x;
    const T lx = (T)cb * lEp;
    A.lE[C][q] = (T)ca * lEp;
    // x = (d1 + psi1') - (d2 + psi2') - J, psi' = b psi + c d
    T ad1 = lx, ad2 = -lx;
    if (s1) {
        const T aps = A.lpsiE[C][C1][q1] + lx;
        A.lpsiE[C][C1][q1] = b1 * aps;
        ad1 = lx + c1 * aps;
    }
    if (s2) {
        const T aps = A.lpsiE[C][C2][q2] - lx;
        A.lpsiE[C][C2][q2] = b2 * aps;
        ad2 = -lx + c2 * aps;
    }
    A.eD[C][0][q] = ad1;
    A.eD[C][1][q] = ad2;
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_estep(AdjParams<T> A) {
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= A.p.n[0] || j >= A.p.n[1]) return;
    const long long step = A.p.step[0];
    adj_edge<T, 0>(A, i, j, k, step);
    adj_edge<T, 1>(A, i, j, k, step);
    adj_edge<T, 2>(A, i, j, k, step);
}

// lambda H += (transposed curl of H) applied to the edges' eD
template <typename T, int C>
__device__ __forceinline__ void adj_curlH(const AdjParams<T> &A, int i, int j, int k) {
    constexpr int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    const KParams<T> &p = A.p;
    // H_C is the H_{C2} of edges E_{C1} (their d1, along C2) and the H_{C1} of
    // edges E_{C2} (their d2, along C1)
    int u1[3] = {i, j, k}, u2[3] = {i, j, k};
    u1[C2] += 1;
    u2[C1] += 1;
    const T a1 = ldz(p, A.eD[C1][0], i, j, k) - ldz(p, A.eD[C1][0], u1[0], u1[1], u1[2]);
    const T a2 = ldz(p, A.eD[C2][1], i, j, k) - ldz(p, A.eD[C2][1], u2[0], u2[1], u2[2]);
    const long long q = p.slot(i, j, k);
    A.lH[C][q] = A.lH[C][q] + (dif(a1, T(0), p.dT[C2], p.invd[C2]) + dif(a2, T(0), p.dT[C1], p.invd[C1]));
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_curlH(AdjParams<T> A) {
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= A.p.n[0] || j >= A.p.n[1]) return;
    adj_curlH<T, 0>(A, i, j, k);
    adj_curlH<T, 1>(A, i, j, k);
    adj_curlH<T, 2>(A, i, j, k);
}

// ---------------------------------------------------------------------------
// the loss: scale * (film EM energy of film f) of the current state -> its
// gradient added to lambda E, lambda H
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ bool film_cell(const KParams<T> &p, const FilmDev &F, int i, int j, int k, double &eps) {
    if (i < F.cb[0] || i >= F.cb[0] + F.cb[3] || j < F.cb[1] || j >= F.cb[1] + F.cb[4] || k < F.cb[2] ||
        k >= F.cb[2] + F.cb[5])
        return false;
    const MatDev &m = p.mat[p.id[p.slot(i, j, k)]];
    eps = m.eps_r;
    return m.Ms > 0.0;
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_loss(AdjParams<T> A, int film, double scale) {
    const KParams<T> &p = A.p;
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= p.n[0] || j >= p.n[1]) return;
    const FilmDev &F = p.films[film];
    const long long q = p.slot(i, j, k);
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        // E_C at the slot: the cells at (C1, C2) offsets -1 / 0
        double se = 0.0;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int cc[3] = {i, j, k};
                cc[C1] -= u;
                cc[C2] -= v;
                double eps;
                if (film_cell(p, F, cc[0], cc[1], cc[2], eps)) se += eps;
            }
        if (se != 0.0) A.lE[C][q] += (T)(scale * p.dV * p.eps0 * se * 0.25 * (double)p.E[C][q]);
        // H_C at the slot: the cells at C offsets -1 / 0
        int nc = 0;
        for (int u = 0; u < 2; u++) {
            int cc[3] = {i, j, k};
            cc[C] -= u;
            double eps;
            if (film_cell(p, F, cc[0], cc[1], cc[2], eps)) nc++;
        }
        if (nc) A.lH[C][q] += (T)(scale * p.dV * p.mu0 * 0.5 * nc * (double)p.H[C][q]);
    }
}

// lambda M of the initial magnetisation M0 = Ms u at every magnetic face ->
// dL/dMs of the face
__global__ void __launch_bounds__(256) k_adj_init_ms(const int4 *blocktab, const FilmDev *films,
                                                     const AdjFilmDev *af, double u0, double u1, double u2) {
    const int4 bt = blocktab[blockIdx.x];
    const FilmDev &F = films[bt.x];
    const AdjFilmDev &G = af[bt.x];
    const int c = bt.y;
    const long long l = (long long)bt.z + threadIdx.x;
    if (l >= F.ns || !(F.prm[(c * 3) * F.ns + l] > 0.0)) return;
    G.gMs[c * F.ns + l] += G.lM[(c * 3 + 0) * F.ns + l] * u0 + G.lM[(c * 3 + 1) * F.ns + l] * u1 +
                           G.lM[(c * 3 + 2) * F.ns + l] * u2;
}

// dL/d eps_r of the cells of a box from the accumulated dL/dca, dL/dcb of
// the twelve edges around each cell (eps of an edge: eps0 x the mean over
// its four cells)
template <typename T>
__global__ void __launch_bounds__(256) k_adj_eps(AdjParams<T> A, int4 b0, int4 bn, double *out) {
    const KParams<T> &p = A.p;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long ncell = (long long)bn.x * bn.y * bn.z;
    if (t >= ncell) return;
    const int ci = b0.x + (int)(t % bn.x), cj = b0.y + (int)((t / bn.x) % bn.y), ck = b0.z + (int)(t / ((long long)bn.x * bn.y));
    double g = 0.0;
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int e[3] = {ci, cj, ck};
                e[C1] += u;
                e[C2] += v;
                for (int a = 0; a < 3; a++) e[a] = fold(e[a], p.n[a], p.per[a]);
                if (e[0] < 0 || e[1] < 0 || e[2] < 0) continue;
                bool valid = true;
                for (int a = 0; a < 3; a++)
                    if (!p.per[a] && a != C && e[a] == 0) valid = false;
                if (!valid) continue;
                int m[4];
                for (int uu = 0; uu < 2; uu++)
                    for (int vv = 0; vv < 2; vv++) {
                        int cc[3] = {e[0], e[1], e[2]};
                        cc[C1] -= 1 - uu;
                        cc[C2] -= 1 - vv;
                        for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                        m[2 * uu + vv] = p.id[p.slot(cc[0], cc[1], cc[2])];
                    }
                const MatDev &M0 = p.mat[m[0]], &M1 = p.mat[m[1]], &M2 = p.mat[m[2]], &M3 = p.mat[m[3]];
                if (M0.is_pec || M1.is_pec || M2.is_pec || M3.is_pec) continue;
                const double eps = p.eps0 * ((M0.eps_r + M1.eps_r + M2.eps_r + M3.eps_r) / 4);
                const double sig = (M0.sigma + M1.sigma + M2.sigma + M3.sigma) / 4;
                const double den = sig / 2.0 + eps / p.dt;
                // ca = (eps/dt - sig/2)/den, cb = 1/den
                const double dca = (sig / p.dt) / (den * den), dcb = -(1.0 / p.dt) / (den * den);
                const long long q = p.slot(e[0], e[1], e[2]);
                g += (A.gca[C][q] * dca + A.gcb[C][q] * dcb) * (p.eps0 / 4.0);
            }
    }
    out[t] = g;
}

// the film EM energy of film f in the current state (the film-energy probe's
// sum): per-block partials, summed on the host in block order
template <typename T>
__global__ void __launch_bounds__(256) k_film_energy(KParams<T> p, int film, double *part) {
    __shared__ double red[256];
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    const int tid = threadIdx.y * 64 + threadIdx.x;
    double w = 0.0;
    const FilmDev &F = p.films[film];
    double eps;
    if (i < p.n[0] && j < p.n[1] && film_cell(p, F, i, j, k, eps)) {
        const int cc[3] = {i, j, k};
        double we = 0.0, wh = 0.0;
        for (int c = 0; c < 3; c++) {
            const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
            double e2 = 0.0;
            for (int u = 0; u < 2; u++)
                for (int v = 0; v < 2; v++) {
                    int q[3] = {cc[0], cc[1], cc[2]};
                    q[c1] += u;
                    q[c2] += v;
                    const double e = (double)ldz(p, p.E[c], q[0], q[1], q[2]);
                    e2 += e * e;
                }
            we += e2 / 4.0;
            double h2 = 0.0;
            for (int u = 0; u < 2; u++) {
                int q[3] = {cc[0], cc[1], cc[2]};
                q[c] += u;
                const double h = (double)ldz(p, p.H[c], q[0], q[1], q[2]);
                h2 += h * h;
            }
            wh += h2 / 2.0;
        }
        w = (0.5 * p.eps0 * eps * we + 0.5 * p.mu0 * wh) * p.dV;
    }
    red[tid] = w;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) part[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)] = red[0];
}

__global__ void k_set_step(long long *step, long long v) {
    if (threadIdx.x == 0) step[0] = v;
}

// acc += scale * (sum of the partials in order), one thread: deterministic
__global__ void k_accum(const double *part, int n, double *acc, double scale) {
    if (threadIdx.x != 0) return;
    double s = 0.0;
    for (int q = 0; q < n; q++) s += part[q];
    acc[0] += scale * s;
}

// ---------------------------------------------------------------------------
// tape schedule
// ---------------------------------------------------------------------------

// region index of the slot e (unfolded, inside [b0, b0 + r) or its wrap), -1
// for no slot
__device__ __forceinline__ long long region_index(const int *n, const int *per, const int *b0, const int *r,
                                                  const int *e) {
    int loc[3];
    for (int a = 0; a < 3; a++) {
        int v = e[a];
        if (v >= n[a]) {
            if (!per[a]) return -1;
            if (v - n[a] >= b0[a]) v -= n[a];
        }
        loc[a] = v - b0[a];
        if (loc[a] < 0 || loc[a] >= r[a]) return -1;
    }
    return (long long)loc[0] + (long long)r[0] * ((long long)loc[1] + (long long)r[1] * loc[2]);
}

template <typename T>
__global__ void __launch_bounds__(256) k_tape_loss(KParams<T> p, int film, int merged, double *dst) {
    tape_loss_body(p, film, merged, dst, blockIdx.x);
}

// the loss term of the state a tape slot holds: scale x the gradient of the
// film EM energy added to lambda E and lambda H; no-op unless the slot's
// time index seg0 + m is past loss_from (seg0 null: always)
template <typename T>
__global__ void __launch_bounds__(256) k_adj_loss_tape(AdjParams<T> A, int film, double scale, const double *tape,
                                                       const long long *seg0, int m, long long loss_from) {
    if (seg0 && seg0[0] + m <= loss_from) return;
    const KParams<T> &p = A.p;
    const FilmDev &F = p.films[film];
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long tb = (long long)r[0] * r[1] * r[2];
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    int q[3];
    if (t >= tb || !region_slot(p.n, p.per, b0, r, t, q)) return;
    const long long sl = p.slot(q[0], q[1], q[2]);
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        double se = 0.0, eps;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int cc[3] = {q[0], q[1], q[2]};
                cc[C1] -= u;
                cc[C2] -= v;
                for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                if (cc[0] >= 0 && cc[1] >= 0 && cc[2] >= 0 && film_cell(p, F, cc[0], cc[1], cc[2], eps)) se += eps;
            }
        if (se != 0.0) A.lE[C][sl] += (T)(scale * p.dV * p.eps0 * se * 0.25 * tape[C * tb + t]);
        int nc = 0;
        for (int u = 0; u < 2; u++) {
            int cc[3] = {q[0], q[1], q[2]};
            cc[C] -= u;
            for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
            if (cc[0] >= 0 && cc[1] >= 0 && cc[2] >= 0 && film_cell(p, F, cc[0], cc[1], cc[2], eps)) nc++;
        }
        if (nc) A.lH[C][sl] += (T)(scale * p.dV * p.mu0 * 0.5 * nc * tape[(3 + C) * tb + t]);
    }
}

// The loss's own dependence on eps_r: the film energy holds
// 1/2 eps0 eps_r dV times the mean over its four edges of E_C^2 (summed over
// C) for each film cell, so dL/d eps_r of a film cell collects that sum of
// every state in the loss window, x scale.  acc is [film cell box] (x
// fastest).  From a film-region tape slot (seg0 null: always; else only when
// seg0 + m is past loss_from) ...
template <typename T>
__global__ void __launch_bounds__(256) k_adj_loss_eps_tape(KParams<T> p, int film, double scale, const double *tape,
                                                           const long long *seg0, int m, long long loss_from,
                                                           double *acc) {
    if (seg0 && seg0[0] + m <= loss_from) return;
    const FilmDev &F = p.films[film];
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long tb = (long long)r[0] * r[1] * r[2];
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= (long long)F.cb[3] * F.cb[4] * F.cb[5]) return;
    const int cell[3] = {F.cb[0] + (int)(t % F.cb[3]), F.cb[1] + (int)((t / F.cb[3]) % F.cb[4]),
                         F.cb[2] + (int)(t / ((long long)F.cb[3] * F.cb[4]))};
    double eps;
    if (!film_cell(p, F, cell[0], cell[1], cell[2], eps)) return;
    double we = 0.0;
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        double e2 = 0.0;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int e[3] = {cell[0], cell[1], cell[2]};
                e[C1] += u;
                e[C2] += v;
                const long long ri = region_index(p.n, p.per, b0, r, e);
                if (ri < 0) continue; // a wall edge: E = 0
                const double x = tape[C * tb + ri];
                e2 += x * x;
            }
        we += e2 / 4.0;
    }
    acc[t] += scale * 0.5 * p.eps0 * p.dV * we;
}

// ... or from the current state (the plain schedule)
template <typename T>
__global__ void __launch_bounds__(256) k_adj_loss_eps_state(KParams<T> p, int film, double scale, double *acc) {
    const FilmDev &F = p.films[film];
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= (long long)F.cb[3] * F.cb[4] * F.cb[5]) return;
    const int cell[3] = {F.cb[0] + (int)(t % F.cb[3]), F.cb[1] + (int)((t / F.cb[3]) % F.cb[4]),
                         F.cb[2] + (int)(t / ((long long)F.cb[3] * F.cb[4]))};
    double eps;
    if (!film_cell(p, F, cell[0], cell[1], cell[2], eps)) return;
    double we = 0.0;
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        double e2 = 0.0;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int q[3] = {cell[0], cell[1], cell[2]};
                q[C1] += u;
                q[C2] += v;
                const double x = (double)ldz(p, p.E[C], q[0], q[1], q[2]);
                e2 += x * x;
            }
        we += e2 / 4.0;
    }
    acc[t] += scale * 0.5 * p.eps0 * p.dV * we;
}

// dL/d eps_r of the box's cells from the box accumulators (eps of an edge:
// eps0 x the mean over its four cells)
template <typename T>
__global__ void __launch_bounds__(256) k_adj_eps_box(KParams<T> p, int4 bb, int4 bs, const double *gca,
                                                     const double *gcb, double *out) {
    const int b0[3] = {bb.x, bb.y, bb.z}, r[3] = {bs.x + 1, bs.y + 1, bs.z + 1};
    const long long tb = (long long)r[0] * r[1] * r[2];
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long ncell = (long long)bs.x * bs.y * bs.z;
    if (t >= ncell) return;
    const int cell[3] = {bb.x + (int)(t % bs.x), bb.y + (int)((t / bs.x) % bs.y),
                         bb.z + (int)(t / ((long long)bs.x * bs.y))};
    double g = 0.0;
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        for (int u = 0; u < 2; u++)
            for (int v = 0; v < 2; v++) {
                int e[3] = {cell[0], cell[1], cell[2]};
                e[C1] += u;
                e[C2] += v;
                const long long ri = region_index(p.n, p.per, b0, r, e);
                if (ri < 0) continue;
                int f[3];
                for (int a = 0; a < 3; a++) f[a] = fold(e[a], p.n[a], p.per[a]);
                bool valid = true;
                for (int a = 0; a < 3; a++)
                    if (!p.per[a] && a != C && f[a] == 0) valid = false;
                if (!valid) continue;
                double se = 0.0, ss = 0.0;
                bool pec = false;
                for (int uu = 0; uu < 2; uu++)
                    for (int vv = 0; vv < 2; vv++) {
                        int cc[3] = {f[0], f[1], f[2]};
                        cc[C1] -= 1 - uu;
                        cc[C2] -= 1 - vv;
                        for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                        const MatDev &M = p.mat[p.id[p.slot(cc[0], cc[1], cc[2])]];
                        pec = pec || M.is_pec;
                        se += M.eps_r;
                        ss += M.sigma;
                    }
                if (pec) continue;
                const double eps = p.eps0 * (se / 4), sig = ss / 4;
                const double den = sig / 2.0 + eps / p.dt;
                const double dca = (sig / p.dt) / (den * den), dcb = -(1.0 / p.dt) / (den * den);
                g += (gca[C * tb + ri] * dca + gcb[C * tb + ri] * dcb) * (p.eps0 / 4.0);
            }
    }
    out[t] = g;
}

// ---------------------------------------------------------------------------
// fused schedule: one stencil pass per transposed map
// ---------------------------------------------------------------------------

// E-step coefficients of the edge of family C at slot idx (in the domain):
// ok = false for an edge on a lower wall or with a PEC cell (E' = 0).  The
// mixed-slot case is out of line with scalar arguments (a reference to the
// kernel's parameter block would make the compiler copy it to scratch).
template <typename T>
struct EdgeCoef {
    T ca, cb;
    bool ok;
};

template <typename T>
__device__ __forceinline__ EdgeCoef<T> edge_coef_mixed(const uint8_t *id, const MatDev *mat, int n0, int n1, int n2,
                                                     int per0, int per1, int per2, int px, double eps0, double dt,
                                                     int C, int i, int j, int k) {
    const int n[3] = {n0, n1, n2}, per[3] = {per0, per1, per2};
    const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
    double se = 0.0, ss = 0.0;
    EdgeCoef<T> r{T(0), T(0), false};
    for (int u = 0; u < 2; u++)
        for (int v = 0; v < 2; v++) {
            int cc[3] = {i, j, k};
            cc[C1] -= 1 - u;
            cc[C2] -= 1 - v;
            for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], n[a], per[a]);
            const MatDev &M = mat[id[(long long)cc[0] + (long long)px * ((long long)cc[1] + (long long)n1 * cc[2])]];
            if (M.is_pec) return r;
            se += M.eps_r;
            ss += M.sigma;
        }
    const double eps = eps0 * (se / 4), sig = ss / 4;
    const double den = sig / 2.0 + eps / dt;
    r.ca = (T)(-(sig / 2.0 - eps / dt) / den);
    r.cb = (T)(1.0 / den);
    r.ok = true;
    return r;
}

// the E-step coefficients of a slot's three edges: its class (the 16-bit one
// on a grid with extended triples), then the class's packed row in one or two
// wide loads (a PEC edge has ca = cb = 0, every other edge cb > 0)
struct EdgeRow {
    int c;
    bool mixed; // on the mixed list: the general path from the cell ids
};

template <typename T>
__device__ __forceinline__ EdgeRow edge_class(const KParams<T> &p, int i, int j, int k, long long zo) {
    const unsigned o = (unsigned)i + (unsigned)j * (unsigned)p.px;
    EdgeRow e;
    if (p.cls16) { // uniform
        e.c = row_ld(p.cls16 + zo, 2u * o);
        e.mixed = e.c == 0xffff;
    } else {
        e.c = row_ld(p.cls + zo, o);
        e.mixed = e.c == kMixed;
    }
    return e;
}

template <typename T>
__device__ __forceinline__ void edge_row_coefs(const KParams<T> &p, const EdgeRow &e, int i, int j, int k, T *ca,
                                               T *cb, bool *ok) {
    // one class for the whole wavefront: its row through the scalar cache
    CoefRow<T> r;
    const int cu = __builtin_amdgcn_readfirstlane(e.c);
    if (__builtin_amdgcn_ballot_w64(e.c != cu || e.mixed) == 0) {
        const T *q = p.coefv + kCoefRow<T> * (long long)cu;
#pragma unroll
        for (int C = 0; C < 3; C++) {
            r.ca[C] = scalar_ld(q, 2 * C);
            r.cb[C] = scalar_ld(q, 2 * C + 1);
        }
    } else {
        r = coef_row<T>(p.coefv, e.mixed ? 0 : e.c);
    }
    // an edge on a lower wall (a non-periodic axis other than its own) is held
    // at zero; a mixed slot's edges read the four cells around them, which
    // exist off the walls only
    const bool ox = i > 0 || p.per[0], oy = j > 0 || p.per[1], oz = k > 0 || p.per[2];
    const bool off[3] = {oy && oz, ox && oz, ox && oy};
#pragma unroll
    for (int C = 0; C < 3; C++) {
        ca[C] = r.ca[C];
        cb[C] = r.cb[C];
        ok[C] = off[C] && r.cb[C] != T(0);
    }
    if (e.mixed) {
        for (int C = 0; C < 3; C++) {
            ok[C] = false;
            if (!off[C]) continue;
            const EdgeCoef<T> m = edge_coef_mixed<T>(p.id, p.mat, p.n[0], p.n[1], p.n[2], p.per[0], p.per[1],
                                                     p.per[2], p.px, p.eps0, p.dt, C, i, j, k);
            ca[C] = m.ca;
            cb[C] = m.cb;
            ok[C] = m.ok;
        }
    }
}

// the first film whose reach holds the face slot idx, its region index lr
template <typename T>
__device__ __forceinline__ int first_region(const AdjParams<T> &A, const int *idx, long long &lr) {
    for (int f = 0; f < A.p.nfilm; f++) {
        const AdjFilmDev G = scalar_desc(A.af, f);
        const int r0 = idx[0] - G.r0[0], r1 = idx[1] - G.r0[1], r2 = idx[2] - G.r0[2];
        if (r0 >= 0 && r0 < G.rn[0] && r1 >= 0 && r1 < G.rn[1] && r2 >= 0 && r2 < G.rn[2]) {
            lr = (long long)r0 + (long long)G.rn[0] * ((long long)r1 + (long long)G.rn[1] * r2);
            return f;
        }
    }
    return -1;
}

// region index of the folded slot t in the region [b0, b0 + r) (which may
// wrap on a periodic axis), -1 outside
__device__ __forceinline__ long long region_index_folded(const int *n, const int *per, const int *b0, const int *r,
                                                         const int *t) {
    long long li = 0, mul = 1;
    for (int a = 0; a < 3; a++) {
        int loc = t[a] - b0[a];
        if (loc < 0 && per[a]) loc += n[a];
        if (loc < 0 || loc >= r[a]) return -1;
        li += mul * loc;
        mul *= r[a];
    }
    return li;
}

// the loss term's lambda H part (film-energy gradient of the state at the
// step's start, scaled) of the face of family C at slot idx, zero off the
// film's cells; used where the merged field pass takes the lambda E part
template <typename T>
__device__ __forceinline__ T face_loss(const AdjParams<T> &A, int C, const int *idx) {
    const KParams<T> &p = A.p;
    const FilmDev F = film_desc(p.films, A.lfilm);
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long ri = region_index_folded(p.n, p.per, b0, r, idx);
    const long long tb = (long long)r[0] * r[1] * r[2], o = (3 + C) * tb + (ri < 0 ? 0 : ri);
    const double nc = A.lw[o], x = A.ltape[o];
    return ri < 0 || nc == 0.0 ? T(0) : (T)(A.lscale * p.dV * p.mu0 * 0.5 * nc * x);
}

// adj_face_core for a face of family C at slot idx inside the reach of film F
// that no other film's reach meets (G.alone), off the CPML slabs: only this
// film's faces matter, and every load goes out at once (a face outside the
// face box reads its element 0, and what it does not use is dropped)
template <typename T, int C>
__device__ __forceinline__ void adj_face_alone(const AdjParams<T> &A, const FilmDev &F, const AdjFilmDev &G,
                                               const int *idx, T loss, T &ad0, T &ad1) {
    const KParams<T> &p = A.p;
    const long long q = p.slot(idx[0], idx[1], idx[2]);
    double lHp = (double)A.lH[C][q];
    bool in0;
    const long long lm = film_local<T>(F, idx, in0);
    double own = F.prm[(C * 3) * F.ns + lm], olp = G.lp[(C * 3 + C) * F.ns + lm], olq = G.lq[(C * 3 + C) * F.ns + lm],
           omo = G.lMout[(C * 3 + C) * F.ns + lm];
    // the magnetic faces s = t + a e_cs - b e_C of each other family cs with
    // this face in their four-face mean
    double tms[2][2][2], tlp[2][2][2], tlq[2][2][2];
    bool tin[2][2][2];
#pragma unroll
    for (int v = 0; v < 2; v++) {
        // families in the order of adj_face_core: the lower of the two first
        const int cs = v == 0 ? (C == 0 ? 1 : 0) : (C == 2 ? 1 : 2);
#pragma unroll
        for (int aa = 0; aa < 2; aa++)
#pragma unroll
            for (int bb = 0; bb < 2; bb++) {
                int s[3] = {idx[0], idx[1], idx[2]};
                s[cs] = fold(s[cs] + aa, p.n[cs], p.per[cs]);
                s[C] = fold(s[C] - bb, p.n[C], p.per[C]);
                bool in;
                const long long ls = film_local<T>(F, s, in); // false for a folded -1 too
                tin[v][aa][bb] = in;
                tms[v][aa][bb] = F.prm[(cs * 3) * F.ns + ls];
                tlp[v][aa][bb] = G.lp[(cs * 3 + C) * F.ns + ls];
                tlq[v][aa][bb] = G.lq[(cs * 3 + C) * F.ns + ls];
            }
    }
    hold(lHp);
    hold(own);
    hold(olp);
    hold(olq);
    hold(omo);
#pragma unroll
    for (int v = 0; v < 8; v++) {
        hold((&tms[0][0][0])[v]);
        hold((&tlp[0][0][0])[v]);
        hold((&tlq[0][0][0])[v]);
    }
    const bool mag = in0 && own > 0.0;
    double lbs_f = 0.0, lbn = 0.0;
    if (mag) {
        lbs_f += olp;
        lbn += olq;
    }
#pragma unroll
    for (int v = 0; v < 2; v++)
#pragma unroll
        for (int aa = 0; aa < 2; aa++)
#pragma unroll
            for (int bb = 0; bb < 2; bb++)
                if (tin[v][aa][bb] && tms[v][aa][bb] > 0.0) {
                    lbs_f += 0.25 * tlp[v][aa][bb];
                    lbn += 0.25 * tlq[v][aa][bb];
                }
    if (mag) {
        const double lbs = lHp + lbs_f;
        const double lbt = lbn + lbs;
        A.lH[C][q] = (T)lbt + loss;
        G.lMout[(C * 3 + C) * F.ns + lm] = omo + lbt;
        ad0 = (T)(-p.hcd * lbs);
        ad1 = (T)(p.hcd * lbs);
    } else {
        A.lH[C][q] = (T)(lHp + lbn + lbs_f) + loss;
        ad0 = (T)(-(double)p.hc * lHp - p.hcd * lbs_f);
        ad1 = (T)((double)p.hc * lHp + p.hcd * lbs_f);
    }
}

// the film region's faces: the general face adjoint (magnetic faces, faces
// the solves read), lambda H and lambda M updated in place, the curl-part
// adjoints stored for the field pass.  A film apart from the others and off
// the slabs (G.alone, decided once by the host) takes the straight-line form:
// the general one's film loop and tests put up to eleven round trips in a row
// (12.4 us on the reach of a 64 x 12 x 4 film, 19.6 us of 256 x 48 x 4; 4.9
// and 9.8 us without them)
template <typename T>
__global__ void __launch_bounds__(256) k_adj_film_faces(AdjParams<T> A, int f) {
    const AdjFilmDev G = scalar_desc(A.af, f);
    const FilmDev FD = film_desc(A.p.films, f);
    const unsigned lr = blockIdx.x * 256u + threadIdx.x;
    if (lr >= (unsigned)G.nr) return;
    int idx[3];
    box_split(lr, G.rn, idx);
    for (int a = 0; a < 3; a++) idx[a] += G.r0[a];
    // one face family per grid row
    T a0, a1, loss = T(0);
    const int F = blockIdx.y;
    if (A.loss_h && A.seg0[0] + A.m > A.loss_from) loss = face_loss(A, F, idx);
    if (G.alone) {
        if (F == 0)
            adj_face_alone<T, 0>(A, FD, G, idx, loss, a0, a1);
        else if (F == 1)
            adj_face_alone<T, 1>(A, FD, G, idx, loss, a0, a1);
        else
            adj_face_alone<T, 2>(A, FD, G, idx, loss, a0, a1);
        G.aDr[(2 * F) * G.nr + lr] = (double)a0;
        G.aDr[(2 * F + 1) * G.nr + lr] = (double)a1;
        return;
    }
    long long l2;
    if (first_region(A, idx, l2) != f) return;
    if (F == 0)
        adj_face_core<T, 0>(A, idx, A.lpsiH[0][1], A.lpsiH[0][2], A.lpsiHo[0][1], A.lpsiHo[0][2], a0, a1);
    else if (F == 1)
        adj_face_core<T, 1>(A, idx, A.lpsiH[1][2], A.lpsiH[1][0], A.lpsiHo[1][2], A.lpsiHo[1][0], a0, a1);
    else
        adj_face_core<T, 2>(A, idx, A.lpsiH[2][0], A.lpsiH[2][1], A.lpsiHo[2][0], A.lpsiHo[2][1], a0, a1);
    if (loss != T(0)) A.lH[F][A.p.slot(idx[0], idx[1], idx[2])] += loss;
    G.aDr[(2 * F) * G.nr + lr] = (double)a0;
    G.aDr[(2 * F + 1) * G.nr + lr] = (double)a1;
}

// the weights of the film-energy gradient over the loss film's region (its
// cell box grown by one slot), once per adjoint run: [6][region], the sum of
// eps_r over the film cells that share the E_C edge, the number of them that
// share the H_C face
template <typename T>
__global__ void __launch_bounds__(256) k_adj_loss_weights(KParams<T> p, int film, double *dst) {
    const FilmDev F = film_desc(p.films, film);
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long tb = (long long)r[0] * r[1] * r[2];
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    if (t >= tb) return;
    int q[3];
    const bool slot = region_slot(p.n, p.per, b0, r, t, q);
    for (int C = 0; C < 3; C++) {
        const int C1 = (C + 1) % 3, C2 = (C + 2) % 3;
        double se = 0.0, eps;
        int nc = 0;
        if (slot) {
            for (int u = 0; u < 2; u++)
                for (int v = 0; v < 2; v++) {
                    int cc[3] = {q[0], q[1], q[2]};
                    cc[C1] -= u;
                    cc[C2] -= v;
                    for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                    if (cc[0] >= 0 && cc[1] >= 0 && cc[2] >= 0 && film_cell(p, F, cc[0], cc[1], cc[2], eps)) se += eps;
                }
            for (int u = 0; u < 2; u++) {
                int cc[3] = {q[0], q[1], q[2]};
                cc[C] -= u;
                for (int a = 0; a < 3; a++) cc[a] = fold(cc[a], p.n[a], p.per[a]);
                if (cc[0] >= 0 && cc[1] >= 0 && cc[2] >= 0 && film_cell(p, F, cc[0], cc[1], cc[2], eps)) nc++;
            }
        }
        dst[C * tb + t] = se;
        dst[(3 + C) * tb + t] = (double)nc;
    }
}

// the loss term of the state at the start of the step (film-energy
// gradient, scaled) for the slot t: added to its three lambda E values (in
// registers) and to lambda H of its three faces (film faces: no other thread
// of the pass reads them)
// (PART: 0 both terms, 1 the lambda E term only)
template <typename T, int PART = 0>
__device__ __forceinline__ void loss_term(const AdjParams<T> &A, const int *t, long long q, T &l0, T &l1, T &l2) {
    const KParams<T> &p = A.p;
    const FilmDev F = film_desc(p.films, A.lfilm);
    const int b0[3] = {F.cb[0], F.cb[1], F.cb[2]}, r[3] = {F.cb[3] + 1, F.cb[4] + 1, F.cb[5] + 1};
    const long long ri = region_index_folded(p.n, p.per, b0, r, t);
    if (ri < 0) return;
    const long long tb = (long long)r[0] * r[1] * r[2];
    T le[3] = {l0, l1, l2};
#pragma unroll
    for (int C = 0; C < 3; C++) {
        {
            const double se = A.lw[C * tb + ri], x = A.ltape[C * tb + ri];
            const T v = (T)(A.lscale * p.dV * p.eps0 * se * 0.25 * x);
            le[C] = se != 0.0 ? le[C] + v : le[C];
        }
        if (PART != 1) {
            const double nc = A.lw[(3 + C) * tb + ri], x = A.ltape[(3 + C) * tb + ri];
            const T h = A.lH[C][q];
            const T v = (T)(A.lscale * p.dV * p.mu0 * 0.5 * nc * x);
            if (nc != 0.0) A.lH[C][q] = h + v;
        }
    }
    l0 = le[0];
    l1 = le[1];
    l2 = le[2];
}

// the flag byte of this block's tile, read through the scalar cache (the
// aligned word that holds it; the table is whole words), so that the wait for
// it does not hold vector loads issued before its first use
__device__ __forceinline__ int adj_tile_flag(const uint8_t *tab) {
    typedef __attribute__((address_space(4))) const uint32_t cword;
    const unsigned ti = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const uint32_t w = ((cword *)tab)[ti >> 2];
    return (int)((w >> (8 * (ti & 3))) & 0xffu);
}

// ---------------------------------------------------------------------------
// the field passes of the tape schedule, by wavefront rows (rows.h): each of
// the six differences of a transposed curl runs along one axis and is
// stretched by that axis's CPML alone, so a row's y and z slabs are uniform
// and only the x slab is a lane's matter
// ---------------------------------------------------------------------------

// the adjoint psi of a wavefront's slots and of their neighbours one slot off
// (D = -1: faces below; +1: edges above) along one axis, for the two
// components that differentiate along it
template <typename T>
struct AdjAxis {
    bool s = false, sn = false; // in a slab: the slot, its neighbour (x: per lane; y, z: uniform)
    T b = T(0), c = T(0), bn = T(0), cn = T(0);
    T pa = T(0), pan = T(0), pb = T(0), pbn = T(0); // psi of the components axis + 1 and axis + 2
    unsigned o = 0;                                 // byte offset of the slot's psi in its row
    long long q = 0;                                // first element of that row
};

template <typename T>
__device__ __forceinline__ unsigned x_psi_off(const KParams<T> &p, int i, bool in) {
    const int sp = i < p.nlo[0] ? i : p.nlo[0] + (i - (p.n[0] - p.nhi[0]));
    return (unsigned)(in ? sp : 0) * (unsigned)sizeof(T);
}

// pa, pb: the psi arrays (null without slabs on the axis); bt, ct: the
// recursion's tables; io: the lane's byte offset in a padded row
template <typename T, int D>
__device__ __forceinline__ void adj_axis_x(const KParams<T> &p, const RowPos &r, const T *pa, const T *pb, const T *bt,
                                           const T *ct, AdjAxis<T> &m) {
    if (p.nlo[0] + p.nhi[0] == 0) return;
    if (!(r.w0 + (D < 0 ? D : 0) < p.nlo[0] || r.w0 + 63 + (D > 0 ? D : 0) >= p.n[0] - p.nhi[0])) return; // uniform
    const int i = min(r.i, p.n[0] - 1), in = i + D;
    m.s = in_slab(p, 0, i);
    m.sn = in >= 0 && in < p.n[0] && in_slab(p, 0, in);
    m.q = row_psi(p, 0, r.j, r.k);
    m.o = x_psi_off(p, i, m.s);
    const unsigned on = x_psi_off(p, in, m.sn), es = (unsigned)sizeof(T);
    const unsigned io = (unsigned)i * es, inn = (unsigned)(m.sn ? in : i) * es;
    m.pa = row_ld(pa + m.q, m.o);
    m.pan = row_ld(pa + m.q, on);
    m.pb = row_ld(pb + m.q, m.o);
    m.pbn = row_ld(pb + m.q, on);
    m.b = row_ld(bt, io);
    m.c = row_ld(ct, io);
    m.bn = row_ld(bt, inn);
    m.cn = row_ld(ct, inn);
}

template <typename T, int D, int W>
__device__ __forceinline__ void adj_axis_yz(const KParams<T> &p, const RowPos &r, const T *pa, const T *pb,
                                            const T *bt, const T *ct, unsigned io, AdjAxis<T> &m) {
    if (p.nlo[W] + p.nhi[W] == 0) return;
    const int x = W == 1 ? r.j : r.k, xn = x + D;
    m.s = in_slab(p, W, x);
    m.sn = xn >= 0 && xn < p.n[W] && in_slab(p, W, xn);
    m.o = io;
    if (m.s) {
        m.q = row_psi(p, W, r.j, r.k);
        m.pa = row_ld(pa + m.q, io);
        m.pb = row_ld(pb + m.q, io);
        m.b = scalar_ld(bt, x);
        m.c = scalar_ld(ct, x);
    }
    if (m.sn) {
        const long long qn = W == 1 ? row_psi(p, W, xn, r.k) : row_psi(p, W, r.j, xn);
        m.pan = row_ld(pa + qn, io);
        m.pbn = row_ld(pb + qn, io);
        m.bn = scalar_ld(bt, xn);
        m.cn = scalar_ld(ct, xn);
    }
}

// the curl-part adjoint of a face from g = -/+ hc lambda H through its CPML
// recursion (a: the first half step transposed; with PAIR the psi goes on
// through the second, h); ps becomes the psi after the maps
template <typename T, bool PAIR>
__device__ __forceinline__ void adj_stretch(bool s, T g, T b, T c, T &ps, T &a, T &h) {
    a = h = g;
    const T aps = ps + g;
    const T a1 = g + c * aps;
    T out = b * aps, h1 = g;
    if (PAIR) {
        const T aps2 = b * aps + g;
        h1 = g + c * aps2;
        out = b * aps2;
    }
    a = s ? a1 : a;
    h = s ? h1 : h;
    ps = s ? out : ps;
}

// what a half-step field pass runs: the second half step of a step transposed
// (writes mu for the E step's transpose), the first (scaling lambda E by ca
// before, with the eps-box sums and the loss of the step's input state), or
// the first of step m and the second of step m - 1 together
enum { HF_SECOND = 0, HF_FIRST = 1, HF_PAIR = 2 };

// inside a film's reach the curl-part adjoints come from the tables of the film
// kernels: part w (2 F + part) of the slot's own face (o, h: of the first and
// the second half step) and of the one before it along axis AX (n, hn).  The
// first film that holds a face counts; returns whether one holds the slot's.
template <typename T, bool PAIR, int AX>
__device__ __forceinline__ bool film_part_values(const RowPos &r, int w, T &o, T &n, T &h, T &hn) {
    const AdjParams<T> &A = args_again<AdjParams<T>>();
    const KParams<T> &p = A.p;
    int nb[3] = {r.i, r.j, r.k};
    nb[AX] = nb[AX] > 0 ? nb[AX] - 1 : (p.per[AX] ? p.n[AX] - 1 : -1);
    bool own = false;
    for (int f = p.nfilm - 1; f >= 0; f--) {
        const AdjFilmDev G = scalar_desc(A.af, f);
        const double *t2 = G.aDr;
        if (PAIR) t2 = scalar_desc(A.afb, f).aDr;
        const int x = r.i - G.r0[0], y = r.j - G.r0[1], z = r.k - G.r0[2];
        const int xn = nb[0] - G.r0[0], yn = nb[1] - G.r0[1], zn = nb[2] - G.r0[2];
        const bool in = r.in && y >= 0 && y < G.rn[1] && z >= 0 && z < G.rn[2] && x >= 0 && x < G.rn[0];
        const bool inn = r.in && yn >= 0 && yn < G.rn[1] && zn >= 0 && zn < G.rn[2] && xn >= 0 && xn < G.rn[0];
        // a reach holds fewer than 2^31 sites; all four loads go out at once,
        // at a part's first site where the face is outside (then dropped)
        const int q = in ? x + G.rn[0] * (y + G.rn[1] * z) : 0, qn = inn ? xn + G.rn[0] * (yn + G.rn[1] * zn) : 0;
        const double *d = G.aDr + w * G.nr, *d2 = t2 + w * G.nr;
        const T vo = (T)d[q], vn = (T)d[qn], vh = PAIR ? (T)d2[q] : T(0), vhn = PAIR ? (T)d2[qn] : T(0);
        o = in ? vo : o;
        n = inn ? vn : n;
        if (PAIR) {
            h = in ? vh : h;
            hn = inn ? vhn : hn;
        }
        own = own || in;
    }
    return own;
}

// the transposed half step(s) on the E side: lambda E_C += the transposed curl
// of the faces' curl-part adjoints.  Six differences, by face family F and part
// (index 2 F + part; part 0 runs along axis F + 1, part 1 along F + 2), each of
// the slot's face and the one before it along that axis.
// One pass for HF_PAIR: non-film faces see the same lambda H in both maps, the
// film region's come from the film kernels' tables; every value follows the
// two single passes' operation sequence, so the results are theirs, bitwise
// (only where no film's reach meets a CPML slab: the film-region kernels keep
// their psi per half step).
// HF_PAIR moves 49 bytes a slot in float32 (lambda E, lambda H, the class in;
// lambda E, mu out) and 16 a slab slot and axis: 175 us on a 512 x 256 x 128 grid
// with CPML 10 at the rate of a copy.  With each slot walking its faces'
// recursions by branches it took 390 us (252 vector instructions and nine
// dependent psi fetches a wavefront); by rows 211 us, with the tables of a film
// tile in one round trip a difference, one class's coefficients through the
// scalar cache and the last part's arguments fetched there (92 scalar registers
// had gone through vector lanes, now 20) 193; 128 x 64 x 64 15.7 -> 13.6 us, 96 x
// 64 x 48 float64 17.2 -> 15.8.
template <typename T, int MODE, int TX, int TY>
__global__ void __launch_bounds__(256) k_adj_hfield(AdjParams<T> A) {
    constexpr bool PAIR = MODE == HF_PAIR;
    const KParams<T> &p = A.p;
    const RowPos r = row_pos<TX>(p.n, blockIdx.x, blockIdx.y, TY, blockIdx.z);
    if (r.j >= p.n[1]) return;
    const unsigned es = (unsigned)sizeof(T);
    const int ic = min(r.i, p.n[0] - 1), j = r.j, k = r.k;
    const long long sz = (long long)p.px * p.n[1];
    const unsigned io = (unsigned)ic * es, rowb = (unsigned)p.px * es, vo = io + (unsigned)j * rowb;
    const bool okx = ic > 0 || p.per[0], oky = j > 0 || p.per[1], okz = k > 0 || p.per[2];
    const unsigned vxm = ic > 0 ? vo - es : (p.per[0] ? vo + (unsigned)(p.n[0] - 1) * es : vo);
    const unsigned vym = io + (unsigned)(j > 0 ? j - 1 : (p.per[1] ? p.n[1] - 1 : j)) * rowb;
    const long long zo = k * sz, zb = (k > 0 ? k - 1 : (p.per[2] ? p.n[2] - 1 : k)) * sz;
    const EdgeRow e = edge_class(p, ic, j, k, zo);
    const T *Hx = A.lH[0] + zo, *Hy = A.lH[1] + zo, *Hz = A.lH[2] + zo;
    const T x0 = row_ld(Hx, vo), x_z = row_ld(A.lH[0] + zb, vo), x_y = row_ld(Hx, vym);
    const T y0 = row_ld(Hy, vo), y_z = row_ld(A.lH[1] + zb, vo), y_x = row_ld(Hy, vxm);
    const T z0 = row_ld(Hz, vo), z_x = row_ld(Hz, vxm), z_y = row_ld(Hz, vym);
    // the slot's lambda E is touched once per pass: non-temporal (the lambda
    // H the neighbouring slots read again stays in L2)
    T *Ex = A.lE[0] + zo, *Ey = A.lE[1] + zo, *Ez = A.lE[2] + zo;
    T l[3] = {row_ld<true>(Ex, vo), row_ld<true>(Ey, vo), row_ld<true>(Ez, vo)};
    AdjAxis<T> ax, ay, az;
    adj_axis_x<T, -1>(p, r, A.lpsiH[1][0], A.lpsiH[2][0], p.bH[0], p.cH[0], ax);
    adj_axis_yz<T, -1, 1>(p, r, A.lpsiH[2][1], A.lpsiH[0][1], p.bH[1], p.cH[1], io, ay);
    adj_axis_yz<T, -1, 2>(p, r, A.lpsiH[0][2], A.lpsiH[1][2], p.bH[2], p.cH[2], io, az);
    T ca[3], cb[3];
    bool ok[3];
    edge_row_coefs<T>(p, e, ic, j, k, ca, cb, ok);
    // the differences one by one (a film tile's table values are then not all
    // live at once): part 0 takes -hc lambda H, part 1 +hc lambda H
    const T hn = -p.hc, hp = p.hc;
    const int fl = p.nfilm ? adj_tile_flag(A.aflags) : 0;
    bool film_own = false;
#define MPX_DIFF(AX, W, HC, V0, VN, M, PS, PSN, OK, D, E)                                              \
    {                                                                                                  \
        T o = (HC) * (V0), n = (HC) * (VN), h = o, g = n;                                              \
        if (AX == 0) {                                                                                 \
            if (M.s || M.sn) {                                                                         \
                adj_stretch<T, PAIR>(M.s, o, M.b, M.c, M.PS, o, h);                                    \
                adj_stretch<T, PAIR>(M.sn, n, M.bn, M.cn, M.PSN, n, g);                                \
            }                                                                                          \
        } else {                                                                                       \
            if (M.s) adj_stretch<T, PAIR>(true, o, M.b, M.c, M.PS, o, h);                              \
            if (M.sn) adj_stretch<T, PAIR>(true, n, M.bn, M.cn, M.PSN, n, g);                          \
        }                                                                                              \
        if (fl & 4) film_own = film_part_values<T, PAIR, AX>(r, W, o, n, h, g);                     \
        D = dif((OK ? n : T(0)) - o, T(0), p.dT[AX], p.invd[AX]);                                      \
        if (PAIR) E = dif((OK ? g : T(0)) - h, T(0), p.dT[AX], p.invd[AX]);                            \
    }
    T d, d2, e1 = T(0), e2 = T(0), dd[3], de[3] = {T(0), T(0), T(0)};
    MPX_DIFF(2, 2, hn, y0, y_z, az, pb, pbn, okz, d, e1);
    MPX_DIFF(1, 5, hp, z0, z_y, ay, pa, pan, oky, d2, e2);
    dd[0] = d + d2;
    if (PAIR) de[0] = e1 + e2;
    MPX_DIFF(0, 4, hn, z0, z_x, ax, pb, pbn, okx, d, e1);
    MPX_DIFF(2, 1, hp, x0, x_z, az, pa, pan, okz, d2, e2);
    dd[1] = d + d2;
    if (PAIR) de[1] = e1 + e2;
    MPX_DIFF(1, 0, hn, x0, x_y, ay, pb, pbn, oky, d, e1);
    MPX_DIFF(0, 3, hp, y0, y_x, ax, pa, pan, okx, d2, e2);
    dd[2] = d + d2;
    if (PAIR) de[2] = e1 + e2;
#undef MPX_DIFF
    const AdjParams<T> &B = args_again<AdjParams<T>>();
    const long long q = zo + (long long)B.p.px * j + ic;
    const int t[3] = {ic, j, k};
    const T lp[3] = {l[0], l[1], l[2]}; // lambda E' of the step
    if (MODE != HF_SECOND) {
#pragma unroll
        for (int C = 0; C < 3; C++) l[C] = ok[C] ? ca[C] * l[C] : T(0);
    }
    l[0] = l[0] + dd[0];
    l[1] = l[1] + dd[1];
    l[2] = l[2] + dd[2];
    if (MODE != HF_SECOND) {
        if (B.ltape && (fl & 4) && B.seg0[0] + B.m > B.loss_from && r.in)
            loss_term<T, PAIR ? 1 : 0>(B, t, q, l[0], l[1], l[2]);
        if (B.pw && q == B.pw_slot && r.in) {
            // the weighted trace's term of the state at the step's start (time n)
            const long long n = B.seg0[0] + B.m;
            if (n >= 1) {
                const T v = (T)(B.pw_scale * B.pw[n - 1]);
                if (B.pw_comp == 0)
                    l[0] += v;
                else if (B.pw_comp == 1)
                    l[1] += v;
                else
                    l[2] += v;
            }
        }
    }
    if (PAIR) {
        // the second half step of step m - 1
        l[0] = l[0] + de[0];
        l[1] = l[1] + de[1];
        l[2] = l[2] + de[2];
    }
    if (!r.in) return;
    row_st<true>(B.lE[0] + zo, vo, l[0]);
    row_st<true>(B.lE[1] + zo, vo, l[1]);
    row_st<true>(B.lE[2] + zo, vo, l[2]);
    if (MODE != HF_FIRST) {
        // the E-step adjoint's input: cb lambda E' (zero on a wall or PEC edge)
        row_st(B.mu[0] + zo, vo, ok[0] ? cb[0] * l[0] : T(0));
        row_st(B.mu[1] + zo, vo, ok[1] ? cb[1] * l[1] : T(0));
        row_st(B.mu[2] + zo, vo, ok[2] ? cb[2] * l[2] : T(0));
    }
    // lambda psiH after the map(s), of the slot's own faces (a film region's
    // faces: the film kernels')
    if (film_own) ax.s = ay.s = az.s = false;
    if (ax.s) {
        row_st(B.lpsiHo[1][0] + ax.q, ax.o, ax.pa);
        row_st(B.lpsiHo[2][0] + ax.q, ax.o, ax.pb);
    }
    if (ay.s) {
        row_st(B.lpsiHo[2][1] + ay.q, io, ay.pa);
        row_st(B.lpsiHo[0][1] + ay.q, io, ay.pb);
    }
    if (az.s) {
        row_st(B.lpsiHo[0][2] + az.q, io, az.pa);
        row_st(B.lpsiHo[1][2] + az.q, io, az.pb);
    }
    if (MODE != HF_SECOND) {
        if (B.btape) {
            // dL/dca += lambda E' E^n, dL/dcb += lambda E' x^n over the eps box
            // (last: its float64 values are then live with little else)
            const int rb[3] = {B.bs[0] + 1, B.bs[1] + 1, B.bs[2] + 1};
            int lj = j - B.bb[1], lk = k - B.bb[2], li = ic - B.bb[0];
            if (lj < 0 && B.p.per[1]) lj += B.p.n[1];
            if (lk < 0 && B.p.per[2]) lk += B.p.n[2];
            if (lj >= 0 && lj < rb[1] && lk >= 0 && lk < rb[2]) { // uniform
                if (li < 0 && B.p.per[0]) li += B.p.n[0];
                if (li >= 0 && li < rb[0]) {
                    const long long ri = (long long)li + (long long)rb[0] * ((long long)lj + (long long)rb[1] * lk);
                    const long long tb = (long long)rb[0] * rb[1] * rb[2];
                    double ga[3], gb[3], ta[3], tx[3];
#pragma unroll
                    for (int C = 0; C < 3; C++) {
                        ga[C] = B.gca_box[C * tb + ri];
                        gb[C] = B.gcb_box[C * tb + ri];
                        ta[C] = B.btape[C * tb + ri];
                        tx[C] = B.btape[(3 + C) * tb + ri];
                    }
#pragma unroll
                    for (int C = 0; C < 3; C++) {
                        B.gca_box[C * tb + ri] = ga[C] + (double)lp[C] * ta[C];
                        B.gcb_box[C * tb + ri] = gb[C] + (double)lp[C] * tx[C];
                    }
                }
            }
        }
    }
}

// the curl-part adjoint of an edge from +/- mu through its CPML recursion
template <typename T>
__device__ __forceinline__ void adj_edge_stretch(bool s, T b, T c, T &ps, T &v) {
    const T aps = ps + v;
    const T w = v + c * aps, out = b * aps;
    v = s ? w : v;
    ps = s ? out : ps;
}

// the transposed E step on the H side: lambda H_C += the transposed curl of
// the edges' curl-part adjoints (mu = cb lambda E'; part 0 of edge family X
// runs along axis X + 1 with +mu, part 1 along X + 2 with -mu); lambda E'
// itself is scaled by ca in the next half-step pass.  On a wall or PEC edge mu
// is zero, and so stays its lambda psiE.  36 bytes a slot in float32: 133 us on
// that grid at the rate of a copy; 234 us before the row form, 123 with it (part
// of mu is still in the last-level cache).
template <typename T, int TX, int TY>
__global__ void __launch_bounds__(256) k_adj_efield(AdjParams<T> A) {
    const KParams<T> &p = A.p;
    const RowPos r = row_pos<TX>(p.n, blockIdx.x, blockIdx.y, TY, blockIdx.z);
    if (r.j >= p.n[1]) return;
    const unsigned es = (unsigned)sizeof(T);
    const int ic = min(r.i, p.n[0] - 1), j = r.j, k = r.k;
    const long long sz = (long long)p.px * p.n[1];
    const unsigned io = (unsigned)ic * es, rowb = (unsigned)p.px * es, vo = io + (unsigned)j * rowb;
    const bool okx = ic + 1 < p.n[0] || p.per[0], oky = j + 1 < p.n[1] || p.per[1], okz = k + 1 < p.n[2] || p.per[2];
    const unsigned vxp = ic + 1 < p.n[0] ? vo + es : (p.per[0] ? vo - (unsigned)(p.n[0] - 1) * es : vo);
    const unsigned vyp = io + (unsigned)(j + 1 < p.n[1] ? j + 1 : (p.per[1] ? 0 : j)) * rowb;
    const long long zo = k * sz, za = (k + 1 < p.n[2] ? k + 1 : (p.per[2] ? 0 : k)) * sz;
    const T *Mx = A.mu[0] + zo, *My = A.mu[1] + zo, *Mz = A.mu[2] + zo;
    const T x0 = row_ld(Mx, vo), x_y = row_ld(Mx, vyp), x_z = row_ld(A.mu[0] + za, vo);
    const T y0 = row_ld(My, vo), y_x = row_ld(My, vxp), y_z = row_ld(A.mu[1] + za, vo);
    const T z0 = row_ld(Mz, vo), z_x = row_ld(Mz, vxp), z_y = row_ld(Mz, vyp);
    // the slot's lambda H is touched once per pass: non-temporal (the mu the
    // neighbouring edges read again stays in L2)
    T *Hx = A.lH[0] + zo, *Hy = A.lH[1] + zo, *Hz = A.lH[2] + zo;
    const T h0 = row_ld<true>(Hx, vo), h1 = row_ld<true>(Hy, vo), h2 = row_ld<true>(Hz, vo);
    // lambda psiE of step n: read set n & 1, write the other
    const bool par = ((A.seg0[0] + A.m) & 1) != 0;
    AdjAxis<T> ax, ay, az;
    adj_axis_x<T, 1>(p, r, par ? A.lpsiE2[1][0] : A.lpsiE[1][0], par ? A.lpsiE2[2][0] : A.lpsiE[2][0], p.bE[0],
                     p.cE[0], ax);
    adj_axis_yz<T, 1, 1>(p, r, par ? A.lpsiE2[2][1] : A.lpsiE[2][1], par ? A.lpsiE2[0][1] : A.lpsiE[0][1], p.bE[1],
                         p.cE[1], io, ay);
    adj_axis_yz<T, 1, 2>(p, r, par ? A.lpsiE2[0][2] : A.lpsiE[0][2], par ? A.lpsiE2[1][2] : A.lpsiE[1][2], p.bE[2],
                         p.cE[2], io, az);
    // by edge family X and part: part 0 +mu along X + 1, part 1 -mu along X + 2
    T o[6] = {x0, -x0, y0, -y0, z0, -z0};
    T n[6] = {x_y, -x_z, y_z, -y_x, z_x, -z_y};
    if (ax.s || ax.sn) {
        adj_edge_stretch(ax.s, ax.b, ax.c, ax.pa, o[3]);
        adj_edge_stretch(ax.s, ax.b, ax.c, ax.pb, o[4]);
        adj_edge_stretch(ax.sn, ax.bn, ax.cn, ax.pan, n[3]);
        adj_edge_stretch(ax.sn, ax.bn, ax.cn, ax.pbn, n[4]);
    }
    if (ay.s) {
        adj_edge_stretch(true, ay.b, ay.c, ay.pa, o[5]);
        adj_edge_stretch(true, ay.b, ay.c, ay.pb, o[0]);
    }
    if (ay.sn) {
        adj_edge_stretch(true, ay.bn, ay.cn, ay.pan, n[5]);
        adj_edge_stretch(true, ay.bn, ay.cn, ay.pbn, n[0]);
    }
    if (az.s) {
        adj_edge_stretch(true, az.b, az.c, az.pa, o[1]);
        adj_edge_stretch(true, az.b, az.c, az.pb, o[2]);
    }
    if (az.sn) {
        adj_edge_stretch(true, az.bn, az.cn, az.pan, n[1]);
        adj_edge_stretch(true, az.bn, az.cn, az.pbn, n[2]);
    }
    const T dx = p.dT[0], dy = p.dT[1], dz = p.dT[2], ix = p.invd[0], iy = p.invd[1], iz = p.invd[2];
    const T d0 = dif(o[2] - (okz ? n[2] : T(0)), T(0), dz, iz) + dif(o[5] - (oky ? n[5] : T(0)), T(0), dy, iy);
    const T d1 = dif(o[4] - (okx ? n[4] : T(0)), T(0), dx, ix) + dif(o[1] - (okz ? n[1] : T(0)), T(0), dz, iz);
    const T d2 = dif(o[0] - (oky ? n[0] : T(0)), T(0), dy, iy) + dif(o[3] - (okx ? n[3] : T(0)), T(0), dx, ix);
    if (!r.in) return;
    row_st<true>(Hx, vo, h0 + d0);
    row_st<true>(Hy, vo, h1 + d1);
    row_st<true>(Hz, vo, h2 + d2);
    if (ax.s) {
        row_st((par ? A.lpsiE[1][0] : A.lpsiE2[1][0]) + ax.q, ax.o, ax.pa);
        row_st((par ? A.lpsiE[2][0] : A.lpsiE2[2][0]) + ax.q, ax.o, ax.pb);
    }
    if (ay.s) {
        row_st((par ? A.lpsiE[2][1] : A.lpsiE2[2][1]) + ay.q, io, ay.pa);
        row_st((par ? A.lpsiE[0][1] : A.lpsiE2[0][1]) + ay.q, io, ay.pb);
    }
    if (az.s) {
        row_st((par ? A.lpsiE[0][2] : A.lpsiE2[0][2]) + az.q, io, az.pa);
        row_st((par ? A.lpsiE[1][2] : A.lpsiE2[1][2]) + az.q, io, az.pb);
    }
}

__global__ void __launch_bounds__(256) k_copy_segs(const CopySeg *segs) {
    const CopySeg S = segs[blockIdx.y];
    const long long n16 = S.bytes >> 4;
    const uint4 *src = (const uint4 *)S.src;
    uint4 *dst = (uint4 *)S.dst;
    const long long stride = (long long)gridDim.x * 256;
    for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < n16; t += stride) dst[t] = src[t];
    const long long rem = (S.bytes - (n16 << 4)) >> 2;
    if (blockIdx.x == 0 && threadIdx.x < rem)
        ((uint32_t *)S.dst)[n16 * 4 + threadIdx.x] = ((const uint32_t *)S.src)[n16 * 4 + threadIdx.x];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static dim3 slot_grid(const int *n) { return dim3((n[0] + 63) / 64, (n[1] + 3) / 4, n[2]); }

// lambda of the state before a half step from lambda after it; the B^
// prepass of the input state must have run (launch_film phase-1 prepass)
template <typename T>
hipError_t launch_adj_half(const AdjParams<T> &A, int nblk, hipStream_t s) {
    if (nblk) k_adj_film<T><<<dim3(nblk), dim3(256), 0, s>>>(A);
    k_adj_face<T><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
    if (nblk) k_adj_film_commit<<<dim3(nblk), dim3(256), 0, s>>>(A.p.blocktab, A.p.films, A.af);
    k_adj_curlE<T><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_estep(const AdjParams<T> &A, hipStream_t s) {
    k_adj_estep<T><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
    k_adj_curlH<T><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_loss(const AdjParams<T> &A, int film, double scale, hipStream_t s) {
    k_adj_loss<T><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A, film, scale);
    return hipGetLastError();
}

hipError_t launch_adj_init_ms(const int4 *blocktab, int nblk, const FilmDev *films, const AdjFilmDev *af,
                              const double *u, hipStream_t s) {
    if (nblk) k_adj_init_ms<<<dim3(nblk), dim3(256), 0, s>>>(blocktab, films, af, u[0], u[1], u[2]);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_film_energy(const KParams<T> &p, int film, double *part, double *acc, double scale, hipStream_t s) {
    const dim3 g = slot_grid(p.n);
    k_film_energy<T><<<g, dim3(64, 4), 0, s>>>(p, film, part);
    k_accum<<<dim3(1), dim3(64), 0, s>>>(part, (int)(g.x * g.y * g.z), acc, scale);
    return hipGetLastError();
}

hipError_t launch_set_step(long long *step, long long v, hipStream_t s) {
    k_set_step<<<dim3(1), dim3(64), 0, s>>>(step, v);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_eps(const AdjParams<T> &A, const int *box, double *out, hipStream_t s) {
    const long long nc = (long long)box[3] * box[4] * box[5];
    if (nc == 0) return hipSuccess;
    k_adj_eps<T><<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s>>>(
        A, make_int4(box[0], box[1], box[2], 0), make_int4(box[3], box[4], box[5], 0), out);
    return hipGetLastError();
}

long long film_tape_size(const int *cb) { return 6LL * (cb[3] + 1) * (cb[4] + 1) * (cb[5] + 1); }
long long box_tape_size(const int *box) { return 6LL * (box[3] + 1) * (box[4] + 1) * (box[5] + 1); }

// cb: the film's cell box (it sizes the grid)
template <typename T>
hipError_t launch_tape_loss(const KParams<T> &p, int film, int merged, double *dst, hipStream_t s, const int *cb) {
    const long long tb = film_tape_size(cb) / 6;
    k_tape_loss<T><<<dim3((unsigned)((tb + 255) / 256)), dim3(256), 0, s>>>(p, film, merged, dst);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_loss_tape(const AdjParams<T> &A, int film, double scale, const double *tape,
                                const long long *seg0, int m, long long loss_from, hipStream_t s, const int *cb) {
    const long long tb = film_tape_size(cb) / 6;
    k_adj_loss_tape<T><<<dim3((unsigned)((tb + 255) / 256)), dim3(256), 0, s>>>(A, film, scale, tape, seg0, m,
                                                                               loss_from);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_loss_eps_tape(const KParams<T> &p, int film, double scale, const double *tape,
                                    const long long *seg0, int m, long long loss_from, double *acc, hipStream_t s,
                                    const int *cb) {
    const long long nc = (long long)cb[3] * cb[4] * cb[5];
    k_adj_loss_eps_tape<T><<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s>>>(p, film, scale, tape, seg0, m,
                                                                                    loss_from, acc);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_loss_eps_state(const KParams<T> &p, int film, double scale, double *acc, hipStream_t s,
                                     const int *cb) {
    const long long nc = (long long)cb[3] * cb[4] * cb[5];
    k_adj_loss_eps_state<T><<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s>>>(p, film, scale, acc);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_eps_box(const KParams<T> &p, const int *box, const double *gca, const double *gcb, double *out,
                              hipStream_t s) {
    const long long nc = (long long)box[3] * box[4] * box[5];
    if (nc == 0) return hipSuccess;
    k_adj_eps_box<T><<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s>>>(
        p, make_int4(box[0], box[1], box[2], 0), make_int4(box[3], box[4], box[5], 0), gca, gcb, out);
    return hipGetLastError();
}

// the field passes' tiles: 256 x 1 slots on the grids whose forward passes use
// them, else 64 x 4 (the flag table is of the same shape)
static dim3 wide_grid(const int *n) { return dim3((n[0] + kWideTX - 1) / kWideTX, n[1], n[2]); }

template <typename T, int MODE>
static void launch_hfield(const AdjParams<T> &A, hipStream_t s) {
    if (A.wide)
        k_adj_hfield<T, MODE, kWideTX, kWideTY><<<wide_grid(A.p.n), dim3(kWideTX, kWideTY), 0, s>>>(A);
    else
        k_adj_hfield<T, MODE, 64, 4><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
}

template <typename T>
hipError_t launch_adj_loss_weights(const KParams<T> &p, int film, double *dst, hipStream_t s, const int *cb) {
    const long long tb = film_tape_size(cb) / 6;
    k_adj_loss_weights<T><<<dim3((unsigned)((tb + 255) / 256)), dim3(256), 0, s>>>(p, film, dst);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_half_fused(const AdjParams<T> &A, int nblk, int scale, const long long *film_nr,
                                 hipStream_t s) {
    if (nblk) k_adj_film<T><<<dim3(nblk), dim3(256), 0, s>>>(A);
    for (int f = 0; f < A.p.nfilm; f++)
        if (film_nr[f] > 0)
            k_adj_film_faces<T><<<dim3((unsigned)((film_nr[f] + 255) / 256), 3), dim3(256), 0, s>>>(A, f);
    if (scale)
        launch_hfield<T, HF_FIRST>(A, s);
    else
        launch_hfield<T, HF_SECOND>(A, s);
    return hipGetLastError();
}

// the film part of a half-step transpose (the magnetic faces' LLG transpose,
// the film reach's faces and their table), then the merged field pass
template <typename T>
hipError_t launch_adj_film_part(const AdjParams<T> &A, int nblk, const long long *film_nr, hipStream_t s) {
    if (nblk) k_adj_film<T><<<dim3(nblk), dim3(256), 0, s>>>(A);
    for (int f = 0; f < A.p.nfilm; f++)
        if (film_nr[f] > 0)
            k_adj_film_faces<T><<<dim3((unsigned)((film_nr[f] + 255) / 256), 3), dim3(256), 0, s>>>(A, f);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_hfield2(const AdjParams<T> &A, hipStream_t s) {
    launch_hfield<T, HF_PAIR>(A, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_estep_fused(const AdjParams<T> &A, hipStream_t s) {
    if (A.wide)
        k_adj_efield<T, kWideTX, kWideTY><<<wide_grid(A.p.n), dim3(kWideTX, kWideTY), 0, s>>>(A);
    else
        k_adj_efield<T, 64, 4><<<slot_grid(A.p.n), dim3(64, 4), 0, s>>>(A);
    return hipGetLastError();
}

// a[q] += v on the stream (one thread)
template <typename T>
__global__ void __launch_bounds__(64) k_add_one(T *a, long long q, double v) {
    if (threadIdx.x == 0) a[q] += (T)v;
}

template <typename T>
hipError_t launch_add_one(T *a, long long q, double v, hipStream_t s) {
    k_add_one<T><<<dim3(1), dim3(64), 0, s>>>(a, q, v);
    return hipGetLastError();
}

hipError_t launch_copy_segs(const CopySeg *segs, int nseg, int nblk, hipStream_t s) {
    if (nseg == 0) return hipSuccess;
    k_copy_segs<<<dim3(nblk, nseg), dim3(256), 0, s>>>(segs);
    return hipGetLastError();
}

#define MPX_ADJ(T)                                                                              \
    template hipError_t launch_adj_half<T>(const AdjParams<T> &, int, hipStream_t);            \
    template hipError_t launch_adj_estep<T>(const AdjParams<T> &, hipStream_t);                \
    template hipError_t launch_adj_loss<T>(const AdjParams<T> &, int, double, hipStream_t);    \
    template hipError_t launch_adj_eps<T>(const AdjParams<T> &, const int *, double *, hipStream_t);      \
    template hipError_t launch_film_energy<T>(const KParams<T> &, int, double *, double *, double, hipStream_t); \
    template hipError_t launch_adj_half_fused<T>(const AdjParams<T> &, int, int, const long long *, hipStream_t); \
    template hipError_t launch_adj_estep_fused<T>(const AdjParams<T> &, hipStream_t);                           \
    template hipError_t launch_adj_film_part<T>(const AdjParams<T> &, int, const long long *, hipStream_t);     \
    template hipError_t launch_adj_hfield2<T>(const AdjParams<T> &, hipStream_t);                               \
    template hipError_t launch_adj_loss_weights<T>(const KParams<T> &, int, double *, hipStream_t, const int *); \
    template hipError_t launch_add_one<T>(T *, long long, double, hipStream_t);                                 \
    template hipError_t launch_tape_loss<T>(const KParams<T> &, int, int, double *, hipStream_t, const int *);   \
    template hipError_t launch_adj_loss_tape<T>(const AdjParams<T> &, int, double, const double *,              \
                                                const long long *, int, long long, hipStream_t, const int *);   \
    template hipError_t launch_adj_loss_eps_tape<T>(const KParams<T> &, int, double, const double *,             \
                                                    const long long *, int, long long, double *, hipStream_t,    \
                                                    const int *);                                                \
    template hipError_t launch_adj_loss_eps_state<T>(const KParams<T> &, int, double, double *, hipStream_t,     \
                                                     const int *);                                               \
    template hipError_t launch_adj_eps_box<T>(const KParams<T> &, const int *, const double *, const double *,   \
                                              double *, hipStream_t);
MPX_ADJ(float)
MPX_ADJ(double)

} // namespace mpx
