// kernels.hip -- gfx950 device code of libmpx: the Yee curl updates, the
// CPML recursions, the soft source, the trapezoidal LLG site solve and the
// probe / energy reductions.
//
// Scheme: arXiv:2510.22221, Methods, "Numerical Model".
//   H/M half step: B^ = H + M, B^* = B^ - dt/(2 mu0) curl E (eq. iterate_H);
//     non-magnetic faces keep H = B^*; magnetic faces solve the trapezoidal
//     LLG (eqs. llg_tra4-llg_tra6) at its fixed point, normalise to Ms and
//     set H = B^*_c - M_c.
//   E step: E <- ca E + cb (curl H - J), ca, cb from eps and sigma of the
//     edge (the semi-implicit E update closing that subsection).
//
// Layout: every field component lives on an nx*ny*nz slot lattice, x fastest
// with a padded pitch; slot (i,j,k) holds the Yee site with natural index
// (i,j,k).  Sites with natural index N along a non-periodic axis lie on the
// domain wall and are identically zero, so they are not stored.
//
// Arithmetic order: the float64 instantiation evaluates every stored value
// with the same sequence of IEEE operations as the plain definition (the
// library is built with -ffp-contract=off), so repeated runs, tile shapes and
// the fused pass all give bitwise identical float64 results.
#include "film.h"

#include <algorithm>

namespace mpx {

__device__ __forceinline__ int cell_id(const int *n, const int *per, int px, const uint8_t *id, int i, int j,
                                       int k) {
    int ii = fold(i, n[0], per[0]), jj = fold(j, n[1], per[1]), kk = fold(k, n[2], per[2]);
    if (ii < 0 || jj < 0 || kk < 0) return -1;
    return id[(long long)ii + (long long)px * ((long long)jj + (long long)n[1] * kk)];
}

// ---------------------------------------------------------------------------
// magnetic-face test: the face of family c at slot idx is magnetic when it
// lies in a film's site box and one of the two cells sharing it has Ms > 0
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ int film_of_site(const KParams<T> &p, int c, const int *idx) {
    for (int f = 0; f < p.nfilm; f++) {
        const FilmDev &F = p.films[f];
        if (idx[0] >= F.b0[0] && idx[0] < F.b0[0] + F.bn[0] && idx[1] >= F.b0[1] && idx[1] < F.b0[1] + F.bn[1] &&
            idx[2] >= F.b0[2] && idx[2] < F.b0[2] + F.bn[2]) {
            const long long l = (long long)(idx[0] - F.b0[0]) +
                                (long long)F.bn[0] * ((long long)(idx[1] - F.b0[1]) + (long long)F.bn[1] * (idx[2] - F.b0[2]));
            return F.prm[(c * 3) * F.ns + l] > 0.0 ? f : -1;
        }
    }
    return -1;
}

// ---------------------------------------------------------------------------
// film half step (float64 throughout)
//   phase 1: reads the state (H, M); writes the scratch (H1, M1)
//   phase 2: reads the scratch for magnetic faces and recomputes the first
//            half step on the fly for non-magnetic ones; writes the state
// ---------------------------------------------------------------------------
struct SiteRef {
    int film;
    long long l; // local index in the film's site box
};

template <typename T>
__device__ __forceinline__ void site_params(const KParams<T> &p, int c, const int *idx, double &ms, double &al,
                                            double &ga) {
    double sm = 0.0, sa = 0.0, sg = 0.0;
    int cnt = 0, nm = 0;
    for (int u = -1; u <= 0; u++) {
        int cc[3] = {idx[0], idx[1], idx[2]};
        cc[c] += u;
        int m = cell_id(p.n, p.per, p.px, p.id, cc[0], cc[1], cc[2]);
        if (m < 0) continue;
        cnt++;
        sm += p.mat[m].Ms;
        if (p.mat[m].Ms > 0) {
            nm++;
            sa += p.mat[m].alpha;
            sg += p.mat[m].gamma_abs;
        }
    }
    ms = cnt ? sm / cnt : 0.0;
    al = nm ? sa / nm : 0.0;
    ga = nm ? sg / nm : 0.0;
}

// B^ and B^* at the face of family cq at idx (folded), for film f; for a
// non-magnetic face in phase 1 also those of phase 2 (bn2, bs2: the phase-2
// expressions, from the same H and E); mag tells whether the face is
// magnetic, cu is its dt/(2 mu0) (curl E)_cq term
template <typename T>
__device__ __forceinline__ void bhat(const KParams<T> &p, int phase, int f, int cq, const int *idx, double &bn,
                                     double &bs, double &bn2, double &bs2, bool &mag, double &cu) {
    bn2 = bs2 = cu = 0.0;
    mag = false;
    if (idx[0] < 0 || idx[1] < 0 || idx[2] < 0) { // outside the domain (cannot happen for the
        bn = bs = 0.0;                             // film placements set_materials accepts)
        return;
    }
    double d1, d2;
    curl_e64(p, cq, idx, d1, d2);
    const FilmDev F = film_desc(p.films, f);
    bool inside;
    const long long l = film_local<T>(F, idx, inside);
    mag = inside && F.prm[(cq * 3) * F.ns + l] > 0.0;
    cu = p.hcd * (d1 - d2);
    double b;
    if (mag) {
        if (phase == 1)
            b = (double)p.H[cq][p.slot(idx[0], idx[1], idx[2])] + F.M[(cq * 3 + cq) * F.ns + l];
        else
            b = F.H1[cq * F.ns + l] + F.M1[(cq * 3 + cq) * F.ns + l];
    } else {
        const double h0 = (double)p.H[cq][p.slot(idx[0], idx[1], idx[2])];
        double h = h0;
        if (phase == 2) h = h - cu;
        b = h + 0.0;
        if (phase == 1) {
            const double h2 = h0 - cu;
            bn2 = h2 + 0.0;
            bs2 = bn2 - cu;
        }
    }
    bn = b;
    bs = b - cu;
}

// ldz()'s value with its load issued whatever the domain test says (at slot
// 0 when the site lies outside, the value then dropped): a value merged out
// of a branch waits for its load, a selected one does not
template <typename T>
__device__ __forceinline__ T ldz_sel(const KParams<T> &p, const T *a, int i, int j, int k) {
    const int ii = fold(i, p.n[0], p.per[0]), jj = fold(j, p.n[1], p.per[1]), kk = fold(k, p.n[2], p.per[2]);
    const bool ok = ii >= 0 && jj >= 0 && kk >= 0;
    const T v = a[ok ? p.slot(ii, jj, kk) : 0];
    return ok ? v : T(0);
}

// curl_e64() with ldz_sel loads
template <typename T>
__device__ __forceinline__ void curl_e64_sel(const KParams<T> &p, int c, const int *idx, double &d1, double &d2) {
    const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    int u1[3] = {idx[0], idx[1], idx[2]}, u2[3] = {idx[0], idx[1], idx[2]};
    u1[c1] += 1;
    u2[c2] += 1;
    const double e2a = (double)ldz_sel(p, p.E[c2], idx[0], idx[1], idx[2]);
    const double e2b = (double)ldz_sel(p, p.E[c2], u1[0], u1[1], u1[2]);
    const double e1a = (double)ldz_sel(p, p.E[c1], idx[0], idx[1], idx[2]);
    const double e1b = (double)ldz_sel(p, p.E[c1], u2[0], u2[1], u2[2]);
    d1 = over_spacing(p, e2b - e2a, c1);
    d2 = over_spacing(p, e1b - e1a, c2);
}

// bhat() for phase 1 at a face of film F's grown box, by the same
// operations, with every load issued before the film test picks the value (a
// face outside the film reads site 0's entries and drops them)
template <typename T>
__device__ __forceinline__ void bhat_phase1(const KParams<T> &p, const FilmDev &F, int cq, const int *idx,
                                            double &bn, double &bs, double &bn2, double &bs2, bool &mag,
                                            double &cu) {
    double d1, d2;
    curl_e64_sel(p, cq, idx, d1, d2);
    bool inside;
    const long long l = film_local<T>(F, idx, inside); // 0 outside
    const double h0 = (double)p.H[cq][p.slot(idx[0], idx[1], idx[2])];
    const double ms = F.prm[(cq * 3) * F.ns + l];
    const double m = F.M[(cq * 3 + cq) * F.ns + l];
    mag = inside && ms > 0.0;
    cu = p.hcd * (d1 - d2);
    const double b = mag ? h0 + m : h0 + 0.0;
    const double n2 = (h0 - cu) + 0.0;
    bn2 = mag ? 0.0 : n2;
    bs2 = mag ? 0.0 : n2 - cu;
    bn = b;
    bs = b - cu;
}

// B^ prepass: B^n and B^* of every face of the grown face box.  BESIDE: in
// the launch of the film's first half step, whose blocks form what they need
// of it themselves and write the magnetic faces' phase-2 values
template <typename T, bool BESIDE = false>
__device__ __forceinline__ void bhat_body(const KParams<T> &p, int phase, int blk) {
    const int4 bt = block_entry(p.blocktab_ext, blk);
    const int f = bt.x, c = bt.y;
    const FilmDev F = block_desc(p.films, p.nfilm, f);
    const unsigned l = (unsigned)bt.z + threadIdx.x;
    if (l >= (unsigned)F.nse) return;
    int idx[3];
    box_split(l, F.en, idx);
    for (int a = 0; a < 3; a++) idx[a] += F.e0[a];
    double bn, bs, bn2, bs2, cu;
    bool mag;
    if (phase == 1)
        bhat_phase1(p, F, c, idx, bn, bs, bn2, bs2, mag, cu);
    else
        bhat(p, phase, f, c, idx, bn, bs, bn2, bs2, mag, cu);
    F.Bn[c * F.nse + l] = bn;
    F.Bs[c * F.nse + l] = bs;
    if (phase == 1 && F.Bn2) {
        if (!mag) {
            F.Bn2[c * F.nse + l] = bn2;
            F.Bs2[c * F.nse + l] = bs2;
        } else if (!BESIDE) {
            // a magnetic face: the film kernel completes it from its solve;
            // it finds the curl term here (only its own thread reads it)
            F.Bs2[c * F.nse + l] = cu;
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_bhat(KParams<T> p, int phase) {
    bhat_body(p, phase, blockIdx.x);
}

// batched: work[b] = (instance, block of that instance)
template <typename T>
__global__ void __launch_bounds__(256) k_bhat_batch(const KParams<T> *__restrict__ plist, const int2 *__restrict__ work, int phase) {
    const int2 wk = work[blockIdx.x];
    bhat_body(plist[wk.x], phase, wk.y);
}

// the first half step and its prepass in one launch: the film's blocks, then
// the prepass's
template <typename T>
__global__ void __launch_bounds__(256) k_film_first(KParams<T> p, int nblk) {
    if ((int)blockIdx.x < nblk)
        film_body<T, true>(p, 1, 0, blockIdx.x, threadIdx.x);
    else
        bhat_body<T, true>(p, 1, blockIdx.x - nblk);
}

template <typename T>
__global__ void __launch_bounds__(256) k_film_first_batch(const KParams<T> *__restrict__ plist, const int2 *__restrict__ work_ext, const int2 *__restrict__ work, int n) {
    const int b = (int)blockIdx.x;
    const int2 wk = b < n ? work[b] : work_ext[b - n];
    if (b < n)
        film_body<T, true>(plist[wk.x], 1, 0, wk.y, threadIdx.x);
    else
        bhat_body<T, true>(plist[wk.x], 1, wk.y);
}

template <typename T>
__global__ void __launch_bounds__(256) k_film(KParams<T> p, int phase, int inc_step) {
    film_body(p, phase, inc_step, blockIdx.x, threadIdx.x);
}

template <typename T>
__global__ void __launch_bounds__(256) k_film_batch(const KParams<T> *__restrict__ plist, const int2 *__restrict__ work, int phase, int inc_step) {
    const int2 wk = work[blockIdx.x];
    film_body(plist[wk.x], phase, inc_step, wk.y, threadIdx.x);
}

// ---------------------------------------------------------------------------
// probes at an integer time: after the E step and the first H/M half step of
// the merged pair (scratch holds H, M at that time for magnetic faces)
// ---------------------------------------------------------------------------
template <typename T>
__device__ double h_integer_time(const KParams<T> &p, int c, const int *idx) {
    const int f = p.nfilm ? film_of_site(p, c, idx) : -1;
    if (f >= 0) {
        const FilmDev &F = p.films[f];
        bool inside;
        const long long l = film_local<T>(F, idx, inside);
        return F.H1[c * F.ns + l];
    }
    const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
    int u1[3] = {idx[0], idx[1], idx[2]}, u2[3] = {idx[0], idx[1], idx[2]};
    u1[c1] += 1;
    u2[c2] += 1;
    const T d1 = dif(ldz(p, p.E[c2], u1[0], u1[1], u1[2]), ldz(p, p.E[c2], idx[0], idx[1], idx[2]), p.dT[c1],
                     p.invd[c1]);
    const T d2 = dif(ldz(p, p.E[c1], u2[0], u2[1], u2[2]), ldz(p, p.E[c1], idx[0], idx[1], idx[2]), p.dT[c2],
                     p.invd[c2]);
    const T h = ldz(p, p.H[c], idx[0], idx[1], idx[2]);
    return (double)(h - p.hc * (d1 - d2));
}

// The energy kernels' materials: a block's copy in LDS, read by cell id
struct EnergyMat {
    double eps, pec;
};

template <typename T>
__device__ __forceinline__ void energy_mats(const KParams<T> &p, EnergyMat *tab, int t) {
    tab[t].eps = p.mat[t].eps_r;
    tab[t].pec = p.mat[t].is_pec ? 1.0 : 0.0;
}

// the two energy sums of the slot idx: eps E^2 over its three edges (PEC and
// lower-wall edges excluded) and H^2 - (hc curl E)^2 over its three faces (H
// at the integer time times the product of the two neighbouring half-step
// values), H being the stored field between steps (MID = 0) or, during the
// merged pass, the integer-time value of h_integer_time rounded to the field
// type (MID = 1), which is what the bracket half step would store.  The seven
// cells around the slot that its edges touch, nine values of E and three of H
// go out in one round trip; an edge that counts has its four cells in the
// domain.
template <typename T, int MID>
__device__ __forceinline__ void energy_site(const KParams<T> &p, const EnergyMat *tab, const int *idx, double &we,
                                            double &wh) {
    const long long q = p.slot(idx[0], idx[1], idx[2]);
    const long long st[3] = {1, p.px, (long long)p.px * p.n[1]};
    long long lo[3], hi[3];
    bool okl[3], okh[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const int l = fold(idx[a] - 1, p.n[a], p.per[a]), u = fold(idx[a] + 1, p.n[a], p.per[a]);
        okl[a] = l >= 0;
        okh[a] = u >= 0;
        lo[a] = okl[a] ? (l - idx[a]) * st[a] : 0;
        hi[a] = okh[a] ? (u - idx[a]) * st[a] : 0;
    }
    int id[7]; // bit a of the index: one cell down along axis a
    T e[3], h[3], eu[3][3];
#pragma unroll
    for (int b = 0; b < 7; b++)
        id[b] = p.id[q + (b & 1 ? lo[0] : 0) + (b & 2 ? lo[1] : 0) + (b & 4 ? lo[2] : 0)];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        e[c] = p.E[c][q];
        eu[c][c1] = p.E[c][q + hi[c1]];
        eu[c][c2] = p.E[c][q + hi[c2]];
        h[c] = p.H[c][q];
    }
    EnergyMat m[7];
#pragma unroll
    for (int b = 0; b < 7; b++) m[b] = tab[id[b]];
    int f = -1;
    if (MID)
        for (int g = 0; g < p.nfilm; g++) {
            const FilmDev &F = p.films[g];
            if (idx[0] >= F.b0[0] && idx[0] < F.b0[0] + F.bn[0] && idx[1] >= F.b0[1] &&
                idx[1] < F.b0[1] + F.bn[1] && idx[2] >= F.b0[2] && idx[2] < F.b0[2] + F.bn[2])
                f = g;
        }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        const EnergyMat &m11 = m[(1 << c1) | (1 << c2)], &m10 = m[1 << c1], &m01 = m[1 << c2], &m00 = m[0];
        const double eps = p.eps0 * ((((m11.eps + m10.eps) + m01.eps) + m00.eps) * 0.25);
        const double ev = (double)e[c], wn = we + eps * ev * ev;
        const bool counts = okl[c1] && okl[c2] && !(m11.pec + m10.pec + m01.pec + m00.pec > 0.0);
        we = counts ? wn : we;
        const T e2b = okh[c1] ? eu[c2][c1] : T(0), e1b = okh[c2] ? eu[c1][c2] : T(0);
        const double cu = p.hcd * (over_spacing(p, (double)e2b - (double)e[c2], c1) -
                                   over_spacing(p, (double)e1b - (double)e[c1], c2));
        double hv = (double)h[c];
        if (MID) {
            hv = (double)(h[c] - p.hc * (dif(e2b, e[c2], p.dT[c1], p.invd[c1]) - dif(e1b, e[c1], p.dT[c2], p.invd[c2])));
            if (f >= 0) {
                const FilmDev &F = p.films[f];
                bool inside;
                const long long l = film_local<T>(F, idx, inside);
                if (F.prm[(c * 3) * F.ns + l] > 0.0) hv = (double)(T)F.H1[c * F.ns + l];
            }
        }
        wh += hv * hv - cu * cu;
    }
}

// the sums of 256 values a and of 256 values b over a block, a halving tree
// each (the first wavefront's, the second's): its first two levels over LDS,
// one barrier, the rest by shuffles.  Valid in threads 0 (a) and 64 (b); red is
// free again after the block's next barrier.
__device__ __forceinline__ double block_tree2(double (*red)[256], int t, double a, double b) {
    red[0][t] = a;
    red[1][t] = b;
    __syncthreads();
    if (t >= 128) return 0.0;
    const double *r = red[t >> 6];
    const int l = t & 63;
    double s = (r[l] + r[l + 128]) + (r[l + 64] + r[l + 192]);
    for (int st = 32; st > 0; st >>= 1) {
        const double o = __shfl_down(s, st, 64);
        if (l < st) s = s + o;
    }
    return s;
}

template <typename T>
__device__ __forceinline__ void probes_body(const KParams<T> &p, int pb) {
    __shared__ double red[256];
    const ProbeDev &P = p.probes[pb];
    long long sample;
    if (!probe_due(P, p.step[0], sample)) return; // uniform over the block
    double v[3] = {0.0, 0.0, 0.0};
    if (P.kind == 0 && P.field < 3) {
        if (threadIdx.x == 0) v[0] = (double)ldz(p, p.E[P.field], P.i, P.j, P.k);
    } else if (P.kind == 1) {
        // the film's mean M: its film blocks' partials, thread t adding
        // partials t, t + 256, ... then a halving tree (the probe block of the
        // merged H/M launch forms the same additions in one wavefront)
        const FilmDev &F = p.films[P.film];
        for (int w = 0; w < 3; w++) {
            const int b0 = F.blk0[w], nb = F.nblk[w];
            double s = 0.0;
            for (int b = threadIdx.x; b < nb; b += blockDim.x) s += p.partial[b0 + b];
            red[threadIdx.x] = s;
            __syncthreads();
            for (int st = 128; st > 0; st >>= 1) {
                if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
                __syncthreads();
            }
            v[w] = red[0] / F.ncells;
            __syncthreads();
        }
    } else if (P.kind == 0) {
        if (threadIdx.x == 0) {
            // an H component; sites on an upper wall are not stored and are zero
            const int idx[3] = {P.i, P.j, P.k};
            const int c = P.field - 3;
            bool wall = false;
            for (int a = 0; a < 3; a++)
                if (idx[a] >= p.n[a]) wall = true;
            v[0] = wall ? 0.0 : h_integer_time(p, c, idx);
        }
    } else if (P.kind == 2) {
        // film EM energy: the partial sums of k_probe_parts, in block order
        double s = 0.0;
        for (long long b = threadIdx.x; b < P.npart; b += blockDim.x) s += P.part[b];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        v[0] = red[0] * p.dV;
    } else {
        // the grid's EM energy: the (E, H) partial pairs of k_probe_parts
        double sum[2];
        for (int w = 0; w < 2; w++) {
            double s = 0.0;
            for (long long b = threadIdx.x; b < P.npart; b += blockDim.x) s += P.part[2 * b + w];
            red[threadIdx.x] = s;
            __syncthreads();
            for (int st = 128; st > 0; st >>= 1) {
                if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
                __syncthreads();
            }
            sum[w] = red[0];
            __syncthreads();
        }
        v[0] = 0.5 * p.dV * (sum[0] + p.mu0 * sum[1]);
    }
    probe_store(p, P, sample, v);
}

// EM energy density sum of one film cell (eps0 eps_r <E^2>/2 + mu0 <H^2>/2 over
// its twelve edges and six faces, H at the integer time), zero elsewhere.
// Every face of a magnetic cell is magnetic and lies in the film's face box, so
// its H at the integer time is the film's scratch; the loads of all cells of
// the box are issued and a non-magnetic cell's dropped (a probe's partials on
// the 64 x 12 x 4 film of a 128 x 64 x 64 grid: 16.4 to 5.4 us).
template <typename T>
__device__ double film_cell_energy(const KParams<T> &p, const FilmDev &F, unsigned t) {
    int cc[3];
    box_split(t, F.cb + 3, cc);
    for (int a = 0; a < 3; a++) cc[a] += F.cb[a];
    const MatDev &m = p.mat[p.id[p.slot(cc[0], cc[1], cc[2])]];
    // the cell's upper neighbours (folded; -1 past a wall)
    int up[3];
    for (int a = 0; a < 3; a++) up[a] = fold(cc[a] + 1, p.n[a], p.per[a]);
    double we = 0.0, wh = 0.0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        double e2 = 0.0;
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int vv = 0; vv < 2; vv++) {
                int q[3] = {cc[0], cc[1], cc[2]};
                if (u) q[c1] = up[c1];
                if (vv) q[c2] = up[c2];
                const bool ok = q[c1] >= 0 && q[c2] >= 0;
                const double x = (double)p.E[c][ok ? p.slot(q[0], q[1], q[2]) : 0];
                const double e = ok ? x : 0.0;
                e2 += e * e;
            }
        we += e2 / 4.0;
        double h2 = 0.0;
#pragma unroll
        for (int u = 0; u < 2; u++) {
            int q[3] = {cc[0], cc[1], cc[2]};
            if (u) q[c] = up[c];
            bool inside;
            const long long l = film_local<T>(F, q, inside);
            const double h = F.H1[c * F.ns + l];
            h2 += h * h;
        }
        wh += h2 / 2.0;
    }
    const double w = 0.5 * p.eps0 * m.eps_r * we + 0.5 * p.mu0 * wh;
    return m.Ms > 0.0 ? w : 0.0;
}

// energy probes: partial b of probe pb sums cells [256 b, 256 b + 256) of the
// film's cell box into P.part[b] (film energy), or slots [256 b, 256 b + 256)
// of the grid (x fastest) into P.part[2 b], P.part[2 b + 1] (grid energy).  A
// block takes partials blockIdx.x, + gridDim.x, ...: a launch at a step that
// samples nothing is over with its few blocks (160 x 144 x 128: 7.4 us with a
// block a partial, 4.6 us; one that samples: 166 us with the ids of an edge's
// cells and their materials read one after the other, 70 us).
template <typename T>
__device__ __forceinline__ void probe_parts_body(const KParams<T> &p, int pb) {
    __shared__ double red[2][2][256];
    __shared__ EnergyMat tab[256];
    const ProbeDev &P = p.probes[pb];
    if ((P.kind != 2 && P.kind != 3) || (long long)blockIdx.x >= P.npart) return;
    long long sample;
    if (!probe_due(P, p.step[0], sample)) return;
    const int tid = (int)threadIdx.x;
    if (P.kind == 2) {
        const FilmDev F = film_desc(p.films, __builtin_amdgcn_readfirstlane(P.film));
        const unsigned ncell = (unsigned)F.cb[3] * F.cb[4] * F.cb[5];
        int w = 0;
        for (unsigned b = blockIdx.x; b < P.npart; b += gridDim.x, w ^= 1) {
            const unsigned t = b * 256u + tid;
            const double v = t < ncell ? film_cell_energy(p, F, t) : 0.0;
            const double s = block_tree2(red[w], tid, v, 0.0);
            if (tid == 0) P.part[b] = s;
        }
        return;
    }
    energy_mats(p, tab, tid);
    __syncthreads();
    const long long rows = (long long)p.n[1] * p.n[2];
    int w = 0;
    for (long long b = blockIdx.x; b < P.npart; b += gridDim.x, w ^= 1) {
        // the partial's first slot and row (one division of uniform values),
        // then the thread's own from there
        const long long t0 = b * 256;
        long long row;
        unsigned x;
        if (t0 >> 32) {
            row = t0 / p.n[0];
            x = (unsigned)(t0 - row * p.n[0]);
        } else {
            row = (unsigned)t0 / (unsigned)p.n[0];
            x = (unsigned)t0 - (unsigned)row * (unsigned)p.n[0];
        }
        const unsigned xt = x + (unsigned)tid, dr = xt / (unsigned)p.n[0];
        const long long rt = row + dr;
        double we = 0.0, wh = 0.0;
        if (rt < rows) {
            const unsigned k = (unsigned)rt / (unsigned)p.n[1];
            const int idx[3] = {(int)(xt - dr * (unsigned)p.n[0]), (int)((unsigned)rt - k * (unsigned)p.n[1]), (int)k};
            energy_site<T, 1>(p, tab, idx, we, wh);
        }
        const double s = block_tree2(red[w], tid, we, wh);
        if (tid == 0) P.part[2 * b] = s;
        if (tid == 64) P.part[2 * b + 1] = s;
    }
}

// row y < nprobe: probe y's partials; the row after them: the film-region state
// of an adjoint step (both read what the H/M launch will move)
template <typename T>
__global__ void __launch_bounds__(256) k_probe_parts(KParams<T> p, int nprobe, LossTape tape) {
    if ((int)blockIdx.y < nprobe)
        probe_parts_body(p, blockIdx.y);
    else if ((int)blockIdx.x < tape.nblk)
        tape_loss_body(p, tape.film, 1, tape.dst, blockIdx.x);
}

template <typename T>
__global__ void __launch_bounds__(256) k_probe_parts_batch(const KParams<T> *__restrict__ plist,
                                                           const int2 *__restrict__ work) {
    const int2 wk = work[blockIdx.y];
    probe_parts_body(plist[wk.x], wk.y);
}

template <typename T>
__global__ void __launch_bounds__(256) k_probes(KParams<T> p) {
    probes_body(p, blockIdx.x);
}

template <typename T>
__global__ void __launch_bounds__(256) k_probes_batch(const KParams<T> *__restrict__ plist, const int2 *__restrict__ work) {
    const int2 wk = work[blockIdx.x];
    probes_body(plist[wk.x], wk.y);
}

// ---------------------------------------------------------------------------
// discrete energy at an integer time: per-block partials of
// sum eps_e E^2, sum (H^2 - (hc curl E)^2) and sum H0_c M_c
// ---------------------------------------------------------------------------
// (partial b: tile b of 64 x 4 slots, x fastest)
template <typename T>
__global__ void __launch_bounds__(256) k_energy(KParams<T> p, double *part, unsigned gx, unsigned gy, unsigned nb) {
    __shared__ double red[2][2][256];
    __shared__ EnergyMat tab[256];
    const int t = threadIdx.x;
    energy_mats(p, tab, t);
    __syncthreads();
    int w = 0;
    for (unsigned b = blockIdx.x; b < nb; b += gridDim.x, w ^= 1) {
        const unsigned r = b / gx, k = r / gy;
        const int idx[3] = {(int)((b - r * gx) * 64u) + (t & 63), (int)((r - k * gy) * 4u) + (t >> 6), (int)k};
        double we = 0.0, wh = 0.0;
        if (idx[0] < p.n[0] && idx[1] < p.n[1]) energy_site<T, 0>(p, tab, idx, we, wh);
        const double s = block_tree2(red[w], t, we, wh);
        if (t == 0) part[2ll * b] = s;
        if (t == 64) part[2ll * b + 1] = s;
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_zeeman(KParams<T> p) {
    __shared__ double red[256];
    const int4 bt = p.blocktab[blockIdx.x];
    const int f = bt.x, c = bt.y;
    const FilmDev &F = p.films[f];
    const long long l = (long long)bt.z + threadIdx.x;
    double z = 0.0;
    if (l < F.ns) {
        int idx[3];
        idx[0] = F.b0[0] + (int)(l % F.bn[0]);
        idx[1] = F.b0[1] + (int)((l / F.bn[0]) % F.bn[1]);
        idx[2] = F.b0[2] + (int)(l / ((long long)F.bn[0] * F.bn[1]));
        (void)idx;
        if (F.prm[(c * 3) * F.ns + l] > 0.0) z = p.H0[c] * F.M[(c * 3 + c) * F.ns + l];
    }
    red[threadIdx.x] = z;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) p.partial[blockIdx.x] = red[0];
}

__global__ void k_sum_pairs(const double *part, long long n, double *out) {
    __shared__ double red[2][256];
    double a = 0.0, b = 0.0;
    for (long long t = threadIdx.x; t < n; t += blockDim.x) {
        a += part[2 * t];
        b += part[2 * t + 1];
    }
    red[0][threadIdx.x] = a;
    red[1][threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = red[0][0];
        out[1] = red[1][0];
    }
}

__global__ void k_sum(const double *part, long long n, double *out) {
    __shared__ double red[256];
    double a = 0.0;
    for (long long t = threadIdx.x; t < n; t += blockDim.x) a += part[t];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

// ---------------------------------------------------------------------------
// host-side launchers (explicit instantiation for float and double)
// ---------------------------------------------------------------------------
// the B^ prepass alone (the adjoint's view of a half step's input)
template <typename T>
hipError_t launch_bhat(const KParams<T> &p, int phase, hipStream_t s) {
    if (p.nblk_ext == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bhat<T>, dim3(p.nblk_ext), dim3(256), 0, s, p, phase);
    return hipGetLastError();
}

// films of at most this many blocks (of 256 faces, over all families) run
// their first half step and its prepass in one launch: a launch and its
// latency chain less against more loads, which up to some three blocks a CU
// hide in the chain (a face forms what it takes from the prepass itself: some
// 50 loads instead of 32, and the prepass's seven a face of the grown box stay
// beside it, for the second half step).  Two launches : one, us of a step:
// float32 51 blocks (128 x 64 x 64) 24.5 : 22.7, 297 28.5 : 25.6, 531 31.5 : 28.6,
// 798 37.0 : 35.5, 990 39.6 : 39.3; float64 123 blocks 25.9 : 23.7, 531 38.2 : 37.1,
// 654 46.6 : 45.4, 711 45.6 : 46.3, 798 47.8 : 49.1, 990 49.4 : 52.0; us of the
// kernels, 3864 blocks 47 : 60
template <typename T>
constexpr int kFilmFirstMax = sizeof(T) == 8 ? 680 : 1024;

template <typename T>
hipError_t launch_film(const KParams<T> &p, int nblk, int phase, int inc, hipStream_t s) {
    if (nblk == 0) return hipSuccess;
    if (phase == 1 && !inc && nblk <= kFilmFirstMax<T>) {
        hipLaunchKernelGGL(k_film_first<T>, dim3(nblk + p.nblk_ext), dim3(256), 0, s, p, nblk);
        return hipGetLastError();
    }
    // phase 2 follows a phase 1 whose kernels wrote its prepass
    if (phase == 1) hipLaunchKernelGGL(k_bhat<T>, dim3(p.nblk_ext), dim3(256), 0, s, p, phase);
    hipLaunchKernelGGL(k_film<T>, dim3(nblk), dim3(256), 0, s, p, phase, inc);
    return hipGetLastError();
}

__global__ void k_tick(long long *step) {
    if (threadIdx.x == 0) step[0] = step[0] + 1;
}

template <typename T>
__global__ void k_tick_batch(const KParams<T> *plist, const int *inst, int n) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) plist[inst[q]].step[0] = plist[inst[q]].step[0] + 1;
}

hipError_t launch_tick(long long *step, hipStream_t s) {
    hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, s, step);
    return hipGetLastError();
}

// blocks of an energy launch: eight a CU, each looping over its partials
constexpr int kPartBlocks = 2048;

template <typename T>
hipError_t launch_probes(const KParams<T> &p, int nprobe, int maxpart, hipStream_t s, bool folded,
                         const LossTape *tape) {
    const int rows = (maxpart > 0 ? nprobe : 0) + (tape ? 1 : 0);
    const int blocks = std::max(std::min(maxpart, kPartBlocks), tape ? tape->nblk : 0);
    if (rows > 0 && blocks > 0)
        hipLaunchKernelGGL(k_probe_parts<T>, dim3(blocks, rows), dim3(256), 0, s, p, maxpart > 0 ? nprobe : 0,
                           tape ? *tape : LossTape());
    if (nprobe > 0 && !folded) hipLaunchKernelGGL(k_probes<T>, dim3(nprobe), dim3(256), 0, s, p);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_energy(const KParams<T> &p, int nblk, double *part, double *out, hipStream_t s) {
    const unsigned gx = (p.n[0] + 63) / 64, gy = (p.n[1] + 3) / 4;
    const long long nb = (long long)gx * gy * p.n[2];
    hipLaunchKernelGGL(k_energy<T>, dim3((unsigned)std::min<long long>(nb, kPartBlocks)), dim3(256), 0, s, p, part,
                       gx, gy, (unsigned)nb);
    hipLaunchKernelGGL(k_sum_pairs, dim3(1), dim3(256), 0, s, part, nb, out);
    if (nblk) {
        hipLaunchKernelGGL(k_zeeman<T>, dim3(nblk), dim3(256), 0, s, p);
        hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, p.partial, (long long)nblk, out + 2);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_film_batch(const KParams<T> *plist, const int2 *work_ext, int n_ext, const int2 *work, int n,
                             int phase, int inc, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (phase == 1 && !inc && n <= kFilmFirstMax<T>) {
        hipLaunchKernelGGL(k_film_first_batch<T>, dim3(n + n_ext), dim3(256), 0, s, plist, work_ext, work, n);
        return hipGetLastError();
    }
    if (phase == 1) hipLaunchKernelGGL(k_bhat_batch<T>, dim3(n_ext), dim3(256), 0, s, plist, work_ext, phase);
    hipLaunchKernelGGL(k_film_batch<T>, dim3(n), dim3(256), 0, s, plist, work, phase, inc);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_probes_batch(const KParams<T> *plist, const int2 *work, int n, int maxpart, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (maxpart > 0) hipLaunchKernelGGL(k_probe_parts_batch<T>, dim3(std::min(maxpart, kPartBlocks), n), dim3(256), 0, s, plist, work);
    hipLaunchKernelGGL(k_probes_batch<T>, dim3(n), dim3(256), 0, s, plist, work);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tick_batch(const KParams<T> *plist, const int *inst, int n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_tick_batch<T>, dim3((n + 63) / 64), dim3(64), 0, s, plist, inst, n);
    return hipGetLastError();
}

#define MPX_INSTANTIATE(T)                                                                  \
    template hipError_t launch_bhat<T>(const KParams<T> &, int, hipStream_t);               \
    template hipError_t launch_film<T>(const KParams<T> &, int, int, int, hipStream_t);     \
    template hipError_t launch_film_batch<T>(const KParams<T> *, const int2 *, int, const int2 *, int, int, int, \
                                             hipStream_t);                                  \
    template hipError_t launch_probes_batch<T>(const KParams<T> *, const int2 *, int, int, hipStream_t); \
    template hipError_t launch_tick_batch<T>(const KParams<T> *, const int *, int, hipStream_t);   \
    template hipError_t launch_probes<T>(const KParams<T> &, int, int, hipStream_t, bool, const LossTape *); \
    template hipError_t launch_energy<T>(const KParams<T> &, int, double *, double *, hipStream_t);

MPX_INSTANTIATE(float)
MPX_INSTANTIATE(double)

} // namespace mpx
