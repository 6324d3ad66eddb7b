// Fused El-WaveHoltz step on a mapped 3-D grid (Sec. 4.1 in three
// dimensions; the partial toroidal shell of Sec. 5.11).
//
// The unit cube (q, r, s) is mapped to the domain; with G_a = J grad a and
// the 3x3 blocks K^{ab} = (1/J) [lam G_a G_b^T + mu (G_a . G_b) I +
// mu G_b G_a^T], L_h is minus the gradient of the discrete energy
//   E_h = 1/2 sum_a sum_{a-edges} w_e (D+a U)^T Kbar^aa (D+a U)
//       + sum_{a != b} sum_{unknown n} w_n (Dh_a U)_n^T K^ab_n (Dh_b U)_n / 2
// (Kbar the mean over the edge's two nodes, Dh central, one-sided into the
// domain on a free s face, w the trapezoid weights: 1/2 on a free s face).
// Row p of L_h is gathered directly:
//   L_p = sum_a sum_{+-} w_e Kbar^aa (U_{p +- e_a} - U_p) / h_a^2
//       - sum_{a != b} sum_n (Dh_a)_{n,p} w_n K^ab_n (Dh_b U)_n,
// where K^ab v = (lam/J) G_a (G_b . v) + (mu/J) (G_b (G_a . v) + (G_a . G_b) v)
// is formed from lam/J, mu/J and the nine metric values at the node (no 3x3
// block is stored).  The step is the corrected leapfrog of Sec. 4.3 with mass
// rho J (a = c dt^2 / (rho J), forcing J f) and the trapezoid accumulation
// of eq. el_WHI_OP fused in, as in the Cartesian kernels.
//
// Mapping: one thread per node, 64 consecutive q nodes per wavefront, one
// (r, s) row per workgroup, XCD-banded; every neighbour value is loaded
// (the 19-point footprint and the coefficients of the six face neighbours
// are served by the caches) in straight-line code, so a wavefront has its
// whole footprint in flight at once; one time step per launch.
#include <algorithm>

#include "elwh_internal.h"
#include "lanes.h"
#include "xcd.h"

namespace elwh {

struct ArgsC3 {
    int nq, nr, ns;
    int64_t P, PS, CS;
    int klo, khi, free_lo, free_hi;
    double hq, hr, hs;
    double w, w0, fc;
    int final_;
};

template <typename T>
struct Metric3 {
    const T* g[9];   // G_q, G_r, G_s by component
};

__device__ __forceinline__ void acc_add_c3(double& hi, double& lo, double x, bool comp) {
    if (comp) {
        const double t = hi + x;
        const double z = t - hi;
        const double e = (hi - (t - z)) + (x - z);
        hi = t;
        lo += e;
    } else {
        hi += x;
    }
}

template <typename T, typename U, int MODE, bool FORCE, bool COMP>
__global__ __launch_bounds__(64) void curv3d_kernel(const U* __restrict__ u, const T* uprev, T* unext,
                                                   const double* __restrict__ xbase, T* __restrict__ u0out,
                                                   double* __restrict__ acc, float* __restrict__ acclo,
                                                   const T* __restrict__ ca, const T* __restrict__ cl,
                                                   const T* __restrict__ cm, Metric3<T> G, const T* __restrict__ f,
                                                   ArgsC3 A) {
    const int nbx = (A.nq - 1 + 63) / 64, nrr = A.nr - 1, npl = A.khi - A.klo + 1;
    int t;
    if (!xcd_tile((int)blockIdx.x, nbx * nrr * npl, t)) return;
    const int i = 1 + 64 * (t % nbx) + (int)threadIdx.x;
    const int j = 1 + (t / nbx) % nrr;
    const int k = A.klo + t / (nbx * nrr);
    if (i > A.nq - 1) return;
    const int64_t P = A.P, PS = A.PS, CS = A.CS;
    const int64_t o = (int64_t)k * PS + (int64_t)j * P + i;

    // The gather below is straight-line code: every load is issued without a
    // branch between it and the next, so a wavefront has its whole footprint
    // in flight at once.  j and k are uniform over the wavefront (one (r, s)
    // row per workgroup), so every test on them is a uniform branch; the two
    // tests on i (the q neighbours' being unknowns) are masks.
    const bool flo = A.free_lo && k == 0, fhi = A.free_hi && k == A.ns;
    const bool on_free = flo || fhi;
    const T wp = on_free ? (T)0.5 : (T)1;   // node weight of p, and of its in-plane edges
    const T cq = (T)(0.5 / A.hq), cr = (T)(0.5 / A.hr);
    // D_s at the plane of p: central, one-sided on a free face (the missing
    // plane is read clamped, i.e. as the plane of p itself, and the
    // coefficient doubles)
    const T csp = on_free ? (T)(1.0 / A.hs) : (T)(0.5 / A.hs);
    const int64_t sm = k > 0 ? -PS : 0, sp = k < A.ns ? PS : 0;
    const T iq2 = (T)(1.0 / (A.hq * A.hq)), ir2 = (T)(1.0 / (A.hr * A.hr)), is2 = (T)(1.0 / (A.hs * A.hs));

    struct V3 {
        T x, y, z;
    };
    struct Co {
        T l, m;        // lambda / J, mu / J
        V3 g[3];       // G_q, G_r, G_s
    };
    auto ld = [&](int64_t q) { return V3{(T)u[q], (T)u[q + CS], (T)u[q + 2 * CS]}; };
    auto ldc = [&](int64_t q) {
        Co c;
        c.l = cl[q];
        c.m = cm[q];
#pragma unroll
        for (int a = 0; a < 3; ++a) c.g[a] = V3{G.g[3 * a][q], G.g[3 * a + 1][q], G.g[3 * a + 2][q]};
        return c;
    };
    auto dot = [](const V3& p, const V3& q) { return p.x * q.x + p.y * q.y + p.z * q.z; };
    auto sub = [](const V3& p, const V3& q) { return V3{p.x - q.x, p.y - q.y, p.z - q.z}; };
    // K^ab v = (lambda/J) G_a (G_b . v) + (mu/J) (G_b (G_a . v) + (G_a . G_b) v)
    auto kab = [&](const Co& c, int a, int b, const V3& v) {
        const V3& ga = c.g[a];
        const V3& gb = c.g[b];
        const T gbv = dot(gb, v), gav = dot(ga, v), gab = dot(ga, gb);
        return V3{c.l * ga.x * gbv + c.m * (gb.x * gav + gab * v.x), c.l * ga.y * gbv + c.m * (gb.y * gav + gab * v.y),
                  c.l * ga.z * gbv + c.m * (gb.z * gav + gab * v.z)};
    };
    T Lx = 0, Ly = 0, Lz = 0;
    auto acc3 = [&](T s_, const V3& v) {
        Lx += s_ * v.x;
        Ly += s_ * v.y;
        Lz += s_ * v.z;
    };

    // footprint of u: p, its six face neighbours, its twelve in-plane diagonal neighbours
    const V3 u0 = ld(o);
    const V3 uqm = ld(o - 1), uqp = ld(o + 1), urm = ld(o - P), urp = ld(o + P), usm = ld(o + sm), usp = ld(o + sp);
    const V3 qr_mm = ld(o - 1 - P), qr_mp = ld(o - 1 + P), qr_pm = ld(o + 1 - P), qr_pp = ld(o + 1 + P);
    const V3 qs_mm = ld(o - 1 + sm), qs_mp = ld(o - 1 + sp), qs_pm = ld(o + 1 + sm), qs_pp = ld(o + 1 + sp);
    const V3 rs_mm = ld(o - P + sm), rs_mp = ld(o - P + sp), rs_pm = ld(o + P + sm), rs_pp = ld(o + P + sp);
    const V3 dqm = sub(uqm, u0), dqp = sub(uqp, u0), drm = sub(urm, u0), drp = sub(urp, u0);
    const V3 dsm = sub(usm, u0), dsp = sub(usp, u0);   // 0 across a free face (clamped)

    // edge terms, p's half: sum_a sum_+- w_e/2 K^aa_p (U_n - U_p) / h_a^2
    {
        const Co c = ldc(o);
        const T eq = (T)0.5 * wp * iq2, er = (T)0.5 * wp * ir2, es = (T)0.5 * is2;
        acc3(eq, kab(c, 0, 0, dqm));
        acc3(eq, kab(c, 0, 0, dqp));
        acc3(er, kab(c, 1, 1, drm));
        acc3(er, kab(c, 1, 1, drp));
        acc3(es, kab(c, 2, 2, dsm));
        acc3(es, kab(c, 2, 2, dsp));
        if (on_free) {
            // the one-sided D_s at p itself: (D_s)_pp = -+1/h_s, weight 1/2
            const T s0 = (T)(flo ? 0.5 / A.hs : -0.5 / A.hs);   // -(D_s)_pp w_p
            acc3(s0, kab(c, 2, 0, V3{(uqp.x - uqm.x) * cq, (uqp.y - uqm.y) * cq, (uqp.z - uqm.z) * cq}));
            acc3(s0, kab(c, 2, 1, V3{(urp.x - urm.x) * cr, (urp.y - urm.y) * cr, (urp.z - urm.z) * cr}));
        }
    }
    // q neighbours: the other half of their edge term, and their cross terms
    // -(D_q)_np w_n K^qb_n (D_b U)_n, (D_q)_np = -+1/(2 h_q) for n = p +- e_q
    {
        const T mm = i - 1 >= 1 ? (T)1 : (T)0, mp = i + 1 <= A.nq - 1 ? (T)1 : (T)0;   // unknowns
        const Co cm_ = ldc(o - 1), cp_ = ldc(o + 1);
        const T eq = (T)0.5 * wp * iq2;
        acc3(eq, kab(cm_, 0, 0, dqm));
        acc3(eq, kab(cp_, 0, 0, dqp));
        const T sm_ = -cq * wp * mm, sp_ = cq * wp * mp;   // -(D_q)_np w_n, masked
        acc3(sm_, kab(cm_, 0, 1, V3{(qr_mp.x - qr_mm.x) * cr, (qr_mp.y - qr_mm.y) * cr, (qr_mp.z - qr_mm.z) * cr}));
        acc3(sm_, kab(cm_, 0, 2, V3{(qs_mp.x - qs_mm.x) * csp, (qs_mp.y - qs_mm.y) * csp, (qs_mp.z - qs_mm.z) * csp}));
        acc3(sp_, kab(cp_, 0, 1, V3{(qr_pp.x - qr_pm.x) * cr, (qr_pp.y - qr_pm.y) * cr, (qr_pp.z - qr_pm.z) * cr}));
        acc3(sp_, kab(cp_, 0, 2, V3{(qs_pp.x - qs_pm.x) * csp, (qs_pp.y - qs_pm.y) * csp, (qs_pp.z - qs_pm.z) * csp}));
    }
    // r neighbours (uniform tests)
    {
        const Co cm_ = ldc(o - P), cp_ = ldc(o + P);
        const T er = (T)0.5 * wp * ir2;
        acc3(er, kab(cm_, 1, 1, drm));
        acc3(er, kab(cp_, 1, 1, drp));
        if (j - 1 >= 1) {
            const T s_ = -cr * wp;
            acc3(s_, kab(cm_, 1, 0, V3{(qr_pm.x - qr_mm.x) * cq, (qr_pm.y - qr_mm.y) * cq, (qr_pm.z - qr_mm.z) * cq}));
            acc3(s_, kab(cm_, 1, 2, V3{(rs_mp.x - rs_mm.x) * csp, (rs_mp.y - rs_mm.y) * csp, (rs_mp.z - rs_mm.z) * csp}));
        }
        if (j + 1 <= A.nr - 1) {
            const T s_ = cr * wp;
            acc3(s_, kab(cp_, 1, 0, V3{(qr_pp.x - qr_mp.x) * cq, (qr_pp.y - qr_mp.y) * cq, (qr_pp.z - qr_mp.z) * cq}));
            acc3(s_, kab(cp_, 1, 2, V3{(rs_pp.x - rs_pm.x) * csp, (rs_pp.y - rs_pm.y) * csp, (rs_pp.z - rs_pm.z) * csp}));
        }
    }
    // s neighbours (uniform tests): across a free face there is none (its
    // edge difference is 0 by the clamped read); -(D_s)_np w_n is +-1/(2 h_s)
    // also where n lies on a free face (one-sided coefficient 1/h_s, weight 1/2)
    {
        const Co cm_ = ldc(o + sm), cp_ = ldc(o + sp);
        const T es = (T)0.5 * is2;
        acc3(es, kab(cm_, 2, 2, dsm));
        acc3(es, kab(cp_, 2, 2, dsp));
        const T cs2 = (T)(0.5 / A.hs);
        if (k - 1 >= A.klo) {
            acc3(-cs2, kab(cm_, 2, 0, V3{(qs_pm.x - qs_mm.x) * cq, (qs_pm.y - qs_mm.y) * cq, (qs_pm.z - qs_mm.z) * cq}));
            acc3(-cs2, kab(cm_, 2, 1, V3{(rs_pm.x - rs_mm.x) * cr, (rs_pm.y - rs_mm.y) * cr, (rs_pm.z - rs_mm.z) * cr}));
        }
        if (k + 1 <= A.khi) {
            acc3(cs2, kab(cp_, 2, 0, V3{(qs_pp.x - qs_mp.x) * cq, (qs_pp.y - qs_mp.y) * cq, (qs_pp.z - qs_mp.z) * cq}));
            acc3(cs2, kab(cp_, 2, 1, V3{(rs_pp.x - rs_mp.x) * cr, (rs_pp.y - rs_mp.y) * cr, (rs_pp.z - rs_mp.z) * cr}));
        }
    }
    const T uc[3] = {u0.x, u0.y, u0.z};
    const T L[3] = {Lx, Ly, Lz};

    // L_h / w_p, then the corrected leapfrog with the trapezoid accumulation
    const T iw = (T)1 / wp;
    const T a_ = ca[o];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int64_t oq = o + q * CS;
        T Lq = L[q] * iw;
        if constexpr (FORCE) Lq -= (T)A.fc * f[oq];
        double hq = 0.0, lq = 0.0;
        T nq;
        if constexpr (MODE == 0) {
            hq = acc[oq];
            if constexpr (COMP) lq = acclo[oq];
            nq = (T)2 * uc[q] - uprev[oq] + a_ * Lq;
        } else {
            hq = xbase ? xbase[oq] : 0.0;
            nq = uc[q] + (T)0.5 * a_ * Lq;
            acc_add_c3(hq, lq, A.w0 * (double)uc[q], COMP);
            if (u0out) u0out[oq] = uc[q];
        }
        unext[oq] = nq;
        acc_add_c3(hq, lq, A.w * (double)nq, COMP);
        if (COMP && A.final_) {
            acc[oq] = hq + lq;
        } else {
            acc[oq] = hq;
            if constexpr (COMP) acclo[oq] = (float)lq;
        }
    }
}

// ---- FP64, all but small grids: marching workgroups that share the fluxes ----------------
//
// The gather above forms every node's contribution K^ab (D_b U) again at each of
// the nodes that use it: 1353 instructions and 134 loads per node, 171 us per
// step on the shell of 400 x 120 x 40 points, twice what its 216 B per update
// take.  Here a node forms its contributions once and hands them over:
//   F^a = sum_{b != a} K^ab D_b U     the cross flux along axis a,
//   h^+-_a = K^aa (U_{p +- e_a} - U_p)   its halves of the two edge terms,
// and along axis a it exports (to the node below and above it)
//   X^-_a = F^a / (2 h_a) - h^-_a / (2 h_a^2),   X^+_a = -F^a / (2 h_a) - h^+_a / (2 h_a^2),
// so L_p = sum_a [X^-_a of p + e_a, X^+_a of p - e_a, (h^-_a + h^+_a) / (2 h_a^2) of p itself].
// The exports along an axis need only the differences along the other two, so
// one halo node per side is enough.
//
// A workgroup of 8 wavefronts takes 8 rows (r) of 64 nodes (q), of which 6 x 62
// are its own, and marches along s: q exports go by DPP, r exports through LDS
// (two buffers, one barrier per plane), s exports stay in registers.  Every
// array is read once per plane, one plane ahead.  A workgroup's registers fill a CU;
// the march is split along s into the rounds of workgroups that cost least (march3_chunk).
// On a free s face (trapezoid weight 1/2): dividing the row by the weight leaves
// the in-plane terms as they are and doubles those along s; D_s is one-sided, and
// the face's own F^s enters with its own coefficient.
constexpr int M3_NW = 8, M3_Q = 62, M3_R = M3_NW - 2;

struct V3d {
    double x, y, z;
};
__device__ __forceinline__ double dot3(const V3d& a, const V3d& b) { return fma(a.x, b.x, fma(a.y, b.y, a.z * b.z)); }
__device__ __forceinline__ V3d sub3(const V3d& a, const V3d& b) { return V3d{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3d mul3(double s, const V3d& a) { return V3d{s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ V3d fma3(double s, const V3d& a, const V3d& b) {
    return V3d{fma(s, a.x, b.x), fma(s, a.y, b.y), fma(s, a.z, b.z)};
}
__device__ __forceinline__ V3d from_left3(const V3d& a) {
    return V3d{lane_from_left_z(a.x), lane_from_left_z(a.y), lane_from_left_z(a.z)};
}
__device__ __forceinline__ V3d from_right3(const V3d& a) {
    return V3d{lane_from_right_z(a.x), lane_from_right_z(a.y), lane_from_right_z(a.z)};
}

struct Coef3 {
    double l, m;       // lambda / J, mu / J
    V3d g[3];
};

template <int MODE, bool FORCE>
__global__ __launch_bounds__(64 * M3_NW) void curv3d_march_kernel(const double* __restrict__ u, const double* uprev,
                                                                 double* unext, const double* __restrict__ xbase,
                                                                 double* __restrict__ acc,
                                                                 const double* __restrict__ ca,
                                                                 const double* __restrict__ cl,
                                                                 const double* __restrict__ cm, Metric3<double> G,
                                                                 const double* __restrict__ f, ArgsC3 A, int tz) {
    __shared__ double us[2][M3_NW][3][64];   // U of the plane being worked on, and of the next
    __shared__ double xs[2][M3_NW][6][64];   // r exports: to the row below, to the row above
    const int nbq = (A.nq - 1 + M3_Q - 1) / M3_Q, nbr = (A.nr - 1 + M3_R - 1) / M3_R;
    const int nbs = (A.khi - A.klo + tz) / tz;
    int t;
    if (!xcd_tile((int)blockIdx.x, nbq * nbr * nbs, t)) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = (t % nbq) * M3_Q + lane;                 // own columns: lanes 1 .. 62
    const int j = ((t / nbq) % nbr) * M3_R + w;            // own rows: wavefronts 1 .. 6
    const int k0 = A.klo + (t / (nbq * nbr)) * tz, k1 = min(k0 + tz - 1, A.khi);
    const bool in = i <= A.nq && j <= A.nr;
    const bool own = lane >= 1 && lane <= M3_Q && w >= 1 && w <= M3_R && i <= A.nq - 1 && j <= A.nr - 1;
    const bool unk = i >= 1 && i <= A.nq - 1 && j >= 1 && j <= A.nr - 1;   // unknown in its plane
    const int64_t CS = A.CS, PS = A.PS, o0 = (int64_t)j * A.P + i;
    const double cq = 0.5 / A.hq, cr = 0.5 / A.hr, cs = 0.5 / A.hs;
    const double eq = 0.5 / (A.hq * A.hq), er = 0.5 / (A.hr * A.hr), es = 0.5 / (A.hs * A.hs);

    auto ldu = [&](int k) {
        V3d v{0.0, 0.0, 0.0};
        if (in && k >= 0 && k <= A.ns) {
            const int64_t o = o0 + k * PS;
            v = V3d{u[o], u[o + CS], u[o + 2 * CS]};
        }
        return v;
    };
    auto ldc = [&](int k) {
        Coef3 c{};
        if (in && k >= 0 && k <= A.ns) {
            const int64_t o = o0 + k * PS;
            c.l = cl[o];
            c.m = cm[o];
#pragma unroll
            for (int a = 0; a < 3; ++a) c.g[a] = V3d{G.g[3 * a][o], G.g[3 * a + 1][o], G.g[3 * a + 2][o]};
        }
        return c;
    };
    auto put_u = [&](const V3d& v, int b) {
        us[b][w][0][lane] = v.x;
        us[b][w][1][lane] = v.y;
        us[b][w][2][lane] = v.z;
    };

    // planes k0 - 1 (exports upwards only) .. k1 + 1 (exports downwards only)
    const int ka = max(k0 - 1, 0), kb = min(k1 + 1, A.ns);
    V3d um = ldu(ka - 1), uc = ldu(ka), up = ldu(ka + 1);
    Coef3 c = ldc(ka);
    V3d L{0.0, 0.0, 0.0};      // the row of plane kk - 1, all but the export from plane kk
    V3d xup{0.0, 0.0, 0.0};    // s export of plane kk - 1 to plane kk
    put_u(uc, ka & 1);
    __syncthreads();

    // centre values of a plane, loaded at the top of the iteration that finishes it
    struct Centre3 {
        double a;
        V3d old, h, f;
    };
    auto ld_centre = [&](int k) {
        Centre3 e{};
        if (own && k >= k0 && k <= k1) {
            const int64_t o = o0 + k * PS;
            e.a = ca[o];
            const double* hb = MODE == 0 ? acc : xbase;
            if (hb) e.h = V3d{hb[o], hb[o + CS], hb[o + 2 * CS]};
            if constexpr (MODE == 0) e.old = V3d{uprev[o], uprev[o + CS], uprev[o + 2 * CS]};
            if constexpr (FORCE) e.f = V3d{f[o], f[o + CS], f[o + 2 * CS]};
        }
        return e;
    };
    auto finish = [&](int k, const Centre3& e, const V3d& uk, const V3d& down) {   // plane k, with the export of k + 1
        const bool face = (A.free_lo && k == 0) || (A.free_hi && k == A.ns);
        const V3d R = fma3(face ? 2.0 : 1.0, down, L);
        if (own && k >= k0 && k <= k1) {
            const double Lq[3] = {R.x, R.y, R.z}, uq[3] = {uk.x, uk.y, uk.z}, oq[3] = {e.old.x, e.old.y, e.old.z};
            const double hq[3] = {e.h.x, e.h.y, e.h.z}, fq[3] = {e.f.x, e.f.y, e.f.z};
            const int64_t o = o0 + k * PS;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double s = FORCE ? Lq[q] - A.fc * fq[q] : Lq[q];
                if constexpr (MODE == 0) {
                    const double n = fma(e.a, s, fma(2.0, uq[q], -oq[q]));
                    unext[o + q * CS] = n;
                    acc[o + q * CS] = fma(A.w, n, hq[q]);
                } else {
                    const double n = fma(0.5 * e.a, s, uq[q]);
                    unext[o + q * CS] = n;
                    acc[o + q * CS] = fma(A.w, n, fma(A.w0, uq[q], hq[q]));
                }
            }
        }
    };

    for (int kk = ka; kk <= kb; ++kk) {
        const int b = kk & 1;
        const Centre3 e = ld_centre(kk - 1);
        const V3d upp = ldu(kk + 2);
        const Coef3 cn = kk < kb ? ldc(kk + 1) : Coef3{};
        const bool flo = A.free_lo && kk == 0, fhi = A.free_hi && kk == A.ns;
        const bool plane = kk >= A.klo && kk <= A.khi;   // unknown planes
        const double mask = unk && plane ? 1.0 : 0.0;
        // differences: clamped across a free face, where D_s doubles
        const int wm = w > 0 ? w - 1 : w, wn = w < M3_NW - 1 ? w + 1 : w;   // (halo rows need no D_r)
        const V3d rm{us[b][wm][0][lane], us[b][wm][1][lane], us[b][wm][2][lane]};
        const V3d rp{us[b][wn][0][lane], us[b][wn][1][lane], us[b][wn][2][lane]};
        const V3d qm = from_left3(uc), qp = from_right3(uc);
        const V3d sm = flo ? uc : um, sp = fhi ? uc : up;
        const double cs2 = (flo || fhi ? 2.0 : 1.0) * cs;
        const V3d dq = mul3(cq, sub3(qp, qm)), dr = mul3(cr, sub3(rp, rm)), ds = mul3(cs2, sub3(sp, sm));
        // cross fluxes: F^a = l G_a sum_{b != a} G_b . d_b + m sum_{b != a} (G_b (G_a . d_b) + (G_a . G_b) d_b)
        const V3d &gq = c.g[0], &gr = c.g[1], &gs = c.g[2];
        const double qq = dot3(gq, dq), rr = dot3(gr, dr), ss = dot3(gs, ds);
        const double Sqr = dot3(gq, gr), Sqs = dot3(gq, gs), Srs = dot3(gr, gs);
        const double lm = mask * c.l, mm = mask * c.m;
        auto cross = [&](const V3d& ga, double tr, const V3d& gb, double gab, double Sab, const V3d& db, const V3d& gc,
                         double gac, double Sac, const V3d& dc) {
            V3d v = mul3(gab, gb);
            v = fma3(Sab, db, v);
            v = fma3(gac, gc, v);
            v = fma3(Sac, dc, v);
            return fma3(lm * tr, ga, mul3(mm, v));
        };
        const V3d Fq = cross(gq, rr + ss, gr, dot3(gq, dr), Sqr, dr, gs, dot3(gq, ds), Sqs, ds);
        const V3d Fr = cross(gr, qq + ss, gq, dot3(gr, dq), Sqr, dq, gs, dot3(gr, ds), Srs, ds);
        const V3d Fs = cross(gs, qq + rr, gq, dot3(gs, dq), Sqs, dq, gr, dot3(gs, dr), Srs, dr);
        // halves of the edge terms, K^aa d = (l + m) G_a (G_a . d) + m |G_a|^2 d, over 2 h_a^2
        auto half = [&](const V3d& g, double e, double S, const V3d& d) {
            return fma3(e * (c.l + c.m) * dot3(g, d), g, mul3(e * c.m * S, d));
        };
        const double Sqq = dot3(gq, gq), Srr = dot3(gr, gr), Sss = dot3(gs, gs);
        const V3d hqm = half(gq, eq, Sqq, sub3(qm, uc)), hqp = half(gq, eq, Sqq, sub3(qp, uc));
        const V3d hrm = half(gr, er, Srr, sub3(rm, uc)), hrp = half(gr, er, Srr, sub3(rp, uc));
        const V3d hsm = half(gs, es, Sss, sub3(sm, uc)), hsp = half(gs, es, Sss, sub3(sp, uc));
        // r exports and the next plane's U, then the barrier
        {
            const V3d xm = fma3(cr, Fr, mul3(-1.0, hrm)), xp = fma3(-cr, Fr, mul3(-1.0, hrp));
            double(&x)[6][64] = xs[b][w];
            x[0][lane] = xm.x;
            x[1][lane] = xm.y;
            x[2][lane] = xm.z;
            x[3][lane] = xp.x;
            x[4][lane] = xp.y;
            x[5][lane] = xp.z;
        }
        put_u(up, b ^ 1);
        // q and s exports meanwhile
        const V3d xqm = fma3(cq, Fq, mul3(-1.0, hqm)), xqp = fma3(-cq, Fq, mul3(-1.0, hqp));
        const V3d xsm = fma3(cs, Fs, mul3(-1.0, hsm)), xsp = fma3(-cs, Fs, mul3(-1.0, hsp));
        const V3d fromq = from_right3(xqm), fromq2 = from_left3(xqp);
        const double iw = flo || fhi ? 2.0 : 1.0;
        V3d own_s = fma3(1.0, hsm, hsp);
        if (flo) own_s = fma3(cs, Fs, own_s);    // -(D_s)_pp w_p = 1 / (2 h_s) on the lower face
        if (fhi) own_s = fma3(-cs, Fs, own_s);
        V3d Ln{hqm.x + hqp.x + hrm.x + hrp.x + fromq.x + fromq2.x, hqm.y + hqp.y + hrm.y + hrp.y + fromq.y + fromq2.y,
               hqm.z + hqp.z + hrm.z + hrp.z + fromq.z + fromq2.z};
        Ln = fma3(iw, V3d{own_s.x + xup.x, own_s.y + xup.y, own_s.z + xup.z}, Ln);
        __syncthreads();
        {
            const double(&em)[6][64] = xs[b][wm];   // from the row below: its upward export
            const double(&ep)[6][64] = xs[b][wn];   // from the row above: its downward export
            Ln.x += em[3][lane] + ep[0][lane];
            Ln.y += em[4][lane] + ep[1][lane];
            Ln.z += em[5][lane] + ep[2][lane];
        }
        finish(kk - 1, e, um, xsm);
        L = Ln;
        xup = xsp;
        um = uc;
        uc = up;
        up = upp;
        c = cn;
    }
    // the last plane where nothing lies above it (a free face)
    if (kb == k1) finish(k1, ld_centre(k1), um, V3d{0.0, 0.0, 0.0});
}

// Planes per chunk along s, one workgroup per CU at a time: the fewest rounds
// times planes (a chunk works on two planes more than it owns).  The shell's 140
// columns of 40 planes in one round use 140 of 256 CUs: 124 us per step; in five
// chunks (three rounds of 10 planes) 95.
static int march3_chunk(int nb, int np) {
    int tz = np;
    int64_t best = (int64_t)1 << 60;
    for (int z = 1; z <= np; ++z) {
        const int64_t cost = ((int64_t)nb * ((np + z - 1) / z) + 255) / 256 * (z + 2);
        if (cost <= best) {
            best = cost;
            tz = z;
        }
    }
    return tz;
}
static int march3_columns(int nq, int nr) { return ((nq - 1 + M3_Q - 1) / M3_Q) * ((nr - 1 + M3_R - 1) / M3_R); }

// The march works through its planes in turn (3.0 us and 2.25 us per plane); the
// gather has every node in flight at once (3.4 us, 4.2 us per 1000 wavefronts of 64
// nodes along q, and 1 us once a CU has more than eight of them).  Fitted to up to
// 4000 wavefronts, where they cross; us per step, gather against march: 40^3 9.7 /
// 11.8, 44^3 10.8 / 12.0, 63 x 63 x 30 11.2 / 12.3, 120 x 36 x 20 9.3 / 10.2, 300 x 3 x
// 300 15.8 / 17.3; 47^3 13.4 / 12.1, 150 x 45 x 15 13.6 / 12.1, 63 x 63 x 35 14.1 /
// 12.4, 200 x 200 x 2 16.8 / 10.7, 400 x 120 x 40 171 / 95.
bool march3_pays(int nq, int nr, int ns, int np) {
    const int nb = march3_columns(nq, nr), tz = march3_chunk(nb, np);
    const int64_t rounds = ((int64_t)nb * ((np + tz - 1) / tz) + 255) / 256;
    const int64_t waves = (int64_t)((nq - 1 + 63) / 64) * (nr - 1) * np;
    return 3.0 + 2.25 * (double)(rounds * std::min(tz + 2, ns + 1)) <
           3.4 + 4.2e-3 * (double)waves + (waves > 8 * 256 ? 1.0 : 0.0);
}

template <int MODE>
static void launch_march3(bool force, const ArgsC3& A, hipStream_t s, const double* u, const double* uprev,
                          double* unext, const double* xbase, double* acc, const double* ca, const double* cl,
                          const double* cm, const Metric3<double>& G, const double* f) {
    const int nb = march3_columns(A.nq, A.nr), np = A.khi - A.klo + 1, tz = march3_chunk(nb, np);
    const dim3 grid((unsigned)xcd_grid(nb * ((np + tz - 1) / tz)));
    if (force)
        hipLaunchKernelGGL((curv3d_march_kernel<MODE, true>), grid, dim3(64 * M3_NW), 0, s, u, uprev, unext, xbase, acc,
                           ca, cl, cm, G, f, A, tz);
    else
        hipLaunchKernelGGL((curv3d_march_kernel<MODE, false>), grid, dim3(64 * M3_NW), 0, s, u, uprev, unext, xbase,
                           acc, ca, cl, cm, G, f, A, tz);
}

bool tile_valid_curv3(bool fp32, int V, int TY) {
    (void)fp32;
    return V == 1 && TY == 4;
}

template <typename T, typename U, int MODE>
static void launch_c3(bool force, bool comp, const ArgsC3& A, hipStream_t s, const U* u, const T* uprev, T* unext,
                      const double* xbase, T* u0out, double* acc, float* acclo, const T* ca, const T* cl,
                      const T* cm, const Metric3<T>& G, const T* f) {
    const int nbx = (A.nq - 1 + 63) / 64;
    const dim3 grid((unsigned)xcd_grid(nbx * (A.nr - 1) * (A.khi - A.klo + 1)));
#define ELWH_LC3(F, CMP)                                                                                        \
    hipLaunchKernelGGL((curv3d_kernel<T, U, MODE, F, CMP>), grid, dim3(64), 0, s, u, uprev, unext, xbase, u0out, \
                       acc, acclo, ca, cl, cm, G, f, A)
    if (force) {
        if (comp) ELWH_LC3(true, true); else ELWH_LC3(true, false);
    } else {
        if (comp) ELWH_LC3(false, true); else ELWH_LC3(false, false);
    }
#undef ELWH_LC3
}

void run_filter_curv3d(elwh_ctx* c, const double* x, bool with_force, bool amode, bool fp32, double* out) {
    hipStream_t s = c->stream;
    ArgsC3 A;
    A.nq = c->L.nx;
    A.nr = c->L.ny;
    A.ns = c->L.nz;
    A.P = c->L.P;
    A.PS = c->L.PS;
    A.CS = c->L.CS;
    A.klo = c->mr.lo;
    A.khi = c->mr.hi;
    A.free_lo = c->mr.free_lo;
    A.free_hi = c->mr.free_hi;
    A.hq = 1.0 / c->L.nx;
    A.hr = 1.0 / c->L.ny;
    A.hs = 1.0 / c->L.nz;
    A.final_ = 0;
    const int nsteps = c->plan.nt * c->opts.periods;
    const double sgn = amode ? -1.0 : 1.0;
    const bool comp = fp32 && c->opts.compensated;
    double* acc = out;
    float* lo = c->acc_lo;
    A.w0 = sgn * c->w[0];
    A.w = sgn * c->w[1];
    A.fc = c->cosn[0];
    if (!fp32) {
        Metric3<double> G;
        for (int q = 0; q < 9; ++q) G.g[q] = c->cg[q];
        double *b0 = c->s64[0], *b1 = c->s64[1];
        prof_mark(c, 0);
        const bool march = march3_pays(A.nq, A.nr, A.ns, A.khi - A.klo + 1);
        if (march)
            launch_march3<1>(with_force, A, s, x, nullptr, b1, amode ? x : nullptr, acc, c->ca, c->cl, c->cm, G, c->f64);
        else
            launch_c3<double, double, 1>(with_force, false, A, s, x, nullptr, b1, amode ? x : nullptr, nullptr, acc, lo,
                                         c->ca, c->cl, c->cm, G, c->f64);
        prof_mark(c, 1);
        const double* prev = x;
        double* cur = b1;
        for (int n = 1; n < nsteps; ++n) {
            double* nxt = (n == 1) ? b0 : const_cast<double*>(prev);
            A.w = sgn * c->w[n + 1];
            A.fc = c->cosn[n];
            if (march)
                launch_march3<0>(with_force, A, s, cur, prev, nxt, nullptr, acc, c->ca, c->cl, c->cm, G, c->f64);
            else
                launch_c3<double, double, 0>(with_force, false, A, s, cur, prev, nxt, nullptr, nullptr, acc, lo, c->ca,
                                             c->cl, c->cm, G, c->f64);
            prev = cur;
            cur = nxt;
        }
    } else {
        Metric3<float> G;
        for (int q = 0; q < 9; ++q) G.g[q] = c->fg[q];
        float *b0 = c->s32[0], *b1 = c->s32[1];
        prof_mark(c, 0);
        launch_c3<float, double, 1>(with_force, comp, A, s, x, nullptr, b1, amode ? x : nullptr, b0, acc, lo, c->fa,
                                    c->fl, c->fm, G, c->f32);
        prof_mark(c, 1);
        float* prev = b0;
        float* cur = b1;
        for (int n = 1; n < nsteps; ++n) {
            A.w = sgn * c->w[n + 1];
            A.fc = c->cosn[n];
            A.final_ = (n == nsteps - 1);
            launch_c3<float, float, 0>(with_force, comp, A, s, cur, prev, prev, nullptr, nullptr, acc, lo, c->fa,
                                       c->fl, c->fm, G, c->f32);
            float* t = prev;
            prev = cur;
            cur = t;
        }
    }
    prof_mark(c, 2, nsteps - 1);
}

}  // namespace elwh
