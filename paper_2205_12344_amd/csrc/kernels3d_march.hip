// 3-D FP64 El-WaveHoltz step on marching workgroups (Cartesian grids).
//
// The kernel of kernels3d.hip gathers each node's 19-point footprint: 17 loads per
// node and plane next to the accumulator's, three rows of U of which two are its
// neighbours' own, and 81 us per step at 128^3 (3.7 TB/s of the 144 B per update).
// Here each array is read once per node: a workgroup of NW wavefronts takes NW
// rows (y) of 64 nodes (x), of which (NW - 2) x 62 are its own, marches along z and
// shares what its rows need of each other through LDS (two buffers, one barrier
// per plane); x neighbours come by DPP, z neighbours stay in registers.
//
// Every flux is formed once per edge, with d_a the difference between both neighbours
// along a (spacings folded into the constants):
//   x edges: (A, mu, mu)_C+R e_x + P_C + P_R,   P = (lam (d_y v + d_z w), mu d_y u, mu d_z u)
//   y edges: (mu, A, mu)_C+N e_y + Q_C + Q_N,   Q = (mu d_x v, lam (d_x u + d_z w), mu d_z v)
//   z edges: (mu, mu, A)_C+U e_z + S_C + S_U,   S = (mu d_x w, mu d_y w, lam (d_x u + d_y v))
// and L_h U is the difference of the fluxes of its six edges, A = lam + 2 mu.  A
// step moves 320 MB at 128^3 (220 of them reads) in 66 us, 4.85 TB/s, the rate of a
// large copy; loads run one plane ahead, and more lookahead or wavefronts gain nothing.  On a
// traction-free z face the difference and the flux across it mirror those inside:
// the one-sided rows of step3d_common.h, divided by their weight 1/2.
#include <algorithm>

#include "elwh_internal.h"
#include "lanes.h"
#include "step3d_common.h"
#include "xcd.h"

namespace elwh {

namespace {

struct V3d {
    double x, y, z;
};
__device__ __forceinline__ V3d operator+(const V3d& a, const V3d& b) { return V3d{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3d operator-(const V3d& a, const V3d& b) { return V3d{a.x - b.x, a.y - b.y, a.z - b.z}; }
// (p, q, r) * a + b, componentwise
__device__ __forceinline__ V3d fma3(double p, double q, double r, const V3d& a, const V3d& b) {
    return V3d{fma(p, a.x, b.x), fma(q, a.y, b.y), fma(r, a.z, b.z)};
}
__device__ __forceinline__ V3d left3(const V3d& a) {
    return V3d{lane_from_left_z(a.x), lane_from_left_z(a.y), lane_from_left_z(a.z)};
}
__device__ __forceinline__ V3d right3(const V3d& a) {
    return V3d{lane_from_right_z(a.x), lane_from_right_z(a.y), lane_from_right_z(a.z)};
}

// START: the even-in-time start u^1 = u^0 + (a / 2)(L u^0 - f) and the seed of the sum.
constexpr int NW = 8;   // wavefronts (12, which 162 registers allow, gain 1 % at 128^3 and lose 4 % at 256^3)

template <bool START, bool FORCE>
__global__ __launch_bounds__(64 * NW) void march3d_kernel(const double* __restrict__ u, const double* uprev,
                                                         double* unext, const double* __restrict__ base,
                                                         double* __restrict__ acc, const double* __restrict__ ca,
                                                         const double* __restrict__ cl, const double* __restrict__ cm,
                                                         const double* __restrict__ f, Args3D A, int tz) {
    __shared__ double sh[2][NW][8][64];   // per plane and row: U, Q, lam, mu
    const int nbx = (A.nx - 1 + 61) / 62, nby = (A.ny - 1 + NW - 3) / (NW - 2), nbz = (A.khi - A.klo + tz) / tz;
    int t;
    if (!xcd_tile((int)blockIdx.x, nbx * nby * nbz, t)) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = (t % nbx) * 62 + lane;                     // own columns: lanes 1 .. 62
    const int j = ((t / nbx) % nby) * (NW - 2) + w;          // own rows: wavefronts 1 .. NW - 2
    const int k0 = A.klo + (t / (nbx * nby)) * tz, k1 = min(k0 + tz - 1, A.khi);
    const bool in = i <= A.nx && j <= A.ny;
    const bool unk = i >= 1 && i <= A.nx - 1 && j >= 1 && j <= A.ny - 1;   // unknown in its plane
    const bool own = unk && lane >= 1 && lane <= 62 && w >= 1 && w <= NW - 2;
    const int64_t CS = A.CS, PS = A.PS;
    // addresses: a uniform plane and component offset, and the lane's place in the plane
    const uint32_t lo = (uint32_t)(j * (int)A.P + i) * (uint32_t)sizeof(double);
    auto at = [&](const double* p, int64_t o) __attribute__((always_inline)) {
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(p + o) + lo);
    };
    auto at3 = [&](const double* p, int64_t o) __attribute__((always_inline)) {
        return V3d{at(p, o), at(p, o + CS), at(p, o + 2 * CS)};
    };
    auto put3 = [&](double* p, int64_t o, const V3d& v) __attribute__((always_inline)) {
        *reinterpret_cast<double*>(reinterpret_cast<char*>(p + o) + lo) = v.x;
        *reinterpret_cast<double*>(reinterpret_cast<char*>(p + o + CS) + lo) = v.y;
        *reinterpret_cast<double*>(reinterpret_cast<char*>(p + o + 2 * CS) + lo) = v.z;
    };

    auto ldu = [&](int k) __attribute__((always_inline)) {
        V3d v{0.0, 0.0, 0.0};
        if (unk && k >= A.klo && k <= A.khi) v = at3(u, k * PS);
        return v;
    };
    auto ldm = [&](const double* c, int k) __attribute__((always_inline)) {
        return in && k >= 0 && k <= A.nz ? at(c, k * PS) : 0.0;
    };
    struct Centre {
        double a;
        V3d old, h, f;
    };
    auto ld_centre = [&](int k) __attribute__((always_inline)) {
        Centre e{};
        if (own && k >= k0 && k <= k1) {
            const int64_t o = k * PS;
            e.a = at(ca, o);
            const double* hb = START ? base : acc;
            if (hb) e.h = at3(hb, o);
            if constexpr (!START) e.old = at3(uprev, o);
            if constexpr (FORCE) e.f = at3(f, o);
        }
        return e;
    };
    auto finish = [&](int k, const Centre& e, const V3d& c, V3d L) __attribute__((always_inline)) {
        if (own && k >= k0 && k <= k1) {
            if constexpr (FORCE) L = fma3(-A.fc, -A.fc, -A.fc, e.f, L);
            V3d n, h;
            if constexpr (START) {
                const double a = 0.5 * e.a;
                n = fma3(a, a, a, L, c);
                h = fma3(A.w, A.w, A.w, n, fma3(A.w0, A.w0, A.w0, c, e.h));
            } else {
                n = fma3(e.a, e.a, e.a, L, V3d{fma(2.0, c.x, -e.old.x), fma(2.0, c.y, -e.old.y), fma(2.0, c.z, -e.old.z)});
                h = fma3(A.w, A.w, A.w, n, e.h);
            }
            put3(unext, k * PS, n);
            put3(acc, k * PS, h);
        }
    };

    // planes k0 - 1 (its S only) .. k1 + 1
    const int ka = max(k0 - 1, 0), kb = min(k1 + 1, A.nz);
    const int wm = w > 0 ? w - 1 : w, wn = w < NW - 1 ? w + 1 : w;   // (halo rows need neither)
    V3d um = ldu(ka - 1), uc = ldu(ka), up = ldu(ka + 1);
    double lc = ldm(cl, ka), mc = ldm(cm, ka), lm = 0.0, mm = 0.0;
    V3d L{0.0, 0.0, 0.0}, S{0.0, 0.0, 0.0}, K{0.0, 0.0, 0.0};   // of plane kk - 1: all but its upper edge; S; its lower edge
    Centre e{};   // of plane kk - 1
    for (int kk = ka; kk <= kb; ++kk) {
        const Centre en = ld_centre(kk);
        const V3d upp = ldu(kk + 2);
        const double ln = ldm(cl, kk + 1), mn = ldm(cm, kk + 1);
        const bool flo = A.free_lo && kk == 0, fhi = A.free_hi && kk == A.nz;
        V3d eD = uc - um, dz = (up - uc) + eD;
        if (flo || fhi) {   // (the empty asm keeps rare, uniform branches from becoming selects)
            asm volatile("");
            if (flo) dz = up - uc;
            if (fhi) dz = eD;
            dz = dz + dz;
        }
        const V3d eR = right3(uc) - uc, dx = eR + left3(eR);
        const double lxy = A.cxy * lc, mxy = A.cxy * mc, lxz = A.cxz * lc, mxz = A.cxz * mc, lyz = A.cyz * lc,
                     myz = A.cyz * mc;
        const V3d Q{mxy * dx.y, fma(lxy, dx.x, lyz * dz.z), myz * dz.y};
        double(&s)[8][64] = sh[kk & 1][w];
        s[0][lane] = uc.x;
        s[1][lane] = uc.y;
        s[2][lane] = uc.z;
        s[3][lane] = Q.x;
        s[4][lane] = Q.y;
        s[5][lane] = Q.z;
        s[6][lane] = lc;
        s[7][lane] = mc;
        __syncthreads();
        const double(&sm)[8][64] = sh[kk & 1][wm];
        const double(&sn)[8][64] = sh[kk & 1][wn];
        const V3d eN = V3d{sn[0][lane], sn[1][lane], sn[2][lane]} - uc;
        const V3d eS = uc - V3d{sm[0][lane], sm[1][lane], sm[2][lane]};
        const V3d dy = eN + eS;
        const double AC = fma(2.0, mc, lc);
        V3d T;
        {   // y edges
            const double mN = sn[7][lane], mS = sm[7][lane];
            const double aN = A.cyy2 * (AC + fma(2.0, mN, sn[6][lane])), aS = A.cyy2 * (AC + fma(2.0, mS, sm[6][lane]));
            const double bN = A.cyy2 * (mc + mN), bS = A.cyy2 * (mc + mS);
            const V3d QN{sn[3][lane], sn[4][lane], sn[5][lane]}, QS{sm[3][lane], sm[4][lane], sm[5][lane]};
            T = fma3(bN, aN, bN, eN, QN - QS);
            T = fma3(-bS, -aS, -bS, eS, T);
        }
        {   // x edges
            const V3d P{fma(lxy, dy.y, lxz * dz.z), mxy * dy.x, mxz * dz.x};
            const double aR = A.cxx2 * (AC + lane_from_right_z(AC)), bR = A.cxx2 * (mc + lane_from_right_z(mc));
            const V3d G = fma3(aR, bR, bR, eR, P + right3(P));
            T = T + (G - left3(G));
        }
        // z edge below; plane kk - 1 is complete with it
        const V3d Sc{mxz * dx.z, myz * dy.z, fma(lxz, dx.x, lyz * dy.y)};
        const double aD = A.czz2 * (AC + fma(2.0, mm, lm)), bD = A.czz2 * (mc + mm);
        const V3d Kd = fma3(bD, bD, aD, eD, S + Sc);
        if (kk > ka) {
            V3d Lm = L + Kd;
            if (A.free_lo && kk - 1 == 0) {   // (the face's lower edge mirrors this one)
                asm volatile("");
                Lm = Lm + Kd;
            }
            finish(kk - 1, e, um, Lm);
        }
        L = T - Kd;
        if (flo) {
            asm volatile("");
            L = T;
        }
        K = Kd;
        S = Sc;
        um = uc;
        uc = up;
        up = upp;
        lm = lc;
        mm = mc;
        lc = ln;
        mc = mn;
        e = en;
    }
    // the last plane where nothing lies above it: the face's upper edge mirrors its lower one
    if (kb == k1) finish(k1, e, um, L - K);
}

int columns(int nx, int ny) { return ((nx - 1 + 61) / 62) * ((ny - 1 + NW - 3) / (NW - 2)); }

template <bool START>
void launch(bool force, const Args3D& A, hipStream_t s, const double* u, const double* uprev, double* unext,
               const double* base, double* acc, const double* ca, const double* cl, const double* cm,
               const double* f) {
    const int nb = columns(A.nx, A.ny), np = A.khi - A.klo + 1;
    // Chunks along z: the fewest rounds of workgroups (one per CU: 162 registers leave
    // two wavefronts per SIMD) times planes (a chunk works on two more than it owns).
    int tz = np;
    int64_t best = (int64_t)1 << 60;
    for (int z = 1; z <= np; ++z) {
        const int64_t cost = ((int64_t)nb * ((np + z - 1) / z) + 255) / 256 * (z + 2);
        if (cost <= best) {
            best = cost;
            tz = z;
        }
    }
    const dim3 grid((unsigned)xcd_grid(nb * ((np + tz - 1) / tz)));
    if (force)
        hipLaunchKernelGGL((march3d_kernel<START, true>), grid, dim3(64 * NW), 0, s, u, uprev, unext, base, acc, ca,
                           cl, cm, f, A, tz);
    else
        hipLaunchKernelGGL((march3d_kernel<START, false>), grid, dim3(64 * NW), 0, s, u, uprev, unext, base, acc,
                           ca, cl, cm, f, A, tz);
}

}  // namespace

// The march is the faster one on grids that are thick every way (us per step,
// against the tiling that autotuning picks): 16^3 6.4 (11.5), 32^3 6.3 (11.3), 64^3
// 14.1 (16.7), 128^3 66 (81), 200 x 150 x 100 95 (132), 256^3 545 (608).  It launches
// every step and works on two planes and two rows more than it owns, so the
// two-step launches keep the thin grids that caches hold (us for 20 steps, march
// against tilings):
//   few planes: 64 x 64 x 1 118 / 74, x 3 126 / 119, x 4 130 / 141; 200 x 200 x 3 189 /
//   164; 600 x 600 x 2 579 / 546, x 4 879 / 997; 800 x 800 x 1 701 / 649, x 2 957 / 1063
//   (planes unknown);
//   few rows: one row 400 x 400 349 / 284, 400 x 200 222 / 243; two rows 400 x 400 361 /
//   335, 400 x 300 299 / 326, 62 x 2500 327 / 503;
//   one round of workgroups that cannot be split further (129 to 256 columns):
//   200 x 200 x 5 251 / 234, x 9 363 / 368; 240 x 380 x 8 425 / 396; 490 x 180 x 8 418 /
//   469.
// With fuse = 1 the tilings step singly too and keep one plane (64 x 64 118 / 90) and
// one row (400 x 400 349 / 322; two rows 361 / 369, two planes of 200 x 200 159 / 160).
StepRule march3d_rule(int nx, int ny, int np, bool pairs) {
    const int64_t nodes = (int64_t)(nx - 1) * (ny - 1) * np;
    if (nodes > 1500000 && ny > 3) return STEP_OWN;
    if (np <= (pairs ? 3 : 1))
        return nodes <= 500000 ? STEP_TILING : (nodes <= 1000000 ? STEP_TILING_UNTIMED : STEP_OWN_UNTIMED);
    if (ny <= (pairs ? 3 : 2)) {
        if (nodes <= 60000) return STEP_OWN;
        return nx > 200 && nodes > (ny == 2 ? 100000 : 300000) ? STEP_TILING_UNTIMED : STEP_OWN_UNTIMED;
    }
    const int nb = columns(nx, ny);
    if (!pairs || np > 16 || nb <= 64) return STEP_OWN;
    return np <= 8 && nb > 128 && nb <= 256 ? STEP_TILING_UNTIMED : STEP_OWN_UNTIMED;
}

StepRule march3d_rule(const elwh_ctx* c) {
    // (places in a plane are 32-bit byte offsets)
    if (c->L.P * (c->L.ny + 1) >= ((int64_t)1 << 29)) return STEP_TILING;
    return march3d_rule(c->L.nx, c->L.ny, c->mr.hi - c->mr.lo + 1, c->opts.fuse >= 2);
}

void launch_march3d(bool start, bool force, const Args3D& A, hipStream_t s, const double* u, const double* uprev,
                    double* unext, const double* base, double* acc, const double* ca, const double* cl,
                    const double* cm, const double* f) {
    if (start)
        launch<true>(force, A, s, u, uprev, unext, base, acc, ca, cl, cm, f);
    else
        launch<false>(force, A, s, u, uprev, unext, base, acc, ca, cl, cm, f);
}

}  // namespace elwh
