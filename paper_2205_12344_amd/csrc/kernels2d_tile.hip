// 2-D El-WaveHoltz steps on tiles that stay in registers, for grids too small
// to fill the chip with marching wavefronts (FP64).
//
// The marching kernels (kernels2d_multi.hip) walk a strip row by row, one row's
// latency after the other; with K = 4 steps per launch a wavefront spends about
// 1.5 us per row, so a grid of 64 or 256 rows takes 16 us for four steps however
// few wavefronts it needs.  Here a workgroup owns a tile of NW R rows x 64
// columns, wavefront w its rows w R .. w R + R - 1, one column per lane: state,
// accumulator and the stencil coefficients of every node stay in registers for
// all the steps of a launch, and after each step the wavefronts exchange their
// first and last rows through LDS (two buffers, one barrier per step); x
// neighbours come by DPP.  A launch of up to H steps computes the tile's inner
// (64 - 2 H) x (NW R - 2 H) nodes exactly (the outer ones are recomputed by the
// neighbouring tiles) and needs u^n and u^{n-1} on the whole tile, so more steps
// per launch cost redundant arithmetic and save launches and loads.
//
// The coefficients are formed once per launch with a = c dt^2 / rho, the
// metric factors and the boundary closure folded in: 16 per node, and a
// step of one node is 16 differences and 16 fused multiply-adds.  A node that
// is no unknown has zero coefficients and keeps its zero.  A traction-free
// face is the interior stencil with a ghost row (or column) equal to the face's
// own, the face normal's compact and mixed terms doubled and the coefficient of
// the one-sided difference's own node negated; the ghost is the value itself.
//
// Two fields (absorbing faces): any face may be an unknown one, so the ghost
// also exists per column (a select on the lanes of the face, in tiles that
// touch it); face nodes are damped, u^{n+1} <- (u^{n+1} + g u^{n-1}) / (1 + g)
// with g and the reciprocal in LDS, and the centred velocity of every level is
// added to a second accumulator.
//
// The launch that starts an application takes the even-in-time start u^1 = u^0
// + (a/2)(Ltilde u^0 - f) (with a second field, + dt (1 - g) u1) as its first step.
#include <algorithm>

#include "step2d_common.h"

namespace elwh {

namespace {

// Differences and products of one component's row: the eight stencil terms.
struct Coef {
    double xL, xR, yS, yN;   // compact terms (own component): edges to the left, right, below, above
    double cL, cR;           // mixed terms: vertical differences of the other component, left and right column
    double cS, cN;           // mixed terms: horizontal differences of the other component, row below and above
};

__device__ __forceinline__ double stencil_row(const Coef& q, double C, double L, double R, double S, double N,
                                              double oSL, double oSR, double oNL, double oNR) {
    double s = q.xR * (R - C);
    s = fma(-q.xL, C - L, s);
    s = fma(q.yN, N - C, s);
    s = fma(-q.yS, C - S, s);
    s = fma(q.cR, oNR - oSR, s);
    s = fma(-q.cL, oNL - oSL, s);
    s = fma(q.cN, oNR - oNL, s);
    return fma(-q.cS, oSR - oSL, s);
}

// Weights of a launch's steps: w(s) of the level step s computes, f(s) the
// forcing factor of the level it starts from.
struct ArgWeights {
    const Tile2D& A;
    __device__ double w(int s) const { return A.wk[s]; }
    __device__ double f(int s) const { return A.fck[s]; }
};
struct TableWeights {
    const double *wt, *ct;
    double sgn;
    __device__ double w(int s) const { return sgn * wt[s]; }
    __device__ double f(int s) const { return ct[s]; }
};

// Tile (tx, ty) of one problem.
template <int NW, int R, bool FORCE, bool TWO, class Weights>
__device__ __forceinline__ void tile2d_body(int tx, int ty, const double* __restrict__ u,
                                            const double* __restrict__ uprev, double* __restrict__ outA,
                                            double* __restrict__ outB, const double* __restrict__ base,
                                            double* __restrict__ acc, const double* __restrict__ ca,
                                            const double* __restrict__ cl, const double* __restrict__ cm,
                                            const double* __restrict__ f, const Tile2D& A, const TwoField2D& D,
                                            const Weights& W) {
    __shared__ double ex[2][NW][2][2][64];   // [buffer][wavefront][first, last row][u, v][column]
    // a f per node (each lane its own values), in registers where three rows leave
    // room: 64^2 filter with forcing 1.30 us per step, from LDS 1.39
    constexpr bool FREG = FORCE && R <= 3;
    __shared__ double af[FORCE && !FREG ? NW * R : 1][2][64];
    double fu[FREG ? R : 1], fv[FREG ? R : 1];
    // damping of the tile's face nodes: g, 1 / (1 + g) of u, then of v
    __shared__ double dg[TWO ? NW * R : 1][4][64];
    __shared__ double zs[TWO ? NW * R : 1][2][64];   // the second field (first launch)
    const int ilo = TWO && D.xfree_lo ? 0 : 1, ihi = TWO && D.xfree_hi ? A.nx : A.nx - 1;   // unknown columns
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: scalar row indices)
    const int col = ilo + tx * (64 - 2 * A.H) - A.H + lane;
    const int row0 = A.jlo + ty * (NW * R - 2 * A.H) - A.H + w * R;   // first row of this wavefront
    const bool colv = col >= 0 && col <= A.nx, colu = col >= ilo && col <= ihi;
    const int64_t P = A.P, CS = A.CS;

    // rows 0 and R + 1 of these arrays are the neighbours' (row r = grid row row0 + r - 1)
    double u0[R + 2], v0[R + 2], u1[R + 2], v1[R + 2], au[R], av[R], bu[R], bv[R];
    const bool xlo = TWO && D.xfree_lo && col == 0, xhi = TWO && D.xfree_hi && col == A.nx;
    bool damped = false;   // (uniform) this wavefront has nodes of an impedance face
    Coef qu[R], qv[R];
    {
        double l[R + 2], m[R + 2], a[R];
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            const int j = row0 + r - 1;
            const bool in = colv && j >= 0 && j <= A.ny;
            const int64_t o = (int64_t)j * P + col;
            l[r] = in ? cl[o] : 0.0;
            m[r] = in ? cm[o] : 0.0;
            u0[r] = in ? u[o] : 0.0;
            v0[r] = in ? u[o + CS] : 0.0;
            if (r >= 1 && r <= R) {
                const bool unk = colu && j >= A.jlo && j <= A.jhi;
                a[r - 1] = unk ? ca[o] : 0.0;
                const bool older = unk && uprev && !(TWO && A.first);
                u1[r] = older ? uprev[o] : 0.0;
                v1[r] = older ? uprev[o + CS] : 0.0;
                const int q = w * R + r - 1;
                const bool own = unk && lane >= A.H && lane < 64 - A.H && q >= A.H && q < NW * R - A.H;
                const double* b = A.first ? base : acc;
                au[r - 1] = own && b ? b[o] : 0.0;
                av[r - 1] = own && b ? b[o + CS] : 0.0;
                if constexpr (TWO) {
                    const double* b1 = A.first ? D.base1 : D.acc1;
                    bu[r - 1] = own && b1 ? b1[o] : 0.0;
                    bv[r - 1] = own && b1 ? b1[o + CS] : 0.0;
                    double gu = 0.0, gv = 0.0;
                    if (unk && ((D.imp_lo && j == 0) || (D.imp_hi && j == A.ny))) {
                        const double* g = D.dmp + (j == 0 ? 0 : 2) * P + col;
                        gu += g[0];
                        gv += g[P];
                    }
                    if (unk && (xlo || xhi)) {
                        const double* g = D.dmpx + (xlo ? 0 : 2) * (A.ny + 1) + j;
                        gu += g[0];
                        gv += g[A.ny + 1];
                    }
                    if (A.first) {
                        zs[q][0][lane] = unk ? uprev[o] : 0.0;
                        zs[q][1][lane] = unk ? uprev[o + CS] : 0.0;
                    }
                    dg[q][0][lane] = gu;
                    dg[q][1][lane] = 1.0 / (1.0 + gu);
                    dg[q][2][lane] = gv;
                    dg[q][3][lane] = 1.0 / (1.0 + gv);
                    damped |= __any(gu != 0.0 || gv != 0.0);
                }
                if constexpr (FORCE) {
                    const double pu = unk ? ca[o] * f[o] : 0.0, pv = unk ? ca[o] * f[o + CS] : 0.0;
                    if constexpr (FREG) {
                        fu[r - 1] = pu;
                        fv[r - 1] = pv;
                    } else {
                        af[q][0][lane] = pu;
                        af[q][1][lane] = pv;
                    }
                }
            }
        }
        u1[0] = u1[R + 1] = v1[0] = v1[R + 1] = 0.0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int j = row0 + k, r = k + 1;
            const bool top = A.free_hi && j == A.ny, bot = A.free_lo && j == 0;
            const double lL = lane_from_left_z(l[r]), lR = lane_from_right_z(l[r]);
            const double mL = lane_from_left_z(m[r]), mR = lane_from_right_z(m[r]);
            const double AL = lL + 2.0 * mL, AC = l[r] + 2.0 * m[r], AR = lR + 2.0 * mR;
            const double AS = l[r - 1] + 2.0 * m[r - 1], AN = l[r + 1] + 2.0 * m[r + 1];
            const double fy = top || bot ? 2.0 : 1.0, fx = xlo || xhi ? 2.0 : 1.0;
            const double ax = fx * a[k] * A.cxx2, ay = fy * a[k] * A.cyy2, c = fx * fy * a[k] * A.cxy;
            const double yN = top ? 0.0 : ay, yS = bot ? 0.0 : ay, xR = xhi ? 0.0 : ax, xL = xlo ? 0.0 : ax;
            qu[k].xL = xL * (AC + AL);
            qu[k].xR = xR * (AR + AC);
            qu[k].yS = yS * (m[r] + m[r - 1]);
            qu[k].yN = yN * (m[r + 1] + m[r]);
            qu[k].cL = c * (xlo ? -l[r] : lL);
            qu[k].cR = c * (xhi ? -l[r] : lR);
            qu[k].cS = c * (bot ? -m[r] : m[r - 1]);
            qu[k].cN = c * (top ? -m[r] : m[r + 1]);
            qv[k].xL = xL * (m[r] + mL);
            qv[k].xR = xR * (mR + m[r]);
            qv[k].yS = yS * (AC + AS);
            qv[k].yN = yN * (AN + AC);
            qv[k].cL = c * (xlo ? -m[r] : mL);
            qv[k].cR = c * (xhi ? -m[r] : mR);
            qv[k].cS = c * (bot ? -l[r] : l[r - 1]);
            qv[k].cN = c * (top ? -l[r] : l[r + 1]);
        }
    }
    // the array rows (1 .. R) of the free faces in this wavefront, 0 if none
    const int rtop = A.free_hi && A.ny >= row0 && A.ny < row0 + R ? A.ny - row0 + 1 : 0;
    const int rbot = A.free_lo && 0 >= row0 && 0 < row0 + R ? 1 - row0 : 0;
    auto ghosts = [&](double(&U)[R + 2], double(&V)[R + 2]) __attribute__((always_inline)) {
        if (rtop | rbot) {
#pragma unroll
            for (int r = 1; r <= R; ++r) {
                // (the empty asm keeps these rare, uniform branches from becoming selects)
                if (rtop == r) {
                    asm volatile("");
                    U[r + 1] = U[r];
                    V[r + 1] = V[r];
                }
                if (rbot == r) {
                    asm volatile("");
                    U[r - 1] = U[r];
                    V[r - 1] = V[r];
                }
            }
        }
    };
    ghosts(u0, v0);
    const bool xface = TWO && __any(xlo || xhi);
    auto left = [&](double x) __attribute__((always_inline)) {
        double l = lane_from_left_z(x);
        if (TWO && xface) {
            asm volatile("");
            l = xlo ? x : l;
        }
        return l;
    };
    auto right = [&](double x) __attribute__((always_inline)) {
        double r = lane_from_right_z(x);
        if (TWO && xface) {
            asm volatile("");
            r = xhi ? x : r;
        }
        return r;
    };

    if (A.first) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            au[k] = fma(A.w0, u0[k + 1], au[k]);
            av[k] = fma(A.w0, v0[k + 1], av[k]);
        }
    }

    // one step: X, Y the current level with its neighbour rows, U, V the level
    // before, overwritten by the next one (before the start: 0)
    auto step = [&](const double(&X)[R + 2], const double(&Y)[R + 2], double(&U)[R + 2], double(&V)[R + 2], int s,
                    bool more) __attribute__((always_inline)) {
        const bool start = s == 0 && A.first;
        const double wk = W.w(s), fc = FORCE ? W.f(s) : 0.0;
        double xSL = left(X[0]), xSR = right(X[0]), ySL = left(Y[0]), ySR = right(Y[0]);
        double xL = left(X[1]), xR = right(X[1]), yL = left(Y[1]), yR = right(Y[1]);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int r = k + 1;
            const double xNL = left(X[r + 1]), xNR = right(X[r + 1]), yNL = left(Y[r + 1]), yNR = right(Y[r + 1]);
            double su = stencil_row(qu[k], X[r], xL, xR, X[r - 1], X[r + 1], ySL, ySR, yNL, yNR);
            double sv = stencil_row(qv[k], Y[r], yL, yR, Y[r - 1], Y[r + 1], xSL, xSR, xNL, xNR);
            if constexpr (FORCE) {
                su = fma(-fc, FREG ? fu[FREG ? k : 0] : af[FREG ? 0 : w * R + k][0][lane], su);
                sv = fma(-fc, FREG ? fv[FREG ? k : 0] : af[FREG ? 0 : w * R + k][1][lane], sv);
            }
            double nu = fma(2.0, X[r], -U[r]) + su, nv = fma(2.0, Y[r], -V[r]) + sv;
            if (start) {   // half of it, plus the second field
                asm volatile("");
                nu *= 0.5;
                nv *= 0.5;
                if constexpr (TWO) {
                    const double(&g)[4][64] = dg[w * R + k];
                    const double zu = zs[w * R + k][0][lane], zv = zs[w * R + k][1][lane];
                    nu = fma(D.dtw * (1.0 - g[0][lane]), zu, nu);
                    nv = fma(D.dtw * (1.0 - g[2][lane]), zv, nv);
                    bu[k] = fma(D.w0v, zu, bu[k]);
                    bv[k] = fma(D.w0v, zv, bv[k]);
                }
            } else if constexpr (TWO) {
                if (damped) {
                    asm volatile("");
                    const double(&g)[4][64] = dg[w * R + k];
                    nu = fma(g[0][lane], U[r], nu) * g[1][lane];
                    nv = fma(g[2][lane], V[r], nv) * g[3][lane];
                }
                bu[k] = fma(D.wvk[s], nu - U[r], bu[k]);
                bv[k] = fma(D.wvk[s], nv - V[r], bv[k]);
            }
            U[r] = nu;
            V[r] = nv;
            au[k] = fma(wk, nu, au[k]);
            av[k] = fma(wk, nv, av[k]);
            xSL = xL; xSR = xR; ySL = yL; ySR = yR;
            xL = xNL; xR = xNR; yL = yNL; yR = yNR;
        }
        if (more) {
            double(&e)[NW][2][2][64] = ex[s & 1];
            e[w][0][0][lane] = U[1];
            e[w][0][1][lane] = V[1];
            e[w][1][0][lane] = U[R];
            e[w][1][1][lane] = V[R];
            __syncthreads();
            const int wb = w > 0 ? w - 1 : w, wa = w < NW - 1 ? w + 1 : w;   // (the tile's outermost rows are not exact)
            U[0] = e[wb][1][0][lane];
            V[0] = e[wb][1][1][lane];
            U[R + 1] = e[wa][0][0][lane];
            V[R + 1] = e[wa][0][1][lane];
            ghosts(U, V);
        }
    };
    int s = 0;
    for (; s + 2 <= A.steps; s += 2) {
        step(u0, v0, u1, v1, s, true);
        step(u1, v1, u0, v0, s + 1, true);
    }
    // X, Y the level before the last, U, V the last
    auto store = [&](const double(&X)[R + 2], const double(&Y)[R + 2], const double(&U)[R + 2],
                     const double(&V)[R + 2]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int j = row0 + k, q = w * R + k;
            if (colu && j >= A.jlo && j <= A.jhi && lane >= A.H && lane < 64 - A.H && q >= A.H && q < NW * R - A.H) {
                const int64_t o = (int64_t)j * P + col;
                if (A.steps > 1) {
                    outA[o] = X[k + 1];
                    outA[o + CS] = Y[k + 1];
                }
                outB[o] = U[k + 1];
                outB[o + CS] = V[k + 1];
                acc[o] = au[k];
                acc[o + CS] = av[k];
                if constexpr (TWO) {
                    D.acc1[o] = bu[k];
                    D.acc1[o + CS] = bv[k];
                }
            }
        }
    };
    if (s < A.steps) {   // one step more: the roles are exchanged
        step(u0, v0, u1, v1, s, false);
        store(u0, v0, u1, v1);
    } else {
        store(u1, v1, u0, v0);
    }
}

__host__ __device__ __forceinline__ int tiles_x(int cols, int H) { return (cols + 63 - 2 * H) / (64 - 2 * H); }
__host__ __device__ __forceinline__ int tiles_y(int nrows, int rows, int H) {
    return (nrows + rows - 2 * H - 1) / (rows - 2 * H);
}

template <int NW, int R, bool FORCE, bool TWO>
__global__ __launch_bounds__(64 * NW) void tile2d_kernel(const double* __restrict__ u, const double* __restrict__ uprev,
                                                         double* __restrict__ outA, double* __restrict__ outB,
                                                         const double* __restrict__ base, double* __restrict__ acc,
                                                         const double* __restrict__ ca, const double* __restrict__ cl,
                                                         const double* __restrict__ cm, const double* __restrict__ f,
                                                         Tile2D A, TwoField2D D) {
    const int ntx = tiles_x(A.nx - 1 + (TWO ? D.xfree_lo + D.xfree_hi : 0), A.H);
    int t;
    if (!xcd_tile((int)blockIdx.x, ntx * tiles_y(A.jhi - A.jlo + 1, NW * R, A.H), t)) return;
    tile2d_body<NW, R, FORCE, TWO>(t % ntx, t / ntx, u, uprev, outA, outB, base, acc, ca, cl, cm, f, A, D,
                                   ArgWeights{A});
}

template <int NW, int R, bool TWO>
void tile_launch(bool force, hipStream_t s, const double* u, const double* uprev, double* outA, double* outB,
                 const double* base, double* acc, const double* ca, const double* cl, const double* cm, const double* f,
                 const Tile2D& A, const TwoField2D& D) {
    const int cols = A.nx - 1 + (TWO ? D.xfree_lo + D.xfree_hi : 0);
    const dim3 grid((unsigned)xcd_grid(tiles_x(cols, A.H) * tiles_y(A.jhi - A.jlo + 1, NW * R, A.H)));
    if (force)
        hipLaunchKernelGGL((tile2d_kernel<NW, R, true, TWO>), grid, dim3(64 * NW), 0, s, u, uprev, outA, outB, base,
                           acc, ca, cl, cm, f, A, D);
    else
        hipLaunchKernelGGL((tile2d_kernel<NW, R, false, TWO>), grid, dim3(64 * NW), 0, s, u, uprev, outA, outB, base,
                           acc, ca, cl, cm, f, A, D);
}

}  // namespace

// The shape and steps per launch with the least modelled time of an application
// of N steps.  Workgroups run in rounds, one per CU (their registers fill it):
// a launch takes 1.5 us and each round the time of H steps (0.11 + 0.018 rows
// us each: arithmetic of the tile's rows on four SIMDs, then the exchange) plus
// 3 us of load latency and coefficients, 0.04 us per tile row for the loads
// and 2.4 ns per inner node for its stores (two fields: 5 us and 6 ns).  Fitted
// to, and within 15 % of, launches of 64^2 to 1500^2 nodes.  Measured, against
// the marching kernels: 64^2 8 x 3 rows x 11 steps 1.14 us per step (3.91), 256^2
// 8 x 4 x 12 1.46 (4.16), 611 x 373 8 x 4 x 6 2.20 (5.50), 1024^2 8 x 4 x 7 8.60
// (10.75); two fields: 256^2 8 x 3 x 7 2.55 (7.01), 1024^2 8 x 3 x 6 14.8 (26.4),
// where the 8 x 4 tile spills registers (20.8; with the velocity sum in LDS
// instead 14.3 at 1024^2 and slower below).
TileShape tile2d_pick(int nx, int nrows, int N, bool two) {
    static const int shapes[3][2] = {{4, 4}, {8, 3}, {8, 4}};
    const double fixed = two ? 5.0 : 3.0, store = two ? 6e-3 : 2.4e-3;
    TileShape best;
    double tbest = 1e300;
    for (int k = 0; k < (two ? 2 : 3); ++k) {
        const int rows = shapes[k][0] * shapes[k][1];
        for (int H = 3; H <= std::min(kTileMaxSteps, rows / 2 - 1); ++H) {
            const long long tiles = (long long)tiles_x(nx - 1, H) * tiles_y(nrows, rows, H);
            const double rounds = (double)((tiles + 255) / 256), inner = (64 - 2 * H) * (rows - 2 * H);
            const double t = (N + H - 1) / H * (1.5 + rounds * (fixed + 0.04 * rows + store * inner)) +
                             rounds * N * (0.11 + 0.018 * rows);
            if (t < tbest) {
                tbest = t;
                best.NW = shapes[k][0];
                best.R = shapes[k][1];
                best.H = H;
            }
        }
    }
    return best;
}

// Few rows and tens of thousands of columns: a tile computes its 16 to 32 rows
// however few are unknown, and there are several rounds of them, while the
// marching wavefronts stop at the last row.  Tiles against the marching kernels,
// us for 60 steps: 25000 x 2 96 / 154, 28000 x 2 179 / 155, 40000 x 4 246 / 218,
// 100000 x 3 319 / 252; 50000 x 8 294 / 331, 80000 x 8 478 / 432; 80000 x 16 642 /
// 706, 120000 x 12 836 / 706; 40000 x 32 679 / 738, 50000 x 48 1310 / 1227,
// 50000 x 64 1663 / 1655.  Two fields 28000 x 3 276 / 283, 40000 x 3 361 / 297, 100000 x
// 5 847 / 640, 100000 x 8 930 / 1389; mapped 28000 x 3 304 / 324, 40000 x 3 400 / 339,
// 100000 x 5 936 / 825, 100000 x 8 988 / 1197.
StepRule strip2d_rule(int nx, int nrows, bool coupled) {
    if (nx <= 25000 || nrows >= (coupled ? 6 : 64)) return STEP_OWN;
    const int widest = coupled ? (nrows <= 3 ? 27000 : (nrows == 4 ? 36000 : 70000))
                               : (nrows <= 4 ? 27000 : (nrows <= 8 ? 60000 : (nrows <= 23 ? 90000 : 45000)));
    return nx > widest ? STEP_TILING_UNTIMED : STEP_OWN_UNTIMED;
}

StepRule tile2d_rule(const elwh_ctx* c, bool two) {
    if (c->opts.fuse < 4) return STEP_TILING;   // (fewer steps per launch asked for)
    const int rows = c->mr.hi - c->mr.lo + 1;
    // One field: beyond about 2000^2 nodes the marching kernels are level (2048^2:
    // 2261 against 2364 us, 4096^2: 8.40 against 8.39 ms) and need no tile
    // redundancy.  Two fields: they take one step per launch, twice as slow up to
    // the largest grid tried (4096^2: 29.4 against 13.7 ms for 61 steps).
    if (!two && (int64_t)c->L.nx * rows > (int64_t)2100 * 2100) return STEP_TILING;
    return strip2d_rule(c->L.nx, rows, two);
}

TileShape tile2d_shape(const elwh_ctx* c, bool two) {
    if (!own_steps(c, tile2d_rule(c, two), two == has_impedance(c))) return TileShape();
    return tile2d_pick(c->L.nx, c->mr.hi - c->mr.lo + 1, c->plan.nt * c->opts.periods + (two ? 1 : 0), two);
}

Tile2D tile2d_args(const elwh_ctx* c, const TileShape& t) {
    Tile2D A{};
    A.nx = c->L.nx;
    A.ny = c->L.ny;
    A.P = c->L.P;
    A.CS = c->L.CS;
    A.jlo = c->mr.lo;
    A.jhi = c->mr.hi;
    A.free_lo = c->mr.free_lo;
    A.free_hi = c->mr.free_hi;
    A.cxx2 = c->st.cxx2;
    A.cyy2 = c->st.cyy2;
    A.cxy = c->st.cxy;
    A.H = t.H;
    return A;
}

void other_two(const elwh_ctx* c, const double* a, const double* b, double** o) {
    int k = 0;
    for (double* p : c->s64)
        if (k < 2 && p != a && p != b) o[k++] = p;
}

void run_filter_tile2d(elwh_ctx* c, const TileShape& t, const double* x, bool with_force, bool amode, double* out) {
    const int nsteps = c->plan.nt * c->opts.periods;
    const double sgn = amode ? -1.0 : 1.0;
    Tile2D A = tile2d_args(c, t);
    A.w0 = sgn * c->w[0];
    const double *cur = x, *prev = nullptr;
    prof_mark(c, 0);
    prof_mark(c, 1);
    for (int n = 0; n < nsteps; n += A.steps) {
        A.first = n == 0;
        A.steps = std::min(t.H, nsteps - n);
        for (int s = 0; s < A.steps; ++s) {
            A.wk[s] = sgn * c->w[n + s + 1];
            A.fck[s] = c->cosn[n + s];
        }
        double* o[2] = {nullptr, nullptr};
        other_two(c, cur, prev, o);
        const auto launch = t.NW == 4 ? tile_launch<4, 4, false>
                                      : (t.R == 3 ? tile_launch<8, 3, false> : tile_launch<8, 4, false>);
        launch(with_force, c->stream, cur, prev, o[0], o[1], amode ? x : nullptr, out, c->ca, c->cl, c->cm, c->f64, A,
               TwoField2D{});
        prev = A.steps > 1 ? o[0] : cur;
        cur = o[1];
    }
    prof_mark(c, 2, nsteps);
}

void run_filter_twofield_tile2d(elwh_ctx* c, const TileShape& t, const double* x0, const double* z1, bool with_force,
                                bool amode, double s_in, double s_out, double* out0, double* out1) {
    const int N = c->plan.nt * c->opts.periods;   // and one step more, for the velocity of the last level
    const double sgn = amode ? -1.0 : 1.0, dt = c->plan.dt;
    Tile2D A = tile2d_args(c, t);
    A.w0 = sgn * c->w[0];
    TwoField2D D{};
    D.base1 = amode ? z1 : nullptr;
    D.acc1 = out1;
    D.dmp = c->dmp;
    D.dmpx = c->dmpx;
    D.imp_lo = c->imp[0];
    D.imp_hi = c->imp[1];
    D.xfree_lo = c->ximp[0];
    D.xfree_hi = c->ximp[1];
    D.w0v = sgn * c->w[0] * s_in * s_out;
    D.dtw = dt * s_in;
    const double *cur = x0, *prev = z1;
    prof_mark(c, 0);
    prof_mark(c, 1);
    for (int n = 0; n <= N; n += A.steps) {
        A.first = n == 0;
        A.steps = std::min(t.H, N + 1 - n);
        for (int s = 0; s < A.steps; ++s) {
            A.wk[s] = n + s < N ? sgn * c->w[n + s + 1] : 0.0;
            A.fck[s] = c->cosn[n + s];
            D.wvk[s] = sgn * c->w[n + s] * s_out / (2.0 * dt);
        }
        double* o[2] = {nullptr, nullptr};
        other_two(c, cur, prev, o);
        const auto launch = t.NW == 4 ? tile_launch<4, 4, true> : tile_launch<8, 3, true>;
        launch(with_force, c->stream, cur, prev, o[0], o[1], amode ? x0 : nullptr, out0, c->ca, c->cl, c->cm, c->f64, A,
               D);
        prev = A.steps > 1 ? o[0] : cur;
        cur = o[1];
    }
    prof_mark(c, 2, N + 1);
}

// ===========================================================================
// Ragged batch: one register-tile tick advances every active problem by up to H
// steps of its own application (the start included), in one launch over the
// concatenated tiles.
// ===========================================================================
namespace {

constexpr int BNW = 8, BR = 4;

template <bool FORCE>
__global__ __launch_bounds__(64 * BNW) void batch_tile2d_kernel(const BProb2D* __restrict__ pr,
                                                               const BState* __restrict__ st, int np, int H, double sgn,
                                                               int amode) {
    const int p = batch_problem_of(pr, np, (int)blockIdx.x, true);
    const BProb2D& q = pr[p];
    if (!st[p].active) return;
    // Workgroup b runs on XCD b mod 8.  The workgroups of a problem that share an
    // XCD take one contiguous eighth of its tiles, so the XCDs stay even when some
    // problems have finished: dealt in one band over all problems, the tiles of
    // the problems left fell to one or two XCDs (batch of 16 problems of 256^2 to
    // 1024^2: 237 ms for three iterations).  Every workgroup has a tile: a whole
    // number of eights per problem left 1000 problems of 30^2 nodes with seven empty
    // workgroups of eight (four iterations 28.1 ms, now 23.4; three of 48 problems of
    // 256^2 38.5, now 36.2).
    const int slot = (int)blockIdx.x - q.off2, share = q.nblk2 / kXcds, more = q.nblk2 % kXcds, e = slot % kXcds;
    const int local = e * share + min(e, more) + slot / kXcds, n = st[p].end ? 0 : st[p].n;
    if (slot >= q.nblk2) return;
    Tile2D A;
    A.nx = q.A.nx;
    A.ny = q.A.ny;
    A.P = q.A.P;
    A.CS = q.A.CS;
    A.jlo = q.A.jlo;
    A.jhi = q.A.jhi;
    A.free_lo = q.A.free_lo;
    A.free_hi = q.A.free_hi;
    A.cxx2 = q.A.cxx2;
    A.cyy2 = q.A.cyy2;
    A.cxy = q.A.cxy;
    A.H = H;
    A.first = n == 0;
    A.steps = min(H, q.nsteps - n);
    A.w0 = sgn * q.w[0];
    const int ic = n == 0 ? -1 : st[p].ic, ip = n == 0 ? -1 : st[p].ip;
    int x1, x2;
    batch_free_two(ic, ip, x1, x2);
    const double* cur = ic >= 0 ? static_cast<const double*>(q.s[ic]) : q.src;
    const double* prev = n == 0 ? nullptr : (ip >= 0 ? static_cast<const double*>(q.s[ip]) : q.src);
    const TableWeights W{q.w + n + 1, q.cosn + n, sgn};
    tile2d_body<BNW, BR, FORCE, false>(local % q.nbx2, local / q.nbx2, cur, prev, static_cast<double*>(q.s[x1]),
                                       static_cast<double*>(q.s[x2]), amode ? q.src : nullptr, q.out,
                                       static_cast<const double*>(q.ca), static_cast<const double*>(q.cl),
                                       static_cast<const double*>(q.cm), static_cast<const double*>(q.f), A,
                                       TwoField2D{}, W);
}

}  // namespace

int batch_reg_tiles(int nx, int nrows, int H, int* ntx) {
    *ntx = tiles_x(nx - 1, H);
    return *ntx * tiles_y(nrows, BNW * BR, H);
}

// Whether wide problems of a few rows carry the batch: as for one problem
// (strip2d_rule), a tile's other rows are empty and the marching ticks are faster.
// ms for four iterations of 30 steps, tiles against marching ticks: 4 problems of
// 10000 x 3 0.37 / 0.33, 4 of 100000 x 3 (15 steps) 1.72 / 0.85, 48 of 1000 x 3 2.47 / 2.25,
// 4 of 20000 x 8 0.57 / 0.54, 4 of 40000 x 8 0.90 / 0.74; 16 of 2000 x 3 0.47 / 0.48, 400 of
// 60 x 8 9.92 / 9.98, 4 of 40000 x 12 0.98 / 1.25; with 4 problems of 512^2, one of
// 100000 x 3 1.03 / 1.10, four 2.26 / 1.90.
bool batch_strips(const BatchSize* probs, int n) {
    int64_t narrow = 0, wide = 0, strips = 0, tiles = 0;
    for (int p = 0; p < n; ++p) {
        const BatchSize& q = probs[p];
        int ntx;
        const int64_t t = batch_reg_tiles(q.nx, q.nrows, 4, &ntx);
        tiles += t;
        if (q.nrows > 8) continue;
        strips += t;
        (q.nrows <= 4 ? narrow : wide) += q.nx;
    }
    return (narrow > 36000 || narrow + wide > 70000) && 4 * strips > 3 * tiles;
}

// Steps per tick for problems of the given interior sizes and steps per
// application, from the model above: every tick costs its launches (25 us with
// the counters and the CG kernels) and its rounds of tiles; the longest
// application sets the number of ticks, all problems the work.
int batch_reg_steps(const std::vector<BatchSize>& probs) {
    constexpr int rows = BNW * BR;
    int best = 4;
    double tbest = 1e300;
    for (int H = 4; H <= 10; ++H) {
        double work = 0;
        int ticks = 0, ntx;
        const double inner = (64 - 2 * H) * (rows - 2 * H);
        const double round = 3.0 + 0.04 * rows + 2.4e-3 * inner + H * (0.11 + 0.018 * rows);
        for (const BatchSize& q : probs) {
            const int n = (q.nsteps + H - 1) / H;
            work += (double)batch_reg_tiles(q.nx, q.nrows, H, &ntx) * n;
            ticks = std::max(ticks, n);
        }
        const double t = ticks * 25.0 + std::max(work / 256.0, (double)ticks) * round;
        if (t < tbest) {
            tbest = t;
            best = H;
        }
    }
    return best;
}

void launch_batch_tiles(bool force, int ntiles, int H, hipStream_t s, const BProb2D* pr, const BState* st, int np,
                        double sgn, int amode) {
    if (ntiles <= 0) return;
    const dim3 grid((unsigned)ntiles);
    if (force)
        hipLaunchKernelGGL(batch_tile2d_kernel<true>, grid, dim3(64 * BNW), 0, s, pr, st, np, H, sgn, amode);
    else
        hipLaunchKernelGGL(batch_tile2d_kernel<false>, grid, dim3(64 * BNW), 0, s, pr, st, np, H, sgn, amode);
}

}  // namespace elwh
