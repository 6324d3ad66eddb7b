// Mapped 2-D El-WaveHoltz steps on register tiles (FP64): several steps of the
// scheme of kernels2d_curv.hip per launch.
//
// A single step moves 136 B per update and the marching kernel reaches the HBM
// rate with it (80.6 us per step at 801 x 4003 cells), so only fewer passes help.
// As on Cartesian grids (kernels2d_tile.hip), a workgroup of 8 wavefronts keeps
// a tile of 8 R rows x 64 columns (R = 4, 5) in registers for up to H steps, exact
// on its inner (64 - 2 H) x (8 R - 2 H) nodes, and wavefronts exchange their
// first and last rows through LDS once per step.  Half of a launch is its steps
// (1.65 us each), half its loads and stores, near the HBM rate; one workgroup fills a
// CU's registers, so the two do not overlap.
//
// Each difference is taken once per edge: with e_R, e_N the differences to the
// right and upper neighbours, per edge
//   G = (K^qq_C + K^qq_R) e_R + P_C + P_R,   P = K^qr (U_N - U_S),
//   H = (K^rr_C + K^rr_N) e_N + Q_C + Q_N,   Q = (K^qr)^T (U_R - U_L),
// and L_h U = G_right - G_left + H_up - H_down, the spacings folded into the
// coefficients, which are formed from lam, mu and the metric at the load and
// stay in registers (K summed over the edge; both parts of the neighbour's P
// and G by DPP along q).  42 FP64 operations per node and step.  Dirichlet
// nodes keep a = 0 and with it their zero.  On a traction-free r side the
// difference and the flux across it mirror those inside: e_N = e_S, H_up = -H_down
// (the one-sided rows of kernels2d_curv.hip, divided by their weight 1/2).
//
// The sum, f and the neighbours' K^qr wait in LDS: registers hold the rest without
// spilling (240).  Handing each node's contributions on to its neighbours instead (80
// operations per node) took 41.2 instead of 37.3 us per step with 8 x 4 rows.
#include <algorithm>
#include <cmath>

#include "step2d_common.h"

namespace elwh {

namespace {

struct V2d {
    double x, y;
};
__device__ __forceinline__ V2d operator+(const V2d& a, const V2d& b) { return V2d{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ V2d operator-(const V2d& a, const V2d& b) { return V2d{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ V2d left2(const V2d& a) { return V2d{lane_from_left_z(a.x), lane_from_left_z(a.y)}; }
__device__ __forceinline__ V2d right2(const V2d& a) { return V2d{lane_from_right_z(a.x), lane_from_right_z(a.y)}; }
struct Sym2 {
    double a, b, c;   // 00, 01 (= 10), 11
};
struct Mat2 {
    double a, b, c, d;   // 00, 01, 10, 11
};
__device__ __forceinline__ V2d operator*(const Sym2& k, const V2d& v) {
    return V2d{fma(k.a, v.x, k.b * v.y), fma(k.b, v.x, k.c * v.y)};
}
__device__ __forceinline__ V2d operator*(const Mat2& k, const V2d& v) {
    return V2d{fma(k.a, v.x, k.b * v.y), fma(k.c, v.x, k.d * v.y)};
}
__device__ __forceinline__ V2d mul_t(const Mat2& k, const V2d& v) {
    return V2d{fma(k.a, v.x, k.c * v.y), fma(k.b, v.x, k.d * v.y)};
}

struct CurvPtrs {
    const double *l, *m, *g0, *g1, *g2, *g3;
};

template <int NW, int R, bool FORCE>
__global__ __launch_bounds__(64 * NW) void curv_tile_kernel(const double* __restrict__ u,
                                                            const double* __restrict__ uprev,
                                                            double* __restrict__ outA, double* __restrict__ outB,
                                                            const double* __restrict__ base, double* __restrict__ acc,
                                                            const double* __restrict__ ca, CurvPtrs M,
                                                            const double* __restrict__ f, Tile2D A) {
    __shared__ double ex[2][NW][2][2][64];   // [buffer][wavefront][first, last row][u, v][column]
    __shared__ double cf[NW][2][4][64];      // K^qr of the first and last rows
    __shared__ double sm[NW * R][2][64];     // the sum, read and written by its own lane only, as is:
    __shared__ double af[FORCE ? NW * R : 1][2][64];
    const int W = 64 - 2 * A.H, HV = NW * R - 2 * A.H;
    const int ntx = (A.nx - 1 + W - 1) / W, nty = (A.jhi - A.jlo + HV) / HV;
    int t;
    if (!xcd_tile((int)blockIdx.x, ntx * nty, t)) return;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = 1 + (t % ntx) * W - A.H + lane;
    const int row0 = A.jlo + (t / ntx) * HV - A.H + w * R;
    const bool colv = col >= 0 && col <= A.nx, colu = col >= 1 && col < A.nx;
    const int64_t P = A.P, CS = A.CS;

    V2d x0[R + 2], x1[R + 2];   // rows 0 and R + 1 are the neighbours'
    Sym2 qq[R], rr[R];
    Mat2 qr[R];
    double a[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int j = row0 + k, q = w * R + k;
        const bool in = colv && j >= 0 && j <= A.ny;
        const int64_t o = (int64_t)j * P + col;
        const double l = in ? M.l[o] : 0.0, m = in ? M.m[o] : 0.0, lm = l + m;
        const double A0 = in ? M.g0[o] : 0.0, A1 = in ? M.g1[o] : 0.0, B0 = in ? M.g2[o] : 0.0, B1 = in ? M.g3[o] : 0.0;
        const double AA = A0 * A0 + A1 * A1, BB = B0 * B0 + B1 * B1, AB = A0 * B0 + A1 * B1;
        qq[k] = Sym2{A.cxx2 * (lm * A0 * A0 + m * AA), A.cxx2 * (lm * A0 * A1), A.cxx2 * (lm * A1 * A1 + m * AA)};
        rr[k] = Sym2{A.cyy2 * (lm * B0 * B0 + m * BB), A.cyy2 * (lm * B0 * B1), A.cyy2 * (lm * B1 * B1 + m * BB)};
        qr[k] = Mat2{A.cxy * (lm * A0 * B0 + m * AB), A.cxy * (l * A0 * B1 + m * B0 * A1),
                     A.cxy * (l * A1 * B0 + m * B1 * A0), A.cxy * (lm * A1 * B1 + m * AB)};
        const bool unk = colu && j >= A.jlo && j <= A.jhi;
        x0[k + 1] = unk ? V2d{u[o], u[o + CS]} : V2d{0.0, 0.0};
        a[k] = unk ? ca[o] : 0.0;
        x1[k + 1] = unk && uprev ? V2d{uprev[o], uprev[o + CS]} : V2d{0.0, 0.0};
        const bool own = unk && lane >= A.H && lane < 64 - A.H && q >= A.H && q < NW * R - A.H;
        const double* b = A.first ? base : acc;
        V2d sum = own && b ? V2d{b[o], b[o + CS]} : V2d{0.0, 0.0};
        if (A.first) {
            sum.x = fma(A.w0, x0[k + 1].x, sum.x);
            sum.y = fma(A.w0, x0[k + 1].y, sum.y);
        }
        sm[q][0][lane] = sum.x;
        sm[q][1][lane] = sum.y;
        if constexpr (FORCE) {
            af[q][0][lane] = unk ? f[o] : 0.0;
            af[q][1][lane] = unk ? f[o + CS] : 0.0;
        }
    }
    // K of both ends of an edge, summed: along q across lanes, along r across wavefronts
    const int wb = w > 0 ? w - 1 : w, wa = w < NW - 1 ? w + 1 : w;   // (the tile's outermost rows are not exact)
    Sym2 rrS;
    {
        double(&e)[NW][8][64] = reinterpret_cast<double(&)[NW][8][64]>(ex);
        const Sym2 f0 = rr[0], f1 = rr[R - 1];
        e[w][0][lane] = f0.a;
        e[w][1][lane] = f0.b;
        e[w][2][lane] = f0.c;
        e[w][3][lane] = f1.a;
        e[w][4][lane] = f1.b;
        e[w][5][lane] = f1.c;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const Mat2& k = qr[b ? R - 1 : 0];
            cf[w][b][0][lane] = k.a;
            cf[w][b][1][lane] = k.b;
            cf[w][b][2][lane] = k.c;
            cf[w][b][3][lane] = k.d;
        }
        __syncthreads();
        rrS = Sym2{f0.a + e[wb][3][lane], f0.b + e[wb][4][lane], f0.c + e[wb][5][lane]};
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const Sym2 n = k < R - 1 ? rr[k < R - 1 ? k + 1 : 0] : Sym2{e[wa][0][lane], e[wa][1][lane], e[wa][2][lane]};
            rr[k] = Sym2{rr[k].a + n.a, rr[k].b + n.b, rr[k].c + n.c};
            qq[k] = Sym2{qq[k].a + lane_from_right_z(qq[k].a), qq[k].b + lane_from_right_z(qq[k].b),
                         qq[k].c + lane_from_right_z(qq[k].c)};
        }
        __syncthreads();
    }
    auto edge_qr = [&](int v, int b) __attribute__((always_inline)) {
        return Mat2{cf[v][b][0][lane], cf[v][b][1][lane], cf[v][b][2][lane], cf[v][b][3][lane]};
    };
    // the array rows (1 .. R) of the free sides in this wavefront, 0 if none
    const int rtop = A.free_hi && A.ny >= row0 && A.ny < row0 + R ? A.ny - row0 + 1 : 0;
    const int rbot = A.free_lo && 0 >= row0 && 0 < row0 + R ? 1 - row0 : 0;
    auto exchange = [&](V2d(&Y)[R + 2], int buf) __attribute__((always_inline)) {
        double(&e)[NW][2][2][64] = ex[buf];
        e[w][0][0][lane] = Y[1].x;
        e[w][0][1][lane] = Y[1].y;
        e[w][1][0][lane] = Y[R].x;
        e[w][1][1][lane] = Y[R].y;
        __syncthreads();
        Y[0] = V2d{e[wb][1][0][lane], e[wb][1][1][lane]};
        Y[R + 1] = V2d{e[wa][0][0][lane], e[wa][0][1][lane]};
    };
    exchange(x0, 1);

    // one step: X the current level with its neighbour rows, Y the level before,
    // overwritten by the next one (before the start: 0)
    auto step = [&](const V2d(&X)[R + 2], V2d(&Y)[R + 2], int s, bool more) __attribute__((always_inline)) {
        const double wk = A.wk[s], fc = FORCE ? A.fck[s] : 0.0;
        const bool start = s == 0 && A.first;
        V2d eS = X[1] - X[0], eR = right2(X[1]) - X[1], Q, HS;
        {
            const V2d dR = right2(X[0]) - X[0];
            const V2d Q0 = mul_t(edge_qr(wb, 1), dR + left2(dR));
            Q = mul_t(qr[0], eR + left2(eR));
            HS = rrS * eS + (Q0 + Q);
        }
#pragma unroll
        for (int r = 1; r <= R; ++r) {
            const int k = r - 1;
            const V2d dR = right2(X[r + 1]) - X[r + 1];
            const V2d QN = mul_t(r < R ? qr[r < R ? r : 0] : edge_qr(wa, 0), dR + left2(dR));
            V2d eN = X[r + 1] - X[r];
            V2d HN = rr[k] * eN + (Q + QN);
            if (rtop == r || rbot == r) {
                // (the empty asm keeps this rare, uniform branch from becoming selects)
                asm volatile("");
                if (rtop == r) {
                    eN = eS;
                    HN = V2d{-HS.x, -HS.y};
                } else {
                    eS = eN;
                    HS = V2d{-HN.x, -HN.y};
                }
            }
            const V2d p = qr[k] * (eN + eS);
            const V2d G = qq[k] * eR + (p + right2(p));
            V2d T = (G - left2(G)) + (HN - HS);
            if constexpr (FORCE) {
                T.x = fma(-fc, af[w * R + k][0][lane], T.x);
                T.y = fma(-fc, af[w * R + k][1][lane], T.y);
            }
            V2d n{fma(a[k], T.x, fma(2.0, X[r].x, -Y[r].x)), fma(a[k], T.y, fma(2.0, X[r].y, -Y[r].y))};
            if (start) {
                asm volatile("");
                n.x *= 0.5;
                n.y *= 0.5;
            }
            Y[r] = n;
            double(&z)[2][64] = sm[w * R + k];
            z[0][lane] = fma(wk, n.x, z[0][lane]);
            z[1][lane] = fma(wk, n.y, z[1][lane]);
            eS = eN;
            HS = HN;
            eR = dR;
            Q = QN;
        }
        if (more) exchange(Y, s & 1);
    };
    int s = 0;
    for (; s + 2 <= A.steps; s += 2) {
        step(x0, x1, s, true);
        step(x1, x0, s + 1, s + 2 < A.steps);
    }
    // X the level before the last, Y the last
    auto store = [&](const V2d(&X)[R + 2], const V2d(&Y)[R + 2]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int j = row0 + k, q = w * R + k;
            if (colu && j >= A.jlo && j <= A.jhi && lane >= A.H && lane < 64 - A.H && q >= A.H && q < NW * R - A.H) {
                const int64_t o = (int64_t)j * P + col;
                if (A.steps > 1) {
                    outA[o] = X[k + 1].x;
                    outA[o + CS] = X[k + 1].y;
                }
                outB[o] = Y[k + 1].x;
                outB[o + CS] = Y[k + 1].y;
                acc[o] = sm[q][0][lane];
                acc[o + CS] = sm[q][1][lane];
            }
        }
    };
    if (s < A.steps) {   // one step more: the roles are exchanged
        step(x0, x1, s, false);
        store(x0, x1);
    } else {
        store(x1, x0);
    }
}

template <int NW, int R>
void curv_tile_launch(bool force, hipStream_t s, const double* u, const double* uprev, double* outA, double* outB,
                      const double* base, double* acc, const double* ca, const CurvPtrs& M, const double* f,
                      const Tile2D& A) {
    const int W = 64 - 2 * A.H, HV = NW * R - 2 * A.H;
    const dim3 grid((unsigned)xcd_grid(((A.nx - 1 + W - 1) / W) * ((A.jhi - A.jlo + HV) / HV)));
    if (force)
        hipLaunchKernelGGL((curv_tile_kernel<NW, R, true>), grid, dim3(64 * NW), 0, s, u, uprev, outA, outB, base, acc,
                           ca, M, f, A);
    else
        hipLaunchKernelGGL((curv_tile_kernel<NW, R, false>), grid, dim3(64 * NW), 0, s, u, uprev, outA, outB, base, acc,
                           ca, M, f, A);
}

}  // namespace

// Shape and steps per launch from a model of one application, fitted to
// measurements at 40 x 20 to 801 x 4003 cells: a launch costs 3 us and its loads
// and stores at 7 TB/s (halos read from L2), a round of one tile per CU 1.5 us and
// its steps (8 x 4 rows 1.41, 8 x 5 rows 1.65 us each).  At 801 x 4003: 35.1 us per
// step (8 x 5 rows; 8 x 4 rows 38.0, workgroups of 4 wavefronts, two per CU, 36.9, 8 x 6
// rows spill and take 39.1), marching single steps 80.6; 600 x 1000 6.5 against 16.0,
// 300 x 300 2.2 against 8.8, 40 x 20 1.9 against 8.0: they serve wide grids of a few
// rows (strip2d_rule) and a tiling that was asked for.
TileShape curv_tile_shape(const elwh_ctx* c) {
    TileShape best;
    const int nx = c->L.nx, nrows = c->mr.hi - c->mr.lo + 1, N = c->plan.nt * c->opts.periods;
    if (!own_steps(c, strip2d_rule(nx, nrows, true), true)) return best;   // the marching kernel
    double tbest = 1e300;
    for (int R = 4; R <= 5; ++R) {
        const int rows = 8 * R;
        for (int H = 3; H <= std::min(kTileMaxSteps, rows / 2 - 1); ++H) {
            const int W = 64 - 2 * H, HV = rows - 2 * H;
            const double tiles = (double)((nx - 2 + W) / W) * ((nrows - 1 + HV) / HV);
            const double bytes = tiles * (64.0 * rows * 104 + (double)W * HV * 48);
            const double launch = 3.0 + bytes / 7e6 + std::ceil(tiles / 256) * (1.5 + H * (R == 4 ? 1.41 : 1.65));
            const double t = launch * ((N + H - 1) / H);
            if (t < tbest) {
                tbest = t;
                best.NW = 8;
                best.R = R;
                best.H = H;
            }
        }
    }
    return best;
}

void run_filter_curv_tile2d(elwh_ctx* c, const TileShape& t, const double* x, bool with_force, bool amode,
                            double* out) {
    const int nsteps = c->plan.nt * c->opts.periods;
    const double sgn = amode ? -1.0 : 1.0;
    Tile2D A = tile2d_args(c, t);
    A.w0 = sgn * c->w[0];
    const CurvPtrs M{c->cl, c->cm, c->cg[0], c->cg[1], c->cg[2], c->cg[3]};
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
        const auto launch = t.R == 4 ? curv_tile_launch<8, 4> : curv_tile_launch<8, 5>;
        launch(with_force, c->stream, cur, prev, o[0], o[1], amode ? x : nullptr, out, c->ca, M, c->f64, A);
        prev = A.steps > 1 ? o[0] : cur;
        cur = o[1];
    }
    prof_mark(c, 2, nsteps);
}

}  // namespace elwh
