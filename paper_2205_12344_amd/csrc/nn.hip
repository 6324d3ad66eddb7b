// Learned warm start for the Krylov solve (C ABI elwh_ws_* in include/elwh.h).
//
// A convolutional encoder-decoder (U-Net, five resolution levels, 3x3
// convolutions with bias and SiLU, 2x2 average pooling, nearest upsampling,
// skip concatenation; 1 644 578 parameters) maps the problem data on the node
// grid -- log rho, log mu, log(lambda/mu), the forcing normalised by its
// maximum, omega h and omega -- to the displacement, and its output seeds the
// solve (x0).  Convolutions are implicit GEMMs on MFMA with BF16 operands and
// FP32 accumulation (nn_conv.hip); master weights, pre-activations, gradients
// and Adam state are FP32.  Training minimises the relative error in the M-weighted
// norm against solutions computed by the solver itself.
#include <cmath>
#include <cstring>
#include <new>
#include <random>
#include <string>
#include <utility>
#include <vector>

#include "elwh_internal.h"
#include "nn_internal.h"

using namespace elwh;

namespace {

struct Conv {
    int cin, cout, act;
    int64_t woff, boff;   // offsets of W [9 cin][cout] and bias [cout] in the flat parameter vector
};

// Layer table, in parameter order.
const int kLayers[][3] = {
    {7, 32, 1},    {32, 32, 1},   // e0
    {32, 64, 1},   {64, 64, 1},   // e1
    {64, 96, 1},   {96, 96, 1},   // e2
    {96, 128, 1},  {128, 128, 1}, // e3
    {128, 128, 1}, {128, 128, 1}, // e4 (bottleneck)
    {256, 128, 1}, {128, 128, 1}, // d3
    {224, 96, 1},  {96, 96, 1},   // d2
    {160, 64, 1},  {64, 64, 1},   // d1
    {96, 32, 1},   {32, 32, 1},   // d0
    {32, 2, 0},                   // head
};
constexpr int NL = sizeof(kLayers) / sizeof(kLayers[0]);
constexpr int NOUT = 2, NLEV = 5;
static_assert(NL <= nn::kLayersMax, "layer tables");
const int kWidth[NLEV] = {32, 64, 96, 128, 128};

}  // namespace

struct elwh_ws {
    int maxB = 0, H = 0, W = 0;
    hipStream_t stream = nullptr;
    std::string err;
    std::vector<Conv> L;
    char* arena = nullptr;                                // every device buffer below
    std::vector<std::pair<void**, size_t>> want;
    int64_t nparam = 0;
    float *P = nullptr, *G = nullptr, *Mo = nullptr, *Vo = nullptr;   // params, grads, Adam moments
    int step = 0;
    double out_scale = 1.0;
    std::vector<unsigned short*> Wf, Wb;   // packed BF16 weights per layer: forward, input gradient
    bool packed_bwd = false;               // Wb belongs to the current parameters
    // per conv layer: pre-activation (FP32, for the gradient), activation and
    // pre-activation gradient (BF16, the operands of the convolutions)
    std::vector<float*> Z;
    std::vector<unsigned short*> A, dZ;
    unsigned short* pool[NLEV - 1] = {};   // pooled activations (input of level l+1)
    float* dskip[NLEV - 1] = {};           // gradient of the skips, until the pooled one joins it
    float* yout = nullptr;                 // network output
    float* dout = nullptr;                 // its gradient
    std::vector<float*> dbpart;            // bias-gradient partials per layer
    float* bpart = nullptr;
    float* part = nullptr;                 // weight-gradient partials
    int64_t part_elems = 0;
    float* lossb = nullptr;                // per-sample loss
    float* lden = nullptr;                 // per-sample weighted norm of the target
    float* hloss = nullptr;                // pinned
    // feature scratch
    double* fmax = nullptr;
    const double** dptr = nullptr;     // device pointer tables
};

namespace {

thread_local std::string g_ws_err;

#define WCK(expr)                                                               \
    do {                                                                        \
        hipError_t e_ = (expr);                                                 \
        if (e_ != hipSuccess) {                                                 \
            ws->err = std::string(#expr) + ": " + hipGetErrorString(e_);        \
            return ELWH_ERR_HIP;                                                \
        }                                                                       \
    } while (0)

int level_of(int l) {
    // e0..e4: layers 0..9 -> level l/2; d3..d0: layers 10..17 -> 3 - (l-10)/2; head: 0
    if (l < 10) return l / 2;
    if (l < 18) return 3 - (l - 10) / 2;
    return 0;
}

// the layer whose output is upsampled into decoder layer l
int deeper_of(int l) { return l == 10 ? 9 : l - 1; }

struct LayerIn {
    nn::ConvSrc S;
    int src;
};

LayerIn layer_input(const elwh_ws* ws, int l, int B, const float* x) {
    const int lev = level_of(l);
    LayerIn in;
    in.S.B = B;
    in.S.H = ws->H >> lev;
    in.S.W = ws->W >> lev;
    in.src = nn::SRC_PLAIN;
    in.S.c0 = ws->L[l].cin;
    if (l == 0) {
        in.src = nn::SRC_FIRST;
        in.S.f = x;
    } else if (l < 10 && l % 2 == 0) {
        in.S.x0 = ws->pool[lev - 1];   // first conv of encoder level lev > 0
    } else if (l >= 10 && l < 18 && l % 2 == 0) {
        in.src = nn::SRC_CAT;
        in.S.x0 = ws->A[deeper_of(l)];
        in.S.c0 = ws->L[deeper_of(l)].cout;
        in.S.x1 = ws->A[2 * lev + 1];
        in.S.c1 = kWidth[lev];
    } else {
        in.S.x0 = ws->A[l - 1];
    }
    return in;
}

// Pre-activations are kept only when a backward pass follows.
elwh_status forward(elwh_ws* ws, int B, const float* x, float* y, bool keep) {
    // encoder, then decoder level 3 down to 0, then the head: the layer order
    for (int l = 0; l < NL; ++l) {
        const Conv& c = ws->L[l];
        const LayerIn in = layer_input(ws, l, B, x);
        const bool head = l == NL - 1;
        unsigned short* pool = l < 8 && l % 2 == 1 ? ws->pool[l / 2] : nullptr;
        WCK(nn::conv_forward(ws->stream, in.S, in.src, c.cin, c.cout, c.act, ws->Wf[l], ws->P + c.boff,
                             keep ? ws->Z[l] : nullptr, ws->A[l], pool, head ? y : nullptr));
    }
    return ELWH_OK;
}

// BF16 weights of the current parameters in the kernels' layout; those of the
// input gradient (none for the first layer) when a backward pass needs them.
void pack(elwh_ws* ws, bool backward) {
    nn::PackTable T;
    T.backward = backward ? 1 : 0;
    int n = 0;
    for (int l = backward ? 1 : 0; l < NL; ++l) {
        const Conv& c = ws->L[l];
        T.l[n++] = {backward ? ws->Wb[l] : ws->Wf[l], c.woff, c.cin, c.cout, nn::pack_ksteps(c.cin, c.cout, backward)};
    }
    nn::pack_weights(ws->stream, T, n, ws->P);
    if (!backward) ws->packed_bwd = false;
}

// Gradients of every parameter into G; dout holds dL/dy and dbpart[head] its sums.
elwh_status backward(elwh_ws* ws, int B, const float* x) {
    if (!ws->packed_bwd) {
        pack(ws, true);
        ws->packed_bwd = true;
    }
    nn::BiasGrads T;
    auto bias_layer = [&](int l, int64_t rows) {
        T.l[l] = {ws->dbpart[l], ws->G + ws->L[l].boff, rows, ws->L[l].cout};
    };
    bias_layer(NL - 1, nn::loss_blocks((int64_t)B * ws->H * ws->W));
    auto back = [&](int l) -> elwh_status {
        const Conv& c = ws->L[l];
        const LayerIn in = layer_input(ws, l, B, x);
        const bool head = l == NL - 1;
        nn::ConvSrc gz;
        gz.B = B;
        gz.H = in.S.H;
        gz.W = in.S.W;
        gz.c0 = c.cout;
        gz.x0 = head ? nullptr : ws->dZ[l];
        gz.f = head ? ws->dout : nullptr;
        const int srcz = head ? nn::SRC_HEAD : nn::SRC_PLAIN;
        WCK(nn::conv_weight_grad(ws->stream, in.S, in.src, gz, srcz, c.cin, c.cout, ws->part, ws->part_elems,
                                 ws->G + c.woff));
        if (l == 0) return ELWH_OK;
        nn::GradDst D;
        int to = l - 1;   // the layer that produced this input
        if (in.src == nn::SRC_CAT) {
            D.mode = nn::GRAD_CAT;
            to = deeper_of(l);
            D.cup = ws->L[to].cout;
            D.dskip = ws->dskip[level_of(l)];
        } else if (l < 10 && l % 2 == 0) {
            D.mode = nn::GRAD_UNPOOL;
            D.dskip = ws->dskip[level_of(l) - 1];
        }
        D.Z = ws->Z[to];
        D.dZ = ws->dZ[to];
        D.dbpart = ws->dbpart[to];
        WCK(nn::conv_input_grad(ws->stream, gz, srcz, c.cout, c.cin, ws->Wb[l], D));
        bias_layer(to, nn::grad_rows(c.cin, B, gz.H, gz.W));
        return ELWH_OK;
    };
    elwh_status st;
    if ((st = back(NL - 1))) return st;
    for (int lev = 0; lev <= NLEV - 2; ++lev) {
        const int la = 10 + 2 * (NLEV - 2 - lev);
        if ((st = back(la + 1)) || (st = back(la))) return st;
    }
    // encoder, deepest first
    for (int l = 9; l >= 0; --l)
        if ((st = back(l))) return st;
    nn::bias_grads(ws->stream, T, NL, ws->bpart);
    return ELWH_OK;
}

// Every device buffer is a part of one allocation: alloc() notes the pointer and
// its size, commit() allocates the sum and hands out the parts (creating the
// handle with one hipMalloc per buffer spent longer on those calls than on
// anything else).
void alloc(elwh_ws* ws, void** p, size_t bytes) { ws->want.emplace_back(p, (bytes + 255) / 256 * 256); }

elwh_status commit(elwh_ws* ws) {
    size_t total = 0;
    for (const auto& w : ws->want) total += w.second;
    if (hipMalloc(reinterpret_cast<void**>(&ws->arena), total) != hipSuccess) {
        ws->arena = nullptr;
        ws->err = "device allocation failed (" + std::to_string(total) + " bytes)";
        return ELWH_ERR_ALLOC;
    }
    (void)hipMemsetAsync(ws->arena, 0, total, ws->stream);
    size_t off = 0;
    for (const auto& w : ws->want) {
        *w.first = ws->arena + off;
        off += w.second;
    }
    ws->want.clear();
    return ELWH_OK;
}

void free_ws(elwh_ws* ws) {
    if (ws->arena) (void)hipFree(ws->arena);
    if (ws->hloss) (void)hipHostFree(ws->hloss);
}

// ---- problem data <-> network tensors ----------------------------------------
// Network pixel (py, px) <-> node (i = px, j = py + 1) of an n x n-cell grid
// (H = W = n), i.e. the unknown rows 1..n of a Dirichlet-bottom / free-top
// square plus the Dirichlet column i = 0.

__global__ void fmax_kernel(const double* const* __restrict__ f, int nn, double* __restrict__ out) {
    const double* fb = f[blockIdx.x];
    double m = 0.0;
    for (int e = threadIdx.x; e < 2 * nn; e += blockDim.x) m = fmax(m, fabs(fb[e]));
    __shared__ double red[256];
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0] > 0 ? red[0] : 1.0;
}

// Per-sample target normalisation: y[b] /= sqrt(sum w y^2 / (2 sum w)), the
// w-weighted RMS over both components (one block per sample, FP64 sums;
// samples with no weight or a zero target are left as they are).
__global__ void normalize_kernel(float* __restrict__ y, const float* __restrict__ w, int npix) {
    float* yb = y + (int64_t)blockIdx.x * npix * 2;
    const float* wb = w + (int64_t)blockIdx.x * npix;
    double sy = 0.0, sw = 0.0;
    for (int p = threadIdx.x; p < npix; p += blockDim.x) {
        const double wp = wb[p], a = yb[2 * p], c = yb[2 * p + 1];
        sy += wp * (a * a + c * c);
        sw += wp;
    }
    __shared__ double r1[256], r2[256];
    __shared__ float scale;
    r1[threadIdx.x] = sy;
    r2[threadIdx.x] = sw;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            r1[threadIdx.x] += r1[threadIdx.x + st];
            r2[threadIdx.x] += r2[threadIdx.x + st];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double rms = r2[0] > 0 ? sqrt(r1[0] / (2.0 * r2[0])) : 0.0;
        scale = rms > 0 ? (float)(1.0 / rms) : 1.0f;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < 2 * npix; p += blockDim.x) yb[p] *= scale;
}

// x[b,py,px,:] = (log rho/0.2, log mu/0.2, log(lam/mu)/0.5, fx/fmax, fy/fmax, 5 omega h, omega/60)
// w[b,py,px] = M weight of the node (trapezoid weight * rho), 0 on Dirichlet nodes
__global__ void features_kernel(const double* const* __restrict__ rho, const double* const* __restrict__ lam,
                                const double* const* __restrict__ mu, const double* const* __restrict__ f,
                                const double* __restrict__ omega, const double* __restrict__ fmx, int n,
                                float* __restrict__ x, float* __restrict__ w, int B) {
    const int64_t npix = (int64_t)n * n;
    const int64_t total = npix * B;
    const int nn1 = n + 1;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(e / npix);
        const int64_t pix = e - (int64_t)b * npix;
        const int py = (int)(pix / n), px = (int)(pix - (int64_t)py * n);
        const int i = px, j = py + 1;
        const int64_t node = (int64_t)j * nn1 + i;
        const double r = rho[b][node], l = lam[b][node], m = mu[b][node];
        const double s = 1.0 / fmx[b];
        float* xo = x + e * 7;
        xo[0] = (float)(log(r) / 0.2);
        xo[1] = (float)(log(m) / 0.2);
        xo[2] = (float)(log(l / m) / 0.5);
        xo[3] = (float)(f[b][node] * s);
        xo[4] = (float)(f[b][node + (int64_t)nn1 * nn1] * s);
        xo[5] = (float)(5.0 * omega[b] / n);
        xo[6] = (float)(omega[b] / 60.0);
        const bool unknown = i >= 1 && i <= n - 1;
        const double wt = (j == n) ? 0.5 : 1.0;   // free top row carries trapezoid weight 1/2
        w[e] = unknown ? (float)(wt * r) : 0.f;
    }
}

// y[b,py,px,c] = v_c(i,j) * omega^2 / (fmax * k)   (targets from solutions)
__global__ void from_field_kernel(const double* const* __restrict__ v, const double* __restrict__ omega,
                                  const double* __restrict__ fmx, double k, int n, float* __restrict__ y, int B) {
    const int64_t npix = (int64_t)n * n;
    const int nn1 = n + 1;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < npix * B; e += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(e / npix);
        const int64_t pix = e - (int64_t)b * npix;
        const int py = (int)(pix / n), px = (int)(pix - (int64_t)py * n);
        const int64_t node = (int64_t)(py + 1) * nn1 + px;
        const double s = omega[b] * omega[b] / (fmx[b] * k);
        y[e * 2] = (float)(v[b][node] * s);
        y[e * 2 + 1] = (float)(v[b][node + (int64_t)nn1 * nn1] * s);
    }
}

// x0_c(i,j) = y[b,py,px,c] * fmax * k / omega^2 on unknown nodes, 0 elsewhere
__global__ void to_field_kernel(const float* __restrict__ y, const double* __restrict__ omega,
                                const double* __restrict__ fmx, double k, int n, double* const* __restrict__ x0, int B) {
    const int nn1 = n + 1;
    const int64_t nodes = (int64_t)nn1 * nn1;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nodes * B; e += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(e / nodes);
        const int64_t node = e - (int64_t)b * nodes;
        const int j = (int)(node / nn1), i = (int)(node - (int64_t)j * nn1);
        double u = 0.0, v = 0.0;
        if (i >= 1 && i <= n - 1 && j >= 1) {
            const int64_t pix = ((int64_t)b * n + (j - 1)) * n + i;
            const double s = fmx[b] * k / (omega[b] * omega[b]);
            u = y[pix * 2] * s;
            v = y[pix * 2 + 1] * s;
        }
        x0[b][node] = u;
        x0[b][node + nodes] = v;
    }
}

unsigned g1(int64_t n) {
    const int64_t g = (n + 255) / 256;
    return (unsigned)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

elwh_status upload_ptrs(elwh_ws* ws, int B, const double* const* a, int slot) {
    WCK(hipMemcpyAsync(ws->dptr + (size_t)slot * ws->maxB, a, sizeof(double*) * B, hipMemcpyHostToDevice, ws->stream));
    return ELWH_OK;
}

}  // namespace

extern "C" {

elwh_status elwh_ws_create(int max_batch, int H, int W, unsigned long long seed, void* stream, elwh_ws** out) {
    if (!out) return ELWH_ERR_ARG;
    *out = nullptr;
    if (max_batch < 1 || H < 16 || W < 16 || H % 16 || W % 16 || (int64_t)H * W * max_batch > (1LL << 26)) {
        g_ws_err = "network: H, W must be multiples of 16 (>= 16); batch x H x W <= 2^26";
        return ELWH_ERR_ARG;
    }
    elwh_ws* ws = new (std::nothrow) elwh_ws();
    if (!ws) return ELWH_ERR_ALLOC;
    ws->maxB = max_batch;
    ws->H = H;
    ws->W = W;
    ws->stream = reinterpret_cast<hipStream_t>(stream);
    auto fail = [&](elwh_status s) {
        g_ws_err = ws->err;
        free_ws(ws);
        delete ws;
        return s;
    };
    int64_t off = 0;
    for (int l = 0; l < NL; ++l) {
        Conv c{kLayers[l][0], kLayers[l][1], kLayers[l][2], 0, 0};
        c.woff = off;
        off += 9LL * c.cin * c.cout;
        c.boff = off;
        off += c.cout;
        ws->L.push_back(c);
    }
    ws->nparam = off;
    const size_t np = (size_t)off;
    for (float** p : {&ws->P, &ws->G, &ws->Mo, &ws->Vo}) alloc(ws, (void**)p, np * 4);
    const int64_t B = max_batch;
    for (auto* v : {&ws->Wf, &ws->Wb, &ws->A, &ws->dZ}) v->resize(NL);
    ws->Z.resize(NL);
    ws->dbpart.resize(NL);
    int64_t max_w = 0;
    for (int l = 0; l < NL; ++l) {
        const Conv& c = ws->L[l];
        const int lev = level_of(l);
        const int64_t npix = B * (H >> lev) * (W >> lev);
        alloc(ws, (void**)&ws->Wf[l], nn::packed_elems(c.cin, c.cout, false) * 2);
        if (l > 0) alloc(ws, (void**)&ws->Wb[l], nn::packed_elems(c.cin, c.cout, true) * 2);
        max_w = std::max<int64_t>(max_w, 9LL * c.cin * c.cout);
        if (l < NL - 1) {
            alloc(ws, (void**)&ws->Z[l], (size_t)npix * c.cout * 4);
            alloc(ws, (void**)&ws->A[l], (size_t)npix * c.cout * 2);
            alloc(ws, (void**)&ws->dZ[l], (size_t)npix * c.cout * 2);
        }
        // bias partials: the rows written by the layer whose input gradient
        // reaches this layer through its SiLU
        int64_t rows = nn::loss_blocks(npix);
        if (l < NL - 1) {
            const int by = l + 1, lb = level_of(by);
            rows = nn::grad_rows(kLayers[by][0], max_batch, H >> lb, W >> lb);
        }
        alloc(ws, (void**)&ws->dbpart[l], (size_t)rows * c.cout * 4);
    }
    for (int lev = 0; lev < NLEV - 1; ++lev) {
        const int64_t npix1 = B * (H >> (lev + 1)) * (W >> (lev + 1));
        const int64_t npix = B * (H >> lev) * (W >> lev);
        alloc(ws, (void**)&ws->pool[lev], (size_t)npix1 * kWidth[lev] * 2);
        alloc(ws, (void**)&ws->dskip[lev], (size_t)npix * kWidth[lev] * 4);
    }
    // weight-gradient shares: about 512 workgroups of one 32 x 32 channel block each
    ws->part_elems = std::max<int64_t>(512LL * 9 * 32 * 32, max_w);
    alloc(ws, (void**)&ws->dout, (size_t)B * H * W * NOUT * 4);
    alloc(ws, (void**)&ws->yout, (size_t)B * H * W * NOUT * 4);
    alloc(ws, (void**)&ws->bpart, sizeof(float) * nn::kLayersMax * nn::kBiasChunks * 128);
    alloc(ws, (void**)&ws->part, (size_t)ws->part_elems * 4);
    alloc(ws, (void**)&ws->lossb, (size_t)B * 4);
    alloc(ws, (void**)&ws->lden, (size_t)B * 4);
    alloc(ws, (void**)&ws->fmax, (size_t)B * 8);
    alloc(ws, (void**)&ws->dptr, (size_t)B * 8 * sizeof(double*));
    elwh_status st;
    if ((st = commit(ws))) return fail(st);
    if (hipHostMalloc((void**)&ws->hloss, (size_t)B * 4, hipHostMallocDefault) != hipSuccess) return fail(ELWH_ERR_ALLOC);
    // He-style initialisation (seeded), zero biases; the head starts small
    std::vector<float> hp(np, 0.f);
    std::mt19937_64 rng(seed);
    for (int l = 0; l < NL; ++l) {
        const Conv& c = ws->L[l];
        const double sd = std::sqrt(2.0 / (9.0 * c.cin)) * (l == NL - 1 ? 0.1 : 1.0);
        std::normal_distribution<double> nd(0.0, sd);
        for (int64_t k = 0; k < 9LL * c.cin * c.cout; ++k) hp[c.woff + k] = (float)nd(rng);
    }
    if (hipMemcpyAsync(ws->P, hp.data(), np * 4, hipMemcpyHostToDevice, ws->stream) != hipSuccess)
        return fail(ELWH_ERR_HIP);
    pack(ws, false);
    if (hipStreamSynchronize(ws->stream) != hipSuccess) return fail(ELWH_ERR_HIP);
    *out = ws;
    return ELWH_OK;
}

void elwh_ws_destroy(elwh_ws* ws) {
    if (!ws) return;
    (void)hipStreamSynchronize(ws->stream);
    free_ws(ws);
    delete ws;
}

const char* elwh_ws_last_error(const elwh_ws* ws) { return ws ? ws->err.c_str() : g_ws_err.c_str(); }

long long elwh_ws_num_params(const elwh_ws* ws) { return ws ? ws->nparam : -1; }

elwh_status elwh_ws_params(elwh_ws* ws, float* get, const float* set, double* out_scale_get, const double* out_scale_set) {
    if (!ws) return ELWH_ERR_ARG;
    if (set) {
        WCK(hipMemcpyAsync(ws->P, set, ws->nparam * 4, hipMemcpyHostToDevice, ws->stream));
        pack(ws, false);
        WCK(hipMemsetAsync(ws->Mo, 0, ws->nparam * 4, ws->stream));
        WCK(hipMemsetAsync(ws->Vo, 0, ws->nparam * 4, ws->stream));
        ws->step = 0;
    }
    if (out_scale_set) ws->out_scale = *out_scale_set;
    if (out_scale_get) *out_scale_get = ws->out_scale;
    if (get) WCK(hipMemcpyAsync(get, ws->P, ws->nparam * 4, hipMemcpyDeviceToHost, ws->stream));
    WCK(hipStreamSynchronize(ws->stream));
    return ELWH_OK;
}

elwh_status elwh_ws_forward(elwh_ws* ws, int B, const float* x, float* y) {
    if (!ws || !x || !y || B < 1 || B > ws->maxB) return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = forward(ws, B, x, y, false))) return st;
    WCK(hipGetLastError());
    return ELWH_OK;
}

elwh_status elwh_ws_loss_grad(elwh_ws* ws, int B, const float* x, const float* y, const float* w, float* loss,
                              float* grad_host) {
    if (!ws || !x || !y || !w || B < 1 || B > ws->maxB) return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = forward(ws, B, x, ws->yout, true))) return st;
    nn::loss(ws->stream, ws->yout, y, w, B, (int64_t)ws->H * ws->W, ws->dout, ws->lossb, ws->lden, ws->dbpart[NL - 1]);
    if ((st = backward(ws, B, x))) return st;
    WCK(hipMemcpyAsync(ws->hloss, ws->lossb, sizeof(float) * B, hipMemcpyDeviceToHost, ws->stream));
    if (grad_host) WCK(hipMemcpyAsync(grad_host, ws->G, ws->nparam * 4, hipMemcpyDeviceToHost, ws->stream));
    WCK(hipStreamSynchronize(ws->stream));
    if (loss) {
        double s = 0;
        for (int b = 0; b < B; ++b) s += ws->hloss[b];
        *loss = (float)s;
    }
    return ELWH_OK;
}

elwh_status elwh_ws_train_step(elwh_ws* ws, int B, const float* x, const float* y, const float* w, float lr,
                               float* loss) {
    if (!ws || !x || !y || !w || B < 1 || B > ws->maxB || !(lr > 0)) return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = forward(ws, B, x, ws->yout, true))) return st;
    nn::loss(ws->stream, ws->yout, y, w, B, (int64_t)ws->H * ws->W, ws->dout, ws->lossb, ws->lden, ws->dbpart[NL - 1]);
    if ((st = backward(ws, B, x))) return st;
    ws->step++;
    nn::adam(ws->stream, ws->P, ws->G, ws->Mo, ws->Vo, ws->nparam, lr, 0.9f, 0.999f, 1e-8f, ws->step);
    pack(ws, false);
    if (loss) {
        WCK(hipMemcpyAsync(ws->hloss, ws->lossb, sizeof(float) * B, hipMemcpyDeviceToHost, ws->stream));
        WCK(hipStreamSynchronize(ws->stream));
        double s = 0;
        for (int b = 0; b < B; ++b) s += ws->hloss[b];
        *loss = (float)s;
    }
    WCK(hipGetLastError());
    return ELWH_OK;
}

elwh_status elwh_ws_features(elwh_ws* ws, int B, int n, const double* const* rho, const double* const* lam,
                             const double* const* mu, const double* const* f, const double* omega_dev, float* x,
                             float* w) {
    if (!ws || B < 1 || B > ws->maxB || n != ws->H || n != ws->W || !rho || !lam || !mu || !f || !omega_dev || !x ||
        !w)
        return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = upload_ptrs(ws, B, rho, 0)) || (st = upload_ptrs(ws, B, lam, 1)) || (st = upload_ptrs(ws, B, mu, 2)) ||
        (st = upload_ptrs(ws, B, f, 3)))
        return st;
    const double** d = ws->dptr;
    const int M = ws->maxB;
    hipLaunchKernelGGL(fmax_kernel, dim3(B), dim3(256), 0, ws->stream, d + 3 * M, (n + 1) * (n + 1), ws->fmax);
    hipLaunchKernelGGL(features_kernel, dim3(g1((int64_t)B * n * n)), dim3(256), 0, ws->stream, d, d + M, d + 2 * M,
                       d + 3 * M, omega_dev, ws->fmax, n, x, w, B);
    WCK(hipStreamSynchronize(ws->stream));   // the pointer tables are reused by the next call
    WCK(hipGetLastError());
    return ELWH_OK;
}

elwh_status elwh_ws_from_field(elwh_ws* ws, int B, int n, const double* const* f, const double* const* v,
                               const double* omega_dev, float* y) {
    if (!ws || B < 1 || B > ws->maxB || n != ws->H || !f || !v || !omega_dev || !y) return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = upload_ptrs(ws, B, f, 3)) || (st = upload_ptrs(ws, B, v, 4))) return st;
    const double** d = ws->dptr;
    const int M = ws->maxB;
    hipLaunchKernelGGL(fmax_kernel, dim3(B), dim3(256), 0, ws->stream, d + 3 * M, (n + 1) * (n + 1), ws->fmax);
    hipLaunchKernelGGL(from_field_kernel, dim3(g1((int64_t)B * n * n)), dim3(256), 0, ws->stream, d + 4 * M,
                       omega_dev, ws->fmax, ws->out_scale, n, y, B);
    WCK(hipStreamSynchronize(ws->stream));
    WCK(hipGetLastError());
    return ELWH_OK;
}

elwh_status elwh_ws_normalize(elwh_ws* ws, int B, float* y, const float* w) {
    if (!ws || B < 1 || B > ws->maxB || !y || !w) return ELWH_ERR_ARG;
    hipLaunchKernelGGL(normalize_kernel, dim3(B), dim3(256), 0, ws->stream, y, w, ws->H * ws->W);
    WCK(hipGetLastError());
    return ELWH_OK;
}

elwh_status elwh_ws_predict(elwh_ws* ws, int B, int n, const float* x, const double* const* f, const double* omega_dev,
                            double* const* x0) {
    if (!ws || B < 1 || B > ws->maxB || n != ws->H || !x || !f || !omega_dev || !x0) return ELWH_ERR_ARG;
    elwh_status st;
    if ((st = forward(ws, B, x, ws->yout, false))) return st;
    if ((st = upload_ptrs(ws, B, f, 3)) ||
        (st = upload_ptrs(ws, B, reinterpret_cast<const double* const*>(x0), 5)))
        return st;
    const double** d = ws->dptr;
    const int M = ws->maxB;
    hipLaunchKernelGGL(fmax_kernel, dim3(B), dim3(256), 0, ws->stream, d + 3 * M, (n + 1) * (n + 1), ws->fmax);
    hipLaunchKernelGGL(to_field_kernel, dim3(g1((int64_t)B * (n + 1) * (n + 1))), dim3(256), 0, ws->stream,
                       ws->yout, omega_dev, ws->fmax, ws->out_scale, n,
                       reinterpret_cast<double* const*>(const_cast<double**>(d + 5 * M)), B);
    WCK(hipStreamSynchronize(ws->stream));
    WCK(hipGetLastError());
    return ELWH_OK;
}

}  // extern "C"
