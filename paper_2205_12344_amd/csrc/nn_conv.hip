// The 3x3 convolutions of the warm-start network as implicit GEMMs on MFMA:
// forward, gradient with respect to the input, gradient with respect to the
// weights.  Operands are BF16, sums FP32.
//
// What bounds them.  An im2col matrix in HBM makes every input value travel
// nine times at 2 bytes (and its gradient nine times at 4): that form took
// 48.1 ms for the forward pass of 48 problems at 256^2 (0.84 TFLOP) and 52.2 ms
// for loss and gradient of 16, mostly im2col and col2im; these kernels take 2.35
// and 4.99 ms (356 and 167 TFLOP/s), bound by LDS and L2 reads of the operands
// in the main loops and by the FP32 pre-activation traffic of the gradients.
// Here a workgroup stages the input pixels of its tile once, all channels and
// a one-pixel halo, in LDS (pixel rows padded by 16 bytes, so the 16-byte reads
// of neighbouring pixels fall on different banks), and the nine taps are nine
// offsets into it.  Pooling, upsampling and the concatenation with the skip
// are done while staging or in the epilogue, so no tensor is written only to
// be read in another shape.
//
// The weights are the A operand (their 32 output channels the matrix rows) and
// the pixels the B operand: a lane then holds four consecutive channels of
// one pixel per register group and stores them as one vector.  Weight fragments
// are packed once per parameter update in the order the lanes read them, and
// come straight from L2 into registers, two k-steps ahead.
//
// Sums run over taps, then channels in steps of 16, by v_mfma_f32_32x32x16_bf16
// (and, for the input gradient, per tap from zero and then over the taps), the
// order of the im2col GEMMs these replaced: the forward pass and the input
// gradient of given operands are the same bits.  Weight and bias gradients sum over
// pixels, in another order (FP32 as before; 3e-7 apart at 16 samples of 256^2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "nn_internal.h"

namespace elwh {
namespace nn {

typedef unsigned short u16;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// round to nearest even
__device__ __forceinline__ u16 f2bf(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (u16)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}
__device__ __forceinline__ float sigm(float z) { return 1.f / (1.f + __expf(-z)); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = sigm(z);
    return s * (1.f + z * (1.f - s));
}
__device__ __forceinline__ uint2 pack4(const float* v) {
    return make_uint2((unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16),
                      (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16));
}

// ---- staging -------------------------------------------------------------------
// Input kinds: a BF16 tensor; the decoder's concatenation [upsampled low-level
// tensor, skip]; the 7-channel FP32 network input (as 64 columns k = 7 tap + c,
// one zero); the 2-channel FP32 gradient of the output.

__device__ __forceinline__ bool src_pixel(const ConvSrc& S, int b, int yy, int xx, int64_t& pix) {
    pix = ((int64_t)b * S.H + yy) * S.W + xx;
    return yy >= 0 && yy < S.H && xx >= 0 && xx < S.W;
}

// The 8 channels c .. c+7 of pixel (yy, xx) (zero outside the image).
template <int SRC>
__device__ __forceinline__ uint4 src_load8(const ConvSrc& S, int b, int yy, int xx, int c) {
    uint4 v = make_uint4(0, 0, 0, 0);
    int64_t pix;
    if (!src_pixel(S, b, yy, xx, pix)) return v;
    if (SRC == SRC_PLAIN) {
        v = *reinterpret_cast<const uint4*>(S.x0 + pix * S.c0 + c);
    } else if (SRC == SRC_CAT) {
        if (c < S.c0) {
            const int64_t low = ((int64_t)b * (S.H / 2) + yy / 2) * (S.W / 2) + xx / 2;
            v = *reinterpret_cast<const uint4*>(S.x0 + low * S.c0 + c);
        } else {
            v = *reinterpret_cast<const uint4*>(S.x1 + pix * S.c1 + (c - S.c0));
        }
    } else if (SRC == SRC_HEAD) {
        if (c == 0) {
            const float2 d = *reinterpret_cast<const float2*>(S.f + pix * 2);
            v.x = (unsigned)f2bf(d.x) | ((unsigned)f2bf(d.y) << 16);
        }
    }
    return v;
}

// Halo tile (rows y0-1 .., columns x0-1 ..) of (TH + 2) x (TW + 2) pixels, all
// `cin` channels, into lds[pixel][cin + 8].
template <int SRC>
__device__ __forceinline__ void stage_tile(const ConvSrc& S, int b, int y0, int x0, int TH, int TW, int cin, u16* lds) {
    const int G = cin >> 3, TW2 = TW + 2, total = (TH + 2) * TW2 * G, stride = cin + 8;
    const float invG = 1.0f / (float)G, invW = 1.0f / (float)TW2;
    for (int g0 = threadIdx.x; g0 < total; g0 += 4 * blockDim.x) {
        uint4 v[4];
        int off[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int g = g0 + k * (int)blockDim.x;
            off[k] = -1;
            if (g < total) {
                const int pix = (int)(((float)g + 0.5f) * invG), c = (g - pix * G) << 3;
                const int r = (int)(((float)pix + 0.5f) * invW), q = pix - r * TW2;
                v[k] = src_load8<SRC>(S, b, y0 + r - 1, x0 + q - 1, c);
                off[k] = pix * stride + c;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (off[k] >= 0) *reinterpret_cast<uint4*>(lds + off[k]) = v[k];
    }
}

// The network input's halo tile as BF16 rows of 7 (TW + 2) values (a row's values
// are consecutive in memory), then rows of im2col values k = 7 tap + c: the 21
// values of one ky are consecutive in the halo row too, so value k of a pixel
// sits at a fixed offset from its top left neighbour's.
__device__ __forceinline__ void stage_raw(const ConvSrc& S, int b, int y0, int x0, int TH, int TW, u16* raw) {
    const int row = 7 * (TW + 2), lo = 7 * (1 - x0), hi = 7 * (S.W + 1 - x0), total = (TH + 2) * row;
    for (int e0 = threadIdx.x; e0 < total; e0 += 8 * blockDim.x) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = e0 + k * (int)blockDim.x, r = e / row, q = e - r * row, y = y0 + r - 1;
            v[k] = 0.f;
            if (e < total && y >= 0 && y < S.H && q >= lo && q < hi)
                v[k] = S.f[(((int64_t)b * S.H + y) * S.W + x0 - 1) * 7 + q];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (e0 + k * (int)blockDim.x < total) raw[e0 + k * blockDim.x] = f2bf(v[k]);
    }
}

__device__ __forceinline__ int raw_offset(int k, int TW) {
    const int ky = k >= 42 ? 2 : (k >= 21 ? 1 : 0);
    return ky * 7 * (TW + 2) + k - 21 * ky;
}

// nk (a power of two) values k0 .. k0 + nk - 1 of every pixel, two per store
__device__ __forceinline__ void stage_cols(const u16* raw, int TH, int TW, int k0, int nk, int pitch, u16* dst) {
    const int half = nk >> 1, j = threadIdx.x & (half - 1), k = k0 + 2 * j;
    const int oa = raw_offset(k, TW), ob = raw_offset(k + 1, TW);
    const bool last = k + 1 == 63;   // the 64th value is zero
    for (int pix = threadIdx.x / half; pix < TH * TW; pix += blockDim.x / half) {
        const u16* src = raw + ((pix / TW) * (TW + 2) + (pix & (TW - 1))) * 7;
        const unsigned v = (unsigned)src[oa] | (last ? 0u : (unsigned)src[ob] << 16);
        *reinterpret_cast<unsigned*>(dst + pix * pitch + 2 * j) = v;
    }
}

// Tile origin of workgroup t: x tiles fastest, then y tiles, then samples.
__device__ __forceinline__ void tile_origin(int t, int H, int W, int TH, int TW, int& b, int& y0, int& x0) {
    const int nx = (W + TW - 1) / TW, ny = (H + TH - 1) / TH;
    x0 = (t % nx) * TW;
    t /= nx;
    y0 = (t % ny) * TH;
    b = t / ny;
}

__device__ __forceinline__ bf16x8_t frag(const u16* p) {
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(p));
}

// ---- forward ---------------------------------------------------------------------
// Workgroup: wp x wc wavefronts; a wavefront computes MT tiles of 32 output
// channels for PT tiles of 32 pixels (32 x 1 pixels, or 16 x 2 where the image
// is at most 16 wide).  FIRST reads k from the im2col rows (one "tap").
template <int MT, int PT, int TWL, int SRC>
__global__ __launch_bounds__(512) void conv_forward_kernel(ConvSrc S, int cin, int cout, int act, int wc,
                                                           const u16* __restrict__ Wp, const float* __restrict__ bias,
                                                           float* __restrict__ Z, u16* __restrict__ A,
                                                           u16* __restrict__ pool, float* __restrict__ out) {
    extern __shared__ u16 lds[];
    constexpr int TW = 1 << TWL, RT = 32 >> TWL;   // columns and rows of a pixel tile
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wpi = wave / wc, wci = wave - wpi * wc, wp = (blockDim.x >> 6) / wc;
    const int TH = wp * PT * RT;
    int b, y0, x0;
    tile_origin(blockIdx.x, S.H, S.W, TH, TW, b, y0, x0);
    constexpr bool FIRST = SRC == SRC_FIRST;
    if (FIRST) {
        u16* raw = lds + TH * TW * 72;
        stage_raw(S, b, y0, x0, TH, TW, raw);
        __syncthreads();
        stage_cols(raw, TH, TW, 0, 64, 72, lds);
    } else {
        stage_tile<SRC>(S, b, y0, x0, TH, TW, cin, lds);
    }
    __syncthreads();

    const int h = lane >> 5, p = lane & 31, px = p & (TW - 1), pr = p >> TWL;
    const int stride = FIRST ? 72 : cin + 8, rowlen = FIRST ? TW : TW + 2;
    const int KC = FIRST ? 4 : cin >> 4, taps = FIRST ? 1 : 9, nct = (cout + 31) >> 5;
    const int ct0 = wci * MT;
    const u16* base[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) base[t] = lds + (((wpi * PT + t) * RT + pr) * rowlen + px) * stride + 8 * h;
    const u16* w = Wp + ((int64_t)ct0 * 64 + lane) * 8;
    const int64_t wstep = (int64_t)nct * 512;
    float16_t acc[MT][PT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][t][r] = 0.f;
    // weight fragments two k-steps ahead (KC is even; the packed array ends in two spare steps)
    bf16x8_t wf[2][MT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) wf[s][m] = frag(w + s * wstep + m * 512);
    for (int tap = 0; tap < taps; ++tap) {
        const int ky = tap / 3, kx = tap - ky * 3, toff = (ky * rowlen + kx) * stride;
        for (int kc = 0; kc < KC; kc += 2) {
            w += 2 * wstep;
            bf16x8_t wn[2][MT];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) wn[s][m] = frag(w + s * wstep + m * 512);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                bf16x8_t x[PT];
#pragma unroll
                for (int t = 0; t < PT; ++t) x[t] = frag(base[t] + toff + (kc + s) * 16);
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int t = 0; t < PT; ++t)
                        acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s][m], x[t], acc[m][t], 0, 0, 0);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) wf[s][m] = wn[s][m];
        }
    }

#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int cb = (ct0 + m) * 32;
        if (cb >= cout) continue;
        if (out) {   // the head: two channels, FP32
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const int y = y0 + (wpi * PT + t) * RT + pr, x = x0 + px;
                if (h == 0 && y < S.H && x < S.W)
                    *reinterpret_cast<float2*>(out + (((int64_t)b * S.H + y) * S.W + x) * 2) =
                        make_float2(acc[m][t][0] + bias[0], acc[m][t][1] + bias[1]);
            }
            continue;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = cb + 8 * q + 4 * h;
            const float4 bv = *reinterpret_cast<const float4*>(bias + c);
            float a[PT][4];
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const float z[4] = {acc[m][t][4 * q] + bv.x, acc[m][t][4 * q + 1] + bv.y, acc[m][t][4 * q + 2] + bv.z,
                                    acc[m][t][4 * q + 3] + bv.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) a[t][i] = act ? z[i] * sigm(z[i]) : z[i];
                const int y = y0 + (wpi * PT + t) * RT + pr, x = x0 + px;
                if (y < S.H && x < S.W) {
                    const int64_t o = (((int64_t)b * S.H + y) * S.W + x) * cout + c;
                    if (Z) *reinterpret_cast<float4*>(Z + o) = make_float4(z[0], z[1], z[2], z[3]);
                    *reinterpret_cast<uint2*>(A + o) = pack4(a[t]);
                }
            }
            if (pool) {
                // 2x2 mean of the FP32 activations: x + 1 is the next lane, y + 1 the
                // next tile (32-wide tiles) or lane + 16 (16-wide)
#pragma unroll
                for (int t = 0; t < PT; t += RT == 1 ? 2 : 1) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = a[t][i];
                        const float up = RT == 1 ? a[t + (RT == 1 ? 1 : 0)][i] : __shfl_xor(lo, 16);
                        v[i] = 0.25f * (lo + __shfl_xor(lo, 1) + up + __shfl_xor(up, 1));
                    }
                    const int y = y0 + (wpi * PT + t) * RT + pr, x = x0 + px;
                    if (y < S.H && x < S.W && !(x & 1) && !(y & 1))
                        *reinterpret_cast<uint2*>(pool + (((int64_t)b * (S.H / 2) + y / 2) * (S.W / 2) + x / 2) * cout +
                                                  c) = pack4(v);
                }
            }
        }
    }
}

// ---- gradient with respect to the input --------------------------------------------
// Sum of the 32 pixel lanes of each half wavefront: v[r] over the lanes, the
// result for register r in the even lane whose bits 4..1 spell r; that lane
// stores channel 8 (r / 4) + 4 h + r % 4.
__device__ __forceinline__ void store_channel_sum(float (&v)[16], int lane, float* __restrict__ dst) {
    int r = 0;
#pragma unroll
    for (int n = 8, bit = 16; n >= 1; n >>= 1, bit >>= 1) {
        const bool hi = (lane & bit) != 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < n) {
                const float keep = hi ? v[i + n] : v[i], send = hi ? v[i] : v[i + n];
                v[i] = keep + __shfl_xor(send, bit);
            }
        r = 2 * r + (hi ? 1 : 0);
    }
    const float s = v[0] + __shfl_xor(v[0], 1);
    if (!(lane & 1)) dst[8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] = s;
}

// dX of one layer and, in the same pass, the pre-activation gradient dZ (BF16)
// and the bias-gradient partials (FP32 sums per wavefront) of the layer that
// produced that input.  The output channels [0, cup) of a concatenated input
// belong to the upsampled layer (2x2 sum), the others to the skip (kept in
// FP32 until the pooled gradient of the level below joins them); the input of
// a level's first convolution is a pooled tensor (unpool: dA = dskip + dX / 4
// for the four pixels).
template <int MT, int PT, int TWL, int SRC>
__global__ __launch_bounds__(512) void conv_input_grad_kernel(ConvSrc S, int cz, int cin, int wc,
                                                              const u16* __restrict__ Wp, GradDst D) {
    extern __shared__ u16 lds[];
    constexpr int TW = 1 << TWL, RT = 32 >> TWL;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wpi = wave / wc, wci = wave - wpi * wc, wp = (blockDim.x >> 6) / wc;
    const int TH = wp * PT * RT;
    int b, y0, x0;
    tile_origin(blockIdx.x, S.H, S.W, TH, TW, b, y0, x0);
    stage_tile<SRC>(S, b, y0, x0, TH, TW, cz, lds);
    __syncthreads();
    const int nct = cin >> 5;
    const int ct0 = (blockIdx.y * wc + wci) * MT;
    if (ct0 >= nct) return;

    const int h = lane >> 5, p = lane & 31, px = p & (TW - 1), pr = p >> TWL;
    const int stride = cz + 8, KC = cz >> 4;
    const u16* base[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) base[t] = lds + (((wpi * PT + t) * RT + pr) * (TW + 2) + px) * stride + 8 * h;
    const u16* w = Wp + ((int64_t)ct0 * 64 + lane) * 8;
    const int64_t wstep = (int64_t)nct * 512;
    float16_t sum[MT][PT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[m][t][r] = 0.f;
    bf16x8_t wf[2][MT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) wf[s][m] = frag(w + s * wstep + m * 512);
    for (int tap = 0; tap < 9; ++tap) {
        const int ky = tap / 3, kx = tap - ky * 3, toff = ((2 - ky) * (TW + 2) + 2 - kx) * stride;
        float16_t acc[MT][PT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[m][t][r] = 0.f;
        for (int kc = 0; kc < KC; kc += 2) {
            w += 2 * wstep;
            bf16x8_t wn[2][MT];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) wn[s][m] = frag(w + s * wstep + m * 512);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                bf16x8_t x[PT];
#pragma unroll
                for (int t = 0; t < PT; ++t) x[t] = frag(base[t] + toff + (kc + s) * 16);
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int t = 0; t < PT; ++t)
                        acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s][m], x[t], acc[m][t], 0, 0, 0);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) wf[s][m] = wn[s][m];
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < PT; ++t) sum[m][t] += acc[m][t];
    }

    const int64_t prow = (int64_t)blockIdx.x * wp + wpi;   // row of the bias-gradient partials
    auto emit = [&](const float16_t(&g0)[PT], int cb) {
        float db[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) db[r] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = cb + 8 * q + 4 * h;
            if (D.mode == GRAD_CAT && cb < D.cup) {
                // upsampled half: the 2x2 sum is the gradient of the low-level activation
#pragma unroll
                for (int t = 0; t < PT; t += RT == 1 ? 2 : 1) {
                    float g[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = g0[t][4 * q + i];
                        const float up = RT == 1 ? g0[t + (RT == 1 ? 1 : 0)][4 * q + i] : __shfl_xor(lo, 16);
                        g[i] = lo + __shfl_xor(lo, 1) + up + __shfl_xor(up, 1);
                    }
                    const int y = y0 + (wpi * PT + t) * RT + pr, x = x0 + px;
                    if (y < S.H && x < S.W && !(x & 1) && !(y & 1)) {
                        const int64_t o = (((int64_t)b * (S.H / 2) + y / 2) * (S.W / 2) + x / 2) * D.cup + c;
                        const float4 z = *reinterpret_cast<const float4*>(D.Z + o);
                        g[0] *= silu_grad(z.x);
                        g[1] *= silu_grad(z.y);
                        g[2] *= silu_grad(z.z);
                        g[3] *= silu_grad(z.w);
                        *reinterpret_cast<uint2*>(D.dZ + o) = pack4(g);
#pragma unroll
                        for (int i = 0; i < 4; ++i) db[4 * q + i] += g[i];
                    }
                }
                continue;
            }
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const int y = y0 + (wpi * PT + t) * RT + pr, x = x0 + px;
                if (y >= S.H || x >= S.W) continue;
                float g[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) g[i] = g0[t][4 * q + i];
                if (D.mode == GRAD_CAT) {
                    const int64_t o = (((int64_t)b * S.H + y) * S.W + x) * (cin - D.cup) + (c - D.cup);
                    *reinterpret_cast<float4*>(D.dskip + o) = make_float4(g[0], g[1], g[2], g[3]);
                } else if (D.mode == GRAD_PLAIN) {
                    const int64_t o = (((int64_t)b * S.H + y) * S.W + x) * cin + c;
                    const float4 z = *reinterpret_cast<const float4*>(D.Z + o);
                    g[0] *= silu_grad(z.x);
                    g[1] *= silu_grad(z.y);
                    g[2] *= silu_grad(z.z);
                    g[3] *= silu_grad(z.w);
                    *reinterpret_cast<uint2*>(D.dZ + o) = pack4(g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) db[4 * q + i] += g[i];
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int64_t o =
                            (((int64_t)b * 2 * S.H + 2 * y + (k >> 1)) * 2 * S.W + 2 * x + (k & 1)) * cin + c;
                        const float4 z = *reinterpret_cast<const float4*>(D.Z + o);
                        const float4 d = *reinterpret_cast<const float4*>(D.dskip + o);
                        float e[4] = {d.x + 0.25f * g[0], d.y + 0.25f * g[1], d.z + 0.25f * g[2], d.w + 0.25f * g[3]};
                        e[0] *= silu_grad(z.x);
                        e[1] *= silu_grad(z.y);
                        e[2] *= silu_grad(z.z);
                        e[3] *= silu_grad(z.w);
                        *reinterpret_cast<uint2*>(D.dZ + o) = pack4(e);
#pragma unroll
                        for (int i = 0; i < 4; ++i) db[4 * q + i] += e[i];
                    }
                }
            }
        }
        if (D.mode != GRAD_CAT)
            store_channel_sum(db, lane, D.dbpart + prow * cin + cb);
        else if (cb < D.cup)
            store_channel_sum(db, lane, D.dbpart + prow * D.cup + cb);
    };
    emit(sum[0], ct0 * 32);
    if constexpr (MT == 2) emit(sum[1], (ct0 + 1) * 32);
}

// ---- gradient with respect to the weights ------------------------------------------
// dW[tap][ci][o] = sum over pixels of X[pixel + tap][ci] dZ[pixel][o]: pixels
// are the contraction index, 16 consecutive ones of a row per MFMA step.  A
// workgroup owns 32 input and 32 output channels (nine 32x32 accumulators per
// wavefront, one per tap) and walks a share of the pixel tiles (32 x 8, the
// rows split over four wavefronts); tiles are staged as [pixel][32 + 4]
// values, and a lane collects its channel's pixels with 2-byte LDS reads (the
// 36-value pitch puts the two half wavefronts, 8 pixels apart, on different
// banks).  A row's ten pixels serve its three taps, the middle one by funnel
// shifts.  The shares are added in a fixed order by sum_partials_kernel.
constexpr int WG_TW = 32, WG_TH = 8, WG_P = 36;

template <int SRC>
__device__ __forceinline__ void stage_slice(const ConvSrc& S, int b, int y0, int x0, int rows, int cols, int halo,
                                            int c0, u16* lds) {
    const int total = rows * cols * 4;
    for (int g = threadIdx.x; g < total; g += blockDim.x) {
        const int pix = g >> 2, c = (g & 3) << 3, r = pix / cols, q = pix - r * cols;
        const uint4 v = src_load8<SRC>(S, b, y0 + r - halo, x0 + q - halo, c0 + c);
        u16* d = lds + pix * WG_P + c;
        *reinterpret_cast<uint2*>(d) = make_uint2(v.x, v.y);
        *reinterpret_cast<uint2*>(d + 4) = make_uint2(v.z, v.w);
    }
}

template <int SRCX, int SRCZ>
__global__ __launch_bounds__(256) void conv_weight_grad_kernel(ConvSrc X, ConvSrc Gz, int K, int cout, int nci,
                                                               int ntiles, int per, float* __restrict__ part) {
    constexpr bool FIRST = SRCX == SRC_FIRST;
    constexpr int NT = FIRST ? 1 : 9, HALO = FIRST ? 0 : 1;
    constexpr int XC = WG_TW + 2 * HALO, XR = WG_TH + 2 * HALO;
    __shared__ __attribute__((aligned(16))) u16 smem[XR * XC * WG_P + WG_TW * WG_TH * WG_P];
    u16* xs = smem;
    u16* zs = smem + XR * XC * WG_P;
    __shared__ u16 raw[FIRST ? (WG_TH + 2) * (WG_TW + 2) * 7 : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, p = lane & 31;
    const int cib = blockIdx.x % nci, cob = blockIdx.x / nci;
    const int nx = (X.W + WG_TW - 1) / WG_TW, ny = (X.H + WG_TH - 1) / WG_TH;
    float16_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    const int t0 = blockIdx.y * per, t1 = min(ntiles, t0 + per);
    for (int tile = t0; tile < t1; ++tile) {
        const int x0 = (tile % nx) * WG_TW, y0 = ((tile / nx) % ny) * WG_TH, b = tile / (nx * ny);
        __syncthreads();
        if (FIRST) {
            stage_raw(X, b, y0, x0, WG_TH, WG_TW, raw);
            __syncthreads();
            stage_cols(raw, WG_TH, WG_TW, cib * 32, 32, WG_P, xs);
        } else {
            stage_slice<SRCX>(X, b, y0, x0, XR, XC, HALO, cib * 32, xs);
        }
        stage_slice<SRCZ>(Gz, b, y0, x0, WG_TH, WG_TW, 0, cob * 32, zs);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = wave * 2 + (k >> 1), xb = (k & 1) * 16 + 8 * h;
            union {
                unsigned u[4];
                bf16x8_t v;
            } zf, xf;
            const u16* zp = zs + (row * WG_TW + xb) * WG_P + p;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                zf.u[e] = (unsigned)zp[2 * e * WG_P] | ((unsigned)zp[(2 * e + 1) * WG_P] << 16);
            if (FIRST) {
                const u16* xp = xs + (row * WG_TW + xb) * WG_P + p;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    xf.u[e] = (unsigned)xp[2 * e * WG_P] | ((unsigned)xp[(2 * e + 1) * WG_P] << 16);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v, zf.v, acc[0], 0, 0, 0);
            } else {
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const u16* xp = xs + ((row + ky) * XC + xb) * WG_P + p;
                    unsigned pr[5];
#pragma unroll
                    for (int e = 0; e < 5; ++e)
                        pr[e] = (unsigned)xp[2 * e * WG_P] | ((unsigned)xp[(2 * e + 1) * WG_P] << 16);
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            xf.u[e] = kx == 0 ? pr[e]
                                              : (kx == 2 ? pr[e + 1] : __builtin_amdgcn_alignbit(pr[e + 1], pr[e], 16));
                        acc[3 * ky + kx] =
                            __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v, zf.v, acc[3 * ky + kx], 0, 0, 0);
                    }
                }
            }
        }
    }
    // add the four wavefronts, tap by tap, and write this share
    float* red = reinterpret_cast<float*>(smem);   // [4][32][32]
    float* dst = part + (int64_t)blockIdx.y * K * cout;
    const int cin = FIRST ? K : K / 9;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r)
            red[wave * 1024 + (8 * (r >> 2) + 4 * h + (r & 3)) * 32 + p] = acc[t][r];
        __syncthreads();
        for (int e = threadIdx.x; e < 1024; e += 256) {
            const int ci = cib * 32 + (e >> 5), o = cob * 32 + (e & 31);
            if (ci < cin && o < cout)
                dst[((int64_t)t * cin + ci) * cout + o] =
                    red[e] + red[1024 + e] + red[2048 + e] + red[3072 + e];
        }
    }
}

__global__ void sum_partials_kernel(const float* __restrict__ part, int splits, int64_t n, float* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    float s = 0.f;
    int z = 0;
    for (; z + 8 <= splits; z += 8) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = part[(int64_t)(z + k) * n + e];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += v[k];
    }
    for (; z < splits; ++z) s += part[(int64_t)z * n + e];
    out[e] = s;
}

// Bias gradients of every layer: rows of per-wavefront sums, first over
// kBiasChunks shares of the rows, then over the shares, in a fixed order.
__global__ __launch_bounds__(256) void bias_grad_rows_kernel(BiasGrads T, float* __restrict__ part) {
    const BiasGrads::Layer L = T.l[blockIdx.y];
    const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    const int64_t per = (L.rows + kBiasChunks - 1) / kBiasChunks, a = blockIdx.x * per, e = min(L.rows, a + per);
    __shared__ float red[8][32];
    for (int cb = 0; cb < L.C; cb += 32) {
        float s = 0.f;
        if (cb + c < L.C)
            for (int64_t r = a + r0; r < e; r += 8) s += L.in[r * L.C + cb + c];
        __syncthreads();
        red[r0][c] = s;
        __syncthreads();
        if (r0 == 0 && cb + c < L.C) {
            for (int k = 1; k < 8; ++k) s += red[k][c];
            part[((int64_t)blockIdx.y * kBiasChunks + blockIdx.x) * 128 + cb + c] = s;
        }
    }
}

__global__ void bias_grad_sum_kernel(BiasGrads T, const float* __restrict__ part) {
    const BiasGrads::Layer L = T.l[blockIdx.x];
    const int c = threadIdx.x;
    if (c >= L.C) return;
    float s = 0.f;
    for (int k = 0; k < kBiasChunks; ++k) s += part[((int64_t)blockIdx.x * kBiasChunks + k) * 128 + c];
    L.out[c] = s;
}

// ---- packed weights ---------------------------------------------------------------
// Fragment order [tap][k step][32 output channels][lane][8], BF16.  Forward: rows
// are output channels, k the input channels (the first layer: k = 7 tap + c);
// input gradient: rows are input channels, k the output channels.
__global__ void pack_weights_kernel(PackTable T, const float* __restrict__ params) {
    const PackTable::Layer L = T.l[blockIdx.y];
    const float* W = params + L.woff;
    const int rows = T.backward ? L.cin : L.cout, nct = (rows + 31) >> 5;
    const int taps = !T.backward && L.cin % 16 ? 1 : 9, total = taps * L.ks * nct * 512;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int i = e & 7, lane = (e >> 3) & 63;
        int f = e >> 9;
        const int ct = f % nct;
        f /= nct;
        const int kc = f % L.ks, tap = f / L.ks;
        const int row = ct * 32 + (lane & 31), k = kc * 16 + 8 * (lane >> 5) + i;
        float v = 0.f;
        if (T.backward) {
            if (row < L.cin && k < L.cout) v = W[((int64_t)tap * L.cin + row) * L.cout + k];
        } else if (taps == 1) {
            if (k < 9 * L.cin && row < L.cout) v = W[(int64_t)k * L.cout + row];
        } else if (row < L.cout && k < L.cin) {
            v = W[((int64_t)tap * L.cin + k) * L.cout + row];
        }
        L.out[e] = f2bf(v);
    }
}

// ---- launchers ----------------------------------------------------------------------
namespace {

template <typename F>
hipError_t allow_lds(F* kernel, size_t bytes) {
    return bytes > 64 * 1024 ? hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes)
                             : hipSuccess;
}

int tiles(int B, int H, int W, int TH, int TW) { return B * ((H + TH - 1) / TH) * ((W + TW - 1) / TW); }

}  // namespace

int64_t packed_elems(int cin, int cout, bool backward) {
    const int rows = backward ? cin : cout, taps = !backward && cin % 16 ? 1 : 9;
    return (int64_t)(taps * pack_ksteps(cin, cout, backward) + 2) * ((rows + 31) / 32) * 512;
}

int pack_ksteps(int cin, int cout, bool backward) {
    return backward ? std::max(cout, 32) / 16 : (cin % 16 ? 4 : cin / 16);
}

void pack_weights(hipStream_t s, const PackTable& T, int n, const float* params) {
    hipLaunchKernelGGL(pack_weights_kernel, dim3(128, n), dim3(256), 0, s, T, params);
}

// The wavefront arrangement.  A weight fragment read from L2 serves PT pixel
// tiles and a pixel fragment from LDS serves MT channel tiles; PT = 4 where
// the halo tile of 512 (32 channels) or 256 pixels still leaves two workgroups
// per CU, else PT = 2 with the channel tiles spread over wavefronts so that the
// staged pixels are shared.
hipError_t conv_forward(hipStream_t s, const ConvSrc& S, int src, int cin, int cout, int act, const u16* Wp,
                        const float* bias, float* Z, u16* A, u16* pool, float* out) {
    const int n = (cout + 31) / 32;
    const bool narrow = S.W <= 16;
    int wp, wc, MT = 1, PT = 2;
    if (n == 1) {
        wp = 4;
        wc = 1;
        if (src != SRC_FIRST && cin <= 32) PT = 4;
    } else if (n == 2) {
        wp = 2;
        wc = 2;
        if (cin <= 64) PT = 4;
    } else if (n == 3) {
        wp = 2;
        wc = 3;
    } else {
        wp = 2;
        wc = 2;
        MT = 2;
    }
    const int TW = narrow ? 16 : 32, TH = wp * PT * (32 / TW);
    const size_t bytes = src == SRC_FIRST ? ((size_t)TH * TW * 72 + (size_t)(TH + 2) * (TW + 2) * 7) * 2
                                           : (size_t)(TH + 2) * (TW + 2) * (cin + 8) * 2;
    const dim3 g(tiles(S.B, S.H, S.W, TH, TW)), blk(64 * wp * wc);
    hipError_t e = hipErrorInvalidValue;
#define FWD(MT_, PT_, SRC_)                                                                                          \
    if (MT == MT_ && PT == PT_ && src == SRC_) {                                                                     \
        auto* k = narrow ? conv_forward_kernel<MT_, PT_, 4, SRC_> : conv_forward_kernel<MT_, PT_, 5, SRC_>;          \
        if ((e = allow_lds(k, bytes)) == hipSuccess) {                                                               \
            hipLaunchKernelGGL(k, g, blk, bytes, s, S, cin, cout, act, wc, Wp, bias, Z, A, pool, out);               \
            e = hipGetLastError();                                                                                   \
        }                                                                                                            \
    }
    FWD(1, 2, SRC_FIRST)
    FWD(1, 4, SRC_PLAIN)
    FWD(1, 2, SRC_PLAIN)
    FWD(2, 2, SRC_PLAIN)
    FWD(1, 2, SRC_CAT)
    FWD(2, 2, SRC_CAT)
#undef FWD
    return e;
}

// Rows of bias-gradient partials that conv_input_grad writes for a source of this size.
namespace {
void grad_shape(int cin, int W, int* wp, int* wc, int* MT, int* TW, int* TH) {
    const int n = cin / 32;
    *MT = n >= 4 && n % 4 == 0 ? 2 : 1;
    *wc = n == 1 ? 1 : (n == 2 || n % 4 == 0 ? 2 : (n <= 6 ? 3 : 4));
    *wp = n == 1 ? 4 : 2;
    *TW = W <= 16 ? 16 : 32;
    *TH = *wp * 2 * (32 / *TW);
}
}  // namespace

int64_t grad_rows(int cin, int B, int H, int W) {
    int wp, wc, MT, TW, TH;
    grad_shape(cin, W, &wp, &wc, &MT, &TW, &TH);
    return (int64_t)tiles(B, H, W, TH, TW) * wp;
}

hipError_t conv_input_grad(hipStream_t s, const ConvSrc& S, int src, int cz, int cin, const u16* Wp, const GradDst& D) {
    int wp, wc, MT, TW, TH;
    grad_shape(cin, S.W, &wp, &wc, &MT, &TW, &TH);
    const int czp = std::max(cz, 32);
    const size_t bytes = (size_t)(TH + 2) * (TW + 2) * (czp + 8) * 2;
    const int per = wc * MT;
    const dim3 g(tiles(S.B, S.H, S.W, TH, TW), (cin / 32 + per - 1) / per), blk(64 * wp * wc);
    hipError_t e = hipErrorInvalidValue;
#define BWD(MT_, SRC_)                                                                                               \
    if (MT == MT_ && src == SRC_) {                                                                                  \
        auto* k = TW == 16 ? conv_input_grad_kernel<MT_, 2, 4, SRC_> : conv_input_grad_kernel<MT_, 2, 5, SRC_>;      \
        if ((e = allow_lds(k, bytes)) == hipSuccess) {                                                               \
            hipLaunchKernelGGL(k, g, blk, bytes, s, S, czp, cin, wc, Wp, D);                                         \
            e = hipGetLastError();                                                                                   \
        }                                                                                                            \
    }
    BWD(1, SRC_PLAIN)
    BWD(2, SRC_PLAIN)
    BWD(1, SRC_HEAD)
#undef BWD
    return e;
}

hipError_t conv_weight_grad(hipStream_t s, const ConvSrc& X, int srcx, const ConvSrc& Gz, int srcz, int cin, int cout,
                            float* part, int64_t part_elems, float* dW) {
    const int K = 9 * cin, nci = srcx == SRC_FIRST ? 2 : cin / 32, nco = (cout + 31) / 32;
    const int ntiles = tiles(X.B, X.H, X.W, WG_TH, WG_TW);
    // about two workgroups per CU over all channel blocks, each with a whole number of tiles
    int splits = std::max(1, std::min(ntiles, 512 / (nci * nco)));
    splits = (int)std::min<int64_t>(splits, std::max<int64_t>(1, part_elems / ((int64_t)K * cout)));
    const int per = (ntiles + splits - 1) / splits;
    splits = (ntiles + per - 1) / per;
    const dim3 g(nci * nco, splits), blk(256);
#define WGR(SX, SZ)                                                                                                   \
    if (srcx == SX && srcz == SZ)                                                                                     \
        hipLaunchKernelGGL((conv_weight_grad_kernel<SX, SZ>), g, blk, 0, s, X, Gz, K, cout, nci, ntiles, per, part);
    WGR(SRC_FIRST, SRC_PLAIN)
    WGR(SRC_PLAIN, SRC_PLAIN)
    WGR(SRC_CAT, SRC_PLAIN)
    WGR(SRC_PLAIN, SRC_HEAD)
#undef WGR
    const int64_t n = (int64_t)K * cout;
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part, splits, n, dW);
    return hipGetLastError();
}

void bias_grads(hipStream_t s, const BiasGrads& T, int n, float* part) {
    hipLaunchKernelGGL(bias_grad_rows_kernel, dim3(kBiasChunks, n), dim3(256), 0, s, T, part);
    hipLaunchKernelGGL(bias_grad_sum_kernel, dim3(n), dim3(128), 0, s, T, part);
}

}  // namespace nn
}  // namespace elwh
