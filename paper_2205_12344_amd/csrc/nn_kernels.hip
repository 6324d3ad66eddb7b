// Loss and Adam kernels of the warm-start network (FP32).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "nn_internal.h"

namespace elwh {
namespace nn {

// Relative error in the weighted norm, per sample b, C = 2 components:
//   L = (1/B) sum_b sum w (yh - y)^2 / sum w y^2 ;  dyh = (2/B) w (yh - y) / den_b
// The sums: one workgroup per sample, each thread adding every 256th value in
// order.  That serial chain bounds it, so 16 values' loads are in flight at a
// time (the gradient, which needs no sum, has its own launch over the chip;
// 380 us for 16 samples of 256^2 with one load at a time and both in one kernel).
__global__ __launch_bounds__(256) void loss_sums_kernel(const float* __restrict__ yh, const float* __restrict__ y,
                                                        const float* __restrict__ w, int B, int64_t npix_per,
                                                        float* __restrict__ loss_per, float* __restrict__ den_per) {
    const int b = blockIdx.x;
    __shared__ float sn[256], sd[256];
    float num = 0.f, den = 0.f;
    const int64_t n = npix_per * 2;
    const float* yb = y + (int64_t)b * n;
    const float* yhb = yh + (int64_t)b * n;
    const float* wb = w + (int64_t)b * npix_per;
    constexpr int U = 16;
    int64_t e = threadIdx.x;
    for (; e + (U - 1) * 256 < n; e += U * 256) {
        float wv[U], yv[U], hv[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            wv[k] = wb[(e + k * 256) / 2];
            yv[k] = yb[e + k * 256];
            hv[k] = yhb[e + k * 256];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const float ww = wv[k], d = hv[k] - yv[k];
            num += ww * d * d;
            den += ww * yv[k] * yv[k];
        }
    }
    for (; e < n; e += 256) {
        const float ww = wb[e / 2], d = yhb[e] - yb[e];
        num += ww * d * d;
        den += ww * yb[e] * yb[e];
    }
    sn[threadIdx.x] = num;
    sd[threadIdx.x] = den;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sn[threadIdx.x] += sn[threadIdx.x + s];
            sd[threadIdx.x] += sd[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float D = sd[0] > 0.f ? sd[0] : 1.f;
        loss_per[b] = sn[0] / D / B;
        den_per[b] = D;
    }
}

// The output gradient and, per workgroup, its sum over pixels (the output
// layer's bias gradient).
__global__ __launch_bounds__(256) void loss_grad_kernel(const float* __restrict__ yh, const float* __restrict__ y,
                                                        const float* __restrict__ w, const float* __restrict__ den_per,
                                                        int B, int64_t npix_per, int64_t npix, float* __restrict__ dyh,
                                                        float* __restrict__ dbpart) {
    __shared__ float s0[256], s1[256];
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float d[2] = {0.f, 0.f};
    if (p < npix) {
        const float D = den_per[p / npix_per];
        for (int c = 0; c < 2; ++c) {
            const int64_t e = 2 * p + c;
            d[c] = 2.f / B * w[p] * (yh[e] - y[e]) / D;
            dyh[e] = d[c];
        }
    }
    s0[threadIdx.x] = d[0];
    s1[threadIdx.x] = d[1];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            s0[threadIdx.x] += s0[threadIdx.x + s];
            s1[threadIdx.x] += s1[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        dbpart[2 * blockIdx.x] = s0[0];
        dbpart[2 * blockIdx.x + 1] = s1[0];
    }
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const float gg = g[e];
        const float mm = b1 * m[e] + (1.f - b1) * gg;
        const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
        m[e] = mm;
        v[e] = vv;
        p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    }
}

// ---- launchers ----------------------------------------------------------------
int64_t loss_blocks(int64_t npix) { return (npix + 255) / 256; }

void loss(hipStream_t s, const float* yh, const float* y, const float* w, int B, int64_t npix_per, float* dyh,
          float* loss_per, float* sums, float* dbpart) {
    hipLaunchKernelGGL(loss_sums_kernel, dim3(B), dim3(256), 0, s, yh, y, w, B, npix_per, loss_per, sums);
    if (dyh)
        hipLaunchKernelGGL(loss_grad_kernel, dim3((unsigned)loss_blocks(B * npix_per)), dim3(256), 0, s, yh, y, w, sums,
                           B, npix_per, B * npix_per, dyh, dbpart);
}

void adam(hipStream_t s, float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
          float eps, int step) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    const int64_t g1 = (n + 255) / 256;
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)(g1 > 65536 ? 65536 : g1)), dim3(256), 0, s, p, g, m, v, n, lr, b1,
                       b2, eps, c1, c2);
}

}  // namespace nn
}  // namespace elwh
