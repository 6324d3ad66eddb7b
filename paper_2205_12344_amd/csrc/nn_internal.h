// Internal launchers of the warm-start network kernels (nn_conv.hip: the
// convolutions; nn_kernels.hip: loss and Adam).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace elwh {
namespace nn {

// Input of a convolution: BF16 x0 with c0 channels; for a concatenated input
// x0 is the low-level tensor (half the size, c0 channels) and x1 the skip (c1
// channels); f is the FP32 network input (7 channels) or output gradient (2).
// H, W: size of the convolution's output.
struct ConvSrc {
    const unsigned short* x0 = nullptr;
    const unsigned short* x1 = nullptr;
    const float* f = nullptr;
    int c0 = 0, c1 = 0;
    int B = 0, H = 0, W = 0;
};
enum { SRC_PLAIN = 0, SRC_CAT = 1, SRC_FIRST = 2, SRC_HEAD = 3 };

// Where the gradient of a convolution's input goes: through the SiLU (Z) of
// the layer that produced it into dZ (BF16) and the bias partials; for a
// concatenated input its channels below cup go there summed over 2x2 pixels
// and the others to dskip (FP32); for a pooled input dskip is added first.
enum { GRAD_PLAIN = 0, GRAD_CAT = 1, GRAD_UNPOOL = 2 };
struct GradDst {
    int mode = GRAD_PLAIN, cup = 0;
    const float* Z = nullptr;
    unsigned short* dZ = nullptr;
    float* dskip = nullptr;
    float* dbpart = nullptr;
};

// Bias-gradient partials of every layer: rows x C sums each.
constexpr int kBiasChunks = 32, kLayersMax = 19;
struct BiasGrads {
    struct Layer {
        const float* in;
        float* out;
        long long rows;
        int C;
    } l[kLayersMax];
};

// Packed BF16 weights: steps of 16 contracted channels per tap, elements (two
// spare steps at the end: the kernels load two steps ahead), and one launch
// that packs n layers from the FP32 parameters.
struct PackTable {
    struct Layer {
        unsigned short* out;
        long long woff;
        int cin, cout, ks;
    } l[kLayersMax];
    int backward;
};
int pack_ksteps(int cin, int cout, bool backward);
int64_t packed_elems(int cin, int cout, bool backward);
void pack_weights(hipStream_t s, const PackTable& T, int n, const float* params);
hipError_t conv_forward(hipStream_t s, const ConvSrc& S, int src, int cin, int cout, int act, const unsigned short* Wp,
                        const float* bias, float* Z, unsigned short* A, unsigned short* pool, float* out);
int64_t grad_rows(int cin, int B, int H, int W);
hipError_t conv_input_grad(hipStream_t s, const ConvSrc& S, int src, int cz, int cin, const unsigned short* Wp,
                           const GradDst& D);
hipError_t conv_weight_grad(hipStream_t s, const ConvSrc& X, int srcx, const ConvSrc& Gz, int srcz, int cin, int cout,
                            float* part, int64_t part_elems, float* dW);
void bias_grads(hipStream_t s, const BiasGrads& T, int n, float* part);

// loss_per[b] and, with dyh non-null, the output gradient and its per-block
// channel sums dbpart[loss_blocks(B npix)][2]; sums: 2 B floats of scratch
int64_t loss_blocks(int64_t npix);
void loss(hipStream_t s, const float* yh, const float* y, const float* w, int B, int64_t npix_per, float* dyh,
          float* loss_per, float* sums, float* dbpart);
void adam(hipStream_t s, float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
          float eps, int step);

}  // namespace nn
}  // namespace elwh
