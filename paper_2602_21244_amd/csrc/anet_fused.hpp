// Angle network with a batch tile's activations kept in LDS across the
// layers (2 -> hidden widths that are multiples of 128 up to 512 -> 1).
#pragma once
#include "common.hpp"

namespace dsmc {

constexpr int AF_MAX_LAYERS = DSMC_ANET_MAX_LAYERS;
// Rows of FP32 deltas held at a time (2 GB for the paper's network).  The
// kernels of a slab drain before the next one starts: with 32 768 rows the
// backward of 262 144 takes 3.82 ms, as one slab 3.56 ms.
constexpr int64_t AF_SLAB = 1 << 18;
constexpr int AF_SPLITS = 16;   // K splits of the weight-gradient kernel (those of the tiled GEMM's)

struct AnetShape {
    int L;                        // weight layers
    int d[AF_MAX_LAYERS + 1];     // widths, d[0] = 2, d[L] = 1
};

// Whether the kernels of this file take the network's widths.
bool anet_fused_shape(const AnetShape& a);

// Workspace pieces (offsets from a 256-byte aligned base).
struct AnetFusedWs {
    float* x;                     // inputs [R][2]
    float* z[AF_MAX_LAYERS];      // pre-activations of hidden layers (blocks of 32 x 32), output [R]
    __bf16* h[AF_MAX_LAYERS];     // hidden activations [R][d_{l+1}] (backward)
    float* dz[AF_MAX_LAYERS];     // dL/dz_l in FP32 of one slab, laid out as z (backward)
    __bf16* delta[AF_MAX_LAYERS]; // dL/dz_l [R][d_{l+1}], l >= 1 (backward)
    __bf16* wp[AF_MAX_LAYERS];    // weights in fragment order (layers 1 .. L-2)
    float* b[AF_MAX_LAYERS];      // biases, aligned copies
    float* red;                   // per-chunk sums of the bias and layer-0 gradients
    float* partial;               // [splits][weights of layers 1 .. L-1]
    size_t bytes;
};
AnetFusedWs anet_fused_layout(void* base, const AnetShape& a, int64_t R);

struct AnetGrid {                 // rows are nodes of a table grid (n_e = 0: rows are x)
    int32_t n_e, n_b;
};

// Forward.  keep: write the pre-activations (and the inputs) for a backward;
// theta: y is clip(exp(y) - 1, 0, pi) instead of the network's output.
int anet_fused_forward(const dsmc_anet* net, const AnetShape& a, int64_t R, const float* x,
                       float* y, const AnetFusedWs& w, bool keep, const AnetGrid& grid,
                       bool theta, hipStream_t s);
int anet_fused_backward(const dsmc_anet* net, const AnetShape& a, int64_t R, const float* dy,
                        float* const* dW, float* const* db, const AnetFusedWs& w,
                        hipStream_t s);

}  // namespace dsmc
