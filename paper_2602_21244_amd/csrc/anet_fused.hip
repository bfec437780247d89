// Angle network on the matrix cores with the activations of a batch tile kept
// in LDS from the first layer to the last (sections "Neural Network
// Architecture", "Neural Surrogate Training" and "Runtime Acceleration via
// Neural Table Look-up").
//
// Forward: a workgroup of 8 waves takes 32, 64 or 128 rows.  Layer 0 (two
// inputs) runs on the VALU in FP32; every further layer is D = W H^T with
// v_mfma_f32_32x32x16_bf16, H read from LDS ([row][k], padded rows) and W
// streamed from L2 in fragment order (one coalesced 1 KB load per fragment,
// PF fragments ahead), each wave holding the accumulators of its units for
// every row of the tile, so the layer's output overwrites its input in LDS.
// D = W H^T puts four consecutive units of one row in a lane: bias, SiLU,
// one 16-byte store of the pre-activation and one 8-byte LDS write.
//
// What bounds it: 2^20 rows write 8 GB of pre-activations (1.6 ms at the
// 5.1 TB/s a copy reaches) beside 1.45 TFLOP, and take 2.5 ms (layer by layer
// through the tiled GEMM, which also wrote and read the bf16 activations:
// 7.6 ms); the 512 x 512 table, which keeps nothing, is bound by the matrix
// cores and the epilogues they wait for: 0.44 ms, 0.83 PFLOP/s (1.67 ms).
// A training step at 4 096 rows (forward, backward, Adam): 0.17 ms (0.66 ms).
//
// Backward: the same walk from the output down with W^T fragments; the
// epilogue multiplies by SiLU' of the stored pre-activation and writes delta
// in FP32 and bf16 and h = SiLU(z) in bf16.  One launch over all layers'
// 128 x 128 weight-gradient tiles times a K split forms dW = delta^T h (both
// operands transposed in registers while they are staged), one the column
// sums of the FP32 deltas, and one adds the splits and chunks.  Every sum is
// taken in the order of the tiled GEMM's path, so the gradients are the same
// bit for bit: a training run amplifies a rounding (a bf16 weight that flips)
// to 1e-6 of the next loss.  The walk and the column sums go by slabs of AF_SLAB
// rows, whose FP32 deltas share one buffer: 2^20 rows of the paper's network
// take 17.2 GB instead of 23.2 (18.6 layer by layer) and 14.4 ms instead of
// 14.2 (42 ms).
#include <math.h>

#include "anet_fused.hpp"

namespace dsmc {

typedef __bf16 bf16x8a __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef __bf16 bf16x4a __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef float floatx16a __attribute__((__vector_size__(16 * sizeof(float))));
typedef float floatx4a __attribute__((__vector_size__(4 * sizeof(float))));

constexpr int AF_THREADS = 512;
constexpr int AF_WAVES = 8;
constexpr int AF_PAD = 8;       // bf16 of padding per LDS row

// LDS row stride of a tile whose widest layer has d units.
__host__ __device__ inline int af_ld(int d) { return d + AF_PAD; }

struct AfDev {
    int L;
    int d[AF_MAX_LAYERS + 1];
    int ld;                          // LDS row stride
    const __bf16* W0;                // [d1][2]
    const __bf16* Wl;                // [d_{L-1}]
    const __bf16* wp[AF_MAX_LAYERS]; // fragment order (W or W^T)
    const float* b[AF_MAX_LAYERS];
    float* x;
    float* z[AF_MAX_LAYERS];
    __bf16* h[AF_MAX_LAYERS];
    __bf16* delta[AF_MAX_LAYERS];
    float* dz[AF_MAX_LAYERS];
    int64_t slab0;                   // first row of dz
};

__device__ __forceinline__ float af_sigm(float z)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
__device__ __forceinline__ float af_softplus(float z)
{
    return fmaxf(z, 0.0f) +
           0.69314718055994531f *
               __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * fabsf(z)));
}

// ------------------------------------------------------------------------
// Weights in fragment order.  Fragment (u, ks) of a layer holds, for lane l,
// the 8 elements k = 16 ks + 8 (l / 32) + e of unit 32 u + l % 32; forward:
// unit = output, k = input; backward (trans): unit = input, k = output.
// ------------------------------------------------------------------------
struct AfPack {
    int n;                              // layers packed
    const __bf16* W[AF_MAX_LAYERS];     // [out][in]
    int out[AF_MAX_LAYERS], in[AF_MAX_LAYERS];
    __bf16* dst[AF_MAX_LAYERS];
    int first[AF_MAX_LAYERS + 1];       // first 8-element chunk of each layer
    int trans;
    const float* b[AF_MAX_LAYERS];      // biases copied to aligned memory
    float* bdst[AF_MAX_LAYERS];
    int bn[AF_MAX_LAYERS];
    int nb;
};

__global__ void __launch_bounds__(256)
k_anet_pack(AfPack p)
{
    const int total = p.first[p.n];
    for (int q = blockIdx.x * 256 + threadIdx.x; q < total; q += gridDim.x * 256) {
        int l = 0;
        while (q >= p.first[l + 1]) ++l;
        const int c = q - p.first[l], lane = c & 63, f = c >> 6;
        const int units = p.trans ? p.in[l] : p.out[l], K = p.trans ? p.out[l] : p.in[l];
        const int KS = K >> 4, u = f / KS, ks = f - u * KS;
        const int unit = 32 * u + (lane & 31), k = 16 * ks + 8 * (lane >> 5);
        bf16x8a v;
        if (!p.trans) {
            const __bf16* s = p.W[l] + (int64_t)unit * K + k;
            if ((reinterpret_cast<uintptr_t>(s) & 15) == 0) {
                v = *reinterpret_cast<const bf16x8a*>(s);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = s[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = p.W[l][(int64_t)(k + e) * units + unit];
        }
        *reinterpret_cast<bf16x8a*>(p.dst[l] + (int64_t)c * 8) = v;
    }
    for (int l = blockIdx.x; l < p.nb; l += gridDim.x)
        for (int c = threadIdx.x; c < p.bn[l]; c += 256) p.bdst[l][c] = p.b[l][c];
}

// acc[u][r] += W(units of tile u0 + u) H(rows of block rb0 + r)^T over K.
// Fragments are loaded PF k steps ahead (K is a multiple of 16 PF).
template <int NU, int NR, int PF>
__device__ __forceinline__ void af_gemm(const __bf16* __restrict__ wp, int KS, int u0, int rb0,
                                        const __bf16* hs, int ld, floatx16a (&acc)[NU][NR])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[u][r][q] = 0.0f;
    const __bf16* w[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) w[u] = wp + ((int64_t)(u0 + u) * KS * 64 + lane) * 8;
    const __bf16* hb = hs + (rb0 * 32 + (lane & 31)) * ld + 8 * (lane >> 5);
    bf16x8a wr[PF][NU];
#pragma unroll
    for (int p = 0; p < PF; ++p)
#pragma unroll
        for (int u = 0; u < NU; ++u) wr[p][u] = *reinterpret_cast<const bf16x8a*>(w[u] + p * 512);
    for (int k0 = 0; k0 < KS; k0 += PF) {
        const bool more = k0 + PF < KS;
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            bf16x8a hf[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r)
                hf[r] = *reinterpret_cast<const bf16x8a*>(hb + r * 32 * ld + (k0 + p) * 16);
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    acc[u][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[p][u], hf[r], acc[u][r],
                                                                        0, 0, 0);
            if (more)
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    wr[p][u] = *reinterpret_cast<const bf16x8a*>(w[u] + (int64_t)(k0 + PF + p) * 512);
        }
    }
}

// Pre-activations are kept in the order the accumulators hold them: blocks of
// 32 rows x 32 units, in a block element (row, unit 8 q + 4 half + i) at
// (q 64 + 32 half + row) 4 + i, so a wave's 16-byte accesses are one 1 KB
// run.  A row-major layout took twice the time to write (32-byte pieces of 32
// rows per store: 2^20 rows in 4.9 ms against 2.5 ms).
__device__ __forceinline__ int64_t af_zoff(int64_t row0, int rb, int N, int u, int q)
{
    return (((row0 >> 5) + rb) * (N >> 5) + u) * 1024 + q * 256 + (threadIdx.x & 63) * 4;
}

// Epilogue of a forward layer: bias, pre-activation out, SiLU to LDS.
template <int NU, int NR>
__device__ __forceinline__ void af_store_fwd(const floatx16a (&acc)[NU][NR], int u0, int rb0,
                                             const float* __restrict__ bias, float* __restrict__ z,
                                             int N, int64_t row0, int64_t R, __bf16* hs, int ld)
{
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int unit = (u0 + u) * 32 + 8 * q + 4 * half;
            const floatx4a b = *reinterpret_cast<const floatx4a*>(bias + unit);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int row = (rb0 + r) * 32 + col;
                floatx4a v;
                bf16x4a o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[u][r][4 * q + i] + b[i];
                    o[i] = (__bf16)(v[i] * af_sigm(v[i]));
                }
                if (z && row0 + (rb0 + r) * 32 < R)
                    *reinterpret_cast<floatx4a*>(z + af_zoff(row0, rb0 + r, N, u0 + u, q)) = v;
                *reinterpret_cast<bf16x4a*>(hs + row * ld + unit) = o;
            }
        }
}

// One hidden layer of a tile in place in LDS (all 512 threads).
template <int NU, int NR, int PF>
__device__ __forceinline__ void af_layer_fwd(const AfDev& n, int l, int u0, int rb0, bool active,
                                             bool keep, int64_t row0, int64_t R, __bf16* hs)
{
    floatx16a acc[NU][NR];
    if (active) af_gemm<NU, NR, PF>(n.wp[l], n.d[l] >> 4, u0, rb0, hs, n.ld, acc);
    __syncthreads();
    if (active)
        af_store_fwd<NU, NR>(acc, u0, rb0, n.b[l], keep ? n.z[l] : nullptr, n.d[l + 1], row0, R,
                             hs, n.ld);
    __syncthreads();
}

// Units of a layer over the waves: up to 16 tiles of 32 units, two per wave
// above 8, one at 5 .. 8; at 4 (128 units) two waves share a tile's rows.
template <int RB, int PF>
__device__ __forceinline__ void af_layer_fwd_any(const AfDev& n, int l, bool keep, int64_t row0,
                                                 int64_t R, __bf16* hs)
{
    const int w = threadIdx.x >> 6, nt = n.d[l + 1] >> 5;
    if (nt > 8) {
        af_layer_fwd<2, RB, PF>(n, l, 2 * w, 0, 2 * w < nt, keep, row0, R, hs);
    } else if (nt > 4) {
        af_layer_fwd<1, RB, PF>(n, l, w, 0, w < nt, keep, row0, R, hs);
    } else {
        constexpr int NR = RB > 1 ? RB / 2 : 1;
        af_layer_fwd<1, NR, PF>(n, l, w & 3, (w >> 2) * NR, RB > 1 || w < 4, keep, row0, R, hs);
    }
}

template <int RB, int PF>
__global__ void __launch_bounds__(AF_THREADS)
k_anet_fused_fwd(AfDev n, int64_t R, const float* __restrict__ x, float* __restrict__ y, int keep,
                 AnetGrid grid, int theta)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr int ROWS = 32 * RB;
    __bf16* hs = reinterpret_cast<__bf16*>(smem);
    float* xs = reinterpret_cast<float*>(smem + (size_t)ROWS * n.ld * sizeof(__bf16));
    const int t = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    if (t < ROWS) {
        const int64_t g = row0 + t;
        float x0 = 0.0f, x1 = 0.0f;
        if (g < R) {
            if (grid.n_e > 0) {
                const int64_t i = g / grid.n_b, j = g - i * grid.n_b;
                // normalised ln E of node i: 2 i / (n_e - 1) - 1; b / b_max = j / (n_b - 1)
                x0 = (float)(2.0 * (double)i / (double)(grid.n_e - 1) - 1.0);
                x1 = (float)((double)j / (double)(grid.n_b - 1));
            } else {
                x0 = x[2 * g];
                x1 = x[2 * g + 1];
            }
            if (keep) {
                n.x[2 * g] = x0;
                n.x[2 * g + 1] = x1;
            }
        }
        xs[2 * t] = x0;
        xs[2 * t + 1] = x1;
    }
    __syncthreads();
    const int n1 = n.d[1], frags = n1 >> 3;   // (unit tile, q) pairs of a row block
    for (int f = t >> 6; f < RB * frags; f += AF_WAVES) {
        const int rb = f / frags, u = (f - rb * frags) >> 2, q = f & 3;
        const int row = rb * 32 + (t & 31), unit = u * 32 + 8 * q + 4 * ((t >> 5) & 1);
        const float x0 = xs[2 * row], x1 = xs[2 * row + 1];
        const floatx4a b = *reinterpret_cast<const floatx4a*>(n.b[0] + unit);
        floatx4a v;
        bf16x4a o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float wa = (float)n.W0[2 * (unit + i)], wb = (float)n.W0[2 * (unit + i) + 1];
            v[i] = __builtin_fmaf(wa, x0, wb * x1) + b[i];
            o[i] = (__bf16)(v[i] * af_sigm(v[i]));
        }
        if (keep && row0 + rb * 32 < R)
            *reinterpret_cast<floatx4a*>(n.z[0] + af_zoff(row0, rb, n1, u, q)) = v;
        *reinterpret_cast<bf16x4a*>(hs + row * n.ld + unit) = o;
    }
    __syncthreads();
    for (int l = 1; l < n.L - 1; ++l) af_layer_fwd_any<RB, PF>(n, l, keep != 0, row0, R, hs);
    // output layer: wave r takes row block r; unit 0 of a fragment whose
    // other 31 units are zero
    const int w = t >> 6, lane = t & 63, col = lane & 31, half = lane >> 5;
    if (w < RB) {
        floatx16a acc;
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
        const __bf16* hb = hs + (w * 32 + col) * n.ld + 8 * half;
        for (int k = 0; k < n.d[n.L - 1]; k += 16) {
            bf16x8a wf;
#pragma unroll
            for (int e = 0; e < 8; ++e) wf[e] = col == 0 ? n.Wl[k + 8 * half + e] : (__bf16)0.0f;
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                wf, *reinterpret_cast<const bf16x8a*>(hb + k), acc, 0, 0, 0);
        }
        const int64_t g = row0 + w * 32 + col;
        if (half == 0 && g < R) {
            const float v = acc[0] + n.b[n.L - 1][0];
            if (keep) n.z[n.L - 1][g] = v;
            float o = af_softplus(v);
            if (theta) {
                o = expm1f(o);
                o = o < 0.f ? 0.f : (o > 3.14159265358979f ? 3.14159265358979f : o);
            }
            y[g] = o;
        }
    }
}

// ------------------------------------------------------------------------
// Backward
// ------------------------------------------------------------------------
// Epilogue of dL/dz of layer j (width N): acc * SiLU'(z) in FP32 (blocks, for
// the column sums; zero past the last row), delta and h in bf16.
template <int NU, int NR>
__device__ __forceinline__ void af_store_bwd(const AfDev& n, int j, const floatx16a (&acc)[NU][NR],
                                             int u0, int rb0, int64_t row0, int64_t R, __bf16* hs)
{
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int N = n.d[j + 1];
    const float* __restrict__ z = n.z[j];
    float* __restrict__ dz = n.dz[j];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int row = (rb0 + r) * 32 + col;
            const bool in = row0 + row < R, blk = row0 + (rb0 + r) * 32 < R;
            const int64_t o = (row0 + row) * N + (u0 + u) * 32 + 4 * half;
            floatx4a zz[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                zz[q] = in ? *reinterpret_cast<const floatx4a*>(
                                 z + af_zoff(row0, rb0 + r, N, u0 + u, q))
                           : floatx4a{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4a dv, hv;
                floatx4a d4;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float zi = zz[q][i], sg = af_sigm(zi);
                    const float d = acc[u][r][4 * q + i] * (sg * (1.0f + zi * (1.0f - sg)));
                    dv[i] = (__bf16)d;
                    hv[i] = (__bf16)(zi * sg);
                    d4[i] = in ? d : 0.0f;
                }
                if (blk)
                    *reinterpret_cast<floatx4a*>(
                        dz + af_zoff(row0 - n.slab0, rb0 + r, N, u0 + u, q)) = d4;
                if (in) *reinterpret_cast<bf16x4a*>(n.h[j] + o + 8 * q) = hv;
                if (j > 0) {
                    if (in) *reinterpret_cast<bf16x4a*>(n.delta[j] + o + 8 * q) = dv;
                    *reinterpret_cast<bf16x4a*>(hs + row * n.ld + (u0 + u) * 32 + 8 * q +
                                                4 * half) = dv;
                }
            }
        }
    }
}

template <int NU, int NR, int PF>
__device__ __forceinline__ void af_layer_bwd(const AfDev& n, int j, int u0, int rb0, bool active,
                                             const __bf16* d_out, int64_t row0, int64_t R,
                                             __bf16* hs)
{
    floatx16a acc[NU][NR];
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    if (active) {
        if (d_out) {
            // the output layer's single unit: W_l^T delta is one k step with k = 0
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    bf16x8a wf, df;
#pragma unroll
                    for (int e = 0; e < 8; ++e) wf[e] = df[e] = (__bf16)0.0f;
                    if (half == 0) {
                        wf[0] = n.Wl[(u0 + u) * 32 + col];
                        df[0] = d_out[(rb0 + r) * 32 + col];
                    }
                    floatx16a zero;
#pragma unroll
                    for (int q = 0; q < 16; ++q) zero[q] = 0.0f;
                    acc[u][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, df, zero, 0, 0, 0);
                }
        } else {
            af_gemm<NU, NR, PF>(n.wp[j + 1], n.d[j + 2] >> 4, u0, rb0, hs, n.ld, acc);
        }
    }
    __syncthreads();
    if (active) af_store_bwd<NU, NR>(n, j, acc, u0, rb0, row0, R, hs);
    __syncthreads();
}

template <int RB, int PF>
__global__ void __launch_bounds__(AF_THREADS)
k_anet_fused_bwd(AfDev n, int64_t R, const float* __restrict__ dy)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr int ROWS = 32 * RB;
    __bf16* hs = reinterpret_cast<__bf16*>(smem);
    __bf16* ds = reinterpret_cast<__bf16*>(smem + (size_t)ROWS * n.ld * sizeof(__bf16));
    const int t = threadIdx.x, w = t >> 6;
    const int64_t row0 = n.slab0 + (int64_t)blockIdx.x * ROWS;
    if (t < ROWS) {
        const int64_t g = row0 + t;
        float d = 0.0f;
        if (g < R) {
            d = dy[g] / (1.0f + expf(-n.z[n.L - 1][g]));
            n.dz[n.L - 1][g - n.slab0] = d;
            n.delta[n.L - 1][g] = (__bf16)d;
        }
        ds[t] = (__bf16)d;
    }
    __syncthreads();
    for (int j = n.L - 2; j >= 0; --j) {
        const __bf16* d_out = j == n.L - 2 ? ds : nullptr;
        const int nt = n.d[j + 1] >> 5;
        if (nt > 8) {
            af_layer_bwd<2, RB, PF>(n, j, 2 * w, 0, 2 * w < nt, d_out, row0, R, hs);
        } else if (nt > 4) {
            af_layer_bwd<1, RB, PF>(n, j, w, 0, w < nt, d_out, row0, R, hs);
        } else {
            constexpr int NR = RB > 1 ? RB / 2 : 1;
            af_layer_bwd<1, NR, PF>(n, j, w & 3, (w >> 2) * NR, RB > 1 || w < 4, d_out, row0, R,
                                    hs);
        }
    }
}

// Column sums of dL/dz in the order of the tiled GEMM's path (so a network
// trains the same whichever path its widths take): chunks of 256 rows, in a
// chunk rows w, w + 4, ... of each w < 4 one after the other, the four sums
// added in order.  A wave takes one chunk and 64 units of a layer: lane
// (block, four units, w) reads 16 bytes a row from the FP32 blocks.
struct AfCols {
    int L;
    int d[AF_MAX_LAYERS + 1];
    const float* dz[AF_MAX_LAYERS];
    const float* x;
    int first[AF_MAX_LAYERS + 1];    // first group of 64 units of each hidden layer
    int red_off[AF_MAX_LAYERS];      // first column of layer l's sums in a chunk's row of red
    int red_ld;
    int64_t R, chunks;               // rows and chunks of the slab
    float* red;                      // [chunks][red_ld]
};
constexpr int AC_ROWS = 256;
static_assert(AF_SLAB % AC_ROWS == 0, "whole chunks (and tiles) in a slab");

__global__ void __launch_bounds__(64)
k_anet_cols(AfCols g)
{
    const int lane = threadIdx.x, ph = lane & 3;
    const int groups = g.first[g.L - 1];
    const int64_t job = blockIdx.x;
    if (job >= g.chunks * groups) {
        // the output's single column: 16 chunks per wave
        const int64_t ch = (job - g.chunks * groups) * 16 + (lane >> 2);
        float s = 0.0f;
        if (ch < g.chunks) {
            const int64_t r1 = (ch + 1) * AC_ROWS < g.R ? (ch + 1) * AC_ROWS : g.R;
            const float* dz = g.dz[g.L - 1];
#pragma unroll 8
            for (int64_t r = ch * AC_ROWS + ph; r < r1; r += 4) s += dz[r];
        }
        const int b = lane & ~3;
        const float a0 = __shfl(s, b, 64), a1 = __shfl(s, b + 1, 64), a2 = __shfl(s, b + 2, 64),
                    a3 = __shfl(s, b + 3, 64);
        if (ph == 0 && ch < g.chunks)
            g.red[ch * g.red_ld + g.red_off[g.L - 1]] = ((a0 + a1) + a2) + a3;
        return;
    }
    const int64_t ch = job / groups;
    const int gr = (int)(job - ch * groups);
    int l = 0;
    while (gr >= g.first[l + 1]) ++l;
    const int N = g.d[l + 1], u = 2 * (gr - g.first[l]) + (lane >> 5), qh = (lane >> 2) & 7;
    const float* dz = g.dz[l] + (int64_t)u * 1024 + (qh >> 1) * 256 + (qh & 1) * 128 + ph * 4;
    floatx4a s = {0.f, 0.f, 0.f, 0.f}, s0 = s, s1 = s;
    const int64_t b0 = ch * (AC_ROWS / 32), nb = (g.R + 31) / 32;
    const int64_t b1 = b0 + AC_ROWS / 32 < nb ? b0 + AC_ROWS / 32 : nb;
    for (int64_t b = b0; b < b1; ++b) {
        floatx4a v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = *reinterpret_cast<const floatx4a*>(dz + b * (N >> 5) * 1024 + e * 16);
        if (l == 0) {
            float x0[8], x1[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t r = b * 32 + 4 * e + ph;
                x0[e] = r < g.R ? g.x[2 * r] : 0.0f;
                x1[e] = r < g.R ? g.x[2 * r + 1] : 0.0f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    s0[i] = __builtin_fmaf(v[e][i], x0[e], s0[i]);
                    s1[i] = __builtin_fmaf(v[e][i], x1[e], s1[i]);
                }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += v[e][i];
    }
    // lane ph of the four writes unit ph
    const int base = lane & ~3, unit = u * 32 + 4 * qh + ph;
    auto total = [&](const floatx4a& a) {
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a0 = __shfl(a[i], base, 64), a1 = __shfl(a[i], base + 1, 64);
            const float a2 = __shfl(a[i], base + 2, 64), a3 = __shfl(a[i], base + 3, 64);
            const float q = ((a0 + a1) + a2) + a3;
            t = ph == i ? q : t;
        }
        return t;
    };
    float* o = g.red + ch * g.red_ld + g.red_off[l] + (l == 0 ? 3 * unit : unit);
    o[0] = total(s);
    if (l == 0) {
        o[1] = total(s0);
        o[2] = total(s1);
    }
}

// dW_l = delta_l^T h_{l-1} for all layers l >= 1 at once: 128 x 128 tiles,
// K (the batch) split over AF_SPLITS workgroups, in the tiled GEMM's lengths
// (and so with its results).  Rows are staged 64 at a time, both
// operands transposed in registers (8 rows x 4 units per thread) into
// [unit][k] LDS rows of 128 bytes whose eight 16-byte chunks are permuted by
// (unit ^ unit / 4) & 7, which keeps the writes and the fragment reads free
// of bank conflicts.
constexpr int AD_T = 128, AD_K = 64;

struct AdLayer {
    const __bf16* d;     // [R][M]
    const __bf16* h;     // [R][N]
    int M, N;
    int tiles_n, first;  // tiles of 128 columns; first tile of the layer
    int64_t off;         // first element in a split's partial
};
struct AdArgs {
    int n;
    AdLayer l[AF_MAX_LAYERS];
    int tiles;
    int64_t R, kc, total;
    float* partial;
};

__device__ __forceinline__ int ad_slot(int unit, int chunk)
{
    return unit * AD_K + ((chunk ^ unit ^ (unit >> 2)) & 7) * 8;
}

struct AdRegs {
    bf16x4a v[8];
};

__device__ __forceinline__ void ad_load(const __bf16* __restrict__ p, int ld, int c0,
                                        int64_t k0, int64_t kend, AdRegs& g)
{
    const int c = c0 + (threadIdx.x & 31) * 4;
    const int64_t k = k0 + (threadIdx.x >> 5) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bf16x4a v = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
        if (k + e < kend) {
            if (ld >= 4) {
                if (c < ld) v = *reinterpret_cast<const bf16x4a*>(p + (k + e) * ld + c);
            } else if (c == 0) {
                v[0] = p[k + e];
            }
        }
        g.v[e] = v;
    }
}

__device__ __forceinline__ void ad_store(const AdRegs& g, __bf16* tile)
{
    const int c = (threadIdx.x & 31) * 4, kg = threadIdx.x >> 5;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bf16x8a o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = g.v[e][i];
        *reinterpret_cast<bf16x8a*>(tile + ad_slot(c + i, kg)) = o;
    }
}

__global__ void __launch_bounds__(256)
k_anet_dw(AdArgs g)
{
    __shared__ __attribute__((aligned(16))) __bf16 As[2][AD_T * AD_K];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][AD_T * AD_K];
    const int split = blockIdx.x % AF_SPLITS, tile = blockIdx.x / AF_SPLITS;
    int l = 0;
    while (l + 1 < g.n && tile >= g.l[l + 1].first) ++l;
    const AdLayer& y = g.l[l];
    const int q = tile - y.first;
    const int m0 = (q / y.tiles_n) * AD_T, n0 = (q % y.tiles_n) * AD_T;
    const int64_t kbeg = split * g.kc, kend = kbeg + g.kc < g.R ? kbeg + g.kc : g.R;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
    const int wm = (w >> 1) * 64, wn = (w & 1) * 64;
    floatx16a acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    AdRegs ra, rb;
    if (kbeg < kend) {
        ad_load(y.d, y.M, m0, kbeg, kend, ra);
        ad_load(y.h, y.N, n0, kbeg, kend, rb);
        ad_store(ra, As[0]);
        ad_store(rb, Bs[0]);
    }
    __syncthreads();
    int cur = 0;
    for (int64_t k0 = kbeg; k0 < kend; k0 += AD_K) {
        const bool more = k0 + AD_K < kend;
        if (more) {
            ad_load(y.d, y.M, m0, k0 + AD_K, kend, ra);
            ad_load(y.h, y.N, n0, k0 + AD_K, kend, rb);
        }
#pragma unroll
        for (int ks = 0; ks < AD_K / 16; ++ks) {
            bf16x8a fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fa[i] = *reinterpret_cast<const bf16x8a*>(
                    As[cur] + ad_slot(wm + i * 32 + col, 2 * ks + half));
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fb[i] = *reinterpret_cast<const bf16x8a*>(
                    Bs[cur] + ad_slot(wn + i * 32 + col, 2 * ks + half));
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j],
                                                                        0, 0, 0);
        }
        if (more) {
            ad_store(ra, As[cur ^ 1]);
            ad_store(rb, Bs[cur ^ 1]);
        }
        __syncthreads();
        cur ^= 1;
    }
    float* p = g.partial + (int64_t)split * g.total + y.off;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                const int c = n0 + wn + j * 32 + col;
                if (m < y.M && c < y.N) p[(int64_t)m * y.N + c] = acc[i][j][r];
            }
}

// The weight gradients: the AF_SPLITS partials of an element, sums of every
// fourth one added in order.  The bias and layer-0 gradients: 16 sums of every
// 16th chunk, added in order; 64 columns per workgroup.
struct AfFinal {
    float* dW[AF_MAX_LAYERS];     // layers 1 .. n
    int64_t off[AF_MAX_LAYERS + 1];
    const float* partial;
    int64_t total;
    int wblocks;                  // workgroups of the weight part
    const float* red;
    int red_ld;
    int64_t chunks;
    int red_off[AF_MAX_LAYERS + 1];
    float* db[AF_MAX_LAYERS];
    float* dW0;
};

__global__ void __launch_bounds__(256)
k_anet_final(AfFinal g)
{
    static_assert(AF_SPLITS == 16, "four sums of four partials");
    if ((int)blockIdx.x < g.wblocks) {
        for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < g.total;
             q += (int64_t)g.wblocks * 256) {
            float a[AF_SPLITS], v[4];
#pragma unroll
            for (int s = 0; s < AF_SPLITS; ++s) a[s] = g.partial[s * g.total + q];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                v[w] = 0.0f;
#pragma unroll
                for (int s = w; s < AF_SPLITS; s += 4) v[w] += a[s];
            }
            int l = 0;
            while (q >= g.off[l + 1]) ++l;
            g.dW[l][q - g.off[l]] = ((v[0] + v[1]) + v[2]) + v[3];
        }
        return;
    }
    __shared__ float part[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c = ((int)blockIdx.x - g.wblocks) * 64 + lane;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (c < g.red_ld) {
        const float* p = g.red + c;
        for (int64_t r = 0; r < g.chunks; r += 16)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (r + 4 * w + e < g.chunks) v[e] += p[(r + 4 * w + e) * g.red_ld];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) part[4 * w + e][lane] = v[e];
    __syncthreads();
    if (w == 0 && c < g.red_ld) {
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < 16; ++q) sum += part[q][lane];
        int l = 0;
        while (c >= g.red_off[l + 1]) ++l;
        const int k = c - g.red_off[l];
        if (l > 0) g.db[l][k] = sum;
        else if (k % 3 == 0) g.db[0][k / 3] = sum;
        else g.dW0[2 * (k / 3) + k % 3 - 1] = sum;
    }
}

// ------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------
bool anet_fused_shape(const AnetShape& a)
{
    if (a.L < 2) return false;
    for (int l = 1; l < a.L; ++l)
        if (a.d[l] % 128 != 0 || a.d[l] > 512) return false;
    return true;
}

static int widest(const AnetShape& a)
{
    int m = 0;
    for (int l = 1; l < a.L; ++l) m = a.d[l] > m ? a.d[l] : m;
    return m;
}

// Row blocks (of 32) per workgroup, forward and backward.  Every workgroup
// streams all weights (1.3 MB for the paper's network) from L2, so few rows
// want many small tiles to spread over the CUs (4 096 rows are 128 tiles of
// 32) and many rows want large ones to reuse each fragment; the backward's
// epilogue holds too many values for 128 rows (76 registers spilled).
// Forward with 32, 64 and 128 rows a tile: 8 192 rows 39, 48 and 71 us; 12 288
// 63, 49 and 71; 16 384 66, 51 and 71; 24 576 92, 88 and 76; 32 768 118, 96 and
// 84; 49 152 176, 140 and 150; 65 536 223, 187 and 167 (between 16 384 and
// 65 536 the better of 64 and 128 alternates with how full the last wave is).
// Backward with 32 and 64: 4 096 rows 88 and 108 us, 8 192 119 and 131, 16 384
// 247 and 250, 65 536 908 and 935.
static int fwd_row_blocks(int64_t R) { return R <= 8192 ? 1 : (R <= 32768 ? 2 : 4); }
static int bwd_row_blocks(int64_t R) { return R <= 8192 ? 1 : 2; }

static int64_t tiles_of(int64_t R, int rb) { return (R + 32 * rb - 1) / (32 * rb); }

// Columns of a chunk's row of sums: three per unit of layer 0, one per unit
// of every other layer.
static int red_columns(const AnetShape& a, int* off)
{
    int c = 0;
    for (int l = 0; l < a.L; ++l) {
        if (off) off[l] = c;
        c += l == 0 ? 3 * a.d[1] : a.d[l + 1];
    }
    if (off) off[a.L] = c;
    return c;
}

static int64_t chunks_of(int64_t R) { return (R + AC_ROWS - 1) / AC_ROWS; }

static int64_t weights_of(const AnetShape& a)
{
    int64_t n = 0;
    for (int l = 1; l < a.L; ++l) n += (int64_t)a.d[l] * a.d[l + 1];
    return n;
}

AnetFusedWs anet_fused_layout(void* base, const AnetShape& a, int64_t R)
{
    AnetFusedWs w{};
    uint8_t* p = reinterpret_cast<uint8_t*>(align_up(reinterpret_cast<uintptr_t>(base)));
    size_t o = 0;
    auto take = [&](size_t b) { uint8_t* r = base ? p + o : nullptr; o += align_up(b); return r; };
    w.x = reinterpret_cast<float*>(take(sizeof(float) * 2 * (size_t)R));
    for (int l = 0; l < a.L; ++l) {
        const size_t n = (size_t)R * a.d[l + 1], blocks = ((size_t)R + 31) / 32 * 32;
        w.z[l] = reinterpret_cast<float*>(
            take(sizeof(float) * (l < a.L - 1 ? blocks * a.d[l + 1] : n)));
        if (l < a.L - 1) w.h[l] = reinterpret_cast<__bf16*>(take(sizeof(__bf16) * n));
        w.dz[l] = reinterpret_cast<float*>(
            take(sizeof(float) * (blocks < AF_SLAB ? blocks : AF_SLAB) * a.d[l + 1]));
        if (l > 0) w.delta[l] = reinterpret_cast<__bf16*>(take(sizeof(__bf16) * n));
        w.b[l] = reinterpret_cast<float*>(take(sizeof(float) * a.d[l + 1]));
        if (l > 0 && l < a.L - 1)
            w.wp[l] = reinterpret_cast<__bf16*>(take(sizeof(__bf16) * (size_t)a.d[l] * a.d[l + 1]));
    }
    w.red = reinterpret_cast<float*>(
        take(sizeof(float) * (size_t)chunks_of(R) * (size_t)red_columns(a, nullptr)));
    w.partial = reinterpret_cast<float*>(take(sizeof(float) * AF_SPLITS * (size_t)weights_of(a)));
    w.bytes = o;
    return w;
}

static AfDev dev_of(const dsmc_anet* net, const AnetShape& a, const AnetFusedWs& w)
{
    AfDev n{};
    n.L = a.L;
    for (int l = 0; l <= a.L; ++l) n.d[l] = a.d[l];
    n.ld = af_ld(widest(a));
    n.W0 = static_cast<const __bf16*>(net->W[0]);
    n.Wl = static_cast<const __bf16*>(net->W[a.L - 1]);
    n.x = w.x;
    for (int l = 0; l < a.L; ++l) {
        n.wp[l] = w.wp[l];
        n.b[l] = w.b[l];
        n.z[l] = w.z[l];
        n.h[l] = w.h[l];
        n.delta[l] = w.delta[l];
        n.dz[l] = w.dz[l];
    }
    return n;
}

static int pack(const dsmc_anet* net, const AnetShape& a, const AnetFusedWs& w, bool trans,
                hipStream_t s)
{
    AfPack p{};
    p.trans = trans ? 1 : 0;
    int c = 0;
    for (int l = 1; l < a.L - 1; ++l) {
        p.W[p.n] = static_cast<const __bf16*>(net->W[l]);
        p.out[p.n] = a.d[l + 1];
        p.in[p.n] = a.d[l];
        p.dst[p.n] = w.wp[l];
        p.first[p.n++] = c;
        c += a.d[l] * a.d[l + 1] / 8;
    }
    p.first[p.n] = c;
    if (!trans)
        for (int l = 0; l < a.L; ++l) {
            p.b[l] = net->b[l];
            p.bdst[l] = w.b[l];
            p.bn[l] = a.d[l + 1];
            p.nb = l + 1;
        }
    if (!c && !p.nb) return DSMC_OK;
    const int blocks = c > 256 ? (c + 255) / 256 : 1;
    k_anet_pack<<<blocks, 256, 0, s>>>(p);
    DSMC_LAUNCH_CHECK("anet:pack");
    return DSMC_OK;
}

static size_t lds_bytes(const AnetShape& a, int rb)
{
    return (size_t)32 * rb * (af_ld(widest(a)) * sizeof(__bf16) + 2 * sizeof(float) + sizeof(__bf16)) +
           16;
}

template <int RB, int PF>
static int fwd_launch(const AfDev& n, const AnetShape& a, int64_t R, const float* x, float* y,
                      bool keep, const AnetGrid& grid, bool theta, hipStream_t s)
{
    const size_t lds = lds_bytes(a, RB);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_anet_fused_fwd<RB, PF>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_check(e, "anet:fwd LDS");
    k_anet_fused_fwd<RB, PF><<<(unsigned)tiles_of(R, RB), AF_THREADS, lds, s>>>(n, R, x, y,
                                                                           keep ? 1 : 0, grid,
                                                                           theta ? 1 : 0);
    DSMC_LAUNCH_CHECK("anet:fwd");
    return DSMC_OK;
}

// One slab of the walk back: rows n.slab0 .. below R1.
template <int RB, int PF>
static int bwd_launch(const AfDev& n, const AnetShape& a, int64_t R1, const float* dy,
                      hipStream_t s)
{
    const size_t lds = lds_bytes(a, RB);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_anet_fused_bwd<RB, PF>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_check(e, "anet:bwd LDS");
    k_anet_fused_bwd<RB, PF><<<(unsigned)tiles_of(R1 - n.slab0, RB), AF_THREADS, lds, s>>>(n, R1,
                                                                                       dy);
    DSMC_LAUNCH_CHECK("anet:bwd");
    return DSMC_OK;
}

int anet_fused_forward(const dsmc_anet* net, const AnetShape& a, int64_t R, const float* x,
                       float* y, const AnetFusedWs& w, bool keep, const AnetGrid& grid,
                       bool theta, hipStream_t s)
{
    const int rb = fwd_row_blocks(R);
    if (tiles_of(R, rb) > 2147483647) return arg_error("anet: too many rows");
    int rc = pack(net, a, w, false, s);
    if (rc) return rc;
    const AfDev n = dev_of(net, a, w);
    switch (rb) {
    case 1: return fwd_launch<1, 8>(n, a, R, x, y, keep, grid, theta, s);
    case 2: return fwd_launch<2, 8>(n, a, R, x, y, keep, grid, theta, s);
    default: return fwd_launch<4, 4>(n, a, R, x, y, keep, grid, theta, s);
    }
}

int anet_fused_backward(const dsmc_anet* net, const AnetShape& a, int64_t R, const float* dy,
                        float* const* dW, float* const* db, const AnetFusedWs& w,
                        hipStream_t s)
{
    const int rb = bwd_row_blocks(R);
    if (tiles_of(R, rb) > 2147483647) return arg_error("anet: too many rows");
    int rc = pack(net, a, w, true, s);
    if (rc) return rc;

    AdArgs g{};
    AfFinal f{};
    int64_t off = 0;
    for (int l = 1; l < a.L; ++l) {
        AdLayer& y = g.l[g.n];
        y.d = w.delta[l];
        y.h = w.h[l - 1];
        y.M = a.d[l + 1];
        y.N = a.d[l];
        y.tiles_n = (y.N + AD_T - 1) / AD_T;
        y.first = g.tiles;
        y.off = off;
        g.tiles += (y.M + AD_T - 1) / AD_T * y.tiles_n;
        f.dW[g.n] = dW[l];
        f.off[g.n] = off;
        off += (int64_t)y.M * y.N;
        f.off[++g.n] = off;
    }
    g.R = R;
    g.total = off;
    g.kc = ((R + AF_SPLITS - 1) / AF_SPLITS + 31) / 32 * 32;   // trailing splits may be empty
    g.partial = w.partial;

    AfCols q{};
    q.L = a.L;
    for (int l = 0; l <= a.L; ++l) q.d[l] = a.d[l];
    for (int l = 0; l < a.L; ++l) {
        q.dz[l] = w.dz[l];
        if (l + 1 < a.L) q.first[l + 1] = q.first[l] + a.d[l + 1] / 64;
    }
    q.red_ld = red_columns(a, f.red_off);
    for (int l = 0; l < a.L; ++l) q.red_off[l] = f.red_off[l];

    AfDev n = dev_of(net, a, w);
    for (int64_t r0 = 0; r0 < R; r0 += AF_SLAB) {
        const int64_t r1 = r0 + AF_SLAB < R ? r0 + AF_SLAB : R;
        n.slab0 = r0;
        rc = rb == 1 ? bwd_launch<1, 8>(n, a, r1, dy, s) : bwd_launch<2, 8>(n, a, r1, dy, s);
        if (rc) return rc;
        if (r1 == R) {   // (before the sums: delta and h are still in the cache)
            k_anet_dw<<<(unsigned)(g.tiles * AF_SPLITS), 256, 0, s>>>(g);
            DSMC_LAUNCH_CHECK("anet:dw");
        }
        q.x = w.x + 2 * r0;
        q.R = r1 - r0;
        q.chunks = chunks_of(q.R);
        q.red = w.red + r0 / AC_ROWS * q.red_ld;
        const int64_t jobs = q.chunks * q.first[a.L - 1] + (q.chunks + 15) / 16;
        k_anet_cols<<<(unsigned)jobs, 64, 0, s>>>(q);
        DSMC_LAUNCH_CHECK("anet:cols");
    }

    f.partial = w.partial;
    f.total = off;
    int64_t wb = (off + 255) / 256;
    const int pb = persistent_blocks(256);
    f.wblocks = (int)(wb < pb ? wb : pb);
    f.red = w.red;
    f.red_ld = q.red_ld;
    f.chunks = chunks_of(R);
    for (int l = 0; l < a.L; ++l) f.db[l] = db[l];
    f.dW0 = dW[0];
    k_anet_final<<<f.wblocks + (f.red_ld + 63) / 64, 256, 0, s>>>(f);
    DSMC_LAUNCH_CHECK("anet:final");
    return DSMC_OK;
}

}  // namespace dsmc
