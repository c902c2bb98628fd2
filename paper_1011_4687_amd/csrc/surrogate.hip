// gfx950 kernels of the coordinate-MLP surrogate of V(r) inside the QM region.
//
// Network: gamma(r) = [cos 2 pi B r, sin 2 pi B r] (BF16) -> 4 x (Linear 128 x 128
// in BF16 on the matrix cores with FP32 accumulation, bias, SiLU, BF16) ->
// Linear 128 -> 1 in FP32; V_hat = poly(r/R) + sigma * y.  Training: MSE,
// straight-through BF16 rounding, Adam on FP32 master weights.
//
// Inference is one kernel; a training step is three: k_train (features,
// forward and backward chain of every row), k_weight_grads (partials of
// dW = dZ^T H) and k_reduce_grads (their sums in a fixed order).  Products run on
// v_mfma_f32_32x32x16_bf16.  Operand layout of the instruction (verified on
// the device): lane l, g = l / 32, r = l % 32 holds A[r][g*8 .. g*8+7] and
// Bt[r][g*8 .. g*8+7]; result register i holds C[(i/4)*8 + g*4 + i%4][r].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "surrogate_internal.h"

namespace envpot {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

constexpr double kTwoPi = 6.283185307179586476925286766559;

__device__ __forceinline__ uint16_t to_bf16(float x) {  // round to nearest even
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Adam on the FP32 master weights.  The step number comes from the device
// training state (so one captured step graph serves every step): step =
// st->step + 1, learning rate by cosine decay from lr0 to lr1 over `total`
// steps, bias corrections 1 - b^step.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int64_t n,
                                              const TrainState* __restrict__ st, double lr0, double lr1,
                                              int64_t total, float b1, float b2, float eps) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t step = st->step + 1;
    const double frac = fmin(1.0, (double)(step - st->step0) / (double)(total > 0 ? total : 1));
    const float lr = (float)(lr1 + 0.5 * (lr0 - lr1) * (1.0 + cos(3.14159265358979323846 * frac)));
    const float bc1 = (float)(1.0 - pow((double)b1, (double)step));
    const float bc2 = (float)(1.0 - pow((double)b2, (double)step));
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// End of a training step: advance the device step counter.
__global__ void k_advance(TrainState* st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) st->step += 1;
}

// BF16 copies of the four hidden weight matrices, as stored (out x in) and transposed.
__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ params, uint16_t* __restrict__ W,
                                              uint16_t* __restrict__ WT) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)kLayers * kHidden * kHidden) return;
    const int l = (int)(idx / (kHidden * kHidden));
    const int e = (int)(idx % (kHidden * kHidden));
    const int o = e / kHidden, i = e % kHidden;
    const uint16_t b = to_bf16(params[(int64_t)l * kLayerStride + e]);
    W[idx] = b;
    WT[(int64_t)l * kHidden * kHidden + i * kHidden + o] = b;
}

constexpr int kLdsLd = kHidden + 8;     // padded LDS rows (bank spread of the 16-byte row reads)

// num / den of den >= 1 (or NaN): the quotient of v_rcp_f32 (1 ulp), corrected
// by its exact remainder, is rounded correctly but for the quotients within
// 2^-22 of a tie; v_div_fixup handles infinities and NaN.
__device__ __forceinline__ float div_ge1(float num, float den) {
    const float y = __builtin_amdgcn_rcpf(den);
    const float q = num * y;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-den, q, num), y, q), den, num);
}

__device__ __forceinline__ float silu(float z) { return div_ge1(z, 1.0f + __expf(-z)); }

__device__ __forceinline__ float dsilu(float z) {
    const float s = div_ge1(1.0f, 1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// cos and sin of 2 pi t in FP64: t modulo 1 is exact, then to the nearest
// quarter; on |u| <= 1/8 the Taylor polynomials of cos 2 pi u and sin 2 pi u
// (next terms below 3e-18).  No large-argument path: the general sincos of
// 64 phases took 40 % of an inference.
__device__ __forceinline__ void sincos_turns(double t, float& sn, float& cs) {
    t -= __builtin_rint(t);
    const double q = __builtin_rint(4.0 * t);
    const double u = __builtin_fma(-0.25, q, t), w = u * u;
    double s = -0.7181223017785006;                       // -(2 pi)^15 / 15!
    s = __builtin_fma(s, w, 3.819952584848282);
    s = __builtin_fma(s, w, -15.09464257682299);
    s = __builtin_fma(s, w, 42.058693944897655);
    s = __builtin_fma(s, w, -76.70585975306139);
    s = __builtin_fma(s, w, 81.60524927607506);
    s = __builtin_fma(s, w, -41.34170224039976);
    s = __builtin_fma(s, w, 6.283185307179586);
    s *= u;
    double c = 0.28200596845579123;                          // (2 pi)^16 / 16!
    c = __builtin_fma(c, w, -1.714390711088672);
    c = __builtin_fma(c, w, 7.903536371318469);
    c = __builtin_fma(c, w, -26.4262567833744);
    c = __builtin_fma(c, w, 60.24464137187666);
    c = __builtin_fma(c, w, -85.45681720669373);
    c = __builtin_fma(c, w, 64.9393940226683);
    c = __builtin_fma(c, w, -19.739208802178716);
    c = __builtin_fma(c, w, 1.0);
    // a quarter turn swaps the two, the signs follow
    const int k = (int)q;
    const float fs = (float)s, fc = (float)c;
    sn = (k & 1) ? fc : fs;
    cs = (k & 1) ? fs : fc;
    if (k & 2) sn = -sn;
    if ((k + 1) & 2) cs = -cs;
}

// Two floats to BF16 (nearest even).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float bf16_low(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16_high(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// poly(r/R): the coefficients (LDS) in nested order (x, y, z exponents
// descending, zero above the baseline's degree).  The empty asm makes the
// loads of one power of x wait for the value of the one before: all 165 at
// once took the registers of the weights.
__device__ __forceinline__ double baseline(double x, double y, double z, const double* coef, double inv_r) {
    const double ux = x * inv_r, uy = y * inv_r, uz = z * inv_r;
    double v = 0.0;
    int k = 0;
#pragma unroll
    for (int a = kMaxPolyDegree; a >= 0; --a) {
        int at = k;
        asm volatile("" : "+v"(at), "+v"(v));
        const double* c0 = coef + at;
        double va = 0.0;
#pragma unroll
        for (int b = kMaxPolyDegree - a; b >= 0; --b) {
            double vb = 0.0;
#pragma unroll
            for (int c = kMaxPolyDegree - a - b; c >= 0; --c) {
                vb = __builtin_fma(vb, uz, *c0++);
                ++k;
            }
            va = __builtin_fma(va, uy, vb);
        }
        v = __builtin_fma(v, ux, va);
    }
    return v;
}

// ---------------------------------------------------------- the network
//
// A workgroup of four waves takes tiles of 32 rows; wave w owns the outputs
// 32 w .. 32 w + 31 of every layer and keeps its rows of the four weight
// matrices in registers for all its tiles (128 registers), so a layer reads
// only activations: each wave multiplies its weights by the tile's rows
// (C[output][row], 8 instructions of K = 16), adds the bias, applies SiLU and
// writes four consecutive outputs of a row at a time back to LDS, where two
// buffers alternate.  The vector unit bounds it (SiLU's exponential and
// division, the FP64 features), not the matrix cores.

struct NetShared {
    float bias[kLayers][kHidden];
    float w_out[kHidden + 4];        // the output layer's weights, then its bias
    double B[3 * kFreq];
};

__device__ __forceinline__ void stage_net(NetShared& sh, const double* __restrict__ B,
                                          const float* __restrict__ params) {
    for (int k = threadIdx.x; k < kLayers * kHidden; k += 256)
        sh.bias[k / kHidden][k % kHidden] = params[(int64_t)(k / kHidden) * kLayerStride + kHidden * kHidden +
                                                   k % kHidden];
    for (int k = threadIdx.x; k <= kHidden; k += 256) sh.w_out[k] = params[kOutOffset + k];
    for (int k = threadIdx.x; k < 3 * kFreq; k += 256) sh.B[k] = B[k];
}

// The shared data as a loop should read it anew: hoisted out of the loop over
// tiles, its 200 words spilled the weights.
__device__ __forceinline__ const NetShared& reread(const NetShared& sh) {
    int zero = 0;
    asm volatile("" : "+v"(zero));
    return *reinterpret_cast<const NetShared*>(reinterpret_cast<const char*>(&sh) + zero);
}

// Rows 32 w .. + 31 of a 128 x 128 BF16 matrix as operands.
__device__ __forceinline__ void load_rows(const uint16_t* __restrict__ W, int wave, int r, int g, bf16x8 (&a)[8]) {
    const uint16_t* p = W + (wave * 32 + r) * kHidden + g * 8;
#pragma unroll
    for (int s = 0; s < 8; ++s) a[s] = *reinterpret_cast<const bf16x8*>(p + 16 * s);
}

// Features of one row: frequencies 16 w + 8 g .. + 7, two at a time (more at
// once cost the registers of the weights), packed cosines and sines to
// put(frequency, cosines, sines).
template <typename Put>
__device__ __forceinline__ void features(const NetShared& sh, double x, double y, double z, int wave, int g, Put put) {
    const int f0 = 16 * wave + 8 * g;
#pragma unroll 1
    for (int f = f0; f < f0 + 8; f += 2) {
        float cv[2], sv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double* b = sh.B + 3 * (f + h);
            sincos_turns(b[0] * x + b[1] * y + b[2] * z, sv[h], cv[h]);
        }
        put(f, pack_bf16(cv[0], cv[1]), pack_bf16(sv[0], sv[1]));
    }
}

// a (32 outputs x 128) times the rows of h (32 x 128, padded): register i is
// output 32 w + out_of(i, g) of row r.
__device__ __forceinline__ f32x16 multiply(const bf16x8 (&a)[8], const uint16_t* h, int r, int g) {
    f32x16 acc = {};
    const uint16_t* p = h + r * kLdsLd + g * 8;
#pragma unroll
    for (int s = 0; s < 8; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], *reinterpret_cast<const bf16x8*>(p + 16 * s), acc, 0, 0, 0);
    return acc;
}
__device__ __forceinline__ int out_of(int i, int g) { return (i >> 2) * 8 + g * 4 + (i & 3); }

// Four consecutive outputs of row r per group q, packed, to LDS.
__device__ __forceinline__ void put_rows(uint16_t* h, const uint32_t (&p)[8], int wave, int r, int g) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint2*>(h + r * kLdsLd + wave * 32 + 8 * q + 4 * g) = make_uint2(p[2 * q], p[2 * q + 1]);
}

// Pre-activations of layer l, and its packed activations.
__device__ __forceinline__ void activate(const f32x16& acc, const float* bias, int wave, int g, float (&z)[16],
                                         uint32_t (&p)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4*>(bias + wave * 32 + 8 * q + 4 * g);
        z[4 * q] = acc[4 * q] + b.x;
        z[4 * q + 1] = acc[4 * q + 1] + b.y;
        z[4 * q + 2] = acc[4 * q + 2] + b.z;
        z[4 * q + 3] = acc[4 * q + 3] + b.w;
        p[2 * q] = pack_bf16(silu(z[4 * q]), silu(z[4 * q + 1]));
        p[2 * q + 1] = pack_bf16(silu(z[4 * q + 2]), silu(z[4 * q + 3]));
    }
}

// Output layer of the row whose top activations are h: one FP32 sum in order.
__device__ __forceinline__ float output_row(const uint16_t* h, const float* w_out) {
    float s = 0.0f;
#pragma unroll 4
    for (int j = 0; j < kHidden; j += 8) {
        const uint4 v = *reinterpret_cast<const uint4*>(h + j);
        const float4 w0 = *reinterpret_cast<const float4*>(w_out + j), w1 = *reinterpret_cast<const float4*>(w_out + j + 4);
        s = __builtin_fmaf(bf16_low(v.x), w0.x, s);
        s = __builtin_fmaf(bf16_high(v.x), w0.y, s);
        s = __builtin_fmaf(bf16_low(v.y), w0.z, s);
        s = __builtin_fmaf(bf16_high(v.y), w0.w, s);
        s = __builtin_fmaf(bf16_low(v.z), w1.x, s);
        s = __builtin_fmaf(bf16_high(v.z), w1.y, s);
        s = __builtin_fmaf(bf16_low(v.w), w1.z, s);
        s = __builtin_fmaf(bf16_high(v.w), w1.w, s);
    }
    return s + w_out[kHidden];
}

// Inference: features, the four layers, the output, the baseline and the
// optional exact part.  RB row blocks of 32 per tile: two where they fill the
// chip, so that two independent products are in flight between barriers.
// 1,000,003 rows 1.19 -> 0.39 ms (its products alone, at the 1.18 PFLOP/s of a
// large one, 0.11); 8192 rows 60 -> 13 us.  Before, a workgroup's four waves
// restaged each layer's weights in LDS for every 128 rows, the features took
// the general FP64 sincos, and the baseline's powers went through scratch.
template <int RB>
__global__ __launch_bounds__(256, 2) void k_infer(const double* __restrict__ pts, int64_t n,
                                                  const double* __restrict__ B, const uint16_t* __restrict__ W,
                                                  const float* __restrict__ params, const double* __restrict__ coef,
                                                  double inv_r, double sigma, const double* __restrict__ add,
                                                  double* __restrict__ out) {
    constexpr int kRows = 32 * RB;
    __shared__ NetShared net;
    __shared__ __attribute__((aligned(16))) uint16_t H[3][kRows * kLdsLd];   // the third for the top layer
    __shared__ double poly[kPolyCoefs];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 5, r = lane & 31;
    bf16x8 a[kLayers][8];
#pragma unroll
    for (int l = 0; l < kLayers; ++l) load_rows(W + l * kHidden * kHidden, wave, r, g, a[l]);
    stage_net(net, B, params);
    if (threadIdx.x < kPolyCoefs) poly[threadIdx.x] = coef[threadIdx.x];
    const int64_t tiles = (n + kRows - 1) / kRows;
    double x[RB][3];
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int64_t row = min(tile * kRows + 32 * b + r, n - 1);
            for (int d = 0; d < 3; ++d) x[b][d] = pts[3 * row + d];
        }
    };
    fetch(blockIdx.x);
    __syncthreads();
    int turn = 0;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const NetShared& sh = reread(net);
        const int64_t row0 = tile * kRows;
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            uint16_t* h = H[0] + (32 * b + r) * kLdsLd;
            features(sh, x[b][0], x[b][1], x[b][2], wave, g, [&](int f, uint32_t cs, uint32_t sn) {
                *reinterpret_cast<uint32_t*>(h + f) = cs;
                *reinterpret_cast<uint32_t*>(h + f + kFreq) = sn;
            });
        }
        if (tile + gridDim.x < tiles) fetch(tile + gridDim.x);
        __syncthreads();
#pragma unroll
        for (int l = 0; l < kLayers; ++l) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                float z[16];
                uint32_t p[8];
                activate(multiply(a[l], H[l & 1] + 32 * b * kLdsLd, r, g), sh.bias[l], wave, g, z, p);
                put_rows(H[l + 1 < kLayers ? (l + 1) & 1 : 2] + 32 * b * kLdsLd, p, wave, r, g);
            }
            __syncthreads();
        }
        // one wave finishes the tile, in turn, while the others go on
        if (wave == turn && lane < kRows && row0 + lane < n) {
            const int64_t row = row0 + lane;
            const float y = output_row(H[2] + lane * kLdsLd, sh.w_out);
            const double v = baseline(pts[3 * row], pts[3 * row + 1], pts[3 * row + 2], poly, inv_r) +
                             sigma * (double)y;
            out[row] = add ? v + add[row] : v;
        }
        turn = (turn + 1) & 3;
    }
}

// Sum over the 32 rows (lanes r) of 16 values: after each exchange a lane
// keeps half of them; the even lane of a pair ends with the sum of value
// keep = bits 4..1 of the lane.
__device__ __forceinline__ float sum_rows(float (&v)[16], int lane) {
#pragma unroll
    for (int w = 16, c = 8; c >= 1; w >>= 1, c >>= 1) {
        const bool up = lane & w;
#pragma unroll
        for (int i = 0; i < c; ++i) {
            const float send = up ? v[i] : v[i + c], keep = up ? v[i + c] : v[i];
            v[i] = keep + __shfl_xor(send, w);
        }
    }
    return v[0] + __shfl_xor(v[0], 1);
}

// One row of a transposed activation: chunks of kChunkRows rows, [output][row].
__device__ __forceinline__ void put_transposed(uint16_t* t, const uint32_t (&p)[8], int64_t row, int wave, int g) {
    uint16_t* o = t + (row / kChunkRows) * (kHidden * kChunkRows) + row % kChunkRows;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        uint16_t* c = o + (wave * 32 + out_of(2 * q, g)) * kChunkRows;
        c[0] = (uint16_t)(p[q] & 0xffffu);
        c[kChunkRows] = (uint16_t)(p[q] >> 16);
    }
}

// Copies of a training step's intermediate tensors, row-major (each or null).
struct TraceOut {
    uint16_t* H[kLayers + 1];
    float* Z[kLayers];
    float* dH[kLayers];
    uint16_t* dZ[kLayers];
    float* y;
    float* dy;
};

__device__ __forceinline__ void trace_bf16(uint16_t* t, const uint32_t (&p)[8], int64_t row, int wave, int g) {
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint2*>(t + row * kHidden + wave * 32 + 8 * q + 4 * g) = make_uint2(p[2 * q], p[2 * q + 1]);
}
__device__ __forceinline__ void trace_f32(float* t, const float (&v)[16], int64_t row, int wave, int g) {
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(t + row * kHidden + wave * 32 + 8 * q + 4 * g) =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

// Forward and backward pass of a training step over tiles of 32 rows, all but
// the weight gradients: features and layers as in k_infer with the
// pre-activations kept in registers, the loss, then per layer dZ = dH
// silu'(Z) (dH = dy w_out for the top one), its column sums (bias gradient; for
// the top layer those of dy H_4 as well) and dH of the layer below = dZ W on
// the matrix cores.  Every row's chain stays in its workgroup, so H and dZ
// leave it once, transposed for k_weight_grads.  8192 rows are one tile per
// compute unit: bound by one tile's chain of eight layers (a kernel per
// layer with 128 rows per workgroup left three quarters of the chip idle and
// passed Z and dH through memory: 65 + 120 us of kernels and 12 reductions,
// now 37 + 11 + 7).
__global__ __launch_bounds__(256, 1) void k_train(const double* __restrict__ pts, const float* __restrict__ target,
                                                  int64_t n, int64_t Np, const double* __restrict__ B,
                                                  const uint16_t* __restrict__ W, const uint16_t* __restrict__ WT,
                                                  const float* __restrict__ params, TrainBuffers tb, TraceOut tr) {
    __shared__ NetShared net;
    __shared__ __attribute__((aligned(16))) uint16_t H[2][32 * kLdsLd];
    __shared__ float dys[32];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 5, r = lane & 31;
    const int64_t tiles = Np / 32;
    const int64_t act = tb.act_stride;   // of one layer's transposed activations
    stage_net(net, B, params);
    __syncthreads();
    // which column the even lanes hold after sum_rows
    const int col = wave * 32 + out_of((lane >> 1) & 15, g);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const NetShared& sh = reread(net);
        // operands of the seven products (layers up, then transposed down), each
        // loaded while the one before is at work
        int zero = 0;
        asm volatile("" : "+s"(zero));
        bf16x8 a[2][8];
        auto load = [&](int l, bool down) {
            load_rows((down ? WT : W) + zero + l * kHidden * kHidden, wave, r, g, a[(l + (down ? 1 : 0)) & 1]);
        };
        load(0, false);
        const int64_t row = tile * 32 + r;
        const bool live = row < n;   // padding rows have zero features
        {
            double x = 0.0, y = 0.0, z = 0.0;
            if (live) {
                x = pts[3 * row];
                y = pts[3 * row + 1];
                z = pts[3 * row + 2];
            }
            uint16_t* ht = tb.HT + (row / kChunkRows) * (kHidden * kChunkRows) + row % kChunkRows;
            features(sh, x, y, z, wave, g, [&](int f, uint32_t cs, uint32_t sn) {
                cs = live ? cs : 0u;
                sn = live ? sn : 0u;
                *reinterpret_cast<uint32_t*>(H[0] + r * kLdsLd + f) = cs;
                *reinterpret_cast<uint32_t*>(H[0] + r * kLdsLd + f + kFreq) = sn;
                ht[f * kChunkRows] = (uint16_t)(cs & 0xffffu);
                ht[(f + 1) * kChunkRows] = (uint16_t)(cs >> 16);
                ht[(f + kFreq) * kChunkRows] = (uint16_t)(sn & 0xffffu);
                ht[(f + kFreq + 1) * kChunkRows] = (uint16_t)(sn >> 16);
                if (tr.H[0]) {
                    *reinterpret_cast<uint32_t*>(tr.H[0] + row * kHidden + f) = cs;
                    *reinterpret_cast<uint32_t*>(tr.H[0] + row * kHidden + f + kFreq) = sn;
                }
            });
        }
        __syncthreads();
        float z[kLayers][16];
        uint32_t p[8];
#pragma unroll
        for (int l = 0; l < kLayers; ++l) {
            if (l + 1 < kLayers) load(l + 1, false);
            else load(kLayers - 1, true);
            activate(multiply(a[l & 1], H[l & 1], r, g), sh.bias[l], wave, g, z[l], p);
            put_rows(H[(l + 1) & 1], p, wave, r, g);
            if (l + 1 < kLayers) put_transposed(tb.HT + (l + 1) * act, p, row, wave, g);
            if (tr.Z[l]) trace_f32(tr.Z[l], z[l], row, wave, g);
            if (tr.H[l + 1]) trace_bf16(tr.H[l + 1], p, row, wave, g);
            __syncthreads();
        }
        if (threadIdx.x < 64) {   // loss and dy, by the first wave (both halves alike)
            const float y = output_row(H[0] + r * kLdsLd, sh.w_out);
            double e2 = 0.0;
            float d = 0.0f;
            if (live) {
                const float e = y - target[row];
                d = 2.0f * e / (float)n;
                e2 = (double)e * (double)e;
            }
            if (g == 0) {
                dys[r] = d;
                if (tr.y) tr.y[row] = y;
                if (tr.dy) tr.dy[row] = d;
            }
#pragma unroll
            for (int w = 16; w > 0; w >>= 1) {
                e2 += __shfl_xor(e2, w);
                d += __shfl_xor(d, w);
            }
            if (lane == 0) {
                tb.loss[tile] = e2;
                tb.dysum[tile] = d;
            }
        }
        __syncthreads();
        const float dy = dys[r];
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = dy * ((i & 1) ? bf16_high(p[i >> 1]) : bf16_low(p[i >> 1]));
        const float so = sum_rows(v, lane);
        if (!(lane & 1)) tb.colout[tile * kHidden + col] = so;
#pragma unroll
        for (int l = kLayers - 1; l >= 0; --l) {
            float dz[16];
            if (l == kLayers - 1) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    dz[i] = dy * sh.w_out[wave * 32 + out_of(i, g)] * dsilu(z[l][i]);
            } else {
                if (l > 0) load(l, true);
                const f32x16 d = multiply(a[l & 1], H[l & 1], r, g);
                if (tr.dH[l]) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = d[i];
                    trace_f32(tr.dH[l], v, row, wave, g);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) dz[i] = d[i] * dsilu(z[l][i]);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) p[q] = pack_bf16(dz[2 * q], dz[2 * q + 1]);
            if (l > 0) put_rows(H[(l - 1) & 1], p, wave, r, g);
            put_transposed(tb.dZT + l * act, p, row, wave, g);
            if (tr.dZ[l]) trace_bf16(tr.dZ[l], p, row, wave, g);
            const float sb = sum_rows(dz, lane);
            if (!(lane & 1)) tb.colsum[(l * tiles + tile) * kHidden + col] = sb;
            __syncthreads();
        }
    }
}

// Partials of dW_l = dZ_l^T H_l over one chunk of rows (FP32 over 128 rows at
// most; k_reduce_grads adds the chunks in FP64), a workgroup per chunk and
// layer, wave w the outputs 32 w .. + 31.  Both operands are read as stored,
// rows contiguous.
__global__ __launch_bounds__(256) void k_weight_grads(int64_t Np, TrainBuffers tb) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 5, r = lane & 31;
    const int64_t chunk = blockIdx.x, l = blockIdx.y, chunks = gridDim.x;
    const int rows = (int)min((int64_t)kChunkRows, Np - chunk * kChunkRows);   // a multiple of 32
    const int64_t at = l * tb.act_stride + chunk * (kHidden * kChunkRows);
    const uint16_t* a = tb.dZT + at + (wave * 32 + r) * kChunkRows + g * 8;
    const uint16_t* b = tb.HT + at + r * kChunkRows + g * 8;
    f32x16 acc[4] = {};
#pragma unroll 4
    for (int k = 0; k < rows; k += 16) {
        const bf16x8 av = *reinterpret_cast<const bf16x8*>(a + k);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                av, *reinterpret_cast<const bf16x8*>(b + t * 32 * kChunkRows + k), acc[t], 0, 0, 0);
    }
    float* gp = tb.gpart + (l * chunks + chunk) * kHidden * kHidden;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) gp[(wave * 32 + out_of(i, g)) * kHidden + t * 32 + r] = acc[t][i];
}

// The gradient from its partials: weights over the chunks, biases and the
// output layer over the tiles, each in FP64 in a fixed order (four groups of
// consecutive partials, then the groups).  Block: 64 parameters.
__global__ __launch_bounds__(256) void k_reduce_grads(int64_t Np, TrainBuffers tb, float* __restrict__ grad) {
    __shared__ double sh[4][64];
    const int jl = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + jl;
    const int64_t tiles = Np / 32, chunks = (Np + kChunkRows - 1) / kChunkRows;
    const float* src = nullptr;
    int64_t P = tiles, stride = kHidden;
    if (j < kOutOffset) {
        const int l = j / kLayerStride, e = j % kLayerStride;
        if (e < kHidden * kHidden) {
            src = tb.gpart + l * chunks * (kHidden * kHidden) + e;
            P = chunks;
            stride = kHidden * kHidden;
        } else {
            src = tb.colsum + l * tiles * kHidden + (e - kHidden * kHidden);
        }
    } else if (j < kOutOffset + kHidden) {
        src = tb.colout + (j - kOutOffset);
    } else if (j < kNParams) {
        src = tb.dysum;
        stride = 1;
    }
    double s = 0.0;
    if (src) {
        const int64_t per = (P + 3) / 4, end = min(P, (g + 1) * per);
#pragma unroll 8
        for (int64_t p = g * per; p < end; ++p) s += src[p * stride];
    }
    sh[g][jl] = s;
    __syncthreads();
    if (g == 0 && j < kNParams) grad[j] = (float)(((sh[0][jl] + sh[1][jl]) + sh[2][jl]) + sh[3][jl]);
}

// Residual targets t = (V - poly(r/R)) / sigma.
__global__ __launch_bounds__(256) void k_residual(const double* __restrict__ pts, const double* __restrict__ V,
                                                  int64_t n, const double* __restrict__ coef, double inv_r,
                                                  double inv_sigma, float* __restrict__ t) {
    __shared__ double poly[kPolyCoefs];
    if (threadIdx.x < kPolyCoefs) poly[threadIdx.x] = coef[threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    t[i] = (float)((V[i] - baseline(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2], poly, inv_r)) * inv_sigma);
}

// SplitMix64 (Steele, Lea, Flood 2014): the counter-based generator of the
// training and gate sample points.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

__device__ __forceinline__ double unif(uint64_t seed, uint64_t ctr) {
    return (double)(splitmix64(seed ^ splitmix64(ctr)) >> 11) * 0x1.0p-53;
}

// n points uniform in the ball of radius R, point i from counters 3i..3i+2.
__global__ __launch_bounds__(256) void k_sample_ball(uint64_t seed, int64_t n, double R, double* __restrict__ pts) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double u0 = unif(seed, 3 * (uint64_t)i), u1 = unif(seed, 3 * (uint64_t)i + 1),
                 u2 = unif(seed, 3 * (uint64_t)i + 2);
    const double r = R * cbrt(u0), ct = 2.0 * u1 - 1.0, st = sqrt(fmax(0.0, 1.0 - ct * ct));
    const double ph = kTwoPi * u2;
    pts[3 * i] = r * st * cos(ph);
    pts[3 * i + 1] = r * st * sin(ph);
    pts[3 * i + 2] = r * ct;
}

// Gate validation points: per voxel v (of the G^3 grid over [-R, R]^3) m
// points uniform in the voxel, pulled radially into the ball when outside it.
__global__ __launch_bounds__(256) void k_sample_voxels(uint64_t seed, int G, int m, double R,
                                                       double* __restrict__ pts) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t nv = (int64_t)G * G * G;
    if (i >= nv * m) return;
    const int64_t v = i / m;
    const int vx = (int)(v % G), vy = (int)((v / G) % G), vz = (int)(v / ((int64_t)G * G));
    const double h = 2.0 * R / G;
    double x = -R + h * (vx + unif(seed, 3 * (uint64_t)i));
    double y = -R + h * (vy + unif(seed, 3 * (uint64_t)i + 1));
    double z = -R + h * (vz + unif(seed, 3 * (uint64_t)i + 2));
    const double rr = sqrt(x * x + y * y + z * z);
    if (rr > R) {
        const double s = R * (1.0 - 1e-12) / rr;
        x *= s;
        y *= s;
        z *= s;
    }
    pts[3 * i] = x;
    pts[3 * i + 1] = y;
    pts[3 * i + 2] = z;
}

// Minibatch of a training step: rows ((step - step0) mod steps_per_epoch)
// * bs .. + bs of the epoch's permutation.
__global__ __launch_bounds__(256) void k_gather(const double* __restrict__ pts, const float* __restrict__ t,
                                                const int32_t* __restrict__ perm, const TrainState* __restrict__ st,
                                                int64_t steps_per_epoch, int64_t bs, double* __restrict__ pb,
                                                float* __restrict__ tb) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= bs) return;
    const int64_t start = ((st->step - st->step0) % steps_per_epoch) * bs;
    const int64_t j = perm[start + i];
    pb[3 * i] = pts[3 * j];
    pb[3 * i + 1] = pts[3 * j + 1];
    pb[3 * i + 2] = pts[3 * j + 2];
    tb[i] = t[j];
}

// Gate: flag[i] = 1 when point i must use the exact kernel (outside the
// ball or in a voxel that failed validation); per-block counts of flags.
__global__ __launch_bounds__(256) void k_gate_flags(const double* __restrict__ pts, int64_t n,
                                                    const uint8_t* __restrict__ pass, int G, double R,
                                                    uint8_t* __restrict__ flag, int32_t* __restrict__ counts) {
    __shared__ int32_t sh[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int f = 0;
    if (i < n) {
        const double x = pts[3 * i], y = pts[3 * i + 1], z = pts[3 * i + 2];
        f = 1;
        if (x * x + y * y + z * z <= R * R) {
            const double h = 2.0 * R / G;
            const int vx = min(G - 1, max(0, (int)floor((x + R) / h)));
            const int vy = min(G - 1, max(0, (int)floor((y + R) / h)));
            const int vz = min(G - 1, max(0, (int)floor((z + R) / h)));
            f = pass[((int64_t)vz * G + vy) * G + vx] ? 0 : 1;
        }
        flag[i] = (uint8_t)f;
    }
    sh[threadIdx.x] = f;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = sh[0];
}

// Exclusive scan of the block counts (one workgroup, sequential chunks).
__global__ __launch_bounds__(256) void k_scan_counts(const int32_t* __restrict__ counts, int nb,
                                                     int64_t* __restrict__ offsets, int64_t* __restrict__ total) {
    __shared__ int64_t sh[256];
    int64_t carry = 0;
    for (int base = 0; base < nb; base += 256) {
        const int i = base + threadIdx.x;
        const int64_t v = i < nb ? counts[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int s = 1; s < 256; s <<= 1) {  // inclusive Hillis-Steele scan
            const int64_t a = threadIdx.x >= s ? sh[threadIdx.x - s] : 0;
            __syncthreads();
            sh[threadIdx.x] += a;
            __syncthreads();
        }
        if (i < nb) offsets[i] = carry + sh[threadIdx.x] - v;
        const int64_t last = sh[255];
        __syncthreads();
        carry += last;
    }
    if (threadIdx.x == 0) *total = carry;
}

// Stable compaction of the flagged points (order of the input kept).
__global__ __launch_bounds__(256) void k_compact(const double* __restrict__ pts, int64_t n,
                                                 const uint8_t* __restrict__ flag,
                                                 const int64_t* __restrict__ offsets,
                                                 int64_t* __restrict__ idx, double* __restrict__ cpts) {
    __shared__ int32_t sh[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int f = (i < n) ? flag[i] : 0;
    sh[threadIdx.x] = f;
    __syncthreads();
    for (int s = 1; s < 256; s <<= 1) {
        const int32_t a = threadIdx.x >= s ? sh[threadIdx.x - s] : 0;
        __syncthreads();
        sh[threadIdx.x] += a;
        __syncthreads();
    }
    if (f) {
        const int64_t o = offsets[blockIdx.x] + sh[threadIdx.x] - 1;
        idx[o] = i;
        cpts[3 * o] = pts[3 * i];
        cpts[3 * o + 1] = pts[3 * i + 1];
        cpts[3 * o + 2] = pts[3 * i + 2];
    }
}

// out[idx[k]] = vals[k] for k < *m (the count is read on the device; the
// grid covers the largest possible count).
__global__ __launch_bounds__(256) void k_scatter(const double* __restrict__ vals, const int64_t* __restrict__ idx,
                                                 const int64_t* __restrict__ m, double* __restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < *m) out[idx[k]] = vals[k];
}

// max |a - b| per voxel (m consecutive samples per voxel), FP64.
__global__ __launch_bounds__(256) void k_voxel_maxerr(const double* __restrict__ a, const double* __restrict__ b,
                                                      int64_t nv, int m, double* __restrict__ err) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= nv) return;
    double e = 0.0;
    for (int k = 0; k < m; ++k) e = fmax(e, fabs(a[v * m + k] - b[v * m + k]));
    err[v] = e;
}

inline int64_t blocks64(int64_t n, int64_t per) { return (n + per - 1) / per; }
inline unsigned blocks(int64_t n, int per = 256) { return (unsigned)blocks64(n, per); }

}  // namespace

#define SG_LAUNCH(k, g, b, st, ...) hipLaunchKernelGGL(k, g, b, 0, static_cast<hipStream_t>(st), __VA_ARGS__)

void sg_adam(float* p, const float* g, float* m, float* v, int64_t n, const TrainState* ts, double lr0,
             double lr1, int64_t total, float b1, float b2, float eps, void* st) {
    SG_LAUNCH(k_adam, dim3(blocks(n)), dim3(256), st, p, g, m, v, n, ts, lr0, lr1, total, b1, b2, eps);
}

void sg_advance(TrainState* ts, void* st) { SG_LAUNCH(k_advance, dim3(1), dim3(64), st, ts); }

void sg_pack(const float* params, uint16_t* W, uint16_t* WT, void* st) {
    SG_LAUNCH(k_pack, dim3(blocks((int64_t)kLayers * kHidden * kHidden)), dim3(256), st, params, W, WT);
}

void sg_infer(const double* pts, int64_t n, const double* B, const uint16_t* W, const float* params,
              const double* coef, double inv_r, double sigma, const double* add, double* out, int cu_count, void* st) {
    if (n <= 0) return;
    const int64_t room = 2 * int64_t(cu_count);   // workgroups resident at once
    if (blocks64(n, 64) >= room)
        SG_LAUNCH(k_infer<2>, dim3((unsigned)std::min(blocks64(n, 64), room)), dim3(256), st, pts, n, B, W, params, coef,
                  inv_r, sigma, add, out);
    else
        SG_LAUNCH(k_infer<1>, dim3((unsigned)std::min(blocks64(n, 32), room)), dim3(256), st, pts, n, B, W, params, coef,
                  inv_r, sigma, add, out);
}

void sg_train(const double* pts, const float* target, int64_t n, int64_t Np, const double* B, const uint16_t* W,
              const uint16_t* WT, const float* params, const TrainBuffers& tb, const TrainTrace& trace, float* grad,
              int cu_count, void* st) {
    if (Np <= 0) return;
    TraceOut tr = {};
    for (int l = 0; l <= kLayers; ++l) tr.H[l] = trace.H ? trace.H + int64_t(l) * Np * kHidden : nullptr;
    for (int l = 0; l < kLayers; ++l) {
        tr.Z[l] = trace.Z ? trace.Z + int64_t(l) * Np * kHidden : nullptr;
        tr.dH[l] = trace.dH ? trace.dH + int64_t(l) * Np * kHidden : nullptr;
        tr.dZ[l] = trace.dZ ? trace.dZ + int64_t(l) * Np * kHidden : nullptr;
    }
    tr.y = trace.y;
    tr.dy = trace.dy;
    SG_LAUNCH(k_train, dim3((unsigned)std::min<int64_t>(Np / 32, cu_count)), dim3(256), st, pts, target, n, Np, B, W, WT,
              params, tb, tr);
    SG_LAUNCH(k_weight_grads, dim3((unsigned)blocks64(Np, kChunkRows), kLayers), dim3(256), st, Np, tb);
    SG_LAUNCH(k_reduce_grads, dim3(blocks(kNParams, 64)), dim3(256), st, Np, tb, grad);
}

void sg_residual(const double* pts, const double* V, int64_t n, const double* coef, double inv_r, double inv_sigma,
                 float* t, void* st) {
    SG_LAUNCH(k_residual, dim3(blocks(n)), dim3(256), st, pts, V, n, coef, inv_r, inv_sigma, t);
}

void sg_sample_ball(uint64_t seed, int64_t n, double R, double* pts, void* st) {
    SG_LAUNCH(k_sample_ball, dim3(blocks(n)), dim3(256), st, seed, n, R, pts);
}

void sg_sample_voxels(uint64_t seed, int G, int m, double R, double* pts, void* st) {
    SG_LAUNCH(k_sample_voxels, dim3(blocks((int64_t)G * G * G * m)), dim3(256), st, seed, G, m, R, pts);
}

void sg_gather(const double* pts, const float* t, const int32_t* perm, const TrainState* ts,
               int64_t steps_per_epoch, int64_t bs, double* pb, float* tb, void* st) {
    SG_LAUNCH(k_gather, dim3(blocks(bs)), dim3(256), st, pts, t, perm, ts, steps_per_epoch, bs, pb, tb);
}

int sg_gate_flags(const double* pts, int64_t n, const uint8_t* pass, int G, double R, uint8_t* flag,
                  int32_t* counts, void* st) {
    SG_LAUNCH(k_gate_flags, dim3(blocks(n)), dim3(256), st, pts, n, pass, G, R, flag, counts);
    return (int)blocks(n);
}

void sg_scan_counts(const int32_t* counts, int nb, int64_t* offsets, int64_t* total, void* st) {
    SG_LAUNCH(k_scan_counts, dim3(1), dim3(256), st, counts, nb, offsets, total);
}

void sg_compact(const double* pts, int64_t n, const uint8_t* flag, const int64_t* offsets, int64_t* idx,
                double* cpts, void* st) {
    SG_LAUNCH(k_compact, dim3(blocks(n)), dim3(256), st, pts, n, flag, offsets, idx, cpts);
}

void sg_scatter(const double* vals, const int64_t* idx, const int64_t* m, int64_t n_max, double* out, void* st) {
    if (n_max <= 0) return;
    SG_LAUNCH(k_scatter, dim3(blocks(n_max)), dim3(256), st, vals, idx, m, out);
}

void sg_voxel_maxerr(const double* a, const double* b, int64_t nv, int m, double* err, void* st) {
    SG_LAUNCH(k_voxel_maxerr, dim3(blocks(nv)), dim3(256), st, a, b, nv, m, err);
}

int sg_last_error() { return hipGetLastError() == hipSuccess ? 0 : -1; }

}  // namespace envpot
