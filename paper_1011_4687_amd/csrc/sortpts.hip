// Spatial order of the evaluation points: a Morton (Z-order) key on a
// 0.25-bohr grid, a radix sort of the keys (hipCUB), a gather of the points
// in key order and, after the evaluation, a scatter of the values back to
// the caller's order.  Points that are close in space then share waves, so
// fewer waves meet a pair (or cluster) inside its far-field radius with only
// some of their lanes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include <hipcub/hipcub.hpp>

#include "sort_internal.h"

namespace envpot {
namespace {

constexpr int kSortBlock = 256;
constexpr double kInvCell = 4.0;  // grid cells per bohr

// The 10 low bits of v spread to every third bit.
__device__ __forceinline__ uint32_t spread10(uint32_t v) {
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t cell(double x) {
    double c = floor(x * kInvCell) + 512.0;  // the grid covers +-128 bohr; outside, the key saturates
    c = c < 0.0 ? 0.0 : (c > 1023.0 ? 1023.0 : c);
    return uint32_t(c);
}

__global__ __launch_bounds__(kSortBlock) void k_morton(const double* __restrict__ pts, int64_t n,
                                                       uint32_t* __restrict__ key, uint32_t* __restrict__ idx) {
    const int64_t i = int64_t(blockIdx.x) * kSortBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t x = cell(pts[3 * i]), y = cell(pts[3 * i + 1]), z = cell(pts[3 * i + 2]);
    key[i] = spread10(x) | (spread10(y) << 1) | (spread10(z) << 2);
    idx[i] = uint32_t(i);
}

__global__ __launch_bounds__(kSortBlock) void k_gather(const double* __restrict__ pts,
                                                       const uint32_t* __restrict__ order, int64_t n,
                                                       double* __restrict__ out) {
    const int64_t i = int64_t(blockIdx.x) * kSortBlock + threadIdx.x;
    if (i >= n) return;
    const int64_t j = order[i];
    out[3 * i] = pts[3 * j];
    out[3 * i + 1] = pts[3 * j + 1];
    out[3 * i + 2] = pts[3 * j + 2];
}

__global__ __launch_bounds__(kSortBlock) void k_scatter(const double* __restrict__ v,
                                                        const uint32_t* __restrict__ order, int64_t n,
                                                        double* __restrict__ out) {
    const int64_t i = int64_t(blockIdx.x) * kSortBlock + threadIdx.x;
    if (i >= n) return;
    out[order[i]] = v[i];
}

__global__ __launch_bounds__(kSortBlock) void k_scatter4(const double* __restrict__ v,
                                                         const uint32_t* __restrict__ order, int64_t n,
                                                         double* __restrict__ out) {
    const int64_t i = int64_t(blockIdx.x) * kSortBlock + threadIdx.x;
    if (i >= n) return;
    const int64_t j = order[i];
#pragma unroll
    for (int c = 0; c < 4; ++c) out[4 * j + c] = v[4 * i + c];
}

__global__ __launch_bounds__(kSortBlock) void k_scatter_multi(const ScatterDesc* __restrict__ d) {
    const ScatterDesc q = d[blockIdx.y];
    const int64_t i = int64_t(blockIdx.x) * kSortBlock + threadIdx.x;
    if (i >= q.n) return;
    q.out[q.order[i]] = q.v[i];
}

// Spatial order of up to kOrderSmallMax points by one workgroup: the cells of
// a 32^3 grid over the points (the bounding box of a sample within three
// standard deviations of its mean, so a few far points do not coarsen it) in
// Morton order, points of a cell in the caller's order.  A stable radix sort in LDS,
// 3 bits a pass: every thread counts and moves its own contiguous share.
// Bound by LDS latency: no launch, allocation or library call beside it.
constexpr int kOrderThreads = 1024;
constexpr int kOrderEach = int(kOrderSmallMax / kOrderThreads);
constexpr int kOrderSlots = int(kOrderSmallMax + kOrderSmallMax / 32);  // padded: strided reads meet all banks

__device__ __forceinline__ int slot(int i) { return i + (i >> 5); }

__device__ __forceinline__ uint32_t spread5(uint32_t v) {
    return (v & 1u) | ((v & 2u) << 2) | ((v & 4u) << 4) | ((v & 8u) << 6) | ((v & 16u) << 8);
}

__device__ __forceinline__ void order_small_body(const double* __restrict__ pts, int n, uint32_t base,
                                                 uint32_t* __restrict__ order) {
    __shared__ uint32_t el[kOrderSlots];
    __shared__ uint16_t at[8 * kOrderThreads];
    __shared__ float red[4][13];
    __shared__ uint32_t wsum[16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int each = (n + kOrderThreads - 1) / kOrderThreads;
    const int b = min(n, t * each), e = min(n, b + each);
    // mean, spread and box of up to 256 of the points (finite ones, evenly
    // taken, relative to the first of them; fixed order)
    float st[13];
#pragma unroll
    for (int k = 0; k < 13; ++k) st[k] = k < 6 ? HUGE_VALF : 0.0f;
    auto finite = [](double x, double y, double z) { return fabs(x) < 1e30 && fabs(y) < 1e30 && fabs(z) < 1e30; };
    const double ref[3] = {pts[0], pts[1], pts[2]};
    const bool okref = finite(ref[0], ref[1], ref[2]);
    if (wave < 4) {
        const int i = int(int64_t(t) * n >> 8);
        const double x = pts[3 * i], y = pts[3 * i + 1], z = pts[3 * i + 2];
        if (finite(x, y, z)) {
            const float d[3] = {float(x - (okref ? ref[0] : 0.0)), float(y - (okref ? ref[1] : 0.0)),
                                float(z - (okref ? ref[2] : 0.0))};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                st[k] = d[k];
                st[3 + k] = -d[k];
                st[6 + k] = d[k];
                st[9 + k] = d[k] * d[k];
            }
            st[12] = 1.0f;
        }
#pragma unroll
        for (int k = 0; k < 13; ++k) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float w = __shfl_xor(st[k], o);
                st[k] = k < 6 ? fminf(st[k], w) : st[k] + w;
            }
            if (lane == 0) red[wave][k] = st[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 13; ++k)
        st[k] = k < 6 ? fminf(fminf(red[0][k], red[1][k]), fminf(red[2][k], red[3][k]))
                      : (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    const float cnt = fmaxf(st[12], 1.0f);
    double lo[3];
    float edge = 0.0f;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float m = st[6 + d] / cnt, sd = 3.0f * sqrtf(fmaxf(st[9 + d] / cnt - m * m, 0.0f));
        const float l = fmaxf(st[d], m - sd), h = fminf(-st[3 + d], m + sd);
        lo[d] = (okref ? ref[d] : 0.0) + double(l);
        edge = fmaxf(edge, h - l);
    }
    const double inv = edge > 0.0f && edge < 1e30f ? 32.0 / double(edge) : 0.0;
    for (int i = t; i < n; i += kOrderThreads) {
        const double x[3] = {pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]};
        uint32_t key = 0x7fffu;
        if (finite(x[0], x[1], x[2])) {
            key = 0;
            for (int d = 0; d < 3; ++d) {
                const double c = (x[d] - lo[d]) * inv;
                key |= spread5(c <= 0.0 ? 0u : (c >= 31.0 ? 31u : uint32_t(c))) << d;
            }
        }
        el[slot(i)] = (key << 15) | uint32_t(i);
    }
    uint32_t v[kOrderEach];
    for (int sh = 15; sh < 30; sh += 3) {
        __syncthreads();
        uint64_t c = 0;  // 8 counts of up to 32
#pragma unroll
        for (int k4 = 0; k4 < kOrderEach; k4 += 4)
            if (k4 < each) {  // the same for every thread
#pragma unroll
                for (int k = k4; k < k4 + 4; ++k)
                    if (b + k < e) {
                        v[k] = el[slot(b + k)];
                        c += uint64_t(1) << (8 * ((v[k] >> sh) & 7u));
                    }
            }
#pragma unroll
        for (int d = 0; d < 8; ++d) at[d * kOrderThreads + t] = uint16_t((c >> (8 * d)) & 255u);
        __syncthreads();
        // exclusive prefix over (digit, thread)
        uint32_t x[8], sum = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            x[k] = at[8 * t + k];
            sum += x[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        uint32_t place = inc - sum;
        for (int w = 0; w < wave; ++w) place += wsum[w];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            at[8 * t + k] = uint16_t(place);
            place += x[k];
        }
        __syncthreads();
#pragma unroll
        for (int k4 = 0; k4 < kOrderEach; k4 += 4)
            if (k4 < each) {
#pragma unroll
                for (int k = k4; k < k4 + 4; ++k)
                    if (b + k < e) {
                        const int d = int((v[k] >> sh) & 7u);
                        const uint32_t o = at[d * kOrderThreads + t];
                        at[d * kOrderThreads + t] = uint16_t(o + 1);
                        el[slot(int(o))] = v[k];
                    }
            }
    }
    __syncthreads();
    for (int i = t; i < n; i += kOrderThreads) order[i] = base + (el[slot(i)] & 0x7fffu);
}

// A workgroup per slice; counts outside the range (up to n_host, which the grid
// and the buffer are for) are left alone: their order is not read.
__global__ __launch_bounds__(kOrderThreads) void k_order_small(const double* __restrict__ pts, int64_t n_host,
                                                               const int64_t* __restrict__ n_dev,
                                                               uint32_t* __restrict__ order) {
    const int64_t n = n_dev ? *n_dev : n_host, per = order_slice(n), base = blockIdx.x * per;
    if (n < kOrderMin || n > n_host || base >= n) return;
    order_small_body(pts + 3 * base, int(min(per, n - base)), uint32_t(base), order + base);
}

// One workgroup per instance or slice.
__global__ __launch_bounds__(kOrderThreads) void k_order_multi(const OrderDesc* __restrict__ d) {
    const OrderDesc q = d[blockIdx.x];
    if (q.n > 0 && q.n <= kOrderSmallMax) order_small_body(q.pts, int(q.n), uint32_t(q.base), q.order);
}

unsigned blocks(int64_t n) { return unsigned((n + kSortBlock - 1) / kSortBlock); }

}  // namespace

int sort_order(const double* pts, int64_t n, uint32_t* order, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n <= 0 || n > int64_t(INT32_MAX)) return -1;
    uint32_t *key = nullptr, *key2 = nullptr, *idx = nullptr;
    void* tmp = nullptr;
    size_t tmp_bytes = 0;
    int rc = 0;
    if (hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, key, key2, idx, order, int(n), 0, 30, st) !=
        hipSuccess)
        return -1;
    if (hipMallocAsync(reinterpret_cast<void**>(&key), size_t(n) * 4, st) != hipSuccess) return -1;
    if (hipMallocAsync(reinterpret_cast<void**>(&key2), size_t(n) * 4, st) != hipSuccess) rc = -1;
    if (rc == 0 && hipMallocAsync(reinterpret_cast<void**>(&idx), size_t(n) * 4, st) != hipSuccess) rc = -1;
    if (rc == 0 && hipMallocAsync(&tmp, std::max<size_t>(tmp_bytes, 1), st) != hipSuccess) rc = -1;
    if (rc == 0) {
        hipLaunchKernelGGL(k_morton, dim3(blocks(n)), dim3(kSortBlock), 0, st, pts, n, key, idx);
        if (hipGetLastError() != hipSuccess) rc = -1;
    }
    if (rc == 0 && hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, key, key2, idx, order, int(n), 0, 30, st) !=
                       hipSuccess)
        rc = -1;
    (void)hipFreeAsync(tmp, st);
    (void)hipFreeAsync(idx, st);
    (void)hipFreeAsync(key2, st);
    (void)hipFreeAsync(key, st);
    return rc;
}

int sort_points(const double* pts, int64_t n, double* sorted, uint32_t* order, void* stream) {
    if (sort_order(pts, n, order, stream) != 0) return -1;
    hipLaunchKernelGGL(k_gather, dim3(blocks(n)), dim3(kSortBlock), 0, static_cast<hipStream_t>(stream), pts, order, n,
                       sorted);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int order_points(const double* pts, int64_t n, const int64_t* n_dev, uint32_t* order, void* stream) {
    if (n <= 0 || n > int64_t(UINT32_MAX)) return -1;
    const int64_t slices = (n + order_slice(n) - 1) / order_slice(n);
    hipLaunchKernelGGL(k_order_small, dim3(unsigned(slices)), dim3(kOrderThreads), 0, static_cast<hipStream_t>(stream), pts,
                       n, n_dev, order);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int order_points_multi(const OrderDesc* d, int n_desc, void* stream) {
    if (n_desc <= 0) return 0;
    hipLaunchKernelGGL(k_order_multi, dim3(unsigned(n_desc)), dim3(kOrderThreads), 0, static_cast<hipStream_t>(stream),
                       d);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

bool sort_disabled() {
    const char* ns = std::getenv("ENVPOT_NO_SORT");
    return ns && *ns && std::atoi(ns) != 0;
}

bool tree_orders(int64_t n, void* stream) {
    if (n < kOrderMin || n > int64_t(INT32_MAX) || sort_disabled()) return false;
    return n < kSortMinPoints || !stream_capturing(stream);
}

int tree_order(const double* pts, int64_t n, uint32_t* order, void* stream) {
    return n < kSortMinPoints ? order_points(pts, n, nullptr, order, stream) : sort_order(pts, n, order, stream);
}

bool stream_capturing(void* stream) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (!stream) return false;  // the null stream is never captured here
    if (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &cap) != hipSuccess) return true;
    return cap != hipStreamCaptureStatusNone;
}

int scatter_values(const double* v, const uint32_t* order, int64_t n, double* out, void* stream) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_scatter, dim3(blocks(n)), dim3(kSortBlock), 0, static_cast<hipStream_t>(stream), v, order,
                       n, out);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int scatter_values_multi(const ScatterDesc* d, int n_desc, int64_t max_n, void* stream) {
    if (n_desc <= 0 || max_n <= 0) return 0;
    hipLaunchKernelGGL(k_scatter_multi, dim3(blocks(max_n), unsigned(n_desc)), dim3(kSortBlock), 0,
                       static_cast<hipStream_t>(stream), d);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace envpot

namespace envpot {

int scatter_rows4(const double* v, const uint32_t* order, int64_t n, double* out, void* stream) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_scatter4, dim3(blocks(n)), dim3(kSortBlock), 0, static_cast<hipStream_t>(stream), v,
                       order, n, out);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace envpot
