// Internal interface of the surrogate kernels (surrogate.hip) for the host
// driver (surrogate.cpp).  Not part of the C ABI.
#pragma once

#include <cstdint>

namespace envpot {

constexpr int kHidden = 128;                 // width of every hidden layer
constexpr int kLayers = 4;                   // hidden layers
constexpr int kFreq = 64;                    // Fourier frequencies: 2 x 64 = 128 inputs
constexpr int kLayerStride = kHidden * kHidden + kHidden;   // W (out x in) then b
constexpr int kOutOffset = kLayers * kLayerStride;          // w_out (128) then b_out
constexpr int kNParams = kOutOffset + kHidden + 1;          // 66,177
constexpr int kMaxPolyDegree = 8;
constexpr int kPolyCoefs = 165;              // monomials up to that degree
constexpr int kChunkRows = 128;              // rows of one weight-gradient partial

// Device state of a training run: Adam step count so far and its value at
// the start of the run (the minibatch index and the learning-rate schedule
// are derived from them on the device, so one captured step graph is
// replayed for every step).
struct TrainState {
    int64_t step;
    int64_t step0;
};

void sg_adam(float* p, const float* g, float* m, float* v, int64_t n, const TrainState* ts, double lr0,
             double lr1, int64_t total, float b1, float b2, float eps, void* st);
void sg_advance(TrainState* ts, void* st);
void sg_pack(const float* params, uint16_t* W, uint16_t* WT, void* st);
// The whole network at inference (features, four layers, output, baseline,
// optional exact part) in one launch: out[i] = poly + sigma y (+ add[i]).
// coef: kPolyCoefs coefficients in nested order (exponents of x, y, z
// descending from kMaxPolyDegree, zero above the baseline's degree).
void sg_infer(const double* pts, int64_t n, const double* B, const uint16_t* W, const float* params,
              const double* coef, double inv_r, double sigma, const double* add, double* out, int cu_count, void* st);

// Workspace of a training step of Np rows (a multiple of 32).
struct TrainBuffers {
    uint16_t* HT = nullptr;    // H_0..H_3, per chunk of kChunkRows rows [feature][row], BF16
    uint16_t* dZT = nullptr;   // dZ_0..dZ_3, likewise
    int64_t act_stride = 0;    // values from one layer to the next in both
    float* gpart = nullptr;    // dW partials: [layer][chunk][128][128]
    float* colsum = nullptr;   // column sums of dZ: [layer][tile of 32 rows][128]
    float* colout = nullptr;   // column sums of dy H_4: [tile][128]
    double* loss = nullptr;    // squared errors per tile
    float* dysum = nullptr;    // sum of dy per tile
};
// Where the intermediate tensors of a step go as well, each or null
// (row-major, Np rows per layer; dH of the layers below the top).
struct TrainTrace {
    uint16_t* H = nullptr;
    float* Z = nullptr;
    float* dH = nullptr;
    uint16_t* dZ = nullptr;
    float* y = nullptr;
    float* dy = nullptr;
};
// Forward and backward pass of n rows (padded to Np; rows >= n have zero
// features and no gradient): loss partials and the whole gradient.
void sg_train(const double* pts, const float* target, int64_t n, int64_t Np, const double* B, const uint16_t* W,
              const uint16_t* WT, const float* params, const TrainBuffers& tb, const TrainTrace& trace, float* grad,
              int cu_count, void* st);
void sg_residual(const double* pts, const double* V, int64_t n, const double* coef, double inv_r, double inv_sigma,
                 float* t, void* st);
void sg_sample_ball(uint64_t seed, int64_t n, double R, double* pts, void* st);
void sg_sample_voxels(uint64_t seed, int G, int m, double R, double* pts, void* st);
void sg_gather(const double* pts, const float* t, const int32_t* perm, const TrainState* ts,
               int64_t steps_per_epoch, int64_t bs, double* pb, float* tb, void* st);
int sg_gate_flags(const double* pts, int64_t n, const uint8_t* pass, int G, double R, uint8_t* flag,
                  int32_t* counts, void* st);
void sg_scan_counts(const int32_t* counts, int nb, int64_t* offsets, int64_t* total, void* st);
void sg_compact(const double* pts, int64_t n, const uint8_t* flag, const int64_t* offsets, int64_t* idx,
                double* cpts, void* st);
void sg_scatter(const double* vals, const int64_t* idx, const int64_t* m, int64_t n_max, double* out, void* st);
void sg_voxel_maxerr(const double* a, const double* b, int64_t nv, int m, double* err, void* st);
int sg_last_error();

}  // namespace envpot
