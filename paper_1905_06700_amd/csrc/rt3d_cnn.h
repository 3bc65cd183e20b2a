// rt3d_cnn.h -- shapes and buffers of the learned depth denoiser (internal).
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "rt3d_dev.h"

namespace rt3d {

constexpr int CNN_LAYERS = 4;
constexpr double CNN_GATE = 3.0;   // neighbour depth gate of the features, in sigma_h
// master (trained) channel counts and the counts stored for the matrix cores
constexpr int CNN_CIN[CNN_LAYERS] = {16, 32, 32, 32};
constexpr int CNN_COUT[CNN_LAYERS] = {32, 32, 32, 3};
constexpr int CNN_CIS[CNN_LAYERS] = {16, 32, 32, 32};
constexpr int CNN_COS[CNN_LAYERS] = {32, 32, 32, 16};
// offsets of each layer in the flat master vector ([3][3][cin][cout] then bias)
constexpr int CNN_L0 = 9 * 16 * 32 + 32, CNN_L1 = 9 * 32 * 32 + 32;
constexpr int CNN_OFF[CNN_LAYERS] = {0, CNN_L0, CNN_L0 + CNN_L1, CNN_L0 + 2 * CNN_L1};
constexpr int CNN_PARAMS = (9 * 16 * 32 + 32) + 2 * (9 * 32 * 32 + 32) + (9 * 32 * 3 + 3);

struct CnnWeights {
    float* master = nullptr;        // FP32 master weights [CNN_PARAMS]
    float* m = nullptr;             // Adam first moment
    float* v = nullptr;             // Adam second moment
    __half* wt[CNN_LAYERS] = {};    // forward layout [cos][9 * cis]
    __half* wb[CNN_LAYERS] = {};    // backward-data layout [cis][9 * cos] (layers 1, 2), [cis][64] (layer 3)
    float* bias[CNN_LAYERS] = {};   // [cos]
    long long step = 0;
};

// Weight-gradient partial sums of one workgroup: per layer [9 cis][cos], then
// the layers' bias sums [cos].
constexpr int CNN_POFF[CNN_LAYERS] = {0, 9 * 16 * 32, 9 * 16 * 32 + 9 * 32 * 32, 9 * 16 * 32 + 2 * 9 * 32 * 32};
constexpr int CNN_PB0 = 9 * 16 * 32 + 2 * 9 * 32 * 32 + 9 * 32 * 16;
constexpr int CNN_PBIAS[CNN_LAYERS] = {CNN_PB0, CNN_PB0 + 32, CNN_PB0 + 64, CNN_PB0 + 96};
constexpr int CNN_PART = CNN_PB0 + 112;

// Pairs of loss sums a training step keeps (at most, one per workgroup).
constexpr unsigned CNN_LOSS_PARTS = 1024;

struct CnnBuffers {
    __half* act[4] = {};            // features [P][16], three hidden activations [P][32]
    __half* dact[4] = {};           // gradients of the hidden activations [P][32] (1 .. 3)
    __half* dy4 = nullptr;          // output gradient [P][4]
    float* lpart = nullptr;         // loss partials [2 CNN_LOSS_PARTS]
    float* part = nullptr;          // weight-gradient partials [cnn_wgrad_partials(groups)][CNN_PART]
    float* grad = nullptr;          // flat gradient [CNN_PARAMS]
};

struct CnnAdam {
    float lr, beta1, beta2, eps;
};

unsigned cnn_wgrad_groups(const Shape& sh);
unsigned cnn_wgrad_partials(unsigned groups);
hipError_t launch_cnn_prepare(const CnnWeights& w, hipStream_t st);
// The network's output y [3][P] (corrections in sigma_h units).
hipError_t launch_cnn_output(const Shape& sh, DevState s, float sigma_h, const CnnWeights& w, const CnnBuffers& b,
                             float* y, hipStream_t st);
// The same, applied: slot k < 3 of a pixel with at most three points moves by
// sigma_h y_k, clamped to [0, tmax].
hipError_t launch_cnn_apply(const Shape& sh, DevState s, float sigma_h, const CnnWeights& w, const CnnBuffers& b,
                            double tmax, hipStream_t st);
hipError_t launch_cnn_train_step(const Shape& sh, DevState s, float sigma_h, const float* truth, int S,
                                 CnnWeights& w, const CnnBuffers& b, const CnnAdam& opt, float* loss,
                                 hipStream_t st);

}  // namespace rt3d
