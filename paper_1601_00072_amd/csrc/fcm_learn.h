// Internal launchers of the learned warm start (fcm_learn.hip); not part of the ABI.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

struct fcm_mlp;

namespace fcm {

// Output width C of a network, and its warm start: BF16 inference of `count`
// normalised histograms and the post-processing into start centroids d_v0
// (count x C doubles; a row of NaN where no valid start exists).  Enqueued on s; returns an FCM_* status.
int mlp_clusters(const fcm_mlp* net);
int mlp_warm(fcm_mlp* net, const float* d_hist, int count, double* d_v0, hipStream_t s);

// The network's BF16 parameters, brought up to date on stream s (for the
// persistent solve's in-kernel inference); *rc receives an FCM_* status.
const uint16_t* mlp_bf16_weights(fcm_mlp* net, hipStream_t s, int* rc);

// Histograms of `count` instances: counts is a workspace of
// count * histogram_copies(count) * 256 words, unused (may be null) unless
// histogram_needs_counts; hist[count][256] receives the normalised
// histograms.  The split follows from the host's copy of the offsets
// (count + 1) and the largest instance; a kHistList also needs `first` (host,
// count + 1 values, written then; unused for one instance) on the device.
int histogram_copies(int count);
enum HistForm : int { kHistRect = 0, kHistList = 1, kHistWaves = 2 };
struct HistSplit {
    int form;
    int blocks;  // kHistRect: of each instance, else in all
};
HistSplit histogram_split(const int64_t* offsets, int count, int64_t max_n, int32_t* first);
hipError_t launch_histogram(const uint8_t* x, const int64_t* d_offsets, const int32_t* d_first, HistSplit sp, int count,
                            uint32_t* counts, float* hist, hipStream_t s);
bool histogram_needs_counts(HistSplit sp);
// the same on counters that are already zero (no memset)
hipError_t launch_histogram_counts(const uint8_t* x, const int64_t* d_offsets, const int32_t* d_first, HistSplit sp,
                                   int count, uint32_t* counts, float* hist, hipStream_t s);
// One training step on `rows` samples (rows of X [.][256] and T [.][C] picked
// by idx, or the first ones if idx is null): loss and gradient at theta, then
// one Adam update (step counts from 1) -- or, with grad set, the gradient
// alone.  Offsets o* of the parameter blocks in the flat vector; activations
// and derivatives hold one row per sample.
struct TrainStep {
    const float *X, *T;
    const int32_t* idx;
    int rows, C;
    int64_t oW1, ob1, oW2, ob2, oW3, ob3;
    float *theta, *m, *v, *grad;
    float *h1, *h2, *d, *dy, *dz2, *dz1;
    float* loss;
    float scale, lr;                 // 1 / (rows C), Adam's step size
    float b1, b2, eps, c1, c2;       // set by the launcher
};
hipError_t launch_train_step(TrainStep a, int step, hipStream_t s);
// BF16 inference copy (output-major rows; see fcm_learn_dev.h) of the flat parameters
hipError_t launch_to_bf16(const float* theta, uint16_t* out, int C, hipStream_t s);
hipError_t launch_mlp_infer(const void* w, bool bf16, const float* X, int count, int C, float* Y, hipStream_t s);
hipError_t launch_mlp_starts(const void* w, const float* X, int count, int C, double* v0, hipStream_t s);

}  // namespace fcm
