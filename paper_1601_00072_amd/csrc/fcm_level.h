// Level solve (Algorithm 1 over the grey levels): what the host runtime and
// the kernels of fcm_levels.hip share (not part of the ABI).
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

#include "fcm_internal.h"

namespace fcm {

constexpr int kLvBlock = 512;   // threads per block: two blocks of 64 KB of counters per CU
constexpr int kLvCopies = 16;   // copies of the global counters (blocks spread their atomics)

struct LevelArgs {
    const uint8_t* x;
    int64_t n, head, nbody;
    DevState* st;
    DevState* host;          // pinned copy of the state's result fields, for the host to read after a wait;
                             // its ticket becomes `seq` once the others are written
    uint32_t* counts;        // [kLvCopies][256] counters, zero at entry and at the end of every launch
    double* hist_v;
    double* hist_d;
    double* hist_J;
    double eps, m;
    int32_t max_iter;
    int32_t do_init;         // compute the data range and v^0 first
    int32_t given;           // start mode: 0 evenly spaced, 1 v0 below, 2 dv0 (device), 3 learned (mlp_w)
    int32_t max_passes;      // passes this launch may run
    int32_t fp32_range;      // report starts whose FP32 distances overflow as non-finite
    uint32_t seq;
    double v0[kMaxC];
    const double* dv0;
    const uint16_t* mlp_w;
};

// Batched level solve: one block per tile of an instance.
struct LevelBatchArgs {
    const uint8_t* x;
    const BatchInst* inst;
    const BatchTile* tiles;  // in launch order
    const int32_t* ntiles;   // [I] tiles of the instance
    const double* m;         // [I] fuzziness
    uint32_t* counts;        // [I][256] counters, zero at entry and at the end of every launch
    uint32_t* ticket;        // [I] tiles counted, zero at entry and at the end of every launch
    BatchRec* recs;
    BatchRec* host_recs;     // pinned: the same records, for the host to read after a wait
    uint64_t* host_start;    // pinned: wall clock at the start of the launch
    double* hist;
};
hipError_t launch_levels_batch(const LevelBatchArgs& a, int grid, hipStream_t s);

hipError_t launch_levels(const LevelArgs& a, int C, int mclass, int grid, hipStream_t s);

}  // namespace fcm
