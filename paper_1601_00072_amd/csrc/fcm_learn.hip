// Learned warm start: grey-level histograms, and the histogram -> centroid
// network (256 -> 128 ReLU -> 64 ReLU -> C) trained and run by these kernels.
//
// Parameters live in one flat FP32 vector: W1 [256][128], b1, W2 [128][64], b2,
// W3 [64][C], b3 (row-major [in][out]).  Training: FP32 forward/backward on
// minibatches, mean squared error on the centroids divided by 255, Adam.
// Inference: BF16 weights and activations (round to nearest even), FP32
// accumulation, one block per histogram.  All reductions run in a fixed order
// (no floating-point atomics), so training is reproducible run to run.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "fcm.h"
#include "fcm_host.h"
#include "fcm_internal.h"
#include "fcm_learn.h"
#include "fcm_learn_dev.h"
#include "fcm_level_dev.h"

namespace fcm {

// ---------------------------------------------------------------------------
// histogram of each instance (integer counts, then normalised to sum 1)
// ---------------------------------------------------------------------------

// A block counts its share of an instance with one counter column per lane
// (level_count; 4 tables shared by all lanes of a wave serialised on busy
// levels: 1,024 slices of 256x256 took 63 us with
// the normalisation, 23 us so).  A single block per
// instance writes the normalised histogram itself; more blocks
// add into copy x % copies of the instance's counters ([count][copies][256],
// zero at entry; the copies spread the adds to a busy level).  Block (x, y) of
// a rectangular grid takes share x of instance y; block x of a list (LIST)
// belongs to the instance whose blocks first[i] .. first[i + 1] contain x.
template <bool LIST>
__global__ __launch_bounds__(kLvBlock) void hist_count_kernel(const uint8_t* x, const int64_t* offsets,
                                                              const int32_t* first, int count, uint32_t* counts,
                                                              float* hist, int copies) {
    __shared__ __align__(16) uint32_t tab[256 * 64];
    const int tid = threadIdx.x;
    int inst = blockIdx.y, share = blockIdx.x, shares = gridDim.x;
    if constexpr (LIST) {
        const int b = blockIdx.x, lane = tid & 63;
        int lo = 0, hi = count;  // first[lo] <= b < first[hi]; 64 places looked at together
        while (hi - lo > 1) {
            const int step = (hi - lo + 63) / 64, i = lo + lane * step;
            const uint64_t below = __ballot(i < hi && first[i < hi ? i : lo] <= b);  // a run of lanes from lane 0
            lo += (__popcll(below) - 1) * step;
            hi = lo + step < hi ? lo + step : hi;
        }
        inst = lo;
        share = b - first[inst];
        shares = first[inst + 1] - first[inst];
    }
    level_clear(tab);  // while the offsets are on their way
    const int64_t b0 = offsets[inst], n = offsets[inst + 1] - b0;
    const uint8_t* xi = x + b0;
    const int64_t lead = (int64_t)((16 - ((uintptr_t)xi & 15)) & 15);
    const int64_t head = n < lead ? n : lead;
    const int64_t nbody = (n - head) / 16;
    if (share && (int64_t)share * kLvBlock >= nbody) return;  // a smaller instance than the grid's largest
    __syncthreads();
    char* t8 = reinterpret_cast<char*>(tab);
    level_count(t8, reinterpret_cast<const uint4*>(xi + head), (int64_t)share * kLvBlock + tid, nbody,
                (int64_t)shares * kLvBlock);
    if (share == 0) level_ragged(t8, xi, n, head, nbody);
    __syncthreads();
    const uint32_t c = level_total(tab);
    if (tid >= 256) return;
    if (!LIST && shares == 1)
        hist[(int64_t)inst * 256 + tid] = hist_norm(c, n);
    else if (c)
        atomicAdd(counts + ((int64_t)inst * copies + share % copies) * 256 + tid, c);
}

// Small instances: one wave each, with a table of its own.  Clearing and
// adding up 64 columns takes a block 2.4 us whatever it counts, and two blocks
// fill a CU; for few voxels the adds that serialise on a busy level cost less
// (65,536 instances of 64 voxels: 302 us a block each, 36 a wave each; 10,000
// of 1,024, half of them on one level: 50 and 25; 4,096 of 4,096: 24 and 33).
constexpr int64_t kHistWaveVoxels = 1024;

__global__ __launch_bounds__(512) void hist_waves_kernel(const uint8_t* x, const int64_t* offsets, int count,
                                                         float* hist) {
    __shared__ uint32_t tabs[8][256];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t inst = (int64_t)blockIdx.x * 8 + wid;
    if (inst >= count) return;  // waves share nothing: no barrier below
    uint32_t* tab = tabs[wid];
#pragma unroll
    for (int j = 0; j < 4; ++j) tab[64 * j + lane] = 0u;
    const int64_t b0 = offsets[inst], n = offsets[inst + 1] - b0;
    const uint8_t* xi = x + b0;
    const int64_t lead = (int64_t)((16 - ((uintptr_t)xi & 15)) & 15);
    const int64_t head = n < lead ? n : lead;
    const int64_t nbody = (n - head) / 16, tail0 = head + 16 * nbody, nr = head + (n - tail0);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint4* body = reinterpret_cast<const uint4*>(xi + head);
    for (int64_t c = lane; c < nbody; c += 64) {
        const uint4 w = body[c];
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < 4; ++b) atomicAdd(tab + ((words[q] >> (8 * b)) & 0xFFu), 1u);
    }
    if (lane < nr) atomicAdd(tab + xi[lane < head ? lane : tail0 + (lane - head)], 1u);  // nr < 32
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t c = tab[64 * j + lane];
        hist[inst * 256 + 64 * j + lane] = hist_norm(c, n);
    }
}

// totals of the copies, as count / n (FP64, stored FP32)
__global__ __launch_bounds__(kBlock) void hist_norm_kernel(const uint32_t* counts, const int64_t* offsets, float* hist,
                                                           int copies) {
    const int inst = blockIdx.x;
    const uint32_t* ci = counts + (int64_t)inst * copies * 256;
    uint32_t total = 0u;
    for (int c = 0; c < copies; ++c) total += ci[c * 256 + threadIdx.x];
    hist[(int64_t)inst * 256 + threadIdx.x] = hist_norm(total, offsets[inst + 1] - offsets[inst]);
}

int histogram_copies(int count) { return count == 1 ? kHistCopies : 1; }

// How the instances are dealt to blocks.  A block's share is between 16,384
// (below that a block's clearing and totals outweigh its count) and 131,072
// voxels, such that the launch gives every CU two blocks; a single instance
// takes at most one per CU (the reads of two are no faster).  Equal numbers of
// blocks for every instance (kHistRect) unless that would launch more than
// twice the blocks that the instances need, most of them without a share
// (one volume of 67M voxels and 512 slices of 256x256: the call took
// 940 us, 92 as a list of blocks; with 5,000 slices of 64x64: 8,420 and 354):
// then kHistList.  More small instances than fit at once: a wave each (kHistWaves).
HistSplit histogram_split(const int64_t* offsets, int count, int64_t max_n, int32_t* first) {
    static constexpr int64_t kCus = 256, kMin = 16384, kMax = 131072;
    auto clamped = [](int64_t v) { return std::min(std::max(v, kMin), kMax); };
    auto blocks = [](int64_t n, int64_t share) { return std::min<int64_t>((n + share - 1) / share, 4096); };
    if (count >= 2 * kCus && max_n <= kHistWaveVoxels) return {kHistWaves, (count + 7) / 8};
    if (count == 1) return {kHistRect, (int)std::min(blocks(max_n, std::max(kMin, max_n / (2 * kCus))), kCus)};
    const int64_t gx = blocks(max_n, clamped(max_n * count / (2 * kCus)));
    if (gx <= 2) return {kHistRect, (int)gx};
    const int64_t share = clamped(offsets[count] / (2 * kCus));
    int64_t need = 0;
    for (int i = 0; i < count; ++i) need += blocks(offsets[i + 1] - offsets[i], share);
    if (gx * count <= 2 * need) return {kHistRect, (int)gx};
    first[0] = 0;
    for (int i = 0; i < count; ++i) first[i + 1] = first[i] + (int32_t)blocks(offsets[i + 1] - offsets[i], share);
    return {kHistList, (int)need};
}

bool histogram_needs_counts(HistSplit sp) { return sp.form == kHistList || (sp.form == kHistRect && sp.blocks > 1); }

// counting and normalisation on counters that are already zero (where that is needed)
hipError_t launch_histogram_counts(const uint8_t* x, const int64_t* d_offsets, const int32_t* d_first, HistSplit sp,
                                   int count, uint32_t* counts, float* hist, hipStream_t s) {
    const int copies = histogram_copies(count);
    hipError_t e;
    if (sp.form == kHistWaves) {
        hipLaunchKernelGGL(hist_waves_kernel, dim3(sp.blocks), dim3(512), 0, s, x, d_offsets, count, hist);
        return hipGetLastError();
    }
    if (sp.form == kHistList) {
        hipLaunchKernelGGL(hist_count_kernel<true>, dim3(sp.blocks), dim3(kLvBlock), 0, s, x, d_offsets, d_first, count,
                           counts, hist, copies);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        constexpr int kMaxY = 65535;  // grid y limit: instances per launch
        for (int c0 = 0; c0 < count; c0 += kMaxY) {
            const int cnt = count - c0 < kMaxY ? count - c0 : kMaxY;
            hipLaunchKernelGGL(hist_count_kernel<false>, dim3(sp.blocks, cnt), dim3(kLvBlock), 0, s, x, d_offsets + c0,
                               static_cast<const int32_t*>(nullptr), cnt, counts + (int64_t)c0 * copies * 256,
                               hist + (int64_t)c0 * 256, copies);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (sp.blocks == 1) return hipSuccess;
    }
    hipLaunchKernelGGL(hist_norm_kernel, dim3(count), dim3(256), 0, s, counts, d_offsets, hist, copies);
    return hipGetLastError();
}

hipError_t launch_histogram(const uint8_t* x, const int64_t* d_offsets, const int32_t* d_first, HistSplit sp, int count,
                            uint32_t* counts, float* hist, hipStream_t s) {
    if (histogram_needs_counts(sp)) {
        const int64_t words = 256 * (int64_t)count * histogram_copies(count);
        hipError_t e = hipMemsetAsync(counts, 0, sizeof(uint32_t) * (size_t)words, s);
        if (e != hipSuccess) return e;
    }
    return launch_histogram_counts(x, d_offsets, d_first, sp, count, counts, hist, s);
}

// ---------------------------------------------------------------------------
// training step in two launches
// ---------------------------------------------------------------------------
//
// A step is 63 MFLOP at the usual 256 rows: launches, and inside them the
// latency of reading what another XCD has just written (about 1 us), bound
// it, not arithmetic (one kernel per product, bias, loss and update took 14
// launches and 100 us per step).  So each block issues all its reads at once,
// as 16-byte loads into registers, and multiplies the wide operand there: a
// thread holds four columns of every 8th (128 columns) or 16th row, the
// narrow operand is broadcast from LDS, and the partial sums of the row
// groups meet in two half-wave exchanges and one LDS add over the four waves.
// Passing the wide operand through LDS instead, one chain per output, took
// 10.9 us for the first launch and 8.75 us for the second; 6.2 and 6.3 us so.
// The first launch does what a row needs by itself -- forward, loss
// derivative, the backward pass to both hidden layers -- for kTrainRows rows
// per block; the second forms every gradient as a sum over the rows and
// updates its parameter at once.  Every output is a fixed tree of FP32 chains
// of fused multiply-adds over its inner index, whatever block computes it, so
// results do not depend on the split.

typedef float vec4 __attribute__((ext_vector_type(4)));

constexpr int kTrainRows = 2;   // rows per block: 128 blocks for the usual batch, each reads W1 once (128 KB)
constexpr int kTileK1 = 4;      // rows of W1 per block of the second launch
constexpr int kTileK2 = 8;      // rows of W2 per block
constexpr int kRowChunk = 128;  // rows of the batch read at a time
constexpr int kColTile = 16, kRowGroups = 16;  // bias sums

__device__ __forceinline__ int64_t train_row(const TrainStep& a, int i) { return a.idx ? (int64_t)a.idx[i] : i; }

// (a, b) -> the sums of a over lanes l and l + 32 in the lower half of the
// wave, of b in the upper half.
__device__ __forceinline__ float half_add(float a, float b) {
    const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                    false, false);
    return __builtin_bit_cast(float, (uint32_t)p[0]) + __builtin_bit_cast(float, (uint32_t)p[1]);
}

// The same between rows of 16 lanes: a's sums in rows 0 and 2, b's in 1 and 3.
__device__ __forceinline__ float row_add(float a, float b) {
    const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                    false, false);
    return __builtin_bit_cast(float, (uint32_t)p[0]) + __builtin_bit_cast(float, (uint32_t)p[1]);
}

__device__ __forceinline__ vec4 half_add(vec4 a, vec4 b) {
    return vec4{half_add(a.x, b.x), half_add(a.y, b.y), half_add(a.z, b.z), half_add(a.w, b.w)};
}
__device__ __forceinline__ vec4 row_add(vec4 a, vec4 b) {
    return vec4{row_add(a.x, b.x), row_add(a.y, b.y), row_add(a.z, b.z), row_add(a.w, b.w)};
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppMirror = 0x140, kDppHalfMirror = 0x141, kDppXor2 = 0x4E, kDppXor1 = 0xB1;

__device__ __forceinline__ vec4 fma4(float s, vec4 q, vec4 z) {
    return vec4{fmaf(s, q.x, z.x), fmaf(s, q.y, z.y), fmaf(s, q.z, z.z), fmaf(s, q.w, z.w)};
}

__global__ __launch_bounds__(256) void train_rows_kernel(TrainStep a) {
    // inner index k of a layer's input at [k mod groups][k div groups]: a
    // thread's rows of the weights are consecutive
    __shared__ __align__(16) float Xs[kTrainRows][8][36], h1s[kTrainRows][16][8];
    __shared__ __align__(16) float part[4][kTrainRows][128];
    __shared__ __align__(16) float h2s[kTrainRows][64], dz2s[kTrainRows][64];
    __shared__ float W3s[64 * kMaxC], dys[kTrainRows][kMaxC];
    static_assert(kTrainRows == 2, "the half-wave exchange takes one row per half");
    const int t = threadIdx.x, C = a.C, lane = t & 63, w = t >> 6;
    const int row0 = blockIdx.x * kTrainRows;
    const int nr = a.rows - row0 < kTrainRows ? a.rows - row0 : kTrainRows;
    const float* th = a.theta;
    const int u1 = t & 127, r1 = t >> 7;       // (row, unit) of the first hidden layer
    const int u2 = t & 63, r2 = (t >> 6) & 1;  // of the second (threads below 128)
    const int l16 = t & 15, o3 = t >> 4;       // 16 lanes per output of the last layer
    const int r3 = o3 / C, c3 = o3 - r3 * C;
    const bool out3 = r3 < nr;
    // every read of the block, in flight together
    const vec4* w1 = reinterpret_cast<const vec4*>(th + a.oW1);
    const vec4* w2 = reinterpret_cast<const vec4*>(th + a.oW2);
    int64_t xr[kTrainRows];
#pragma unroll
    for (int r = 0; r < kTrainRows; ++r) xr[r] = r < nr ? train_row(a, row0 + r) : 0;
    vec4 q1[32], q2[8];
    float x[kTrainRows], w3[2];
#pragma unroll
    for (int i = 0; i < 32; ++i) q1[i] = w1[i * 256 + t];
#pragma unroll
    for (int i = 0; i < 8; ++i) q2[i] = w2[i * 256 + t];
#pragma unroll
    for (int i = 0; i < 2; ++i) w3[i] = i * 256 + t < 64 * C ? th[a.oW3 + i * 256 + t] : 0.f;
    const float bias1 = th[a.ob1 + u1], bias2 = th[a.ob2 + u2], bias3 = out3 ? th[a.ob3 + c3] : 0.f;
#pragma unroll
    for (int r = 0; r < kTrainRows; ++r) x[r] = r < nr ? a.X[xr[r] * 256 + t] : 0.f;
    const float want = out3 ? a.T[(r3 ? xr[1] : xr[0]) * C + c3] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < kTrainRows; ++r) Xs[r][t & 7][t >> 3] = x[r];
#pragma unroll
    for (int i = 0; i < 2; ++i) W3s[i * 256 + t] = w3[i];
    __syncthreads();
    {
        vec4 z0{}, z1{};  // units 4 (t mod 32) .. + 3 over the rows t div 32 + 8 i
        const int g = t >> 5;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            z0 = fma4(Xs[0][g][i], q1[i], z0);
            z1 = fma4(Xs[1][g][i], q1[i], z1);
        }
        *reinterpret_cast<vec4*>(&part[w][lane >> 5][4 * (t & 31)]) = half_add(z0, z1);
    }
    __syncthreads();
    const float h1 =
        fmaxf(((part[0][r1][u1] + part[1][r1][u1]) + (part[2][r1][u1] + part[3][r1][u1])) + bias1, 0.f);
    h1s[r1][u1 & 15][u1 >> 4] = h1;
    if (r1 < nr) a.h1[(int64_t)(row0 + r1) * 128 + u1] = h1;
    __syncthreads();
    {
        vec4 z0{}, z1{};  // units 4 (t mod 16) .. + 3 over the rows t div 16 + 16 i
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            z0 = fma4(h1s[0][o3][i], q2[i], z0);
            z1 = fma4(h1s[1][o3][i], q2[i], z1);
        }
        const vec4 z = half_add(z0, z1);
        float* d = &part[w][lane >> 5][4 * l16 + ((lane >> 4) & 1)];
        d[0] = row_add(z.x, z.y);
        d[2] = row_add(z.z, z.w);
    }
    __syncthreads();
    float h2 = 0.f;
    if (t < 128) {
        h2 = fmaxf(((part[0][r2][u2] + part[1][r2][u2]) + (part[2][r2][u2] + part[3][r2][u2])) + bias2, 0.f);
        h2s[r2][u2] = h2;
        if (r2 < nr) a.h2[(int64_t)(row0 + r2) * 64 + u2] = h2;
    }
    __syncthreads();
    {
        float y = 0.f;
        if (r3 < kTrainRows)
#pragma unroll
            for (int q = 0; q < 4; ++q) y = fmaf(h2s[r3][4 * l16 + q], W3s[(4 * l16 + q) * C + c3], y);
        y += dpp_f32<kDppXor1>(y);
        y += dpp_f32<kDppXor2>(y);
        y += dpp_f32<kDppHalfMirror>(y);
        y += dpp_f32<kDppMirror>(y);
        if (l16 == 0 && r3 < kTrainRows) {
            const float d = (y + bias3) - want;
            const float dy = out3 ? 2.f * d * a.scale : 0.f;
            if (out3) {
                a.d[(int64_t)(row0 + r3) * C + c3] = d;
                a.dy[(int64_t)(row0 + r3) * C + c3] = dy;
            }
            dys[r3][c3] = dy;
        }
    }
    __syncthreads();
    if (t < 128) {
        float g = 0.f;
        for (int c = 0; c < C; ++c) g = fmaf(dys[r2][c], W3s[u2 * C + c], g);
        if (!(h2 > 0.f)) g = 0.f;  // the ReLU's derivative, from the activation
        dz2s[r2][u2] = g;
        if (r2 < nr) a.dz2[(int64_t)(row0 + r2) * 64 + u2] = g;
    }
    __syncthreads();
    {
        // rows of W2 times dz2: four columns per lane, then the sum over 16
        // lanes by halving: lane l ends with value l of 2 rows x 8
        float v[16];
        const vec4 d0 = *reinterpret_cast<const vec4*>(&dz2s[0][4 * l16]);
        const vec4 d1 = *reinterpret_cast<const vec4*>(&dz2s[1][4 * l16]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = fmaf(d0.w, q2[i].w, fmaf(d0.z, q2[i].z, fmaf(d0.y, q2[i].y, d0.x * q2[i].x)));
            v[8 + i] = fmaf(d1.w, q2[i].w, fmaf(d1.z, q2[i].z, fmaf(d1.y, q2[i].y, d1.x * q2[i].x)));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = ((l16 & 8) ? v[j + 8] : v[j]) + dpp_f32<kDppMirror>((l16 & 8) ? v[j] : v[j + 8]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = ((l16 & 4) ? v[j + 4] : v[j]) + dpp_f32<kDppHalfMirror>((l16 & 4) ? v[j] : v[j + 4]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            v[j] = ((l16 & 2) ? v[j + 2] : v[j]) + dpp_f32<kDppXor2>((l16 & 2) ? v[j] : v[j + 2]);
        const float g = ((l16 & 1) ? v[1] : v[0]) + dpp_f32<kDppXor1>((l16 & 1) ? v[0] : v[1]);
        part[0][l16 >> 3][(l16 & 7) * 16 + o3] = g;
    }
    __syncthreads();
    if (r1 < nr) a.dz1[(int64_t)(row0 + r1) * 128 + u1] = h1 > 0.f ? part[0][r1][u1] : 0.f;
}

// Parameter i with its moments, read before the gradient is known.
struct TrainParam {
    int64_t i;
    float m, v, th;
    __device__ __forceinline__ void load(const TrainStep& a, int64_t index) {
        i = index;
        if (a.grad) return;
        m = a.m[i];
        v = a.v[i];
        th = a.theta[i];
    }
    // Adam update with gradient gi, or (no update) the gradient itself.
    __device__ __forceinline__ void apply(const TrainStep& a, float gi) const {
        if (a.grad) {
            a.grad[i] = gi;
            return;
        }
        const float mi = a.b1 * m + (1.f - a.b1) * gi;
        const float vi = a.b2 * v + (1.f - a.b2) * gi * gi;
        a.m[i] = mi;
        a.v[i] = vi;
        a.theta[i] = th - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    }
};

// A chunk of kRowChunk rows of G [rows][N] in registers, a thread's rows N / 4
// threads apart; rows beyond the batch are zero and add nothing.
template <int N>
struct RowChunk {
    static constexpr int Q = kRowChunk * N / 4 / 256;
    vec4 q[Q];
    __device__ __forceinline__ void load(const float* G, int i0, int rows) {
        const int64_t base = (int64_t)i0 * N / 4, end = (int64_t)rows * N / 4;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int64_t e = base + i * 256 + threadIdx.x;
            q[i] = e < end ? reinterpret_cast<const vec4*>(G)[e] : vec4{};
        }
    }
};

// Sums over the batch's rows i of A[i][k] G[i][n], k < TK, n < N: A's row i at
// arow(i), `width` <= TK consecutive values; output (k, n) belongs to
// parameter at(k, n).  TK x N = 512: every thread ends with two outputs.
template <int TK, int N, typename ARow, typename At>
__device__ __forceinline__ void train_tile(const TrainStep& a, const ARow& arow, int width, const float* G,
                                           const At& at, float (*part)[512], float* sa) {
    constexpr int LANES = N / 4, GROUPS = 256 / LANES, STEPS = kRowChunk / GROUPS;
    static_assert(TK * N == 512 && (N == 128 || N == 64), "two outputs per thread");
    const int t = threadIdx.x, lane = t & 63, g = t / LANES;
    RowChunk<N> cur, next;
    float av[TK], an[TK];
    auto load = [&](int i0, RowChunk<N>& c, float (&v)[TK]) {
        const float* src = t < kRowChunk && i0 + t < a.rows ? arow(i0 + t) : nullptr;
        c.load(G, i0, a.rows);
#pragma unroll
        for (int q = 0; q < TK; ++q) v[q] = src && q < width ? src[q] : 0.f;  // the caller's histograms: 4-byte alignment
    };
    load(0, cur, av);
    TrainParam prm[2];
    int kk[2], nn[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int e = p * 256 + t;
        kk[p] = e / N;
        nn[p] = e % N;
        if (kk[p] < width) prm[p].load(a, at(kk[p], nn[p]));
    }
    vec4 acc[TK] = {};
    for (int i0 = 0; i0 < a.rows; i0 += kRowChunk) {
        const bool more = i0 + kRowChunk < a.rows;
        if (more) load(i0 + kRowChunk, next, an);
        if (i0) __syncthreads();  // the rows of A before are used
        if (t < kRowChunk)
#pragma unroll
            for (int q = 0; q < TK; ++q) sa[t * TK + q] = av[q];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
#pragma unroll
            for (int k = 0; k < TK; ++k) acc[k] = fma4(sa[(i * GROUPS + g) * TK + k], cur.q[i], acc[k]);
        if (more) {
            cur = next;
#pragma unroll
            for (int q = 0; q < TK; ++q) av[q] = an[q];
        }
    }
    // the wave's row groups: halves, then rows of 16; each step leaves half the
    // values in either part
    int k0 = (lane >> 5) * (TK / 2);
#pragma unroll
    for (int k = 0; k < TK / 2; ++k) acc[k] = half_add(acc[k], acc[k + TK / 2]);
    if constexpr (N == 64) {
#pragma unroll
        for (int k = 0; k < TK / 4; ++k) acc[k] = row_add(acc[k], acc[k + TK / 4]);
        k0 += ((lane >> 4) & 1) * (TK / 4);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
        *reinterpret_cast<vec4*>(&part[t >> 6][(k0 + k) * N + 4 * (t % LANES)]) = acc[k];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int e = p * 256 + t;
        if (kk[p] < width) prm[p].apply(a, (part[0][e] + part[1][e]) + (part[2][e] + part[3][e]));
    }
}

// Column sums of G [rows][N], 16 columns per block: 16 row groups (thread (g,
// c) adds rows g, g + 16, ... of column c), then the groups in order.
__device__ __forceinline__ void train_bias(const TrainStep& a, const float* G, int N, int block, int64_t out,
                                           float* s) {
    const int c = threadIdx.x % kColTile, g = threadIdx.x / kColTile;
    const int j = block * kColTile + c;
    TrainParam prm;
    if (g == 0 && j < N) prm.load(a, out + j);
    float v = 0.f;
    if (j < N)
#pragma unroll 16
        for (int i = g; i < a.rows; i += kRowGroups) v += G[(int64_t)i * N + j];
    s[g * (kColTile + 1) + c] = v;
    __syncthreads();
    if (g == 0 && j < N) {
        float t = s[c];
        for (int r = 1; r < kRowGroups; ++r) t += s[r * (kColTile + 1) + c];
        prm.apply(a, t);
    }
}

constexpr int kBlocksW1 = 256 / kTileK1, kBlocksW2 = 128 / kTileK2;
constexpr int kBlocksB1 = 128 / kColTile, kBlocksB2 = 64 / kColTile;
constexpr int kTrainBlocks = kBlocksW1 + kBlocksW2 + kBlocksB1 + kBlocksB2 + 3;  // and W3, b3, the loss

__global__ __launch_bounds__(256) void train_update_kernel(TrainStep a) {
    __shared__ __align__(16) float part[4][512];
    __shared__ __align__(16) float sa[kRowChunk * 8];
    static_assert(kTileK1 <= 8 && kTileK2 <= 8 && kMaxC <= 8, "sa holds a chunk of the narrow operand");
    const int t = threadIdx.x, C = a.C;
    float* s = &part[0][0];
    int b = blockIdx.x;
    if (b < kBlocksW1) {
        const int64_t k0 = b * kTileK1, out = a.oW1 + k0 * 128;
        train_tile<kTileK1, 128>(a, [&](int i) { return a.X + train_row(a, i) * 256 + k0; }, kTileK1, a.dz1,
                                 [=](int k, int n) { return out + k * 128 + n; }, part, sa);
        return;
    }
    b -= kBlocksW1;
    if (b < kBlocksW2) {
        const int64_t k0 = b * kTileK2, out = a.oW2 + k0 * 64;
        train_tile<kTileK2, 64>(a, [&](int i) { return a.h1 + (int64_t)i * 128 + k0; }, kTileK2, a.dz2,
                                [=](int k, int n) { return out + k * 64 + n; }, part, sa);
        return;
    }
    b -= kBlocksW2;
    if (b == 0) {  // W3 [64][C], transposed: the wide operand is the activation
        const int64_t out = a.oW3;
        train_tile<8, 64>(a, [&](int i) { return a.dy + (int64_t)i * C; }, C, a.h2,
                          [=](int k, int n) { return out + (int64_t)n * C + k; }, part, sa);
        return;
    }
    --b;
    if (b < kBlocksB1) return train_bias(a, a.dz1, 128, b, a.ob1, s);
    b -= kBlocksB1;
    if (b < kBlocksB2) return train_bias(a, a.dz2, 64, b, a.ob2, s);
    b -= kBlocksB2;
    if (b == 0) return train_bias(a, a.dy, C, 0, a.ob3, s);
    // the batch's loss: sum (Y - T)^2 / (rows C), FP64, in a fixed order
    double* sum = reinterpret_cast<double*>(s);
    double v = 0.0;
    const int64_t n = (int64_t)a.rows * C;
    for (int64_t i = t; i < n; i += 256) {
        const float d = a.d[i];
        v += (double)d * d;
    }
    sum[t] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) sum[t] += sum[t + w];
        __syncthreads();
    }
    if (t == 0) *a.loss = (float)(sum[0] * a.scale);
}

hipError_t launch_train_step(TrainStep a, int step, hipStream_t s) {
    a.b1 = 0.9f;
    a.b2 = 0.999f;
    a.eps = 1e-8f;
    a.c1 = 1.f - powf(a.b1, (float)step);
    a.c2 = 1.f - powf(a.b2, (float)step);
    hipLaunchKernelGGL(train_rows_kernel, dim3((a.rows + kTrainRows - 1) / kTrainRows), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(train_update_kernel, dim3(kTrainBlocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BF16 inference
// ---------------------------------------------------------------------------

// BF16 inference copy (InferLayout) of the flat FP32 parameters, one thread
// per element of the copy.
__global__ void to_bf16_kernel(const float* theta, uint16_t* out, int C) {
    using L = InferLayout;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t fW1 = 0, fb1 = fW1 + 256 * 128, fW2 = fb1 + 128, fb2 = fW2 + 128 * 64, fW3 = fb2 + 64;
    const int64_t fb3 = fW3 + 64 * (int64_t)C;
    int64_t src;
    if (e < L::b1) src = fW1 + (e % 256) * 128 + e / 256;                      // W1t[o][i] = W1[i][o]
    else if (e < L::W2) src = fb1 + (e - L::b1);
    else if (e < L::b2) src = fW2 + ((e - L::W2) % 128) * 64 + (e - L::W2) / 128;
    else if (e < L::W3) src = fb2 + (e - L::b2);
    else if (e < L::b3(C)) src = fW3 + ((e - L::W3) % 64) * C + (e - L::W3) / 64;
    else if (e < L::b3(C) + C) src = fb3 + (e - L::b3(C));
    else return;
    out[e] = to_bf16(theta[src]);
}

hipError_t launch_to_bf16(const float* theta, uint16_t* out, int C, hipStream_t s) {
    const int64_t n = InferLayout::b3(C) + C;
    hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, out, C);
    return hipGetLastError();
}

// What follows the network where start centroids are wanted (warm_post_one):
// `range`, the histogram's levels above zero, is collected as the histogram is
// read, so the inference launch ends with the starts.  A launch of its own for
// this, with the outputs and the histograms read again, took 5.4 us for 1,024
// instances and a launch gap (histograms and starts of 1,024 slices: 92.6 us
// so, 89.2 in one launch).
__device__ __forceinline__ void start_row(const uint64_t (&range)[4], const float* y, int C, double* v0) {
    int lo = 255, hi = 0;  // what a walk over no positive level ends with
#pragma unroll
    for (int q = 3; q >= 0; --q)
        if (range[q]) lo = 64 * q + __builtin_ctzll(range[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (range[q]) hi = 64 * q + 63 - __builtin_clzll(range[q]);
    warm_post_one(y, lo, hi, C, v0);
}

// One block (256 threads) per histogram (mlp_block_forward); outputs to Y, or
// (STARTS) start centroids to v0.
template <bool BF16, bool STARTS>
__global__ __launch_bounds__(256) void mlp_infer_kernel(const void* w, const float* X, int C, float* Y, double* v0) {
    __shared__ float a0[256];
    __shared__ float a1[128];
    __shared__ float a2[64];
    __shared__ float tmp[256];
    const int64_t s = blockIdx.x;
    if constexpr (STARTS) {
        __shared__ uint64_t range[4];
        __shared__ float y[kMaxC];
        const int t = threadIdx.x;
        const uint64_t m = __ballot(X[s * 256 + t] > 0.f);
        if ((t & 63) == 0) range[t >> 6] = m;
        mlp_block_forward<BF16>(w, X + s * 256, C, a0, a1, a2, tmp, y);
        __syncthreads();
        if (t == 0) start_row(range, y, C, v0 + s * C);
    } else {
        mlp_block_forward<BF16>(w, X + s * 256, C, a0, a1, a2, tmp, Y + s * C);
    }
}

// The BF16 network on kInferRows histograms per block: the arithmetic and its
// order are mlp_block_forward's, but a block reads the weights (83 KB) once for
// all of them.
constexpr int kInferRows = 4;  // one per wave for the starts

template <bool STARTS>
__global__ __launch_bounds__(256) void mlp_infer_rows_kernel(const uint16_t* w, const float* X, int count, int C,
                                                             float* Y, double* v0) {
    using L = InferLayout;
    __shared__ float a0[kInferRows][256], a1[kInferRows][128], a2[kInferRows][64], tmp[kInferRows][256];
    __shared__ uint64_t range[kInferRows][4];
    __shared__ float ys[kInferRows][kMaxC];
    const int t = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * kInferRows;
    const int m = count - s0 < kInferRows ? (int)(count - s0) : kInferRows;
#pragma unroll
    for (int h = 0; h < kInferRows; ++h) {
        const float x = h < m ? X[(s0 + h) * 256 + t] : 0.f;
        a0[h][t] = act<true>(x);
        if constexpr (STARTS) {
            const uint64_t r = __ballot(x > 0.f);
            if ((t & 63) == 0) range[h][t >> 6] = r;
        }
    }
    uint4 w2[16], w3[8];
    if (t < 64) load_bf16<16>(w + L::W2 + t * 128, w2);
    if (t < C) load_bf16<8>(w + L::W3 + t * 64, w3);
    __syncthreads();
    const int o = t & 127, half = t >> 7;
    float z[kInferRows];
#pragma unroll
    for (int h = 0; h < kInferRows; ++h) z[h] = half ? 0.f : from_bf16(w[L::b1 + o]);
#pragma unroll
    for (int c = 0; c < 128; c += 64) {
        uint4 q[8];
        load_bf16<8>(w + L::W1 + o * 256 + 128 * half + c, q);
#pragma unroll
        for (int h = 0; h < kInferRows; ++h) z[h] = dot_bf16_regs<8>(z[h], a0[h] + 128 * half + c, q);
    }
#pragma unroll
    for (int h = 0; h < kInferRows; ++h) tmp[h][t] = z[h];
    __syncthreads();
    for (int e = t; e < kInferRows * 128; e += 256) {
        const int h = e >> 7, u = e & 127;
        a1[h][u] = act<true>(fmaxf(tmp[h][u] + tmp[h][u + 128], 0.f));
    }
    __syncthreads();
    if (t < 64)
#pragma unroll
        for (int h = 0; h < kInferRows; ++h)
            a2[h][t] = act<true>(fmaxf(dot_bf16_regs<16>(from_bf16(w[L::b2 + t]), a1[h], w2), 0.f));
    __syncthreads();
    if (t < C)
#pragma unroll
        for (int h = 0; h < kInferRows; ++h) {
            const float y = dot_bf16_regs<8>(from_bf16(w[L::b3(C) + t]), a2[h], w3);
            if constexpr (STARTS)
                ys[h][t] = y;
            else if (h < m)
                Y[(s0 + h) * C + t] = y;
        }
    if constexpr (STARTS) {
        __syncthreads();
        const int h = t >> 6;
        if ((t & 63) == 0 && h < m) start_row(range[h], ys[h], C, v0 + (s0 + h) * C);
    }
}

// Several histograms per block from the count on that still gives every second
// CU a block (1,024 histograms: 19 us one per block, 12 us four per block).
template <bool STARTS>
static hipError_t launch_bf16(const void* w, const float* X, int count, int C, float* Y, double* v0, hipStream_t s) {
    if (count >= 128 * kInferRows)
        hipLaunchKernelGGL(mlp_infer_rows_kernel<STARTS>, dim3((count + kInferRows - 1) / kInferRows), dim3(256), 0, s,
                           static_cast<const uint16_t*>(w), X, count, C, Y, v0);
    else
        hipLaunchKernelGGL((mlp_infer_kernel<true, STARTS>), dim3(count), dim3(256), 0, s, w, X, C, Y, v0);
    return hipGetLastError();
}

hipError_t launch_mlp_infer(const void* w, bool bf16, const float* X, int count, int C, float* Y, hipStream_t s) {
    if (bf16) return launch_bf16<false>(w, X, count, C, Y, nullptr, s);
    hipLaunchKernelGGL((mlp_infer_kernel<false, false>), dim3(count), dim3(256), 0, s, w, X, C, Y,
                       static_cast<double*>(nullptr));
    return hipGetLastError();
}

hipError_t launch_mlp_starts(const void* w, const float* X, int count, int C, double* v0, hipStream_t s) {
    return launch_bf16<true>(w, X, count, C, nullptr, v0, s);
}

// ---------------------------------------------------------------------------
// histograms without allocation (fcm_histogram_noalloc)
// ---------------------------------------------------------------------------

// The workspace of fcm_histogram in a fixed device array: the instance
// offsets, the first blocks of a list, then the counters ([count][copies][256]; one instance uses
// kHistCopies copies, more instances one copy each).  Each device holds its
// own copy of the array for the life of the process.
constexpr int kNoAllocMaxCount = 1024;
constexpr size_t kNoAllocOffBytes =
    ((sizeof(int64_t) + sizeof(int32_t)) * (kNoAllocMaxCount + 1) + 255) / 256 * 256;
constexpr size_t kNoAllocCountWords = 256 * (size_t)kNoAllocMaxCount;
static_assert((size_t)kHistCopies <= (size_t)kNoAllocMaxCount, "one instance's copies fit");
static __device__ __align__(256) unsigned char scratch[kNoAllocOffBytes + sizeof(uint32_t) * kNoAllocCountWords];

__global__ __launch_bounds__(kBlock) void zero_words_kernel(uint32_t* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = 0u;
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (in host code the array's
// name is not a device address); looked up once per device.
int scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return dev_err(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return FCM_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return dev_err(e == hipSuccess ? hipErrorInvalidSymbol : e, "hipGetSymbolAddress");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return FCM_OK;
}

}  // namespace

}  // namespace fcm

extern "C" int fcm_histogram_noalloc(const uint8_t* d_x, const int64_t* offsets, int32_t count, float* d_hist,
                                     void* stream) {
    using namespace fcm;
    if (!d_x || !offsets || !d_hist || count < 1 || offsets[0] != 0) return FCM_EINVAL;
    int64_t max_n = 0;
    for (int32_t i = 0; i < count; ++i) {
        if (offsets[i + 1] <= offsets[i]) return FCM_EINVAL;
        max_n = offsets[i + 1] - offsets[i] > max_n ? offsets[i + 1] - offsets[i] : max_n;
    }
    if (max_n > (int64_t)UINT32_MAX) return FCM_EINVAL;
    if (count > kNoAllocMaxCount) {
        last_error() = "fcm_histogram_noalloc: more instances than its fixed workspace holds (1024)";
        return FCM_EINVAL;
    }
    void* base = nullptr;
    int rc = scratch_address(&base);
    if (rc != FCM_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    int64_t* d_off = reinterpret_cast<int64_t*>(base);
    int32_t* d_first = reinterpret_cast<int32_t*>(d_off + kNoAllocMaxCount + 1);
    uint32_t* d_counts = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(base) + kNoAllocOffBytes);
    int32_t first[kNoAllocMaxCount + 1];
    const HistSplit sp = histogram_split(offsets, count, max_n, first);
    FCM_HIP(hipMemcpyAsync(d_off, offsets, sizeof(int64_t) * ((size_t)count + 1), hipMemcpyHostToDevice, s));
    if (sp.form == kHistList)
        FCM_HIP(hipMemcpyAsync(d_first, first, sizeof(int32_t) * ((size_t)count + 1), hipMemcpyHostToDevice, s));
    if (histogram_needs_counts(sp)) {
        // the array keeps the previous call's counts: clear them (a kernel, no memset node)
        const int64_t words = 256 * (int64_t)count * histogram_copies(count);
        const int zgrid = (int)((words + kBlock - 1) / kBlock < 1024 ? (words + kBlock - 1) / kBlock : 1024);
        hipLaunchKernelGGL(zero_words_kernel, dim3(zgrid), dim3(kBlock), 0, s, d_counts, words);
        FCM_HIP(hipGetLastError());
    }
    FCM_HIP(launch_histogram_counts(d_x, d_off, d_first, sp, count, d_counts, d_hist, s));
    FCM_HIP(hipStreamSynchronize(s));
    return FCM_OK;
}
