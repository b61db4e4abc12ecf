// Algorithm 1 over the grey levels of an 8-bit input (device code shared by
// the single and the batched solver).
//
// Every sum of Eq.1 and Eq.3 over the voxels regroups exactly by grey level,
// sum_i f(x_i) = sum_g h_g f(g), and the memberships of Eq.4 depend on a
// voxel only through its grey level, so the largest membership change of
// Algorithm 1 is the largest change over the levels present.  So the voxels
// are read once, into 256 counts, and the iteration runs on at most 256
// levels, in FP64, inside one block (the binning idea the paper cites in
// Sec. 3, exact here because the data are 8-bit).
//
// Two parts:
//   level_count    a block's voxels into 256 counts;
//   level_iterate  Algorithm 1 on the counts.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fcm.h"
#include "fcm_device.h"
#include "fcm_internal.h"
#include "fcm_level.h"

namespace fcm {

// ---------------------------------------------------------------------------
// counting
// ---------------------------------------------------------------------------

constexpr int kLvWaves = kLvBlock / 64;
constexpr int kLvIterWaves = 5;  // four waves of 64 levels, one that records the history

// One counter column per lane, bin-major: the 64 lanes of a wave touch 64
// different banks whatever their voxels hold (a brain slice is half
// background: one shared table would serialise up to 64 adds to one word).
// The block's waves share the columns.
using LevelTable = uint32_t[256 * 64];

__device__ __forceinline__ void level_clear(uint32_t* tab) {
    uint4* t4 = reinterpret_cast<uint4*>(tab);
#pragma unroll
    for (int i = 0; i < 256 * 64 / 4 / kLvBlock; ++i) t4[i * kLvBlock + threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ void level_bump(char* tab, uint32_t off) {
    // relaxed add without return: a fire-and-forget ds_add
    __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(tab + off), 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The 16 voxels of a chunk.  The byte offset of a counter is (level << 8) |
// (lane << 2), so the level's byte is masked where it lies or shifted once.
__device__ __forceinline__ void level_chunk(char* tab, uint32_t lane4, uint4 w) {
    const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t v = words[i];
        level_bump(tab, ((v << 8) & 0xFF00u) | lane4);
        level_bump(tab, (v & 0xFF00u) | lane4);
        level_bump(tab, ((v >> 8) & 0xFF00u) | lane4);
        level_bump(tab, ((v >> 16) & 0xFF00u) | lane4);
    }
}

constexpr int kLvUnroll = 4;  // chunks a thread counts while the next as many are on their way

// Chunks c0 + first, + step, ... below c1 of `body` into the table.
__device__ __forceinline__ void level_count(char* tab, const uint4* body, int64_t first, int64_t c1, int64_t step) {
    const uint32_t lane4 = (threadIdx.x & 63u) << 2;
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    int64_t c = first;
    uint4 cur[kLvUnroll];
#pragma unroll
    for (int u = 0; u < kLvUnroll; ++u) cur[u] = c + u * step < c1 ? body[c + u * step] : z;
    while (c + (kLvUnroll - 1) * step < c1) {
        const int64_t cn = c + kLvUnroll * step;
        uint4 nxt[kLvUnroll];
#pragma unroll
        for (int u = 0; u < kLvUnroll; ++u) nxt[u] = cn + u * step < c1 ? body[cn + u * step] : z;
#pragma unroll
        for (int u = 0; u < kLvUnroll; ++u) level_chunk(tab, lane4, cur[u]);
#pragma unroll
        for (int u = 0; u < kLvUnroll; ++u) cur[u] = nxt[u];
        c = cn;
    }
#pragma unroll
    for (int u = 0; u < kLvUnroll; ++u)
        if (c + u * step < c1) level_chunk(tab, lane4, cur[u]);
}

// Unaligned head and tail of an instance (fewer than 16 voxels each).
__device__ __forceinline__ void level_ragged(char* tab, const uint8_t* x, int64_t n, int64_t head, int64_t nbody) {
    const int64_t tail0 = head + 16 * nbody;
    const int64_t nr = head + (n - tail0);
    const int64_t t = threadIdx.x;
    if (t < nr) {
        const uint32_t v = x[t < head ? t : tail0 + (t - head)];
        level_bump(tab, (v << 8) | ((threadIdx.x & 63u) << 2));
    }
}

// Count of level t in threads t < 256 after a block-wide call (the first 256
// threads add the 64 columns of their level four at a time, each starting at
// its own columns so that a quarter wave's 16-byte reads lie in different
// banks; single words took 0.9 us, 0.3 us so).
__device__ __forceinline__ uint32_t level_total(const uint32_t* tab) {
    uint32_t c = 0u;
    const uint32_t t = threadIdx.x;
    if (t < 256u) {
        const uint4* row = reinterpret_cast<const uint4*>(tab) + t * 16u;
        uint4 s = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (uint32_t i = 0; i < 16u; ++i) {
            const uint4 q = row[(i + t) & 15u];
            s.x += q.x;
            s.y += q.y;
            s.z += q.z;
            s.w += q.w;
        }
        c = (s.x + s.y) + (s.z + s.w);
    }
    return c;
}

// ---------------------------------------------------------------------------
// iteration
// ---------------------------------------------------------------------------

// What one instance needs to iterate; the same for every thread of the block.
struct LevelProblem {
    double eps, m, alpha;     // alpha = 1 / (m - 1)
    int32_t max_iter, max_passes;
    int32_t do_init;          // start from v^0; else continue at `pass` from the history
    int32_t given;            // start mode: 0 evenly spaced, 1 v0, 2 dv0 (device); LEARNED: the network's (mlp_w)
    int32_t pass;             // do_init == 0: index of the next pass (0: v^0 is committed, no pass has run)
    int32_t fp32_range;       // report starts whose FP32 distances overflow as non-finite
    int64_t n;
    const double* v0;
    const double* dv0;
    const uint16_t* mlp_w;
    double* hist_v;
    double* hist_d;
    double* hist_J;
    uint64_t* times;          // commit times (wall clock), entry 0 the start, entry p + 1 pass p; or null
};

// Result of level_iterate, in the recording wave (the centroids, v^pass and
// v^iters, are in LevelScratch::v and vp).
struct LevelOutcome {
    int32_t pass, iters, passes, status, done, lo, hi;
    double delta, J;
};

// Shared memory of level_iterate (lies over the counting table).
constexpr int kLvRetry = 1, kLvEnd = 2, kLvStatusShift = 8, kLvStatus0 = 64;
constexpr int kExpSteps = 32, kLogSteps = 64;

struct LevelScratch {
    double red[2][8][2][4];   // [attempt parity][cluster][num, den][wave]
    int flag[2][4];           // wave: a level changed by eps or more
    // of an attempt, for the recording wave, which is one barrier behind
    double dm[3][256];        // largest membership change of a level
    double jt[3][256];        // its term of Eq.1
    double vnext[3][8];
    int dec[3];               // kLvRetry, or status + kLvStatus0 and kLvEnd
    double v[8], vp[8];
    double ex[kExpSteps];     // 2^(j / kExpSteps)
    double lg[kLogSteps][2];  // 1 / f_j and log2 f_j, f_j = 1 + (j + 1/2) / kLogSteps
    uint64_t mask[4];
    float h[256], a0[256], a1[128], a2[64], tmp[256], y[8];
    double w0[8];
};
static_assert(sizeof(LevelScratch) <= sizeof(LevelTable), "scratch lies over the counting table");

// Block barrier that orders shared memory only: __syncthreads also waits for
// the wave's global stores, and the recording wave stores a row of the
// history in every pass (0.5 us each time).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ double readfirst_d(double v) { return readlane_d(v, 0); }

// (a, b) -> the sums of a over lanes l and l + 32 in the lower half of the
// wave, of b in the upper half: the instruction swaps a's upper half with b's
// lower half.
__device__ __forceinline__ double swap32_add(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
           __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}

// The same between rows of 16: a's rows 1 and 3 change places with b's rows 0
// and 2, so a's row pairs end in rows 0 and 2, b's in rows 1 and 3.
__device__ __forceinline__ double swap16_add(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
           __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
}

// Sum over the lane's row of 16, in every lane of the row.
__device__ __forceinline__ double row_sum_f64(double v) {
    v += dpp_mov_f64<0xB1>(v);
    v += dpp_mov_f64<0x4E>(v);
    v += dpp_mov_f64<0x141>(v);
    v += dpp_mov_f64<0x140>(v);
    return v;
}

// Sums of four values over the wave, value r in row r: each swap folds two
// values into one register, 21 instructions for four sums in a chain of six
// adds (one value at a time with moves and adds: 72 in the same chain).  Sums
// by the 4x4x4 FP64 matrix instruction need fewer instructions still but wait
// for each other's results: the same time per pass within 5 %.
__device__ __forceinline__ double quad_sum_f64(double v0, double v1, double v2, double v3) {
    return row_sum_f64(swap16_add(swap32_add(v0, v2), swap32_add(v1, v3)));
}

// max over the wave of non-negative values, valid in lane 63 (row butterflies,
// then the rows' last lanes broadcast upwards; lanes without a source read 0)
__device__ __forceinline__ double wave_max_pos_f64(double v) {
    v = fmax(v, dpp_mov_f64<0xB1>(v));
    v = fmax(v, dpp_mov_f64<0x4E>(v));
    v = fmax(v, dpp_mov_f64<0x141>(v));
    v = fmax(v, dpp_mov_f64<0x140>(v));
    v = fmax(v, dpp_mov_f64<0x142>(v));  // row_bcast:15
    v = fmax(v, dpp_mov_f64<0x143>(v));  // row_bcast:31
    return v;
}

// 1 / s to the last bit or two: hardware estimate and two Newton steps.
__device__ __forceinline__ double recip_f64(double s) {
    double r = __builtin_amdgcn_rcp(s);
    r = fma(r, fma(-s, r, 1.0), r);
    r = fma(r, fma(-s, r, 1.0), r);
    return r;
}

// log2 of a positive normal number: exponent + log2 f_j + log2(1 + r), where f
// is the mantissa, f_j the middle of its 1/64 interval and r = f / f_j - 1
// (|r| <= 2^-7), by the series of the logarithm (next term below 3e-18).
__device__ __forceinline__ double log2_tab(double x, const LevelScratch& sh) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t hi = (uint32_t)(b >> 32);
    const int e = (int)(hi >> 20) - 1023, j = (int)(hi >> 14) & (kLogSteps - 1);
    const double f =
        __builtin_bit_cast(double, (b & 0xFFFFFFFFull) | ((uint64_t)((hi & 0xFFFFFu) | 0x3FF00000u) << 32));
    constexpr double K = 1.4426950408889634074;  // 1 / ln 2
    const double r = fma(f, sh.lg[j][0], -1.0);
    double p = fma(r, K / 7, -K / 6);
    p = fma(r, p, K / 5);
    p = fma(r, p, -K / 4);
    p = fma(r, p, K / 3);
    p = fma(r, p, -K / 2);
    p = fma(r, p, K);
    return fma(r, p, (double)e + sh.lg[j][1]);
}

// 2^y (0 far below): y = n / 32 + r, the table's 2^((n mod 32) / 32) times the
// exponential series in r (|r| <= 2^-6, next term below 4e-18), times 2^(n div 32).
__device__ __forceinline__ double exp2_tab(double y, const LevelScratch& sh) {
    y = fmax(y, -1100.0);
    const double nd = rint(y * kExpSteps);
    const int n = (int)nd;
    constexpr double L = 0.69314718055994530942;
    const double r = fma(nd, -1.0 / kExpSteps, y);
    double p = fma(r, L * L * L * L * L * L / 720, L * L * L * L * L / 120);
    p = fma(r, p, L * L * L * L / 24);
    p = fma(r, p, L * L * L / 6);
    p = fma(r, p, L * L / 2);
    p = fma(r, p, L);
    p = fma(r, p, 1.0);
    return ldexp(p * sh.ex[n & (kExpSteps - 1)], n >> 5);
}

// Eq.4 and u^m by distance ratios, u_k = w_k / sum_j w_j with
// w_k = (d_min / d_k)^(2/(m-1)) <= 1, and the zero-distance rule (equal split
// over the clusters at distance 0): the form that holds for any centroids, and
// gives equal ones equal memberships to the last bit.
template <int C>
__device__ __noinline__ double level_u_any(double x, const double* v, double m, double* u, double* a) {
    double d[C];
    double dmin = 1.0e308;
    int nz = 0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        d[k] = fabs(x - v[k]);
        dmin = fmin(dmin, d[k]);
        nz += d[k] == 0.0;
    }
    if (nz) {
        const double un = 1.0 / nz, an = m == 2.0 ? un * un : pow(un, m);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = d[k] == 0.0 ? un : 0.0;
            a[k] = d[k] == 0.0 ? an : 0.0;
        }
        return 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const double r = dmin / d[k];
        u[k] = m == 2.0 ? r * r : pow(r, 2.0 / (m - 1.0));
        s += u[k];
    }
#pragma unroll
    for (int k = 0; k < C; ++k) {
        u[k] /= s;
        a[k] = m == 2.0 ? u[k] * u[k] : pow(u[k], m);
    }
    double j = 0.0;
#pragma unroll
    for (int k = 0; k < C; ++k) j += a[k] * d[k] * d[k];
    return j;
}

// Memberships u (Eq.4) and a = u^m of grey level x.  With q_k = (x - v_k)^2,
// the m = 2 memberships are u2_k = P_k / sum_j P_j, P_k = prod_{j != k} q_j
// (one reciprocal); other m follow from w_k = u2_k^alpha, u_k = w_k / S,
// S = sum w, and u_k^m = w_k u2_k / S^m because alpha (m - 1) = 1 -- so only
// the generic m needs logarithms, one log2 and one exp2 per cluster.  Returns
// the level's term of Eq.1, sum_k u_k^m q_k = u2_0 q_0 S^(1-m) (u2_k q_k is the
// same for every k).  `safe`: by the ratio form.  The caller asks for it in
// every pass where two centroids are equal -- their products round differently,
// and Algorithm 1 moves away from coinciding centroids exponentially once they
// differ -- and from the pass on in which products out of range (centroids far
// beyond the grey levels) gave non-finite sums.  (Equal products and the
// zero-distance rule inside the product form, or anything else that touches
// this branch in a pass, costs every other solve 1 to 10 % of a pass.)
template <int C, int MK>
__device__ __forceinline__ double level_u(double x, const double (&v)[C], double m, double alpha, bool safe, bool on,
                                          const LevelScratch& sh, double (&u)[C], double (&a)[C]) {
    if (safe) {
        double cv[C], cu[C], ca[C];  // copies: only they live in memory
#pragma unroll
        for (int k = 0; k < C; ++k) cv[k] = v[k];
        // a level that no voxel has takes the cheap way out of the rule
        const double j = level_u_any<C>(on ? x : v[0], cv, m, cu, ca);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = cu[k];
            a[k] = ca[k];
        }
        return j;
    }
    double q[C], P[C], pre[C], suf[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const double d = x - v[k];
        q[k] = d * d;
    }
    pre[1] = q[0];
#pragma unroll
    for (int k = 2; k < C; ++k) pre[k] = pre[k - 1] * q[k - 1];
    suf[C - 1] = q[C - 1];
#pragma unroll
    for (int k = C - 2; k >= 1; --k) suf[k] = q[k] * suf[k + 1];
    P[0] = suf[1];
    P[C - 1] = pre[C - 1];
#pragma unroll
    for (int k = 1; k < C - 1; ++k) P[k] = pre[k] * suf[k + 1];
    double S = P[0];
#pragma unroll
    for (int j = 1; j < C; ++j) S += P[j];
    const double r = recip_f64(S);
#pragma unroll
    for (int k = 0; k < C; ++k) P[k] *= r;  // u2
    const double j2 = P[0] * q[0];
    if constexpr (MK == kM2) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = P[k];
            a[k] = P[k] * P[k];
        }
        return j2;
    } else if constexpr (MK == kM15) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = P[k] * P[k];
            s += u[k];
        }
        const double rs = recip_f64(s), t = rs * sqrt(rs);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            a[k] = u[k] * P[k] * t;
            u[k] *= rs;
        }
        return j2 * (s * t);
    } else {
        double L[C], top = -1.0e300;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            L[k] = log2_tab(fmax(P[k], 1.0e-290), sh);
            top = fmax(top, L[k]);
        }
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const double w = exp2_tab(alpha * (L[k] - top), sh);  // largest 1
            u[k] = P[k] > 1.0e-290 ? w : 0.0;
            s += u[k];
        }
        const double rs = recip_f64(s);
        // u^m = w_k (u2_k / u2_max) s^-m
        const double t = exp2_tab(fma(-m, log2_tab(s, sh), -top), sh);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            a[k] = u[k] * P[k] * t;
            u[k] *= rs;
        }
        return j2 * (s * t);
    }
}

// Whether any two of the centroids (the same in every lane) are equal.
template <int C>
__device__ __forceinline__ bool any_equal(const double (&v)[C]) {
    bool eq = false;
#pragma unroll
    for (int k = 1; k < C; ++k)
#pragma unroll
        for (int j = 0; j < k; ++j) eq = eq || v[j] == v[k];
    return __builtin_amdgcn_readfirstlane(eq) != 0;
}

// Algorithm 1 on the counts: thread t < 256 holds the count of level t.
// Called by kLvIterWaves waves (the block's other waves have ended).  Waves
// 0..3 own 64 levels each, one per lane; per attempt at a pass a wave
// evaluates Eq.4 once (U^(p-1) stays in registers), sums its levels and writes
// its partial sums; after the attempt's only barrier every wave adds the four
// partial sums in wave order and takes the decision itself (same bits in
// every lane).  The stopping test needs only one bit per wave; the change and
// the objective of the history are reduced and recorded by the fifth wave,
// one barrier behind, off the others' path.  One wave per SIMD runs a chain of
// dependent instructions, an LDS round trip and a barrier per pass: latency is
// what there is to save, and one CU is all that 256 levels can use (a second
// one would cost two exchanges of 1.1 us).  Per pass, C = 4, m = 2: 0.82 us
// with a chain of moves and adds per sum and the record in the same
// interval, 0.65 us so; C = 8, m = 2.5: 3.0 us with the library's log2 and
// exp2, 1.8 us with the tables above.
template <int C, int MK, bool LEARNED>
__device__ __forceinline__ void level_iterate(const LevelProblem& pb, uint32_t cnt, LevelScratch& sh,
                                              LevelOutcome& out) {
    constexpr int SETS = (C + 3) / 4;  // clusters a lane sums: kc, kc + 4
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool work = wid < 4;
    const double c = (double)cnt, x = (double)tid;
    int lo = 0, hi = 255, p = 0;
    double v[C];
    double uo[C];
#pragma unroll
    for (int k = 0; k < C; ++k) uo[k] = 0.0;
    bool huge = false, twins = false;
    if constexpr (MK == kMGeneric) {
        if (tid < kExpSteps) sh.ex[tid] = exp2((double)tid / kExpSteps);
        if (tid < kLogSteps) {
            const double f = 1.0 + (tid + 0.5) / kLogSteps, r = 1.0 / f;
            sh.lg[tid][0] = r;
            sh.lg[tid][1] = -log2(r);
        }
        lds_barrier();
    }
    if (pb.do_init) {
        if (work) {
            const uint64_t m = __ballot(cnt != 0u);
            if (lane == 0) sh.mask[wid] = m;
        }
        __syncthreads();
        lo = 255;
        hi = 0;
#pragma unroll
        for (int w = 3; w >= 0; --w)
            if (sh.mask[w]) lo = 64 * w + __builtin_ctzll(sh.mask[w]);
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (sh.mask[w]) hi = 64 * w + 63 - __builtin_clzll(sh.mask[w]);
        const double* dv0 = pb.dv0;
        if constexpr (LEARNED) {
            if (work) sh.h[tid] = hist_norm(cnt, pb.n);
            __syncthreads();
            mlp_block_forward<true>(pb.mlp_w, sh.h, C, sh.a0, sh.a1, sh.a2, sh.tmp, sh.y);
            __syncthreads();
            if (tid == 0) warm_post_one(sh.y, lo, hi, C, sh.w0);
            __syncthreads();
            dv0 = sh.w0;
        }
        if (tid == 0) {
            double s[C];
            start_centroids(C, (uint32_t)lo, (uint32_t)hi, LEARNED ? 2 : pb.given, pb.v0, dv0, s);
            for (int k = 0; k < C; ++k) sh.v[k] = s[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = readfirst_d(sh.v[k]);
        twins = LEARNED || pb.given ? any_equal<C>(v) : lo == hi;  // evenly spaced
        if (wid == 4) {
            if (lane < C) pb.hist_v[lane] = sh.v[lane];
            if (pb.times && lane == 0) pb.times[0] = wall_clock64();
        }
    } else {
        p = pb.pass;
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = readfirst_d(pb.hist_v[(int64_t)p * C + k]);
        twins = any_equal<C>(v);
        if (work && p > 0) {
            double vp[C], t[C];
#pragma unroll
            for (int k = 0; k < C; ++k) vp[k] = pb.hist_v[(int64_t)(p - 1) * C + k];
            level_u<C, MK>(x, vp, pb.m, pb.alpha, twins, cnt != 0u, sh, uo, t);
            bool fin = true;
#pragma unroll
            for (int k = 0; k < C; ++k) fin = fin && isfinite(uo[k]);
            if (!fin) level_u<C, MK>(x, vp, pb.m, pb.alpha, true, cnt != 0u, sh, uo, t);
        }
    }
    // also where v^0 was committed before this launch (a query or labels first)
    if (pb.fp32_range && p == 0)
#pragma unroll
        for (int k = 0; k < C; ++k) huge = huge || !(fabs(v[k]) < 1.8e19);
    const bool owner = (lane & 15) == 0;  // one lane per cluster of a set
    int kc[SETS];       // the clusters whose sums this lane holds
    double vk[SETS], vr[SETS];  // their centroids in this pass; in the last pass run
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int k = (lane >> 4) + 4 * s;
        kc[s] = k < C ? k : C - 1;
        vk[s] = v[0];
#pragma unroll
        for (int q = 1; q < C; ++q)
            if (kc[s] == q) vk[s] = v[q];
        vr[s] = vk[s];
    }
    if (pb.max_passes <= 0) return;
    if (work) {
        // passes below `calm` go on unless they converge or turn non-finite
        const int64_t stop_at = (int64_t)p + pb.max_passes - 1;
        const int calm = huge ? -1 : (int)(stop_at < pb.max_iter ? stop_at : pb.max_iter);
        int par = 0, slot = 0;
        bool safe = twins;
        while (true) {
            double u[C], a[C];
            const double jt = level_u<C, MK>(x, v, pb.m, pb.alpha, safe, cnt != 0u, sh, u, a);
#pragma unroll
            for (int k = 0; k < C; ++k) a[k] *= c;
            double num[SETS], den[SETS];
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                double t[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) t[k] = 4 * s + k < C ? a[4 * s + k < C ? 4 * s + k : 0] : 0.0;
                num[s] = quad_sum_f64(t[0] * x, t[1] * x, t[2] * x, t[3] * x);
                den[s] = quad_sum_f64(t[0], t[1], t[2], t[3]);
            }
            double dm = 0.0;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const double d = u[k] - uo[k];
                dm = fmax(dm, fmax(d, -d));
            }
            if (!cnt) dm = 0.0;
            const bool moved = __any(dm >= pb.eps);
            sh.dm[slot][tid] = dm;
            sh.jt[slot][tid] = c * jt;
            if (owner) {
#pragma unroll
                for (int s = 0; s < SETS; ++s)
                    if (kc[s] == (lane >> 4) + 4 * s) {
                        sh.red[par][kc[s]][0][wid] = num[s];
                        sh.red[par][kc[s]][1][wid] = den[s];
                    }
                if (lane == 0) sh.flag[par][wid] = moved;
            }
            lds_barrier();
            double rn[SETS][8];
#pragma unroll
            for (int s = 0; s < SETS; ++s)
#pragma unroll
                for (int i = 0; i < 8; ++i) rn[s][i] = sh.red[par][kc[s]][0][i];
            const int any = (sh.flag[par][0] | sh.flag[par][1]) | (sh.flag[par][2] | sh.flag[par][3]);
            __builtin_amdgcn_sched_barrier(0);  // all reads are on their way before anything waits for one
            double vn[SETS];
            bool fin = true;
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                const double nt = ((rn[s][0] + rn[s][1]) + rn[s][2]) + rn[s][3];
                const double dt = ((rn[s][4] + rn[s][5]) + rn[s][6]) + rn[s][7];
                const double q = nt / dt;
                vn[s] = dt > 0.0 ? q : vk[s];
                fin = fin && isfinite(vn[s]) && dt >= 0.0;
            }
            const bool ok = __all(fin);
            const bool go = ok && __builtin_amdgcn_readfirstlane(any) != 0;
            int dec = (FCM_RUNNING + kLvStatus0) << kLvStatusShift;
            bool run = true;
            if (!(go && p < calm)) {
                const bool retry = !ok && !safe;  // again, with the form that holds for any centroids
                const int status = !ok || huge ? FCM_ENUMERIC
                                               : (p >= 1 && !go ? FCM_OK : (p >= pb.max_iter ? FCM_NOT_CONVERGED
                                                                                             : FCM_RUNNING));
                run = !retry && status == FCM_RUNNING && p < stop_at;
                dec = retry ? kLvRetry : ((status + kLvStatus0) << kLvStatusShift) | (run ? 0 : kLvEnd);
            }
            if (wid == 0 && owner) {
#pragma unroll
                for (int s = 0; s < SETS; ++s)
                    if (kc[s] == (lane >> 4) + 4 * s) sh.vnext[slot][kc[s]] = vn[s];
                if (lane == 0) sh.dec[slot] = dec;
            }
            par ^= 1;
            slot = slot == 2 ? 0 : slot + 1;
            if (run) {
#pragma unroll
                for (int k = 0; k < C; ++k) v[k] = readlane_d(vn[k / 4], 16 * (k % 4));
#pragma unroll
                for (int k = 0; k < C; ++k) uo[k] = u[k];
#pragma unroll
                for (int s = 0; s < SETS; ++s) vk[s] = vn[s];
                ++p;
            } else if (dec & kLvRetry) {
                safe = true;
            } else {
#pragma unroll
                for (int s = 0; s < SETS; ++s) {
                    vr[s] = vk[s];
                    if ((dec >> kLvStatusShift) - kLvStatus0 == FCM_RUNNING) vk[s] = vn[s];  // out of passes only
                }
                break;
            }
        }
        if (wid == 0 && owner)
#pragma unroll
            for (int s = 0; s < SETS; ++s)
                if (kc[s] == (lane >> 4) + 4 * s) {
                    sh.v[kc[s]] = vk[s];   // v^pass
                    sh.vp[kc[s]] = vr[s];  // v^iters
                }
        lds_barrier();
    } else {
        int slot = 0, passes = 0;
        out.lo = lo;
        out.hi = hi;
        lds_barrier();
        while (true) {
            lds_barrier();  // of the next attempt, or the one after the last
            const int dec = __builtin_amdgcn_readfirstlane(sh.dec[slot]);
            if (!(dec & kLvRetry)) {
                const int status = (dec >> kLvStatusShift) - kLvStatus0;
                const double* dr = sh.dm[slot];
                const double* jr = sh.jt[slot];
                const double j = (jr[lane] + jr[lane + 64]) + (jr[lane + 128] + jr[lane + 192]);
                double d = fmax(fmax(dr[lane], dr[lane + 64]), fmax(dr[lane + 128], dr[lane + 192]));
                const double vn = sh.vnext[slot][lane & 7];
                const double J = quad_sum_f64(j, 0.0, 0.0, 0.0);
                d = wave_max_pos_f64(d);
                const double delta = p > 0 ? readlane_d(d, 63) : __builtin_nan("");
                if (lane == 0) {
                    pb.hist_J[p] = J;
                    pb.hist_d[p] = delta;
                    if (pb.times) pb.times[p + 1] = wall_clock64();
                }
                ++passes;
                out.iters = p;
                out.delta = delta;
                out.J = readlane_d(J, 0);
                out.status = status;
                if (status == FCM_RUNNING) {
                    ++p;
                    if (lane < C) pb.hist_v[(int64_t)p * C + lane] = vn;
                }
                if (dec & kLvEnd) break;
            }
            slot = slot == 2 ? 0 : slot + 1;
        }
        if (huge) {  // ended with pass 0: its objective as FP32 terms would make it
            out.J = __builtin_nan("");
            if (lane == 0) pb.hist_J[0] = out.J;
        }
        out.pass = p;
        out.passes = passes;
        out.done = out.status != FCM_RUNNING;
    }
}

}  // namespace fcm
