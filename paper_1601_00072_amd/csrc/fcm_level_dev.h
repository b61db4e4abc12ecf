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

// Count of level t in threads t < 256 after a block-wide call (the first
// 256 threads add the 64 columns of their level, each starting at its own
// column so that a wave's lanes read different banks).
__device__ __forceinline__ uint32_t level_total(const uint32_t* tab) {
    uint32_t c = 0u;
    const uint32_t t = threadIdx.x;
    if (t < 256u) {
        const uint32_t* row = tab + t * 64u;
#pragma unroll 16
        for (uint32_t i = 0; i < 64u; ++i) c += row[(i + t) & 63u];
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
    int32_t pass;             // do_init == 0: index of the next pass (>= 1)
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

// Shared memory of level_iterate (lies over the counting table).  The weights
// u^m h of a wave's 64 levels pass from "lane = level" to "lane = (cluster,
// part of the levels)" through `w`; the row stride keeps both directions free
// of bank conflicts.
template <int C>
struct LevelGeom {
    static constexpr int CP = C <= 2 ? 2 : (C <= 4 ? 4 : 8);  // clusters rounded up
    static constexpr int PARTS = CP == 8 ? 8 : 16;            // lanes that share a cluster's levels
    static constexpr int PER = 64 / PARTS;                    // levels per such lane
    static constexpr int STRIDE = CP == 8 ? 72 : 80;
};

struct LevelScratch {
    double w[4][8 * 80];
    double red[2][8][3][4];   // [pass parity][cluster][num, den, J][wave]
    double dmax[2][4];
    double v[8], vp[8];
    uint64_t mask[4];
    float h[256], a0[256], a1[128], a2[64], tmp[256], y[8];
    double w0[8];
};
static_assert(sizeof(LevelScratch) <= sizeof(LevelTable), "scratch lies over the counting table");

__device__ __forceinline__ double readfirst_d(double v) { return readlane_d(v, 0); }

template <int CTRL>
__device__ __forceinline__ double dpp_add_f64(double v) {
    return v + dpp_mov_f64<CTRL>(v);
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

// Eq.4 and u^m by distance ratios, u_k = w_k / sum_j w_j with
// w_k = (d_min / d_k)^(2/(m-1)) <= 1, and the zero-distance rule (equal split
// over the clusters at distance 0): the form that holds for any centroids.
template <int C>
__device__ __noinline__ void level_u_any(double x, const double* v, double m, double* u, double* a) {
    double d[C];
    double dmin = 1.0e308;
    int nz = 0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        d[k] = fabs(x - v[k]);
        dmin = fmin(dmin, d[k]);
        nz += d[k] == 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        if (nz) {
            u[k] = d[k] == 0.0 ? 1.0 : 0.0;
        } else {
            const double r = dmin / d[k];
            u[k] = m == 2.0 ? r * r : pow(r, 2.0 / (m - 1.0));
        }
        s += u[k];
    }
#pragma unroll
    for (int k = 0; k < C; ++k) {
        u[k] /= s;
        a[k] = m == 2.0 ? u[k] * u[k] : pow(u[k], m);
    }
}

// Memberships u (Eq.4) and a = u^m of grey level x.  With q_k = (x - v_k)^2,
// the m = 2 memberships are u2_k = P_k / sum_j P_j, P_k = prod_{j != k} q_j
// (one reciprocal); other m follow from w_k = u2_k^alpha, u_k = w_k / S,
// S = sum w, and u_k^m = w_k u2_k / S^m because alpha (m - 1) = 1 -- so only
// the generic m needs logarithms, one log2 and one exp2 per cluster.  Two
// centroids on the same level (all P zero) and products out of range take
// the ratio form.
template <int C, int MK>
__device__ __forceinline__ void level_u(double x, const double (&v)[C], double m, double alpha, double (&u)[C],
                                        double (&a)[C]) {
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
    if (!(S > 1.0e-280 && S < 1.0e280)) {
        double cv[C], cu[C], ca[C];  // copies: only they live in memory
#pragma unroll
        for (int k = 0; k < C; ++k) cv[k] = v[k];
        level_u_any<C>(x, cv, m, cu, ca);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = cu[k];
            a[k] = ca[k];
        }
        return;
    }
    const double r = recip_f64(S);
    if constexpr (MK == kM2) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = P[k] * r;
            a[k] = u[k] * u[k];
        }
    } else if constexpr (MK == kM15) {
        double s = 0.0, w[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            P[k] *= r;
            w[k] = P[k] * P[k];
            s += w[k];
        }
        const double rs = recip_f64(s), t = rs * sqrt(rs);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = w[k] * rs;
            a[k] = w[k] * P[k] * t;
        }
    } else {
        double L[C], top = -1.0e300;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            P[k] *= r;
            L[k] = P[k] > 0.0 ? log2(P[k]) : -1.0e300;
            top = fmax(top, L[k]);
        }
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            u[k] = exp2(alpha * (L[k] - top));  // w_k, largest 1
            s += u[k];
        }
        const double rs = recip_f64(s);
        // u^m = w_k (u2_k / u2_max) s^-m
        const double t = exp2(-m * log2(s) - top);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            a[k] = u[k] * P[k] * t;
            u[k] *= rs;
        }
    }
}

// Algorithm 1 on the counts: thread t < 256 holds the count of level t.
// Called by kLvIterWaves waves (the block's other waves have ended).  Waves
// 0..3 own 64 levels each, one per lane; per pass a wave evaluates Eq.4 once
// (U^(p-1) stays in registers), turns its weights through LDS so that a
// cluster's sums need only 3 or 4 cross-lane steps, and writes its partial
// sums; after the pass's only barrier every wave adds the four partial sums
// in wave order and takes the decision itself (same bits in every lane), and
// the fifth wave records it, off the others' path.
template <int C, int MK, bool LEARNED>
__device__ __forceinline__ void level_iterate(const LevelProblem& pb, uint32_t cnt, LevelScratch& sh,
                                              LevelOutcome& out) {
    using Gm = LevelGeom<C>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool work = wid < 4;
    const double c = (double)cnt, x = (double)tid;
    int lo = 0, hi = 255, p = 0;
    double v[C];
    double uo[C];
#pragma unroll
    for (int k = 0; k < C; ++k) uo[k] = 0.0;
    bool huge = false;
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
        if (pb.fp32_range)
#pragma unroll
            for (int k = 0; k < C; ++k) huge = huge || !(fabs(v[k]) < 1.8e19);
        if (wid == 4) {
            if (lane < C) pb.hist_v[lane] = sh.v[lane];
            if (pb.times && lane == 0) pb.times[0] = wall_clock64();
        }
    } else {
        p = pb.pass;
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = readfirst_d(pb.hist_v[(int64_t)p * C + k]);
        if (work && p > 0) {
            double vp[C], t[C];
#pragma unroll
            for (int k = 0; k < C; ++k) vp[k] = pb.hist_v[(int64_t)(p - 1) * C + k];
            level_u<C, MK>(x, vp, pb.m, pb.alpha, uo, t);
        }
    }
    const int part = lane % Gm::PARTS;
    const int kc = lane / Gm::PARTS < C ? lane / Gm::PARTS : C - 1;  // the cluster whose sums this lane adds
    double vk = v[0];  // v[kc]
#pragma unroll
    for (int k = 1; k < C; ++k)
        if (kc == k) vk = v[k];
    double* w = sh.w[work ? wid : 0];
    int status = FCM_RUNNING, passes = 0;
    double delta = __builtin_nan(""), Jt = __builtin_nan("");
    double vr = vk;  // centroid kc of the last pass run
    int last = p;
    for (int budget = pb.max_passes; budget > 0; --budget) {
        const int par = p & 1;
        if (work) {
            double u[C], a[C];
            level_u<C, MK>(x, v, pb.m, pb.alpha, u, a);
            double dm = 0.0;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                w[k * Gm::STRIDE + lane] = c * a[k];
                dm = fmax(dm, fabs(u[k] - uo[k]));
                uo[k] = u[k];
            }
            if (!cnt) dm = 0.0;
            // the wave's own LDS writes are visible to its lanes (in order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            double num = 0.0, den = 0.0, jk = 0.0;
#pragma unroll
            for (int i = 0; i < Gm::PER; ++i) {
                const int l = part + Gm::PARTS * i;
                const double wv = w[kc * Gm::STRIDE + l];
                const double xl = (double)(64 * wid + l), e = xl - vk;
                den += wv;
                num = fma(wv, xl, num);
                jk = fma(wv, e * e, jk);
            }
            num = dpp_add_f64<0xB1>(num);
            den = dpp_add_f64<0xB1>(den);
            jk = dpp_add_f64<0xB1>(jk);
            num = dpp_add_f64<0x4E>(num);
            den = dpp_add_f64<0x4E>(den);
            jk = dpp_add_f64<0x4E>(jk);
            num = dpp_add_f64<0x141>(num);
            den = dpp_add_f64<0x141>(den);
            jk = dpp_add_f64<0x141>(jk);
            if constexpr (Gm::PARTS == 16) {
                num = dpp_add_f64<0x140>(num);
                den = dpp_add_f64<0x140>(den);
                jk = dpp_add_f64<0x140>(jk);
            }
            if (part == 0 && lane < C * Gm::PARTS) {
                sh.red[par][kc][0][wid] = num;
                sh.red[par][kc][1][wid] = den;
                sh.red[par][kc][2][wid] = jk;
            }
            dm = wave_max_pos_f64(dm);
            if (lane == 63) sh.dmax[par][wid] = dm;
        }
        __syncthreads();
        const double* rn = sh.red[par][kc][0];
        const double num = ((rn[0] + rn[1]) + rn[2]) + rn[3];
        const double den = ((rn[4] + rn[5]) + rn[6]) + rn[7];
        const double dmx = fmax(fmax(sh.dmax[par][0], sh.dmax[par][1]), fmax(sh.dmax[par][2], sh.dmax[par][3]));
        const double vn = den > 0.0 ? num / den : vk;
        const bool bad = __any(!isfinite(vn)) || huge;
        const int stop = __builtin_amdgcn_readfirstlane((int)(p >= 1 && dmx < pb.eps));
        status = bad ? FCM_ENUMERIC : (stop ? FCM_OK : (p >= pb.max_iter ? FCM_NOT_CONVERGED : FCM_RUNNING));
        if (!work) {
            const double jk = ((rn[8] + rn[9]) + rn[10]) + rn[11];
            Jt = 0.0;
#pragma unroll
            for (int k = 0; k < C; ++k) Jt += readlane_d(jk, k * Gm::PARTS);
            delta = p > 0 ? dmx : __builtin_nan("");
            if (lane == 0) {
                pb.hist_J[p] = Jt;
                pb.hist_d[p] = delta;
                if (pb.times) pb.times[p + 1] = wall_clock64();
            }
            if (status == FCM_RUNNING && part == 0 && lane < C * Gm::PARTS) pb.hist_v[(int64_t)(p + 1) * C + kc] = vn;
        }
        ++passes;
        last = p;
        vr = vk;
        if (status != FCM_RUNNING) break;
        vk = vn;
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = readlane_d(vn, k * Gm::PARTS);
        ++p;
    }
    if (wid == 4 && part == 0 && lane < C * Gm::PARTS) {
        sh.v[kc] = vk;   // v^pass
        sh.vp[kc] = vr;  // v^iters
    }
    if (wid == 4) {
        out.pass = p;
        out.iters = passes ? last : -1;
        out.passes = passes;
        out.status = status;
        out.done = status != FCM_RUNNING;
        out.lo = lo;
        out.hi = hi;
        out.delta = delta;
        out.J = Jt;
    }
}

}  // namespace fcm
