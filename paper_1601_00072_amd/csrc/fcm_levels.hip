// Solve of one instance over its grey levels: one launch counts the levels of
// the whole input and runs Algorithm 1 on the counts (fcm_level_dev.h).
//
// The blocks count their share of the voxels into LDS and add the 256 counts
// to global counters; the last block to arrive (atomic ticket) takes the
// totals and iterates, the others are gone by then.  Nobody waits for another
// block, so the grid need not be resident at once.  The history and the state
// are written in the same layout as the per-voxel drivers', so results,
// trajectories and labels read the same way and the drivers can be mixed.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fcm.h"
#include "fcm_device.h"
#include "fcm_internal.h"
#include "fcm_level.h"
#include "fcm_level_dev.h"

namespace fcm {

namespace {

// The result fields of a state record (one thread).
template <int C>
__device__ __forceinline__ void level_commit(DevState* st, const LevelArgs& a, const LevelOutcome& o,
                                             const LevelScratch& sh, int64_t total) {
    if (a.do_init) {
        st->lo = o.lo;
        st->hi = o.hi;
    }
    if (o.iters >= 0 || a.do_init) {
        st->pass = o.pass;
        st->iters = o.iters;
        st->passes = o.iters + 1;
        st->status = o.status;
        st->done = o.done;
        st->delta = o.delta;
        st->J = o.J;
        for (int k = 0; k < C; ++k) {
            st->vres[k] = sh.vp[k];
            st->v32[o.pass & 1][k] = (float)sh.v[k];
            st->v32[(o.pass + 1) & 1][k] = (float)sh.vp[k];
        }
    }
    st->sync.passes_total = (uint64_t)total;
}

template <int C, int MK, bool LEARNED>
__global__ __launch_bounds__(kLvBlock, LEARNED ? 2 : 4) void fcm_level_kernel(LevelArgs a) {
    __shared__ __align__(16) uint32_t tab[256 * 64];
    __shared__ int s_last;
    const int tid = threadIdx.x, G = gridDim.x;
    DevState* st = a.st;
    if (!a.do_init && st->done) return;
    level_clear(tab);
    __syncthreads();
    char* t8 = reinterpret_cast<char*>(tab);
    level_count(t8, reinterpret_cast<const uint4*>(a.x + a.head), (int64_t)blockIdx.x * kLvBlock + tid, a.nbody,
                (int64_t)G * kLvBlock);
    if (blockIdx.x == 0) level_ragged(t8, a.x, a.n, a.head, a.nbody);
    __syncthreads();
    uint32_t cnt = level_total(tab);
    if (G > 1) {
        const int copies = G < kLvCopies ? G : kLvCopies;
        if (cnt) {
            // the returned value is consumed, so the wave goes on only when
            // its add has been performed
            const uint32_t old = __hip_atomic_fetch_add(a.counts + (blockIdx.x % copies) * 256 + tid, cnt,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::"v"(old));
        }
        __syncthreads();
        if (tid == 0) {
            // the block's adds have been performed; the release orders them
            // before its arrival.  No acquire on the other side: what the last
            // block reads of the others are the counters, with atomic loads
            // issued after this add's value is known, which are served where
            // the adds were performed (an acquire invalidates the XCD's L2).
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const uint32_t prev =
                __hip_atomic_fetch_add(&st->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = prev == (uint32_t)G - 1u;
        }
        __syncthreads();
        if (!s_last) return;
        if (tid < 256) {
            // atomic loads are served where the adds were performed
            uint32_t part[kLvCopies];
#pragma unroll
            for (int c = 0; c < kLvCopies; ++c) part[c] = load_coherent(a.counts + c * 256 + tid);
            cnt = 0u;
#pragma unroll
            for (int c = 0; c < kLvCopies; ++c) {
                cnt += part[c];
                store_coherent(a.counts + c * 256 + tid, 0u);
            }
        }
        if (tid == 0) st->ticket = 0;
    }
    __syncthreads();  // the table is read out: its memory becomes the iteration's scratch
    if (tid >= 64 * kLvIterWaves) return;
    LevelScratch& sh = *reinterpret_cast<LevelScratch*>(tab);
    LevelProblem pb{};
    pb.eps = a.eps;
    pb.m = a.m;
    pb.alpha = 1.0 / (a.m - 1.0);
    pb.max_iter = a.max_iter;
    pb.max_passes = a.max_passes;
    pb.do_init = a.do_init;
    pb.given = a.given;
    pb.pass = a.do_init ? 0 : st->pass;
    pb.fp32_range = a.fp32_range;
    pb.n = a.n;
    pb.v0 = a.v0;
    pb.dv0 = a.dv0;
    pb.mlp_w = a.mlp_w;
    pb.hist_v = a.hist_v;
    pb.hist_d = a.hist_d;
    pb.hist_J = a.hist_J;
    pb.times = nullptr;
    LevelOutcome o{};
    level_iterate<C, MK, LEARNED>(pb, cnt, sh, o);
    if (tid >= 256) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (tid == 256) {
            const int64_t total = (int64_t)st->sync.passes_total + o.passes;
            if (!a.do_init) {
                o.lo = st->lo;
                o.hi = st->hi;
            }
            level_commit<C>(st, a, o, sh, total);
            level_commit<C>(a.host, a, o, sh, total);
            a.host->lo = o.lo;
            a.host->hi = o.hi;
            // the host may see this before the runtime reports the launch done
            __hip_atomic_store(&a.host->ticket, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

template <int C, bool LEARNED>
hipError_t launch_c(const LevelArgs& a, int mclass, int grid, hipStream_t s) {
    if (mclass == kM2)
        hipLaunchKernelGGL((fcm_level_kernel<C, kM2, LEARNED>), dim3(grid), dim3(kLvBlock), 0, s, a);
    else if (mclass == kM15)
        hipLaunchKernelGGL((fcm_level_kernel<C, kM15, LEARNED>), dim3(grid), dim3(kLvBlock), 0, s, a);
    else
        hipLaunchKernelGGL((fcm_level_kernel<C, kMGeneric, LEARNED>), dim3(grid), dim3(kLvBlock), 0, s, a);
    return hipGetLastError();
}

template <int C>
hipError_t launch_c(const LevelArgs& a, int mclass, int grid, hipStream_t s) {
    return a.do_init && a.given == 3 ? launch_c<C, true>(a, mclass, grid, s) : launch_c<C, false>(a, mclass, grid, s);
}

}  // namespace

hipError_t launch_levels(const LevelArgs& a, int C, int mclass, int grid, hipStream_t s) {
    switch (C) {
        case 2: return launch_c<2>(a, mclass, grid, s);
        case 3: return launch_c<3>(a, mclass, grid, s);
        case 4: return launch_c<4>(a, mclass, grid, s);
        case 5: return launch_c<5>(a, mclass, grid, s);
        case 6: return launch_c<6>(a, mclass, grid, s);
        case 7: return launch_c<7>(a, mclass, grid, s);
        case 8: return launch_c<8>(a, mclass, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fcm
