// Batched solve over the grey levels: many instances in one launch.
//
// One block per tile: it counts the tile's grey levels (fcm_level_dev.h) and
// adds them to its instance's counters; the block that counts an instance's
// last tile iterates the instance to its end.  No block waits for another, so
// the instances overlap freely: while some iterate (five waves of a block,
// latency-bound), other blocks of the same CU count or iterate.  The host
// orders the tiles so that the instances that take most passes come first
// (more clusters converge later): the longest chain of passes starts early
// and the rest fills the other CUs meanwhile.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fcm.h"
#include "fcm_device.h"
#include "fcm_internal.h"
#include "fcm_level.h"
#include "fcm_level_dev.h"

namespace fcm {

namespace {

template <int C>
__device__ __forceinline__ void iterate_c(const LevelProblem& pb, int mclass, uint32_t cnt, LevelScratch& sh,
                                          LevelOutcome& o) {
    if (mclass == kM2)
        level_iterate<C, kM2, false>(pb, cnt, sh, o);
    else if (mclass == kM15)
        level_iterate<C, kM15, false>(pb, cnt, sh, o);
    else
        level_iterate<C, kMGeneric, false>(pb, cnt, sh, o);
}

__device__ __forceinline__ void write_rec(BatchRec* r, const LevelOutcome& o, const LevelScratch& sh, int C) {
    r->pass = o.pass;
    r->done = o.done;
    r->iters = o.iters;
    r->status = o.status;
    r->passes = o.passes;
    r->lo = o.lo;
    r->hi = o.hi;
    r->delta = o.delta;
    r->J = o.J;
    for (int k = 0; k < C; ++k) r->vres[k] = sh.vp[k];
}

__global__ __launch_bounds__(kLvBlock, 4) void fcm_level_batch_kernel(LevelBatchArgs a) {
    __shared__ __align__(16) uint32_t tab[256 * 64];
    __shared__ int s_last;
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid == 0) *a.host_start = wall_clock64();
    const BatchTile tile = a.tiles[blockIdx.x];
    const int i = tile.inst;
    const BatchInst& in = a.inst[i];
    const uint8_t* x = a.x + in.base;
    level_clear(tab);
    __syncthreads();
    char* t8 = reinterpret_cast<char*>(tab);
    level_count(t8, reinterpret_cast<const uint4*>(x + in.head), tile.c0 + tid, tile.c1, kLvBlock);
    if (tile.ragged) level_ragged(t8, x, in.n, in.head, in.nbody);
    __syncthreads();
    uint32_t cnt = level_total(tab);
    const int nt = a.ntiles[i];
    if (nt > 1) {
        uint32_t* counts = a.counts + (int64_t)i * 256;
        if (cnt) {
            // consumed, so the wave goes on only when its add has been performed
            const uint32_t old =
                __hip_atomic_fetch_add(counts + tid, cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::"v"(old));
        }
        __syncthreads();
        if (tid == 0) {
            // as in the single solve: released, and read with atomic loads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const uint32_t prev =
                __hip_atomic_fetch_add(a.ticket + i, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = prev == (uint32_t)nt - 1u;
        }
        __syncthreads();
        if (!s_last) return;
        if (tid < 256) {
            cnt = load_coherent(counts + tid);  // served where the adds were performed
            store_coherent(counts + tid, 0u);
        }
        if (tid == 0) a.ticket[i] = 0u;
    }
    __syncthreads();  // the table is read out: its memory becomes the iteration's scratch
    if (tid >= 64 * kLvIterWaves) return;
    LevelScratch& sh = *reinterpret_cast<LevelScratch*>(tab);
    LevelProblem pb{};
    const int C = __builtin_amdgcn_readfirstlane(in.C), mclass = __builtin_amdgcn_readfirstlane(in.mclass);
    const int64_t rows = (int64_t)in.max_iter + 2;
    pb.eps = in.eps;
    pb.m = a.m[i];
    pb.alpha = 1.0 / (pb.m - 1.0);
    pb.max_iter = in.max_iter;
    pb.max_passes = in.max_iter + 1;
    pb.do_init = 1;
    pb.given = in.given;
    pb.fp32_range = 1;
    pb.n = in.n;
    pb.v0 = in.v0;
    pb.dv0 = in.dv0;
    pb.hist_v = a.hist + in.hist;
    pb.hist_d = pb.hist_v + rows * C;
    pb.hist_J = pb.hist_d + rows;
    pb.times = reinterpret_cast<uint64_t*>(pb.hist_J + rows);
    LevelOutcome o{};
    switch (C) {
        case 2: iterate_c<2>(pb, mclass, cnt, sh, o); break;
        case 3: iterate_c<3>(pb, mclass, cnt, sh, o); break;
        case 4: iterate_c<4>(pb, mclass, cnt, sh, o); break;
        case 5: iterate_c<5>(pb, mclass, cnt, sh, o); break;
        case 6: iterate_c<6>(pb, mclass, cnt, sh, o); break;
        case 7: iterate_c<7>(pb, mclass, cnt, sh, o); break;
        default: iterate_c<8>(pb, mclass, cnt, sh, o); break;
    }
    if (tid >= 256) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (tid == 256) {
            write_rec(a.recs + i, o, sh, C);
            write_rec(a.host_recs + i, o, sh, C);
        }
    }
}

}  // namespace

hipError_t launch_levels_batch(const LevelBatchArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL(fcm_level_batch_kernel, dim3(grid), dim3(kLvBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace fcm
