// Persistent batched executor of one precision.
#pragma once

#include "batch_tasks.hpp"

namespace psv {
namespace {

// Persistent executor. Tasks are int4 {problem, level, tile, tiles of the
// previous level of that problem}; the queue holds every level of every
// problem, level by level, problems largest first, so whatever a task waits
// for was dequeued earlier by a running block and the wait always ends.
// A wait that exceeds the spin budget sets *error and the block carries on
// (the kernel always drains); the host then reports the failure.
constexpr long long SPIN_LIMIT = 1ll << 22;  // x s_sleep(2): well above any legitimate wait

template <typename T>
__device__ __forceinline__ void run_kind(int kind, const ProblemDesc& D, const ProblemIO& io, int b,
                                         unsigned char* smem, double* red) {
    switch (kind) {
#define PSV_K(k) case k: run_task<T, k>(D, io, b, smem, red); break;
        PSV_K(K_MINP) PSV_K(K_MINF) PSV_K(K_FWD) PSV_K(K_MEAN) PSV_K(K_Y) PSV_K(K_Z) PSV_K(K_Z2)
        PSV_K(K_YI) PSV_K(K_INV) PSV_K(K_INVADD) PSV_K(K_RES) PSV_K(K_NRM) PSV_K(K_CHK)
        PSV_K(K_CHKF)
#undef PSV_K
        default: break;
    }
}

// Tickets hand out TICKET_TASKS consecutive tasks at a time. The queue is
// ordered by pass, so a run of tasks usually shares its (problem, pass): the
// block waits on that group's dependency once and releases its completions
// with one counter update. The smallest unfinished task always has its
// dependencies (earlier in the queue) done and is the current task of its
// block, so the executor cannot deadlock.
// Synchronisation is costly on a multi-XCD GPU: each XCD has its own L2, so
// a release at device scope writes the L2's dirty lines back and an acquire
// invalidates the caches. Only thread 0 of a block releases (one atomic per
// run of completions, no separate fence) and acquires (the wait's atomic
// load, then a block barrier). Longer tickets mean fewer of both but leave
// fewer blocks working on each pass while the others wait on it: on a batch
// of 64 problems of 0.26-3.1 million cells, 8 tasks per ticket took 25.6 ms,
// 4 took 29.2, 32 took 30.6 and 128 took 57.5.
constexpr int TICKET_TASKS = 8;

template <typename T>
__global__ void __launch_bounds__(256) k_batch_persistent(PersistArgs A) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[16];
    __shared__ int s_task;
    for (;;) {
        __syncthreads();  // the previous task is done with LDS and s_task
        if (threadIdx.x == 0) s_task = atomicAdd(A.ticket, A.chunk);
        __syncthreads();
        const int t0 = s_task;
        if (t0 >= A.ntasks) break;
        const int t1 = min(t0 + A.chunk, A.ntasks);
        int* cnt_done = nullptr;  // counter of the group whose completions are pending
        int pending = 0;
        for (int t = t0; t < t1; ++t) {
            const int4 tk = A.tasks[t];
            int* cnt = A.counters + (size_t)tk.x * A.nlevels;
            if (cnt + tk.y != cnt_done) {
                if (pending && threadIdx.x == 0)
                    __hip_atomic_fetch_add(cnt_done, pending, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                pending = 0;
                cnt_done = cnt + tk.y;
                if (threadIdx.x == 0 && tk.y > 0) {
                    long long spins = 0;
                    while (__hip_atomic_load(cnt + tk.y - 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < tk.w) {
                        __builtin_amdgcn_s_sleep(2);
                        if (++spins > SPIN_LIMIT) {
                            atomicOr(A.error, 1);
                            break;
                        }
                        // once any wait has failed, no block waits again: the drain is bounded
                        if ((spins & 255) == 0 &&
                            __hip_atomic_load(A.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                            break;
                    }
                }
                __syncthreads();  // thread 0's acquire covers the block (one L1 per CU)
            }
            run_kind<T>(A.kinds[tk.y], A.desc[tk.x], A.io[tk.x], tk.z, smem_raw, red);
            __syncthreads();  // the tile is complete and its LDS free
            ++pending;
        }
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(cnt_done, pending, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <typename T>
void launch_queue(const PersistArgs& A, size_t lds, int device, hipStream_t s) {
    int per_cu = 0, ncu = 0;
    allow_lds(k_batch_persistent<T>, lds);
    PSV_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch_persistent<T>, 256, lds));
    PSV_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device));
    PersistArgs a = A;
    a.chunk = TICKET_TASKS;
    hipLaunchKernelGGL(k_batch_persistent<T>, dim3(std::max(1, std::min(per_cu, 8) * ncu)), dim3(256),
                       lds, s, a);
    PSV_HIP(hipGetLastError());
}

}  // namespace
}  // namespace psv
