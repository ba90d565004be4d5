// Block-pass kernels: the interpreted pass (k2) and the batched passes (k6),
// both around k2_body and K2Interp of k2_device.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "k2_device.h"
#include "launch.h"
#include "plan.h"

namespace svk {

// ---------------------------------------------------------------- k2

// Interpreted block pass: the op list of the pass runs on every block (see
// k2_body and K2Interp in k2_device.h).
template <typename T, int LOGR, bool MFMA>
__global__ void __launch_bounds__((k2_max_threads<T, LOGR>()))
k2_kernel(typename CT<T>::type *__restrict__ S, const svp::K2Op *__restrict__ ops, svp::K2Args args)
{
    extern __shared__ unsigned char lds_raw[];
    // the build with matrix-core windows keeps no prefetch set (registers)
    k2_body_any<T, LOGR, K2Interp<MFMA>, MFMA ? 0 : 1>(S, args, lds_raw, K2Interp<MFMA>{ops, args.nops, args.l},
                                                        blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------- k6

// Barrier of the work-groups that share one instance. Thread 0 releases the
// group's stores device-wide, counts itself in, and waits (bounded) until the
// count reaches `target`; a wait that exceeds `limit` polls, or an error
// raised by another group, sets *err and makes every waiter leave, so the
// grid always drains.
__device__ __forceinline__ bool group_barrier(unsigned *ctr, unsigned target, int *err, unsigned limit, int *ok)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicAdd(ctr, 1u);
        unsigned spins = 0;
        int good = 1;
        while (__hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > limit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                atomicExch(err, 1);
                good = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        __threadfence();
        *ok = good;
    }
    __syncthreads();
    // the same for every thread after the barrier: read as a uniform value,
    // so that code after a barrier stays uniform for the compiler too
    return __builtin_amdgcn_readfirstlane(*ok) != 0;
}

// The passes of one instance on this work-group's share of its blocks
// (rank among group_size work-groups). Work-groups that share an instance
// meet at the counter barrier between passes; a work-group that runs an
// instance alone meets its own waves there, since the next pass reads what
// other waves stored.
template <typename T, int LOGR, bool MFMA>
__device__ __forceinline__ bool k6_run(const svp::BatchInst &I, uint64_t rank, const svp::BatchPass *__restrict__ passes,
                       const svp::K2Op *__restrict__ ops, unsigned *ctrs, int *err, unsigned limit,
                       unsigned char *lds, int *ok)
{
    using C = typename CT<T>::type;
    for (int p = 0; p < I.npass; ++p) {
        const svp::BatchPass &P = passes[I.pass_off + p];
        // no prefetch of the next block: measured no faster here, and its
        // registers would push the interpreter into spills
        k2_body_any<T, LOGR, K2Interp<MFMA>, 0>((C *)I.S, P.args, lds,
                                                 K2Interp<MFMA>{ops + P.op_begin, P.args.nops, P.args.l}, rank,
                                                 (uint64_t)I.group_size);
        if (p + 1 == I.npass) break;
        if (I.group_size > 1) {
            if (!group_barrier(&ctrs[I.ctr], (unsigned)((p + 1) * I.group_size), err, limit, ok)) return false;
        } else {
            __syncthreads();
        }
    }
    return true;
}

// Many states in one persistent launch. Work-group w runs the jobs
// wg_off[w] .. wg_off[w+1]-1 in order; a job is (instance, rank). An
// instance spread over several work-groups is their only job; small
// instances are packed several to a work-group. Every instance uses the
// launch's work-group size: its block has l = r + log2(threads) local qubits
// with its own register tile r (I.logr, 3 .. LMAX), so a small state runs
// with smaller tiles instead of shrinking every instance's block.
template <typename T, int LMAX, bool MFMA>
__global__ void __launch_bounds__((k2_max_threads<T, LMAX>()))
k6_batch_kernel(const svp::BatchInst *__restrict__ insts, const int32_t *__restrict__ wg_off,
                const int2 *__restrict__ jobs, const svp::BatchPass *__restrict__ passes,
                const svp::K2Op *__restrict__ ops, unsigned *ctrs, int *err, unsigned limit)
{
    extern __shared__ unsigned char lds_raw[];
    __shared__ int ok;
    const int j0 = wg_off[blockIdx.x], j1 = wg_off[blockIdx.x + 1];
    for (int j = j0; j < j1; ++j) {
        if (j > j0) __syncthreads();  // the previous job's last reads of LDS
        const int2 J = jobs[j];
        const svp::BatchInst I = insts[J.x];
        bool good = true;
        if (I.logr == 3) good = k6_run<T, 3, MFMA>(I, (uint64_t)J.y, passes, ops, ctrs, err, limit, lds_raw, &ok);
        if constexpr (LMAX >= 4)
            if (I.logr == 4) good = k6_run<T, 4, MFMA>(I, (uint64_t)J.y, passes, ops, ctrs, err, limit, lds_raw, &ok);
        if constexpr (LMAX >= 5)
            if (I.logr == 5) good = k6_run<T, 5, MFMA>(I, (uint64_t)J.y, passes, ops, ctrs, err, limit, lds_raw, &ok);
        if (!good) return;
    }
}

__global__ void __launch_bounds__(256) zero_u32_kernel(unsigned *p, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

hipError_t zero_u32(unsigned *p, uint32_t n, hipStream_t st)
{
    zero_u32_kernel<<<grid_for(n, 256, 1024), 256, 0, st>>>(p, n);
    return hipGetLastError();
}

template <typename T>
static const void *k6_fn(int lmax, bool mfma)
{
    switch (lmax * 2 + (mfma ? 1 : 0)) {
    case 6: return (const void *)k6_batch_kernel<T, 3, false>;
    case 7: return (const void *)k6_batch_kernel<T, 3, true>;
    case 8: return (const void *)k6_batch_kernel<T, 4, false>;
    case 9: return (const void *)k6_batch_kernel<T, 4, true>;
    case 10: return (const void *)k6_batch_kernel<T, 5, false>;
    case 11: return (const void *)k6_batch_kernel<T, 5, true>;
    default: return nullptr;
    }
}

int k6_max_threads(int dtype, int lmax)
{
    if (lmax < 3 || lmax > 5) return 0;
    const int bumped = lmax + (dtype == 0 ? 0 : 1);
    return bumped >= 5 ? (bumped >= 6 ? 256 : 512) : 1024;
}

int k6_occupancy(int dtype, int lmax, unsigned threads, size_t lds, bool mfma)
{
    const void *fn = dtype == 0 ? k6_fn<float>(lmax, mfma) : k6_fn<double>(lmax, mfma);
    if (!fn) return 0;
    if (lds > 64 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return 0;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)threads, lds) != hipSuccess) return 0;
    return per_cu;
}

hipError_t k6_batch(int dtype, int lmax, unsigned grid, unsigned threads, size_t lds, const svp::BatchInst *insts,
                    const int32_t *wg_off, const void *jobs, const svp::BatchPass *passes, const svp::K2Op *ops,
                    unsigned *ctrs, int *err, unsigned limit, bool mfma, hipStream_t st)
{
    const void *fn = dtype == 0 ? k6_fn<float>(lmax, mfma) : k6_fn<double>(lmax, mfma);
    if (!fn) return hipErrorInvalidValue;
    void *args[] = {&insts, &wg_off, &jobs, &passes, &ops, &ctrs, &err, &limit};
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), args, lds, st);
}

template <typename T, int LOGR, bool MFMA>
static hipError_t k2_launch_t(void *S, const K2Args &a, const svp::K2Op *ops, hipStream_t st)
{
    using C = typename CT<T>::type;
    const size_t lds = svp::k2_lds_layout(a.l, (int)sizeof(C), a.nug, a.tab_count, a.nut, a.half_lds).total;
    static size_t attr_bytes = 64 * 1024;
    if (lds > attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void *)k2_kernel<T, LOGR, MFMA>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_bytes = lds;
    }
    const unsigned threads = 1u << (a.l - LOGR);
    const uint64_t blocks = 1ull << a.nblk_bits;
    if (threads > (unsigned)k2_max_threads<T, LOGR>()) return hipErrorInvalidConfiguration;
    // persistent grid: as many work-groups as fit on the device at once
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
    }
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k2_kernel<T, LOGR, MFMA>,
                                                                (int)threads, lds);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    const uint64_t grid = svp::k2_grid((uint64_t)per_cu * (uint64_t)cus, blocks);
    k2_kernel<T, LOGR, MFMA><<<(unsigned)grid, threads, lds, st>>>((C *)S, ops, a);
    return hipGetLastError();
}

template <typename T, bool MFMA>
static hipError_t k2_dispatch(void *S, int logr, const K2Args &a, const svp::K2Op *ops, hipStream_t st)
{
    switch (logr) {
    case 1: return k2_launch_t<T, 1, MFMA>(S, a, ops, st);
    case 2: return k2_launch_t<T, 2, MFMA>(S, a, ops, st);
    case 3: return k2_launch_t<T, 3, MFMA>(S, a, ops, st);
    case 4: return k2_launch_t<T, 4, MFMA>(S, a, ops, st);
    case 5: return k2_launch_t<T, 5, MFMA>(S, a, ops, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t k2_pass(void *S, int n, int dtype, int logr, const K2Args &a, const svp::K2Op *ops, bool mfma,
                   hipStream_t st)
{
    if (a.l < logr || a.l > n || logr < 1) return hipErrorInvalidValue;
    if (mfma)
        return dtype == 0 ? k2_dispatch<float, true>(S, logr, a, ops, st)
                          : k2_dispatch<double, true>(S, logr, a, ops, st);
    return dtype == 0 ? k2_dispatch<float, false>(S, logr, a, ops, st)
                      : k2_dispatch<double, false>(S, logr, a, ops, st);
}

}  // namespace svk
