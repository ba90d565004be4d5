// Batched block passes (k6), around k2_body and K2Interp of k2_device.h.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "k2_device.h"
#include "launch.h"
#include "plan.h"

namespace svk {

// ---------------------------------------------------------------- k6

// One block pass of many states in one launch. Work-group w starts with chunk
// w and takes the next one from the counter *ctr (zero at the start) until none
// is left; chunks come most expensive first, so the launch ends within one
// small chunk's time on every work-group. Every chunk uses the launch's
// work-group size: its block has l = r + log2(threads) local qubits with its
// own register tile r (3 .. LMAX), so a small state runs with smaller tiles
// instead of shrinking every instance's block.
constexpr size_t kK6Tail = 16;  // bytes of LDS after the pass's: the next chunk

template <typename T, int LMAX, bool MFMA>
__global__ void __launch_bounds__((k2_max_threads<T, LMAX>()))
k6_batch_kernel(const svp::BatchPass *passes, const svp::BatchChunk *chunks, unsigned nchunks,
                const svp::K2Op *ops, unsigned *ctr, unsigned lds)
{
    using C = typename CT<T>::type;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    // after the pass's LDS, which then starts at address 0 (a variable of its own is
    // placed first, and every access of the pass gets an addition)
    unsigned &next = *reinterpret_cast<unsigned *>(lds_raw + lds);
    for (unsigned c = blockIdx.x; c < nchunks;) {
        const auto &J = as_const<svp::BatchChunk>(chunks)[c];
        const auto &P = as_const<svp::BatchPass>(passes)[J.pass];
        const K2Interp<MFMA> prog{as_const<svp::K2Op>(ops) + P.op_begin, P.args.nops, P.args.l};
        // no prefetch of the next block: measured no faster here, and its
        // registers would push the interpreter into spills
        auto run = [&](auto logr) {
            k2_body_any<T, decltype(logr)::value, K2Interp<MFMA>, 0>((C *)P.S, P.args, lds_raw, prog, (uint64_t)J.first,
                                                                     (uint64_t)J.stride);
        };
        if (J.logr == 3) run(K2Int<3>{});
        if constexpr (LMAX >= 4)
            if (J.logr == 4) run(K2Int<4>{});
        if constexpr (LMAX >= 5)
            if (J.logr == 5) run(K2Int<5>{});
        __syncthreads();  // this chunk's last reads of LDS; every thread has read next
        if (threadIdx.x == 0) next = gridDim.x + atomicAdd(ctr, 1u);
        __syncthreads();
        c = __builtin_amdgcn_readfirstlane(next);
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
    lds += kK6Tail;
    if (lds > 64 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return 0;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)threads, lds) != hipSuccess) return 0;
    return per_cu;
}

hipError_t k6_batch(int dtype, int lmax, unsigned grid, unsigned threads, size_t lds, const svp::BatchPass *passes,
                    const svp::BatchChunk *chunks, unsigned nchunks, const svp::K2Op *ops, unsigned *ctr, bool mfma,
                    hipStream_t st)
{
    const void *fn = dtype == 0 ? k6_fn<float>(lmax, mfma) : k6_fn<double>(lmax, mfma);
    if (!fn) return hipErrorInvalidValue;
    unsigned tail = (unsigned)lds;
    void *args[] = {&passes, &chunks, &nchunks, &ops, &ctr, &tail};
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), args, lds + kK6Tail, st);
}

}  // namespace svk
