// The interpreted block pass (k2), around k2_body and K2Interp of k2_device.h.
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
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    // the build with matrix-core windows keeps no prefetch set (registers)
    k2_body_any<T, LOGR, K2Interp<MFMA>, MFMA ? 0 : 1>(S, args, lds_raw,
                                                        K2Interp<MFMA>{as_const<svp::K2Op>(ops), args.nops, args.l},
                                                        blockIdx.x, gridDim.x);
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
