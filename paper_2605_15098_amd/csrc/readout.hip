// Readout kernels: bandwidth probe, FP64 probabilities, marginals, argmax and
// norm (k5), measurement, and logical-order export and import of the state.
// Indices are physical, sto() gives the storage index (k2_device.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>

#include "k2_device.h"
#include "launch.h"
#include "plan.h"

namespace svk {

// ---------------------------------------------------------------- measurement

// Inclusive prefix sums of FP64 values in a fixed order (deterministic):
// tiles of SCAN_TILE values, each thread summing SCAN_PER consecutive values,
// a work-group scan of the thread sums, then the tiles' totals scanned the
// same way (recursively) and added back.
constexpr int SCAN_THREADS = 256, SCAN_PER = 8, SCAN_TILE = SCAN_THREADS * SCAN_PER;

__device__ double block_exclusive_scan(double v, double *sh, double *total)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int d = 1; d < SCAN_THREADS; d <<= 1) {
        const double x = t >= d ? sh[t - d] : 0.0;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    const double incl = sh[t];
    *total = sh[SCAN_THREADS - 1];
    __syncthreads();
    return incl - v;
}

__global__ void __launch_bounds__(SCAN_THREADS) scan_tiles(const double *__restrict__ in, double *__restrict__ out,
                                                            uint64_t m, double *__restrict__ tile_sums)
{
    __shared__ double sh[SCAN_THREADS];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_PER;
    double v[SCAN_PER], s = 0.0;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) {
        v[k] = base + k < m ? in[base + k] : 0.0;
        s += v[k];
        v[k] = s;
    }
    double total;
    const double off = block_exclusive_scan(s, sh, &total);
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k)
        if (base + k < m) out[base + k] = off + v[k];
    if (threadIdx.x == 0 && tile_sums) tile_sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(SCAN_THREADS) scan_add(double *__restrict__ out, uint64_t m,
                                                          const double *__restrict__ tile_incl)
{
    if (blockIdx.x == 0) return;
    const double off = tile_incl[blockIdx.x - 1];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_PER;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k)
        if (base + k < m) out[base + k] += off;
}

size_t scan_scratch_bytes(uint64_t m)
{
    size_t b = 0;
    for (uint64_t x = (m + SCAN_TILE - 1) / SCAN_TILE; x > 1; x = (x + SCAN_TILE - 1) / SCAN_TILE) b += x * 8;
    return b + 64;
}

hipError_t scan_inclusive(const double *in, double *out, uint64_t m, void *scratch, hipStream_t st)
{
    const uint64_t tiles = (m + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles > 0xffffffffull) return hipErrorInvalidValue;
    double *sums = tiles > 1 ? (double *)scratch : nullptr;
    scan_tiles<<<(unsigned)tiles, SCAN_THREADS, 0, st>>>(in, out, m, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || tiles <= 1) return e;
    e = scan_inclusive(sums, sums, tiles, (double *)scratch + tiles, st);
    if (e != hipSuccess) return e;
    scan_add<<<(unsigned)tiles, SCAN_THREADS, 0, st>>>(out, m, sums);
    return hipGetLastError();
}

// Inverse CDF: the smallest m with cdf[m] > u * cdf[M - 1] (clamped to M - 1).
__global__ void __launch_bounds__(256) sample_search(const double *__restrict__ cdf, uint64_t M,
                                                     const double *__restrict__ u, uint64_t shots,
                                                     uint64_t *__restrict__ out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= shots) return;
    const double target = u[i] * cdf[M - 1];
    uint64_t lo = 0, hi = M;  // first index in [lo, hi) with cdf > target
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (cdf[mid] > target) hi = mid;
        else lo = mid + 1;
    }
    out[i] = lo < M ? lo : M - 1;
}

hipError_t sample_outcomes(const double *cdf, uint64_t M, const double *u, uint64_t shots, uint64_t *out,
                           hipStream_t st)
{
    if (shots == 0) return hipSuccess;
    sample_search<<<grid_for(shots, 256, 0x7fffffffu), 256, 0, st>>>(cdf, M, u, shots, out);
    return hipGetLastError();
}

// Projective collapse over the storage order: amplitudes whose physical
// bits in `mask` differ from `val` become 0, the others are scaled.
template <typename C>
__global__ void __launch_bounds__(256) collapse_kernel(C *__restrict__ S, uint64_t N, uint64_t mask, uint64_t val,
                                                       double scale)
{
    using T = decltype(C::x);
    const T sc = (T)scale;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const uint64_t p = sto<C>(i);  // storage position i holds physical index sto(i)
        C a = S[i];
        if ((p & mask) != val) {
            a.x = 0;
            a.y = 0;
        } else {
            a.x *= sc;
            a.y *= sc;
        }
        S[i] = a;
    }
}

hipError_t collapse(void *S, int n, int dtype, uint64_t mask, uint64_t val, double scale, hipStream_t st)
{
    const uint64_t N = 1ull << n;
    const unsigned g = grid_for(N, 256, 16384);
    if (dtype == 0) collapse_kernel<float2><<<g, 256, 0, st>>>((float2 *)S, N, mask, val, scale);
    else collapse_kernel<double2><<<g, 256, 0, st>>>((double2 *)S, N, mask, val, scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------- bandwidth probe

// Plain HBM streams, the reference for the block passes' bandwidth: mode 0
// copies src to dst, mode 1 rewrites dst in place (read and write of the
// same addresses, as a block pass does). 16-byte accesses, four in flight
// per thread, grid-stride over whole-device work-groups.
__global__ void __launch_bounds__(256) stream_probe_kernel(float4 *__restrict__ dst, const float4 *__restrict__ src,
                                                            uint64_t n16, float scale)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = src[i + k * stride];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k].x *= scale;
            v[k].y *= scale;
            v[k].z *= scale;
            v[k].w *= scale;
            dst[i + k * stride] = v[k];
        }
    }
    for (; i < n16; i += stride) {
        float4 v = src[i];
        v.x *= scale;
        v.y *= scale;
        v.z *= scale;
        v.w *= scale;
        dst[i] = v;
    }
}

hipError_t stream_probe(void *dst, const void *src, uint64_t bytes, int mode, hipStream_t st)
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const uint64_t n16 = bytes / 16;
    const unsigned grid = grid_for(n16, 256, (unsigned)cus * 8u);
    stream_probe_kernel<<<grid, 256, 0, st>>>((float4 *)dst, (const float4 *)(mode == 1 ? dst : src), n16, 1.0f);
    return hipGetLastError();
}

// ---------------------------------------------------------------- k5 readouts

struct PermArg {
    int8_t p[48];
    int n;
    int ident;
};

static PermArg make_perm(const int *perm, int n)
{
    PermArg pa{};
    pa.n = n;
    pa.ident = 1;
    for (int q = 0; q < n; ++q) {
        pa.p[q] = (int8_t)(perm ? perm[q] : q);
        if (pa.p[q] != q) pa.ident = 0;
    }
    return pa;
}

__device__ __forceinline__ uint64_t phys_of(uint64_t x, const PermArg &pa)
{
    if (pa.ident) return x;
    uint64_t p = 0;
    for (int q = 0; q < pa.n; ++q) p |= ((x >> q) & 1ull) << pa.p[q];
    return p;
}

template <typename C> __device__ __forceinline__ double prob(C a)
{
    const double re = (double)a.x, im = (double)a.y;
    return re * re + im * im;
}

template <typename C>
__global__ void __launch_bounds__(256)
probs_kernel(const C *__restrict__ S, PermArg pa, double *__restrict__ out, uint64_t off, uint64_t cnt)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride)
        out[i] = prob(S[sto<C>(phys_of(off + i, pa))]);
}

hipError_t probabilities(const void *S, int n, int dtype, const int *perm, double *out,
                         uint64_t offset, uint64_t count, hipStream_t st)
{
    const PermArg pa = make_perm(perm, n);
    const unsigned g = grid_for(count, 256, 16384);
    if (dtype == 0) probs_kernel<float2><<<g, 256, 0, st>>>((const float2 *)S, pa, out, offset, count);
    else probs_kernel<double2><<<g, 256, 0, st>>>((const double2 *)S, pa, out, offset, count);
    return hipGetLastError();
}

struct BitList {
    int8_t b[48];
    int cnt;
    int low;  // 1: b[k] == k + first (the bits form one contiguous run), first = b[0]
};

// Place bit k of v at position bl.b[k]. A contiguous run is one shift.
__device__ __forceinline__ uint64_t deposit(uint64_t v, const BitList &bl)
{
    if (bl.low) return bl.cnt ? (v << bl.b[0]) : 0ull;
    uint64_t r = 0;
    for (int k = 0; k < bl.cnt; ++k) r |= ((v >> k) & 1ull) << bl.b[k];
    return r;
}

// Each thread owns one marginal entry m and sums its 2^(n-nq) terms in order.
template <typename C>
__global__ void __launch_bounds__(256)
marg_direct_kernel(const C *__restrict__ S, BitList qb, BitList ob, double *__restrict__ out)
{
    const uint64_t M = 1ull << qb.cnt, O = 1ull << ob.cnt;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t m = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; m < M; m += stride) {
        const uint64_t bm = deposit(m, qb);
        double s = 0.0;
        for (uint64_t o = 0; o < O; ++o) s += prob(S[sto<C>(bm | deposit(o, ob))]);
        out[m] = s;
    }
}

// Small marginals: work-group (m, g) reduces chunk g of m's terms; the
// partials are then summed in fixed order. Deterministic.
constexpr int MARG_G = 256;

template <typename C>
__global__ void __launch_bounds__(256)
marg_chunk_kernel(const C *__restrict__ S, BitList qb, BitList ob, double *__restrict__ part)
{
    __shared__ double red[256];
    const uint64_t m = blockIdx.y;
    const uint64_t O = 1ull << ob.cnt;
    const uint64_t per = (O + MARG_G - 1) / MARG_G;
    const uint64_t o0 = (uint64_t)blockIdx.x * per;
    uint64_t o1 = o0 + per;
    if (o1 > O) o1 = O;
    const uint64_t bm = deposit(m, qb);
    double s = 0.0;
    for (uint64_t o = o0 + threadIdx.x; o < o1; o += blockDim.x) s += prob(S[sto<C>(bm | deposit(o, ob))]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[m * MARG_G + blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) marg_finish_kernel(const double *__restrict__ part, uint64_t M,
                                                          double *__restrict__ out)
{
    const uint64_t m = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    double s = 0.0;
    for (int g = 0; g < MARG_G; ++g) s += part[m * MARG_G + g];
    out[m] = s;
}

static BitList make_bits(const int *b, int cnt)
{
    BitList bl{};
    bl.cnt = cnt;
    bl.low = 1;
    for (int k = 0; k < cnt; ++k) {
        bl.b[k] = (int8_t)b[k];
        if (b[k] != b[0] + k) bl.low = 0;
    }
    return bl;
}

size_t marginal_scratch_bytes(int n, int nq)
{
    if (n - nq <= 12) return 0;
    return (size_t)sizeof(double) * MARG_G << nq;
}

template <typename C>
static hipError_t marginal_t(const C *S, int n, const int *qbits, int nq, const int *obits,
                             double *out, void *scratch, hipStream_t st)
{
    const BitList qb = make_bits(qbits, nq), ob = make_bits(obits, n - nq);
    const uint64_t M = 1ull << nq;
    if (n - nq <= 12) {
        marg_direct_kernel<C><<<grid_for(M, 256, 65535), 256, 0, st>>>(S, qb, ob, out);
        return hipGetLastError();
    }
    if (M > 65535) return hipErrorInvalidValue;
    double *part = (double *)scratch;
    dim3 grid(MARG_G, (unsigned)M);
    marg_chunk_kernel<C><<<grid, 256, 0, st>>>(S, qb, ob, part);
    marg_finish_kernel<<<grid_for(M, 256, 65535), 256, 0, st>>>(part, M, out);
    return hipGetLastError();
}

hipError_t marginal(const void *S, int n, int dtype, const int *qbits, int nq, const int *obits,
                    double *out, void *scratch, hipStream_t st)
{
    return dtype == 0 ? marginal_t((const float2 *)S, n, qbits, nq, obits, out, scratch, st)
                      : marginal_t((const double2 *)S, n, qbits, nq, obits, out, scratch, st);
}

// argmax with the lowest index winning ties
__device__ __forceinline__ bool better(double v1, uint64_t i1, double v2, uint64_t i2)
{
    return v1 > v2 || (v1 == v2 && i1 < i2);
}

constexpr int AM_BLOCKS = 8192;

__device__ void block_argmax(double v, uint64_t i, double *rv, uint64_t *ri, double *outv, uint64_t *outi)
{
    __shared__ double sv[256];
    __shared__ uint64_t si[256];
    sv[threadIdx.x] = v;
    si[threadIdx.x] = i;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            const double v2 = sv[threadIdx.x + w];
            const uint64_t i2 = si[threadIdx.x + w];
            if (better(v2, i2, sv[threadIdx.x], si[threadIdx.x])) {
                sv[threadIdx.x] = v2;
                si[threadIdx.x] = i2;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *outv = sv[0];
        *outi = si[0];
    }
    (void)rv;
    (void)ri;
}

__global__ void __launch_bounds__(256) argmax_stage1(const double *__restrict__ p, uint64_t len,
                                                     double *pv, uint64_t *pi)
{
    double bv = -1.0;
    uint64_t bi = ~0ull;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += stride)
        if (better(p[i], i, bv, bi)) { bv = p[i]; bi = i; }
    block_argmax(bv, bi, nullptr, nullptr, &pv[blockIdx.x], &pi[blockIdx.x]);
}

__global__ void __launch_bounds__(256) argmax_stage2(const double *pv, const uint64_t *pi, int nparts,
                                                     uint64_t *res_idx, double *res_val)
{
    double bv = -1.0;
    uint64_t bi = ~0ull;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x)
        if (better(pv[i], pi[i], bv, bi)) { bv = pv[i]; bi = pi[i]; }
    block_argmax(bv, bi, nullptr, nullptr, res_val, res_idx);
}

size_t argmax_scratch_bytes(uint64_t) { return (size_t)AM_BLOCKS * (sizeof(double) + sizeof(uint64_t)); }

hipError_t argmax(const double *p, uint64_t len, void *scratch, uint64_t *res_idx, double *res_val,
                  hipStream_t st)
{
    double *pv = (double *)scratch;
    uint64_t *pi = (uint64_t *)(pv + AM_BLOCKS);
    const unsigned g = grid_for(len, 256, AM_BLOCKS);
    argmax_stage1<<<g, 256, 0, st>>>(p, len, pv, pi);
    argmax_stage2<<<1, 256, 0, st>>>(pv, pi, (int)g, res_idx, res_val);
    return hipGetLastError();
}

// The marginal's physical bits in ascending order, as runs of consecutive
// bits (a permuted layout usually leaves one or two), and the logical bit of
// each: the marginal is walked in memory order so that neighbouring threads
// read neighbouring amplitudes, and the logical index is formed only for
// entries that can win.
struct PhysMarg {
    int8_t src[48], dst[48], len[48];  // run r: bits src..src+len-1 of p -> dst..
    int8_t lbit[48];                   // logical bit of the k-th physical bit (ascending)
    int nruns, cnt;
};

__device__ __forceinline__ uint64_t deposit_runs(uint64_t p, const PhysMarg &q)
{
    uint64_t r = 0;
    for (int k = 0; k < q.nruns; ++k) r |= ((p >> q.src[k]) & ((1ull << q.len[k]) - 1ull)) << q.dst[k];
    return r;
}

template <typename C>
__global__ void __launch_bounds__(256) marg_argmax_stage1(const C *__restrict__ S, PhysMarg qm, BitList ob,
                                                          double *pv, uint64_t *pi)
{
    const uint64_t M = 1ull << qm.cnt, O = 1ull << ob.cnt;
    double bv = -1.0;
    uint64_t bi = ~0ull;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < M; p += stride) {
        const uint64_t bm = deposit_runs(p, qm);
        double s = 0.0;
        for (uint64_t o = 0; o < O; ++o) s += prob(S[sto<C>(bm | deposit(o, ob))]);
        if (s >= bv) {
            uint64_t m = 0;
            for (int k = 0; k < qm.cnt; ++k) m |= ((p >> k) & 1ull) << qm.lbit[k];
            if (better(s, m, bv, bi)) { bv = s; bi = m; }
        }
    }
    block_argmax(bv, bi, nullptr, nullptr, &pv[blockIdx.x], &pi[blockIdx.x]);
}

// Scratch of the allocation-free readout: partial maxima of the fused
// marginal/argmax kernels, then the result (index, value). One copy per GPU
// for the life of the process; in host code the name below is not a device
// address: kernels get the per-device address from static_scratch().
constexpr size_t kStaticScratchBytes = (size_t)AM_BLOCKS * (sizeof(double) + sizeof(uint64_t)) + 256;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t static_scratch_bytes() { return kStaticScratchBytes; }

hipError_t static_scratch(void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = ptr;
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t marginal_argmax(const void *S, int n, int dtype, const int *qbits, int nq, const int *obits,
                           void *scratch, uint64_t *res_idx, double *res_val, hipStream_t st)
{
    const BitList ob = make_bits(obits, n - nq);
    PhysMarg qm{};
    qm.cnt = nq;
    {
        int order[64];
        for (int j = 0; j < nq; ++j) order[j] = j;
        for (int a = 1; a < nq; ++a)  // ascending physical bit
            for (int b = a; b > 0 && qbits[order[b]] < qbits[order[b - 1]]; --b) {
                const int t = order[b];
                order[b] = order[b - 1];
                order[b - 1] = t;
            }
        for (int k = 0; k < nq; ++k) {
            qm.lbit[k] = (int8_t)order[k];
            const int phys = qbits[order[k]];
            if (qm.nruns > 0 && qm.dst[qm.nruns - 1] + qm.len[qm.nruns - 1] == phys) {
                qm.len[qm.nruns - 1] += 1;
            } else {
                qm.src[qm.nruns] = (int8_t)k;
                qm.dst[qm.nruns] = (int8_t)phys;
                qm.len[qm.nruns] = 1;
                qm.nruns += 1;
            }
        }
    }
    double *pv = (double *)scratch;
    uint64_t *pi = (uint64_t *)(pv + AM_BLOCKS);
    const unsigned g = grid_for(1ull << nq, 256, AM_BLOCKS);
    if (dtype == 0) marg_argmax_stage1<float2><<<g, 256, 0, st>>>((const float2 *)S, qm, ob, pv, pi);
    else marg_argmax_stage1<double2><<<g, 256, 0, st>>>((const double2 *)S, qm, ob, pv, pi);
    argmax_stage2<<<1, 256, 0, st>>>(pv, pi, (int)g, res_idx, res_val);
    return hipGetLastError();
}

template <typename C>
__global__ void __launch_bounds__(256) norm_stage1(const C *__restrict__ S, uint64_t N, double *part)
{
    __shared__ double red[256];
    double s = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) s += prob(S[i]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) norm_stage2(const double *part, int nparts, double *res)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *res = red[0];
}

size_t norm_scratch_bytes(int) { return (size_t)AM_BLOCKS * sizeof(double); }

hipError_t norm2(const void *S, int n, int dtype, void *scratch, double *res, hipStream_t st)
{
    const uint64_t N = 1ull << n;
    const unsigned g = grid_for(N, 256, AM_BLOCKS);
    double *part = (double *)scratch;
    if (dtype == 0) norm_stage1<float2><<<g, 256, 0, st>>>((const float2 *)S, N, part);
    else norm_stage1<double2><<<g, 256, 0, st>>>((const double2 *)S, N, part);
    norm_stage2<<<1, 256, 0, st>>>(part, (int)g, res);
    return hipGetLastError();
}

template <typename C>
__global__ void __launch_bounds__(256) gather_kernel(const C *__restrict__ S, PermArg pa, C *__restrict__ out,
                                                     uint64_t off, uint64_t cnt)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride)
        out[i] = S[sto<C>(phys_of(off + i, pa))];
}

template <typename C>
__global__ void __launch_bounds__(256) scatter_kernel(C *__restrict__ S, PermArg pa, const C *__restrict__ in,
                                                      uint64_t off, uint64_t cnt)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride)
        S[sto<C>(phys_of(off + i, pa))] = in[i];
}

hipError_t gather_logical(const void *S, int n, int dtype, const int *perm, void *out, uint64_t offset,
                          uint64_t count, hipStream_t st)
{
    const PermArg pa = make_perm(perm, n);
    const unsigned g = grid_for(count, 256, 16384);
    if (dtype == 0) gather_kernel<float2><<<g, 256, 0, st>>>((const float2 *)S, pa, (float2 *)out, offset, count);
    else gather_kernel<double2><<<g, 256, 0, st>>>((const double2 *)S, pa, (double2 *)out, offset, count);
    return hipGetLastError();
}

hipError_t scatter_logical(void *S, int n, int dtype, const int *perm, const void *in, uint64_t offset,
                           uint64_t count, hipStream_t st)
{
    const PermArg pa = make_perm(perm, n);
    const unsigned g = grid_for(count, 256, 16384);
    if (dtype == 0) scatter_kernel<float2><<<g, 256, 0, st>>>((float2 *)S, pa, (const float2 *)in, offset, count);
    else scatter_kernel<double2><<<g, 256, 0, st>>>((double2 *)S, pa, (const double2 *)in, offset, count);
    return hipGetLastError();
}

}  // namespace svk
