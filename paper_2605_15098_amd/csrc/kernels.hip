// gfx950 kernels of the state-vector simulator.
//
//  k1  plain sweep: one gate over the whole state (Algorithm 1, Section III-A,
//      with the single-control predicate). Pairs are enumerated by inserting
//      the fixed bits into a dense counter, so consecutive lanes touch
//      consecutive amplitudes and every sweep is a coalesced HBM stream.
//  k3  explicit qubit exchange (the SWAP of Section III-B) as an in-place
//      pass over the amplitudes whose two bits differ.
//  kq  extended gates: a k-qubit unitary with controls.
//
// The block-resident passes are in block.hip, the readouts in readout.hip.
//
// Complex values are interleaved (re, im): float2 for complex64 and double2
// for complex128. Gate matrices arrive in binary64 and are rounded once.
// The single-gate arithmetic (cmul, cmad2, hbfly in k2_device.h) is shared by
// k1 and k2 so an unfused partitioned run reproduces the plain run bit for
// bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "grid.h"
#include "k2_device.h"
#include "launch.h"
#include "plan.h"

namespace svk {

// ---------------------------------------------------------------- init

// |0...0>: one 16-byte store per thread, 4 KiB per work-group. More per
// work-group is slower up to 4 GiB of complex64: 64 MiB alone 12.6 us here,
// 21-25 with 16, 32 or 64 KiB, 14 in a grid-stride loop (the runtime's fill 13.2);
// after a readout of the same state 18.1 against 20.9, and 4 GiB 612 against 685
// us (7.0 TB/s). From 64 GiB on that is more threads than one launch may have.
template <typename V>
__global__ void __launch_bounds__(256) init_kernel(V *S, uint64_t count, uint64_t group0, V first)
{
    const uint64_t i = (group0 + blockIdx.x) * 256 + threadIdx.x;
    if (i < count) S[i] = i == 0 ? first : V{};
}

template <typename V> static hipError_t init_launch(void *S, uint64_t bytes, int dtype, hipStream_t st)
{
    V first{};
    const float one32 = 1.0f;
    const double one64 = 1.0;
    if (dtype == 0) std::memcpy(&first, &one32, sizeof one32);
    else std::memcpy(&first, &one64, sizeof one64);
    const uint64_t count = bytes / sizeof(V);
    return split_launch((count + 255) / 256, 256, [&](uint64_t group0, unsigned groups) {
        init_kernel<V><<<groups, 256, 0, st>>>((V *)S, count, group0, first);
        return hipGetLastError();
    });
}

hipError_t init_zero_state(void *S, int n, int dtype, hipStream_t st)
{
    const uint64_t bytes = (dtype == 0 ? 8ull : 16ull) << n;  // 16 or more
    // (a borrowed buffer may start between two 16-byte units)
    if ((uintptr_t)S % 16 == 0) return init_launch<float4>(S, bytes, dtype, st);
    return init_launch<float2>(S, bytes, dtype, st);
}

// Logical-to-storage order in place (sto is its own inverse, so each pair
// {i, sto(i)} is swapped once, by the thread of the smaller index).
template <typename C> __global__ void __launch_bounds__(256) sto_inplace_kernel(C *S, uint64_t N)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const uint64_t j = sto<C>(i);
        if (j <= i) continue;
        const C a = S[i];
        S[i] = S[j];
        S[j] = a;
    }
}

hipError_t to_storage_order(void *S, int n, int dtype, hipStream_t st)
{
    const uint64_t N = 1ull << n;
    const int s0 = dtype == 0 ? 5 : 4;
    if (n < s0 + 10) return hipSuccess;  // stored in plain order
    const unsigned g = grid_for(N, 256, 8192);
    if (dtype == 0) sto_inplace_kernel<float2><<<g, 256, 0, st>>>((float2 *)S, N);
    else sto_inplace_kernel<double2><<<g, 256, 0, st>>>((double2 *)S, N);
    return hipGetLastError();
}

bool plain_storage(int n, int dtype) { return n < (dtype == 0 ? 5 : 4) + 10; }

// ---------------------------------------------------------------- k1

constexpr int K1_BLOCK = 256;
constexpr int K1_PER = 4;

enum { K1_DENSE = 0, K1_H = 1, K1_X = 2 };

// Pairs (j, j + 2^t) with bit t of j clear and, if c >= 0, bit c set.
template <typename C>
__global__ void __launch_bounds__(K1_BLOCK)
k1_pair_kernel(C *__restrict__ S, uint64_t npairs, uint64_t group0, int t, int c, int kind, C u00, C u01, C u10, C u11)
{
    const uint64_t base = (group0 + blockIdx.x) * (K1_BLOCK * K1_PER) + threadIdx.x;
    const int lo = (c >= 0 && c < t) ? c : t;
    const int hi = (c >= 0 && c > t) ? c : t;
    const uint64_t cbit = c >= 0 ? (1ull << c) : 0ull;
    const uint64_t h = 1ull << t;
#pragma unroll
    for (int i = 0; i < K1_PER; ++i) {
        const uint64_t p = base + (uint64_t)i * K1_BLOCK;
        if (p >= npairs) break;
        uint64_t j = insert0(p, lo);
        if (c >= 0) j = insert0(j, hi);
        j |= cbit;
        // storage order: sto(j + h) = sto(j) ^ sto(h), bit t of j being clear
        const uint64_t sj = sto<C>(j), sk = sj ^ sto<C>(h);
        C a = S[sj], b = S[sk];
        if (kind == K1_H) {
            hbfly(a, b);
            S[sj] = a;
            S[sk] = b;
        } else if (kind == K1_X) {
            S[sj] = b;
            S[sk] = a;
        } else {
            S[sj] = cmad2(u00, a, u01, b);
            S[sk] = cmad2(u10, a, u11, b);
        }
    }
}

// Diagonal gates. Amplitudes with every bit of `ones` (at most two bits, lo
// <= hi) set are multiplied by d1 when tsel < 0, else by d0 or d1 according
// to bit tsel. (The first group as the last argument: 18 qubits complex128 3.28
// us a gate, 3.30 as the third.)
template <typename C>
__global__ void __launch_bounds__(K1_BLOCK)
k1_diag_kernel(C *__restrict__ S, uint64_t namps, int nones, int lo, int hi, int tsel, C d0, C d1, uint64_t group0)
{
    const uint64_t base = (group0 + blockIdx.x) * (K1_BLOCK * K1_PER) + threadIdx.x;
    uint64_t ones = 0;
    if (nones >= 1) ones |= 1ull << lo;
    if (nones >= 2) ones |= 1ull << hi;
#pragma unroll
    for (int i = 0; i < K1_PER; ++i) {
        const uint64_t p = base + (uint64_t)i * K1_BLOCK;
        if (p >= namps) break;
        uint64_t j = p;
        if (nones >= 1) j = insert0(j, lo);
        if (nones >= 2) j = insert0(j, hi);
        j |= ones;
        const uint64_t sj = sto<C>(j);
        C a = S[sj];
        const C d = csel(tsel >= 0 && !((j >> tsel) & 1ull), d0, d1);
        S[sj] = cmul(d, a);
    }
}

// Work-groups of a sweep over `work` pairs or amplitudes.
static uint64_t k1_groups(uint64_t work) { return (work + K1_BLOCK * K1_PER - 1) / (K1_BLOCK * K1_PER); }

template <typename T> static hipError_t k1_launch(void *Sv, int n, const svp::MGate &g, hipStream_t st)
{
    using C = typename CT<T>::type;
    C *S = (C *)Sv;
    const double *u = g.u;
    if (g.cls == svp::GC_DIAG) {
        const bool ptype = (u[0] == 1.0 && u[1] == 0.0);
        int bits[2], nb = 0;
        if (g.c >= 0) bits[nb++] = g.c;
        if (ptype) bits[nb++] = g.t;
        if (nb == 2 && bits[0] > bits[1]) { int x = bits[0]; bits[0] = bits[1]; bits[1] = x; }
        const uint64_t namps = 1ull << (n - nb);
        return split_launch(k1_groups(namps), K1_BLOCK, [&](uint64_t group0, unsigned groups) {
            k1_diag_kernel<C><<<groups, K1_BLOCK, 0, st>>>(S, namps, nb, nb > 0 ? bits[0] : 0,
                                                           nb > 1 ? bits[1] : 0, ptype ? -1 : g.t,
                                                           mk<C>(u[0], u[1]), mk<C>(u[6], u[7]), group0);
            return hipGetLastError();
        });
    }
    const uint64_t npairs = 1ull << (n - 1 - (g.c >= 0 ? 1 : 0));
    const int kind = g.op == 0 ? K1_H : (g.cls == svp::GC_PERM ? K1_X : K1_DENSE);
    return split_launch(k1_groups(npairs), K1_BLOCK, [&](uint64_t group0, unsigned groups) {
        k1_pair_kernel<C><<<groups, K1_BLOCK, 0, st>>>(S, npairs, group0, g.t, g.c, kind, mk<C>(u[0], u[1]),
                                                       mk<C>(u[2], u[3]), mk<C>(u[4], u[5]),
                                                       mk<C>(u[6], u[7]));
        return hipGetLastError();
    });
}

hipError_t k1_gate(void *S, int n, int dtype, const svp::MGate &g, hipStream_t st)
{
    return dtype == 0 ? k1_launch<float>(S, n, g, st) : k1_launch<double>(S, n, g, st);
}

// ---------------------------------------------------------------- plain circuits of small states

// Every gate of a plain circuit on a state that fits in LDS, in one launch: one
// work-group holds the state and applies the gates in order, a barrier
// after each, with k1_pair_kernel's and k1_diag_kernel's arithmetic (the same
// bits). A launch per gate is bound by the launches: 3.2 us each against less
// than a microsecond of work on up to 2^14 amplitudes (10 qubits complex128,
// 64 gates of a phase estimation: 205 us in launches). What is left is each wave's
// own instructions, a thousand cycles a gate. So a thread has as few amplitudes
// as there are threads for (PER, 0: any number), consecutive diagonal gates
// keep them in registers, without LDS and barriers between the gates (for PER
// = 0 their tests of every amplitude cost more: a controlled phase touches a
// quarter), and the scalar cache has the records before the first gate needs
// them. us with reset, export and readout of a phase estimation, before these -> now: 10
// qubits complex64 72 -> 62, 12 qubits 106 -> 81, 14 qubits 238 -> 205.
// ops: K2_PHASE / K2_DIAG / K2_H / K2_X / K2_DENSE records with a: target, b:
// control or -1, v: the matrix.
template <typename C, int PER>
__global__ void __launch_bounds__(1024) k1_small_kernel(C *__restrict__ S, int n, const svp::K2Op *ops, int nops)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char small_lds[];
    C *st = reinterpret_cast<C *>(small_lds);
    const uint32_t N = 1u << n, nt = blockDim.x, tid = threadIdx.x;
    const k2_const<svp::K2Op> op = as_const<svp::K2Op>(ops);
    auto diagonal = [&](int g) { return op[g].kind == svp::K2_PHASE || op[g].kind == svp::K2_DIAG; };
    {
        // one word of each 64-byte line of the first records (the scalar cache
        // is 16 KiB), eight lines in flight
        const int lines = min(nops, 128) * (int)sizeof(svp::K2Op) / 64;
        const k2_const<int32_t> w = as_const<int32_t>(ops);
        for (int i = 0; i + 8 <= lines; i += 8) {
            int32_t x = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) x ^= w[(i + k) * 16];
            asm volatile("" ::"s"(x));
        }
    }
    for (uint32_t i = tid; i < N; i += nt) st[i] = S[i];
    __syncthreads();
    for (int g = 0; g < nops;) {
        const int t = op[g].a, c = op[g].b, kind = op[g].kind;
        const k2_const<double> v = &op[g].v[0];
        if (kind == svp::K2_PHASE || kind == svp::K2_DIAG) {
            if constexpr (PER > 0) {
                C a[PER];
#pragma unroll
                for (int k = 0; k < PER; ++k) a[k] = st[tid + k * nt];
                do {
                    const int gt = op[g].a, gc = op[g].b;
                    const uint32_t cb = gc >= 0 ? 1u << gc : 0u, tb = 1u << gt;
                    const k2_const<double> d = &op[g].v[0];
                    if (op[g].kind == svp::K2_PHASE) {
                        const C d1 = mk<C>(d[6], d[7]);
                        const uint32_t ones = cb | tb;
#pragma unroll
                        for (int k = 0; k < PER; ++k)
                            if (((tid + k * nt) & ones) == ones) a[k] = cmul(d1, a[k]);
                    } else {
                        const C d0 = mk<C>(d[0], d[1]), d1 = mk<C>(d[6], d[7]);
#pragma unroll
                        for (int k = 0; k < PER; ++k) {
                            const uint32_t j = tid + k * nt;
                            if ((j & cb) == cb) a[k] = cmul(csel((j & tb) != 0u, d1, d0), a[k]);
                        }
                    }
                    ++g;
                } while (g < nops && diagonal(g));
#pragma unroll
                for (int k = 0; k < PER; ++k) st[tid + k * nt] = a[k];
                __syncthreads();
                continue;
            }
            // amplitudes with every condition bit set: the control, and for a phase the target
            const C d0 = mk<C>(v[0], v[1]), d1 = mk<C>(v[6], v[7]);
            const bool phase = kind == svp::K2_PHASE;
            int lo = phase ? t : c, hi = phase ? c : -1;
            if (lo < 0) lo = hi, hi = -1;
            if (hi >= 0 && hi < lo) {
                const int x = lo;
                lo = hi;
                hi = x;
            }
            const uint32_t ones = (lo >= 0 ? 1u << lo : 0u) | (hi >= 0 ? 1u << hi : 0u);
            const uint32_t cnt = N >> ((lo >= 0) + (hi >= 0));
            for (uint32_t p = tid; p < cnt; p += nt) {
                uint32_t j = p;
                if (lo >= 0) j = insert0_32(j, lo);
                if (hi >= 0) j = insert0_32(j, hi);
                j |= ones;
                const C d = csel(!phase && !((j >> t) & 1u), d0, d1);
                st[j] = cmul(d, st[j]);
            }
        } else {
            const int lo = (c >= 0 && c < t) ? c : t, hi = (c >= 0 && c > t) ? c : t;
            const uint32_t cbit = c >= 0 ? 1u << c : 0u, pairs = N >> (c >= 0 ? 2 : 1);
            auto each = [&](auto &&f) {
                for (uint32_t p = tid; p < pairs; p += nt) {
                    uint32_t j = insert0_32(p, lo);
                    if (c >= 0) j = insert0_32(j, hi);
                    j |= cbit;
                    f(st[j], st[j | (1u << t)]);
                }
            };
            if (kind == svp::K2_H) {
                each([](C &x, C &y) {
                    C a = x, b = y;
                    hbfly(a, b);
                    x = a;
                    y = b;
                });
            } else if (kind == svp::K2_X) {
                each([](C &x, C &y) {
                    const C a = x, b = y;
                    x = b;
                    y = a;
                });
            } else {
                const C u00 = mk<C>(v[0], v[1]), u01 = mk<C>(v[2], v[3]), u10 = mk<C>(v[4], v[5]), u11 = mk<C>(v[6], v[7]);
                each([&](C &x, C &y) {
                    const C a = x, b = y;
                    x = cmad2(u00, a, u01, b);
                    y = cmad2(u10, a, u11, b);
                });
            }
        }
        ++g;
        __syncthreads();
    }
    for (uint32_t i = tid; i < N; i += nt) S[i] = st[i];
}

int k1_small_max(int dtype) { return dtype == 0 ? 14 : 13; }

svp::K2Op k1_small_op(const svp::MGate &g)
{
    svp::K2Op op{};
    if (g.cls == svp::GC_DIAG) op.kind = (g.u[0] == 1.0 && g.u[1] == 0.0) ? svp::K2_PHASE : svp::K2_DIAG;
    else op.kind = g.op == 0 ? svp::K2_H : (g.cls == svp::GC_PERM ? svp::K2_X : svp::K2_DENSE);
    op.a = g.t;
    op.b = g.c;
    for (int k = 0; k < 8; ++k) op.v[k] = g.u[k];
    return op;
}

template <typename C, int PER>
static hipError_t k1_small_launch(void *S, int n, const svp::K2Op *ops, int nops, hipStream_t st)
{
    const size_t lds = sizeof(C) << n;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)k1_small_kernel<C, PER>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    k1_small_kernel<C, PER><<<1, n >= 10 ? 1024u : 1u << n, lds, st>>>((C *)S, n, ops, nops);
    return hipGetLastError();
}

template <typename C> static hipError_t k1_small_any(void *S, int n, const svp::K2Op *ops, int nops, hipStream_t st)
{
    if (n <= 10) return k1_small_launch<C, 1>(S, n, ops, nops, st);
    if (n == 11) return k1_small_launch<C, 2>(S, n, ops, nops, st);
    if (n == 12) return k1_small_launch<C, 4>(S, n, ops, nops, st);
    return k1_small_launch<C, 0>(S, n, ops, nops, st);
}

hipError_t k1_small(void *S, int n, int dtype, const svp::K2Op *dev_ops, int nops, hipStream_t st)
{
    if (n > k1_small_max(dtype)) return hipErrorInvalidValue;
    return dtype == 0 ? k1_small_any<float2>(S, n, dev_ops, nops, st) : k1_small_any<double2>(S, n, dev_ops, nops, st);
}

// ---------------------------------------------------------------- extended gates

// A k-qubit unitary (2^k x 2^k, row-major, the state's precision; bit b of
// the row index = target b) on physical target bits where every physical
// bit of cmask is 1: one thread per group of 2^k amplitudes. The group base
// inserts zeros at the fixed bits (targets and controls, ascending) into
// the thread number and sets the controls; the matrix is read at uniform
// addresses (scalar loads), the 2^k outputs are stored after all inputs are
// in registers.
template <typename C, int K>
__global__ void __launch_bounds__(128) kq_kernel(C *__restrict__ S, uint64_t ngroups, KqArg a, const C *__restrict__ U, uint64_t group0)
{
    constexpr int D = 1 << K;
    const uint64_t g = (group0 + blockIdx.x) * 128 + threadIdx.x;
    if (g >= ngroups) return;
    uint64_t j = g;
    for (int i = 0; i < a.nfixed; ++i) j = insert0(j, a.fixed[i]);
    j |= a.cmask;
    const uint64_t sj = sto<C>(j);
    // storage offset of group member x (the order is linear, so offsets XOR)
    auto at = [&](int x) {
        uint64_t off = sj;
#pragma unroll
        for (int b = 0; b < K; ++b)
            if ((x >> b) & 1) off ^= a.toff[b];
        return off;
    };
    C v[D];
#pragma unroll
    for (int x = 0; x < D; ++x) v[x] = S[at(x)];
#pragma unroll
    for (int x = 0; x < D; ++x) {
        C acc = mk<C>(0.0, 0.0);
#pragma unroll
        for (int y = 0; y < D; ++y) {
            const C u = U[x * D + y];
            acc.x = xfma(u.x, v[y].x, xfma(-u.y, v[y].y, acc.x));
            acc.y = xfma(u.x, v[y].y, xfma(u.y, v[y].x, acc.y));
        }
        S[at(x)] = acc;
    }
}

// The same for k = 4..6 on the matrix cores: the gate is a contraction of 2^k
// complex products per amplitude, and a thread per group can hold neither 2^6
// amplitudes in registers nor the matrix in the scalar cache. A wave takes NB
// batches of 16 groups, the columns of the 16x16x4 products: lane 16 q + n
// loads amplitudes 4 s + q of group n (both components), and all of a wave's
// inputs are in registers before its first store (the gate is in place).
// With PAIR (complex64, memory bit 0 neither target nor control) a lane's two
// batches are neighbouring groups, 16 bytes per access: half the accesses,
// runs of 256 bytes. The matrix is staged once per work-group in operand
// order as (re, im) pairs: one LDS read feeds four products, re and im rows
// against re and im inputs. Lane 16 q + n gets rows 4 q + r (FP32) or 4 r + q
// (FP64) of group n. Up to k = 5 this is bound by HBM; k = 6 needs 512 flop
// per amplitude, about as long on the matrix cores as the memory takes.
// One gate on scattered targets, a thread per group -> this: 26 qubits
// complex64 k = 5 280-336 -> 211-257 us, k = 6 1122 -> 355-384 us; 25 qubits
// complex128 k = 5 262-341 -> 205-220 us, k = 6 2619 -> 306-332 us.
template <typename C, int K, int NB, bool PAIR>
__global__ void __launch_bounds__(256, K == 6 && PAIR ? 4 : 1) kq_mfma_kernel(C *__restrict__ S, uint64_t nbatch, KqArg a, const C *__restrict__ U)
{
    using T = decltype(C::x);
    using V = typename K2Mfma<T>::V;
    constexpr int D = 1 << K, TILES = D / 16, STEPS = D / 4;
    constexpr bool F32 = sizeof(T) == 4;
    __shared__ C ul[D * D];
    for (int e = threadIdx.x; e < D * D; e += 256) {
        const int l = e & 63, s = (e >> 6) % STEPS, t = (e >> 6) / STEPS;
        ul[e] = U[(16 * t + (l & 15)) * D + 4 * s + (l >> 4)];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
    // storage offsets of the lane's part of the input and output amplitudes (the order is linear, offsets XOR)
    const uint64_t qin = ((q & 1) ? a.toff[0] : 0ull) ^ ((q & 2) ? a.toff[1] : 0ull);
    const uint64_t qout = F32 ? ((q & 1) ? a.toff[2] : 0ull) ^ ((q & 2) ? a.toff[3] : 0ull) : qin;
    auto off = [&](int x, int first, int bits) {
        uint64_t o = 0;
#pragma unroll
        for (int b = 0; b < bits; ++b)
            if ((x >> b) & 1) o ^= a.toff[first + b];
        return o;
    };
    const uint64_t stride = (uint64_t)gridDim.x * 4;
    for (uint64_t b = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); b < nbatch; b += stride) {
        uint64_t base[NB];
        C v[NB][STEPS];
        if constexpr (PAIR) {
            uint64_t j = (b * 16 + n) * 2;
            for (int f = 0; f < a.nfixed; ++f) j = insert0(j, a.fixed[f]);
            base[0] = sto<C>(j | a.cmask);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const float4 p = *reinterpret_cast<const float4 *>(S + (base[0] ^ qin ^ off(s, 2, K - 2)));
                v[0][s] = mk<C>(p.x, p.y);
                v[1][s] = mk<C>(p.z, p.w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                uint64_t j = (b * NB + i) * 16 + n;
                for (int f = 0; f < a.nfixed; ++f) j = insert0(j, a.fixed[f]);
                base[i] = sto<C>(j | a.cmask);
#pragma unroll
                for (int s = 0; s < STEPS; ++s) v[i][s] = S[base[i] ^ qin ^ off(s, 2, K - 2)];
            }
        }
        // (not unrolled: the operand reads of all tiles together would take the registers of two more waves)
#pragma unroll 1
        for (int t = 0; t < TILES; ++t) {
            V re[NB], im[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) re[i] = im[i] = V{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const C u = ul[(t * STEPS + s) * 64 + lane];
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    re[i] = K2Mfma<T>::mma(u.x, v[i][s].x, re[i]);
                    im[i] = K2Mfma<T>::mma(u.y, v[i][s].x, im[i]);
                    re[i] = K2Mfma<T>::mma(-u.y, v[i][s].y, re[i]);
                    im[i] = K2Mfma<T>::mma(u.x, v[i][s].y, im[i]);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t o = qout ^ off(r, F32 ? 0 : 2, 2) ^ off(t, 4, K - 4);
                if constexpr (PAIR) {
                    *reinterpret_cast<float4 *>(S + (base[0] ^ o)) =
                        make_float4((float)re[0][r], (float)im[0][r], (float)re[1][r], (float)im[1][r]);
                } else {
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        C z;
                        z.x = re[i][r];
                        z.y = im[i][r];
                        S[base[i] ^ o] = z;
                    }
                }
            }
        }
    }
}

template <typename C, int K> static hipError_t kq_mfma_launch(C *S, uint64_t ngroups, const KqArg &a, const C *U, hipStream_t st)
{
    constexpr int NB = sizeof(C) == 8 ? 2 : 1;
    const uint64_t nbatch = ngroups / (16 * NB);
    const unsigned grid = grid_for(nbatch, 4, 1024);
    if (NB == 2 && a.fixed[0] > 0 && (uintptr_t)S % 16 == 0) kq_mfma_kernel<C, K, NB, NB == 2><<<grid, 256, 0, st>>>(S, nbatch, a, U);
    else kq_mfma_kernel<C, K, NB, false><<<grid, 256, 0, st>>>(S, nbatch, a, U);
    return hipGetLastError();
}

// ngroups is a power of two, so from 32 on there is a whole number of batches;
// smaller states keep the thread per group. k = 4 takes the matrix cores too:
// no difference on scattered targets (212 and 208 us at 26 qubits complex64),
// but 335 against 476 us on the lowest ones, where a thread's amplitudes are
// neighbours and its accesses touch a line each. k <= 3 stays with the threads
// (at the memory's rate, 180-205 us).
template <typename C> static hipError_t kq_launch(void *S, int n, const KqArg &a, const void *U, hipStream_t st)
{
    const uint64_t ngroups = 1ull << (n - a.nfixed);
    const bool mfma = ngroups >= 32;
    if (mfma && a.k == 4) return kq_mfma_launch<C, 4>((C *)S, ngroups, a, (const C *)U, st);
    if (mfma && a.k == 5) return kq_mfma_launch<C, 5>((C *)S, ngroups, a, (const C *)U, st);
    if (mfma && a.k == 6) return kq_mfma_launch<C, 6>((C *)S, ngroups, a, (const C *)U, st);
    return split_launch((ngroups + 127) / 128, 128, [&](uint64_t group0, unsigned groups) {
        switch (a.k) {
        case 1: kq_kernel<C, 1><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        case 2: kq_kernel<C, 2><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        case 3: kq_kernel<C, 3><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        case 4: kq_kernel<C, 4><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        case 5: kq_kernel<C, 5><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        case 6: kq_kernel<C, 6><<<groups, 128, 0, st>>>((C *)S, ngroups, a, (const C *)U, group0); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    });
}

hipError_t kq_gate(void *S, int n, int dtype, const int *tbits, int k, const int *cbits, int nc, const void *U,
                   hipStream_t st)
{
    if (k < 1 || k > 6 || nc < 0 || k + nc > n || k + nc > 24) return hipErrorInvalidValue;
    KqArg a{};
    a.k = k;
    int fixed[24];
    for (int b = 0; b < k; ++b) fixed[b] = tbits[b];
    for (int b = 0; b < nc; ++b) {
        fixed[k + b] = cbits[b];
        a.cmask |= 1ull << cbits[b];
    }
    a.nfixed = k + nc;
    std::sort(fixed, fixed + a.nfixed);
    for (int i = 0; i < a.nfixed; ++i) a.fixed[i] = (int8_t)fixed[i];
    for (int b = 0; b < k; ++b)
        a.toff[b] = dtype == 0 ? sto<float2>(1ull << tbits[b]) : sto<double2>(1ull << tbits[b]);
    return dtype == 0 ? kq_launch<float2>(S, n, a, U, st) : kq_launch<double2>(S, n, a, U, st);
}

// ---------------------------------------------------------------- k3

// Exchange memory bits p and v: amplitude i with bit p = 1, bit v = 0 trades
// places with i ^ 2^p ^ 2^v. Pure data movement, exact.
template <typename C>
__global__ void __launch_bounds__(K1_BLOCK) k3_kernel(C *__restrict__ S, uint64_t npairs, uint64_t group0, int p, int v)
{
    const uint64_t base = (group0 + blockIdx.x) * (K1_BLOCK * K1_PER) + threadIdx.x;
    const int lo = p < v ? p : v, hi = p < v ? v : p;
    const uint64_t flip = (1ull << p) | (1ull << v);
#pragma unroll
    for (int i = 0; i < K1_PER; ++i) {
        const uint64_t q = base + (uint64_t)i * K1_BLOCK;
        if (q >= npairs) break;
        uint64_t j = insert0(insert0(q, lo), hi) | (1ull << p);
        const uint64_t sj = sto<C>(j), sk = sto<C>(j ^ flip);
        C a = S[sj], b = S[sk];
        S[sj] = b;
        S[sk] = a;
    }
}

hipError_t k3_swap(void *S, int n, int dtype, int p, int v, hipStream_t st)
{
    const uint64_t npairs = 1ull << (n - 2);
    return split_launch(k1_groups(npairs), K1_BLOCK, [&](uint64_t group0, unsigned groups) {
        if (dtype == 0) k3_kernel<float2><<<groups, K1_BLOCK, 0, st>>>((float2 *)S, npairs, group0, p, v);
        else k3_kernel<double2><<<groups, K1_BLOCK, 0, st>>>((double2 *)S, npairs, group0, p, v);
        return hipGetLastError();
    });
}

}  // namespace svk
