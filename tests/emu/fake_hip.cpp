// Test-only stand-in for the HIP runtime: the program defines the runtime's
// entry points itself, so the simulator library it is linked with allocates
// addresses that nobody reads, and launches kernels that are only written down.
// Host code (launch shapes, error paths, caches, tuners) then runs on a
// machine without a GPU, at sizes that no test machine's memory holds.
//
// A launch is refused as the runtime refuses it, from 2^32 threads in one
// dimension on. Device times are invented: first the number of launches counts, then their
// LDS bytes.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/sv.h"
#include "../../paper_2605_15098_amd/csrc/plan.h"

namespace {

constexpr uintptr_t kDeviceFrom = uintptr_t(1) << 44;
uintptr_t g_next = kDeviceFrom;
hipError_t g_last = hipSuccess;
bool g_fail_launches = false, g_fail_allocations = false, g_capturing = false;
size_t g_allocated = 0, g_most_bytes = ~size_t(0);  // since the last call(); allocations above this fail
int g_launches = 0, g_graphs = 0;
uint64_t g_most_threads = 0;
double g_clock = 0.0;
struct FakeGraph {
    double cost = 0.0;
};
FakeGraph *g_graph = nullptr;
struct FakeEvent {
    double at = 0.0;
};
struct Call {
    dim3 grid, block;
    size_t lds;
    hipStream_t st;
};
std::vector<Call> g_calls;

}  // namespace

extern "C" {

hipError_t hipMalloc(void **p, size_t bytes)
{
    if (g_fail_allocations || bytes > g_most_bytes) return g_last = hipErrorOutOfMemory;
    g_allocated += bytes;
    *p = (void *)g_next;
    g_next += (bytes + 511) / 512 * 512;
    return hipSuccess;
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    *p = std::calloc(1, bytes);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *, size_t bytes, hipMemcpyKind kind, hipStream_t)
{
    if (kind == hipMemcpyDeviceToHost) std::memset(dst, 0, bytes);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::memset(a, 0, sizeof *a);
    a->type = (uintptr_t)p >= kDeviceFrom && (uintptr_t)p < g_next ? hipMemoryTypeDevice : hipMemoryTypeHost;
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t lds, hipStream_t)
{
    const uint64_t threads = (uint64_t)grid.x * block.x;
    if (threads > g_most_threads) g_most_threads = threads;
    if (g_fail_launches || threads >= (1ull << 32) || grid.x == 0) return g_last = hipErrorInvalidConfiguration;
    ++g_launches;
    (g_capturing ? g_graph->cost : g_clock) += 1e6 + (double)lds;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    g_calls.push_back({grid, block, lds, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    const Call c = g_calls.back();
    g_calls.pop_back();
    *grid = c.grid;
    *block = c.block;
    *lds = c.lds;
    *st = c.st;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    g_graph = new FakeGraph();
    g_capturing = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    g_capturing = false;
    *g = reinterpret_cast<hipGraph_t>(g_graph);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    ++g_graphs;
    *x = reinterpret_cast<hipGraphExec_t>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    g_clock += reinterpret_cast<FakeGraph *>(x)->cost;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete reinterpret_cast<FakeGraph *>(g);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = reinterpret_cast<hipEvent_t>(new FakeEvent());
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<FakeEvent *>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    reinterpret_cast<FakeEvent *>(e)->at = g_clock;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(reinterpret_cast<FakeEvent *>(b)->at - reinterpret_cast<FakeEvent *>(a)->at);
    return hipSuccess;
}

}  // extern "C"

namespace {

// One call: its name, status, launches and the most threads of any of them.
template <typename F> void call(const char *name, F &&f)
{
    g_launches = 0;
    g_most_threads = 0;
    g_allocated = 0;
    const sv_status st = f();
    std::printf("%s %d %d %llu\n", name, (int)st, g_launches, (unsigned long long)g_most_threads);
}

void *device(size_t bytes)
{
    void *p = nullptr;
    (void)hipMalloc(&p, bytes);
    return p;
}

sv_gate gate(int op, int t, int c = -1, double theta = 0.0, int t2 = -1)
{
    sv_gate g{};
    g.op = op;
    g.target = t;
    g.control = c;
    g.target2 = t2;
    g.theta = theta;
    return g;
}

int reset(int n, sv_dtype dt)
{
    const size_t bytes = (dt == SV_COMPLEX64 ? 8ull : 16ull) << n;
    sv_handle h = nullptr;
    call("create", [&] { return sv_create(n, dt, &h); });
    call("reset", [&] { return sv_reset(h); });
    sv_destroy(h);
    char *p = (char *)device(bytes + 8);
    call("wrap", [&] { return sv_wrap(n, dt, p + 8, bytes, nullptr, &h); });
    call("reset_between_units", [&] { return sv_reset(h); });
    sv_destroy(h);
    return 0;
}

// One call of everything that sweeps the state or its outcomes.
int sweeps(int n, sv_dtype dt)
{
    const size_t bytes = (dt == SV_COMPLEX64 ? 8ull : 16ull) << n;
    void *user = device(bytes);
    double *out = (double *)device(8ull << n);
    sv_handle h = nullptr;
    call("create", [&] { return sv_create(n, dt, &h); });
    std::vector<int> low(n - 1);
    for (int q = 0; q < n - 1; ++q) low[q] = q;
    const int few[] = {n - 1, 0, 7};
    double u[4] = {0.1, 0.2, 0.3, 0.4}, x = 0.0, y = 0.0;
    uint64_t shots[4], m = 0;
    sv_schedule plain{};
    plain.mode = SV_PLAIN;
    sv_schedule paper{};
    paper.mode = SV_PARTITIONED;
    paper.block_qubits = 10;
    paper.remap = SV_REMAP_EXPLICIT;
    std::vector<double> mat(2 * 64 * 64, 0.0);
    for (int layout = 0; layout < 2; ++layout) {
        call("state", [&] { return sv_state(h, user); });
        call("set_state", [&] { return sv_set_state_range(h, 0, 1ull << n, user); });
        call("probabilities", [&] { return sv_probabilities(h, nullptr, 0, out); });
        call("marginal", [&] { return sv_probabilities(h, low.data(), n - 1, out); });
        call("marginal_of_few", [&] { return sv_probabilities(h, few, 3, out); });
        call("norm", [&] { return sv_norm(h, &x); });
        call("qpe_readout", [&] { return sv_qpe_readout(h, n - 1, &m, &x, &y); });
        call("sample", [&] { return sv_sample(h, nullptr, 0, u, 4, shots); });
        call("sample_of_few", [&] { return sv_sample(h, few, 3, u, 4, shots); });
        const sv_gate sweep[] = {gate(SV_H, n - 1), gate(SV_X, 1), gate(SV_RX, 2, -1, 0.3), gate(SV_RZ, 3, -1, 0.4),
                                 gate(SV_P, 4, -1, 0.5), gate(SV_X, 5, 0)};
        call("plain", [&] { return sv_apply_circuit(h, sweep, 6, &plain); });
        call("explicit_remap", [&] { return sv_apply_circuit(h, sweep, 6, &paper); });
        call("partitioned", [&] { return sv_apply_circuit(h, sweep, 6, nullptr); });
        for (int k = 1; k <= 6; ++k) {
            sv_gate_ex g{};
            g.op = SV_UK;
            g.ntargets = k;
            for (int b = 0; b < k; ++b) g.targets[b] = n - 1 - 2 * b;
            g.uk = mat.data();
            call("unitary", [&] { return sv_apply_circuit_ex(h, &g, 1, nullptr); });
        }
        const sv_gate rename[] = {gate(SV_SWAP, 0, -1, 0.0, n - 1), gate(SV_SWAP, 2, -1, 0.0, 9)};
        call("swap", [&] { return sv_apply_circuit(h, rename, 2, nullptr); });
    }
    sv_destroy(h);
    return 0;
}

// A reset whose launch fails, from a layout that SWAPs permuted: status, then the layout.
int failed_reset()
{
    sv_handle h = nullptr;
    sv_create(5, SV_COMPLEX64, &h);
    const sv_gate g[] = {gate(SV_SWAP, 0, -1, 0.0, 3), gate(SV_SWAP, 1, -1, 0.0, 4)};
    call("swap", [&] { return sv_apply_circuit(h, g, 2, nullptr); });
    g_fail_launches = true;
    call("reset", [&] { return sv_reset(h); });
    g_fail_launches = false;
    int lay[5];
    sv_layout(h, lay);
    std::printf("layout %d %d %d %d %d\n", lay[0], lay[1], lay[2], lay[3], lay[4]);
    call("reset", [&] { return sv_reset(h); });
    sv_layout(h, lay);
    std::printf("layout %d %d %d %d %d\n", lay[0], lay[1], lay[2], lay[3], lay[4]);
    sv_destroy(h);
    return 0;
}

// The marginal of the nq qubits from `first` on (of all: in reversed order).
int marginal(int n, int nq, int first)
{
    sv_handle h = nullptr;
    sv_create(n, SV_COMPLEX64, &h);
    std::vector<int> q(nq);
    for (int k = 0; k < nq; ++k) q[k] = nq == n ? n - 1 - k : first + k;
    double *out = (double *)device(8ull << nq);
    call("marginal", [&] { return sv_probabilities(h, q.data(), nq, out); });
    sv_destroy(h);
    return 0;
}

// Shots (their logarithm; -1: a projective measurement) of a full register in the
// identity or a permuted layout, and the scratch that they took; little: with
// no memory for an array of the probabilities.
int shots(int n, sv_dtype dt, int log_shots, bool permuted, bool little)
{
    sv_handle h = nullptr;
    sv_create(n, dt, &h);
    const sv_gate g = gate(SV_SWAP, 0, -1, 0.0, n - 1);
    if (permuted) sv_apply_circuit(h, &g, 1, nullptr);
    const size_t count = size_t(1) << (log_shots > 0 ? log_shots : 0);
    double *u = (double *)device(8 * count);
    uint64_t *out = (uint64_t *)device(8 * count), m = 0;
    double p = 0.0;
    if (little) g_most_bytes = (size_t(1) << n) + 16 * count + 4096;
    call("shots", [&] { return log_shots < 0 ? sv_measure(h, nullptr, 0, 0.5, &m, &p) : sv_sample(h, nullptr, 0, u, count, out); });
    std::printf("scratch %zu\n", g_allocated);
    sv_destroy(h);
    return 0;
}

// An allocation that fails, then a call that needs none.
int failed_allocation()
{
    sv_handle h = nullptr;
    sv_create(12, SV_COMPLEX64, &h);
    double p[4096], x = 0.0;
    g_fail_allocations = true;
    call("probabilities", [&] { return sv_probabilities(h, nullptr, 0, p); });
    call("norm", [&] { return sv_norm(h, &x); });
    call("reset", [&] { return sv_reset(h); });
    g_fail_allocations = false;
    call("norm", [&] { return sv_norm(h, &x); });
    sv_destroy(h);
    return 0;
}

// A circuit without its gate array, after one of as many gates was applied.
int null_gates()
{
    sv_handle h = nullptr;
    sv_create(5, SV_COMPLEX64, &h);
    const sv_gate g[] = {gate(SV_H, 0), gate(SV_X, 1, 0), gate(SV_RZ, 2, -1, 0.3)};
    call("apply", [&] { return sv_apply_circuit(h, g, 3, nullptr); });
    call("null", [&] { return sv_apply_circuit(h, nullptr, 3, nullptr); });
    call("apply", [&] { return sv_apply_circuit(h, g, 3, nullptr); });
    sv_destroy(h);
    return 0;
}

// Batches of one instance, with the number of graphs built so far after each:
// a circuit, the same again, under another fusion rule, and a circuit with
// another angle whose 64-bit mixed hash, words in the order of the inputs, is
// that of the first.
int batch()
{
    const int n = 10;
    const void *buf = (void *)g_next;
    sv_handle h = nullptr;
    sv_create(n, SV_COMPLEX64, &h);
    sv_gate a[] = {gate(SV_H, 0), gate(SV_X, 1, 0), gate(SV_RZ, 9, -1, 0.3)}, b[3];
    std::memcpy(b, a, sizeof a);
    b[2].theta = 1.7;
    auto salt = [](uint64_t k) { return 0x9e3779b97f4a7c15ull + (k << 6) + (k >> 2); };
    auto mix = [&](uint64_t k, uint64_t x) {
        k = (k ^ (x + salt(k))) * 0xff51afd7ed558ccdull;
        return k ^ (k >> 33);
    };
    auto words = [&](uint64_t k, const void *p, size_t count) {
        for (size_t i = 0; i < count; ++i) {
            uint64_t w;
            std::memcpy(&w, (const char *)p + 8 * i, 8);
            k = mix(k, w);
        }
        return k;
    };
    svp::PlanConfig c;
    c.n = n;
    c.dtype = SV_COMPLEX64;
    c.mode = 1;
    c.policy = SV_SWAP_GRAPH;
    c.diag_free = 1;
    c.fuse_k = 1;
    c.auto_pins = 1;
    int l2p[n];
    for (int q = 0; q < n; ++q) l2p[q] = q;
    static_assert(sizeof c % 8 == 0 && sizeof l2p % 8 == 0, "whole words");
    uint64_t k = mix(mix(0x5eed, 1), 7);
    k = mix(words(k, &c, sizeof c / 8), sizeof c);
    k = mix(mix(k, (uint64_t)(uintptr_t)buf), n);
    k = mix(words(k, l2p, sizeof l2p / 8), sizeof l2p);
    k = words(k, a, 24);  // all but the last gate's angle and matrix, which an RZ does not read
    uint64_t ta, tb, ua = 0, ub;
    std::memcpy(&ta, &a[2].theta, 8);
    std::memcpy(&tb, &b[2].theta, 8);
    const uint64_t ka = mix(k, ta), kb = mix(k, tb);
    ub = (kb ^ ka ^ (ua + salt(ka))) - salt(kb);
    std::memcpy(&b[2].u[0], &ub, 8);
    const sv_gate *la = a, *lb = b;
    const size_t m = 3;
    auto apply = [&](const char *name, const sv_gate *const *list) {
        call(name, [&] { return sv_apply_batch(&h, 1, list, &m, nullptr); });
        std::printf("graphs %d\n", g_graphs);
    };
    apply("first", &la);
    apply("same", &la);
    apply("other_angle", &lb);
    setenv("SV_FUSE_ALL", "1", 1);
    apply("other_rule", &la);
    unsetenv("SV_FUSE_ALL");
    apply("same", &la);
    sv_destroy(h);
    return 0;
}

// The exhaustive tuner's pick for a Fourier transform, and the untuned schedule's block.
int tune(int n, sv_dtype dt)
{
    sv_handle h = nullptr;
    sv_create(n, dt, &h);
    std::vector<sv_gate> g;
    for (int q = n - 1; q >= 0; --q) {
        g.push_back(gate(SV_H, q));
        for (int c = 0; c < q; ++c) g.push_back(gate(SV_P, q, c, 0.1 + c));
    }
    sv_schedule s{};
    call("tune", [&] { return sv_tune(h, g.data(), g.size(), SV_TUNER_EXHAUSTIVE, &s); });
    float f[SV_FEATURES];
    sv_features(n, dt, g.data(), g.size(), nullptr, f);
    std::printf("pick %d %d %d\n", s.block_qubits, s.reg_qubits, s.pin_qubits);
    std::printf("default %d %d %d\n", (int)f[2], (int)f[3], (int)f[4]);
    sv_destroy(h);
    return 0;
}

// The batch tuner's pick for Fourier transforms of two sizes.
int tune_batch(int n0, int n1, sv_dtype dt)
{
    sv_handle hs[2] = {};
    std::vector<sv_gate> g[2];
    const int ns[2] = {n0, n1};
    for (int i = 0; i < 2; ++i) {
        sv_create(ns[i], dt, &hs[i]);
        for (int q = ns[i] - 1; q >= 0; --q) {
            g[i].push_back(gate(SV_H, q));
            for (int c = 0; c < q; ++c) g[i].push_back(gate(SV_P, q, c, 0.1 + c));
        }
    }
    const sv_gate *lists[] = {g[0].data(), g[1].data()};
    const size_t m[] = {g[0].size(), g[1].size()};
    sv_schedule s{};
    s.block_qubits = -1;
    call("tune", [&] { return sv_tune_batch(hs, 2, lists, m, &s); });
    std::printf("pick %d %d %d\n", s.block_qubits, s.reg_qubits, s.pin_qubits);
    sv_stats st{};
    call("default", [&] { return sv_apply_batch(hs, 2, lists, m, nullptr); });
    sv_stats_get(hs[1], &st);
    std::printf("passes %d\n", (int)st.passes);
    return 0;
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    auto num = [&](int i) { return argc > i ? std::atoi(argv[i]) : 0; };
    if (what == "reset") return reset(num(2), (sv_dtype)num(3));
    if (what == "sweeps") return sweeps(num(2), (sv_dtype)num(3));
    if (what == "failed_reset") return failed_reset();
    if (what == "null_gates") return null_gates();
    if (what == "batch") return batch();
    if (what == "tune") return tune(num(2), (sv_dtype)num(3));
    if (what == "tune_batch") return tune_batch(num(2), num(3), (sv_dtype)num(4));
    if (what == "failed_allocation") return failed_allocation();
    if (what == "shots") return shots(num(2), (sv_dtype)num(3), num(4), num(5) != 0, num(6) != 0);
    if (what == "marginal") return marginal(num(2), num(3), num(4));
    return 2;
}
