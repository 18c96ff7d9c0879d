// Host-only driver of the library's host runtime (tests/test_host_path_cpu.py
// builds and runs it).  The HIP runtime functions that libhwr calls are defined
// here, in the executable, and so take the place of the runtime's: device and
// pinned memory are host allocations, copies are done at once, kernels are
// recorded by name and not run, streams and events are counters.  Allocations
// can be made to fail and every call of interest is logged, so a scenario can
// check what a host batch does when memory is short, how often its blocks are
// allocated, which stream a copy is put on and which kernels a batch takes.
//
//   host_path <scenario>       prints "ok", or the failed checks (exit 1)
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "hwr.h"

namespace {

struct Op {
    std::string what;             // copy, launch, record, wait
    void *stream, *obj;           // obj: the event, or the copy's destination
    size_t bytes;
    std::string kernel;
};
std::vector<Op> g_log;
std::map<const void *, std::string> &kernels() {      // registered before main
    static std::map<const void *, std::string> m;
    return m;
}
std::map<char *, size_t> g_dev, g_pinned;
int g_dev_mallocs = 0, g_pinned_mallocs = 0;
size_t g_fail_pinned = SIZE_MAX, g_fail_dev = SIZE_MAX;    // allocations of this many bytes or more fail
int g_cus = 256;
bool g_busy = false;             // streams have work left
uintptr_t g_next = 0x1000;
dim3 g_grid, g_block;
size_t g_shm;
hipStream_t g_stream;

bool inside(const std::map<char *, size_t> &m, const void *p) {
    for (const auto &kv : m)
        if (p >= kv.first && p < kv.first + kv.second) return true;
    return false;
}
template <class T>
T handle() {
    return reinterpret_cast<T>(g_next += 16);
}
hipError_t launch(const void *f, hipStream_t s) {
    g_log.push_back({"launch", s, nullptr, 0, kernels()[f]});
    return hipSuccess;
}

}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, hipStream_t s) {
    g_grid = g, g_block = b, g_shm = shm, g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shm, hipStream_t *s) {
    *g = g_grid, *b = g_block, *shm = g_shm, *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s) { return launch(f, s); }
hipError_t hipExtLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s, hipEvent_t, hipEvent_t, int) {
    return launch(f, s);
}
hipError_t hipMalloc(void **p, size_t n) {
    if (n >= g_fail_dev) return hipErrorOutOfMemory;
    ++g_dev_mallocs;
    *p = std::calloc(1, n);
    g_dev[static_cast<char *>(*p)] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    g_dev.erase(static_cast<char *>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    if (n >= g_fail_pinned) return hipErrorOutOfMemory;
    ++g_pinned_mallocs;
    *p = std::calloc(1, n);
    g_pinned[static_cast<char *>(*p)] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    g_pinned.erase(static_cast<char *>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    if (inside(g_dev, p)) a->type = hipMemoryTypeDevice;
    else if (inside(g_pinned, p)) a->type = hipMemoryTypeHost;
    else return hipErrorInvalidValue;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    g_log.push_back({"copy", st, d, n, ""});
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static std::vector<unsigned char> scratch(size_t(64) << 20);
    *p = scratch.data();
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    *p = {};
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = g_cus;
    return hipSuccess;
}
const char *hipGetErrorName(hipError_t) { return "error"; }
const char *hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = handle<hipEvent_t>(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = handle<hipEvent_t>(), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    g_log.push_back({"record", s, e, 0, ""});
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = handle<hipStream_t>(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return g_busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    g_log.push_back({"wait", s, e, 0, ""});
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}

namespace {

int g_bad = 0;
void check(bool ok, const std::string &what) {
    if (!ok) {
        std::printf("FAIL %s\n", what.c_str());
        ++g_bad;
    }
}

// A context of 4 models on 2 GPU types (bf16, H = 64, all weights zero) and
// host batches for it.
struct Rig {
    static constexpr int M = 4, N = 8, F = 16, H = 64;
    int D;
    hwr_ctx *ctx = nullptr;
    std::vector<uint16_t> emb;
    std::vector<int32_t> len, nout, choice;
    std::vector<uint8_t> feasible;
    std::vector<float> slo, utility, cand;

    explicit Rig(int d, int max_chunk = 0, int weights = 0) : D(d) {
        std::vector<int32_t> dep_model(N), dep_gpu(N), arch(M, 0);
        for (int i = 0; i < N; ++i) dep_model[i] = i % M, dep_gpu[i] = i / M;
        std::vector<float> params(M, 7.0f), zf(static_cast<size_t>(H), 0.0f);
        std::vector<uint16_t> z(static_cast<size_t>(D) * M + F * H + H * H + H * 3, 0);
        hwr_config c{};
        c.n_models = M, c.n_gpu_types = 2, c.n_deployments = N, c.arch_width = 2, c.gpu_width = 2;
        c.embed_dim = D, c.feat_dim = F, c.hidden = H, c.emb_dtype = c.weight_dtype = HWR_BF16;
        c.max_chunk = max_chunk, c.cost_weight = 0.5f, c.default_slo_s = 1.0f;
        c.dep_model = dep_model.data(), c.dep_gpu = dep_gpu.data(), c.model_arch = arch.data();
        c.model_params_b = params.data(), c.wq = c.w1 = c.w2 = c.w3 = z.data();
        c.bq = c.b1 = c.b2 = c.b3 = zf.data();
        const std::vector<float> cw(8, 0.5f);
        c.n_weights = weights, c.cost_weights = cw.data();
        c.stream = handle<void *>();
        check(hwr_init(&c, &ctx) == HWR_OK, "init");
        stream = c.stream;
        std::vector<hwr_hw_state> st(N, hwr_hw_state{1, 1, 0.5f, 0.5f, 0.1f, 0.01f});
        check(ctx && hwr_update_hw_state(ctx, st.data(), N) == HWR_OK, "state");
    }
    ~Rig() { hwr_free(ctx); }
    hwr_status route(int n, hwr_mem mem = HWR_MEM_HOST, bool candidates = false, int weights = 1) {
        emb.assign(static_cast<size_t>(n) * D, 0x3F80);
        len.assign(n, 100), nout.assign(n, 10), slo.assign(n, 1.0f);
        choice.assign(static_cast<size_t>(n) * weights, -1);
        feasible.assign(choice.size(), 9), utility.assign(choice.size(), -1.0f);
        cand.assign(candidates ? static_cast<size_t>(n) * N : 0, -1.0f);
        const hwr_query_batch q{n, mem, emb.data(), len.data(), nout.data(), slo.data()};
        hwr_route_result r{};
        r.choice = choice.data(), r.feasible = feasible.data(), r.utility = utility.data();
        if (candidates) r.cand_ttft = cand.data();
        g_log.clear();
        return hwr_route_batch(ctx, &q, &r);
    }
    // every output of the last batch came back (kernels write nothing here, so
    // as the zeros of a fresh allocation)
    bool written() const {
        for (int32_t c : choice)
            if (c != 0) return false;
        for (uint8_t f : feasible)
            if (f != 0) return false;
        return true;
    }
    void *stream;
};

int launches(const std::string &name) {
    int n = 0;
    for (const Op &o : g_log) n += o.what == "launch" && o.kernel.find(name) != std::string::npos;
    return n;
}

// No pinned memory, or no device memory for the embeddings' block: the batch
// is routed chunk by chunk through device staging.
void memory_short() {
    Rig r(768);
    g_fail_pinned = 0;
    for (int n : {24, 1500}) {
        check(r.route(n) == HWR_OK && r.written(), "no pinned block: " + std::to_string(n) + " queries");
        check(launches("k_route") == 1, "one decision launch");
    }
    g_fail_pinned = SIZE_MAX;
    check(r.route(24) == HWR_OK && r.written(), "pinned memory is back");
    check(r.route(2000, HWR_MEM_HOST, true) == HWR_OK, "candidates take the device staging");
    g_fail_dev = size_t(1) << 20;
    check(r.route(2000) == HWR_OK && r.written(), "no device block for the embeddings");
    g_fail_dev = SIZE_MAX;
    check(r.route(2000) == HWR_OK, "device memory is back");
}

// Batches of every size, growing: the blocks are allocated a few times, not at
// each new largest batch.  A block that cannot be had at its rounded size is
// allocated at the size that the batch needs.
void growing_batches() {
    Rig r(768);
    const int pinned = g_pinned_mallocs, dev = g_dev_mallocs;
    for (int n = 2; n <= 1500; ++n) check(r.route(n) == HWR_OK, std::to_string(n) + " queries");
    check(g_pinned_mallocs - pinned <= 4, std::to_string(g_pinned_mallocs - pinned) + " pinned allocations");
    check(g_dev_mallocs - dev <= 4, std::to_string(g_dev_mallocs - dev) + " device allocations");
    Rig s(768);
    const size_t emb = size_t(2100) * 768 * 2;    // over 3 MB, rounded up to 4
    g_fail_dev = emb + 1;
    check(s.route(2100) == HWR_OK && inside(g_dev, g_log[0].obj) && g_log[0].bytes == emb, "2100 queries, no room to round up");
    check(g_log[0].what == "copy" && !launches("k_gather"), "through the block");
    g_fail_dev = SIZE_MAX;
}

// On a device of few compute units, batches that fill it while their table rows
// are still by query: k_route_stream reads the map of rows by value, so they
// take the form that does not.
void few_compute_units() {
    g_cus = 4;
    Rig r(64);
    for (int n : {200, 300}) {
        check(r.route(n, HWR_MEM_DEVICE) == HWR_OK && launches("k_route") == 1, "one decision launch");
        check(launches("k_route_stream") == 0 && launches("k_table") == 1, std::to_string(n) + " queries: rows by query");
    }
    check(r.route(3000, HWR_MEM_DEVICE) == HWR_OK && launches("k_route_stream") == 1, "rows by value: streamed");
    g_cus = 256;
}

// Embeddings that go up by themselves do so on a stream of their own, beside
// whatever the context's stream still has to run; the kernels wait for them.
// With nothing left to run there, they take the context's stream.
// Both copies: the caller's memory directly, and through the pinned ring.
void upload_beside_the_stream() {
    for (int n : {1500, 12000}) {
        Rig r(768);
        check(r.route(n) == HWR_OK, "idle");
        for (const Op &o : g_log) check(o.stream == r.stream && o.what != "wait", "idle: one stream");
        g_busy = true;
        for (int call = 0; call < 2; ++call) {
            check(r.route(n) == HWR_OK, std::to_string(n) + " queries");
            size_t up = 0, copied = 0;
            void *upload = nullptr, *event = nullptr;
            bool waits = false, after = false;
            for (const Op &o : g_log) {
                if (o.what == "copy" && o.stream != r.stream) up += o.bytes, upload = o.stream, copied = up;
                // the event recorded after the whole copy is the one waited for
                if (o.what == "record" && o.stream == upload && copied == r.emb.size() * 2) event = o.obj;
                if (o.what == "wait" && o.stream == r.stream && o.obj == event && event) waits = true;
                if (o.what == "launch" && o.kernel.find("k_state") == std::string::npos) after = after || !waits;
            }
            check(up == r.emb.size() * 2, "every byte of the embeddings on the upload stream");
            check(waits && !after, "the kernels wait for the upload");
        }
        g_busy = false;
    }
}

// Results in device memory are copied there, not written by the host; a block
// over 8 MB is not pinned.
void chunk_path_instead() {
    Rig r(64);
    void *choice = nullptr;
    check(hipMalloc(&choice, 300 * 4) == hipSuccess, "result");
    check(r.route(300) == HWR_OK, "host result");
    for (const Op &o : g_log) check(o.what != "copy", "host result: no copy");
    hwr_query_batch q{300, HWR_MEM_HOST, r.emb.data(), r.len.data(), r.nout.data(), r.slo.data()};
    hwr_route_result res{};
    res.choice = static_cast<int32_t *>(choice);
    g_log.clear();
    check(hwr_route_batch(r.ctx, &q, &res) == HWR_OK, "device result");
    bool copied = false;
    for (const Op &o : g_log) copied = copied || (o.what == "copy" && o.obj == choice && o.bytes == 1200);
    check(copied, "device result: copied");
    const int pinned = g_pinned_mallocs;
    Rig w(64, 0, 8);
    const int own = g_pinned_mallocs - pinned;
    check(w.route(40000, HWR_MEM_HOST, false, 8) == HWR_OK && g_pinned_mallocs == pinned + own, "block over 8 MB: none pinned");
    check(w.route(38000, HWR_MEM_HOST, false, 8) == HWR_OK && g_pinned_mallocs == pinned + own + 1, "block under 8 MB");
    (void)hipFree(choice);
}

struct Scenario {
    const char *name;
    void (*run)();
};
const Scenario kScenarios[] = {{"memory_short", memory_short}, {"growing_batches", growing_batches},
                               {"few_compute_units", few_compute_units},
                               {"upload_beside_the_stream", upload_beside_the_stream},
                               {"chunk_path_instead", chunk_path_instead}};

}  // namespace

int main(int argc, char **argv) {
    if (argc != 2) return 2;
    for (const Scenario &s : kScenarios)
        if (std::strcmp(argv[1], s.name) == 0) {
            s.run();
            std::printf(g_bad ? "%d failed\n" : "ok\n", g_bad);
            return g_bad ? 1 : 0;
        }
    return 2;
}
