// The host side of libdba on a stand-in for the HIP runtime: kernels are only noted down and "run" when a scenario says so, so
// that calls can be watched while the GPU is behind, and errors come when they are wanted.  (This program's definitions
// go before those of the runtime library that libdba.so is linked to.)
//   host_side_driver LIBDBA.so SCENARIO
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <chrono>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../include/dba.h"

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); fflush(stdout); _exit(1); } } while (0)
extern "C" void _exit(int) __attribute__((noreturn));

// ---------------------------------------------------------------------------
// the stand-in
// ---------------------------------------------------------------------------
struct Dim3 { uint32_t x, y, z; };
constexpr int kOk = 0, kErrorInvalidValue = 1, kErrorLaunchOutOfResources = 701;
constexpr size_t kParamBytes = 176;                // of a step kernel's last argument

struct Work {                                      // a kernel that has been launched
    std::string name;
    void *stream = nullptr;
    uint32_t *seen = nullptr, *told = nullptr;     // host words it will write, of sentences 0 .. B - 1
    const uint32_t *words = nullptr;               // host words it will read
    int B = 0;
    uint32_t value = 0;
    std::vector<unsigned char *> pointers;         // of a step's or dba_init's parameters: those into the workspace
};

static std::map<const void *, std::string> g_names;
static std::map<unsigned char *, size_t> g_host;   // host memory that kernels may use
static std::set<unsigned char *> g_released;
static std::vector<Work> g_queue, g_done;
static int g_last_error, g_calls, g_launches, g_syncs, g_fail_launch = -1;
static bool g_capturing;
static unsigned char *g_ws;
static size_t g_ws_bytes;
static int g_B, g_step;                            // of the step that is about to be launched: sentences, its number from 1

static int error(int e) { if (e != kOk) g_last_error = e; return e; }

static void run(const Work &w)
{
    for (int b = 0; w.seen && b < w.B; ++b) w.seen[b] = 1;
    for (int b = 0; w.told && b < w.B; ++b) w.told[b] = w.value;
    g_done.push_back(w);
}
static void gpu_runs()                             // all that has been launched
{
    for (const Work &w : g_queue) run(w);
    g_queue.clear();
}
static void gpu_runs(void *stream, int most = 1 << 30)
{
    std::vector<Work> left;
    for (const Work &w : g_queue)
        if (w.stream == stream && most-- > 0) run(w);
        else left.push_back(w);
    g_queue.swap(left);
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { g_names[host] = name; }
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}

static struct { Dim3 grid, block; size_t lds; void *stream; } g_config;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream)
{
    ++g_calls;
    g_config = {grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    ++g_calls;
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return kOk;
}
int hipGetLastError() { ++g_calls; const int e = g_last_error; g_last_error = kOk; return e; }
const char *hipGetErrorString(int) { return "an error"; }
int hipGetDevice(int *dev) { ++g_calls; *dev = 0; return kOk; }
int hipGetSymbolAddress(void **p, const void *) { ++g_calls; *p = reinterpret_cast<void *>(uintptr_t(1) << 40); return kOk; }
int hipHostMalloc(void **p, size_t n, unsigned)
{
    ++g_calls;
    *p = calloc(1, n);
    g_host[static_cast<unsigned char *>(*p)] = n;
    return kOk;
}
int hipHostFree(void *p)                           // (never handed out again, so that late writes do no harm)
{
    ++g_calls;
    CHECK(g_host.count(static_cast<unsigned char *>(p)) && g_released.insert(static_cast<unsigned char *>(p)).second);
    return kOk;
}
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { ++g_calls; return kOk; }
int hipStreamIsCapturing(void *, int *status) { ++g_calls; *status = g_capturing; return kOk; }
int hipThreadExchangeStreamCaptureMode(int *) { ++g_calls; return kOk; }
int hipStreamSynchronize(void *stream) { ++g_calls; ++g_syncs; gpu_runs(stream); return kOk; }

static bool in_host_memory(const unsigned char *p)
{
    for (auto &h : g_host)
        if (p >= h.first && p < h.first + h.second) return true;
    return false;
}
int hipLaunchKernel(const void *kernel, Dim3 grid, Dim3, void **args, size_t, void *stream)
{
    ++g_calls;
    if (g_fail_launch >= 0 && g_fail_launch-- == 0) return error(kErrorLaunchOutOfResources);
    ++g_launches;
    Work w;
    w.name = g_names[kernel];
    w.stream = stream;
    auto params = [&](const void *from) {
        for (size_t at = 0; at < kParamBytes; at += 8) {
            unsigned char *p;
            memcpy(&p, static_cast<const unsigned char *>(from) + at, 8);
            if (p >= g_ws && p < g_ws + g_ws_bytes) w.pointers.push_back(p);
            if (in_host_memory(p)) w.told = reinterpret_cast<uint32_t *>(p);
        }
    };
    if (w.name.find("dba_init_kernel") != std::string::npos) {
        w.B = (int)grid.x;
        w.words = *static_cast<const uint32_t **>(args[2]);
        w.seen = *static_cast<uint32_t **>(args[3]);
        params(args[4]);
    } else if (w.name.find("dba_sentence_kernel") != std::string::npos) {
        params(args[4]);
    } else if (w.name.find("dba_step_kernel") != std::string::npos) {
        params(args[8]);
    } else if (w.name.find("dba_merge_kernel") != std::string::npos) {
        params(args[3]);
    }
    if (w.told) {
        w.B = g_B;
        w.value = (uint32_t)g_step << 2;
    }
    g_queue.push_back(w);
    return kOk;
}
}  // extern "C"

// ---------------------------------------------------------------------------
// libdba
// ---------------------------------------------------------------------------
static void *g_lib;
#define LIB(name) reinterpret_cast<decltype(&name)>(dlsym(g_lib, #name))

static unsigned char *workspace(int B, int k, int V, int N)
{
    g_ws_bytes = LIB(dba_workspace_bytes)(B, k, V, N, 64);
    return g_ws = static_cast<unsigned char *>(aligned_alloc(256, (g_ws_bytes + 255) / 256 * 256));
}

static int init(dba_ctx **ctx, int B, int k, int V, int N, void *stream = nullptr)
{
    std::vector<int32_t> none(B + 1, 0);
    g_B = B;
    workspace(B, k, V, N);
    return LIB(dba_init)(ctx, B, k, V, N, 2, 0, nullptr, none.data(), none.data(), g_ws, g_ws_bytes, stream);
}

static int step(dba_ctx *ctx)
{
    g_step = LIB(dba_steps_done)(ctx) + 1;
    return LIB(dba_step)(ctx, reinterpret_cast<const float *>(uintptr_t(1) << 41), nullptr, nullptr, nullptr, nullptr);
}

static void ask(dba_ctx *ctx)
{
    std::vector<uint8_t> flags(g_B);
    CHECK(LIB(dba_get_finished)(ctx, flags.data()) == DBA_OK);
}

// the host memory block of the ctx that dba_init has launched last (for a kernel that has run or not)
static unsigned char *block_of_last_init()
{
    for (auto *list : {&g_queue, &g_done})
        for (size_t i = list->size(); i-- > 0;)
            if ((*list)[i].seen) return reinterpret_cast<unsigned char *>((*list)[i].seen);
    return nullptr;
}

// ---------------------------------------------------------------------------
// scenarios
// ---------------------------------------------------------------------------
// An error that is not the step's own, or its own: whatever the call makes of it, the block must not go to the next ctx
// while a kernel that may have been launched can still write to it.
static void a_step_that_reports_an_error(int told_before, bool own)
{
    dba_ctx *a = nullptr, *b = nullptr;
    CHECK(init(&a, 3, 4, 50, 9) == DBA_OK);
    ask(a);
    unsigned char *block = block_of_last_init();
    for (int i = 0; i < told_before; ++i) CHECK(step(a) == DBA_OK);
    gpu_runs();
    if (own) g_fail_launch = 0;
    else g_last_error = kErrorInvalidValue;
    const int rc = step(a);
    CHECK(rc == DBA_EHIP || (!own && rc == DBA_OK));
    CHECK(LIB(dba_steps_done)(a) == told_before + (rc == DBA_OK));
    bool under_way = false;
    for (const Work &w : g_queue) under_way = under_way || w.told;
    CHECK(under_way == !own);
    LIB(dba_destroy)(a);
    bool writes = false;
    for (const Work &w : g_queue) writes = writes || (w.told && reinterpret_cast<unsigned char *>(w.told) == block);
    CHECK(init(&b, 3, 4, 50, 9) == DBA_OK);
    CHECK(!writes || block_of_last_init() != block);
    gpu_runs();
    LIB(dba_destroy)(b);
}

static void launch_errors()
{
    for (int told = 0; told < 3; ++told)
        for (int own = 0; own < 2; ++own) a_step_that_reports_an_error(told, own != 0);
    // the same for dba_init, whose kernel reads the constraints from the block and writes to it
    for (int own = 0; own < 2; ++own) {
        dba_ctx *a = nullptr, *b = nullptr;
        if (own) g_fail_launch = 0;
        else g_last_error = kErrorInvalidValue;
        const int rc = init(&a, 3, 4, 50, 9);
        CHECK(own ? rc == DBA_EHIP : rc == DBA_EHIP || rc == DBA_OK);
        unsigned char *block = g_queue.empty() ? nullptr : block_of_last_init();
        CHECK((block == nullptr) == (own != 0));
        CHECK(init(&b, 3, 4, 50, 9) == DBA_OK);
        CHECK(block_of_last_init() != block);
        gpu_runs();
        if (rc == DBA_OK) LIB(dba_destroy)(a);
        LIB(dba_destroy)(b);
    }
    // calls that fail again and again keep nothing
    dba_ctx *c = nullptr;
    CHECK(init(&c, 3, 4, 50, 9) == DBA_OK);
    ask(c);
    CHECK(step(c) == DBA_OK);
    const size_t blocks = g_host.size();
    for (int i = 0; i < 100; ++i) {
        dba_ctx *none = nullptr;
        g_fail_launch = 0;
        CHECK(init(&none, 3, 4, 50, 9) == DBA_EHIP && !none);
        g_fail_launch = 0;
        CHECK(step(c) == DBA_EHIP);
    }
    CHECK(g_host.size() <= blocks + 1);
    CHECK(step(c) == DBA_OK && g_queue.back().told);       // (and the ctx goes on as before)
    gpu_runs();
    LIB(dba_destroy)(c);
}

// A step asks whether its stream is being captured and launches its kernels: the error that another call has left on the
// thread is not looked at, and stays there.
static void calls_of_a_step()
{
    const struct { int B, k, V, launches; const char *first, *last; } shapes[] = {
        {1, 5, 1000, 1, "dba_sentence_kernel", "dba_sentence_kernel"}, {1, 5, 1025, 1, "dba_step_kernel", "dba_step_kernel"},
        {16, 10, 32000, 1, "dba_step_kernel", "dba_step_kernel"}, {2, 40, 1000, 2, "dba_stream_kernel", "dba_merge_kernel"}};
    for (auto &s : shapes) {
        dba_ctx *c = nullptr;
        g_last_error = kErrorInvalidValue;
        CHECK(init(&c, s.B, s.k, s.V, 9) == DBA_OK);
        for (int t = 0; t < 4; ++t) {
            const int calls = g_calls, launches = g_launches;
            CHECK(step(c) == DBA_OK);
            CHECK(g_launches == launches + s.launches && g_calls == calls + 1 + s.launches);
            CHECK(g_queue[g_queue.size() - s.launches].name.find(s.first) != std::string::npos);
            CHECK(g_queue.back().name.find(s.last) != std::string::npos);
        }
        ask(c);
        CHECK(g_last_error == kErrorInvalidValue);
        // the first of two launches fails: there is nothing for the second
        g_fail_launch = 0;
        const int launches = g_launches;
        CHECK(step(c) == DBA_EHIP && g_launches == launches && LIB(dba_steps_done)(c) == 4);
        gpu_runs();
        LIB(dba_destroy)(c);
    }
}

// dba_destroy does not wait for steps and uses no stream for them; the block goes to another ctx only when the last step that
// writes to it has.
static void steps_under_way()
{
    auto stream = [](int i) { return reinterpret_cast<void *>(uintptr_t(i + 1)); };
    constexpr int kMany = 60;
    std::set<unsigned char *> blocks;
    const auto begin = std::chrono::steady_clock::now();
    for (int i = 0; i < kMany; ++i) {
        dba_ctx *c = nullptr;
        CHECK(init(&c, 5, 3, 60, 9, stream(i)) == DBA_OK);
        CHECK(blocks.insert(block_of_last_init()).second);
        ask(c);
        for (int t = 0; t < 2; ++t) CHECK(step(c) == DBA_OK && g_queue.back().told && g_queue.back().stream == stream(i));
        if (i % 2) gpu_runs(stream(i), 1);                 // the first of the two
        const int syncs = g_syncs;
        LIB(dba_destroy)(c);
        CHECK(g_syncs == syncs);
    }
    CHECK(std::chrono::steady_clock::now() - begin < std::chrono::seconds(1));
    CHECK(g_queue.size() == kMany + kMany / 2 && g_released.empty());
    for (int i = 0; i < kMany; i += 3) gpu_runs(stream(i));
    std::set<unsigned char *> again;
    for (int i = 0; i < kMany / 3; ++i) {                  // (all held at a time)
        dba_ctx *c = nullptr;
        CHECK(init(&c, 5, 3, 60, 9, stream(kMany)) == DBA_OK);
        CHECK(blocks.count(block_of_last_init()) && again.insert(block_of_last_init()).second);
    }
    for (const Work &w : g_queue) CHECK(!w.told || !again.count(reinterpret_cast<unsigned char *>(w.told)));
    dba_ctx *c = nullptr;
    CHECK(init(&c, 5, 3, 60, 9, stream(kMany)) == DBA_OK && !blocks.count(block_of_last_init()));
    gpu_runs();
    LIB(dba_destroy)(c);
    // all are through: what the store does not keep has been freed once the next block comes back
    CHECK(init(&c, 5, 3, 60, 9, stream(kMany)) == DBA_OK);
    ask(c);
    CHECK(step(c) == DBA_OK);
    gpu_runs();
    LIB(dba_destroy)(c);
    CHECK(g_host.size() - g_released.size() <= 32 + again.size());
}

// dba_init empties the places of steps of one launch where a step of some element type uses them, and there alone.
static void places_made_empty()
{
    const struct { int B, k, V; bool used; } shapes[] = {
        {16, 10, 32000, true}, {1, 5, 1000, false} /* a workgroup per sentence */, {1, 5, 1025, true} /* with 32 bits */, {1, 5, 2049, true},
        {89, 8, 41000, true} /* with 16 bits */, {89, 8, 82000, false}, {64, 20, 32000, true} /* with 16 bits */, {64, 29, 32000, false},
        {30, 17, 1000, true} /* with 32 bits */, {30, 17, 7500, false}, {30, 17, 8192, true}, {1409, 1, 1000, false}};
    for (auto &s : shapes) {
        dba_ctx *c = nullptr;
        CHECK(init(&c, s.B, s.k, s.V, 9) == DBA_OK);
        // the beam, the constraints, the flags and the records, then the lists and the keys
        const size_t n = g_queue.back().pointers.size();
        if (n != (s.used ? 6u : 4u)) printf("%d x %d x %d: %zu\n", s.B, s.k, s.V, n);
        CHECK(n == (s.used ? 6u : 4u));
        gpu_runs();
        LIB(dba_destroy)(c);
    }
}

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> scenarios = {
        {"launch_errors", launch_errors},
        {"calls_of_a_step", calls_of_a_step},
        {"steps_under_way", steps_under_way},
        {"places_made_empty", places_made_empty},
    };
    if (argc != 3 || !scenarios.count(argv[2])) return 2;
    g_lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!g_lib) { printf("%s\n", dlerror()); return 2; }
    CHECK(!g_names.empty());                               // (libdba has found the stand-in)
    scenarios.at(argv[2])();
    printf("%s ok\n", argv[2]);
    fflush(stdout);
    _exit(0);                                              // (nothing of the runtime library is shut down)
}
