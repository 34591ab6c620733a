// Drives hs_runtime.cpp on the CPU: the HIP calls and kernel launches that it makes are replaced by the
// stand-ins below ("device" memory is host memory, launches compute nothing, copies are done at once),
// which count what is alive and can be told to fail.  One check per name given on the command line.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../paper_2506_23917_amd/csrc/hs_common.hpp"

namespace {

struct FakeStream {
    int device;
    bool busy;                 // work enqueued and not waited for
};
struct FakeEvent {
    int device;
    FakeStream *on;
};

int g_device = 0;              // the calling thread's current device
int g_streams = 0, g_events = 0, g_pinned = 0;       // alive
int g_streams_made = 0;
size_t g_pinned_bytes = 0;    // page-locked so far
int g_fail_stream = -1;        // number of the stream whose creation fails
bool g_overlap = true;         // what the probe of a side stream sees
bool g_no_memory = false;      // operator new throws

FakeStream *fs(hipStream_t s) { return (FakeStream *)s; }
FakeEvent *fe(hipEvent_t e) { return (FakeEvent *)e; }
void work(void *stream) { ((FakeStream *)stream)->busy = true; }

}  // namespace

void *operator new(size_t n)
{
    void *p = g_no_memory ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return g_no_memory ? nullptr : std::malloc(n ? n : 1); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

extern "C" {

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    if (g_streams_made++ == g_fail_stream) return hipErrorOutOfMemory;
    ++g_streams;
    *s = (hipStream_t) new FakeStream{g_device, false};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    --g_streams;
    delete fs(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    fs(s)->busy = false;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    ++g_events;
    *e = (hipEvent_t) new FakeEvent{g_device, nullptr};
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    --g_events;
    delete fe(e);
    return hipSuccess;
}
// as the runtime has it: an event and the stream it is recorded on belong to one device
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (fe(e)->device != fs(s)->device) return hipErrorInvalidHandle;
    fe(e)->on = fs(s);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    if (fe(e)->on) fe(e)->on->busy = false;
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.f;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }

hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::malloc(n);
    ++g_pinned;
    g_pinned_bytes += n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    --g_pinned;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind)
{
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t s)
{
    work((void *)s);
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t s)
{
    work((void *)s);
    std::memset(p, v, n);
    return hipSuccess;
}

}  // extern "C"

namespace hsk {

void Launch::init_cells(const Ctx &, void *s) { work(s); }
void Launch::init_count(const Ctx &, void *s) { work(s); }
void Launch::init_fill(const Ctx &, void *s) { work(s); }
void Launch::init_finish(const Ctx &, void *s) { work(s); }
void Launch::scan_cells(const Ctx &, void *s) { work(s); }
void Launch::tile_table(const Ctx &, void *s) { work(s); }
void Launch::inject(const Ctx &, void *s) { work(s); }
void Launch::move_count(const Ctx &, void *s, int, int) { work(s); }
void Launch::scatter(const Ctx &, void *s) { work(s); }
void Launch::gather(const Ctx &, void *s) { work(s); }
void Launch::scalars(const Ctx &, void *s) { work(s); }
void Launch::collide(const Ctx &, void *s) { work(s); }
void Launch::dense(const Ctx &, void *s) { work(s); }
void Launch::finish_step(const Ctx &, void *s) { work(s); }
void Launch::philox(uint64_t, uint32_t, uint64_t, uint32_t, uint32_t, int64_t, uint32_t *, void *s) { work(s); }
// the output kernels leave 1, 2, 3, .. in the order of the fields
void launch_finalize(const Ctx &, void *s, int, int ncells, double *out)
{
    work(s);
    for (int k = 0; k < 8 * ncells; ++k) out[k] = k + 1;
}
void launch_moments_now(const Ctx &c, void *s, int k, int ncells, double *out) { launch_finalize(c, s, k, ncells, out); }
void launch_build_big(const Ctx &, void *s) { work(s); }
void launch_surface_finalize(const Ctx &, void *s, int, double *) { work(s); }
void launch_dsmc_ratio(const Ctx &, void *s, int, int, double *) { work(s); }
void launch_surface_reduce(const Ctx &, void *s, int, double *) { work(s); }
void launch_queue_probe(void *first, void *second, unsigned long long *t)
{
    work(first);
    work(second);
    t[0] = 100;
    t[1] = g_overlap ? 50 : 150;
}
int static_scratch(void **, size_t *) { return 1; }
int cap_wave() { return 192; }
int tile_width() { return 256; }
int cap_block(int) { return kCapBlockLds; }

}  // namespace hsk

namespace {

#define CHECK(x)                                                                     \
    do {                                                                             \
        if (!(x)) {                                                                  \
            std::printf("line %d: %s does not hold\n", __LINE__, #x);                \
            std::exit(1);                                                            \
        }                                                                            \
    } while (0)

// A sim of `n` one-dimensional cases of `ncells` cells on a stream of device `dev`.
struct Fixture {
    hs_gas gas;
    std::vector<hs_case> cases;
    std::vector<char> ws;
    FakeStream main;
    hs_sim *sim = nullptr;
    hs_status made;

    Fixture(int n, int ncells, int dev = 0, uint32_t flags = 0) : main{dev, false}
    {
        gas = {6.63e-26, 4.17e-10, 273.0, 0.81, 2.117e-5, 2.0 / 3.0, 5.0 / 3.0};
        hs_case c;
        std::memset(&c, 0, sizeof(c));
        c.dim = 1;
        c.nx = ncells;
        c.ny = c.nz = 1;
        for (double &h : c.h) h = 1.0;
        c.bc[0] = c.bc[1] = HS_BC_SPECULAR;
        for (int k = 2; k < 6; ++k) c.bc[k] = HS_BC_OUTFLOW;
        c.inflow.T = 1.0;
        c.F_N = 1.0;
        c.dt_G = 1e-3;
        c.T_sigma = 300.0;
        c.capacity = 64;
        cases.assign((size_t)n, c);
        for (int k = 0; k < n; ++k) cases[k].seed = 1 + k;       // (each its own random numbers)
        size_t bytes = 0;
        CHECK(hs_plan(&gas, cases.data(), n, HS_FP64, flags, &bytes) == HS_OK);
        ws.assign(bytes, 0);
        g_device = dev;
        made = hs_init_particles(&gas, cases.data(), n, HS_FP64, flags | HS_FLAG_NO_PARTICLES, ws.data(), bytes, (void *)&main, &sim);
    }
    ~Fixture()
    {
        hs_destroy(sim);
        if (g_streams || g_events || g_pinned) std::printf("left alive: %d streams, %d events, %d pinned\n", g_streams, g_events, g_pinned);
        if (g_streams || g_events || g_pinned) std::exit(1);
    }
};

// Reads the fields of a case into arrays of their own and checks them.
hs_status read_fields(hs_sim *sim, int c)
{
    const size_t nc = (size_t)hs_num_cells(sim, c);
    std::vector<double> f[4];
    for (int k = 0; k < 4; ++k) f[k].assign(k == 0 || k == 2 ? nc : 3 * nc, 0.0);
    const hs_status st = hs_sample_moments(sim, c, 0, f[0].data(), f[1].data(), f[2].data(), f[3].data(), nullptr);
    double want = 0.0;
    if (st == HS_OK)
        for (const auto &a : f)
            for (const double x : a) CHECK(x == ++want);
    return st;
}

// A side stream: the first that overlaps, else the last, also where a later one cannot be made.
void side_stream()
{
    for (int overlap = 0; overlap < 2; ++overlap)
        for (int fail = -1; fail < 4; ++fail) {
            g_overlap = overlap;
            g_streams_made = 0;
            g_fail_stream = fail;
            Fixture f(1, 8);
            g_fail_stream = -1;
            if (fail == 0) {
                CHECK(f.made != HS_OK && !f.sim);
            } else {
                CHECK(f.made == HS_OK && f.sim && g_streams == 1);
                CHECK(hs_step(f.sim, 2) == HS_OK);
            }
        }
    g_overlap = true;
}

// Steps and reads of a sim while another device is the thread's current one.
void other_device()
{
    Fixture f(2, 300, 1);
    CHECK(f.made == HS_OK);
    g_device = 0;
    for (int k = 0; k < 3; ++k) {
        CHECK(hs_step(f.sim, 1) == HS_OK);
        for (int c = 0; c < 2; ++c) CHECK(read_fields(f.sim, c) == HS_OK);
    }
}

// What a program that reads a sim once pays for: page-locking a megabyte or more costs more than it saves.
void first_read()
{
    for (const int ncells : {200, 10080, 100000}) {
        g_pinned_bytes = 0;
        Fixture f(2, ncells);
        CHECK(g_pinned_bytes == 0);
        for (int k = 0; k < 2; ++k)
            for (int c = 0; c < 2; ++c) CHECK(read_fields(f.sim, c) == HS_OK);
        CHECK(g_pinned_bytes < 1000000);
    }
}

// No exception leaves a read where the host's memory has run out (they need none).
void no_memory()
{
    Fixture f(3, 40000);
    std::vector<double> a(8 * 40000);
    int64_t out[HS_NUM_COUNTERS];
    double *n = a.data(), *u = n + 40000, *T = u + 3 * 40000, *q = T + 40000;
    for (int k = 0; k < 2; ++k) {
        g_no_memory = true;
        hs_status st = hs_counters(f.sim, 2, out);
        if (!st) st = hs_sample_moments(f.sim, 1, k, n, u, T, q, nullptr);
        if (!st) st = hs_sample_moments(f.sim, 1, k, T, n, nullptr, u, nullptr);
        g_no_memory = false;
        CHECK(st == HS_OK);
    }
}

// A read waits for its kernel also where no array is asked for.
void no_arrays()
{
    Fixture f(1, 500);
    for (int k = 0; k < 3; ++k) {
        int64_t samples = -1;
        CHECK(hs_sample_moments(f.sim, 0, 0, nullptr, nullptr, nullptr, nullptr, &samples) == HS_OK);
        CHECK(samples == 0 && !f.main.busy);
    }
}

struct Named {
    const char *name;
    void (*run)();
};
const Named kChecks[] = {{"side_stream", side_stream}, {"other_device", other_device}, {"first_read", first_read},
                         {"no_memory", no_memory}, {"no_arrays", no_arrays}};

}  // namespace

int main(int argc, char **argv)
{
    for (int k = 1; k < argc; ++k) {
        bool known = false;
        for (const Named &c : kChecks)
            if (std::string(argv[k]) == c.name) {
                known = true;
                c.run();
                std::printf("%s: ok\n", c.name);
            }
        if (!known) return 2;
    }
    return 0;
}
