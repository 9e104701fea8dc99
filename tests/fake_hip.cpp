// A stand-in for the HIP runtime and the kernel launchers, so that the library's host code (contexts, plans,
// steps, staging, the tuner) runs without a GPU: device memory is host memory, copies happen at once, launches
// are recorded.  A launcher told to fail returns an error.  One scenario per argument; see test_host_runtime.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <string>
#include <vector>

#include "sg_host.h"

using namespace sg;

struct Op {
    std::string what;
    const void* a;   // stream
    const void* b;   // event or counter
};
static std::vector<Op> g_ops;
static std::vector<const void*> g_waited;   // events the host waited for
static int g_pinned = 0;                   // pinned allocations
static int g_fail_psf_at = -1;             // the PSF launch that fails (counted from 0), -1: none
static int g_psf = 0;
static int g_fail_tx = 0;                  // every PSF launch of this tile width fails (-1: of any)
static void op(const char* w, const void* a = nullptr, const void* b = nullptr) { g_ops.push_back(Op{w, a, b}); }

#define CHECK(x)                                                               \
    do {                                                                       \
        if (!(x)) {                                                            \
            std::printf("line %d: %s\n", __LINE__, #x);                        \
            return 1;                                                          \
        }                                                                      \
    } while (0)

extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipMalloc(void** p, size_t n) { return *p = std::malloc(n), std::memset(*p, 0x5A, n), hipSuccess; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return ++g_pinned, *p = std::malloc(n), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memmove(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { return std::memmove(d, s, n), hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)std::malloc(8), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free(s), hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)std::calloc(1, 8), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    *(size_t*)e = g_ops.size();   // "time": operations so far
    return op("record", s, e), hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return g_waited.push_back(e), hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { return *ms = 0.01f * (float)(*(size_t*)b - *(size_t*)a), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { return op("wait", s, e), hipSuccess; }
}

namespace sg {
hipError_t launch_queue_reset(QueueDev* q, int n, hipStream_t s)
{
    for (int k = 0; k < n; ++k)
        for (auto& c : q[k].q) c.next = 0;
    return op("reset", s, q), hipSuccess;
}
hipError_t launch_upload(void* d, const void* h, size_t n, hipStream_t s) { return std::memcpy(d, h, n), op("upload", s), hipSuccess; }
hipError_t launch_upload_small(void* d, const void* h, size_t n, hipStream_t s) { return launch_upload(d, h, n, s); }
hipError_t launch_ray(const PhysArgs&, QueueDev* q, int, hipStream_t s)
{
    for (auto& c : q->q) c.next += 1;
    return op("ray", s, q), hipSuccess;
}
hipError_t launch_psf(const PhysArgs& a, int tx, int, hipStream_t s)
{
    if (g_psf++ == g_fail_psf_at || tx == g_fail_tx || g_fail_tx < 0) return hipErrorInvalidConfiguration;
    if (a.ray_queue)
        for (auto& c : a.ray_queue->q) c.next = 0;
    return op("psf", s, a.ray_queue), hipSuccess;
}
hipError_t launch_max_label(const uint8_t*, int64_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_brick_labels(const uint8_t*, int32_t, int32_t, int32_t, uint8_t*, hipStream_t) { return hipSuccess; }
int ray_grid(int n_cu, bool, bool, bool) { return 6 * n_cu; }
int psf_grid(int, int, int n_cu) { return 2 * n_cu; }
size_t psf_lds_bytes(int, int) { return 0; }
bool psf_tile_supported(int) { return true; }
hipError_t noalloc_init(int) { return hipSuccess; }
void surrogate_release_all(sg_ctx*) {}
void recon_release_all(sg_ctx*) {}
void SurrogateDeleter::operator()(Surrogate*) const {}
void ReconDeleter::operator()(Recon*) const {}
}  // namespace sg

struct World {
    sg_ctx* c = nullptr;
    int n;
    std::vector<uint8_t> labels = std::vector<uint8_t>(8 * 8 * 8, 1);
    std::vector<int32_t> vids;
    std::vector<sg_probe> probes;
    std::vector<int64_t> offs;
    std::vector<double> poses;
    std::vector<float> out;
    explicit World(int n_) : n(n_)
    {
        sg_create(&c, 0, nullptr);
        sg_volume_desc d;
        std::memset(&d, 0, sizeof(d));
        d.labels = labels.data();
        d.nx = d.ny = d.nz = 8;
        for (double& s : d.spacing_mm) s = 1.0;
        int32_t v = 0;
        sg_volume_register(c, &d, &v);
        sg_tissue t[2];
        std::memset(t, 0, sizeof(t));
        t[0].Z_mrayl = t[1].Z_mrayl = 1.5f;
        sg_tissue_table_set(c, t, 2);
        sg_probe p;
        std::memset(&p, 0, sizeof(p));
        p.W = 8;
        p.H = 16;
        p.dx_mm = p.dy_mm = 0.5;
        p.f_mhz = 5.0;
        p.E0 = 1.0;
        p.psf_frac = 0.01;
        p.dr_db = 60.0;
        p.n_elev = 1;
        vids.assign(n, v);
        probes.assign(n, p);
        for (int i = 0; i < n; ++i) {
            offs.push_back(128 * i);
            const double P[12] = {1, 0, 0, 4, 0, 1, 0, 4, 0, 0, 1, 0};
            poses.insert(poses.end(), P, P + 12);
        }
        out.resize(128 * (size_t)n);
    }
    ~World() { sg_destroy(c); }
    int plan()
    {
        int32_t id = -1;
        if (sg_batch_plan_create(c, n, vids.data(), probes.data(), offs.data(), &id) != SG_OK) std::printf("%s\n", sg_last_error());
        return id;
    }
    bool counters_zero(int id)
    {
        const QueueDev* q = (const QueueDev*)c->plans[id]->d_queue.p;
        for (int k = 0; k < kMaxChunks; ++k)
            for (const auto& s : q[k].q)
                if (s.next != 0) return false;
        return true;
    }
};

static const void* aux_of(World& w, int id) { return w.c->plans[id]->aux; }

// operations since `from`: the main stream waits for an event recorded on aux, and nothing is launched on aux later
static bool joined(size_t from, const void* aux)
{
    for (size_t i = from; i < g_ops.size(); ++i) {
        if (g_ops[i].what != "record" || g_ops[i].a != aux) continue;
        for (size_t j = i + 1; j < g_ops.size(); ++j)
            if (g_ops[j].what == "wait" && g_ops[j].a == nullptr && g_ops[j].b == g_ops[i].b) return true;
    }
    return false;
}

// a step cut short: the second stream joined, the counters cleared after that, on each entry point
static int failed_step()
{
    for (int profiled = 0; profiled < 2; ++profiled)
        for (int chunks = 1; chunks <= 4; chunks += 3)
            for (int at = 0; at < chunks; ++at) {
                World w(800);   // (more ray items than fit at once: the chunked step uses its second stream)
                const int id = w.plan();
                CHECK(id >= 0 && sg_batch_set_config(w.c, id, 4, 64, chunks) == SG_OK && w.counters_zero(id));
                g_ops.clear();
                g_psf = 0;
                g_fail_psf_at = at;
                float a, b;
                CHECK((profiled ? sg_batch_step_profiled(w.c, id, w.out.data(), &a, &b) : sg_batch_step(w.c, id, w.out.data())) == SG_EHIP);
                g_fail_psf_at = -1;
                CHECK(w.counters_zero(id));
                CHECK(g_ops.back().what == "reset");
                CHECK(chunks == 1 || joined(0, aux_of(w, id)));
                CHECK(sg_batch_step(w.c, id, w.out.data()) == SG_OK && w.counters_zero(id));
            }
    return 0;
}

// a launch shape whose steps fail is neither the tuner's choice nor in its cache, and leaves nothing behind
static int failed_tuning(const char* cache)
{
    World w(8);
    const int id = w.plan();
    CHECK(id >= 0);
    g_fail_tx = 64;
    CHECK(sg_autotune(w.c, id, cache) == SG_OK);
    g_fail_tx = 0;
    int32_t spw, tx, ty, ch;
    CHECK(sg_batch_config(w.c, id, &spw, &tx, &ty, &ch) == SG_OK && tx != 64);
    CHECK(w.counters_zero(id));
    std::ifstream f(cache);
    std::string line;
    int lines = 0;
    while (std::getline(f, line)) {
        ++lines;
        CHECK(line.find("\"tx\": 64") == std::string::npos);
    }
    CHECK(lines == 1);
    // every shape fails: the plan keeps its own, and nothing more is cached
    World v(9);
    const int iv = v.plan();
    CHECK(sg_batch_set_config(v.c, iv, 8, 16, 1) == SG_OK);
    g_fail_tx = -1;
    CHECK(sg_autotune(v.c, iv, cache) == SG_OK);
    g_fail_tx = 0;
    CHECK(sg_batch_config(v.c, iv, &spw, &tx, &ty, &ch) == SG_OK && spw == 8 && tx == 16 && ch == 1);
    CHECK(v.counters_zero(iv));
    std::ifstream again(cache);
    while (std::getline(again, line)) --lines;
    CHECK(lines == 0);
    return 0;
}

// the counters of single calls are at zero once the context is there, whether or not its first call runs (a call
// that a graph records does not)
static int first_call()
{
    World w(2);
    CHECK(w.c->queue.p);
    for (const auto& q : ((const QueueDev*)w.c->queue.p)->q) CHECK(q.next == 0);
    g_ops.clear();
    CHECK(sg_simulate(w.c, w.n, w.vids.data(), w.probes.data(), w.poses.data(), w.out.data(), w.offs.data(), nullptr) == SG_OK);
    for (const Op& o : g_ops) CHECK(o.what != "reset");
    return 0;
}

// uploads past the by-value limit: one pinned allocation for a series of calls, slots in turn, each waited for
// before it is written again, also where the sizes grow
static int staging()
{
    World w(40);   // 3840 bytes of poses
    const int id = w.plan();
    CHECK(id >= 0);
    g_pinned = 0;
    for (int k = 0; k < 9; ++k) {
        w.poses[12 * k + 3] = 0.5 * k;
        g_ops.clear();
        g_waited.clear();
        CHECK(sg_batch_set_poses(w.c, id, w.poses.data()) == SG_OK);
        CHECK(!std::memcmp(w.c->plans[id]->d_poses.p, w.poses.data(), 96 * 40));
        // the event waited for is the one recorded after this slot's upload, and each slot has its own
        CHECK(g_ops.size() == 2 && g_ops[0].what == "upload" && g_ops[1].what == "record");
        CHECK(k < kStagingSlots || (!g_waited.empty() && g_waited.front() == g_ops[1].b));
    }
    CHECK(g_pinned == 1);
    World v(200);
    const int iv = v.plan();
    g_pinned = 0;
    for (int k = 0; k < 9; ++k) {
        CHECK(sg_simulate(v.c, v.n, v.vids.data(), v.probes.data(), v.poses.data(), v.out.data(), v.offs.data(), nullptr) == SG_OK);
        CHECK(sg_batch_set_poses(v.c, iv, v.poses.data()) == SG_OK);
        CHECK(!std::memcmp(v.c->plans[iv]->d_poses.p, v.poses.data(), 96 * 200));
    }
    CHECK(g_pinned == 1);
    return 0;
}

int main(int argc, char** argv)
{
    const std::string s = argc > 1 ? argv[1] : "";
    if (s == "failed_step") return failed_step();
    if (s == "first_call") return first_call();
    if (s == "staging") return staging();
    if (s == "failed_tuning") return failed_tuning(argv[2]);
    std::printf("unknown scenario\n");
    return 2;
}
