// The library's host side (api.hip, compiled for the host alone) on a
// pretended device: memory is the host's, a stream is a queue of operations
// that run when the host waits for them, and the kernels' launchers are
// stand-ins that leave what the host reads of them.  Allocations and launches
// can be made to fail.  Each scenario prints "<name> <what it found>".
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <string>
#include <vector>

#include "fastmdp.h"
#include "planner.h"

namespace {

struct Stream {
    std::deque<std::function<void()>> q;
    void run_one() {
        auto f = std::move(q.front());
        q.pop_front();
        f();
    }
    void drain() {
        while (!q.empty()) run_one();
    }
};
struct Event {
    Stream *on = nullptr;
    bool done = true;
};
std::vector<Stream *> g_streams;
Stream g_null;
hipError_t g_last = hipSuccess;
size_t g_host_limit = ~(size_t)0, g_dev_limit = ~(size_t)0;   // larger allocations fail
bool g_fail_gather = false;
int g_range_launches = 0, g_other_launches = 0;

Stream *stream(hipStream_t s) { return s ? reinterpret_cast<Stream *>(s) : &g_null; }
Event *event(hipEvent_t e) { return reinterpret_cast<Event *>(e); }
hipError_t fail(hipError_t e) { return g_last = e; }
size_t pending() {
    size_t n = g_null.q.size();
    for (Stream *s : g_streams) n += s->q.size();
    return n;
}

}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *mem = std::calloc(1, (size_t)16 << 20);
    *p = mem;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
    if (n > g_dev_limit) return fail(hipErrorOutOfMemory);
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    if (n > g_host_limit) return fail(hipErrorOutOfMemory);
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 4;
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t *s) {
    g_streams.push_back(new Stream);
    *s = reinterpret_cast<hipStream_t>(g_streams.back());
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    stream(s)->drain();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    delete event(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    Event *v = event(e);
    v->on = stream(s);
    v->done = false;
    v->on->q.push_back([v] { v->done = true; });
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    while (!event(e)->done) event(e)->on->run_one();
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    stream(s)->q.push_back([e] { (void)hipEventSynchronize(e); });
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    g_null.drain();
    for (Stream *q : g_streams) q->drain();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    if (kind == hipMemcpyHostToDevice) {
        std::vector<char> held((const char *)s, (const char *)s + n);
        stream(st)->q.push_back([d, held] { std::memcpy(d, held.data(), held.size()); });
    } else {
        stream(st)->q.push_back([=] { std::memcpy(d, s, n); });
    }
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    stream(st)->q.push_back([=] { std::memset(d, v, n); });
    return hipSuccess;
}
}  // extern "C"

namespace fmdp {

bool planner_shape_supported(int, int, int) { return true; }
size_t features_workspace(int) { return 1; }
int mlp_weights(const fastmdp_mlp *, PropNet *) { return -1; }

// Every running request reaches its goal in 600 + id % 3 points of its own.
hipError_t launch_planner(int nblk, hipStream_t st, const DevCfg &c, const DevTable &t, Slot *s, const int *list,
                          const Traj &tr, int budget, int, int, const EvalOut &ev, const PropArgs &prop,
                          const LaunchStop &, const MatePeaks &) {
    const bool range = uses_range_planner(c, prop.mode) && !ev.V && budget > 1;
    if (range && (!t.Q || !t.grec || !t.goff || !t.gn)) return hipErrorInvalidValue;
    (range ? g_range_launches : g_other_launches) += 1;
    stream(st)->q.push_back([=] {
        for (int b = 0; b < nblk; ++b) {
            const int slot = list ? list[b] : b;
            Slot &S = s[slot];
            if (S.status != kRunning || budget < 1) continue;
            S.n_points = 600 + S.req % 3;
            for (int k = 0; k < S.n_points; ++k) {
                const size_t p = (size_t)slot * tr.stride + k;
                for (int a = 0; a < 3; ++a) tr.xyz[3 * p + a] = 100.0 * S.req + 10.0 * k + a;
                tr.act[p] = S.req + k;
                tr.val[p] = S.t0 + 0.5 * k;
            }
            S.status = FASTMDP_OK;
            S.valid = 1;
        }
    });
    return hipSuccess;
}
hipError_t launch_features(const DevCfg &, const DevTable &, int, const double *, const double *, const int *,
                           const int *, float *, int *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_fill_int(int *p, int v, int n, hipStream_t st) {
    stream(st)->q.push_back([=] { std::fill(p, p + n, v); });
    return hipSuccess;
}
hipError_t launch_quantise_table(const DevTable &, hipStream_t) { return hipSuccess; }
hipError_t launch_build_grid(const DevTable &t, int, hipStream_t) { return t.gn ? hipSuccess : hipErrorInvalidValue; }
hipError_t launch_scatter_points(const DevTable &, const float *, const int *, const int *, int, int, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_append_plans(const DevTable &, const int *, const int *, int, const float *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_commit(const DevCfg &, const DevTable &, const double *, int, int, int, int *, int *result,
                         hipStream_t st) {
    stream(st)->q.push_back([=] { *result = 0; });
    return hipSuccess;
}
hipError_t launch_gather_traj(const Slot *slots, const int *list, int n, const long long *off, long long total,
                              const Traj &tr, void *dst, hipStream_t st) {
    if (g_fail_gather) return hipErrorUnknown;
    stream(st)->q.push_back([=] {
        double *xyz = static_cast<double *>(dst), *val = xyz + 3 * total;
        int *act = reinterpret_cast<int *>(val + total);
        for (int i = 0; i < n; ++i)
            for (int k = 0; k < slots[list[i]].n_points; ++k) {
                const size_t p = (size_t)list[i] * tr.stride + k;
                for (int a = 0; a < 3; ++a) xyz[3 * (off[i] + k) + a] = tr.xyz[3 * p + a];
                act[off[i] + k] = tr.act[p];
                val[off[i] + k] = tr.val[p];
            }
    });
    return hipGetLastError();
}
hipError_t launch_batch_step(const DevCfg &, Slot *s, int n, const Traj &, const BatchState &bs, int, hipStream_t st) {
    stream(st)->q.push_back([=] {
        *bs.any = 0;
        for (int i = 0; i < n; ++i) *bs.any |= s[i].status == kRunning;
    });
    return hipSuccess;
}
hipError_t launch_fcfs_begin(const DevTable &, const PassBufs &, const DeathLog &, const DeathLog &, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_fcfs_pass(const DevCfg &, const DevTable &, Slot *s, const int *list, int n, const Traj &,
                            const DeathLog &, const DeathLog &, const PassBufs &pb, int, hipStream_t st) {
    stream(st)->q.push_back([=] {
        for (int i = 0; i < n; ++i) pb.mirror[list[i]] = s[list[i]];
    });
    return hipSuccess;
}
hipError_t launch_fcfs_abort(const DevTable &, Slot *, const int *, int, const Traj &, int, int, hipStream_t) {
    return hipSuccess;
}

}  // namespace fmdp

namespace {

fastmdp_config config(int range_query, int max_slots) {
    fastmdp_config c;
    std::memset(&c, 0, sizeof(c));
    for (int k = 0; k < 3; ++k) c.box_max[k] = 10000.0;
    c.dt = 1.0;
    c.gamma = c.gamma_intr = c.gamma_terr = 0.99;
    c.r_goal = c.r_intr = c.r_terr = 1.0;
    c.R_intr = c.R_sep = c.R_terr = 150.0;
    c.n_head = 9;
    c.n_climb = c.n_speed = 3;
    for (int k = 0; k < 3; ++k) {
        c.climb[k] = 5.0 * (k - 1);
        c.speed[k] = 20.0 + 10.0 * k;
    }
    c.max_steps = 3600;
    c.plan_capacity = 64;
    c.max_rows = 3601;
    c.max_slots = max_slots;
    c.tie_rel = 1e-9;
    c.range_query = range_query;
    return c;
}

struct Plans {
    std::vector<fastmdp_plan> p;
    std::vector<std::vector<double>> xyz, val;
    std::vector<std::vector<int>> act;
    explicit Plans(int n) : p(n), xyz(n), val(n), act(n) {
        for (int i = 0; i < n; ++i) {
            xyz[i].assign(3 * 3601, -1.0);
            val[i].assign(3601, -1.0);
            act[i].assign(3601, -1);
            p[i] = fastmdp_plan{-9, 0, 0, 3601, xyz[i].data(), act[i].data(), val[i].data()};
        }
    }
    // plan i is request i's as the stand-in left it
    bool whole() const {
        for (int i = 0; i < (int)p.size(); ++i) {
            if (p[i].status != FASTMDP_OK || p[i].n_points != 600 + i % 3) return false;
            for (int k = 0; k < p[i].n_points; ++k)
                if (xyz[i][3 * k] != 100.0 * i + 10.0 * k || xyz[i][3 * k + 2] != 100.0 * i + 10.0 * k + 2 ||
                    act[i][k] != i + k || val[i][k] != p[i].t0 + 0.5 * k)
                    return false;
        }
        return true;
    }
};

void tell(const char *name, int rc, bool whole) {
    std::printf("%s rc=%d pending=%zu whole=%d range=%d other=%d\n", name, rc, pending(), (int)whole, g_range_launches,
                g_other_launches);
    std::fflush(stdout);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    const int n = argc > 2 ? std::atoi(argv[2]) : 8;
    const bool no_index = what == "no_index", no_host = argc > 3 && std::string(argv[3]) == "no_host_memory";
    g_fail_gather = argc > 3 && std::string(argv[3]) == "no_gather";
    // the index's records are the table's largest arrays
    if (no_index) g_dev_limit = (size_t)3601 * 64 * 4;
    fastmdp_ctx *ctx = nullptr;
    int rc = fastmdp_create(nullptr, &ctx);
    const fastmdp_config cfg = config(1, no_index ? 1 : 80);
    rc = fastmdp_create(&cfg, &ctx);
    if (rc) {
        tell("create", rc, false);
        return 0;
    }
    std::vector<fastmdp_request> reqs(n);
    std::vector<int> t0(n), committed(n);
    for (int i = 0; i < n; ++i) {
        reqs[i] = fastmdp_request{(uint64_t)i, {1.0, 2.0, 3.0}, {4.0, 5.0, 6.0}, 0};
        t0[i] = 3 * i;
    }
    if (no_host) g_host_limit = 0;
    for (int pass = 0; pass < 2; ++pass) {               // the second once there is memory again
        Plans plans(n);
        int chosen = -2;
        if (what == "request" || no_index) rc = fastmdp_plan_request(ctx, &reqs[0], &plans.p[0]);
        else if (what == "departures") rc = fastmdp_plan_departures(ctx, &reqs[0], n, t0.data(), plans.p.data(), &chosen);
        else if (what == "batch") rc = fastmdp_plan_batch(ctx, n, reqs.data(), plans.p.data());
        else if (what == "fcfs") rc = fastmdp_plan_fcfs(ctx, n, reqs.data(), nullptr, plans.p.data(), committed.data(), nullptr);
        tell(what.c_str(), rc, plans.whole());
        g_host_limit = ~(size_t)0;
        g_fail_gather = false;
    }
    fastmdp_destroy(ctx);
    return 0;
}
