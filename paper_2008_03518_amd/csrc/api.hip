// api.hip -- host side of libfastmdp: the C ABI declared in include/fastmdp.h.
//
// The context owns the device state: the time-major SoA known-plan table,
// the terrain heightmap, per-slot trajectory buffers and small scratch.  A
// host mirror of the per-row entry counts is kept for capacity checks and
// for loading plans.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <thread>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "fastmdp.h"
#include "planner.h"

using fmdp::DeathLog;
using fmdp::DevCfg;
using fmdp::DevTable;
using fmdp::EvalOut;
using fmdp::Slot;
using fmdp::Traj;

// Staging of fastmdp_load_plans_noalloc: a fixed device array, one copy on
// every GPU the library runs on, held until the process ends.  Plan starts
// and lengths take the first kNoallocPlanBytes, the FP32 points the rest.
// Host code never passes `scratch` itself (its name is a host-side stand-in,
// not a device address): it uses the address hipGetSymbolAddress returns on
// each device (noalloc_scratch).
constexpr int kNoallocMaxPlans = 65536;
constexpr int kNoallocMaxPoints = 655360;
constexpr size_t kNoallocPlanBytes = (size_t)2 * kNoallocMaxPlans * sizeof(int);
constexpr size_t kNoallocBytes = kNoallocPlanBytes + (size_t)3 * kNoallocMaxPoints * sizeof(float);   // 8 MiB
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch[kMaxDevices] = {};

// Device address of `scratch` on device dev (current), looked up once per
// device.  nullptr if the lookup fails.
void *noalloc_scratch(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) {
            std::fprintf(stderr, "libfastmdp: hipGetSymbolAddress(scratch) failed on device %d\n", dev);
            return nullptr;
        }
        g_scratch[dev] = p;
    }
    return g_scratch[dev];
}
}  // namespace

struct fastmdp_ctx {
    fastmdp_config cfg{};
    DevCfg dc{};
    DevTable tb{};
    int A = 0;
    hipStream_t own = nullptr, stream = nullptr;
    std::vector<int> hRowN;
    int n_plans = 0;
    int seq = 0;                          // next request sequence number (table entry owners are below it)
    // the rows' grids (fmdp::DevTable): built, over at most gridRowN entries
    // of each row (empty: built during a planning call, whose row counts the
    // host does not hold) when the table held grid_plans plans
    bool grid_ok = false;
    std::vector<int> gridRowN;
    int grid_plans = 0;
    std::vector<int> snapRowN;            // table snapshot (row counts)
    int snap_plans = 0;
    float *dTerr = nullptr;
    int max_slots = 1, stride = 0;
    int n_cu = 256;                       // compute units of the device
    int dev = 0;                          // HIP device of the context
    void *dScratch = nullptr;             // this device's `scratch` (allocation-free plan loading)
    std::vector<int> hRowTmp;             // row counts being checked by fastmdp_load_plans_noalloc
    Slot *dSlots = nullptr;
    Traj tr{};
    // pinned host memory of the calls for one state or plan, which the
    // kernels read and write in place: eval outputs (4 * A), a trajectory to
    // commit (stride * 3), and hInt = {best action, commit result, aircraft of
    // a batch still flying}
    double *hIo = nullptr, *hPts = nullptr;
    int *hInt = nullptr;
    int *dFlag = nullptr;         // commit check: per point
    int *dFeatWs = nullptr;       // fastmdp_features: grouping of the states by row (made when first used)
    DeathLog dl[2]{};                     // FCFS withdrawals: of the last pass and of the one running
    int *dRowNPre = nullptr, *dInsN = nullptr;   // acceptance-pass work buffers (fmdp::PassBufs)
    int4 *dIns = nullptr;
    float4 *dBox = nullptr;
    // pinned host mirrors and the trajectory gather buffers of the FCFS engine
    Slot *hSlots = nullptr;
    void *hGather = nullptr;
    size_t gather_cap = 0;                // bytes
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipEvent_t eGather = nullptr;         // after the last trajectory gather's copy to the host
    hipStream_t gstream = nullptr;        // the gathers' stream: their copies leave the planning stream free
    // pinned lists of the engine's rounds, read by the kernels in place (each
    // is rewritten only after the round's synchronisation): gather offsets,
    // the launch list, the pass list and the gather list
    void *hRound = nullptr;
    long long *hOff = nullptr;
    int *hList = nullptr, *hPass = nullptr, *hList2 = nullptr;
    // learned action proposal
    fmdp::PropArgs prop{};
    float *dEvF = nullptr;        // proposal eval outputs: features, logits
    int *dEvI = nullptr;          // top-k, certified, proposal's action
    int *dStop = nullptr;         // finished-workgroup counter of a planner launch
    fmdp::BatchState bs{};        // co-simulated batch: peaks and step bookkeeping
    std::mutex mu;
    // counters of the last call
    long long st_pairs = 0, st_steps = 0, st_resumes = 0, st_launches = 0, st_entries = 0;
    long long st_hit = 0, st_miss = 0;
    double st_ms = 0.0;
};

namespace {

#define HIP_TRY(x)                                                                                  \
    do {                                                                                            \
        hipError_t e_ = (x);                                                                        \
        if (e_ != hipSuccess) {                                                                     \
            std::fprintf(stderr, "libfastmdp: %s failed: %s\n", #x, hipGetErrorString(e_));         \
            return FASTMDP_E_DEVICE;                                                                \
        }                                                                                           \
    } while (0)

template <class T>
int dev_alloc(T **p, size_t n) {
    *p = nullptr;
    if (n == 0) return 0;
    if (hipMalloc(reinterpret_cast<void **>(p), n * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();           // reported here, not by the next launch
        *p = nullptr;
        return FASTMDP_E_NOMEM;
    }
    return 0;
}

void free_all(fastmdp_ctx *c) {
    hipFree(c->tb.X); hipFree(c->tb.Y); hipFree(c->tb.Z); hipFree(c->tb.rowN);
    hipFree(c->tb.vis); hipFree(c->tb.own); hipFree(c->tb.dead);
    hipFree(c->tb.Q); hipFree(c->tb.grec); hipFree(c->tb.goff); hipFree(c->tb.gn);
    for (DeathLog &d : c->dl) {
        hipFree(d.x); hipFree(d.y); hipFree(d.z); hipFree(d.col);
        hipFree(d.seg); hipFree(d.seg_box); hipFree(d.box); hipFree(d.n);
    }
    hipFree(c->dRowNPre); hipFree(c->dIns); hipFree(c->dInsN); hipFree(c->dBox);
    hipFree(c->dTerr);
    hipFree(c->dSlots);
    hipFree(c->tr.xyz); hipFree(c->tr.act); hipFree(c->tr.val); hipFree(c->tr.seen); hipFree(c->tr.top);
    hipFree(c->tr.ep); hipFree(c->tr.col); hipFree(c->tr.nd); hipFree(c->tr.seenw);
    hipFree(c->dFlag); hipFree(c->dFeatWs);
    if (c->hIo) hipHostFree(c->hIo);
    if (c->hSlots) hipHostFree(c->hSlots);
    if (c->hGather) hipHostFree(c->hGather);
    hipFree(c->dEvF); hipFree(c->dEvI); hipFree(c->dStop);
    hipFree(c->bs.pk); hipFree(c->bs.owner); hipFree(c->bs.n); hipFree(c->bs.active); hipFree(c->bs.prev_n);
    
    if (c->e0) hipEventDestroy(c->e0);
    if (c->e1) hipEventDestroy(c->e1);
    if (c->eGather) hipEventDestroy(c->eGather);
    if (c->hRound) hipHostFree(c->hRound);
    if (c->own) hipStreamDestroy(c->own);
    if (c->gstream) hipStreamDestroy(c->gstream);
}

int check_cfg(const fastmdp_config *c) {
    if (!c) return FASTMDP_E_INVAL;
    if (c->n_head < 1 || c->n_head > fmdp::kMaxHeads) return FASTMDP_E_INVAL;
    if (c->n_climb < 1 || c->n_climb > FASTMDP_MAX_ACT_DIM) return FASTMDP_E_INVAL;
    if (c->n_speed < 1 || c->n_speed > FASTMDP_MAX_ACT_DIM) return FASTMDP_E_INVAL;
    if ((long)c->n_head * c->n_climb * c->n_speed > fmdp::kMaxActions) return FASTMDP_E_INVAL;
    if (!(c->dt > 0.0) || !(c->gamma > 0.0 && c->gamma < 1.0)) return FASTMDP_E_INVAL;
    if (!(c->gamma_intr > 0.0 && c->gamma_intr < 1.0) || !(c->gamma_terr > 0.0 && c->gamma_terr < 1.0))
        return FASTMDP_E_INVAL;
    for (int v = 0; v < c->n_speed; ++v)
        if (!(c->speed[v] > 0.0)) return FASTMDP_E_INVAL;
    if (c->max_steps < 1 || c->max_steps + 1 > fmdp::kMaxPoints || c->max_rows < 2) return FASTMDP_E_INVAL;
    // rows are read four entries (16 bytes) per lane
    if (c->plan_capacity < 4 || c->plan_capacity % 4 != 0)
        return FASTMDP_E_INVAL;
    if (!(c->tie_rel >= 0.0)) return FASTMDP_E_INVAL;
    if (c->lookahead < 0 || c->lookahead > fmdp::kMaxLookahead) return FASTMDP_E_INVAL;
    if (c->range_query != 0 && c->range_query != 1) return FASTMDP_E_INVAL;
    if (c->planner_threads != 0 && c->planner_threads != fmdp::kPlanThreads &&
        !((c->planner_threads == fmdp::kRangeThreads || c->planner_threads == fmdp::kRangeThreadsSolo) &&
          c->range_query == 1 && c->lookahead <= 1 && c->n_head <= fmdp::kRangeMaxHeads))
        return FASTMDP_E_INVAL;
    if (!(c->peak_growth >= 0.0)) return FASTMDP_E_INVAL;
    return 0;
}

void make_devcfg(const fastmdp_config &c, DevCfg &d) {
    std::memset(&d, 0, sizeof(d));
    for (int k = 0; k < 3; ++k) { d.box_lo[k] = c.box_min[k]; d.box_hi[k] = c.box_max[k]; }
    double vmax = 0.0;
    for (int v = 0; v < c.n_speed; ++v) vmax = std::max(vmax, c.speed[v]);
    d.dt = c.dt;
    d.ell = vmax * c.dt;
    d.gamma = c.gamma; d.r_goal = c.r_goal;
    d.r_intr = c.r_intr; d.R_intr = c.R_intr; d.gamma_intr = c.gamma_intr;
    d.R_sep = c.R_sep;
    d.r_terr = c.r_terr; d.R_terr = c.R_terr; d.gamma_terr = c.gamma_terr;
    d.clear_terr = std::max(c.R_terr, 0.0);
    d.log_gamma = std::log(c.gamma);
    d.log_gamma_intr = std::log(c.gamma_intr);
    d.log_gamma_terr = std::log(c.gamma_terr);
    d.abs_r_goal = std::fabs(c.r_goal);
    d.abs_r_intr = std::fabs(c.r_intr);
    d.abs_r_terr = std::fabs(c.r_terr);
    d.log2_gamma_f = (float)std::log2(c.gamma);
    d.inv_ell_f = (float)(1.0 / d.ell);
    d.abs_r_goal_f = (float)d.abs_r_goal;
    for (int k = 0; k < FASTMDP_MAX_ACT_DIM; ++k) {
        d.climb[k] = c.climb[k];
        d.speed[k] = c.speed[k];
        d.climb_f[k] = (float)c.climb[k];
        d.kv[k] = (float)(-2.0 * c.speed[k] * c.dt);
    }
    d.zeta_scale = (float)(-2.0 * c.dt);
    d.tie_rel = c.tie_rel;
    d.reach = std::max(c.R_intr, c.R_sep) + 1.0;
    d.band_lo2 = std::max(c.R_intr - fmdp::kBand, 0.0) * std::max(c.R_intr - fmdp::kBand, 0.0);
    d.band_hi2 = (c.R_intr + fmdp::kBand) * (c.R_intr + fmdp::kBand);
    double cmax = 0.0;
    for (int k = 0; k < c.n_climb; ++k) cmax = std::max(cmax, std::fabs(c.climb[k]));
    d.reach_state = d.reach + std::sqrt(vmax * vmax + cmax * cmax) * c.dt;
    d.n_head = c.n_head; d.n_climb = c.n_climb; d.n_speed = c.n_speed;
    d.n_actions = c.n_head * c.n_climb * c.n_speed;
    const int mid = c.n_climb / 2;
    d.zero_climb = (c.climb[mid] == 0.0) ? mid : -1;
    d.max_steps = c.max_steps;
    d.lookahead = c.lookahead > 1 ? c.lookahead : 1;
    d.max_step = std::sqrt(vmax * vmax + cmax * cmax) * c.dt;
    d.range_query = c.range_query ? 1 : 0;
    d.peak_growth = c.peak_growth;
    // every point scored in a step lies within lookahead * max_step of the
    // state; a plan farther than reach from all of them changes nothing
    const double rc = d.reach + d.lookahead * d.max_step + 1.0;
    d.cull_r2 = (float)(rc * rc);
    // Box test of the range-query planner: an entry the exact test keeps has
    // |q_x|, |q_y| < sqrt(cull_r2) (1 + 2^-23), and the FP32 offset of the
    // box test differs from q_x by under |state| 2^-24 plus 2 |q_x| 2^-24.
    double max_abs = 0.0;
    for (int k = 0; k < 3; ++k) max_abs = std::max({max_abs, std::fabs(c.box_min[k]), std::fabs(c.box_max[k])});
    d.cull_box = (float)(std::sqrt((double)d.cull_r2) * 1.001 + 1.0 + max_abs * 1e-6);
    // Two goal terms differ by more than the tie band when their distances
    // differ by more than m ell / |log gamma|, m = -log(1 - tie_rel) plus
    // what the rounding of the two computed terms can hide: below 1e-12
    // while the exponent |log gamma| d / ell is at most 600 (the exponent's
    // relative error is a few 2^-53, the exponential's as well).
    d.run_ok = d.abs_r_goal > 0.0 && c.tie_rel <= 1e-3 ? 1 : 0;
    d.run_c1 = c.n_head > 1 ? std::cos(2.0 * M_PI / c.n_head) : -1e9;
    // half-widths of the box test on 16-bit coordinates: the staging radius
    // plus both roundings (half a step each), the FP32 arithmetic's (under a
    // step) and the FP32 state's (2^-24 of the coordinates)
    d.run_r = d.run_w = d.run_step = 0u;
    for (int k = 0; k < 2; ++k) {
        const double scale = 65535.0 / (c.box_max[k] - c.box_min[k]);
        const double r = std::ceil((std::sqrt((double)d.cull_r2) * 1.001 + max_abs * 1e-6) * scale) + 3.0;
        const double m = std::ceil(d.max_step * scale);
        const bool fits = r > 0.0 && m >= 0.0 && r + 32.0 * m < 32000.0;
        if (!fits) d.run_ok = 0;
        d.run_r |= (fits ? (uint32_t)r : 0u) << (16 * k);
        d.run_w |= (fits ? 2u * (uint32_t)r : 0xffffu) << (16 * k);
        d.run_step |= (fits ? (uint32_t)m : 0u) << (16 * k);
    }
    // The goal terms of a step's actions differ by at most the factor
    // gamma^-(2 max_step / ell); an action inside a well loses at least the
    // well's value at its radius.
    const double well = d.abs_r_intr * std::exp(d.log_gamma_intr * (c.R_intr / d.ell)) * (1.0 - 1e-9);
    const double spread = std::exp(-d.log_gamma * (2.0 * d.max_step / d.ell)) - 1.0;
    d.detour_ok = d.run_ok && d.abs_r_goal * (spread * (1.0 + 1e-9) + 2.0 * c.tie_rel + 1e-9) < well ? 1 : 0;
    d.run_margin = (-std::log1p(-std::min(c.tie_rel, 0.5)) * 1.001 + 2e-12) * d.ell / std::fabs(d.log_gamma);
    d.run_dmax = 600.0 * d.ell / std::fabs(d.log_gamma);
    d.run_v = 0;
    for (int v = 1; v < c.n_speed; ++v)
        if (c.speed[v] > c.speed[d.run_v]) d.run_v = v;
    d.planner_threads = c.planner_threads;
    d.n_cu = 256;                          // the device's count is set once the context knows it
}

// Adds the last planner launch's duration (its events have completed).
int planner_time(fastmdp_ctx *c) {
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, c->e0, c->e1));
    c->st_ms += ms;
    c->st_launches += 1;
    return 0;
}

int timed_planner(fastmdp_ctx *c, int nblk, const int *list, int budget, int validate, int epoch,
                  const EvalOut &ev, Slot *slots, int stop_target = 0, bool sync = true) {
    HIP_TRY(hipEventRecord(c->e0, c->stream));
    const fmdp::LaunchStop stop{c->dStop, stop_target};
    hipError_t e = fmdp::launch_planner(nblk, c->stream, c->dc, c->tb, slots, list, c->tr, budget, validate,
                                        epoch, ev, c->prop, stop, fmdp::MatePeaks{});
    if (e != hipSuccess) {
        std::fprintf(stderr, "libfastmdp: planner launch failed: %s\n", hipGetErrorString(e));
        return FASTMDP_E_DEVICE;
    }
    HIP_TRY(hipEventRecord(c->e1, c->stream));
    if (!sync) return 0;                     // the caller synchronises, then calls planner_time
    HIP_TRY(hipEventSynchronize(c->e1));
    return planner_time(c);
}

// The range-query planner's index of the rows, after everything a context
// cannot do without.  Where there is no memory for it (20 bytes an entry and
// 4 KB a row, beside the table's 24 bytes an entry) the requests are planned
// on the 1024-thread kernel, which reads the table itself: the same plans.
void alloc_index(fastmdp_ctx *c) {
    DevTable &t = c->tb;
    const size_t rows = (size_t)c->cfg.max_rows, entries = rows * c->cfg.plan_capacity;
    if (dev_alloc(&t.Q, entries) == 0 && dev_alloc(&t.grec, entries) == 0 &&
        dev_alloc(&t.goff, rows * (fmdp::kGridCells + 1)) == 0 && dev_alloc(&t.gn, rows) == 0)
        return;
    hipFree(t.Q); hipFree(t.grec); hipFree(t.goff); hipFree(t.gn);
    t.Q = nullptr;
    t.grec = nullptr;
    t.goff = t.gn = nullptr;
    c->dc.planner_threads = fmdp::kPlanThreads;
}

// The rows' grids, before a range-query planner launch: built when there are
// none, or when the entries appended since (searched one by one) have grown
// to a quarter of the indexed ones.  `limit` as launch_build_grid; in_call:
// during a planning call.
int refresh_grid(fastmdp_ctx *c, int limit, bool in_call) {
    if (!fmdp::uses_range_planner(c->dc, c->prop.mode)) return 0;
    if (c->grid_ok && c->n_plans - c->grid_plans < std::max(in_call ? 1024 : 256, c->grid_plans / 4)) return 0;
    HIP_TRY(fmdp::launch_build_grid(c->tb, limit, c->stream));
    c->grid_ok = true;
    c->grid_plans = c->n_plans;
    if (in_call) c->gridRowN.clear();
    else c->gridRowN = c->hRowN;
    return 0;
}

// The table's rows, for the choice of the kernel of launches of many requests.
void note_rows(fastmdp_ctx *c) { c->dc.longest_row = *std::max_element(c->hRowN.begin(), c->hRowN.end()); }

void reset_stats(fastmdp_ctx *c) {
    c->st_pairs = c->st_steps = c->st_resumes = c->st_launches = c->st_entries = 0;
    c->st_hit = c->st_miss = 0;
    c->st_ms = 0.0;
}

Slot fresh_slot(const fastmdp_request &r, int req_index, int seq) {
    Slot s;
    std::memset(&s, 0, sizeof(s));
    s.seq = seq;
    s.origin[0] = r.origin.x; s.origin[1] = r.origin.y; s.origin[2] = r.origin.z;
    s.goal[0] = r.goal.x; s.goal[1] = r.goal.y; s.goal[2] = r.goal.z;
    s.t0 = r.t0;
    s.n_points = 0;
    s.status = fmdp::kRunning;
    s.req = req_index;
    s.resume_at = -1;
    return s;
}

// Accepted trajectories on their way to the caller's plans: the device
// packs them into one pinned host buffer; the host unpacks after a later
// synchronisation.
struct PendingPlans {
    std::vector<int> slots, reqs, n, status, t0;
    std::vector<long long> off;
    long long total = 0;
    bool empty() const { return reqs.empty(); }
};

constexpr size_t kPointBytes = 4 * sizeof(double) + sizeof(int);      // a gathered point

// A call that returns early waits for what it has enqueued: the kernels read
// and write the context's pinned memory in place, and the next call fills it
// anew.  (Behind the context's lock, so that the lock is held meanwhile.)
struct Drain {
    fastmdp_ctx *c;
    bool done = false;                     // nothing is left in flight
    ~Drain() {
        if (done) return;
        (void)hipStreamSynchronize(c->stream);
        (void)hipStreamSynchronize(c->gstream);
    }
};

// The pinned gather buffer, grown to `bytes` (no copy into it is in flight);
// without memory for that the one there is stays.
int gather_reserve(fastmdp_ctx *c, size_t bytes) {
    if (bytes <= c->gather_cap) return 0;
    size_t cap = std::max(bytes, 2 * c->gather_cap);
    void *p = nullptr;
    if (hipHostMalloc(&p, cap) != hipSuccess) {
        (void)hipGetLastError();
        cap = bytes;
        if (hipHostMalloc(&p, cap) != hipSuccess) {
            (void)hipGetLastError();
            return FASTMDP_E_NOMEM;
        }
    }
    if (c->hGather) hipHostFree(c->hGather);
    c->hGather = p;
    c->gather_cap = cap;
    return 0;
}

// No pinned buffer to be had: the trajectories copied one by one into the
// caller's plans (the streams that wrote them have been waited for).
int plans_copy(fastmdp_ctx *c, const std::vector<int> &slots, const std::vector<int> &reqs, const Slot *hs,
               fastmdp_plan *plans) {
    for (size_t i = 0; i < slots.size(); ++i) {
        const Slot &s = hs[slots[i]];
        fastmdp_plan &p = plans[reqs[i]];
        const size_t base = (size_t)slots[i] * c->stride, n = (size_t)s.n_points;
        HIP_TRY(hipMemcpy(p.xyz, c->tr.xyz + base * 3, n * 3 * sizeof(double), hipMemcpyDeviceToHost));
        HIP_TRY(hipMemcpy(p.action, c->tr.act + base, n * sizeof(int), hipMemcpyDeviceToHost));
        HIP_TRY(hipMemcpy(p.value, c->tr.val + base, n * sizeof(double), hipMemcpyDeviceToHost));
        p.status = s.status;
        p.t0 = s.t0;
        p.n_points = s.n_points;
    }
    return 0;
}

// pp: the trajectories that are on their way (none without memory for the
// buffer: they are in the caller's plans on return).

int gather_enqueue(fastmdp_ctx *c, const Slot *dslots, const std::vector<int> &slots, const std::vector<int> &reqs, const Slot *hs,
                   fastmdp_plan *plans, PendingPlans &pp) {
    const int m = (int)slots.size();
    pp = PendingPlans();
    PendingPlans q;
    q.slots = slots;
    q.reqs = reqs;
    q.off.resize(m);
    for (int i = 0; i < m; ++i) {
        const Slot &s = hs[slots[i]];
        if (plans[reqs[i]].capacity < s.n_points) return FASTMDP_E_CAPACITY;
        q.off[i] = q.total;
        q.total += s.n_points;
        q.n.push_back(s.n_points);
        q.status.push_back(s.status);
        q.t0.push_back(s.t0);
    }
    if (m > c->max_slots) return FASTMDP_E_CAPACITY;
    if (gather_reserve(c, (size_t)q.total * kPointBytes)) return plans_copy(c, slots, reqs, hs, plans);
    std::memcpy(c->hList2, q.slots.data(), m * sizeof(int));
    std::memcpy(c->hOff, q.off.data(), m * sizeof(long long));
    // on the gathers' own stream, so that the planning stream's next launch
    // does not wait for the copy; the caller has synchronised the planning
    // stream, and nothing it runs before these slots are reused writes them
    HIP_TRY(fmdp::launch_gather_traj(dslots, c->hList2, m, c->hOff, q.total, c->tr, c->hGather, c->gstream));
    HIP_TRY(hipEventRecord(c->eGather, c->gstream));
    pp = std::move(q);
    return 0;
}

// After a synchronisation that follows gather_enqueue.
void gather_unpack(fastmdp_ctx *c, PendingPlans &pp, fastmdp_plan *plans) {
    const double *xyz = static_cast<const double *>(c->hGather);
    const double *val = xyz + 3 * pp.total;
    const int *act = reinterpret_cast<const int *>(val + pp.total);
    for (size_t i = 0; i < pp.reqs.size(); ++i) {
        fastmdp_plan &p = plans[pp.reqs[i]];
        const int n = pp.n[i];
        std::memcpy(p.xyz, xyz + 3 * pp.off[i], (size_t)n * 3 * sizeof(double));
        std::memcpy(p.action, act + pp.off[i], (size_t)n * sizeof(int));
        std::memcpy(p.value, val + pp.off[i], (size_t)n * sizeof(double));
        p.status = pp.status[i];
        p.t0 = pp.t0[i];
        p.n_points = n;
    }
    pp = PendingPlans();
}

// The trajectories of slots 0..n-1 to the caller's plans, for the calls that
// plan them in one go: enqueued behind the planner, before their lengths are
// known, each in a place of a whole trajectory's size -- one synchronisation,
// where three copies to pageable memory per plan took 45 us each call.  Many
// or long ones (above kDirectBytes) are packed once their lengths are known.
constexpr size_t kDirectBytes = (size_t)8 << 20;

// Before the planner's launch (the buffer may have to grow): whether the
// trajectories go that way.
bool plans_reserve(fastmdp_ctx *c, int n) {
    const size_t bytes = (size_t)n * c->stride * kPointBytes;
    return bytes <= kDirectBytes && gather_reserve(c, bytes) == 0;
}

int plans_enqueue(fastmdp_ctx *c, const Slot *slots, int n, bool direct) {
    if (!direct) return 0;
    for (int i = 0; i < n; ++i) {
        c->hList2[i] = i;
        c->hOff[i] = (long long)i * c->stride;
    }
    HIP_TRY(fmdp::launch_gather_traj(slots, c->hList2, n, c->hOff, (long long)n * c->stride, c->tr, c->hGather,
                                     c->stream));
    return 0;
}

// After the synchronisation that follows plans_enqueue; hs: the slots as the
// planner left them.
int plans_collect(fastmdp_ctx *c, const Slot *slots, const Slot *hs, int n, bool direct, fastmdp_plan *plans) {
    PendingPlans pp;
    if (direct) {
        pp.total = (long long)n * c->stride;
        for (int i = 0; i < n; ++i) {
            pp.reqs.push_back(i);
            pp.off.push_back((long long)i * c->stride);
            pp.n.push_back(hs[i].n_points);
            pp.status.push_back(hs[i].status);
            pp.t0.push_back(hs[i].t0);
        }
    } else {
        std::vector<int> all(n);
        for (int i = 0; i < n; ++i) all[i] = i;
        const int rc = gather_enqueue(c, slots, all, all, hs, plans, pp);
        if (rc) return rc;
        HIP_TRY(hipStreamSynchronize(c->gstream));
    }
    gather_unpack(c, pp, plans);
    return 0;
}

}  // namespace

extern "C" {

int fastmdp_create(const fastmdp_config *cfg, fastmdp_ctx **out) {
    if (!out) return FASTMDP_E_INVAL;
    int rc = check_cfg(cfg);
    if (rc) return rc;
    fastmdp_ctx *c = new (std::nothrow) fastmdp_ctx();
    if (!c) return FASTMDP_E_NOMEM;
    c->cfg = *cfg;
    make_devcfg(*cfg, c->dc);
    if (!fmdp::planner_shape_supported(cfg->n_climb, cfg->n_speed, c->dc.zero_climb)) {
        delete c;
        return FASTMDP_E_INVAL;
    }
    c->A = c->dc.n_actions;
    c->max_slots = std::max(1, cfg->max_slots);
    c->stride = cfg->max_steps + 1;
    c->tb.cap = cfg->plan_capacity;
    c->tb.rows = cfg->max_rows;
    c->tb.qx0 = (float)cfg->box_min[0];
    c->tb.qy0 = (float)cfg->box_min[1];
    c->tb.qsx = (float)(65535.0 / (cfg->box_max[0] - cfg->box_min[0]));
    c->tb.qsy = (float)(65535.0 / (cfg->box_max[1] - cfg->box_min[1]));
    c->tb.gsx = (float)(fmdp::kGrid / (cfg->box_max[0] - cfg->box_min[0]));
    c->tb.gsy = (float)(fmdp::kGrid / (cfg->box_max[1] - cfg->box_min[1]));
    const size_t tsz = (size_t)cfg->max_rows * cfg->plan_capacity;
    const size_t ssz = (size_t)c->max_slots * c->stride;
    rc = 0;
    rc = rc ? rc : dev_alloc(&c->tb.X, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.Y, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.Z, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.vis, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.own, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.dead, tsz);
    rc = rc ? rc : dev_alloc(&c->tb.rowN, (size_t)cfg->max_rows);
    rc = rc ? rc : dev_alloc(&c->dSlots, (size_t)c->max_slots);
    rc = rc ? rc : dev_alloc(&c->tr.xyz, ssz * 3);
    rc = rc ? rc : dev_alloc(&c->tr.act, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.val, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.seen, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.top, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.ep, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.col, ssz);
    rc = rc ? rc : dev_alloc(&c->tr.nd, ssz);
    if (c->dc.lookahead > 1) rc = rc ? rc : dev_alloc(&c->tr.seenw, ssz * c->dc.lookahead);
    for (DeathLog &d : c->dl) {            // a slot withdraws one piece a pass
        d.cap = (int)std::min<size_t>(ssz, (size_t)1 << 22);
        d.seg_cap = c->max_slots;
        d.box_cap = (int)std::min<size_t>((size_t)c->max_slots * fmdp::kRowBlocks,
                                          (size_t)d.cap / fmdp::kRowBlock + 2 * (size_t)c->max_slots);
        rc = rc ? rc : dev_alloc(&d.x, (size_t)d.cap);
        rc = rc ? rc : dev_alloc(&d.y, (size_t)d.cap);
        rc = rc ? rc : dev_alloc(&d.z, (size_t)d.cap);
        rc = rc ? rc : dev_alloc(&d.col, (size_t)d.cap);
        rc = rc ? rc : dev_alloc(&d.seg, (size_t)d.seg_cap);
        rc = rc ? rc : dev_alloc(&d.seg_box, (size_t)d.seg_cap);
        rc = rc ? rc : dev_alloc(&d.box, (size_t)d.box_cap);
        rc = rc ? rc : dev_alloc(&d.n, (size_t)3);
    }
    rc = rc ? rc : dev_alloc(&c->dRowNPre, (size_t)cfg->max_rows);
    rc = rc ? rc : dev_alloc(&c->dIns, (size_t)c->max_slots);
    rc = rc ? rc : dev_alloc(&c->dInsN, (size_t)1);
    rc = rc ? rc : dev_alloc(&c->dBox, (size_t)c->max_slots * fmdp::kRowBlocks);
    rc = rc ? rc : dev_alloc(&c->dFlag, (size_t)c->stride);
    rc = rc ? rc : dev_alloc(&c->dEvF, (size_t)FASTMDP_N_FEAT + fmdp::kMaxActions);
    rc = rc ? rc : dev_alloc(&c->dEvI, (size_t)FASTMDP_MAX_TOPK + 2);
    rc = rc ? rc : dev_alloc(&c->dStop, (size_t)1);
    rc = rc ? rc : dev_alloc(&c->bs.pk, (size_t)fmdp::kMaxBatch * fmdp::kMatePeaks * 4);
    rc = rc ? rc : dev_alloc(&c->bs.owner, (size_t)fmdp::kMaxBatch * fmdp::kMatePeaks);
    rc = rc ? rc : dev_alloc(&c->bs.n, (size_t)1);
    rc = rc ? rc : dev_alloc(&c->bs.active, (size_t)fmdp::kMaxBatch);
    rc = rc ? rc : dev_alloc(&c->bs.prev_n, (size_t)fmdp::kMaxBatch);
    if (!rc && hipHostMalloc(reinterpret_cast<void **>(&c->hSlots), (size_t)c->max_slots * sizeof(Slot)) != hipSuccess)
        rc = FASTMDP_E_NOMEM;
    if (!rc) {
        const size_t d = (size_t)4 * c->A + (size_t)c->stride * 3;
        if (hipHostMalloc(reinterpret_cast<void **>(&c->hIo), d * sizeof(double) + 3 * sizeof(int)) != hipSuccess) {
            rc = FASTMDP_E_NOMEM;
        } else {
            c->hPts = c->hIo + (size_t)4 * c->A;
            c->hInt = reinterpret_cast<int *>(c->hIo + d);
            c->bs.any = c->hInt + 2;
        }
    }
    rc = rc ? rc : gather_reserve(c, (size_t)c->stride * kPointBytes);
    if (!rc && hipStreamCreate(&c->own) != hipSuccess) rc = FASTMDP_E_DEVICE;
    if (!rc && hipStreamCreate(&c->gstream) != hipSuccess) rc = FASTMDP_E_DEVICE;
    if (!rc && hipEventCreate(&c->e0) != hipSuccess) rc = FASTMDP_E_DEVICE;
    if (!rc && hipEventCreate(&c->e1) != hipSuccess) rc = FASTMDP_E_DEVICE;
    if (!rc && hipEventCreateWithFlags(&c->eGather, hipEventDisableTiming) != hipSuccess) rc = FASTMDP_E_DEVICE;
    if (!rc) {
        const size_t ms = (size_t)c->max_slots;
        if (hipHostMalloc(&c->hRound, ms * sizeof(long long) + 3 * ms * sizeof(int)) != hipSuccess) {
            rc = FASTMDP_E_NOMEM;
        } else {
            c->hOff = static_cast<long long *>(c->hRound);
            c->hList = reinterpret_cast<int *>(c->hOff + ms);
            c->hPass = c->hList + ms;
            c->hList2 = c->hPass + ms;
        }
    }
    if (rc) {
        free_all(c);
        delete c;
        return rc;
    }
    if (fmdp::uses_range_planner(c->dc, FASTMDP_PROPOSE_NONE)) alloc_index(c);
    c->stream = c->own;
    c->tr.stride = c->stride;
    {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess) {
            c->dev = dev;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
                c->n_cu = cus;
        }
    }
    c->dc.n_cu = c->n_cu;
    c->dScratch = noalloc_scratch(c->dev);
    if (!c->dScratch) {
        free_all(c);
        delete c;
        return FASTMDP_E_DEVICE;
    }
    c->hRowN.assign(cfg->max_rows, 0);
    c->hRowTmp.assign(cfg->max_rows, 0);
    if (fmdp::launch_fill_int(c->tb.rowN, 0, cfg->max_rows, c->stream) != hipSuccess ||
        (c->tb.gn && fmdp::launch_fill_int(c->tb.gn, 0, cfg->max_rows, c->stream) != hipSuccess) ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        free_all(c);
        delete c;
        return FASTMDP_E_DEVICE;
    }
    *out = c;
    return 0;
}

void fastmdp_destroy(fastmdp_ctx *ctx) {
    if (!ctx) return;
    hipStreamSynchronize(ctx->stream);
    free_all(ctx);
    delete ctx;
}

int fastmdp_set_stream(fastmdp_ctx *ctx, void *hip_stream) {
    if (!ctx) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    ctx->stream = hip_stream ? static_cast<hipStream_t>(hip_stream) : ctx->own;
    return 0;
}

int fastmdp_load_plans(fastmdp_ctx *ctx, int32_t n, const int32_t *t0, const int32_t *len, const float *xyz) {
    if (!ctx || n < 0 || (n > 0 && (!t0 || !len || !xyz))) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    size_t total = 0;
    for (int j = 0; j < n; ++j) {
        if (t0[j] < 0 || len[j] < 1) return FASTMDP_E_INVAL;
        if ((long)t0[j] + len[j] > ctx->tb.rows) return FASTMDP_E_CAPACITY;
        total += (size_t)len[j];
    }
    std::vector<int> rowN = ctx->hRowN;
    std::vector<int> rows(total), cols(total);
    size_t p = 0;
    for (int j = 0; j < n; ++j)
        for (int k = 0; k < len[j]; ++k, ++p) {
            const int r = t0[j] + k;
            if (rowN[r] >= ctx->tb.cap) return FASTMDP_E_CAPACITY;
            rows[p] = r;
            cols[p] = rowN[r]++;
        }
    if (total) {
        float *dP = nullptr;
        int *dR = nullptr, *dC = nullptr;
        int rc = dev_alloc(&dP, total * 3);
        rc = rc ? rc : dev_alloc(&dR, total);
        rc = rc ? rc : dev_alloc(&dC, total);
        if (rc) { hipFree(dP); hipFree(dR); hipFree(dC); return rc; }
        hipError_t e = hipMemcpyAsync(dP, xyz, total * 3 * sizeof(float), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(dR, rows.data(), total * sizeof(int), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(dC, cols.data(), total * sizeof(int), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = fmdp::launch_scatter_points(ctx->tb, dP, dR, dC, (int)total, -1, ctx->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(ctx->tb.rowN, rowN.data(), rowN.size() * sizeof(int), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        hipFree(dP); hipFree(dR); hipFree(dC);
        if (e != hipSuccess) {
            std::fprintf(stderr, "libfastmdp: load_plans: %s\n", hipGetErrorString(e));
            return FASTMDP_E_DEVICE;
        }
    }
    ctx->hRowN.swap(rowN);
    ctx->n_plans += n;
    return 0;
}

int fastmdp_load_plans_noalloc(fastmdp_ctx *ctx, int32_t n, const int32_t *t0, const int32_t *len,
                               const float *xyz) {
    if (!ctx || n < 0 || (n > 0 && (!t0 || !len || !xyz))) return FASTMDP_E_INVAL;
    if (n > kNoallocMaxPlans) return FASTMDP_E_CAPACITY;
    std::lock_guard<std::mutex> lk(ctx->mu);
    long long total = 0;
    for (int j = 0; j < n; ++j) {
        if (t0[j] < 0 || len[j] < 1) return FASTMDP_E_INVAL;
        if ((long)t0[j] + len[j] > ctx->tb.rows) return FASTMDP_E_CAPACITY;
        total += len[j];
    }
    if (total > kNoallocMaxPoints) return FASTMDP_E_CAPACITY;
    if (n == 0) return 0;
    // row counts after the load, in the context's own host buffer
    std::vector<int> &rowN = ctx->hRowTmp;
    std::copy(ctx->hRowN.begin(), ctx->hRowN.end(), rowN.begin());
    for (int j = 0; j < n; ++j)
        for (int k = 0; k < len[j]; ++k)
            if (++rowN[t0[j] + k] > ctx->tb.cap) return FASTMDP_E_CAPACITY;
    unsigned char *base = static_cast<unsigned char *>(ctx->dScratch);
    int *dT0 = reinterpret_cast<int *>(base);
    int *dLen = dT0 + kNoallocMaxPlans;
    float *dXyz = reinterpret_cast<float *>(base + kNoallocPlanBytes);
    hipError_t e = hipMemcpyAsync(dT0, t0, (size_t)n * sizeof(int), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(dLen, len, (size_t)n * sizeof(int), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(dXyz, xyz, (size_t)total * 3 * sizeof(float), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = fmdp::launch_append_plans(ctx->tb, dT0, dLen, n, dXyz, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        std::fprintf(stderr, "libfastmdp: load_plans_noalloc: %s\n", hipGetErrorString(e));
        return FASTMDP_E_DEVICE;
    }
    ctx->hRowN.swap(rowN);
    ctx->n_plans += n;
    return 0;
}

int fastmdp_set_terrain(fastmdp_ctx *ctx, int32_t nx, int32_t ny, const float *h, double x0, double y0, double cell) {
    if (!ctx || nx < 2 || ny < 2 || !h || !(cell > 0.0)) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    float *d = nullptr;
    int rc = dev_alloc(&d, (size_t)nx * ny);
    if (rc) return rc;
    if (hipMemcpy(d, h, (size_t)nx * ny * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(d);
        return FASTMDP_E_DEVICE;
    }
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    hipFree(ctx->dTerr);
    ctx->dTerr = d;
    ctx->tb.terr = d;
    ctx->tb.tnx = nx; ctx->tb.tny = ny;
    ctx->tb.tx0 = x0; ctx->tb.ty0 = y0; ctx->tb.tcell = cell;
    return 0;
}

int fastmdp_eval_step(fastmdp_ctx *ctx, const fastmdp_state *state, double *values, double *goal_term,
                      double *intr_term, double *terr_term, int32_t *best) {
    if (!ctx || !state || state->t < 0) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    reset_stats(ctx);
    fastmdp_request r{};
    r.origin = state->pos;
    r.goal = state->goal;
    r.t0 = state->t;
    Slot &s = ctx->hSlots[0];                          // the kernel reads and writes it in place
    s = fresh_slot(r, 0, ctx->seq);
    const int A = ctx->A;
    double *h = ctx->hIo;
    EvalOut ev{h, h + A, h + 2 * A, h + 3 * A, ctx->hInt};
    Drain drain{ctx};
    int rc = timed_planner(ctx, 1, nullptr, 1, 0, 0, ev, ctx->hSlots);
    if (rc) return rc;
    drain.done = true;
    if (values) std::memcpy(values, h, A * sizeof(double));
    if (goal_term) std::memcpy(goal_term, h + A, A * sizeof(double));
    if (intr_term) std::memcpy(intr_term, h + 2 * A, A * sizeof(double));
    if (terr_term) std::memcpy(terr_term, h + 3 * A, A * sizeof(double));
    if (best) *best = ctx->hInt[0];
    ctx->st_pairs = s.pairs;
    ctx->st_entries = s.entries;
    ctx->st_steps = s.steps;
    return 0;
}

int fastmdp_plan_request(fastmdp_ctx *ctx, const fastmdp_request *req, fastmdp_plan *out) {
    if (!ctx || !req || !out || req->t0 < 0) return FASTMDP_E_INVAL;
    if (out->capacity < ctx->stride || !out->xyz || !out->action || !out->value) return FASTMDP_E_CAPACITY;
    std::lock_guard<std::mutex> lk(ctx->mu);
    reset_stats(ctx);
    Slot &s = ctx->hSlots[0];                          // the kernel reads and writes it in place
    s = fresh_slot(*req, 0, ctx->seq);
    const bool direct = plans_reserve(ctx, 1);
    Drain drain{ctx};
    int rc = refresh_grid(ctx, ctx->seq, false);
    if (rc) return rc;
    EvalOut none{nullptr, nullptr, nullptr, nullptr, nullptr};
    rc = timed_planner(ctx, 1, nullptr, ctx->cfg.max_steps + 1, 0, 0, none, ctx->hSlots, 0, false);
    rc = rc ? rc : plans_enqueue(ctx, ctx->hSlots, 1, direct);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    rc = planner_time(ctx);
    rc = rc ? rc : plans_collect(ctx, ctx->hSlots, ctx->hSlots, 1, direct, out);
    if (rc) return rc;
    drain.done = true;
    ctx->st_pairs = s.pairs;
    ctx->st_entries = s.entries;
    ctx->st_steps = s.steps;
    ctx->st_hit = s.cert_hit;
    ctx->st_miss = s.cert_miss;
    return 0;
}

int fastmdp_plan_departures(fastmdp_ctx *ctx, const fastmdp_request *req, int32_t n, const int32_t *t0,
                            fastmdp_plan *plans, int32_t *chosen) {
    if (!ctx || !req || n < 1 || !t0 || !plans || !chosen) return FASTMDP_E_INVAL;
    if (n > ctx->max_slots) return FASTMDP_E_CAPACITY;
    for (int i = 0; i < n; ++i) {
        if (t0[i] < 0) return FASTMDP_E_INVAL;
        if (plans[i].capacity < ctx->stride || !plans[i].xyz || !plans[i].action || !plans[i].value)
            return FASTMDP_E_CAPACITY;
    }
    std::lock_guard<std::mutex> lk(ctx->mu);
    reset_stats(ctx);
    note_rows(ctx);
    Slot *hs = ctx->hSlots;
    for (int i = 0; i < n; ++i) {
        fastmdp_request r = *req;
        r.t0 = t0[i];
        hs[i] = fresh_slot(r, i, ctx->seq);            // every candidate sees the same table
    }
    const bool direct = plans_reserve(ctx, n);
    Drain drain{ctx};
    int rc = refresh_grid(ctx, ctx->seq, false);
    if (rc) return rc;
    EvalOut none{nullptr, nullptr, nullptr, nullptr, nullptr};
    rc = timed_planner(ctx, n, nullptr, ctx->cfg.max_steps + 1, 1, 0, none, hs, 0, false);
    rc = rc ? rc : plans_enqueue(ctx, hs, n, direct);
    if (rc) return rc;
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    rc = planner_time(ctx);
    rc = rc ? rc : plans_collect(ctx, hs, hs, n, direct, plans);
    if (rc) return rc;
    drain.done = true;
    int best = -1;
    for (int i = 0; i < n; ++i) {
        ctx->st_pairs += hs[i].pairs;
        ctx->st_entries += hs[i].entries;
        ctx->st_steps += hs[i].steps;
        // the earliest departure whose plan reached the goal and would be accepted
        if (hs[i].status == FASTMDP_OK && hs[i].valid && (best < 0 || t0[i] < t0[best])) best = i;
    }
    *chosen = best;
    return 0;
}

int fastmdp_plan_batch(fastmdp_ctx *ctx, int32_t n, const fastmdp_request *reqs, fastmdp_plan *plans) {
    if (!ctx || n < 1 || !reqs || !plans) return FASTMDP_E_INVAL;
    if (n > fmdp::kMaxBatch || n > ctx->max_slots) return FASTMDP_E_CAPACITY;
    if (ctx->dc.lookahead > 1 || ctx->prop.mode != FASTMDP_PROPOSE_NONE) return FASTMDP_E_INVAL;
    for (int i = 0; i < n; ++i) {
        if (reqs[i].t0 < 0 || reqs[i].t0 != reqs[0].t0) return FASTMDP_E_INVAL;     // lockstep from one row
        if (plans[i].capacity < ctx->stride || !plans[i].xyz || !plans[i].action || !plans[i].value)
            return FASTMDP_E_CAPACITY;
    }
    std::lock_guard<std::mutex> lk(ctx->mu);
    reset_stats(ctx);
    Slot *hs = ctx->hSlots;
    for (int i = 0; i < n; ++i) hs[i] = fresh_slot(reqs[i], i, ctx->seq);
    const bool direct = plans_reserve(ctx, n);
    Drain drain{ctx};
    HIP_TRY(hipMemcpyAsync(ctx->dSlots, hs, n * sizeof(Slot), hipMemcpyHostToDevice, ctx->stream));
    const fmdp::MatePeaks mates{ctx->bs.pk, ctx->bs.owner, ctx->bs.n};
    EvalOut none{nullptr, nullptr, nullptr, nullptr, nullptr};
    const fmdp::LaunchStop nostop{ctx->dStop, 0};
    HIP_TRY(hipEventRecord(ctx->e0, ctx->stream));
    // the origin checks (no step), then each step: one planner step of every
    // aircraft still flying, then the batch's own rules and the next peaks
    auto planner = [&](int budget) -> int {
        hipError_t e = fmdp::launch_planner(n, ctx->stream, ctx->dc, ctx->tb, ctx->dSlots, nullptr,
                                            ctx->tr, budget, 0, 0, none, ctx->prop, nostop,
                                            budget > 0 ? mates : fmdp::MatePeaks{});
        if (e != hipSuccess) {
            std::fprintf(stderr, "libfastmdp: planner launch failed: %s\n", hipGetErrorString(e));
            return FASTMDP_E_DEVICE;
        }
        ctx->st_launches += 1;
        return 0;
    };
    int rc = planner(0);
    if (rc) return rc;
    HIP_TRY(fmdp::launch_batch_step(ctx->dc, ctx->dSlots, n, ctx->tr, ctx->bs, 1, ctx->stream));
    int any = ctx->hInt[2] = 1;
    for (int k = 0; any; ++k) {
        rc = planner(1);
        if (rc) return rc;
        HIP_TRY(fmdp::launch_batch_step(ctx->dc, ctx->dSlots, n, ctx->tr, ctx->bs, 0, ctx->stream));
        if ((k & 7) == 7) {
            // the steps enqueued up to the last such point have ended; the
            // eight since then run meanwhile
            if (k > 7) HIP_TRY(hipEventSynchronize(ctx->eGather));
            any = __atomic_load_n(ctx->hInt + 2, __ATOMIC_RELAXED);
            HIP_TRY(hipEventRecord(ctx->eGather, ctx->stream));
            if (k > ctx->cfg.max_steps + 1) break;                 // every aircraft has hit the step limit
        }
    }
    HIP_TRY(hipEventRecord(ctx->e1, ctx->stream));
    rc = plans_enqueue(ctx, ctx->dSlots, n, direct);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(hs, ctx->dSlots, n * sizeof(Slot), hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, ctx->e0, ctx->e1));
    ctx->st_ms = ms;
    for (int i = 0; i < n; ++i) {
        ctx->st_pairs += hs[i].pairs;
        ctx->st_entries += hs[i].entries;
        ctx->st_steps += hs[i].steps;
    }
    rc = plans_collect(ctx, ctx->dSlots, hs, n, direct, plans);
    drain.done = rc == 0;
    return rc;
}

int fastmdp_commit_plan(fastmdp_ctx *ctx, const fastmdp_plan *plan) {
    if (!ctx || !plan || !plan->xyz || plan->n_points < 1 || plan->t0 < 0) return FASTMDP_E_INVAL;
    if (plan->status != FASTMDP_OK) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const int n = plan->n_points, t0 = plan->t0;
    if ((long)t0 + n > ctx->tb.rows || n > ctx->stride) return FASTMDP_E_CAPACITY;
    for (int k = 0; k < n; ++k)
        if (ctx->hRowN[t0 + k] >= ctx->tb.cap) return FASTMDP_E_CAPACITY;
    std::memcpy(ctx->hPts, plan->xyz, (size_t)n * 3 * sizeof(double));
    Drain drain{ctx};
    HIP_TRY(fmdp::launch_commit(ctx->dc, ctx->tb, ctx->hPts, t0, n, ctx->seq, ctx->dFlag, ctx->hInt + 1, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    drain.done = true;
    const int flag = ctx->hInt[1];
    if (flag & 2) return FASTMDP_E_CAPACITY;
    if (flag) return FASTMDP_E_CONFLICT;
    for (int k = 0; k < n; ++k) ctx->hRowN[t0 + k] += 1;
    ctx->n_plans += 1;
    ctx->seq += 1;
    return 0;
}

int fastmdp_num_plans(const fastmdp_ctx *ctx) { return ctx ? ctx->n_plans : FASTMDP_E_INVAL; }

int fastmdp_plan_fcfs(fastmdp_ctx *ctx, int32_t n, const fastmdp_request *reqs, const double *arrival_s,
                      fastmdp_plan *plans, int32_t *committed, double *done_s) {
    if (!ctx || n < 0 || (n > 0 && (!reqs || !plans || !committed))) return FASTMDP_E_INVAL;
    for (int i = 0; i < n; ++i) {
        if (reqs[i].t0 < 0) return FASTMDP_E_INVAL;
        if (arrival_s && (i > 0 && arrival_s[i] < arrival_s[i - 1])) return FASTMDP_E_INVAL;
        if (plans[i].capacity < ctx->stride || !plans[i].xyz || !plans[i].action || !plans[i].value)
            return FASTMDP_E_CAPACITY;
    }
    std::lock_guard<std::mutex> lk(ctx->mu);
    reset_stats(ctx);
    note_rows(ctx);
    using clk = std::chrono::steady_clock;
    const auto t_start = clk::now();
    auto now_s = [&]() { return std::chrono::duration<double>(clk::now() - t_start).count(); };
    const int S = std::min(ctx->max_slots, std::max(n, 1));
    const int budget = ctx->cfg.steps_per_launch > 0 ? ctx->cfg.steps_per_launch : 512;
    const int seq0 = ctx->seq;
    Slot *hs = ctx->hSlots;                  // pinned mirror of the slots
    std::vector<int> slot_req(S, -1);        // request held by each slot
    std::vector<int> req_slot(n, -1);
    int next_req = 0, next_commit = 0;
    std::vector<int> list, pass;
    PendingPlans pending;                    // accepted trajectories still being copied
    bool gathered = false;                   // a gather was enqueued in this call
    int epoch = 0;                           // acceptance passes run
    const fmdp::PassBufs pbufs{ctx->dRowNPre, ctx->dIns, ctx->dInsN, ctx->dBox, ctx->dStop, ctx->hSlots};
    HIP_TRY(fmdp::launch_fcfs_begin(ctx->tb, pbufs, ctx->dl[0], ctx->dl[1], ctx->stream));
    auto finish = [&](int rc) {
        // the device row counts include tentative and withdrawn entries
        if (hipMemcpyAsync(ctx->hRowN.data(), ctx->tb.rowN, ctx->hRowN.size() * sizeof(int), hipMemcpyDeviceToHost,
                           ctx->stream) != hipSuccess ||
            hipStreamSynchronize(ctx->stream) != hipSuccess)
            return FASTMDP_E_DEVICE;
        return rc;
    };
    auto run = [&]() -> int {
        int rc0 = refresh_grid(ctx, seq0, false);
        if (rc0) return rc0;
        while (next_commit < n) {
            // a call that grows the table far: its accepted plans indexed too
            if (next_commit > 0) rc0 = refresh_grid(ctx, seq0 + next_commit, true);
            if (rc0) return rc0;
            // admit arrived requests into free slots, in request order
            bool dirty = false;
            const double t_now = arrival_s ? now_s() : 0.0;
            for (int s = 0; s < S && next_req < n; ++s)
                if (slot_req[s] < 0) {
                    if (arrival_s && arrival_s[next_req] > t_now) break;
                    hs[s] = fresh_slot(reqs[next_req], next_req, seq0 + next_req);
                    slot_req[s] = next_req;
                    req_slot[next_req] = s;
                    ++next_req;
                    dirty = true;
                }
            if (dirty) {
                // a reused slot: its accepted trajectory's gather comes first
                if (gathered) HIP_TRY(hipStreamWaitEvent(ctx->stream, ctx->eGather, 0));
                HIP_TRY(hipMemcpyAsync(ctx->dSlots, hs, S * sizeof(Slot), hipMemcpyHostToDevice, ctx->stream));
            }
            // plan the oldest running requests, two per compute unit (with the
            // proposal or the window one: their workgroups take a CU each; the
            // range-query planner could hold four, but the oldest requests,
            // which the later ones depend on, then step more slowly; the full
            // sweep, ms a pass with two and with one: 1000 requests at 3000
            // plans 77 and 75, 92 and 85, 78 and 84 by the inputs, at 1500
            // plans 57 and 65, 2000 requests at 800 plans 91 and 108), for up
            // to `budget` steps: a
            // request that waits for the next launch plans against the plans its
            // predecessors finish in this one instead of re-planning after them
            list.clear();
            for (int s = 0; s < S; ++s)
                if (slot_req[s] >= 0 && hs[s].status == fmdp::kRunning) list.push_back(s);
            const int per_launch =
                ctx->n_cu * (fmdp::uses_range_planner(ctx->dc, ctx->prop.mode) ||
                                     fmdp::uses_pairs(ctx->dc, ctx->prop.mode)
                                 ? fmdp::kLaunchPerCU
                                 : 1);
            if ((int)list.size() > per_launch) {
                std::nth_element(list.begin(), list.begin() + per_launch, list.end(),
                                 [&](int a, int b) { return hs[a].req < hs[b].req; });
                list.resize(per_launch);
            }
            if (list.empty() && next_commit == next_req) {
                // idle until the next arrival
                const double wait = arrival_s[next_req] - now_s();
                if (wait > 0) std::this_thread::sleep_for(std::chrono::duration<double>(std::min(wait, 0.001)));
                continue;
            }
            // One synchronisation per round: the planner launch and the
            // acceptance pass over every admitted, not yet accepted request,
            // in stream order, the slots written to the host's mirror by the
            // pass itself; the trajectories accepted in the previous round
            // reach the caller's plans meanwhile.
            const bool planned = !list.empty();
            if (planned) {
                std::memcpy(ctx->hList, list.data(), list.size() * sizeof(int));
                EvalOut none{nullptr, nullptr, nullptr, nullptr, nullptr};
                // the launch ends once a quarter of its requests have finished:
                // the others resume after the acceptance pass, with new requests
                // in the freed compute units.  In the range-query planner's
                // launches few requests wait for a place after the first ones, so
                // they run until half have finished (half the acceptance passes;
                // three streams of 1000 requests: 9.4, 10.2 and 10.0 ms a pass,
                // with a quarter 9.7, 10.1 and 11.3; the full sweep, whose steps
                // cost more than a pass, takes 76, 91 and 77 ms with a quarter
                // and 92, 102 and 90 with half)
                const int stop_div = fmdp::uses_range_planner(ctx->dc, ctx->prop.mode) ? 2 : 4;
                const int stop_target = std::max(1, (int)list.size() / stop_div);
                int rc = timed_planner(ctx, (int)list.size(), ctx->hList, budget, 1, epoch, none, ctx->dSlots, stop_target, false);
                if (rc) return finish(rc);
            }
            pass.clear();
            for (int r = next_commit; r < next_req; ++r) pass.push_back(req_slot[r]);
            epoch += 1;
            std::memcpy(ctx->hPass, pass.data(), pass.size() * sizeof(int));
            HIP_TRY(fmdp::launch_fcfs_pass(ctx->dc, ctx->tb, ctx->dSlots, ctx->hPass, (int)pass.size(), ctx->tr,
                                           ctx->dl[(epoch - 1) & 1], ctx->dl[epoch & 1], pbufs, epoch, ctx->stream));
            // the trajectories accepted last round were gathered ahead of this
            // round's launch: hand them to the caller while the planner runs
            if (!pending.empty()) {
                HIP_TRY(hipEventSynchronize(ctx->eGather));
                gather_unpack(ctx, pending, plans);
            }
            HIP_TRY(hipStreamSynchronize(ctx->stream));
            if (planned) {
                int rc = planner_time(ctx);
                if (rc) return finish(rc);
            }
            for (int s : pass) {
                if (hs[s].err) return finish(FASTMDP_E_CAPACITY);
            }
            // accept in request order: a finished request whose predecessors are
            // all accepted is final; one that withdrew entries in this pass ends
            // the walk (later requests are checked against it next pass)
            const double t_done = now_s();
            std::vector<int> acc_slots, acc_reqs;
            while (next_commit < next_req) {
                const int s = req_slot[next_commit];
                if (hs[s].status == fmdp::kRunning) break;
                const int r = next_commit;
                committed[r] = (hs[s].status == FASTMDP_OK && hs[s].valid) ? 1 : 0;
                if (done_s) done_s[r] = t_done;
                ctx->n_plans += committed[r];
                ctx->st_pairs += hs[s].pairs;
                ctx->st_entries += hs[s].entries;
                ctx->st_steps += hs[s].steps;
                ctx->st_hit += hs[s].cert_hit;
                ctx->st_miss += hs[s].cert_miss;
                ctx->st_resumes += hs[s].resumes;
                acc_slots.push_back(s);
                acc_reqs.push_back(r);
                ++next_commit;
                if (hs[s].killed) break;
            }
            if (!acc_slots.empty()) {
                int rc = gather_enqueue(ctx, ctx->dSlots, acc_slots, acc_reqs, hs, plans, pending);
                if (rc) return finish(rc);
                gathered = gathered || !pending.empty();
                for (int s : acc_slots) slot_req[s] = -1;   // reusable: the gather precedes any new planning
            }
        }
        if (!pending.empty()) {
            HIP_TRY(hipEventSynchronize(ctx->eGather));
            gather_unpack(ctx, pending, plans);
        }
        return 0;
    };
    const int rc = run();
    if (rc == 0) {
        ctx->seq = seq0 + n;
        return finish(0);
    }
    // An interrupted call keeps exactly the accepted requests: their plans
    // stay in the table and are visible to every later request (sequence
    // numbers below ctx->seq); the entries of every admitted request not yet
    // accepted are withdrawn.  Accepted trajectories still on their way to
    // the caller are delivered; committed[] is 0 from the first unaccepted
    // request on.
    (void)hipStreamSynchronize(ctx->stream);
    const bool gathered_all = hipStreamSynchronize(ctx->gstream) == hipSuccess;
    if (!pending.empty() && gathered_all) gather_unpack(ctx, pending, plans);
    int m = 0;
    for (int s = 0; s < S; ++s)
        if (slot_req[s] >= 0) ctx->hPass[m++] = s;
    if (m > 0)
        fmdp::launch_fcfs_abort(ctx->tb, ctx->dSlots, ctx->hPass, m, ctx->tr, seq0 + next_commit, epoch + 1,
                                ctx->stream);
    for (int r = next_commit; r < n; ++r) committed[r] = 0;
    ctx->seq = seq0 + next_commit;
    return finish(rc);
}

int fastmdp_table_snapshot(fastmdp_ctx *ctx) {
    if (!ctx) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    ctx->snapRowN = ctx->hRowN;
    ctx->snap_plans = ctx->n_plans;
    return 0;
}

int fastmdp_table_rewind(fastmdp_ctx *ctx) {
    if (!ctx) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    if (ctx->snapRowN.empty()) {
        ctx->snapRowN.assign(ctx->tb.rows, 0);
        ctx->snap_plans = 0;
    }
    HIP_TRY(hipMemcpyAsync(ctx->tb.rowN, ctx->snapRowN.data(), ctx->snapRowN.size() * sizeof(int),
                           hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    // the grids stand while they index no entry that is dropped here
    bool covered = ctx->gridRowN.size() == ctx->snapRowN.size();
    for (size_t r = 0; covered && r < ctx->snapRowN.size(); ++r) covered = ctx->gridRowN[r] <= ctx->snapRowN[r];
    ctx->grid_ok = ctx->grid_ok && covered;
    ctx->hRowN = ctx->snapRowN;
    ctx->n_plans = ctx->snap_plans;
    return 0;
}

int fastmdp_last_stats(const fastmdp_ctx *ctx, int64_t *pairs, int64_t *steps, int64_t *resumes, int64_t *launches,
                       double *kernel_ms, int64_t *row_entries) {
    if (!ctx) return FASTMDP_E_INVAL;
    if (pairs) *pairs = ctx->st_pairs;
    if (row_entries) *row_entries = ctx->st_entries;
    if (steps) *steps = ctx->st_steps;
    if (resumes) *resumes = ctx->st_resumes;
    if (launches) *launches = ctx->st_launches;
    if (kernel_ms) *kernel_ms = ctx->st_ms;
    return 0;
}

int fastmdp_features(fastmdp_ctx *ctx, int32_t n, const double *states, const double *goals, const int32_t *rows,
                     const int32_t *seqs, float *feat) {
    if (!ctx || n < 0 || (n > 0 && (!states || !goals || !rows || !seqs || !feat))) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    if (n >= fmdp::kFeatGrouped && !ctx->dFeatWs &&
        dev_alloc(&ctx->dFeatWs, fmdp::features_workspace(ctx->tb.rows)))
        (void)hipGetLastError();                       // no memory for it: one workgroup per state
    HIP_TRY(fmdp::launch_features(ctx->dc, ctx->tb, n, states, goals, rows, seqs, feat, ctx->dFeatWs, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return 0;
}

int fastmdp_next_seq(const fastmdp_ctx *ctx) { return ctx ? ctx->seq : FASTMDP_E_INVAL; }

int fastmdp_set_proposal(fastmdp_ctx *ctx, int32_t mode, int32_t top_k, int32_t refresh, const fastmdp_mlp *net) {
    if (!ctx || refresh < 1) return FASTMDP_E_INVAL;
    fmdp::PropArgs p{};
    p.mode = mode;
    p.k = top_k;
    p.refresh = refresh;
    if (mode == FASTMDP_PROPOSE_NONE) {
        p.k = 0;
    } else if (mode == FASTMDP_PROPOSE_MLP || mode == FASTMDP_PROPOSE_GOAL) {
        if (ctx->dc.lookahead > 1) return FASTMDP_E_INVAL;      // the window runs the full sweep
        if (top_k < 1 || top_k > FASTMDP_MAX_TOPK || top_k > ctx->A) return FASTMDP_E_INVAL;
        if (mode == FASTMDP_PROPOSE_MLP) {
            if (fmdp::mlp_weights(net, &p.net)) return FASTMDP_E_INVAL;
            if (p.net.n_in != FASTMDP_N_FEAT || p.net.n_hid != FASTMDP_MLP_HIDDEN || p.net.n_out < ctx->A)
                return FASTMDP_E_INVAL;
        }
    } else {
        return FASTMDP_E_INVAL;
    }
    std::lock_guard<std::mutex> lk(ctx->mu);
    ctx->prop = p;
    return 0;
}

int fastmdp_eval_proposal(fastmdp_ctx *ctx, const fastmdp_state *state, float *features, float *logits,
                          int32_t *topk, int32_t *certified, int32_t *best) {
    if (!ctx || !state || state->t < 0) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    if (ctx->prop.mode == FASTMDP_PROPOSE_NONE) return FASTMDP_E_INVAL;
    reset_stats(ctx);
    fastmdp_request r{};
    r.origin = state->pos;
    r.goal = state->goal;
    r.t0 = state->t;
    Slot s = fresh_slot(r, 0, ctx->seq);
    Drain drain{ctx};
    HIP_TRY(hipMemcpyAsync(ctx->dSlots, &s, sizeof(Slot), hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(hipMemsetAsync(ctx->dEvF, 0, (FASTMDP_N_FEAT + fmdp::kMaxActions) * sizeof(float), ctx->stream));
    const int A = ctx->A;
    EvalOut ev{nullptr, nullptr, nullptr, nullptr, ctx->hInt, ctx->dEvF, ctx->dEvF + FASTMDP_N_FEAT,
               ctx->dEvI, ctx->dEvI + FASTMDP_MAX_TOPK, ctx->dEvI + FASTMDP_MAX_TOPK + 1};
    int rc = timed_planner(ctx, 1, nullptr, 1, 0, 0, ev, ctx->dSlots);
    if (rc) return rc;
    std::vector<float> hf(FASTMDP_N_FEAT + (size_t)A);
    int hi[FASTMDP_MAX_TOPK + 2];
    HIP_TRY(hipMemcpyAsync(hf.data(), ctx->dEvF, hf.size() * sizeof(float), hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(hipMemcpyAsync(hi, ctx->dEvI, sizeof(hi), hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    drain.done = true;
    if (features) std::memcpy(features, hf.data(), FASTMDP_N_FEAT * sizeof(float));
    if (logits) std::memcpy(logits, hf.data() + FASTMDP_N_FEAT, A * sizeof(float));
    if (topk) std::memcpy(topk, hi, ctx->prop.k * sizeof(int));
    if (certified) *certified = hi[FASTMDP_MAX_TOPK];
    if (best) *best = hi[FASTMDP_MAX_TOPK + 1];
    return 0;
}

int fastmdp_proposal_stats(const fastmdp_ctx *ctx, int64_t *certified, int64_t *fallbacks) {
    if (!ctx) return FASTMDP_E_INVAL;
    if (certified) *certified = ctx->st_hit;
    if (fallbacks) *fallbacks = ctx->st_miss;
    return 0;
}

// Checkpoint file: "FMDPTAB2", rows, cap, n_plans, live entries per row
// [rows], then for each row its live entries' x, y and z (FP32).  Withdrawn
// entries are dropped; loaded entries are owned by no request.
int fastmdp_save_table(fastmdp_ctx *ctx, const char *path) {
    if (!ctx || !path) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const int rows = ctx->tb.rows, cap = ctx->tb.cap;
    std::vector<int> dead((size_t)cap), live(rows, 0);
    std::vector<float> buf[3];
    for (auto &b : buf) b.resize((size_t)cap);
    std::vector<std::vector<float>> keep(rows);
    for (int r = 0; r < rows; ++r) {
        const int m = std::min(ctx->hRowN[r], cap);
        if (!m) continue;
        const size_t off = (size_t)r * cap;
        float *src[3] = {ctx->tb.X, ctx->tb.Y, ctx->tb.Z};
        if (hipMemcpy(dead.data(), ctx->tb.dead + off, m * sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
            return FASTMDP_E_DEVICE;
        for (int a = 0; a < 3; ++a)
            if (hipMemcpy(buf[a].data(), src[a] + off, m * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
                return FASTMDP_E_DEVICE;
        for (int a = 0; a < 3; ++a)
            for (int j = 0; j < m; ++j)
                if (dead[j] == fmdp::kAlive) keep[r].push_back(buf[a][j]);
        live[r] = (int)keep[r].size() / 3;
    }
    FILE *f = std::fopen(path, "wb");
    if (!f) return FASTMDP_E_IO;
    int hdr[3] = {rows, cap, ctx->n_plans};
    bool ok = std::fwrite("FMDPTAB2", 1, 8, f) == 8 && std::fwrite(hdr, sizeof(int), 3, f) == 3 &&
              std::fwrite(live.data(), sizeof(int), rows, f) == (size_t)rows;
    for (int r = 0; ok && r < rows; ++r)
        if (!keep[r].empty()) ok = std::fwrite(keep[r].data(), sizeof(float), keep[r].size(), f) == keep[r].size();
    ok = (std::fclose(f) == 0) && ok;
    return ok ? 0 : FASTMDP_E_IO;
}

int fastmdp_load_table(fastmdp_ctx *ctx, const char *path) {
    if (!ctx || !path) return FASTMDP_E_INVAL;
    std::lock_guard<std::mutex> lk(ctx->mu);
    FILE *f = std::fopen(path, "rb");
    if (!f) return FASTMDP_E_IO;
    char magic[8];
    int hdr[3];
    if (std::fread(magic, 1, 8, f) != 8 || std::memcmp(magic, "FMDPTAB2", 8) != 0 ||
        std::fread(hdr, sizeof(int), 3, f) != 3) {
        std::fclose(f);
        return FASTMDP_E_IO;
    }
    const int rows = hdr[0];
    if (rows != ctx->tb.rows || hdr[2] < 0) {
        std::fclose(f);
        return FASTMDP_E_CAPACITY;
    }
    std::vector<int> rowN(rows);
    if (std::fread(rowN.data(), sizeof(int), rows, f) != (size_t)rows) {
        std::fclose(f);
        return FASTMDP_E_IO;
    }
    for (int r = 0; r < rows; ++r)
        if (rowN[r] < 0 || rowN[r] > ctx->tb.cap) {
            std::fclose(f);
            return FASTMDP_E_CAPACITY;
        }
    const int cap = ctx->tb.cap;
    std::vector<float> buf((size_t)cap * 3);
    std::vector<int> own((size_t)cap, -1), alive((size_t)cap, fmdp::kAlive);
    ctx->grid_ok = false;                              // rows are overwritten from here on
    int rc = 0;
    for (int r = 0; r < rows && !rc; ++r) {
        const int m = rowN[r];
        if (!m) continue;
        if (std::fread(buf.data(), sizeof(float), (size_t)m * 3, f) != (size_t)m * 3) {
            rc = FASTMDP_E_IO;
            break;
        }
        const size_t off = (size_t)r * cap;
        float *dst[3] = {ctx->tb.X, ctx->tb.Y, ctx->tb.Z};
        bool ok = true;
        for (int a = 0; a < 3 && ok; ++a)
            ok = hipMemcpy(dst[a] + off, buf.data() + (size_t)a * m, m * sizeof(float), hipMemcpyHostToDevice) ==
                 hipSuccess;
        ok = ok && hipMemcpy(ctx->tb.vis + off, own.data(), m * sizeof(int), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(ctx->tb.own + off, own.data(), m * sizeof(int), hipMemcpyHostToDevice) == hipSuccess;
        ok = ok && hipMemcpy(ctx->tb.dead + off, alive.data(), m * sizeof(int), hipMemcpyHostToDevice) == hipSuccess;
        if (!ok) rc = FASTMDP_E_DEVICE;
    }
    std::fclose(f);
    if (!rc && hipMemcpy(ctx->tb.rowN, rowN.data(), rows * sizeof(int), hipMemcpyHostToDevice) != hipSuccess)
        rc = FASTMDP_E_DEVICE;
    // the 16-bit coordinates follow the points, also of the rows read before
    // a file breaks off
    if (ctx->tb.Q && (fmdp::launch_quantise_table(ctx->tb, ctx->stream) != hipSuccess ||
                      hipStreamSynchronize(ctx->stream) != hipSuccess))
        rc = rc ? rc : FASTMDP_E_DEVICE;
    if (rc) return rc;
    ctx->hRowN.swap(rowN);
    ctx->n_plans = hdr[2];
    return 0;
}

const char *fastmdp_strerror(int code) {
    switch (code) {
        case 0: return "ok";
        case FASTMDP_E_INVAL: return "invalid argument or unsupported configuration";
        case FASTMDP_E_CAPACITY: return "table or buffer capacity exceeded";
        case FASTMDP_E_DEVICE: return "HIP runtime error";
        case FASTMDP_E_CONFLICT: return "commit refused: separation or terrain conflict";
        case FASTMDP_E_NOMEM: return "out of memory";
        case FASTMDP_E_IO: return "file input/output error";
        default: return "unknown code";
    }
}

}  // extern "C"
