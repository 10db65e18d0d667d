// range.hip -- the range-query planner for gfx950: one request per workgroup
// of 256 or 512 threads (Sec. VII: only the trajectories within reach of the
// state are considered).
//
// With the range query most steps have no plan within reach, and a step is a
// chain of dependent operations, bound by latency and not by bytes or
// arithmetic: scoring every action in FP64 against the few plans near it, on
// the whole workgroup, took 3.5 us a step for a request alone (2.4 GHz: 8400
// cycles), whether or not a plan was near.  Here a step is taken in one of
// three ways, all of which give the same plans, values and records bit for
// bit:
//   - in a run, where no plan changes the choice: an action's value is at
//     most its goal term, so the goal-directed action is the choice while no
//     well reaches its successor.  One wave computes the run's states ahead
//     (about 300 cycles a step: a reciprocal square root and its
//     refinements), the others check them against the table;
//   - in a detour batch, among the plans near them: the action nearest the
//     goal outside every well, one workgroup barrier a step and no
//     exponential;
//   - singly, where those rules do not decide (a tie, no action outside the
//     wells, a distance within 1 mm of the radius that is inside): every
//     action scored in FP64, tie-band argmax, as in the 1024-thread kernel
//     (the same functions).
// The entries near a state come from a grid over the row (table.hip,
// build_grid_kernel: a 30 km row of 2600 entries has about ten in the cells a
// query covers, where reading x and y of the row took 21 KB of the compute
// unit's 64 B/clk); columns appended since the grid was built are searched by
// their 16-bit coordinates, 4 bytes an entry.  Points are written 64 at a
// time, a run's values evaluated 64 at a time.
//   Measured (MI355X, 3000 plans, 360 actions): a request alone 3.5 us a step
// before, now 0.2 (no plan near) to 3 (in traffic all the way), 0.4 in the
// middle of 180 flights; the 1000-request stream's planner time 22.3 -> 7.4 ms.
#include "bearing.h"
#include "planner.h"
#include "row_window.h"
#include "score.h"
#include "wave.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace fmdp {

namespace {

constexpr int HMAX = kRangeMaxHeads;

__device__ __forceinline__ int lanes_below(uint64_t bal) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
}

// NT threads per request: kRangeThreads with OCC requests resident per CU
// (kRangePerCU: up to 128 VGPRs each; 2: up to 256, no register spills), or
// kRangeThreadsSolo (one action per thread) for launches that hold at most
// one request per CU.
template <int NT, int OCC, int NC, int NV, int ZC>
__global__ __attribute__((amdgpu_flat_work_group_size(NT, NT),
                          amdgpu_waves_per_eu(NT == kRangeThreads ? OCC : 2))) void range_planner_kernel(
    DevCfg cfg, DevTable tb, Slot *slots, const int *slot_list, Traj tr, int budget, int validate, int epoch,
    LaunchStop stop) {
    constexpr int NW = NT / 64;
    constexpr int TILE = NT;                     // staged entries per round: one candidate per thread
    constexpr int APT = kMaxActions / NT;        // actions per thread
    constexpr int RUN = kRunSteps;               // steps of a run: four lanes of the checking wave each
    constexpr int DS = 8;                        // steps of a detour batch
    constexpr int DL = 32;                       // entries listed per detour step
    constexpr int RING = 128;                    // points on their way to the trajectory
    static_assert(64 + 4 * RUN <= RING, "points are written before the ring wraps");
    static_assert(NW >= 3 && DS % NW == 0 && DS <= RUN, "a run's roles and a detour batch's rows are dealt to the waves");
    static_assert(kMaxActions % NT == 0, "actions are dealt to threads in whole rounds");
    static_assert(HMAX <= NT, "one thread per heading");
    __shared__ float4 sList[DS][DL];            // detour batch: each row's entries near the batch's states
    __shared__ int sListN[DS];
    // detour step, per wave (alternate steps): its nearest action outside
    // the wells: distance to the goal, successor, nearest plan, action, how
    // many of its lanes come as near
    __shared__ double sR[2][NW][5];
    __shared__ int sRa[2][NW], sRn[2][NW];
    __shared__ double sC0[HMAX], sS0[HMAX];              // heading offsets (cos, sin of 2*pi*h/H)
    __shared__ float4 tile[TILE];               // staged entries of one round
    __shared__ double sCos[2][HMAX], sSin[2][HMAX];      // heading directions, alternate steps
    __shared__ double sStep[FASTMDP_MAX_ACT_DIM], sDz[FASTMDP_MAX_ACT_DIM];   // speed*dt, climb*dt
    __shared__ float sKv[FASTMDP_MAX_ACT_DIM], sClf[FASTMDP_MAX_ACT_DIM];      // FP32 sweep constants
    __shared__ unsigned sBand[kMaxActions / 32];
    __shared__ double red_d[NW];
    __shared__ int s_wsum[NW], s_rem[2][NW];
    __shared__ int s_wli[NW], s_wti[NW], s_wfl[NW];      // per wave: choice, largest, choice's flags
    __shared__ double s_wv[NW], s_wd2[NW];               // per wave: choice's value, nearest distance
    __shared__ int s_any, s_flag, s_stop, s_stop_run[2];
    // the points taken last, written to the trajectory 64 at a time: point i
    // in slot i % RING; value (runs leave it to the write), nearest squared
    // distance, action | run << 16, row entries seen, top action
    __shared__ double sP[RING][3], sPv[RING], sPd[RING];
    __shared__ int sPa[RING], sPs[RING], sPt[RING];
    // runs (alternate batches): steps and action, directions and distances;
    // per step the findings among the indexed and the later columns: nearest
    // (sweep expression), entries in reach, and whether the rest holds
    __shared__ double sQ[2][RUN][3];
    __shared__ int sNb[2], sAg[2];
    __shared__ float sMg[2][RUN], sMt[2][RUN];
    __shared__ int sNg[2][RUN], sNt[2][RUN], sOk[2][RUN];
    __shared__ int sCnt[kCountRows], sGn[kCountRows];    // entry counts and indexed columns of rows wb .. wb + 127
    const ActTab at{sStep, sDz};

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int slot = slot_list ? slot_list[blockIdx.x] : (int)blockIdx.x;
    Slot &S = slots[slot];
    if (S.status != kRunning) return;           // a finished request (uniform: one slot per workgroup)

    const int H = cfg.n_head, A = cfg.n_actions;
    const double g[3] = {S.goal[0], S.goal[1], S.goal[2]};
    const int t0 = S.t0;
    const int seq = S.seq;
    const size_t pt_base = (size_t)slot * tr.stride;

    // this thread's heading offset 2*pi*h/H (h = tid < H)
    if (tid < H) {
        const double th = 2.0 * M_PI * (double)tid / (double)H;
        sC0[tid] = cos(th);
        sS0[tid] = sin(th);
    }
    if (tid < FASTMDP_MAX_ACT_DIM) {
        sStep[tid] = cfg.speed[tid] * cfg.dt;
        sDz[tid] = cfg.climb[tid] * cfg.dt;
        sKv[tid] = cfg.kv[tid];
        sClf[tid] = cfg.climb_f[tid];
    }
    for (int w = tid; w < kMaxActions / 32; w += NT) sBand[w] = 0u;
    if (tid == 0) {
        s_any = 0;
        s_flag = 0;
        s_stop = 0;
    }
    // the state, the point count and the status live in every thread's
    // registers (the same values in all)
    int n = S.n_points;
    double s[3];
    if (n == 0) {
        s[0] = S.origin[0]; s[1] = S.origin[1]; s[2] = S.origin[2];
    } else {
        const double *p = tr.xyz + (pt_base + n - 1) * 3;
        s[0] = p[0]; s[1] = p[1]; s[2] = p[2];
    }
    int status = kRunning;
    __syncthreads();

    // Origin check of a fresh request: inside the box, clear of terrain, and
    // no plan active at the departure row closer than R_sep.
    if (n == 0) {
        const int n_row = t0 < tb.rows ? min(tb.rowN[t0], tb.cap) : 0;
        const size_t rb = (size_t)t0 * tb.cap;
        int hit = 0;
        for (int j = tid; j < n_row; j += NT)
            if (entry_visible(tb, rb + j, seq) &&
                entry_d2(s[0], s[1], s[2], tb.X[rb + j], tb.Y[rb + j], tb.Z[rb + j]) < cfg.R_sep * cfg.R_sep)
                hit = 1;
        if (hit) s_flag = 1;        // benign race: every writer stores 1
        __syncthreads();
        bool blocked = s_flag != 0 || outside_box(cfg, s[0], s[1], s[2]);
        if (tb.terr && s[2] - terrain_height(tb, s[0], s[1]) < 0.0) blocked = true;
        if (tid == 0) {
            double *p = tr.xyz + pt_base * 3;
            p[0] = s[0]; p[1] = s[1]; p[2] = s[2];
            tr.act[pt_base] = -1;
            tr.val[pt_base] = 0.0;
            tr.seen[pt_base] = n_row;
            tr.ep[pt_base] = epoch;
            tr.top[pt_base] = -1;
            tr.col[pt_base] = -1;
            tr.nd[pt_base] = INFINITY;
        }
        n = 1;
        if (blocked) status = FASTMDP_REJECT_ORIGIN;
    }

    // Entry counts and indexed columns of 128 rows from wb on (the table does
    // not change during a launch), 64 rows at a time by one wave
    // (row_window.h)
    int wb = t0 + n;
    auto read_counts = [&](int first) {
        const int r = first + lane;
        const bool in = r >= 0 && r < tb.rows;
        sCnt[count_slot(r)] = in ? min(tb.rowN[r], tb.cap) : 0;
        sGn[count_slot(r)] = in ? tb.gn[r] : 0;
    };
    if (wave < 2) read_counts(wb + kCountLoad * wave);
    auto row_count = [&](int row) { return sCnt[count_slot(row)]; };
    auto row_indexed = [&](int row) { return sGn[count_slot(row)]; };
    auto shift_counts = [&](int row) {                    // uniform; `row`: the next batch's first
        if (count_load_due(wb, row)) {
            if (wave == NW - 1) read_counts(wb + kCountRows);
            wb += kCountLoad;
        }
    };
    // The exact test of the range query for one entry (x, y, z, visibility)
    // against a state: e its staged form.
    auto near_entry = [&](const float4 r, double x, double y, double z, float4 &e) {
        const float qx = (float)((double)r.x - x);
        const float qy = (float)((double)r.y - y);
        const float qz = (float)((double)r.z - z);
        const float w = fmaf(qx, qx, fmaf(qy, qy, qz * qz));
        e = make_float4(qx, qy, cfg.zeta_scale * qz, w);
        return __float_as_int(r.w) < seq && w < cfg.cull_r2;
    };
    auto table_entry = [&](size_t idx) {
        return make_float4(tb.X[idx], tb.Y[idx], tb.Z[idx], __int_as_float(tb.vis[idx]));
    };
    // 16-bit box test: both offsets from the box's corner at most its width
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 q_half = __builtin_bit_cast(u16x2, cfg.run_r), q_width = __builtin_bit_cast(u16x2, cfg.run_w);
    auto q_corner = [&](double x, double y, u16x2 half) {
        return (u16x2)(__builtin_bit_cast(u16x2, quantised(tb, (float)x, (float)y)) - half);
    };
    // bits of the entries j .. j + 3 (columns [from, n_row) only) inside the box
    auto q_inside = [&](const uint4 q, u16x2 corner, u16x2 q_width, int j, int from, int n_row) -> uint32_t {
        const uint32_t e4[4] = {q.x, q.y, q.z, q.w};
        uint32_t o[4], bits = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = __builtin_bit_cast(
                uint32_t, __builtin_elementwise_sub_sat((u16x2)(__builtin_bit_cast(u16x2, e4[i]) - corner), q_width));
        if (__ballot(min(min(o[0], o[1]), min(o[2], o[3])) == 0u)) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o[i] == 0u && j + i >= from && j + i < n_row) bits |= 1u << i;
        }
        return bits;
    };
    // cells a query around (x, y) covers (one metre more than the box test)
    const float g_half = cfg.cull_box + 1.0f;
    struct Cells {
        int x0, x1, y0, y1;
    };
    auto cells = [&](float x, float y, float g_half) {
        Cells c;
        c.x0 = __builtin_amdgcn_readfirstlane(grid_cell(x - g_half, tb.qx0, tb.gsx));
        c.x1 = __builtin_amdgcn_readfirstlane(grid_cell(x + g_half, tb.qx0, tb.gsx));
        c.y0 = __builtin_amdgcn_readfirstlane(grid_cell(y - g_half, tb.qy0, tb.gsy));
        c.y1 = __builtin_amdgcn_readfirstlane(grid_cell(y + g_half, tb.qy0, tb.gsy));
        return c;
    };
    // records [a, b) of this lane's row of cells: y on lanes below 32, y + 1
    // above; this lane's first record in a, later ones 32 on
    auto cell_range = [&](int row, const Cells &c, int y, int &a, int &b) {
        const int yy = y + (lane >> 5);
        a = b = 0;
        if (yy <= c.y1) {
            const int *off = tb.goff + (size_t)row * (kGridCells + 1) + yy * kGrid;
            a = off[c.x0];
            b = off[c.x1 + 1];
        }
    };

    long long pairs = 0, entries = 0;                     // this thread's share (counted by one thread or one lane per step)
    int steps_here = 0, stop_v = 0, buf = 0, dpar = 0;
    bool stop_now = false;
    enum { STEP = 0, DETOUR = 1, STRAIGHT = 2 };          // how the next step is taken: singly, in a detour batch, in a run
    int mode = cfg.run_ok ? STRAIGHT : STEP;
    int singly = 0, wait = 1;                             // single steps left before the next detour batch; their next number
    // goal-directed choices in a row that end a detour: doubled by a run that
    // stops within half a batch (a flight along the edge of a well, which a
    // run does not decide, would pay for a run every other step)
    int need = 2, direct = 0;
    // Points [fl, to) from the ring to the trajectory, one per lane of the
    // calling wave.  A run's point has its goal term for a value (no penalty
    // reaches it), evaluated here for 64 points at a time instead of once per
    // step by a whole wave.
    int fl = n;
    auto write_points = [&](int from, int to) {
        const int i = from + lane;
        if (i >= to) return;
        const int r = i % RING;
        const size_t p = pt_base + i;
        const double x = sP[r][0], y = sP[r][1], z = sP[r][2];
        const int pa = sPa[r];
        tr.xyz[p * 3 + 0] = x;
        tr.xyz[p * 3 + 1] = y;
        tr.xyz[p * 3 + 2] = z;
        tr.val[p] = (pa >> 16) ? goal_term(cfg, x, y, z, g) : sPv[r];
        tr.nd[p] = sPd[r];
        tr.act[p] = pa & 0xffff;
        tr.seen[p] = sPs[r];
        tr.top[p] = sPt[r];
        tr.ep[p] = epoch;
        tr.col[p] = -1;
    };
    // 64 points at a time; a run's last points may not be visible to the
    // writing wave before the next barrier: they stay
    auto flush_points = [&]() {                           // uniform
        if (n - fl >= 64 + RUN) {
            if (wave == NW - 1) write_points(fl, fl + 64);
            fl += 64;
        }
    };
    // The launch stop counter, by one thread per batch: the value on its way
    // since an earlier batch, and every fourth time a new read (all workgroups
    // of a launch read this one word, past their caches)
    int polls = 0;
    auto poll_stop = [&](int &flag) {
        flag = stop.target > 0 && stop_v >= stop.target;
        if (stop.target > 0 && (polls++ & 3) == 0)
            stop_v = __hip_atomic_load(stop.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // the state's component of this lane (x, y, z, x of every four lanes)
    const int comp = (lane & 3) == 3 ? 0 : lane & 3;
    const double ell2_hi = cfg.ell * cfg.ell * (1.0 + 1e-9);
    if (tid < 3) sP[(n - 1) % RING][tid] = s[tid];        // the state a run starts from
    __syncthreads();
    // scoring rounds q that hold an action of this wave (wave-uniform)
    const int nq = min(APT, max(0, (A - wave * 64 + NT - 1) / NT));

    for (;;) {
        if (status != kRunning) break;                    // uniform (registers)
        const int k = n - 1;                              // steps taken so far
        const int t = t0 + k;
        {
            const double ex = g[0] - s[0], ey = g[1] - s[1], ez = g[2] - s[2];
            const double e2 = norm2(ex, ey, ez);
            if (e2 <= ell2_hi && sqrt(e2) <= cfg.ell) {
                status = FASTMDP_OK;
                break;
            }
            if (k >= cfg.max_steps) {
                status = FASTMDP_TIMEOUT;
                break;
            }
            if (steps_here >= budget || stop_now) break;  // resumable: stays running
        }
        shift_counts(t + 1);
        flush_points();

        // 0. A run: steps whose choice no plan can change, RUN at a time.
        //    While no well reaches the goal-directed action's successor
        //    (heading 0, the fastest speed, the climb nearest the goal's
        //    altitude), its value is its goal term, and no other action's
        //    value exceeds its own goal term (the penalties are
        //    non-negative); so where every other successor is farther from
        //    the goal by more than run_margin, it is the choice, alone inside
        //    the tie band.  The states of a batch follow from one another
        //    without the table: wave 0 computes the next batch's while wave
        //    1, four lanes per step, checks this batch's actions, box,
        //    terrain and indexed entries and the other waves its rows' later
        //    columns, so a batch takes what the chain of its states takes and
        //    one barrier.  The steps before the first unconfirmed one are
        //    taken, with the records the single step would leave; that one
        //    is left to the modes below.
        if (mode == STRAIGHT) {                           // uniform
            const int left = min(cfg.max_steps - k, budget - steps_here);
            // wave 0: the batch p of the states from point n0 - 1 (component
            // s_l) on, at most lim of them: successors into the ring,
            // directions and distances into sQ
            double s_l = comp == 0 ? s[0] : comp == 1 ? s[1] : s[2];
            const double g_l = comp == 0 ? g[0] : comp == 1 ? g[1] : g[2];
            const double v_step = sStep[cfg.run_v];
            auto chain = [&](int p, int n0, int lim) {
                // the climb, and for how many steps it can stay the best (a
                // step past that is caught by the check)
                const double z0 = dpp_bcast_f64<2>(s_l);
                int cg = 0;
                double e0 = INFINITY;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const double e = fabs(g[2] - (z0 + sDz[c]));
                    if (e < e0) {
                        e0 = e;
                        cg = c;
                    }
                }
                const double c_dz = sDz[cg];
                int nb = max(0, min(RUN, lim));
                if (c_dz != 0.0) {
                    const float m = (float)fabs(g[2] - z0) / (float)fabs(c_dz);
                    nb = min(nb, max(1, (int)fminf(m, 1e4f)));
                }
                nb = __builtin_amdgcn_readfirstlane(nb);
                if (lane == 0) {
                    sNb[p] = nb;
                    sAg[p] = cg * NV + cfg.run_v;         // heading 0
                }
                for (int i = 0; i < nb; ++i) {            // uniform
                    // one step of all three components: the horizontal
                    // distance and the quotients b / br from one reciprocal
                    // square root, rounded as the square root and the
                    // divisions of the single step (bearing.h; r2 is far from
                    // the ends of the range: checked with the step)
                    const double b = g_l - s_l;
                    const double bx = dpp_bcast_f64<0>(b), by = dpp_bcast_f64<1>(b);
                    const double r2 = dot2(bx, bx, by, by);
                    const Bearing v = bearing(r2, __builtin_amdgcn_rsq(r2));
                    const double br = v.br, q = bearing_quotient(b, v);
                    s_l = comp == 2 ? s_l + c_dz : __builtin_fma(v_step, q, s_l);
                    if (lane < 3) {
                        sQ[p][i][lane] = lane == 2 ? br : q;
                        sP[(n0 + i) % RING][lane] = s_l;
                    }
                }
            };
            int par = 0, taken = 0;
            if (wave == 0) chain(0, n, left);
            lds_barrier();
            for (;;) {                                    // uniform
                const int nb = sNb[par], ag = sAg[par];
                const int tr0 = t0 + n;                   // row of the batch's first step (t + 1)
                if (wave == 0) {
                    chain(par ^ 1, n + nb, left - taken - nb);
                } else if (wave == 1) {
                    const int st = lane >> 2, sub = lane & 3;
                    const int row = tr0 + st;
                    const bool act = st < nb;
                    const int idn = act ? row_indexed(row) : 0;
                    const int r0 = (n + st - 1) % RING, r1 = (n + st) % RING;
                    const double x = sP[r0][0], y = sP[r0][1], z = sP[r0][2];
                    // the step's row of cells: its first records are on
                    // their way during the checks
                    const int x0 = grid_cell((float)x - g_half, tb.qx0, tb.gsx);
                    const int x1 = grid_cell((float)x + g_half, tb.qx0, tb.gsx);
                    int cy = grid_cell((float)y - g_half, tb.qy0, tb.gsy);
                    const int y1 = grid_cell((float)y + g_half, tb.qy0, tb.gsy);
                    const int *off = tb.goff + (size_t)row * (kGridCells + 1);
                    const float4 *rec = tb.grec + (size_t)row * tb.cap;
                    int a = 0, b = 0;
                    if (idn > 0) {
                        a = off[cy * kGrid + x0];
                        b = off[cy * kGrid + x1 + 1];
                    }
                    const double nx = sP[r1][0], ny = sP[r1][1], nz = sP[r1][2];
                    const double cb = sQ[par][st][0], sb = sQ[par][st][1], br = sQ[par][st][2];
                    bool good = act && !outside_box(cfg, nx, ny, nz);
                    const double bx = g[0] - x, by = g[1] - y, bz = g[2] - z;
                    const double r2 = dot2(bx, bx, by, by), e2 = __builtin_fma(bz, bz, r2);
                    const double far = br + fabs(bz);     // at least the state's distance to the goal
                    good = good && far <= cfg.run_dmax && e2 > ell2_hi && r2 > 1e-100;
                    {
                        const double ex = g[0] - nx, ey = g[1] - ny, ez = g[2] - nz;
                        const double d2g = norm2(ex, ey, ez);
                        const double lim = d2g * (1.0 + 1e-14) + cfg.run_margin * (2.0 * far + cfg.run_margin) * 1.0001;
                        // heading 0's actions exactly as scored, and the
                        // nearest that any other heading's can come
#pragma unroll
                        for (int i = 0; i < (NC * NV + 3) / 4; ++i) {
                            const int q = min(sub + 4 * i, NC * NV - 1);
                            const double stp = sStep[q % NV];
                            const double fx = g[0] - __builtin_fma(stp, cb, x), fy = g[1] - __builtin_fma(stp, sb, y);
                            const double fz = g[2] - (z + sDz[q / NV]);
                            const double fz2 = fz * fz;
                            const double d2h = norm2(fx, fy, fz);
                            const double d2o = r2 + stp * (stp - 2.0 * br * cfg.run_c1) + fz2 - (1e-6 + 1e-12 * r2);
                            good = good && (q == ag || d2h > lim) && d2o > lim;
                        }
                    }
                    if (tb.terr) good = good && nz - terrain_height(tb, nx, ny) >= cfg.clear_terr;
                    // the indexed entries near the state, every fourth of its
                    // cells' records
                    const float ch = (float)cb, sh = (float)sb, kvv = sKv[cfg.run_v], clv = sClf[ag / NV];
                    int nkeep = 0;
                    float m = INFINITY;
                    a += sub;
                    while (__ballot(a < b || (idn > 0 && cy < y1))) {       // uniform
                        if (a < b) {
                            float4 e;
                            if (near_entry(rec[a], x, y, z, e)) {
                                const float hq = fmaf(e.x, ch, e.y * sh);
                                const float uu = fmaf(kvv, hq, e.w);
                                m = fminf(m, ag / NV == ZC ? uu : fmaf(clv, e.z, uu));
                                nkeep += 1;
                            }
                            a += 4;
                        } else if (idn > 0 && cy < y1) {
                            cy += 1;
                            a = off[cy * kGrid + x0] + sub;
                            b = off[cy * kGrid + x1 + 1];
                        }
                    }
                    m = fminf(m, dpp_f32<kDppQuad1032>(m));
                    m = fminf(m, dpp_f32<kDppQuad2301>(m));
                    nkeep += dpp_i32<kDppQuad1032>(nkeep);
                    nkeep += dpp_i32<kDppQuad2301>(nkeep);
                    const uint64_t gb = __ballot(good);
                    if (sub == 0) {
                        sMg[par][st] = m;
                        sNg[par][st] = nkeep;
                        sOk[par][st] = (gb >> (4 * st) & 15u) == 15u;
                    }
                    if (lane == 0) poll_stop(s_stop_run[par]);
                } else {
                    for (int st = wave - 2; st < nb; st += NW - 2) {        // uniform per wave
                        const int row = tr0 + st, n_row = row_count(row), idn = row_indexed(row);
                        int nkeep = 0;
                        float m = INFINITY;
                        if (idn < n_row) {
                            const int r0 = (n + st - 1) % RING;
                            const double x = sP[r0][0], y = sP[r0][1], z = sP[r0][2];
                            const float ch = (float)sQ[par][st][0], sh = (float)sQ[par][st][1];
                            const float kvv = sKv[cfg.run_v], clv = sClf[ag / NV];
                            const size_t rb = (size_t)row * tb.cap;
                            const u16x2 corner = q_corner(x, y, q_half);
                            for (int base = idn & ~3; base < n_row; base += 4 * 256) {   // uniform per wave
                                uint4 q[4];
#pragma unroll
                                for (int u = 0; u < 4; ++u) {
                                    const int j = base + 256 * u + 4 * lane;
                                    q[u] = make_uint4(0u, 0u, 0u, 0u);
                                    if (j < n_row) q[u] = *reinterpret_cast<const uint4 *>(tb.Q + rb + j);
                                }
                                uint32_t cm = 0u;
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    if (base + 256 * u < n_row)             // uniform per wave
                                        cm |= q_inside(q[u], corner, q_width, base + 256 * u + 4 * lane, idn, n_row) << (4 * u);
                                while (__ballot(cm != 0u)) {                // uniform per wave
                                    bool keep = false;
                                    if (cm) {
                                        const int bit = __builtin_ctz(cm);
                                        cm &= cm - 1u;
                                        float4 e;
                                        keep = near_entry(table_entry(rb + base + 256 * (bit >> 2) + 4 * lane + (bit & 3)),
                                                          x, y, z, e);
                                        if (keep) {
                                            const float hq = fmaf(e.x, ch, e.y * sh);
                                            const float uu = fmaf(kvv, hq, e.w);
                                            m = fminf(m, ag / NV == ZC ? uu : fmaf(clv, e.z, uu));
                                        }
                                    }
                                    nkeep += __popcll(__ballot(keep));
                                }
                            }
                            if (nkeep) m = wave_min_f32(m);
                        }
                        if (lane == 0) {
                            sMt[par][st] = m;
                            sNt[par][st] = nkeep;
                        }
                    }
                }
                lds_barrier();
                // one lane per step: the nearest plan of its successor, and
                // whether the step stands
                const int st = lane & (RUN - 1);
                const int nk = sNg[par][st] + sNt[par][st];
                const float m = fminf(sMg[par][st], sMt[par][st]);
                const double d2n = nk > 0 ? nearest_d2<NC, NV>(at, ag, m) : INFINITY;
                const uint64_t undecided = __ballot(st >= nb || !sOk[par][st] || !(d2n >= cfg.band_hi2));
                const int f = min(nb, undecided ? __builtin_ctzll(undecided) : RUN);       // steps taken
                if (wave == 0 && lane < f) {
                    const int ri = (n + lane) % RING, cnt = row_count(tr0 + lane);
                    sPd[ri] = d2n;
                    sPa[ri] = ag | 1 << 16;
                    sPs[ri] = cnt;
                    sPt[ri] = -1;
                    pairs += (long long)A * nk;
                    entries += cnt;
                }
                stop_now = s_stop_run[par];
                n += f;
                steps_here += f;
                taken += f;
                par ^= 1;
                if (f < nb) {
                    mode = cfg.detour_ok ? DETOUR : STEP;
                    need = taken < RUN / 2 ? min(2 * need, 64) : 2;
                }
                if (f < nb || stop_now || sNb[par] == 0) break;
                shift_counts(t0 + n);
                flush_points();
            }
            const int ri = (n - 1) % RING;
            s[0] = sP[ri][0]; s[1] = sP[ri][1]; s[2] = sP[ri][2];
            lds_barrier();                                // the last batch is read before the next run writes its own
            continue;
        }

        // 0b. A detour batch: up to DS steps among the plans near them, one
        //    barrier each.  An action outside every well has its goal term
        //    for a value (terrain aside) and beats every action inside one
        //    (detour_ok), so the choice is the action nearest the goal among
        //    those outside, where no other of them comes as near to within
        //    run_margin.  The entries within reach of the batch's states
        //    (each lies within the steps taken so far of the first) are
        //    listed first, one row per wave at a time; each step then reads
        //    no memory and evaluates no exponential.  Whatever this rule does
        //    not decide (no action outside the wells, a tie, terrain within
        //    reach) is left to the single step below.
        if (mode == DETOUR) {                             // uniform
            const int kb = min(DS, min(cfg.max_steps - k, budget - steps_here));
#pragma unroll
            for (int i = 0; i < DS / NW; ++i) {
                const int kk = wave + NW * i;             // the row of step kk
                if (kk >= kb) continue;                   // uniform per wave
                const int row = t + 1 + kk, n_row = row_count(row), idn = row_indexed(row);
                const size_t rb = (size_t)row * tb.cap;
                const float reach = cfg.cull_box + 1.0f + (float)kk * (float)cfg.max_step;
                int cnt = 0;
                auto list = [&](bool have, const float4 p) {
                    float4 e;
                    near_entry(p, s[0], s[1], s[2], e);
                    const bool keep = have && __float_as_int(p.w) < seq && e.w < reach * reach;
                    const uint64_t bal = __ballot(keep);
                    const int at_i = cnt + lanes_below(bal);
                    if (keep && at_i < DL) sList[kk][at_i] = p;
                    cnt += __popcll(bal);
                };
                if (idn > 0) {
                    const Cells cl = cells((float)s[0], (float)s[1], reach);
                    for (int cy = cl.y0; cy <= cl.y1; cy += 2) {            // uniform
                        int a, b;
                        cell_range(row, cl, cy, a, b);
                        for (a += lane & 31; __ballot(a < b); a += 32) {    // uniform per wave
                            float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                            if (a < b) p = tb.grec[rb + a];
                            list(a < b, p);
                        }
                    }
                }
                if (idn < n_row) {
                    const u16x2 half = q_half + __builtin_bit_cast(u16x2, cfg.run_step) * (uint16_t)kk;
                    const u16x2 corner = q_corner(s[0], s[1], half);
                    for (int base = idn & ~3; base < n_row; base += 256) {  // uniform
                        const int j = base + 4 * lane;
                        uint4 q = make_uint4(0u, 0u, 0u, 0u);
                        if (j < n_row) q = *reinterpret_cast<const uint4 *>(tb.Q + rb + j);
                        uint32_t cm = q_inside(q, corner, half + half, j, idn, n_row);
                        while (__ballot(cm != 0u)) {      // uniform per wave
                            const bool have = cm != 0u;
                            float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                            if (have) {
                                p = table_entry(rb + j + __builtin_ctz(cm));
                                cm &= cm - 1u;
                            }
                            list(have, p);
                        }
                    }
                }
                if (lane == 0) sListN[kk] = cnt;
            }
            if (tid == 0) poll_stop(s_stop_run[0]);
            lds_barrier();
            stop_now = s_stop_run[0];
            double x = s[0], y = s[1], z = s[2];
            int f = 0;
            for (; f < kb; ++f) {                         // uniform: every wave decides alike
                mode = STEP;
                const int cnt = sListN[f];
                if (cnt > DL) break;
                // this state's entries, one per lane
                float4 e = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
                bool keep = false;
                if (lane < cnt) keep = near_entry(sList[f][lane], x, y, z, e);
                const uint64_t near = __ballot(keep);
                const double bx = g[0] - x, by = g[1] - y, bz = g[2] - z;
                const double r2 = dot2(bx, bx, by, by), e2 = __builtin_fma(bz, bz, r2);
                // the direction, as a run's chain has it
                const Bearing dir = bearing(r2, __builtin_amdgcn_rsq(r2));
                const double br = dir.br, cb = bearing_quotient(bx, dir), sb = bearing_quotient(by, dir);
                const double far = br + fabs(bz);
                if (!(e2 > ell2_hi && r2 > 1e-100 && far <= cfg.run_dmax)) break;
                // this thread's actions: squared distance to the goal, and
                // infinity inside a well (or out of the box)
                const double xyz[3] = {x, y, z};
                double b1 = INFINITY, b2 = INFINITY, bn = INFINITY, qx = x, qy = y, qz = z;
                double d2q[APT], dnq[APT];
                int ba = 0;
#pragma unroll
                for (int q = 0; q < APT; ++q) {
                    d2q[q] = dnq[q] = INFINITY;
                    if (wave * 64 + q * NT >= A) continue;                  // uniform per wave
                    const int a = min(tid + q * NT, A - 1), h = a / (NC * NV), c = (a / NV) % NC, v = a % NV;
                    const double dx = dot2(cb, sC0[h], -sb, sS0[h]), dy = dot2(sb, sC0[h], cb, sS0[h]);
                    double px, py, pz;
                    successor(cfg, at, a, xyz, dx, dy, px, py, pz);
                    const double ex = g[0] - px, ey = g[1] - py, ez = g[2] - pz;
                    double d2 = norm2(ex, ey, ez);
                    const float ch = (float)dx, sh = (float)dy, kvv = sKv[v], clv = sClf[c];
                    float m = INFINITY;
                    for (uint64_t nb = near; nb; nb &= nb - 1) {            // uniform
                        const int l = __builtin_ctzll(nb);
                        const float ux = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.x), l));
                        const float uy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.y), l));
                        const float uz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.z), l));
                        const float uw = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.w), l));
                        const float hq = fmaf(ux, ch, uy * sh);
                        const float uu = fmaf(kvv, hq, uw);
                        m = fminf(m, c == ZC ? uu : fmaf(clv, uz, uu));
                    }
                    const double dn = nearest_d2<NC, NV>(at, a, m);
                    if (tid + q * NT >= A || outside_box(cfg, px, py, pz) || dn <= cfg.band_lo2) d2 = INFINITY;
                    d2q[q] = d2;
                    dnq[q] = dn;
                    const bool less = d2 < b1;
                    b2 = fmin(b2, less ? b1 : d2);
                    if (less) {
                        b1 = d2;
                        bn = dn;
                        ba = a;
                        qx = px;
                        qy = py;
                        qz = pz;
                    }
                }
                // the wave's nearest, then the workgroup's
                const double slack = cfg.run_margin * (2.0 * (far + cfg.max_step) + cfg.run_margin) * 1.0001;
                {
                    const double d1 = -wave_max(-b1);
                    const double lim = d1 * (1.0 + 1e-14) + slack;
                    const uint64_t first = __ballot(b1 == d1), close = __ballot(b1 <= lim), second = __ballot(b2 <= lim);
                    if (lane == __builtin_ctzll(first)) {
                        sR[dpar][wave][0] = d1;
                        sR[dpar][wave][1] = qx;
                        sR[dpar][wave][2] = qy;
                        sR[dpar][wave][3] = qz;
                        sR[dpar][wave][4] = bn;
                        sRa[dpar][wave] = ba;
                        sRn[dpar][wave] = __popcll(close) + __popcll(second);
                    }
                }
                lds_barrier();
                double d1 = INFINITY;
                int w1 = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const double d = sR[dpar][w][0];
                    if (d < d1) {
                        d1 = d;
                        w1 = w;
                    }
                }
                const double lim = d1 * (1.0 + 1e-14) + slack;
                int close = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) close += w != w1 && sR[dpar][w][0] <= lim;
                int best = sRa[dpar][w1], top = -1;
                double px = sR[dpar][w1][1], py = sR[dpar][w1][2], pz = sR[dpar][w1][3];
                double dn = sR[dpar][w1][4];
                const bool alone = close == 0 && sRn[dpar][w1] == 1;
                dpar ^= 1;
                if (!(d1 < INFINITY)) break;              // no action outside the wells
                if (alone) {
                    if (dn < cfg.band_hi2) {
                        // within kBand of the radius: the nearest distance in
                        // FP64 over the entries in reach, as the single step
                        // has it
                        double dd = INFINITY;
                        if (keep) {
                            const float4 p = sList[f][lane];
                            dd = entry_d2(px, py, pz, p.x, p.y, p.z);
                        }
                        dn = -wave_max(-dd);
                        if (!(dn >= cfg.R_intr * cfg.R_intr)) break;
                    }
                    if (tb.terr && !(pz - terrain_height(tb, px, py) >= cfg.clear_terr)) break;
                } else {
                    // several come as near (the two headings beside a plan on
                    // the track): their goal terms, then the single step's
                    // argmax among them
                    double V[APT], v1 = -INFINITY;
                    bool bad = false;
#pragma unroll
                    for (int q = 0; q < APT; ++q) {
                        V[q] = -INFINITY;
                        if (!(d2q[q] <= lim)) continue;
                        const int a = tid + q * NT, h = a / (NC * NV);
                        double ux, uy, uz;
                        successor(cfg, at, a, xyz, dot2(cb, sC0[h], -sb, sS0[h]), dot2(sb, sC0[h], cb, sS0[h]), ux, uy, uz);
                        V[q] = goal_term(cfg, ux, uy, uz, g);
                        v1 = fmax(v1, V[q]);
                        bad = bad || !(dnq[q] >= cfg.band_hi2) ||
                              (tb.terr && !(uz - terrain_height(tb, ux, uy) >= cfg.clear_terr));
                    }
                    v1 = wave_max(v1);
                    const uint64_t undecided = __ballot(bad);
                    if (lane == 0) {
                        red_d[wave] = v1;
                        s_wfl[wave] = undecided != 0;
                    }
                    lds_barrier();
                    double vm = -INFINITY;
                    bool any_bad = false;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        vm = fmax(vm, red_d[w]);
                        any_bad = any_bad || s_wfl[w];
                    }
                    const double thr = vm - cfg.tie_rel * fabs(vm);
                    int li = 0x7fffffff, ti = 0x7fffffff;
#pragma unroll
                    for (int q = APT - 1; q >= 0; --q) {  // lowest index last
                        if (V[q] > -INFINITY && V[q] >= thr) li = tid + q * NT;
                        if (V[q] > -INFINITY && V[q] == vm) ti = tid + q * NT;
                    }
                    li = wave_min(li);
                    ti = wave_min(ti);
                    if (lane == 0) {
                        s_wli[wave] = li;
                        s_wti[wave] = ti;
                    }
#pragma unroll
                    for (int q = 0; q < APT; ++q)
                        if (tid + q * NT == li) s_wd2[wave] = dnq[q];
                    lds_barrier();
                    best = top = 0x7fffffff;
                    int bw = 0;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        if (s_wli[w] < best) {
                            best = s_wli[w];
                            bw = w;
                        }
                        top = min(top, s_wti[w]);
                    }
                    // (the next writes to these follow at least one barrier)
                    if (any_bad || best == 0x7fffffff) break;
                    dn = s_wd2[bw];
                    top = top != best ? top : -1;
                    const int h = best / (NC * NV);
                    successor(cfg, at, best, xyz, dot2(cb, sC0[h], -sb, sS0[h]), dot2(sb, sC0[h], cb, sS0[h]), px, py, pz);
                }
                mode = DETOUR;
                if (tid == 0) {
                    const int ri = n % RING, rc = row_count(t + 1 + f);
                    sP[ri][0] = px;
                    sP[ri][1] = py;
                    sP[ri][2] = pz;
                    sPd[ri] = dn;
                    sPa[ri] = best | 1 << 16;
                    sPs[ri] = rc;
                    sPt[ri] = top;
                    pairs += (long long)A * __popcll(near);
                    entries += rc;
                }
                // back to runs after `need` goal-directed choices in a row
                {
                    double ez = INFINITY;
                    int cg = 0;
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const double d = fabs(g[2] - (z + sDz[c]));
                        if (d < ez) {
                            ez = d;
                            cg = c;
                        }
                    }
                    direct = best == cg * NV + cfg.run_v ? direct + 1 : 0;
                }
                x = px; y = py; z = pz;
                n += 1;
                if (direct >= need) {
                    mode = STRAIGHT;
                    direct = 0;
                    ++f;
                    break;
                }
            }
            s[0] = x; s[1] = y; s[2] = z;
            steps_here += f;
            if (f > 0) wait = 1;
            if (mode == STEP) {                           // undecided: single steps, more of them each time in a row
                singly = wait;
                wait = min(2 * wait, 16);
            }
            lds_barrier();                                // the lists are read before the next batch writes its own
            continue;
        }

        // heading directions: the goal bearing rotated by each offset
        {
            const double bx = g[0] - s[0], by = g[1] - s[1];
            const double br = sqrt(dot2(bx, bx, by, by));
            const double cb = br > 0.0 ? bx / br : 1.0, sb = br > 0.0 ? by / br : 0.0;
            if (tid < H) {
                sCos[buf][tid] = dot2(cb, sC0[tid], -sb, sS0[tid]);
                sSin[buf][tid] = dot2(sb, sC0[tid], cb, sS0[tid]);
            }
        }
        const double *hc = sCos[buf], *hs = sSin[buf];
        const int row = t + 1;
        const int n_row = row_count(row);
        if (tid == 0) entries += n_row;
        const size_t rb = (size_t)row * tb.cap;
        int n_vis = 0;
        float mA[APT];
#pragma unroll
        for (int i = 0; i < APT; ++i) mA[i] = INFINITY;
        if (tid == 0 && stop.target > 0)
            stop_v = __hip_atomic_load(stop.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // 1. the row's entries near the state, one per lane and round: the
        //    records of the cells around it (wave 0) and the later columns
        //    inside the 16-bit box (groups of 256 dealt to the waves, 8 * NW
        //    of them per pass), by the exact test; staged, then swept by
        //    every thread for its actions
        if (n_row > 0) {
            const int idn = row_indexed(row);
            const Cells cl = cells((float)s[0], (float)s[1], g_half);
            const u16x2 corner = q_corner(s[0], s[1], q_half);
            int cy = cl.y0, ia = 0, ib = 0;
            if (wave == 0 && idn > 0) {
                cell_range(row, cl, cy, ia, ib);
                ia += lane & 31;
            }
            int base = idn & ~3;                          // the next pass over the later columns
            uint32_t cm = 0u;
            int cbase = 0;
            bool more = true;
            int par = 0;                                  // alternate s_rem buffer (see below)
            while (more) {                                // uniform
                // a pass's candidates: bit 4 i + m of cm marks column cbase +
                // 256 NW i + m
                if (!__ballot(cm != 0u) && base < n_row) {                 // uniform per wave
                    cbase = base + 256 * wave + 4 * lane;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int j = cbase + 256 * NW * i;
                        if (base + 256 * (wave + NW * i) < n_row) {        // uniform per wave
                            uint4 q = make_uint4(0u, 0u, 0u, 0u);
                            if (j < n_row) q = *reinterpret_cast<const uint4 *>(tb.Q + rb + j);
                            cm |= q_inside(q, corner, q_width, j, idn, n_row) << (4 * i);
                        }
                    }
                    base += 8 * 256 * NW;
                }
                bool keep = false;
                float4 e = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
                if (ia < ib) {
                    keep = near_entry(tb.grec[rb + ia], s[0], s[1], s[2], e);
                    ia += 32;
                } else if (cm) {
                    const int bit = __builtin_ctz(cm);
                    cm &= cm - 1u;
                    keep = near_entry(table_entry(rb + cbase + 256 * NW * (bit >> 2) + (bit & 3)), s[0], s[1], s[2], e);
                }
                if (wave == 0 && idn > 0 && !__ballot(ia < ib) && cy + 2 <= cl.y1) {   // the next rows of cells
                    cy += 2;
                    cell_range(row, cl, cy, ia, ib);
                    ia += lane & 31;
                }
                const uint64_t kb = __ballot(keep);
                const bool rem = __ballot(cm != 0u || ia < ib) || base < n_row ||
                                 (wave == 0 && idn > 0 && cy + 2 <= cl.y1);
                par ^= 1;
                if (lane == 0) {
                    s_wsum[wave] = __popcll(kb);
                    s_rem[par][wave] = rem;
                }
                // the flags of remaining candidates alternate between two
                // buffers: a buffer is rewritten only after a barrier that
                // follows every read of its previous contents
                lds_barrier();                            // also: this step's heading directions visible
                int tp = 0, tn = 0;
                more = false;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const int c = s_wsum[w];
                    tp += w < wave ? c : 0;
                    tn += c;
                    more = more || s_rem[par][w];
                }
                if (keep) tile[tp + lanes_below(kb)] = e;
                lds_barrier();
                n_vis += tn;
                // every thread's actions over the staged entries: the
                // 1024-thread sweep's FP32 expression, minimum over plans
#pragma unroll
                for (int q = 0; q < APT; ++q) {
                    const int a = tid + q * NT;
                    if (a < A && tn > 0) {
                        const int h = a / (NC * NV), c = (a / NV) % NC, v = a % NV;
                        const float ch = (float)hc[h], sh = (float)hs[h];
                        const float kvv = sKv[v], clv = sClf[c];
                        float m = mA[q];
                        for (int u = 0; u < tn; ++u) {
                            const float4 p = tile[u];
                            const float hq = fmaf(p.x, ch, p.y * sh);
                            const float uu = fmaf(kvv, hq, p.w);
                            m = fminf(m, (c == ZC) ? uu : fmaf(clv, p.z, uu));
                        }
                        mA[q] = m;
                    }
                }
                // (the next round writes the tile after its first barrier,
                // which every thread reaches after this sweep)
            }
        }
        if (n_row == 0) lds_barrier();                    // heading directions visible
        // 3. per-action value in FP64 (the 1024-thread kernel's scoring);
        //    actions whose nearest distance lies within kBand of the well
        //    radius get it recomputed exactly first.  Kept per action: value,
        //    nearest distance and whether the successor is inside a well or
        //    below the terrain.  The rounds of a wave that holds an action in
        //    each are scored unconditionally (a past the last action reads
        //    the last one), so that their FP64 chains interleave; a round
        //    with no action of the wave is skipped.
        auto flags = [](const Scored &c) { return (c.I > 0.0 ? 1 : 0) | (c.clr < 0.0 ? 2 : 0); };
        double V[APT], d2v[APT];
        int fl[APT];
        bool band[APT];
        double vloc = -INFINITY;
        bool mine_band = false;
        auto score_rounds = [&](auto nq_c) {
            constexpr int NQ = decltype(nq_c)::value;
#pragma unroll
            for (int q = 0; q < APT; ++q) {
                const int a = tid + q * NT;
                if (q >= NQ) {                            // every action of the round is past the last
                    V[q] = -INFINITY;
                    d2v[q] = INFINITY;
                    fl[q] = 0;
                    band[q] = false;
                    continue;
                }
                const int ac = a < A ? a : A - 1;
                const int h = ac / (NC * NV);
                const double d2 = nearest_d2<NC, NV>(at, ac, mA[q]);
                d2v[q] = d2;
                band[q] = a < A && d2 > cfg.band_lo2 && d2 < cfg.band_hi2;
                const Scored c = score_action(cfg, tb, at, ac, s, g, hc[h], hs[h], d2);
                V[q] = (a < A && !band[q]) ? c.V : -INFINITY;
                fl[q] = flags(c);
                if (band[q]) atomicOr(&sBand[a >> 5], 1u << (a & 31));
                mine_band = mine_band || band[q];
                vloc = fmax(vloc, V[q]);
            }
        };
        static_assert(APT <= 2, "one or two scoring rounds");
        if (nq >= APT) score_rounds(std::integral_constant<int, APT>());
        else if (nq == 1) score_rounds(std::integral_constant<int, 1>());
        else score_rounds(std::integral_constant<int, 0>());
        double wv = wave_max(vloc);
        if (lane == 0) red_d[wave] = wv;
        if (mine_band) s_any = 1;
        lds_barrier();
        if (s_any) {                                      // uniform; almost never taken
            lds_barrier();                                // every thread has read the flag
            if (tid == 0) s_any = 0;
            // exact FP64 nearest distance over the row's visible entries for
            // each flagged action; its owner thread takes the result
            for (int w = 0; w < (A + 31) / 32; ++w) {
                unsigned bits = sBand[w];
                while (bits) {
                    const int a = w * 32 + __builtin_ctz(bits);
                    bits &= bits - 1;
                    const int h = a / (NC * NV);
                    double qx, qy, qz;
                    successor(cfg, at, a, s, hc[h], hs[h], qx, qy, qz);
                    double dmin = INFINITY;
                    for (int j = tid; j < n_row; j += NT)
                        if (entry_visible(tb, rb + j, seq))
                            dmin = fmin(dmin, entry_d2(qx, qy, qz, tb.X[rb + j], tb.Y[rb + j], tb.Z[rb + j]));
                    dmin = -wave_max(-dmin);
                    if (lane == 0) red_d[wave] = dmin;
                    lds_barrier();
                    if (a % NT == tid) {
                        double d2 = red_d[0];
#pragma unroll
                        for (int q = 1; q < NW; ++q) d2 = fmin(d2, red_d[q]);
#pragma unroll
                        for (int q = 0; q < APT; ++q)
                            if (q == a / NT) d2v[q] = d2;
                    }
                    lds_barrier();
                }
            }
            vloc = -INFINITY;
#pragma unroll
            for (int q = 0; q < APT; ++q) {
                const int a = tid + q * NT;
                if (band[q]) {
                    const int h = a / (NC * NV);
                    const Scored c = score_action(cfg, tb, at, a, s, g, hc[h], hs[h], d2v[q]);
                    V[q] = c.V;
                    fl[q] = flags(c);
                }
                vloc = fmax(vloc, V[q]);
            }
            wv = wave_max(vloc);
            if (lane == 0) red_d[wave] = wv;
            lds_barrier();
        }
        // argmax: the largest value vm, then the lowest index inside the tie
        // band [vm - tie |vm|, vm], and the lowest-index largest action; each
        // wave publishes its lowest candidate with what the step needs of it
        double vm = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) vm = fmax(vm, red_d[w]);
        const double thr = vm - cfg.tie_rel * fabs(vm);
        int li = 0x7fffffff, ti = 0x7fffffff;
#pragma unroll
        for (int q = APT - 1; q >= 0; --q) {              // lowest index last
            const int a = tid + q * NT;
            if (a < A && V[q] >= thr) li = a;
            if (a < A && V[q] == vm) ti = a;
        }
        li = wave_min(li);
        ti = wave_min(ti);
        if (lane == 0) {
            s_wli[wave] = li;
            s_wti[wave] = ti;
        }
#pragma unroll
        for (int q = 0; q < APT; ++q)
            if (tid + q * NT == li) {
                s_wv[wave] = V[q];
                s_wd2[wave] = d2v[q];
                s_wfl[wave] = fl[q];
            }
        if (tid == 0 && stop.target > 0) s_stop = stop_v >= stop.target;
        lds_barrier();
        stop_now = s_stop;
        int best = 0x7fffffff, top = 0x7fffffff, bw = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int l = s_wli[w];
            if (l < best) {
                best = l;
                bw = w;
            }
            top = min(top, s_wti[w]);
        }
        if (vm == -INFINITY) best = -1;
        if (best < 0) {
            status = FASTMDP_NO_VALID_ACTION;
        } else {
            // every thread takes the step: the chosen action's successor (the
            // point its scoring was computed at), recorded as the pending point
            const int h = best / (NC * NV);
            double x, y, z;
            successor(cfg, at, best, s, hc[h], hs[h], x, y, z);
            const int flb = s_wfl[bw];
            if (tid == 0) pairs += (long long)A * n_vis;  // pairs with the plans this request sees
            if (tid == 0) {
                const int ri = n % RING;
                sP[ri][0] = x;
                sP[ri][1] = y;
                sP[ri][2] = z;
                sPv[ri] = s_wv[bw];
                sPd[ri] = s_wd2[bw];
                sPa[ri] = best;
                sPs[ri] = n_row;
                sPt[ri] = top != best ? top : -1;
            }
            // a detour batch next (it ends in a run once the goal-directed
            // action is the choice), unless those decided nothing lately
            if (cfg.run_ok) {
                singly -= singly > 0;
                direct = 0;
                if (singly == 0) mode = cfg.detour_ok ? DETOUR : STRAIGHT;
            }
            s[0] = x; s[1] = y; s[2] = z;
            n += 1;
            if (flb & 1) status = FASTMDP_REJECT_SEPARATION;
            else if (flb & 2) status = FASTMDP_REJECT_TERRAIN;
        }
        // (the band bits were last read before the barrier above; the next
        // step sets them after its first barrier)
        for (int w = tid; w < kMaxActions / 32; w += NT) sBand[w] = 0u;
        buf ^= 1;
        steps_here += 1;
    }
    __syncthreads();   // the last points' records visible
    for (int i = fl + 64 * wave; i < n; i += 64 * NW) write_points(i, n);
    __syncthreads();   // the trajectory complete for every thread

    // Commit validation (validate_points' rule and arithmetic): the points
    // whose scored nearest plan is within R_sep + 1 m, one per wave at a time,
    // against the records of the cells around each and the later columns
    // that its scoring counted.  (A point kept from an earlier launch may
    // have counted fewer columns than are indexed now; the entries since
    // were checked against it, at a larger distance, when they came.)
    if (validate && status == FASTMDP_OK) {
        const double r2 = cfg.R_sep * cfg.R_sep;
        const double clear2 = (cfg.R_sep + 1.0) * (cfg.R_sep + 1.0);
        int bad = 0;
        for (int k0 = 0; k0 < n; k0 += NT) {              // uniform
            const int k = k0 + NW * lane + wave;
            bool near = false;
            if (k < n) {
                const double *x = tr.xyz + (pt_base + k) * 3;
                if (tb.terr && x[2] - terrain_height(tb, x[0], x[1]) < 0.0) bad = 1;
                near = !(tr.nd[pt_base + k] > clear2);
            }
            for (uint64_t fb = __ballot(near); fb; fb &= fb - 1) {          // uniform per wave
                const int kk = k0 + NW * __builtin_ctzll(fb) + wave;
                const double *x = tr.xyz + (pt_base + kk) * 3;
                const double px = x[0], py = x[1], pz = x[2];
                const int row = t0 + kk, lim = tr.seen[pt_base + kk];
                const int idn = row < tb.rows ? tb.gn[row] : 0;
                const size_t rb = (size_t)row * tb.cap;
                const float fx = (float)px, fy = (float)py;
                const float vb = (float)cfg.R_sep * 1.001f + 1.0f + 1e-6f * fmaxf(fabsf(fx), fabsf(fy));
                if (idn > 0) {
                    const Cells cl = cells(fx, fy, vb);
                    for (int cy = cl.y0; cy <= cl.y1; cy += 2) {            // uniform
                        int a, b;
                        cell_range(row, cl, cy, a, b);
                        for (a += lane & 31; a < b; a += 32) {
                            const float4 p = tb.grec[rb + a];
                            if (__float_as_int(p.w) < seq && entry_d2(px, py, pz, p.x, p.y, p.z) < r2) bad = 1;
                        }
                    }
                }
                for (int j = idn + lane; j < lim; j += 64) {
                    const float ex = tb.X[rb + j], ey = tb.Y[rb + j];
                    if (fabsf(ex - fx) <= vb && fabsf(ey - fy) <= vb && entry_visible(tb, rb + j, seq) &&
                        entry_d2(px, py, pz, ex, ey, tb.Z[rb + j]) < r2)
                        bad = 1;
                }
            }
        }
        bad = __syncthreads_or(bad);
        if (tid == 0) S.valid = bad == 0;
    }

    if (pairs > 0 || entries > 0) {
        atomicAdd(reinterpret_cast<unsigned long long *>(&S.pairs), (unsigned long long)pairs);
        atomicAdd(reinterpret_cast<unsigned long long *>(&S.entries), (unsigned long long)entries);
    }
    if (tid == 0) {
        S.n_points = n;
        S.status = status;
        if (stop.target > 0 && status != kRunning) atomicAdd(stop.ctr, 1);
        S.steps += steps_here;
    }
}

template <int NC, int NV, int ZC>
hipError_t launch_t(int nblk, int nt, hipStream_t st, const DevCfg &c, const DevTable &t, Slot *s, const int *list,
                    const Traj &tr, int budget, int validate, int epoch, const LaunchStop &stop) {
    if (nt == kRangeThreadsSolo)
        hipLaunchKernelGGL((range_planner_kernel<kRangeThreadsSolo, 1, NC, NV, ZC>), dim3(nblk), dim3(nt), 0, st, c,
                           t, s, list, tr, budget, validate, epoch, stop);
    else if (nt == kRangeThreads && nblk <= 2 * c.n_cu)        // two per CU: no spilled registers
        hipLaunchKernelGGL((range_planner_kernel<kRangeThreads, 2, NC, NV, ZC>), dim3(nblk), dim3(nt), 0, st, c, t,
                           s, list, tr, budget, validate, epoch, stop);
    else if (nt == kRangeThreads)
        hipLaunchKernelGGL((range_planner_kernel<kRangeThreads, kRangePerCU, NC, NV, ZC>), dim3(nblk), dim3(nt), 0,
                           st, c, t, s, list, tr, budget, validate, epoch, stop);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_range_planner(int nblk, hipStream_t st, const DevCfg &c, const DevTable &t, Slot *s,
                                const int *list, const Traj &tr, int budget, int validate, int epoch,
                                const LaunchStop &stop) {
    if (!c.range_query || c.lookahead > 1 || c.n_head > kRangeMaxHeads) return hipErrorInvalidValue;
    const int zc = c.zero_climb;
    const int nt = range_planner_threads(c, nblk);
#define FMDP_RANGE_SHAPE(NC, NV, ZC) \
    if (c.n_climb == NC && c.n_speed == NV && zc == ZC) \
        return launch_t<NC, NV, ZC>(nblk, nt, st, c, t, s, list, tr, budget, validate, epoch, stop);
    FMDP_PLANNER_SHAPES(FMDP_RANGE_SHAPE)
#undef FMDP_RANGE_SHAPE
    return hipErrorInvalidValue;
}

}  // namespace fmdp
