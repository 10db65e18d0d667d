// table.hip -- known-plan table kernels: load scatter, commit validation and
// append (the accepted-plan database of Sec. V), and the first-come-first-
// served sequencer that accepts concurrently planned trajectories strictly in
// request order.
#include "planner.h"
#include "wave.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>

namespace fmdp {

namespace {

__device__ double table_terrain_height(const DevTable &tb, double x, double y) {
    double fx = (x - tb.tx0) / tb.tcell;
    double fy = (y - tb.ty0) / tb.tcell;
    fx = fmin(fmax(fx, 0.0), (double)(tb.tnx - 1));
    fy = fmin(fmax(fy, 0.0), (double)(tb.tny - 1));
    int i = (int)floor(fx), j = (int)floor(fy);
    i = i > tb.tnx - 2 ? tb.tnx - 2 : i;
    j = j > tb.tny - 2 ? tb.tny - 2 : j;
    const double ax = fx - i, ay = fy - j;
    const float *h = tb.terr + (size_t)j * tb.tnx + i;
    const double h00 = h[0], h10 = h[1], h01 = h[tb.tnx], h11 = h[tb.tnx + 1];
    return (1.0 - ay) * ((1.0 - ax) * h00 + ax * h10) + ay * ((1.0 - ax) * h01 + ax * h11);
}

__global__ void fill_int_kernel(int *p, int value, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

__global__ void scatter_points_kernel(DevTable tb, const float *pts, const int *rows, const int *cols, int n,
                                      int own) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t idx = (size_t)rows[i] * tb.cap + cols[i];
    tb.X[idx] = pts[3 * i + 0];
    tb.Y[idx] = pts[3 * i + 1];
    tb.Z[idx] = pts[3 * i + 2];
    if (tb.Q) tb.Q[idx] = quantised(tb, pts[3 * i + 0], pts[3 * i + 1]);
    tb.vis[idx] = own;
    tb.own[idx] = own;
    tb.dead[idx] = kAlive;
}

// One workgroup per row, its whole capacity: a file that breaks off has
// replaced points past the row's count too.
__global__ void quantise_table_kernel(DevTable tb) {
    const int row = blockIdx.x;
    for (int j = threadIdx.x; j < tb.cap; j += blockDim.x) {
        const size_t idx = (size_t)row * tb.cap + j;
        tb.Q[idx] = quantised(tb, tb.X[idx], tb.Y[idx]);
    }
}

// One workgroup per row: the indexed prefix, a histogram of its cells, their
// offsets, then the records (a cell's in any order: the planner takes a
// minimum and a count over them).
constexpr int kGridThreads = 256;

__global__ __launch_bounds__(kGridThreads) void build_grid_kernel(DevTable tb, int limit) {
    __shared__ int cell_n[kGridCells], part[kGridThreads], s_np;
    const int row = blockIdx.x, tid = threadIdx.x;
    const int n = min(tb.rowN[row], tb.cap);
    const size_t rb = (size_t)row * tb.cap;
    if (tid == 0) s_np = n;
    for (int c = tid; c < kGridCells; c += kGridThreads) cell_n[c] = 0;
    __syncthreads();
    if (n >= kGridMin) {
        int np = n;
        for (int j = tid; j < n; j += kGridThreads)
            if (tb.vis[rb + j] != kAlive && tb.own[rb + j] >= limit) np = min(np, j);
        if (np < n) atomicMin(&s_np, np);
    }
    __syncthreads();
    const int np = s_np >= kGridMin ? s_np : 0;
    if (tid == 0) tb.gn[row] = np;
    if (np == 0) return;                                     // uniform
    auto cell = [&](size_t idx) {
        return grid_cell(tb.Y[idx], tb.qy0, tb.gsy) * kGrid + grid_cell(tb.X[idx], tb.qx0, tb.gsx);
    };
    for (int j = tid; j < np; j += kGridThreads)
        if (tb.vis[rb + j] != kAlive) atomicAdd(&cell_n[cell(rb + j)], 1);
    __syncthreads();
    constexpr int PER = kGridCells / kGridThreads;           // cells per thread
    int mine[PER], sum = 0;
    for (int i = 0; i < PER; ++i) {
        mine[i] = sum;
        sum += cell_n[tid * PER + i];
    }
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < kGridThreads; d <<= 1) {
        const int v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int *off = tb.goff + (size_t)row * (kGridCells + 1);
    for (int i = 0; i < PER; ++i) {
        const int o = part[tid] - sum + mine[i];
        cell_n[tid * PER + i] = o;
        off[tid * PER + i] = o;
    }
    if (tid == kGridThreads - 1) off[kGridCells] = part[tid];
    __syncthreads();
    for (int j = tid; j < np; j += kGridThreads) {
        const int v = tb.vis[rb + j];
        if (v == kAlive) continue;
        const int p = atomicAdd(&cell_n[cell(rb + j)], 1);
        tb.grec[rb + p] = make_float4(tb.X[rb + j], tb.Y[rb + j], tb.Z[rb + j], __int_as_float(v));
    }
}

// Plans appended in order from one staging buffer, by one workgroup: plan j
// (t0[j], len[j] points from xyz + 3 * off) takes the next column of each row
// it spans.  A plan spans a row at most once, so its points take their
// columns independently; plans follow one another behind a barrier, which
// gives every row its entries in plan order (the columns the host-computed
// scatter of fastmdp_load_plans gives).  The row counts move by device
// atomics, which the next plan reads after the barrier.
__global__ __launch_bounds__(1024) void append_plans_kernel(DevTable tb, const int *t0, const int *len, int n,
                                                            const float *xyz) {
    long long off = 0;
    for (int j = 0; j < n; ++j) {
        const int t = t0[j], L = len[j];
        for (int k = threadIdx.x; k < L; k += blockDim.x) {
            const int row = t + k;
            const int col = atomicAdd(&tb.rowN[row], 1);
            const size_t idx = (size_t)row * tb.cap + col;
            const float *p = xyz + 3 * (off + k);
            tb.X[idx] = p[0];
            tb.Y[idx] = p[1];
            tb.Z[idx] = p[2];
            if (tb.Q) tb.Q[idx] = quantised(tb, p[0], p[1]);
            tb.vis[idx] = -1;
            tb.own[idx] = -1;
            tb.dead[idx] = kAlive;
        }
        off += L;
        __syncthreads();
    }
}

// Commit validation of one trajectory point as planned (FP64) against every
// entry of its row visible to `seq`, as stored (FP32), in FP64; terrain
// clearance; capacity.  flag bit 0: conflict, bit 1: capacity.
__device__ int check_point(const DevCfg &c, const DevTable &tb, const double p[3], int row, int seq, int tid,
                           int nthr) {
    if (row >= tb.rows) return 2;
    const int n_row = tb.rowN[row];
    int f = n_row >= tb.cap ? 2 : 0;
    const double r2 = c.R_sep * c.R_sep;
    const size_t rb = (size_t)row * tb.cap;
    for (int j = tid; j < n_row; j += nthr)
        if (entry_visible(tb, rb + j, seq) && entry_d2(p[0], p[1], p[2], tb.X[rb + j], tb.Y[rb + j], tb.Z[rb + j]) < r2)
            f |= 1;
    if (tid == 0 && tb.terr && p[2] - table_terrain_height(tb, p[0], p[1]) < 0.0) f |= 1;
    return f;
}

__global__ void commit_check_kernel(DevCfg c, DevTable tb, const double *pts, int t0, int n, int seq, int *flags) {
    const int k = blockIdx.x;
    if (k >= n) return;
    const double p[3] = {pts[3 * k], pts[3 * k + 1], pts[3 * k + 2]};
    const int f = check_point(c, tb, p, t0 + k, seq, threadIdx.x, blockDim.x);
    const int conflict = __syncthreads_or(f & 1), full = __syncthreads_or(f & 2);
    if (threadIdx.x == 0) flags[k] = (conflict ? 1 : 0) | (full ? 2 : 0);
}

// Append the trajectory rounded to FP32 (the table's storage format).
// Every workgroup looks at all points' flags; one tells the host.  Points and
// result lie in pinned host memory: check and append take 10 us, where the
// copy of the points, the flag's clearing and its copy added three transfers.
__global__ void commit_append_kernel(DevTable tb, const double *pts, int t0, int n, int own, const int *flags,
                                     int *result) {
    int f = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) f |= flags[i];
    const int conflict = __syncthreads_or(f & 1), full = __syncthreads_or(f & 2);
    if (blockIdx.x == 0 && threadIdx.x == 0) *result = (conflict ? 1 : 0) | (full ? 2 : 0);
    if (conflict || full) return;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int row = t0 + k;
    const int col = tb.rowN[row];
    const size_t idx = (size_t)row * tb.cap + col;
    tb.X[idx] = (float)pts[3 * k + 0];
    tb.Y[idx] = (float)pts[3 * k + 1];
    tb.Z[idx] = (float)pts[3 * k + 2];
    if (tb.Q) tb.Q[idx] = quantised(tb, (float)pts[3 * k + 0], (float)pts[3 * k + 1]);
    tb.vis[idx] = own;
    tb.own[idx] = own;
    tb.dead[idx] = kAlive;
    tb.rowN[row] = col + 1;
}

// ---------------------------------------------------------------------------
// First-come-first-served with concurrent requests and tentative plans.
//
// Request q (sequence number q) plans against the live table entries of
// every earlier request: plans accepted before it and the tentative
// trajectories of earlier requests that finished planning.  A finished
// trajectory with status OK enters the table at once as tentative entries
// owned by q; when q is re-planned from step k its entries from step k on are
// withdrawn (dead = epoch, logged).  Passes run between planner launches over
// every admitted, not yet accepted request, those still planning included;
// in pass e (epoch e):
//   1. insert: every finished OK trajectory enters the table (missing entries);
//   2. check: every trajectory, as far as it is planned, is tested against
//      what changed since it scored each row.  A point is in step with the
//      table when its pass ends (seen = rowN, ep = e - 1), and nothing
//      changes during a launch, so that is
//        - the entries entered in this pass and visible to it: an added plan
//          only adds a penalty, so every value at that step can only fall and
//          the chosen action stays chosen with the same value unless the
//          plan lands within the well radius of the chosen successor (or of
//          the largest action's successor when the choice was made inside
//          the tie band);
//        - for points scored before the last launch, the entries withdrawn
//          in the last pass that it saw (column < seen[k], owner < q): a
//          withdrawal can raise any successor's value, so it matters when
//          within the well radius of any successor, i.e. within `reach_state`
//          of the scored state;
//        - for the origin (k = 0) the test is the origin check.
//      The first affected step is recorded; the steps before it stand;
//   3. withdraw: an affected trajectory drops its points from the first
//      affected step on (their entries die with epoch e) and goes back to
//      (or on) planning; a finished trajectory that is not OK (or failed its
//      commit validation) withdraws all its entries.
// Acceptance (host side) walks the requests in order: a finished request
// whose checks are clean and all of whose predecessors are accepted is
// final; its tentative entries simply stay.  A request that withdrew entries
// in this pass ends the walk, because later requests have not yet been
// checked against the withdrawal.
//
// Three launches a pass.  Before (checks of finished requests only, so that
// a request in its second launch had every entry since its first to scan;
// withdrawn entries tested one by one against every request; counts, lists
// and the slots copied one by one) a pass of the 1000-request stream took 190
// us in eight kernels and 150 us of copies and launches around them.
// ---------------------------------------------------------------------------
constexpr int kPassThreads = 256;

// Bounding box of a wave's points (lanes without one pass infinities).
__device__ __forceinline__ float4 wave_box(bool in, float x, float y) {
    return make_float4(wave_min_f32(in ? x : INFINITY), wave_max_f32(in ? x : -INFINITY),
                       wave_min_f32(in ? y : INFINITY), wave_max_f32(in ? y : -INFINITY));
}

__global__ __launch_bounds__(kPassThreads) void fcfs_insert_kernel(DevTable tb, Slot *slots, const int *list,
                                                                   Traj tr, PassBufs pb) {
    const int slot = list[blockIdx.x];
    Slot &S = slots[slot];
    const int status = S.status;
    if (threadIdx.x == 0) S.first = 0x7fffffff;             // opened here for the checks that follow
    if (status != FASTMDP_OK || !S.valid) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = S.n_points, t0 = S.t0, own = S.seq;
    const size_t base = (size_t)slot * tr.stride;
    int err = 0, added = 0;
    for (int k = threadIdx.x; k < n; k += kPassThreads) {
        if (tr.col[base + k] >= 0) continue;
        added = 1;
        const int row = t0 + k;
        if (row >= tb.rows) { err = 1; continue; }
        const int col = atomicAdd(&tb.rowN[row], 1);
        if (col >= tb.cap) {                          // row full: undo and report
            atomicSub(&tb.rowN[row], 1);
            err = 1;
            continue;
        }
        const double *x = tr.xyz + (base + k) * 3;
        const size_t idx = (size_t)row * tb.cap + col;
        tb.X[idx] = (float)x[0];
        tb.Y[idx] = (float)x[1];
        tb.Z[idx] = (float)x[2];
        if (tb.Q) tb.Q[idx] = quantised(tb, (float)x[0], (float)x[1]);
        tb.vis[idx] = own;
        tb.own[idx] = own;
        tb.dead[idx] = kAlive;
        tr.col[base + k] = col;
    }
    if (err) S.err = 1;
    // a trajectory that entered entries: its row-block boxes (a wave's lanes
    // hold one block's rows), for the check of the entries entered in this pass
    if (!__syncthreads_or(added) || n == 0) return;
    const int b0 = t0 / kRowBlock, nb = (t0 + n - 1) / kRowBlock - b0 + 1;
    for (int b = wave; b < nb; b += kPassThreads / 64) {      // uniform per wave
        const int k = (b0 + b) * kRowBlock + lane - t0;
        const bool in = k >= 0 && k < n;
        const double *x = tr.xyz + (base + (in ? k : 0)) * 3;
        const float4 q = wave_box(in, (float)x[0], (float)x[1]);    // the values the table stores
        if (lane == 0) pb.box[(size_t)slot * kRowBlocks + b] = q;
    }
    if (threadIdx.x == 0) pb.ins[atomicAdd(pb.ins_n, 1)] = make_int4(slot, t0, n, own);
}

// The window's check of added entries takes a request's points in chunks.
constexpr int kCheckPoints = 64;

// The successor the added-entry rule tests besides the chosen one x_k
// (point k): the largest action's, when the step to point k chose inside
// the tie band (top_k >= 0), else x_k itself.
__device__ __forceinline__ void top_successor(const DevCfg &c, const Slot &S, const Traj &tr, size_t base, int k,
                                              int top_k, double y[3]) {
    const double *x = tr.xyz + (base + k) * 3;
    y[0] = x[0];
    y[1] = x[1];
    y[2] = x[2];
    if (top_k < 0) return;
    const double *sp = tr.xyz + (base + k - 1) * 3;
    const double bx = S.goal[0] - sp[0], by = S.goal[1] - sp[1];
    const double r = sqrt(bx * bx + by * by);
    const double cb = r > 0.0 ? bx / r : 1.0, sb = r > 0.0 ? by / r : 0.0;
    const int h = top_k / (c.n_climb * c.n_speed);
    const int cl = (top_k / c.n_speed) % c.n_climb;
    const int v = top_k % c.n_speed;
    const double th = 2.0 * M_PI * (double)h / (double)c.n_head;
    const double c0 = cos(th), s0 = sin(th);
    const double step = c.speed[v] * c.dt;
    y[0] = sp[0] + step * (cb * c0 - sb * s0);
    y[1] = sp[1] + step * (sb * c0 + cb * s0);
    y[2] = sp[2] + c.climb[cl] * c.dt;
}

// Check (one workgroup per request): this request's scored states against
// the trajectories inserted in this pass and the pieces withdrawn in the last
// one, trajectory against trajectory.  The states are boxed per block of
// kRowBlock rows (in LDS); a block of an inserted or withdrawn piece of an
// earlier request whose box comes within reach + the longest step (+ 1 m and
// 1e-6 |coordinate| for the FP32 boxes) of the request's box is a candidate,
// and a wave then tests its rows, one per lane, by the rules above.  Outside
// such blocks no entry can matter.
constexpr int kNewCand = 4 * kPassThreads;             // (piece, block) pairs tested per round

__global__ __launch_bounds__(kPassThreads) void fcfs_check_kernel(DevCfg c, DevTable tb, Slot *slots, const int *list,
                                                                  Traj tr, PassBufs pb, DeathLog dl, int epoch) {
    __shared__ float4 s_box[kRowBlocks];                  // the scored states' boxes
    __shared__ int2 s_cand[kNewCand];                     // (piece, block)
    __shared__ int s_nc, s_first;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slot = list[blockIdx.x];
    Slot &S = slots[slot];
    const int n_ins = *pb.ins_n, n_seg = min(dl.n[1], dl.seg_cap);
    const int n = S.n_points, t0 = S.t0, q = S.seq;
    if (n == 0 || (n_ins == 0 && n_seg == 0)) return;        // uniform
    const size_t base = (size_t)slot * tr.stride;
    const int b0 = t0 / kRowBlock, nb = (t0 + n - 1) / kRowBlock - b0 + 1;
    for (int b = wave; b < nb; b += kPassThreads / 64) {      // uniform per wave
        const int k = (b0 + b) * kRowBlock + lane - t0;
        const bool in = k >= 0 && k < n;
        const double *x = tr.xyz + (base + (in && k > 0 ? k - 1 : 0)) * 3;  // the state point k was scored from
        const float4 v = wave_box(in, (float)x[0], (float)x[1]);
        if (lane == 0) s_box[b] = v;
    }
    if (tid == 0) {
        s_nc = 0;
        s_first = 0x7fffffff;
    }
    __syncthreads();
    const double r2 = c.reach * c.reach;
    const double rs2 = c.reach_state * c.reach_state;
    const double ro2 = (c.R_sep + 1.0) * (c.R_sep + 1.0);
    const float reach_f = (float)(c.reach + c.max_step) + 1.0f;
    // 1. box against box: pieces [0, n_ins) are insertions, the rest withdrawals
    const int total = (n_ins + n_seg) * nb;
    for (int c0 = 0; c0 < total; c0 += kNewCand) {            // uniform
        for (int i = c0 + tid; i < min(total, c0 + kNewCand); i += kPassThreads) {
            const int pi = i / nb, b = i - pi * nb;
            int row0, np, own;
            const float4 *box;
            if (pi < n_ins) {
                const int4 d = pb.ins[pi];
                row0 = d.y;
                np = d.z;
                own = d.w;
                box = pb.box + (size_t)d.x * kRowBlocks;
            } else {
                const int4 d = dl.seg[pi - n_ins];
                row0 = d.z;
                np = d.y;
                own = d.w;
                box = dl.box + dl.seg_box[pi - n_ins];
            }
            if (own >= q) continue;                            // not visible to this request
            const int pb0 = row0 / kRowBlock, pnb = (row0 + np - 1) / kRowBlock - pb0 + 1;
            const int bb = b0 + b - pb0;
            if (bb < 0 || bb >= pnb) continue;
            const float4 e = box[bb];
            const float4 o = s_box[b];
            if (!(o.x <= o.y)) continue;                       // no point of the request in this block
            const float m = reach_f + 1e-6f * fmaxf(fmaxf(fabsf(o.x), fabsf(o.y)), fmaxf(fabsf(o.z), fabsf(o.w)));
            if (e.x > o.y + m || e.y < o.x - m || e.z > o.w + m || e.w < o.z - m) continue;
            s_cand[atomicAdd(&s_nc, 1)] = make_int2(pi, b);
        }
        __syncthreads();
        // 2. the candidate blocks' rows, one per lane
        const int nc = s_nc;
        for (int ci = wave; ci < nc; ci += kPassThreads / 64) {
            const int pi = s_cand[ci].x;
            const int r = (b0 + s_cand[ci].y) * kRowBlock + lane;
            const int k = r - t0;
            if (k < 0 || k >= n || r >= tb.rows) continue;
            if (pi < n_ins) {
                const int4 d = pb.ins[pi];
                const int kp = r - d.y;
                if (kp < 0 || kp >= d.z) continue;
                const int col = tr.col[(size_t)d.x * tr.stride + kp];
                if (col < pb.rowN_pre[r] || col >= tb.cap) continue;  // entered before this pass (or none)
                const size_t idx = (size_t)r * tb.cap + col;
                if (!entry_visible(tb, idx, q)) continue;
                const double *x = tr.xyz + (base + k) * 3;
                double y[3];
                top_successor(c, S, tr, base, k, k > 0 ? tr.top[base + k] : -1, y);
                const float px = tb.X[idx], py = tb.Y[idx], pz = tb.Z[idx];
                if (entry_d2(x[0], x[1], x[2], px, py, pz) < r2 || entry_d2(y[0], y[1], y[2], px, py, pz) < r2)
                    atomicMin(&s_first, k);
            } else {
                const int4 d = dl.seg[pi - n_ins];
                const int i = r - d.z;
                if (i < 0 || i >= d.y) continue;
                if (dl.col[d.x + i] >= tr.seen[base + k] || tr.ep[base + k] >= epoch - 1) continue;
                const double *sp = tr.xyz + (base + (k == 0 ? 0 : k - 1)) * 3;
                if (entry_d2(sp[0], sp[1], sp[2], dl.x[d.x + i], dl.y[d.x + i], dl.z[d.x + i]) < (k == 0 ? ro2 : rs2))
                    atomicMin(&s_first, k);
            }
        }
        __syncthreads();
        if (tid == 0) s_nc = 0;
        __syncthreads();
    }
    if (tid == 0 && s_first != 0x7fffffff) S.first = s_first;
}

// Lookahead window W > 1: the step to point k (from point k-1 at row
// t0 + k - 1) scored rows t0 + k - 1 + w, w = 1..W, and recorded the entry
// counts it saw in seenw.  The same two rules per window row: an added entry
// matters within reach of the chosen action's window point w (or of the
// largest action's, when the choice was made inside the tie band), a
// withdrawn one within reach of any action's point w, i.e. within
// reach + w * max_step of point k - 1.  The origin (k = 0) is the origin
// check, as without the window.

// Window point w of action a from state sp (the action's heading is an
// offset from the goal bearing at sp).
__device__ void table_window_point(const DevCfg &c, const double sp[3], const double goal[3], int a, int w,
                                   double y[3]) {
    const double bx = goal[0] - sp[0], by = goal[1] - sp[1];
    const double r = sqrt(bx * bx + by * by);
    const double cb = r > 0.0 ? bx / r : 1.0, sb = r > 0.0 ? by / r : 0.0;
    const int h = a / (c.n_climb * c.n_speed);
    const int cl = (a / c.n_speed) % c.n_climb;
    const int v = a % c.n_speed;
    const double th = 2.0 * M_PI * (double)h / (double)c.n_head;
    const double c0 = cos(th), s0 = sin(th);
    const double k = (double)w;
    const double step = k * (c.speed[v] * c.dt);
    y[0] = sp[0] + step * (cb * c0 - sb * s0);
    y[1] = sp[1] + step * (sb * c0 + cb * s0);
    y[2] = sp[2] + k * (c.climb[cl] * c.dt);
}

__global__ __launch_bounds__(kPassThreads) void fcfs_check_dead_window_kernel(DevCfg c, DevTable tb, Slot *slots,
                                                                              const int *list, Traj tr, DeathLog dl,
                                                                              int epoch) {
    __shared__ int s_first;
    const int tid = threadIdx.x;
    const int slot = list[blockIdx.x];
    Slot &S = slots[slot];
    const int n = S.n_points, t0 = S.t0, q = S.seq, W = c.lookahead;
    const int n_seg = min(dl.n[1], dl.seg_cap);
    if (n == 0 || n_seg == 0) return;                        // uniform
    const size_t base = (size_t)slot * tr.stride;
    if (tid == 0) s_first = 0x7fffffff;
    __syncthreads();
    const double ro2 = (c.R_sep + 1.0) * (c.R_sep + 1.0);
    for (int si = 0; si < n_seg; ++si) {                      // uniform
        const int4 d = dl.seg[si];
        if (d.w >= q) continue;                               // uniform: not visible to this request
        for (int i = tid; i < d.y; i += kPassThreads) {
            const int r = d.z + i - t0, col = dl.col[d.x + i];
            const float ex = dl.x[d.x + i], ey = dl.y[d.x + i], ez = dl.z[d.x + i];
            if (r == 0 && col < tr.seen[base] && tr.ep[base] < epoch - 1) {       // the origin check
                const double *o = tr.xyz + base * 3;
                if (entry_d2(o[0], o[1], o[2], ex, ey, ez) < ro2) atomicMin(&s_first, 0);
            }
            for (int w = 1; w <= W; ++w) {
                const int k = r - w + 1;                  // the step to point k scored this row as point w
                if (k < 1 || k >= n) continue;
                if (col >= tr.seenw[(base + k) * W + w - 1] || tr.ep[base + k] >= epoch - 1) continue;
                const double *sp = tr.xyz + (base + k - 1) * 3;
                const double rw = c.reach + w * c.max_step;
                if (entry_d2(sp[0], sp[1], sp[2], ex, ey, ez) < rw * rw) atomicMin(&s_first, k);
            }
        }
    }
    __syncthreads();
    if (tid == 0 && s_first != 0x7fffffff) atomicMin(&S.first, s_first);
}

// Added entries, window W > 1: one wave per point at a time, its lanes over
// the new entries of each window row; the wave stops at the first entry in
// reach.
__global__ __launch_bounds__(kPassThreads) void fcfs_check_add_window_kernel(DevCfg c, DevTable tb, Slot *slots,
                                                                             const int *list, Traj tr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = list[blockIdx.x];
    Slot &S = slots[slot];
    const int n = S.n_points, t0 = S.t0, q = S.seq, W = c.lookahead;
    const int k0 = blockIdx.y * kCheckPoints;
    if (k0 >= n) return;
    const size_t base = (size_t)slot * tr.stride;
    const double r2 = c.reach * c.reach;
    constexpr int per_wave = kCheckPoints / (kPassThreads / 64);
    for (int i = 0; i < per_wave; ++i) {
        const int k = k0 + wave * per_wave + i;
        if (k >= n) break;
        int hit = 0;
        if (k == 0) {                                     // the origin check: row t0 against R_sep + 1 m
            const int row = t0;
            if (row < tb.rows) {
                const int lo = tr.seen[base], hi = min(tb.rowN[row], tb.cap);
                const double *x = tr.xyz + base * 3;
                const size_t rb = (size_t)row * tb.cap;
                for (int j = lo + lane; j < hi && !hit; j += 64)
                    hit = entry_visible(tb, rb + j, q) &&
                          entry_d2(x[0], x[1], x[2], tb.X[rb + j], tb.Y[rb + j], tb.Z[rb + j]) < r2;
            }
        } else {
            const double *sp = tr.xyz + (base + k - 1) * 3, *sk = tr.xyz + (base + k) * 3;
            const int top = tr.top[base + k];
            for (int w = 1; w <= W && !__ballot(hit); ++w) {
                const int row = t0 + k - 1 + w;
                if (row >= tb.rows) break;
                const int lo = tr.seenw[(base + k) * W + w - 1], hi = min(tb.rowN[row], tb.cap);
                if (lo >= hi) continue;
                // the chosen action's point w lies on the line through points k-1 and k
                const double y[3] = {sp[0] + w * (sk[0] - sp[0]), sp[1] + w * (sk[1] - sp[1]),
                                     sp[2] + w * (sk[2] - sp[2])};
                double u[3] = {y[0], y[1], y[2]};
                if (top >= 0) table_window_point(c, sp, S.goal, top, w, u);
                const size_t rb = (size_t)row * tb.cap;
                for (int j = lo + lane; j < hi && !hit; j += 64) {
                    if (!entry_visible(tb, rb + j, q)) continue;
                    const float px = tb.X[rb + j], py = tb.Y[rb + j], pz = tb.Z[rb + j];
                    hit = entry_d2(y[0], y[1], y[2], px, py, pz) < r2 || entry_d2(u[0], u[1], u[2], px, py, pz) < r2;
                }
            }
        }
        if (__ballot(hit)) {
            if (lane == 0) atomicMin(&S.first, k);
            break;                                        // later points of this wave cannot be first
        }
    }
}

// Check, last part, and withdrawal (one workgroup per request): the steps
// before the first affected one are in step with the table now; an affected
// trajectory, or one that was refused, withdraws its entries from there on,
// as one segment of the pass's log (inserted points are a prefix of the
// trajectory, so the entries are of consecutive rows).  The slot then goes
// to the host's mirror.  Workgroups past the list prepare the next pass: the
// row counts before its insertions, no insertion, an empty log where the
// last pass's was, a cleared stop counter.
constexpr int kPrepRows = 4 * kPassThreads;            // row counts copied per workgroup

template <bool LOOK>
__global__ __launch_bounds__(kPassThreads) void fcfs_finish_kernel(DevCfg c, DevTable tb, Slot *slots, const int *list,
                                                                   int n_list, Traj tr, DeathLog prev, DeathLog cur,
                                                                   PassBufs pb, int epoch) {
    __shared__ int s_m, s_base, s_box, s_err;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if ((int)blockIdx.x >= n_list) {                         // uniform
        const int p = blockIdx.x - n_list;
        for (int r = p * kPrepRows + tid; r < min(tb.rows, (p + 1) * kPrepRows); r += kPassThreads)
            pb.rowN_pre[r] = tb.rowN[r];
        if (p == 0 && tid < 3) prev.n[tid] = 0;
        if (p == 0 && tid == 3) *pb.ins_n = 0;
        if (p == 0 && tid == 4) *pb.stop = 0;
        return;
    }
    const int slot = list[blockIdx.x];
    Slot &S = slots[slot];
    const int n = S.n_points, t0 = S.t0, first = S.first, status = S.status, W = c.lookahead;
    const size_t base = (size_t)slot * tr.stride;
    for (int k = tid; k < min(n, first); k += kPassThreads) {
        const int row = t0 + k;
        if (row < tb.rows) tr.seen[base + k] = min(tb.rowN[row], tb.cap);
        if (LOOK && k > 0)
            for (int w = 1; w <= W; ++w) {
                const int rw = t0 + k - 1 + w;
                tr.seenw[(base + k) * W + w - 1] = rw < tb.rows ? min(tb.rowN[rw], tb.cap) : 0;
            }
        tr.ep[base + k] = epoch - 1;
    }
    const bool affected = first < n;
    int from = n;
    if (affected) from = first;
    else if (status != kRunning && (status != FASTMDP_OK || !S.valid)) from = 0;
    if (tid == 0) {
        s_m = from;
        s_err = 0;
    }
    __syncthreads();
    int m = from;                                            // one past the last inserted point
    for (int k = from + tid; k < n; k += kPassThreads)
        if (tr.col[base + k] >= 0) m = k + 1;
    if (m > from) atomicMax(&s_m, m);
    __syncthreads();
    m = s_m;
    const int cnt = m - from;
    if (cnt > 0) {                                           // uniform
        const int b0 = (t0 + from) / kRowBlock, nb = (t0 + m - 1) / kRowBlock - b0 + 1;
        if (tid == 0) {
            const int e = atomicAdd(&cur.n[0], cnt), g = atomicAdd(&cur.n[1], 1), x = atomicAdd(&cur.n[2], nb);
            if (e + cnt > cur.cap || g >= cur.seg_cap || x + nb > cur.box_cap) {
                s_err = 1;
                if (g < cur.seg_cap) {                       // (an empty piece: nothing of it is read)
                    cur.seg[g] = make_int4(0, 0, 0, 0x7fffffff);
                    cur.seg_box[g] = 0;
                }
            } else {
                cur.seg[g] = make_int4(e, cnt, t0 + from, S.seq);
                cur.seg_box[g] = x;
            }
            s_base = e;
            s_box = x;
        }
        __syncthreads();
        const bool log = !s_err;
        for (int b = wave; b < nb; b += kPassThreads / 64) {  // uniform per wave
            const int k = (b0 + b) * kRowBlock + lane - t0;
            const int col = k >= from && k < m ? tr.col[base + k] : -1;
            const bool in = col >= 0;
            float x = 0.0f, y = 0.0f;
            if (in) {
                const size_t idx = (size_t)(t0 + k) * tb.cap + col;
                tb.dead[idx] = epoch;
                tb.vis[idx] = kAlive;
                x = tb.X[idx];
                y = tb.Y[idx];
                if (log) {
                    const int i = s_base + k - from;
                    cur.x[i] = x;
                    cur.y[i] = y;
                    cur.z[i] = tb.Z[idx];
                    cur.col[i] = col;
                }
                tr.col[base + k] = -1;
            } else if (k >= from && k < m && log) {
                cur.col[s_base + k - from] = 0x7fffffff;     // (no entry: nobody has seen it)
            }
            const float4 q = wave_box(in, x, y);
            if (lane == 0 && log) cur.box[s_box + b] = q;
        }
    }
    if (tid == 0) {
        S.resume_at = affected ? first : -1;
        S.killed = cnt > 0;
        if (cnt > 0 && s_err) S.err = 1;
        if (affected) {
            S.n_points = first;         // keep points 0..first-1; re-score from the last kept point
            S.status = kRunning;
            S.valid = 0;
            S.resumes += 1;
        }
    }
    __syncthreads();
    static_assert(sizeof(Slot) % sizeof(int) == 0 && sizeof(Slot) / sizeof(int) <= kPassThreads, "one word per thread");
    if (tid < (int)(sizeof(Slot) / sizeof(int)))
        reinterpret_cast<int *>(pb.mirror + slot)[tid] = reinterpret_cast<const int *>(&S)[tid];
}

__global__ void fcfs_begin_kernel(DevTable tb, PassBufs pb, DeathLog a, DeathLog b) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < tb.rows) pb.rowN_pre[i] = tb.rowN[i];
    if (i < 3) a.n[i] = b.n[i] = 0;
    if (i == 3) *pb.ins_n = 0;
    if (i == 4) *pb.stop = 0;
}

// An interrupted call: every table entry of the listed slots (requests that
// were admitted but not accepted) is withdrawn, whatever their state, so
// that only accepted plans stay visible.  Only entries owned by sequence
// numbers from min_own on (the unaccepted requests) are touched.
__global__ __launch_bounds__(kPassThreads) void fcfs_abort_kernel(DevTable tb, Slot *slots, const int *list, Traj tr,
                                                                  int min_own, int epoch) {
    const int slot = list[blockIdx.x];
    const Slot &S = slots[slot];
    const int n = min(S.n_points, tr.stride), t0 = S.t0;
    const size_t base = (size_t)slot * tr.stride;
    for (int k = threadIdx.x; k < n; k += kPassThreads) {
        const int col = tr.col[base + k];
        const int row = t0 + k;
        if (col < 0 || col >= tb.cap || row >= tb.rows) continue;
        if (tb.own[(size_t)row * tb.cap + col] < min_own) continue;
        tb.dead[(size_t)row * tb.cap + col] = epoch;
        tb.vis[(size_t)row * tb.cap + col] = kAlive;
        tr.col[base + k] = -1;
    }
}

// Pack the trajectories of the listed slots into one pinned host buffer: slot
// list[i]'s n_points points go to point offset off[i]; xyz (3 doubles), then action, then value per point, in three
// contiguous sections of `total` points each.
// Consecutive threads write consecutive words (dst may lie across the bus).
__global__ void gather_traj_kernel(const Slot *slots, const int *list, const long long *off, long long total, Traj tr,
                                   double *xyz, int *act, double *val) {
    const int slot = list[blockIdx.x];
    const int n = slots[slot].n_points;
    const long long o = off[blockIdx.x];
    const size_t base = (size_t)slot * tr.stride;
    for (int i = threadIdx.x; i < 3 * n; i += blockDim.x) xyz[o * 3 + i] = tr.xyz[base * 3 + i];
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        act[o + k] = tr.act[base + k];
        val[o + k] = tr.val[base + k];
    }
}

}  // namespace

hipError_t launch_gather_traj(const Slot *slots, const int *list, int n_list, const long long *off, long long total,
                              const Traj &tr, void *dst, hipStream_t st) {
    if (n_list <= 0) return hipSuccess;
    double *xyz = static_cast<double *>(dst);
    double *val = xyz + 3 * total;
    int *act = reinterpret_cast<int *>(val + total);
    hipLaunchKernelGGL(gather_traj_kernel, dim3(n_list), dim3(256), 0, st, slots, list, off, total, tr, xyz, act, val);
    return hipGetLastError();
}

hipError_t launch_fcfs_abort(const DevTable &t, Slot *slots, const int *list, int n_list, const Traj &tr, int min_own,
                             int epoch, hipStream_t st) {
    if (n_list <= 0) return hipSuccess;
    hipLaunchKernelGGL(fcfs_abort_kernel, dim3(n_list), dim3(kPassThreads), 0, st, t, slots, list, tr, min_own, epoch);
    return hipGetLastError();
}

hipError_t launch_fill_int(int *p, int value, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_int_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, value, n);
    return hipGetLastError();
}

hipError_t launch_quantise_table(const DevTable &t, hipStream_t st) {
    hipLaunchKernelGGL(quantise_table_kernel, dim3(t.rows), dim3(256), 0, st, t);
    return hipGetLastError();
}

hipError_t launch_build_grid(const DevTable &t, int limit, hipStream_t st) {
    hipLaunchKernelGGL(build_grid_kernel, dim3(t.rows), dim3(kGridThreads), 0, st, t, limit);
    return hipGetLastError();
}

hipError_t launch_append_plans(const DevTable &t, const int *t0, const int *len, int n, const float *xyz,
                               hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(append_plans_kernel, dim3(1), dim3(1024), 0, st, t, t0, len, n, xyz);
    return hipGetLastError();
}

hipError_t launch_scatter_points(const DevTable &t, const float *pts, const int *rows, const int *cols, int n,
                                 int own, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_points_kernel, dim3((n + 255) / 256), dim3(256), 0, st, t, pts, rows, cols, n, own);
    return hipGetLastError();
}

hipError_t launch_commit(const DevCfg &c, const DevTable &t, const double *pts, int t0, int n, int seq, int *flags,
                         int *result, hipStream_t st) {
    if (n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(commit_check_kernel, dim3(n), dim3(256), 0, st, c, t, pts, t0, n, seq, flags);
    hipLaunchKernelGGL(commit_append_kernel, dim3((n + 255) / 256), dim3(256), 0, st, t, pts, t0, n, seq, flags,
                       result);
    return hipGetLastError();
}

hipError_t launch_fcfs_begin(const DevTable &t, const PassBufs &pb, const DeathLog &a, const DeathLog &b,
                             hipStream_t st) {
    hipLaunchKernelGGL(fcfs_begin_kernel, dim3((std::max(t.rows, 8) + 255) / 256), dim3(256), 0, st, t, pb, a, b);
    return hipGetLastError();
}

hipError_t launch_fcfs_pass(const DevCfg &c, const DevTable &t, Slot *slots, const int *list, int n_list,
                            const Traj &tr, const DeathLog &prev, const DeathLog &cur, const PassBufs &pb, int epoch,
                            hipStream_t st) {
    if (n_list <= 0) return hipSuccess;
    const dim3 blk(kPassThreads), fin(n_list + (t.rows + kPrepRows - 1) / kPrepRows);
    hipLaunchKernelGGL(fcfs_insert_kernel, dim3(n_list), blk, 0, st, t, slots, list, tr, pb);
    if (c.lookahead > 1) {
        if (!tr.seenw) return hipErrorInvalidValue;
        hipLaunchKernelGGL(fcfs_check_dead_window_kernel, dim3(n_list), blk, 0, st, c, t, slots, list, tr, prev, epoch);
        hipLaunchKernelGGL(fcfs_check_add_window_kernel, dim3(n_list, (tr.stride + kCheckPoints - 1) / kCheckPoints),
                           blk, 0, st, c, t, slots, list, tr);
        hipLaunchKernelGGL((fcfs_finish_kernel<true>), fin, blk, 0, st, c, t, slots, list, n_list, tr, prev, cur, pb,
                           epoch);
    } else {
        hipLaunchKernelGGL(fcfs_check_kernel, dim3(n_list), blk, 0, st, c, t, slots, list, tr, pb, prev, epoch);
        hipLaunchKernelGGL((fcfs_finish_kernel<false>), fin, blk, 0, st, c, t, slots, list, n_list, tr, prev, cur, pb,
                           epoch);
    }
    return hipGetLastError();
}

}  // namespace fmdp
